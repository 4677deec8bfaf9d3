// Cross-covariance attention inside every window: the XCA design of the
// linear-attention ablation (Sec. 4.5, Tab. 7), which cites XCiT, run on the
// same window-sorted plan as SLA.  For window w and head h, with the window's q
// and k columns L2-normalised over the window's rows (norms floored at 1e-12):
//     A[e][c] = softmax over c of  tau_h qhat[:, e] . khat[:, c]     (d x d),
//     o_i[e]  = sum_c A[e][c] v_i[c]                                 for i in w.
// Like Eq. (3) it needs one d x d reduction over the window's rows per head,
// here q^T k together with the column norms, and then one d x d product per row,
// so it runs on the attention kernels' work items, row blocks and register
// layouts (sla_attn_core.h): one wave per (chunk, head) or per share of a long
// window, rows held in registers, no barrier but the exchange of a long window's
// partial sums.
//
// The d x d matrices are held as result tiles of their transposes, M[ct][et]: lane
// (i, g) component j is the entry (c, e) = (16 ct + 4 g + j, 16 et + i).  A row e
// of A then lies in one lane per lane group: its softmax is a reduction over a
// lane's own entries and two lane swaps; the tiles are already the operand of the
// products over c (o = v A^T, dqhat = k B_q^T), and one LDS transpose gives the
// operand of those over e.
//
// What bounds it: the chain of dependent steps of a window, at 2 to 4 waves per
// SIMD, as in k_sla_fwd / k_sla_bwd.  The kernels before held one 256-thread workgroup
// per (window, head), whose 5 to 9 barriers and serial column sums set the time.
// Kernel trace, one Waymo-like frame (60k rows, fp16, H = 4, d = 32): forward 24.0
// us against 26.9, backward 56.5 against 85.9 on inputs used before; with ten sets in
// turn, all from HBM, 29.1 against 28.4 and 67.6 against 87.6.  Forward + backward by
// events 79.9 against 105 us, 151 against 328 on 100k rows in log-normal windows
// (bf16).
#include "sla.h"
#include "sla_attn_core.h"

#include <mutex>

namespace sla {

hipError_t launch_xca_vec_fwd(const void* plan, int32_t n, int32_t W, int32_t H, int32_t d, const float* tau,
                              const float* q, const float* k, const float* v, float* o, hipStream_t stream);
hipError_t launch_xca_vec_bwd(const void* plan, int32_t n, int32_t W, int32_t H, int32_t d, const float* tau,
                              const float* q, const float* k, const float* v, const float* dout, float* dq,
                              float* dk, float* dv, float* part, hipStream_t stream);

// The dtau partials of the backward without a workspace (sla_backward_xca_noalloc):
// one fp32 per (window, head), held in static device memory on every GPU the
// library runs on.  In host code `scratch` only names the symbol; its address on
// a device comes from hipGetSymbolAddress, looked up once per device.
constexpr size_t kXcaScratchFloats = 262144;   // SLA_XCA_SCRATCH_FLOATS
static_assert(kXcaScratchFloats == SLA_XCA_SCRATCH_FLOATS, "the header states the scratch size");
static __device__ __align__(256) float scratch[kXcaScratchFloats];

namespace {

constexpr float kXcaFloor = 1e-12f;   // least column norm
// A window's chain is longer than the attention's and worth more parts (up to 8, four
// times the grid): fp16 forward + backward, 1,521 windows, 20k rows 74 us against 84
// with parts that fill the grid once, 3k rows 51 against 54.
constexpr int kXcaPartFill = 400;

// Operands of the d x d matrices (A, B_q, B_k) in the products with rows: 16-bit
// storage at d = 32 rounds them to the storage type, A in bf16 with its rounding residual
// as a second operand, B_q and B_k always; at d = 16, as in fp32 storage, they stay fp32
// and the rows are widened for 16x16x4 products.  60k rows, H = 8, fp16, inputs
// from HBM: forward 30.7 us (29.6 with A in fp16), backward 59.3 (57.5); with a workgroup
// per (window, head) on the vector units, also in fp32, 49.9 and 110.
template <typename T, int D>
using XcaOp = std::conditional_t<Ty<T>::kNarrow && D == 32, T, float>;
template <typename O>
constexpr bool kXcaPair = std::is_same<O, bf16_t>::value;

template <typename T, typename O, int KS>
__device__ __forceinline__ Raw<O, KS> xca_row(Raw<T, KS> x) {
  if constexpr (std::is_same<T, O>::value) {
    return x;
  } else {
    float f[KS];
    Frag<T, KS>::to_f32(x, f);
    return Frag<O, KS>::from_f32(f);
  }
}

// A product with a row, over the head dim.  fp32 operands: 16x16x4 products in pairs, added
// as a tree, so that a sum of 32 terms goes through 10 additions one after the other
// instead of 32 (fp32 o and dv of a 45k-row frame, d = 32: relative
// error 1.03e-7 against 1.30e-7 in one chain and 1.06e-7 on the vector units; same time).
template <typename O, int KS>
__device__ __forceinline__ floatx4 xca_mma(Raw<O, KS> a, Raw<O, KS> b) {
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (Ty<O>::kNarrow) {
    return Frag<O, KS>::mma(a, b, zero);
  } else {
    floatx4 c[KS / 2];
#pragma unroll
    for (int k = 0; k < KS / 2; ++k) {
      c[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2 * k], b[2 * k], zero, 0, 0, 0);
      c[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2 * k + 1], b[2 * k + 1], c[k], 0, 0, 0);
    }
    if constexpr (KS == 8) return (c[0] + c[1]) + (c[2] + c[3]);
    else return c[0] + c[1];
  }
}

// Sums over a window's rows: M[ct][et] = sum k_r[c] q_r[e] (forward and backward),
// P[ct][et] = sum v_r[c] dout_r[e] (backward), and the squared columns of q and k:
// 16-bit storage takes them from the diagonals of the tiles q^T q and k^T k, whose
// operands M needs anyway; fp32 sums them on the vector units, by slots (slot r of
// lane group g: column E(g, r)).
template <int D, bool BWD>
struct XcaSums {
  static constexpr int NT = Geo<D>::NT, KS = Geo<D>::KS;
  static constexpr int kTiles = (BWD ? 2 : 1) * NT * NT + 2 * NT;
  floatx4 M[NT][NT];
  floatx4 P[BWD ? NT : 1][BWD ? NT : 1];
  floatx4 q2[NT], k2[NT];
  __device__ void clear() {
    const floatx4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int a = 0; a < NT; ++a) {
      q2[a] = z;
      k2[a] = z;
#pragma unroll
      for (int b = 0; b < NT; ++b) {
        M[a][b] = z;
        if constexpr (BWD) P[a][b] = z;
      }
    }
  }
  __device__ void publish(floatx4* slot, int lane) const {
    int t = 0;
#pragma unroll
    for (int a = 0; a < NT; ++a) {
#pragma unroll
      for (int b = 0; b < NT; ++b) {
        slot[(t++) * 64 + lane] = M[a][b];
        if constexpr (BWD) slot[(t++) * 64 + lane] = P[a][b];
      }
      slot[(t++) * 64 + lane] = q2[a];
      slot[(t++) * 64 + lane] = k2[a];
    }
  }
  // the sum of the published sums of the waves that share the window, in wave order
  __device__ void combine(const floatx4* slots, int stride, int lane, int wv, bool pair) {
    clear();
    const int w0 = pair ? (wv & ~1) : 0, nw = pair ? 2 : kWaves;
    for (int w = w0; w < w0 + nw; ++w) {
      const floatx4* sl = slots + w * stride;
      int t = 0;
#pragma unroll
      for (int a = 0; a < NT; ++a) {
#pragma unroll
        for (int b = 0; b < NT; ++b) {
          M[a][b] += sl[(t++) * 64 + lane];
          if constexpr (BWD) P[a][b] += sl[(t++) * 64 + lane];
        }
        q2[a] += sl[(t++) * 64 + lane];
        k2[a] += sl[(t++) * 64 + lane];
      }
    }
  }
};

// 16-bit rows of a job in the wave's slot: two matrices of kSliceRows rows, read back by
// columns with the LDS transpose loads.  (A product with a 0/1 selection matrix, as the
// attention kernels transpose, would carry an infinity or NaN of one column into all of
// its row's: 0 x inf.)
template <int D>
constexpr int kXcaStageLd = D + 8;   // 8-byte aligned rows; the writes of 16 rows spread over all banks
template <int D>
constexpr int kXcaMat = kSliceRows * kXcaStageLd<D>;

// A wave's slot, in floatx4: its published sums (KT tiles), and the rows it stages.
template <typename T, int D, int KT>
constexpr int kXcaSlot = Ty<T>::kNarrow ? (KT * 64 > kXcaMat<D> / 4 ? KT * 64 : kXcaMat<D> / 4)
                                        : (KT * 64 > kStageWave<D> / 4 ? KT * 64 : kStageWave<D> / 4);

// M[ct][et] += X^T Y over the rows [a, b) of a job (x, y zero outside); SQ: also
// the diagonal tiles xx += X^T X, yy += Y^T Y (16-bit storage) or the squares by slots.
template <typename T, int D, bool SQ>
__device__ __forceinline__ void rows_product(const Raw<T, Geo<D>::KS> (&x)[2], const Raw<T, Geo<D>::KS> (&y)[2],
                                             int32_t r0, int32_t a, int32_t b, int i, int g, float* stage,
                                             floatx4 (&M)[Geo<D>::NT][Geo<D>::NT],
                                             floatx4 (*xx)[Geo<D>::NT], floatx4 (*yy)[Geo<D>::NT]) {
  constexpr int KS = Geo<D>::KS, NT = Geo<D>::NT;
  if constexpr (!Ty<T>::kNarrow) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      stage_put<D>(stage, s, i, g, x[s]);
      stage_put<D>(stage + kStageMat<D>, s, i, g, y[s]);
      if constexpr (SQ)
#pragma unroll
        for (int r = 0; r < KS; ++r) {
          (*xx)[r >> 2][r & 3] += x[s][r] * x[s][r];
          (*yy)[r >> 2][r & 3] += y[s][r] * y[s][r];
        }
    }
    wave_lds_sync();
    stage_product<D>(stage, stage + kStageMat<D>, r0, a, b, i, g, M);
  } else {
    unsigned short* const sx = reinterpret_cast<unsigned short*>(stage);
    unsigned short* const sy = sx + kXcaMat<D>;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int at = (16 * s + i) * kXcaStageLd<D> + 16 * t + 4 * g;
        *reinterpret_cast<u16x4*>(sx + at) = u16x4{x[s][4 * t], x[s][4 * t + 1], x[s][4 * t + 2], x[s][4 * t + 3]};
        *reinterpret_cast<u16x4*>(sy + at) = u16x4{y[s][4 * t], y[s][4 * t + 1], y[s][4 * t + 2], y[s][4 * t + 3]};
      }
    wave_lds_sync();
    Raw<T, 8> py[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      py[t] = lds_cols<T>(sy, kXcaStageLd<D>, 16 * t, i, g);
      if constexpr (SQ) (*yy)[t] = Frag<T, 8>::mma(py[t], py[t], (*yy)[t]);
    }
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
      const Raw<T, 8> px = lds_cols<T>(sx, kXcaStageLd<D>, 16 * ct, i, g);
      if constexpr (SQ) (*xx)[ct] = Frag<T, 8>::mma(px, px, (*xx)[ct]);
#pragma unroll
      for (int et = 0; et < NT; ++et) M[ct][et] = Frag<T, 8>::mma(px, py[et], M[ct][et]);
    }
  }
  wave_lds_sync();   // the tile may be written again
}

// Rows [a, b) of one job into the sums.  Matrices K, V, Q (and dout).
template <typename T, int D, int NM>
__device__ __forceinline__ void xca_sums_seg(const Slice<T, Geo<D>::KS, NM>& sb, int32_t r0, int32_t a, int32_t b,
                                             int i, int g, float* stage, XcaSums<D, NM == 4>& su) {
  constexpr int KS = Geo<D>::KS;
  using F = Frag<T, KS>;
  Raw<T, KS> x[2], y[2];
  auto rows = [&](int mx, int my) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int32_t row = r0 + 16 * s + i;
      const bool in = sb.ok[s] && row >= a && row < b;
      x[s] = in ? sb.x[mx][s] : F::zero();
      y[s] = in ? sb.x[my][s] : F::zero();
    }
  };
  rows(0, 2);
  rows_product<T, D, true>(x, y, r0, a, b, i, g, stage, su.M, &su.k2, &su.q2);
  if constexpr (NM == 4) {
    rows(1, 3);
    rows_product<T, D, false>(x, y, r0, a, b, i, g, stage, su.P, nullptr, nullptr);
  }
}

// Max over the 4 lane groups.
__device__ __forceinline__ float max_groups(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Column norms of a window and their reciprocals, in the wave's LDS area: [q | k |
// 1 / q | 1 / k], D each, one column a lane.  (The square root is the correctly
// rounded one, so that the norm of a one-row column is its magnitude.)
template <int D>
constexpr int kXcaNorm = 4 * D;

template <typename T, int D, bool BWD>
__device__ __forceinline__ void xca_norms(const XcaSums<D, BWD>& su, float* norms, int lane, int i, int g) {
  constexpr int NT = Geo<D>::NT;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if constexpr (Ty<T>::kNarrow) {
      const int j = i & 3;
      const float x = j < 2 ? (j == 0 ? su.q2[t][0] : su.q2[t][1]) : (j == 2 ? su.q2[t][2] : su.q2[t][3]);
      const float y = j < 2 ? (j == 0 ? su.k2[t][0] : su.k2[t][1]) : (j == 2 ? su.k2[t][2] : su.k2[t][3]);
      if (g == (i >> 2)) {
        norms[16 * t + i] = x;
        norms[D + 16 * t + i] = y;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = sum_rows16(su.q2[t][j]), y = sum_rows16(su.k2[t][j]);
        if (i == 0) {
          norms[16 * t + 4 * g + j] = x;
          norms[D + 16 * t + 4 * g + j] = y;
        }
      }
    }
  }
  wave_lds_sync();
  if (lane < 2 * D) {
    // a norm whose square has overflowed divides to zero: its reciprocal is zero, and the
    // norm itself finite, so that the steps of xca_unit leave that zero
    const float x = fmaxf(sqrtf(norms[lane]), kXcaFloor);
    norms[lane] = fminf(x, 3.0e38f);
    norms[2 * D + lane] = recip<T>(x);
  }
  wave_lds_sync();
}

// Slots c or e = E(g, r) of one of the four parts, read where they are used: held
// in registers through the row passes they cost spills.
template <int D>
__device__ __forceinline__ void xca_slots(const float* s, int g, float (&x)[Geo<D>::KS]) {
#pragma unroll
  for (int t = 0; t < Geo<D>::NT; ++t) {
    const float4 u = *reinterpret_cast<const float4*>(s + 16 * t + 4 * g);
    x[4 * t] = u.x; x[4 * t + 1] = u.y; x[4 * t + 2] = u.z; x[4 * t + 3] = u.w;
  }
}

// exp(x) for x <= 0: 2^(x log2 e) on the hardware's exp2 (1 ulp).  fp32 adds what
// the product's rounding and log2 e's own lost: 2^(t + r) = 2^t (1 + r ln 2) for |r| < 2^-16.
template <typename T>
__device__ __forceinline__ float xca_exp(float x) {
  if constexpr (Ty<T>::kNarrow) {
    return __builtin_amdgcn_exp2f(x * kLog2e);
  } else {
    constexpr float kLo = 1.925963033e-8f;   // log2 e - kLog2e
    x = x < -128.f ? -128.f : x;              // 2^-184 is zero; a NaN stays one
    const float t = x * kLog2e;
    const float r = fmaf(x, kLo, fmaf(x, kLog2e, -t));
    const float e = __builtin_amdgcn_exp2f(t);
    return fmaf(e * 0.69314718f, r, e);
  }
}

// M: raw sums -> A (both transposed); N, when asked for, gets qhat^T khat.  The
// logits lie in [-|tau|, |tau|], so the usual max shift is all the guard needed.
template <typename T, int D, bool KEEP>
__device__ __forceinline__ void xca_softmax(floatx4 (&M)[Geo<D>::NT][Geo<D>::NT], const float* norms, float tau,
                                            int i, int g, floatx4 (*N)[Geo<D>::NT]) {
  constexpr int NT = Geo<D>::NT;
  float rk[Geo<D>::KS];
  xca_slots<D>(norms + 3 * D, g, rk);
#pragma unroll
  for (int et = 0; et < NT; ++et) {
    float mx = -3.0e38f;
    const float rq = norms[2 * D + 16 * et + i];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = M[ct][et][j] * rq * rk[4 * ct + j];
        if constexpr (KEEP) N[ct][et][j] = x;
        M[ct][et][j] = tau * x;
        mx = fmaxf(mx, M[ct][et][j]);
      }
    mx = max_groups(mx);
    float sum = 0.f;
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = M[ct][et][j] - mx;
        M[ct][et][j] = xca_exp<T>(x);
        sum += M[ct][et][j];
      }
    const float inv = recip<T>(sum_groups(sum));
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int j = 0; j < 4; ++j) M[ct][et][j] *= inv;
  }
}

// Operand (type T) of a product over c from transposed tiles: lane (i, g) of tile et holds
// (row e = 16 et + i) the slots c = E(g, r), times mul; `lo` gets the residuals.
template <typename T, int D, bool LO>
__device__ __forceinline__ void xca_operand(const floatx4 (&M)[Geo<D>::NT][Geo<D>::NT], float mul,
                                            Raw<T, Geo<D>::KS> (&hi)[Geo<D>::NT], Raw<T, Geo<D>::KS>* lo) {
  constexpr int KS = Geo<D>::KS, NT = Geo<D>::NT;
  using F = Frag<T, KS>;
#pragma unroll
  for (int et = 0; et < NT; ++et) {
    float x[KS];
#pragma unroll
    for (int r = 0; r < KS; ++r) x[r] = M[r >> 2][et][r & 3] * mul;
    hi[et] = F::from_f32(x);
    if constexpr (LO) {
      float h[KS];
      F::to_f32(hi[et], h);
#pragma unroll
      for (int r = 0; r < KS; ++r) x[r] -= h[r];
      lo[et] = F::from_f32(x);
    }
  }
}

// --------------------------------------------------------------- forward
template <typename T, int D, bool PARTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
void k_xca_fwd_mma(KernelArgs a, const float* __restrict__ tau, const T* __restrict__ q, const T* __restrict__ k,
               const T* __restrict__ v, T* __restrict__ o) {
  constexpr int KS = Geo<D>::KS, NT = Geo<D>::NT;
  constexpr int KT = XcaSums<D, false>::kTiles;
  constexpr int SL = kXcaSlot<T, D, KT>;
  constexpr bool kHold = Ty<T>::kNarrow || D == 16;
  using F = Frag<T, KS>;
  using O = XcaOp<T, D>;
  __shared__ floatx4 s_part[kWaves * SL];
  __shared__ WaveMeta s_meta[kWaves];
  __shared__ __align__(16) float s_norm[kWaves][kXcaNorm<D>];
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const PlanHeader* hdr = a.hdr;
  if (hdr->magic != kPlanMagic || hdr->n != a.n || hdr->num_windows != a.W) return;
  const Items it = work_items<PARTS ? kXcaPartFill : 0, 3>(a, hdr);
  const int32_t* perm = hdr->csr ? nullptr : a.perm;
  const int i = lane & 15, g = lane >> 4;
  const size_t rs = (size_t)a.H * D;
  const int32_t n = a.n, G = gridDim.x;
  floatx4* const slot = s_part + wv * SL;
  float* const stage = reinterpret_cast<float*>(slot);
  float* const norms = s_norm[wv];
  const T* const mats[3] = {k, v, q};
  constexpr unsigned kKQ = 5u, kV = 2u, kAll = 7u;
  WaveMeta& meta = s_meta[wv];
  const bool csr = perm == nullptr;
  int32_t item = blockIdx.x;
  WaveWork wc, wn;
  {
    const Slot s0 = item_slot(it, item, wv), s1 = item_slot(it, item + G, wv);
    wc = decode_work(a, s0, slot_entry(a, s0), wv);
    wn = decode_work(a, s1, slot_entry(a, s1), wv);
  }
  request_perm(wc, perm, meta.perm[0], lane);
  request_perm(wn, perm, meta.perm[1], lane);
  request_offs(wc, a, meta.offs[0], lane);
  request_entry(a, item_slot(it, item + 2 * G, wv), &meta.ent[0], lane);
  int par = 0;   // ring slot of the current item
  while (item < it.total) {
    const WaveWork ww = wc;
    const int col = ww.h * D;
    // a share of more than kBlockRows rows is streamed through the block
    const bool resident = ww.rb - ww.ra <= kBlockRows;
    // fp32 at d = 32 reads v per window, after the sums, and k, q too: three waves per SIMD
    const unsigned first = resident && kHold ? kAll : kKQ;
    // the item's rows and windows, and the entry of the item after next, from LDS;
    // then the requests ahead (see k_sla_fwd)
    wait_vm();
    BlockRows br;
    block_rows_lds(br, ww, meta.perm[par], csr, lane);
    Stream str;
    stream_lds(str, ww, a, it, meta.offs[par], lane);
    const WaveWork wnn = decode_work(a, item_slot(it, item + 2 * G, wv), lds_entry(&meta.ent[par]), wv);
    wait_lgkm();
    request_perm(wnn, perm, meta.perm[par], lane);
    request_offs(wn, a, meta.offs[par ^ 1], lane);
    request_entry(a, item_slot(it, item + 3 * G, wv), &meta.ent[par ^ 1], lane);
    Block<T, D, 3> bk;
    int32_t fa = INT32_MIN, fb = ww.rb;   // the rows of this item's windows
    if constexpr (PARTS) str.rows(fa, fb);
    if (kHold && ww.kind != 0) {
      block_fetch<T, D, 3>(bk, br, ww.ra, fb, n, mats, first, rs, col, g, fa);
      block_arrange<T, D, 3>(bk, first);
    }
    const float th = tau[ww.h];
    WinIter wi;
    for (bool more = wi.first(ww, str); more; more = wi.next(ww, str)) {
      const int32_t wa = wi.wc.ws, wb = wi.wc.we;
      auto refetch = [&](int32_t base, unsigned which) {
        BlockRows br;
        block_rows(br, base, ww.rb, perm, lane);
        block_fetch<T, D, 3>(bk, br, base, wb, n, mats, which, rs, col, g, wa);
        block_arrange<T, D, 3>(bk, which);
      };
      XcaSums<D, false> su;
      su.clear();
      for (int32_t base = ww.ra; base < ww.rb; base += kBlockRows) {
        if (!kHold || base != ww.ra) refetch(base, kKQ);
#pragma unroll
        for (int jj = 0; jj < kBlockJobs; ++jj) {
          const int32_t r0 = base + kSliceRows * jj;
          if (job_overlaps(r0, wa, wb)) xca_sums_seg<T, D, 3>(bk.j[jj], r0, wa, wb, i, g, stage, su);
        }
      }
      if (wi.shared) {
        su.publish(slot, lane);
        lds_barrier();
        su.combine(s_part, SL, lane, wv, ww.pair);
        lds_barrier();  // the slots may be written again
      }
      if (!kHold) refetch(ww.ra, kV);   // in flight under the softmax
      xca_norms<T, D>(su, norms, lane, i, g);
      xca_softmax<T, D, false>(su.M, norms, th, i, g, nullptr);
      Raw<O, KS> op[NT], opl[NT];
      xca_operand<O, D, kXcaPair<O>>(su.M, 1.f, op, opl);
      for (int32_t base = ww.ra; base < ww.rb; base += kBlockRows) {
        if (!(resident && kHold) && (base != ww.ra || kHold)) refetch(base, kV);
#pragma unroll
        for (int jj = 0; jj < kBlockJobs; ++jj)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const int32_t r0 = base + kSliceRows * jj;
            if (!sub_overlaps(r0, s, wa, wb)) continue;
            const int32_t row = r0 + 16 * s + i;
            const Raw<O, KS> vr = xca_row<T, O, KS>(bk.j[jj].x[1][s]);
            float x[KS];
#pragma unroll
            for (int et = 0; et < NT; ++et) {
              floatx4 d4 = xca_mma<O, KS>(op[et], vr);
              if constexpr (kXcaPair<O>) d4 = Frag<O, KS>::mma(opl[et], vr, d4);
#pragma unroll
              for (int j = 0; j < 4; ++j) x[4 * et + j] = d4[j];
            }
            RowIO<T, D>::put(o, row_off(bk.j[jj].o[s], rs, col), g, F::from_f32(x),
                             bk.j[jj].ok[s] && row >= wa && row < wb);
          }
      }
    }
    item += G;
    wc = wn;
    wn = wnn;
    par ^= 1;
  }
}

// -------------------------------------------------------------- backward
// Chain rule of the forward, with N = qhat^T khat, A = softmax_c(tau N):
//   dv_i = A^T do_i,  dA = sum_i do_i v_i^T,  dG = A * (dA - rowsum(A * dA)),
//   dtau partial = sum dG * N,
//   dqh[:, e] = sum_c B_q[e][c] k[:, c] with B_q[e][c] = tau dG[e][c] / nk_c,
//   s_e = sum_r qhat_re dqh_re  (the projection of dqh onto qhat, summed over the
//        window's rows; zero where the norm took the floor),
//   dq[:, e] = (dqh[:, e] - qhat[:, e] s_e) / nq_e,
// and likewise dk with B_k[e][c] = tau dG[e][c] / nq_e and t_c = sum_r khat_rc
// dkh_rc.  s_e comes from the rows themselves, as qhat and dqh round, so that
// the difference keeps the cancellation exact where it is exact in real
// arithmetic: in a one-row window qhat = q / |q| is +-1 exactly (the square
// root of a rounded square is the magnitude again in binary floating point), so
// qhat s_e = dqh and dq = 0, as the chain rule gives.
//
// Three passes over the window's rows: G, the norms and dA (one exchange for a
// long window); dv and the projections (a second exchange); dq and dk, whose dqh
// and dkh are formed again from registers rather than held (matrix products are
// cheap here, registers are not).
//
// 16-bit storage at d = 32: B_q[e][c] = tau dG[e][c] / nk_c spans the range of 1 / nk, and a
// floored norm (a zero column) makes that 1e12 times wider than the rest.  So the
// column factor is split: B_q[e][c] k[r][c] = (tau dG[e][c] s_c / nk_c)(k[r][c] /
// s_c) with s_c = 2^floor(log2 nk_c).  The first factor, within [1/2, 1] of tau dG,
// takes one power-of-two scale into [1, 2) and is carried as a high/residual pair;
// the second is the row rescaled by a power of two, exactly, with |k / s_c| < 2.
// B_k alike with nq.
//
// x / y for the normalised rows: the hardware reciprocal and one correction step,
// exactly +-1 when x = +-y (a one-row window's only entry).
__device__ __forceinline__ float xca_unit(float x, float y, float ry) {
  const float h = x * ry;
  return fmaf(fmaf(-h, y, x), ry, h);
}

// The same where the quotient may overflow (a gradient through a floored norm): to infinity.
__device__ __forceinline__ float xca_div(float x, float y, float ry) {
  const float h = x * ry;
  return fabsf(h) < 3.4e38f ? fmaf(fmaf(-h, y, x), ry, h) : h;
}

// 2^floor(log2 x) for a normal x > 0 (the norms: at least 1e-12)
__device__ __forceinline__ float xca_pow2_floor(float x) {
  return __uint_as_float(__float_as_uint(x) & 0x7f800000u);
}

// A row's slots times powers of two (exact); rows against fp32 operands stay as they are.
template <typename T, typename O, int KS>
__device__ __forceinline__ Raw<O, KS> xca_rescale(Raw<T, KS> x, const float (&nrm)[KS]) {
  if constexpr (!Ty<O>::kNarrow) return xca_row<T, O, KS>(x);
  Raw<O, KS> r;
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    // 1 / 2^e from the exponent bits: norms are normal numbers below 2^126
    const float inv = __uint_as_float(0x7f000000u - (__float_as_uint(nrm[j]) & 0x7f800000u));
    r[j] = f32_to_u16<T>(u16_to_f32<T>(x[j]) * inv);
  }
  return r;
}

template <typename T, int D>
struct XcaBwdOp {
  using O = XcaOp<T, D>;
  static constexpr int NT = Geo<D>::NT, KS = Geo<D>::KS;
  static constexpr int NL = Ty<O>::kNarrow ? NT : 1;
  Raw<O, KS> bq[NT], bql[NL];   // scaled B_q: row e = 16 t + i, slots c (and residual)
  Raw<O, KS> bk[NT], bkl[NL];   // scaled B_k^T: row c = 16 t + i, slots e
  float iq, ik;                 // the scales' inverses
  // dqh and dkh of a row by slots
  __device__ __forceinline__ void grads(const Raw<T, KS>& qr, const Raw<T, KS>& kr, const float (&nq)[KS],
                                        const float (&nk)[KS], float (&gq)[KS], float (&gk)[KS]) const {
    using F = Frag<O, KS>;
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    const Raw<O, KS> kb = xca_rescale<T, O, KS>(kr, nk), qb = xca_rescale<T, O, KS>(qr, nq);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      floatx4 x = F::mma(bq[t], kb, zero), y = F::mma(bk[t], qb, zero);
      if constexpr (Ty<O>::kNarrow) {
        x = F::mma(bql[t], kb, x);
        y = F::mma(bkl[t], qb, y);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        gq[4 * t + j] = x[j] * iq;
        gk[4 * t + j] = y[j] * ik;
      }
    }
  }
};

template <typename T, int D, bool PARTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_xca_bwd_mma(KernelArgs a, const float* __restrict__ tau, const T* __restrict__ q, const T* __restrict__ k,
               const T* __restrict__ v, const T* __restrict__ dout, T* __restrict__ dq, T* __restrict__ dk,
               T* __restrict__ dv, float* __restrict__ part) {
  constexpr int KS = Geo<D>::KS, NT = Geo<D>::NT;
  constexpr int KT = XcaSums<D, true>::kTiles;
  constexpr int SL = kXcaSlot<T, D, KT>;
  constexpr bool NW = Ty<T>::kNarrow;
  // fp32 at d = 32: rows held through a window's three passes leave one wave per
  // SIMD (or 230 spilled registers); read again for each pass, two
  constexpr bool kHold = NW || D == 16;
  using F = Frag<T, KS>;
  using O = XcaOp<T, D>;
  constexpr bool NO = Ty<O>::kNarrow;
  __shared__ floatx4 s_part[kWaves * SL];
  __shared__ WaveMeta s_meta[kWaves];
  __shared__ __align__(16) float s_norm[kWaves][kXcaNorm<D>];
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const PlanHeader* hdr = a.hdr;
  if (hdr->magic != kPlanMagic || hdr->n != a.n || hdr->num_windows != a.W) return;
  const Items it = work_items<PARTS ? kXcaPartFill : 0, 3>(a, hdr);
  const int32_t* perm = hdr->csr ? nullptr : a.perm;
  const int i = lane & 15, g = lane >> 4;
  const size_t rs = (size_t)a.H * D;
  const int32_t n = a.n, G = gridDim.x;
  floatx4* const slot = s_part + wv * SL;
  float* const stage = reinterpret_cast<float*>(slot);
  float* const norms = s_norm[wv];
  const T* const mats[4] = {k, v, q, dout};
  constexpr unsigned kKQ = 5u, kKQD = 13u, kAll = 15u;
  WaveMeta& meta = s_meta[wv];
  const bool csr = perm == nullptr;
  int32_t item = blockIdx.x;
  WaveWork wc, wn;
  {
    const Slot s0 = item_slot(it, item, wv), s1 = item_slot(it, item + G, wv);
    wc = decode_work(a, s0, slot_entry(a, s0), wv);
    wn = decode_work(a, s1, slot_entry(a, s1), wv);
  }
  request_perm(wc, perm, meta.perm[0], lane);
  request_perm(wn, perm, meta.perm[1], lane);
  request_offs(wc, a, meta.offs[0], lane);
  request_entry(a, item_slot(it, item + 2 * G, wv), &meta.ent[0], lane);
  int par = 0;   // ring slot of the current item
  while (item < it.total) {
    const WaveWork ww = wc;
    const int col = ww.h * D;
    // a share of more than kBlockRows rows is streamed through the block; so is every
    // window in fp32 at d = 32
    const bool resident = kHold && ww.rb - ww.ra <= kBlockRows;
    // the item's rows and windows, and the entry of the item after next, from LDS;
    // then the requests ahead (see k_sla_fwd)
    wait_vm();
    BlockRows br;
    block_rows_lds(br, ww, meta.perm[par], csr, lane);
    Stream str;
    stream_lds(str, ww, a, it, meta.offs[par], lane);
    const WaveWork wnn = decode_work(a, item_slot(it, item + 2 * G, wv), lds_entry(&meta.ent[par]), wv);
    wait_lgkm();
    request_perm(wnn, perm, meta.perm[par], lane);
    request_offs(wn, a, meta.offs[par ^ 1], lane);
    request_entry(a, item_slot(it, item + 3 * G, wv), &meta.ent[par ^ 1], lane);
    Block<T, D, 4> bk;
    int32_t fa = INT32_MIN, fb = ww.rb;   // the rows of this item's windows
    if constexpr (PARTS) str.rows(fa, fb);
    if (kHold && ww.kind != 0) {
      block_fetch<T, D, 4>(bk, br, ww.ra, fb, n, mats, kAll, rs, col, g, fa);
      block_arrange<T, D, 4>(bk, kAll);
    }
    const float th = tau[ww.h];
    WinIter wi;
    for (bool more = wi.first(ww, str); more; more = wi.next(ww, str)) {
      const int32_t wa = wi.wc.ws, wb = wi.wc.we;
      auto refetch = [&](int32_t base, unsigned which) {
        BlockRows br;
        block_rows(br, base, ww.rb, perm, lane);
        block_fetch<T, D, 4>(bk, br, base, wb, n, mats, which, rs, col, g, wa);
        block_arrange<T, D, 4>(bk, which);
      };
      auto load_norms = [&](float(&nq)[KS], float(&nk)[KS], float(&rq)[KS], float(&rk)[KS]) {
        asm volatile("" ::: "memory");   // not hoisted out of the loops over rows
        xca_slots<D>(norms, g, nq);
        xca_slots<D>(norms + D, g, nk);
        xca_slots<D>(norms + 2 * D, g, rq);
        xca_slots<D>(norms + 3 * D, g, rk);
      };
      XcaBwdOp<T, D> op;
      Raw<O, KS> at[NT], atl[NT];   // A^T: row c = 16 t + i, slots e
      {
        // pass 1: G, the norms, dA
        XcaSums<D, true> su;
        su.clear();
        for (int32_t base = ww.ra; base < ww.rb; base += kBlockRows) {
          if (!kHold || base != ww.ra) refetch(base, kAll);
#pragma unroll
          for (int jj = 0; jj < kBlockJobs; ++jj) {
            const int32_t r0 = base + kSliceRows * jj;
            if (job_overlaps(r0, wa, wb)) xca_sums_seg<T, D, 4>(bk.j[jj], r0, wa, wb, i, g, stage, su);
          }
        }
        if (wi.shared) {
          su.publish(slot, lane);
          lds_barrier();
          su.combine(s_part, SL, lane, wv, ww.pair);
          lds_barrier();
        }
        xca_norms<T, D>(su, norms, lane, i, g);
        floatx4 N[NT][NT];
        xca_softmax<T, D, true>(su.M, norms, th, i, g, N);
        State<D> tr;   // transposed through LDS
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
          for (int et = 0; et < NT; ++et) tr.M[ct][et] = su.M[ct][et];
        transposed_operand<O, D, kXcaPair<O>>(tr, 1.f, stage, i, g, at, atl);
        // dG (in P), the temperature share, B_q (in M) and B_k (in P)
        float pt = 0.f, mq = 0.f, mk = 0.f;
        float fk[KS];
        {
          float nk[KS];
          xca_slots<D>(norms + D, g, nk);
          xca_slots<D>(norms + 3 * D, g, fk);
#pragma unroll
          for (int r = 0; r < KS; ++r) fk[r] *= th * (NO ? xca_pow2_floor(nk[r]) : 1.f);
        }
#pragma unroll
        for (int et = 0; et < NT; ++et) {
          float rsum = 0.f;
#pragma unroll
          for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int j = 0; j < 4; ++j) rsum += su.M[ct][et][j] * su.P[ct][et][j];
          rsum = sum_groups(rsum);
          const float fq = th * norms[2 * D + 16 * et + i] * (NO ? xca_pow2_floor(norms[16 * et + i]) : 1.f);
#pragma unroll
          for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float dg = su.M[ct][et][j] * (su.P[ct][et][j] - rsum);
              pt += dg * N[ct][et][j];
              su.M[ct][et][j] = dg * fk[4 * ct + j];
              tr.M[ct][et][j] = dg * fq;
              mq = fmaxf(mq, fabsf(su.M[ct][et][j]));
              mk = fmaxf(mk, fabsf(tr.M[ct][et][j]));
            }
        }
        pt = sum_groups(sum_rows16(pt));
        // waves that share a window hold the same sum; the first of them writes it
        if (lane == 0 && ww.rb > ww.ra && (!wi.shared || (ww.pair ? (wv & 1) : wv) == 0))
          part[(size_t)wi.window(ww) * a.H + ww.h] = pt;
        const float sq = NO ? pow2_scale_to_one(wave_reduce<true>(mq)) : 1.f;
        const float sk = NO ? pow2_scale_to_one(wave_reduce<true>(mk)) : 1.f;
        op.iq = 1.f / sq;
        op.ik = 1.f / sk;
        xca_operand<O, D, NO>(su.M, sq, op.bq, op.bql);
        transposed_operand<O, D, NO>(tr, sk, stage, i, g, op.bk, op.bkl);
      }
      // pass 2: dv, and the projections s_e, t_c by slots
      float ps[KS], pk[KS];
#pragma unroll
      for (int r = 0; r < KS; ++r) ps[r] = pk[r] = 0.f;
      for (int32_t base = ww.ra; base < ww.rb; base += kBlockRows) {
        if (!resident) refetch(base, kKQD);
#pragma unroll
        for (int jj = 0; jj < kBlockJobs; ++jj)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const int32_t r0 = base + kSliceRows * jj;
            if (!sub_overlaps(r0, s, wa, wb)) continue;
            const int32_t row = r0 + 16 * s + i;
            const auto& sb = bk.j[jj];
            const bool in = sb.ok[s] && row >= wa && row < wb;
            __builtin_amdgcn_sched_barrier(0);   // one sub-tile's operands live at a time
            const Raw<O, KS> dr = xca_row<T, O, KS>(sb.x[3][s]);
            float x[KS];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              floatx4 d4 = xca_mma<O, KS>(at[t], dr);
              if constexpr (kXcaPair<O>) d4 = Frag<O, KS>::mma(atl[t], dr, d4);
#pragma unroll
              for (int j = 0; j < 4; ++j) x[4 * t + j] = d4[j];
            }
            RowIO<T, D>::put(dv, row_off(sb.o[s], rs, col), g, F::from_f32(x), in);
            float gq[KS], gk[KS], qf[KS], kf[KS], nq[KS], nk[KS], rq[KS], rk[KS];
            load_norms(nq, nk, rq, rk);
            op.grads(sb.x[2][s], sb.x[0][s], nq, nk, gq, gk);
            F::to_f32(sb.x[2][s], qf);
            F::to_f32(sb.x[0][s], kf);
#pragma unroll
            for (int r = 0; r < KS; ++r) {
              ps[r] += in ? xca_unit(qf[r], nq[r], rq[r]) * gq[r] : 0.f;
              pk[r] += in ? xca_unit(kf[r], nk[r], rk[r]) * gk[r] : 0.f;
            }
          }
      }
#pragma unroll
      for (int r = 0; r < KS; ++r) {
        ps[r] = sum_rows16(ps[r]);
        pk[r] = sum_rows16(pk[r]);
      }
      if (wi.shared) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          slot[(2 * t) * 64 + lane] = floatx4{ps[4 * t], ps[4 * t + 1], ps[4 * t + 2], ps[4 * t + 3]};
          slot[(2 * t + 1) * 64 + lane] = floatx4{pk[4 * t], pk[4 * t + 1], pk[4 * t + 2], pk[4 * t + 3]};
        }
        lds_barrier();
#pragma unroll
        for (int r = 0; r < KS; ++r) ps[r] = pk[r] = 0.f;
        const int w0 = ww.pair ? (wv & ~1) : 0, nw = ww.pair ? 2 : kWaves;
        for (int w = w0; w < w0 + nw; ++w)
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const floatx4 x = s_part[w * SL + (2 * t) * 64 + lane], y = s_part[w * SL + (2 * t + 1) * 64 + lane];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              ps[4 * t + j] += x[j];
              pk[4 * t + j] += y[j];
            }
          }
        lds_barrier();   // the slots may be written again
      }
      // a floored norm is a constant: no projection
      {
        float nq[KS], nk[KS];
        xca_slots<D>(norms, g, nq);
        xca_slots<D>(norms + D, g, nk);
#pragma unroll
        for (int r = 0; r < KS; ++r) {
          ps[r] = nq[r] > kXcaFloor ? ps[r] : 0.f;
          pk[r] = nk[r] > kXcaFloor ? pk[r] : 0.f;
        }
      }
      // pass 3: dq, dk
      for (int32_t base = ww.ra; base < ww.rb; base += kBlockRows) {
        if (!resident) refetch(base, kKQ);
#pragma unroll
        for (int jj = 0; jj < kBlockJobs; ++jj)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const int32_t r0 = base + kSliceRows * jj;
            if (!sub_overlaps(r0, s, wa, wb)) continue;
            const int32_t row = r0 + 16 * s + i;
            const auto& sb = bk.j[jj];
            const bool in = sb.ok[s] && row >= wa && row < wb;
            __builtin_amdgcn_sched_barrier(0);
            float gq[KS], gk[KS], qf[KS], kf[KS], nq[KS], nk[KS], rq[KS], rk[KS];
            load_norms(nq, nk, rq, rk);
            op.grads(sb.x[2][s], sb.x[0][s], nq, nk, gq, gk);
            F::to_f32(sb.x[2][s], qf);
            F::to_f32(sb.x[0][s], kf);
#pragma unroll
            for (int r = 0; r < KS; ++r) {
              const float xq = gq[r] - xca_unit(qf[r], nq[r], rq[r]) * ps[r];
              const float xk = gk[r] - xca_unit(kf[r], nk[r], rk[r]) * pk[r];
              gq[r] = NW ? xq * rq[r] : xca_div(xq, nq[r], rq[r]);
              gk[r] = NW ? xk * rk[r] : xca_div(xk, nk[r], rk[r]);
            }
            RowIO<T, D>::put(dq, row_off(sb.o[s], rs, col), g, F::from_f32(gq), in);
            RowIO<T, D>::put(dk, row_off(sb.o[s], rs, col), g, F::from_f32(gk), in);
          }
      }
    }
    item += G;
    wc = wn;
    wn = wnn;
    par ^= 1;
  }
}

// dtau[h] = sum over the windows that hold rows, in window order, of the (window,
// head) partials: 256 strided sums, then a fixed tree.
__global__ __launch_bounds__(256) void k_xca_dtau(KernelArgs a, const float* __restrict__ part,
                                                  float* __restrict__ dtau) {
  __shared__ float s[256];
  const int h = (int)blockIdx.x, tid = (int)threadIdx.x;
  float x = 0.f;
  if (a.hdr->magic == kPlanMagic && a.hdr->n == a.n && a.hdr->num_windows == a.W)
#pragma unroll 4
    for (int32_t w = tid; w < a.W; w += 256) {
      const bool live = max(0, min(a.offs[w], a.n)) < min(a.offs[w + 1], a.n);
      const float y = part[(size_t)w * a.H + h];
      x += live ? y : 0.f;
    }
  s[tid] = x;
  __syncthreads();
  for (int m = 128; m > 0; m >>= 1) {
    if (tid < m) s[tid] += s[tid + m];
    __syncthreads();
  }
  if (tid == 0) dtau[h] = s[0];
}

// fp32 scenes of fewer rows per window slot than this take the vector-unit kernels
// (sla_xca_vec.hip): a thin window costs a wave of the matrix-core kernels its whole
// chain of fp32 products.  Forward + backward, H = 4, d = 32, 1,521 windows (us, vector
// units against matrix cores): 10k rows 78 / 113, 25k 108 / 135, 60k 193 / 158; 612
// log-normal windows, 30k rows: 524 / 172.
constexpr int64_t kXcaVecRows = 28;

template <typename T>
bool xca_vec(int32_t n, int32_t W) {
  return !Ty<T>::kNarrow && (int64_t)n < kXcaVecRows * W;
}

template <typename T, int D>
hipError_t xca_impl(const void* plan, int32_t n, int32_t W, int32_t H, const float* tau,
                    const void* q, const void* k, const void* v, void* o, hipStream_t stream) {
  if constexpr (!Ty<T>::kNarrow)
    if (xca_vec<T>(n, W))
      return launch_xca_vec_fwd(plan, n, W, H, D, tau, static_cast<const T*>(q), static_cast<const T*>(k),
                                static_cast<const T*>(v), static_cast<T*>(o), stream);
  const PlanLayout lay = plan_layout(n, W);
  const KernelArgs a = kernel_args(plan, lay, n, W, H, 0.f);
  const int grid = grid_size(reinterpret_cast<const void*>(&k_xca_fwd_mma<T, D, false>), lay, n, H);
  const auto kern = parts_fit(grid, n, W, H, kXcaPartFill) ? &k_xca_fwd_mma<T, D, true> : &k_xca_fwd_mma<T, D, false>;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), 0, stream, a, tau,
                     static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(v),
                     static_cast<T*>(o));
  return hipGetLastError();
}

template <typename T, int D>
hipError_t xca_bwd_impl(const void* plan, int32_t n, int32_t W, int32_t H, const float* tau,
                        const void* q, const void* k, const void* v, const void* dout, void* dq,
                        void* dk, void* dv, float* dtau, float* part, hipStream_t stream) {
  const PlanLayout lay = plan_layout(n, W);
  const KernelArgs a = kernel_args(plan, lay, n, W, H, 0.f);
  if (n > 0) {
    hipError_t e = hipSuccess;
    bool vec = false;
    if constexpr (!Ty<T>::kNarrow) {
      vec = xca_vec<T>(n, W);
      if (vec)
        e = launch_xca_vec_bwd(plan, n, W, H, D, tau, static_cast<const T*>(q), static_cast<const T*>(k),
                               static_cast<const T*>(v), static_cast<const T*>(dout), static_cast<T*>(dq),
                               static_cast<T*>(dk), static_cast<T*>(dv), part, stream);
    }
    if (!vec) {
      const int grid = grid_size(reinterpret_cast<const void*>(&k_xca_bwd_mma<T, D, false>), lay, n, H);
      const auto kern = parts_fit(grid, n, W, H, kXcaPartFill) ? &k_xca_bwd_mma<T, D, true> : &k_xca_bwd_mma<T, D, false>;
      hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), 0, stream, a,
                         tau, static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(v),
                         static_cast<const T*>(dout), static_cast<T*>(dq), static_cast<T*>(dk),
                         static_cast<T*>(dv), part);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_xca_dtau, dim3((unsigned)H), dim3(256), 0, stream, a, part, dtau);
  return hipGetLastError();
}

}  // namespace

// dtype: 0 f32, 1 f16, 2 bf16; d: 16 or 32
hipError_t launch_forward_xca(const void* plan, int32_t n, int32_t W, int dtype, int32_t H, int32_t d,
                              const float* tau, const void* q, const void* k, const void* v, void* o,
                              hipStream_t stream) {
  if (d == 32) {
    if (dtype == 0) return xca_impl<float, 32>(plan, n, W, H, tau, q, k, v, o, stream);
    if (dtype == 1) return xca_impl<_Float16, 32>(plan, n, W, H, tau, q, k, v, o, stream);
    return xca_impl<bf16_t, 32>(plan, n, W, H, tau, q, k, v, o, stream);
  }
  if (dtype == 0) return xca_impl<float, 16>(plan, n, W, H, tau, q, k, v, o, stream);
  if (dtype == 1) return xca_impl<_Float16, 16>(plan, n, W, H, tau, q, k, v, o, stream);
  return xca_impl<bf16_t, 16>(plan, n, W, H, tau, q, k, v, o, stream);
}

hipError_t launch_backward_xca(const void* plan, int32_t n, int32_t W, int dtype, int32_t H, int32_t d,
                               const float* tau, const void* q, const void* k, const void* v,
                               const void* dout, void* dq, void* dk, void* dv, float* dtau, float* part,
                               hipStream_t stream) {
  if (d == 32) {
    if (dtype == 0) return xca_bwd_impl<float, 32>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, dtau, part, stream);
    if (dtype == 1) return xca_bwd_impl<_Float16, 32>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, dtau, part, stream);
    return xca_bwd_impl<bf16_t, 32>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, dtau, part, stream);
  }
  if (dtype == 0) return xca_bwd_impl<float, 16>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, dtau, part, stream);
  if (dtype == 1) return xca_bwd_impl<_Float16, 16>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, dtau, part, stream);
  return xca_bwd_impl<bf16_t, 16>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, dtau, part, stream);
}

// Device address of `scratch` on the current device (nullptr and the HIP error
// if it cannot be looked up).  Looked up once per device, with that device current.
static float* scratch_address(hipError_t& err) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static float* addr[kMaxDevices] = {};
  int dev = 0;
  err = hipGetDevice(&dev);
  if (err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= kMaxDevices) {
    err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    void* p = nullptr;
    err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess) return nullptr;
    addr[dev] = static_cast<float*>(p);
  }
  err = hipSuccess;
  return addr[dev];
}

// sla_backward_xca with the dtau partials in `scratch` (num_windows * heads <=
// kXcaScratchFloats, checked by the caller).  Every partial of a window with rows is
// written by every call and no other one counts, so nothing is cleared.
hipError_t launch_backward_xca_noalloc(const void* plan, int32_t n, int32_t W, int dtype, int32_t H, int32_t d,
                                       const float* tau, const void* q, const void* k, const void* v,
                                       const void* dout, void* dq, void* dk, void* dv, float* dtau,
                                       hipStream_t stream) {
  hipError_t err;
  float* part = scratch_address(err);
  if (part == nullptr) return err;
  return launch_backward_xca(plan, n, W, dtype, H, d, tau, q, k, v, dout, dq, dk, dv, dtau, part, stream);
}

}  // namespace sla
