// XCA on the matrix cores: the passes over the rows of a window, shared by the kernels on
// work items (sla_xca.hip, which describes the operation and its layouts) and by those
// with a workgroup per (window, head) (sla_xca_win.hip).
#pragma once
#include "sla_attn_core.h"

namespace sla {

constexpr float kXcaFloor = 1e-12f;   // least column norm

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

// -------------------------------------------------- one window, forward
// The rows [wa, wb) of a window of this wave (whole, or `shared`: its rows are this wave's
// share and the sums are added to the other waves'): sums, A, outputs.  HOLD: bk holds the
// item's first block (`resident`: all of it); otherwise every pass reads its rows.
// (k_xca_fwd_mma has the same steps written out, for the reason given there.)
template <typename T, int D, bool HOLD>
__device__ __forceinline__ void xca_fwd_window(Block<T, D, 3>& bk, const T* const (&mats)[3], T* o, const WaveWork& ww,
                                               int32_t wa, int32_t wb, bool shared, bool resident, float th,
                                               const int32_t* perm, int32_t n, size_t rs, floatx4* s_part,
                                               float* norms, int lane, int wv) {
  constexpr int KS = Geo<D>::KS, NT = Geo<D>::NT;
  constexpr int SL = kXcaSlot<T, D, XcaSums<D, false>::kTiles>;
  using F = Frag<T, KS>;
  using O = XcaOp<T, D>;
  constexpr unsigned kKQ = 5u, kV = 2u;
  const int i = lane & 15, g = lane >> 4, col = ww.h * D;
  floatx4* const slot = s_part + wv * SL;
  float* const stage = reinterpret_cast<float*>(slot);
  auto refetch = [&](int32_t base, unsigned which) {
    BlockRows br;
    block_rows(br, base, ww.rb, perm, lane);
    block_fetch<T, D, 3>(bk, br, base, wb, n, mats, which, rs, col, g, wa);
    block_arrange<T, D, 3>(bk, which);
  };
  XcaSums<D, false> su;
  su.clear();
  for (int32_t base = ww.ra; base < ww.rb; base += kBlockRows) {
    if (!HOLD || base != ww.ra) refetch(base, kKQ);
#pragma unroll
    for (int jj = 0; jj < kBlockJobs; ++jj) {
      const int32_t r0 = base + kSliceRows * jj;
      if (job_overlaps(r0, wa, wb)) xca_sums_seg<T, D, 3>(bk.j[jj], r0, wa, wb, i, g, stage, su);
    }
  }
  if (shared) {
    su.publish(slot, lane);
    lds_barrier();
    su.combine(s_part, SL, lane, wv, ww.pair);
    lds_barrier();  // the slots may be written again
  }
  if (!HOLD) refetch(ww.ra, kV);   // in flight under the softmax
  xca_norms<T, D>(su, norms, lane, i, g);
  xca_softmax<T, D, false>(su.M, norms, th, i, g, nullptr);
  Raw<O, KS> op[NT], opl[NT];
  xca_operand<O, D, kXcaPair<O>>(su.M, 1.f, op, opl);
  for (int32_t base = ww.ra; base < ww.rb; base += kBlockRows) {
    if (!(resident && HOLD) && (base != ww.ra || HOLD)) refetch(base, kV);
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
// the second is the row rescaled by a power of two, with |k / s_c| < 2: exactly in bf16,
// in fp16 down to 2^-14, below which it is a subnormal, off by at most 2^-25.
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

// A row's slots times powers of two; rows against fp32 operands stay as they are.
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

// -------------------------------------------------- one window, backward
// As xca_fwd_window; `window` is the window's number, for its temperature share.
template <typename T, int D, bool HOLD>
__device__ __forceinline__ void xca_bwd_window(Block<T, D, 4>& bk, const T* const (&mats)[4], T* dq, T* dk, T* dv,
                                               float* part, const WaveWork& ww, int32_t window, int32_t wa,
                                               int32_t wb, bool shared, bool resident, float th, const int32_t* perm,
                                               int32_t n, int32_t H, floatx4* s_part, float* norms, int lane, int wv) {
  constexpr int KS = Geo<D>::KS, NT = Geo<D>::NT;
  constexpr int SL = kXcaSlot<T, D, XcaSums<D, true>::kTiles>;
  constexpr bool NW = Ty<T>::kNarrow;
  using F = Frag<T, KS>;
  using O = XcaOp<T, D>;
  constexpr bool NO = Ty<O>::kNarrow;
  constexpr unsigned kKQ = 5u, kKQD = 13u, kAll = 15u;
  const int i = lane & 15, g = lane >> 4, col = ww.h * D;
  const size_t rs = (size_t)H * D;
  floatx4* const slot = s_part + wv * SL;
  float* const stage = reinterpret_cast<float*>(slot);
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
      if (!HOLD || base != ww.ra) refetch(base, kAll);
#pragma unroll
      for (int jj = 0; jj < kBlockJobs; ++jj) {
        const int32_t r0 = base + kSliceRows * jj;
        if (job_overlaps(r0, wa, wb)) xca_sums_seg<T, D, 4>(bk.j[jj], r0, wa, wb, i, g, stage, su);
      }
    }
    if (shared) {
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
    if (lane == 0 && ww.rb > ww.ra && (!shared || (ww.pair ? (wv & 1) : wv) == 0))
      part[(size_t)window * H + ww.h] = pt;
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
  if (shared) {
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

// A workgroup per (window, head) (sla_xca_win.hip); long_windows: with the passes above for
// windows of more than 64 rows.
template <typename T, int D>
hipError_t launch_xca_win_fwd(const void* plan, int32_t n, int32_t W, int32_t H, bool long_windows, const float* tau,
                              const T* q, const T* k, const T* v, T* o, hipStream_t stream);
template <typename T, int D>
hipError_t launch_xca_win_bwd(const void* plan, int32_t n, int32_t W, int32_t H, bool long_windows, const float* tau,
                              const T* q, const T* k, const T* v, const T* dout, T* dq, T* dk, T* dv, float* part,
                              hipStream_t stream);
// Workgroups of the kernels with the long passes that the device holds at once.
template <typename T, int D>
int xca_win_resident(bool bwd);

}  // namespace sla
