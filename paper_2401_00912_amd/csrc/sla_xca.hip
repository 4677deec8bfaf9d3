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
// What bounds it: the chain of dependent steps of a window on one wave (some 2.5 us
// forward), at 2 to 4 waves per SIMD.  Against a 256-thread workgroup per (window, head), as
// in sla_xca_win.hip, whose 5 to 9 barriers and serial column sums set the time of large
// scenes: one Waymo-like frame (60k rows, fp16, H = 4, d = 32), inputs from HBM, forward
// 29.1 us against 29.7, backward 67.4 against 91.9; bf16 30.1 against 31.9 and 66.9 against
// 87.2; 60k rows in log-normal windows, fp16, 42.9 against 79.7 and 98.0 against 203;
// H = 8, d = 16, 30.6 against 49.9 and 59.5 against 112.  Scenes of few or of thin windows
// are faster with the workgroups: xca_path below.
#include "sla.h"
#include "sla_xca_core.h"

#include <mutex>

namespace sla {

// The dtau partials of the backward without a workspace (sla_backward_xca_noalloc):
// one fp32 per (window, head), held in static device memory on every GPU the
// library runs on.  In host code `scratch` only names the symbol; its address on
// a device comes from hipGetSymbolAddress, looked up once per device.
constexpr size_t kXcaScratchFloats = 262144;   // SLA_XCA_SCRATCH_FLOATS
static_assert(kXcaScratchFloats == SLA_XCA_SCRATCH_FLOATS, "the header states the scratch size");
static __device__ __align__(256) float scratch[kXcaScratchFloats];

namespace {

// A window's chain is longer than the attention's and worth more parts than fill the grid
// once, up to 8.  In percent of the grid (fp16, H = 8, d = 32, inputs from HBM): forward,
// 3,481 windows of 16k rows, 43.7 us at 400, 51.3 at 200, 49.5 at 100; backward, 1,521
// windows of 8k rows, 79.2, 68.7 and 75.1, 3,481 of 8k 109, 103 and 115.
constexpr int kXcaFwdFill = 400, kXcaBwdFill = 200;

// --------------------------------------------------------------- forward
template <typename T, int D, bool PARTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
void k_xca_fwd_mma(KernelArgs a, const float* __restrict__ tau, const T* __restrict__ q, const T* __restrict__ k,
               const T* __restrict__ v, T* __restrict__ o) {
  constexpr int SL = kXcaSlot<T, D, XcaSums<D, false>::kTiles>;
  constexpr bool kHold = Ty<T>::kNarrow || D == 16;
  __shared__ floatx4 s_part[kWaves * SL];
  __shared__ WaveMeta s_meta[kWaves];
  __shared__ __align__(16) float s_norm[kWaves][kXcaNorm<D>];
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const PlanHeader* hdr = a.hdr;
  if (hdr->magic != kPlanMagic || hdr->n != a.n || hdr->num_windows != a.W) return;
  const Items it = work_items<PARTS ? kXcaFwdFill : 0, 3>(a, hdr);
  const int32_t* perm = hdr->csr ? nullptr : a.perm;
  const int i = lane & 15, g = lane >> 4;
  const size_t rs = (size_t)a.H * D;
  const int32_t n = a.n, G = gridDim.x;
  float* const norms = s_norm[wv];
  const T* const mats[3] = {k, v, q};
  constexpr int KS = Geo<D>::KS, NT = Geo<D>::NT;
  using F = Frag<T, KS>;
  using O = XcaOp<T, D>;
  floatx4* const slot = s_part + wv * SL;
  float* const stage = reinterpret_cast<float*>(slot);
  constexpr unsigned kV = 2u, kKQ = 5u, kAll = 7u;
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
      // xca_fwd_window, written out: as a call its row masks are formed on the scalar unit,
      // the frame above, fp16, 29.8 us against 29.1
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

template <typename T, int D, bool PARTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_xca_bwd_mma(KernelArgs a, const float* __restrict__ tau, const T* __restrict__ q, const T* __restrict__ k,
               const T* __restrict__ v, const T* __restrict__ dout, T* __restrict__ dq, T* __restrict__ dk,
               T* __restrict__ dv, float* __restrict__ part) {
  constexpr int SL = kXcaSlot<T, D, XcaSums<D, true>::kTiles>;
  // fp32 at d = 32: rows held through a window's three passes leave one wave per
  // SIMD (or 230 spilled registers); read again for each pass, two
  constexpr bool kHold = Ty<T>::kNarrow || D == 16;
  __shared__ floatx4 s_part[kWaves * SL];
  __shared__ WaveMeta s_meta[kWaves];
  __shared__ __align__(16) float s_norm[kWaves][kXcaNorm<D>];
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const PlanHeader* hdr = a.hdr;
  if (hdr->magic != kPlanMagic || hdr->n != a.n || hdr->num_windows != a.W) return;
  const Items it = work_items<PARTS ? kXcaBwdFill : 0, 3>(a, hdr);
  const int32_t* perm = hdr->csr ? nullptr : a.perm;
  const int i = lane & 15, g = lane >> 4;
  const size_t rs = (size_t)a.H * D;
  const int32_t n = a.n, G = gridDim.x;
  float* const norms = s_norm[wv];
  const T* const mats[4] = {k, v, q, dout};
  constexpr unsigned kAll = 15u;
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
      xca_bwd_window<T, D, kHold>(bk, mats, dq, dk, dv, part, ww, wi.window(ww), wa, wb, wi.shared, resident, th, perm, n, a.H,
                                  s_part, norms, lane, wv);
    }
    item += G;
    wc = wn;
    wn = wnn;
    par ^= 1;
  }
}

// dtau[h] = sum over the windows that hold rows, in window order, of the (window,
// head) partials: 256 strided sums, then a fixed tree.  ALL: every window's partial is
// written (those without rows as zero), and none is asked for its rows.
template <bool ALL>
__global__ __launch_bounds__(256) void k_xca_dtau(KernelArgs a, const float* __restrict__ part,
                                                  float* __restrict__ dtau) {
  __shared__ float s[256];
  const int h = (int)blockIdx.x, tid = (int)threadIdx.x;
  float x = 0.f;
  if constexpr (ALL) {
    for (int32_t w = tid; w < a.W; w += 256) x += part[(size_t)w * a.H + h];
  } else if (a.hdr->magic == kPlanMagic && a.hdr->n == a.n && a.hdr->num_windows == a.W)
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

// Which kernels a call takes: those on work items (above), or a workgroup per (window,
// head) (sla_xca_win.hip), with or without the passes over long windows.  Items give every
// window one wave: right for many windows and for long ones, and a long chain where the
// chip is not full.  Measured in us, inputs from HBM, forward / backward; plain: a workgroup
// per (window, head) without, long: with the long passes:
//   case                                                  items        plain        long
//   fp16 d = 32, H = 4, 169 windows of 4 rows          11.8 / 27.9   5.1 / 14.8   5.0 / 18.3
//     63 windows of 1 to 60 rows                       11.0 / 24.9   6.5 / 14.5   6.5 / 14.3
//     LiDAR-like, 169 windows, 5k rows                 13.8 / 33.8  17.9 / 48.6  10.3 / 27.1
//     log-normal, 122 windows, 6k rows                 13.9 / 32.2  22.6 / 63.1  11.8 / 32.3
//     LiDAR-like, 900 windows, 8k rows                 14.5 / 36.2  12.5 / 41.0  18.9 / 63.9
//     LiDAR-like, 1,521 windows, 16k rows              24.0 / 52.2  20.2 / 61.1  33.9 / 105
//     the same, H = 8                                  33.3 / 80.2  35.4 / 109   62.1 / 197
//   fp16 d = 16, H = 4, 169 windows of 4 rows           8.9 / 17.9   5.7 / 12.7   5.7 / 12.3
//   fp32 d = 32, H = 4, 63 windows of 1 to 60 rows     17.4 / 37.8  12.0 / 25.0  10.8 / 24.6
//     LiDAR-like, 1,521 windows, 60k rows              52 / 126     59 / 157
// Hence: long where all (window, head) pairs are resident at once, and at d = 32 up to
// twice that where windows are neither thin (below 12 rows a slot, 28 in fp32, few are
// long and the plain kernels' smaller workgroups win) nor, in the backward, likely to be
// very long (40); plain for thin windows up to a number of pairs; items for the rest.
// The plain kernels' time goes with the pairs, that of items with the waves, of which a
// head count that is no multiple of four leaves some idle.
enum class XcaPath { kItems, kWin, kWinLong };

template <typename T, int D>
XcaPath xca_path(int32_t n, int32_t W, int32_t H, bool bwd) {
  const int64_t pairs = (int64_t)W * H, resident = xca_win_resident<T, D>(bwd);
  const auto rows_below = [&](int64_t r) { return (int64_t)n < r * W; };   // rows per window slot
  if (pairs <= resident) return XcaPath::kWinLong;
  if constexpr (D == 32)
    if (pairs <= 2 * resident && !rows_below(Ty<T>::kNarrow ? 12 : 28) && (!bwd || rows_below(40)))
      return XcaPath::kWinLong;
  if constexpr (!Ty<T>::kNarrow) return rows_below(28) ? XcaPath::kWin : XcaPath::kItems;
  if constexpr (D == 16) return rows_below(6) && pairs <= 3700 ? XcaPath::kWin : XcaPath::kItems;
  if (bwd) return rows_below(12) && pairs <= 2000 ? XcaPath::kWin : XcaPath::kItems;
  const int waves = H < 4 ? H * (4 / H) : H, of = (waves + 3) / 4 * 4;
  const int64_t most = std::is_same<T, bf16_t>::value ? 4500 : 7500;   // bf16: A is a pair of operands
  return rows_below(20) && pairs * waves <= most * of ? XcaPath::kWin : XcaPath::kItems;
}

template <typename T, int D>
hipError_t xca_impl(const void* plan, int32_t n, int32_t W, int32_t H, const float* tau,
                    const void* q, const void* k, const void* v, void* o, hipStream_t stream) {
  const T *qt = static_cast<const T*>(q), *kt = static_cast<const T*>(k), *vt = static_cast<const T*>(v);
  const XcaPath path = xca_path<T, D>(n, W, H, false);
  if (path != XcaPath::kItems)
    return launch_xca_win_fwd<T, D>(plan, n, W, H, path == XcaPath::kWinLong, tau, qt, kt, vt, static_cast<T*>(o),
                                    stream);
  const PlanLayout lay = plan_layout(n, W);
  const KernelArgs a = kernel_args(plan, lay, n, W, H, 0.f);
  int grid;
  const auto kern = pick_parts(&k_xca_fwd_mma<T, D, false>, &k_xca_fwd_mma<T, D, true>, lay, n, W, H, kXcaFwdFill, grid);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), 0, stream, a, tau, qt, kt, vt, static_cast<T*>(o));
  return hipGetLastError();
}

template <typename T, int D>
hipError_t xca_bwd_impl(const void* plan, int32_t n, int32_t W, int32_t H, const float* tau,
                        const void* q, const void* k, const void* v, const void* dout, void* dq,
                        void* dk, void* dv, float* dtau, float* part, hipStream_t stream) {
  const T *qt = static_cast<const T*>(q), *kt = static_cast<const T*>(k), *vt = static_cast<const T*>(v),
          *dt = static_cast<const T*>(dout);
  T *dqt = static_cast<T*>(dq), *dkt = static_cast<T*>(dk), *dvt = static_cast<T*>(dv);
  const PlanLayout lay = plan_layout(n, W);
  const KernelArgs a = kernel_args(plan, lay, n, W, H, 0.f);
  const XcaPath path = n > 0 ? xca_path<T, D>(n, W, H, true) : XcaPath::kItems;
  if (n > 0) {
    hipError_t e;
    if (path != XcaPath::kItems) {
      e = launch_xca_win_bwd<T, D>(plan, n, W, H, path == XcaPath::kWinLong, tau, qt, kt, vt, dt, dqt, dkt, dvt, part,
                                   stream);
    } else {
      int grid;
      const auto kern =
          pick_parts(&k_xca_bwd_mma<T, D, false>, &k_xca_bwd_mma<T, D, true>, lay, n, W, H, kXcaBwdFill, grid);
      hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), 0, stream, a, tau, qt, kt, vt, dt, dqt, dkt, dvt, part);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(path == XcaPath::kItems ? &k_xca_dtau<false> : &k_xca_dtau<true>, dim3((unsigned)H), dim3(256), 0,
                     stream, a, part, dtau);
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
