// Cross-covariance attention inside every window, fp32 on the vector units: the
// kernels for scenes of thin windows (the operation and its chain rule are in
// sla_xca.hip, which also says when these run).
//
// One 256-thread workgroup per (window, head), the heads of a window on one XCD.
//   1. 64 rows at a time, the window's q and k rows (this head's d columns)
//      are gathered through the plan's permutation into LDS; thread
//      (e, c-block) accumulates G[e][c] = sum_r q_re k_rc for its EPT columns,
//      and the first wave the squared column norms.
//   2. The logits tau G[e][c] / (|q_e| |k_c|) are bounded by |tau|, so the
//      softmax needs no overflow guard beyond the usual max shift; the row max
//      and sum are reduced over the CPR threads of a row with lane xors.
//   3. Each thread keeps one row e of A in registers and, 64 rows at a time
//      with the v rows in LDS, writes o_i[e] for its rows.  A window of at most
//      64 rows gathers its v rows in step 1 already, into registers, so that
//      their round trip overlaps the sums; longer windows gather v again here.
// Bound by the vector units and their LDS reads (VALU busy 61%, LDS active 48% on a
// Waymo-like frame), with four times the waves per window of the matrix-core kernels.
#include "sla_common.h"

namespace sla {
namespace {

constexpr int kXcaThreads = 256;
constexpr int kXcaRows = 64;   // rows staged in LDS at a time

template <typename T>
struct XcaIo;
template <>
struct XcaIo<float> {
  static constexpr int kPiece = 4;   // elements per 16-byte piece
  __device__ static void unpack(uint4 u, float (&x)[4]) {
    x[0] = __uint_as_float(u.x); x[1] = __uint_as_float(u.y);
    x[2] = __uint_as_float(u.z); x[3] = __uint_as_float(u.w);
  }
  __device__ static void store(float* p, float x) { *p = x; }
};
// Workgroup b -> (window, head) such that the heads of a window share b mod 8:
// workgroups are dealt to the 8 XCDs round-robin, so the heads of a window run
// on one XCD, whose L2 then serves the other heads' quarters of each row's
// 128-byte lines.  The grid is 8 ceil(W / 8) H; workgroups past the last window
// have nothing to do.
__device__ __forceinline__ void xca_item(uint32_t b, int32_t H, int32_t& w, int32_t& h) {
  const uint32_t per = 8u * (uint32_t)H;
  const uint32_t g = b / per, r = b - g * per;
  h = (int32_t)(r >> 3);
  w = (int32_t)(g * 8u + (r & 7u));
}

inline unsigned xca_grid(int32_t W, int32_t H) { return (unsigned)(((int64_t)W + 7) / 8 * 8 * H); }

// LDS row stride of the staged rows: 16-byte aligned rows for float4 reads
template <int D>
constexpr int kXcaLd = D + 4;

// 16-byte pieces of a staged block: piece j = (row r, piece pc); a thread takes
// pieces tid, tid + 256 (at most two: 64 rows of 32 fp32 columns)
template <typename T, int D>
constexpr int kXcaPieces = kXcaRows * D / XcaIo<T>::kPiece;
template <typename T, int D>
constexpr int kXcaPerThread = (kXcaPieces<T, D> + kXcaThreads - 1) / kXcaThreads;

// Gathers the raw pieces of rows [p0, p0 + nr) (sorted positions) of `x` into
// registers (zero past nr or for an out-of-range row) and, when s_row is given,
// records each row's original index there (-1 for none).
template <typename T, int D>
__device__ __forceinline__ void xca_fetch(const int32_t* pm, int32_t p0, int nr, int32_t n,
                                          size_t rs, int col, const T* x,
                                          uint4 (&raw)[kXcaPerThread<T, D>], int32_t* s_row) {
  constexpr int PB = XcaIo<T>::kPiece, PR = D / PB;
#pragma unroll
  for (int u = 0; u < kXcaPerThread<T, D>; ++u) {
    const int j = (int)threadIdx.x + u * kXcaThreads;
    const int r = j / PR, pc = j - r * PR;
    int32_t row = -1;
    if (j < kXcaPieces<T, D> && r < nr) {
      row = pm ? pm[p0 + r] : p0 + r;
      if ((uint32_t)row >= (uint32_t)n) row = -1;
    }
    raw[u] = row >= 0 ? *reinterpret_cast<const uint4*>(x + (size_t)row * rs + col + pc * PB)
                      : make_uint4(0, 0, 0, 0);
    if (s_row && j < kXcaPieces<T, D> && pc == 0) s_row[r] = row;
  }
}

// Raw pieces into an LDS block of fp32 rows.
template <typename T, int D>
__device__ __forceinline__ void xca_put(const uint4 (&raw)[kXcaPerThread<T, D>],
                                        float (*a)[kXcaLd<D>]) {
  constexpr int PB = XcaIo<T>::kPiece, PR = D / PB;
#pragma unroll
  for (int u = 0; u < kXcaPerThread<T, D>; ++u) {
    const int j = (int)threadIdx.x + u * kXcaThreads;
    if (j < kXcaPieces<T, D>) {
      const int r = j / PR, pc = j - r * PR;
      float x[PB];
      XcaIo<T>::unpack(raw[u], x);
#pragma unroll
      for (int e = 0; e < PB; ++e) a[r][pc * PB + e] = x[e];
    }
  }
}

template <typename T, int D>
__global__ __launch_bounds__(kXcaThreads) void k_xca_fwd(
    const PlanHeader* __restrict__ hdr, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ offs, const float* __restrict__ tau, const T* __restrict__ q,
    const T* __restrict__ k, const T* __restrict__ v, T* __restrict__ o, int32_t n, int32_t W,
    int32_t H) {
  constexpr int EPT = D * D / kXcaThreads;   // entries (e, c) per thread: 4 (d = 32) or 1 (d = 16)
  constexpr int CPR = D / EPT;               // threads per row e of G
  constexpr int RPP = kXcaThreads / D;       // output rows per pass of phase 3
  static_assert(D * D % kXcaThreads == 0 && CPR <= 64 && (CPR & (CPR - 1)) == 0, "row groups");
  constexpr int LD = kXcaLd<D>;
  constexpr int NP = kXcaPerThread<T, D>;
  __shared__ __align__(16) float s_a[kXcaRows][LD];   // q rows, then v rows
  __shared__ __align__(16) float s_b[kXcaRows][LD];   // k rows
  __shared__ float s_g[D][D + 1];          // softmax weights A
  __shared__ float s_nrm[2 * D];           // |q_e|, then |k_c|
  __shared__ int32_t s_row[kXcaRows];
  int32_t w, h;
  xca_item(blockIdx.x, H, w, h);
  if (w >= W) return;
  if (hdr->magic != kPlanMagic || hdr->n != n || hdr->num_windows != W) return;
  const int32_t* pm = hdr->csr ? nullptr : perm;
  const int32_t rb = max(0, min(offs[w], n)), re = max(rb, min(offs[w + 1], n));
  if (rb == re) return;
  const int tid = (int)threadIdx.x;
  const size_t rs = (size_t)H * D;
  const int col = h * D;

  // 1. G = q^T k over the window's rows, and the squared column norms
  const int e = tid / CPR, c0 = (tid - e * CPR) * EPT;
  float acc[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) acc[u] = 0.f;
  float nrm = 0.f;
  // a window of at most one block also gathers its v rows now, into registers,
  // so that their round trip overlaps the q^T k sums
  const bool one = re - rb <= kXcaRows;
  uint4 vr[NP];
  for (int32_t p0 = rb; p0 < re; p0 += kXcaRows) {
    const int nr = min(kXcaRows, re - p0);
    if (p0 != rb) __syncthreads();   // the previous block's readers are done
    {
      uint4 qr[NP], kr[NP];
      xca_fetch<T, D>(pm, p0, nr, n, rs, col, q, qr, s_row);
      xca_fetch<T, D>(pm, p0, nr, n, rs, col, k, kr, nullptr);
      if (one) xca_fetch<T, D>(pm, p0, nr, n, rs, col, v, vr, nullptr);
      xca_put<T, D>(qr, s_a);
      xca_put<T, D>(kr, s_b);
    }
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
      const float a = s_a[r][e];
#pragma unroll
      for (int u = 0; u < EPT; ++u) acc[u] += a * s_b[r][c0 + u];
    }
    // the first wave sums the squared columns (q in lanes 0..D-1, k after)
    if (tid < D) {
      for (int r = 0; r < nr; ++r) nrm += s_a[r][tid] * s_a[r][tid];
    } else if (tid < 2 * D) {
      for (int r = 0; r < nr; ++r) nrm += s_b[r][tid - D] * s_b[r][tid - D];
    }
  }
  if (tid < 2 * D) s_nrm[tid] = fmaxf(sqrtf(nrm), 1e-12f);
  __syncthreads();

  // 2. softmax of each row e over c
  const float t = tau[h];
  float g[EPT];
  float mx = -3.0e38f;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    g[u] = t * acc[u] / (s_nrm[e] * s_nrm[D + c0 + u]);
    mx = fmaxf(mx, g[u]);
  }
#pragma unroll
  for (int m = 1; m < CPR; m <<= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    g[u] = expf(g[u] - mx);
    sum += g[u];
  }
#pragma unroll
  for (int m = 1; m < CPR; m <<= 1) sum += __shfl_xor(sum, m, 64);
  const float inv = 1.f / sum;
#pragma unroll
  for (int u = 0; u < EPT; ++u) s_g[e][c0 + u] = g[u] * inv;
  // s_a's last readers (the q^T k sums) passed the barrier above
  if (one) xca_put<T, D>(vr, s_a);
  __syncthreads();

  // 3. o_i[e3] = sum_c A[e3][c] v_i[c]
  const int e3 = tid % D, r3 = tid / D;
  float arow[D];
#pragma unroll
  for (int c = 0; c < D; ++c) arow[c] = s_g[e3][c];
  for (int32_t p0 = rb; p0 < re; p0 += kXcaRows) {
    const int nr = min(kXcaRows, re - p0);
    if (!one) {
      __syncthreads();   // s_a and s_row are free
      uint4 raw[NP];
      xca_fetch<T, D>(pm, p0, nr, n, rs, col, v, raw, s_row);
      xca_put<T, D>(raw, s_a);
      __syncthreads();
    }
    for (int r = r3; r < nr; r += RPP) {
      const int32_t row = s_row[r];
      float s = 0.f;
#pragma unroll
      for (int c = 0; c < D; c += 4) {
        const float4 x = *reinterpret_cast<const float4*>(&s_a[r][c]);
        s += arow[c] * x.x + arow[c + 1] * x.y + arow[c + 2] * x.z + arow[c + 3] * x.w;
      }
      if (row >= 0) XcaIo<T>::store(o + (size_t)row * rs + col + e3, s);
    }
  }
}

// Backward, in passes over the window's rows: q, k (N, as in the forward); dout, v
// (dA and dv); q, k again (dqh, dkh and their projections; then dq, dk, from
// registers for a window of one block, from a further pass over q, k otherwise).
template <typename T, int D>
__global__ __launch_bounds__(kXcaThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 5))) void k_xca_bwd(
    const PlanHeader* __restrict__ hdr, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ offs, const float* __restrict__ tau, const T* __restrict__ q,
    const T* __restrict__ k, const T* __restrict__ v, const T* __restrict__ dout,
    T* __restrict__ dq, T* __restrict__ dk, T* __restrict__ dv, float* __restrict__ part,
    int32_t n, int32_t W, int32_t H) {
  constexpr int EPT = D * D / kXcaThreads;
  constexpr int CPR = D / EPT;
  constexpr int RPP = kXcaThreads / D;
  constexpr int LD = kXcaLd<D>;
  constexpr int NP = kXcaPerThread<T, D>;
  constexpr int NW = kXcaThreads / 64;
  __shared__ __align__(16) float s_a[kXcaRows][LD];
  __shared__ __align__(16) float s_b[kXcaRows][LD];
  // A (rows of D + 1) until pass 2 ends, then B_q[e][c] = tau dG[e][c] / nk_c
  // (rows of LD) in the same place
  __shared__ __align__(16) float s_ab[D * LD];
  float (*const s_g)[D + 1] = reinterpret_cast<float (*)[D + 1]>(s_ab);
  float (*const s_bq)[LD] = reinterpret_cast<float (*)[LD]>(s_ab);
  __shared__ __align__(16) float s_bk[D][LD];   // B_k[c][e] = tau dG[e][c] / nq_e
  __shared__ float s_sp[2 * RPP][D]; // shares of s_e and t_c
  __shared__ float s_nrm[2 * D];     // nq, nk
  __shared__ float s_st[2 * D];      // s_e, t_c
  __shared__ float s_red[NW];
  __shared__ int32_t s_row[kXcaRows];
  const int tid = (int)threadIdx.x;
  int32_t w, h;
  xca_item(blockIdx.x, H, w, h);
  if (w >= W) return;
  const size_t b = (size_t)w * H + h;   // this (window, head)'s temperature partial
  if (hdr->magic != kPlanMagic || hdr->n != n || hdr->num_windows != W) {
    if (tid == 0) part[b] = 0.f;
    return;
  }
  const int32_t* pm = hdr->csr ? nullptr : perm;
  const int32_t rb = max(0, min(offs[w], n)), re = max(rb, min(offs[w + 1], n));
  if (rb == re) {
    if (tid == 0) part[b] = 0.f;
    return;
  }
  const size_t rs = (size_t)H * D;
  const int col = h * D;
  const float t = tau[h];

  // 1. N = qhat^T khat (raw sums and column norms), A
  const int e = tid / CPR, c0 = (tid - e * CPR) * EPT;
  float acc[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) acc[u] = 0.f;
  float nrm = 0.f;
  for (int32_t p0 = rb; p0 < re; p0 += kXcaRows) {
    const int nr = min(kXcaRows, re - p0);
    if (p0 != rb) __syncthreads();
    {
      uint4 qr[NP], kr[NP];
      xca_fetch<T, D>(pm, p0, nr, n, rs, col, q, qr, s_row);
      xca_fetch<T, D>(pm, p0, nr, n, rs, col, k, kr, nullptr);
      xca_put<T, D>(qr, s_a);
      xca_put<T, D>(kr, s_b);
    }
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
      const float x = s_a[r][e];
#pragma unroll
      for (int u = 0; u < EPT; ++u) acc[u] += x * s_b[r][c0 + u];
    }
    if (tid < D) {
      for (int r = 0; r < nr; ++r) nrm += s_a[r][tid] * s_a[r][tid];
    } else if (tid < 2 * D) {
      for (int r = 0; r < nr; ++r) nrm += s_b[r][tid - D] * s_b[r][tid - D];
    }
  }
  if (tid < 2 * D) s_nrm[tid] = fmaxf(sqrtf(nrm), 1e-12f);
  __syncthreads();
  float nn[EPT], a[EPT];
  float mx = -3.0e38f;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    nn[u] = acc[u] / (s_nrm[e] * s_nrm[D + c0 + u]);
    a[u] = t * nn[u];
    mx = fmaxf(mx, a[u]);
  }
#pragma unroll
  for (int m = 1; m < CPR; m <<= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    a[u] = expf(a[u] - mx);
    sum += a[u];
  }
#pragma unroll
  for (int m = 1; m < CPR; m <<= 1) sum += __shfl_xor(sum, m, 64);
  const float inv = 1.f / sum;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    a[u] *= inv;
    s_g[e][c0 + u] = a[u];
  }
  __syncthreads();

  // 2. dA = sum_i do_i v_i^T, and dv_i[x3] = sum_e A[e][x3] do_i[e]
  const int x3 = tid % D, r3 = tid / D;
  float acl[D];
#pragma unroll
  for (int j = 0; j < D; ++j) acl[j] = s_g[j][x3];
  float da[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) da[u] = 0.f;
  for (int32_t p0 = rb; p0 < re; p0 += kXcaRows) {
    const int nr = min(kXcaRows, re - p0);
    __syncthreads();   // s_a, s_b, s_row (and s_g's column reads) are done with
    {
      uint4 dr[NP], vr[NP];
      xca_fetch<T, D>(pm, p0, nr, n, rs, col, dout, dr, s_row);
      xca_fetch<T, D>(pm, p0, nr, n, rs, col, v, vr, nullptr);
      xca_put<T, D>(dr, s_a);
      xca_put<T, D>(vr, s_b);
    }
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
      const float x = s_a[r][e];
#pragma unroll
      for (int u = 0; u < EPT; ++u) da[u] += x * s_b[r][c0 + u];
    }
    for (int r = r3; r < nr; r += RPP) {
      const int32_t row = s_row[r];
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < D; j += 4) {
        const float4 x = *reinterpret_cast<const float4*>(&s_a[r][j]);
        s += acl[j] * x.x + acl[j + 1] * x.y + acl[j + 2] * x.z + acl[j + 3] * x.w;
      }
      if (row >= 0) XcaIo<T>::store(dv + (size_t)row * rs + col + x3, s);
    }
  }

  // 3. dG and the temperature partial
  float rsum = 0.f;
#pragma unroll
  for (int u = 0; u < EPT; ++u) rsum += a[u] * da[u];
#pragma unroll
  for (int m = 1; m < CPR; m <<= 1) rsum += __shfl_xor(rsum, m, 64);
  float dg[EPT], pt = 0.f, srow = 0.f;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    dg[u] = a[u] * (da[u] - rsum);
    pt += dg[u] * nn[u];
  }
  srow = pt;
#pragma unroll
  for (int m = 1; m < CPR; m <<= 1) srow += __shfl_xor(srow, m, 64);   // sum_c dG N over row e
  // the workgroup's sum of dG * N: the rows' sums, wave by wave, in order
  float wsum = (tid - e * CPR) == 0 ? srow : 0.f;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) wsum += __shfl_xor(wsum, m, 64);
  __syncthreads();   // the last block's readers of s_a, s_b and every reader of s_g (A,
                     // whose place B_q takes) are done
  if ((tid & 63) == 0) s_red[tid >> 6] = wsum;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    s_bq[e][c0 + u] = t * dg[u] / s_nrm[D + c0 + u];
    s_bk[c0 + u][e] = t * dg[u] / s_nrm[e];
  }
  __syncthreads();
  if (tid == 0) {
    float tot = 0.f;
#pragma unroll
    for (int j = 0; j < NW; ++j) tot += s_red[j];
    part[b] = tot;
  }

  // 4. dqh[:, x3], dkh[:, x3] for rows r3, r3 + RPP, ... of each block, and their
  //    projections on qhat[:, x3], khat[:, x3]
  const float nq = s_nrm[x3], nk = s_nrm[D + x3];
  constexpr int RPT = kXcaRows / RPP;   // rows of a block per thread
  float gqr[RPT], gkr[RPT];
  // dqh and dkh of this thread's rows of the block in LDS: rows B_q[x3] and
  // B_k[x3] are read 4 columns at a time, outside the loop over the rows, so
  // that only one slice of them is held in registers
  auto grads = [&](int nr) {
#pragma unroll
    for (int m = 0; m < RPT; ++m) {
      gqr[m] = 0.f;
      gkr[m] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < D; j += 4) {
      const float4 bq = *reinterpret_cast<const float4*>(&s_bq[x3][j]);
      const float4 bk = *reinterpret_cast<const float4*>(&s_bk[x3][j]);
#pragma unroll
      for (int m = 0; m < RPT; ++m) {
        const int r = r3 + RPP * m;
        if (r < nr) {
          const float4 kx = *reinterpret_cast<const float4*>(&s_b[r][j]);
          const float4 qx = *reinterpret_cast<const float4*>(&s_a[r][j]);
          gqr[m] += bq.x * kx.x + bq.y * kx.y + bq.z * kx.z + bq.w * kx.w;
          gkr[m] += bk.x * qx.x + bk.y * qx.y + bk.z * qx.z + bk.w * qx.w;
        }
      }
    }
  };
  auto fetch_qk = [&](int32_t p0, int nr) {
    uint4 qr[NP], kr[NP];
    xca_fetch<T, D>(pm, p0, nr, n, rs, col, q, qr, s_row);
    xca_fetch<T, D>(pm, p0, nr, n, rs, col, k, kr, nullptr);
    xca_put<T, D>(qr, s_a);
    xca_put<T, D>(kr, s_b);
  };
  float ps = 0.f, pk = 0.f;   // this thread's share of s_x3 and t_x3, in row order
  for (int32_t p0 = rb; p0 < re; p0 += kXcaRows) {
    const int nr = min(kXcaRows, re - p0);
    __syncthreads();
    fetch_qk(p0, nr);
    __syncthreads();
    grads(nr);
#pragma unroll
    for (int m = 0; m < RPT; ++m) {
      const int r = r3 + RPP * m;
      if (r < nr) {
        ps += (s_a[r][x3] / nq) * gqr[m];
        pk += (s_b[r][x3] / nk) * gkr[m];
      }
    }
  }
  // s_x3 = the RPP shares in order (the floor makes the norm a constant: no projection)
  s_sp[r3][x3] = ps;
  s_sp[RPP + r3][x3] = pk;
  __syncthreads();
  if (tid < 2 * D) {
    const int c = tid & (D - 1), which = tid / D;
    float x = 0.f;
#pragma unroll
    for (int j = 0; j < RPP; ++j) x += s_sp[which * RPP + j][c];
    s_st[tid] = s_nrm[tid] > 1e-12f ? x : 0.f;
  }
  __syncthreads();
  const float sq = s_st[x3], tk = s_st[D + x3];

  // 5. dq[:, x3] and dk[:, x3]; a window of one block still has its q, k rows in
  //    LDS and its dqh, dkh in registers
  const bool one_block = re - rb <= kXcaRows;
  for (int32_t p0 = rb; p0 < re; p0 += kXcaRows) {
    const int nr = min(kXcaRows, re - p0);
    if (!one_block) {
      __syncthreads();
      fetch_qk(p0, nr);
      __syncthreads();
      grads(nr);
    }
#pragma unroll
    for (int m = 0; m < RPT; ++m) {
      const int r = r3 + RPP * m;
      if (r >= nr) continue;
      const int32_t row = s_row[r];
      if (row >= 0) {
        XcaIo<T>::store(dq + (size_t)row * rs + col + x3, (gqr[m] - (s_a[r][x3] / nq) * sq) / nq);
        XcaIo<T>::store(dk + (size_t)row * rs + col + x3, (gkr[m] - (s_b[r][x3] / nk) * tk) / nk);
      }
    }
  }
}

template <int D>
hipError_t fwd_impl(const void* plan, int32_t n, int32_t W, int32_t H, const float* tau, const float* q,
                    const float* k, const float* v, float* o, hipStream_t stream) {
  const PlanLayout lay = plan_layout(n, W);
  const char* base = static_cast<const char*>(plan);
  hipLaunchKernelGGL((k_xca_fwd<float, D>), dim3(xca_grid(W, H)), dim3(kXcaThreads), 0, stream,
                     reinterpret_cast<const PlanHeader*>(base + lay.header),
                     reinterpret_cast<const int32_t*>(base + lay.perm),
                     reinterpret_cast<const int32_t*>(base + lay.offsets), tau, q, k, v, o, n, W, H);
  return hipGetLastError();
}

template <int D>
hipError_t bwd_impl(const void* plan, int32_t n, int32_t W, int32_t H, const float* tau, const float* q,
                    const float* k, const float* v, const float* dout, float* dq, float* dk, float* dv,
                    float* part, hipStream_t stream) {
  const PlanLayout lay = plan_layout(n, W);
  const char* base = static_cast<const char*>(plan);
  hipLaunchKernelGGL((k_xca_bwd<float, D>), dim3(xca_grid(W, H)), dim3(kXcaThreads), 0, stream,
                     reinterpret_cast<const PlanHeader*>(base + lay.header),
                     reinterpret_cast<const int32_t*>(base + lay.perm),
                     reinterpret_cast<const int32_t*>(base + lay.offsets), tau, q, k, v, dout, dq, dk, dv, part,
                     n, W, H);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_xca_vec_fwd(const void* plan, int32_t n, int32_t W, int32_t H, int32_t d, const float* tau,
                              const float* q, const float* k, const float* v, float* o, hipStream_t stream) {
  if (d == 32) return fwd_impl<32>(plan, n, W, H, tau, q, k, v, o, stream);
  return fwd_impl<16>(plan, n, W, H, tau, q, k, v, o, stream);
}

hipError_t launch_xca_vec_bwd(const void* plan, int32_t n, int32_t W, int32_t H, int32_t d, const float* tau,
                              const float* q, const float* k, const float* v, const float* dout, float* dq,
                              float* dk, float* dv, float* part, hipStream_t stream) {
  if (d == 32) return bwd_impl<32>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, part, stream);
  return bwd_impl<16>(plan, n, W, H, tau, q, k, v, dout, dq, dk, dv, part, stream);
}

}  // namespace sla
