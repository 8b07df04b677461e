// The steps of one greedy pick between two streaming passes: six kernels,
// for one selection problem or, along gridDim.z, for several at once (the
// blocks of Algorithm 4, each with its own state and buffers).
//
// With Q the orthonormal FP64 basis of the t picks so far, a the pick's
// column (decoded to FP64 by the previous streaming pass), V = [w_1 .. w_t]
// the history of the target vectors w_s = B B^T q_s (for B = A: (A A^T) q_s),
// and B the explicit target (for B = A, C = A A^T in its place):
//
//   K1  dots   c1 = Q^T a                          (partials over row blocks)
//   K2  rows   e1 = a - Q c1
//   K3  dots   c2 = Q^T e1
//   K4  rows   e2 = e1 - Q c2,  ||e2||^2 per workgroup
//   K5  dots   [B^T e2 ; V^T e2]                   (B = A: [C e2 ; V^T e2])
//   K6  rows   ||e2||^2 and the basis check; with q = e2 / ||e2||:
//              upsilon = B^T q, c3 = V^T q = Q^T (B B^T q), w = B upsilon
//              (B = A: w = C q), z = w - Q c3, V[:, t] = w, Q[:, t] = q;
//              the last workgroup to finish records the pick and the
//              objective decrease ||upsilon||^2 (B = A: q . w).
//
// This is Gram-Schmidt with one re-orthogonalisation (K1-K4) and the target
// operations of Theorem 4 in the q/z form (K5-K6): omega = A^T q and
// gamma = A^T z then come from one streaming pass.  c3 is formed as V^T q
// (equal to Q^T w, since q_s^T B B^T q = w_s^T q), so it needs no reduction
// after w is known.
//
// With the history of the streaming passes' omega (wh, row s holds A^T q_{s+1}
// in binary32, so c1 = column p of it) the first reduction is already done,
// and a workgroup of 32 rows that holds its rows of Q can do a row update and
// the partial dots after it in one go:
//
//   S1  e1 = a - Q c1 (a decoded from column p of A),  partials of Q^T e1
//   S2  e2 = e1 - Q c2, ||e2||^2,  partials of [B^T e2 ; V^T e2]
//   S3  = K6 on partials per 32 rows                   (B = A: K5, then K6)
//
// c1 is off by binary32 rounding (1e-7 ||a||); the second projection, formed
// in FP64 from e1 as it is, takes that out with the rest of Q's span, so e2 is
// orthogonal to Q to FP64 rounding of ||e1||.  That is as good as two projections
// in FP64 while an accepted pick's ||e2|| is far above 1e-7 ||a||, so the
// history is kept for tau >= 1e-6 only (kHistTau in gcss_api.hip).  Over 80
// random problems (m 100 .. 8192, k 10 .. 200, tau 1e-4 .. 1e-6) the largest
// |Q^T Q - I| of the two agree to 3% in the mean, 4e-16 .. 1.2e-14 both.  The partials of a
// consumer grow with m (m / 32 rows of r + t), so this form serves shapes
// whose partials stay small; above, S1 without partials replaces K1 and K2.
// The chain's kernel time per step on MI355X, six kernels -> now: m = 1024,
// r = 128, k = 50: 29 -> 19 us; m = 3001, r = 200, k = 64: 33 -> 23 us; m = 4096,
// B = A, k = 200: 42 -> 37 us; m = 8192, r = 512, k = 500 (no slab): 44 -> 40 us;
// the streaming pass without its last workgroup's work takes 7 us less.
//
// Latency is what these kernels spend: each one reads the device state, then
// issues every load it needs at once (partials of the previous kernel, the
// rows of Q, B or V it multiplies), so a kernel costs about two memory round
// trips.  Dot kernels: workgroup (x, y) forms kDotCols column sums over rows
// [1024 y, 1024 (y + 1)), written as partials P[y][c]; a consumer adds the
// ceil(m / 1024) <= kMaxRB partials of an entry in order.  Row kernels: a
// workgroup of 1024 threads owns 32 rows and its 32 groups of 32 lanes split
// the sum over columns; partial sums meet in LDS in a fixed order.  Every
// reduction has a fixed order, so results do not depend on scheduling.
#include <type_traits>

#include "gcss_device.h"

namespace gcss {

constexpr int kDotRows = 1024;  // rows per block of the dot kernels (4 consecutive per thread)
constexpr int kDotCols = 4;     // columns per dot workgroup
constexpr int kMaxRB = 8;       // row blocks of the dot kernels (m <= 8192)
constexpr int kRowRB = 32;      // rows per row-kernel workgroup
constexpr int kRowGroups = 32;  // column groups per row-kernel workgroup
constexpr int kRowThreads = kRowRB * kRowGroups;  // 1024
// columns per thread loaded in one round: the smallest U of 4, 8, 16 that takes
// a matrix in one round (32 U columns), the largest with further rounds.  A
// thread issues U loads (clamped) whatever the column count, so U = 16 for 20
// columns costs most of a row kernel's issue slots.
constexpr int kRowUMax = 16;

template <typename T>
__device__ __forceinline__ double to_f64(T v) {
  if constexpr (sizeof(T) == 2) return (double)__uint_as_float((uint32_t)v << 16);  // bfloat16
  else return (double)v;
}

// sum over y < nrb (in order) of P[y * lp + c]: all loads in flight at once
// (unconditional: y >= nrb reads row nrb - 1 again, nrb >= 1).
__device__ __forceinline__ double psum(const double *P, int64_t lp, int nrb, int64_t c) {
  double v[kMaxRB];
#pragma unroll
  for (int y = 0; y < kMaxRB; ++y) v[y] = P[(int64_t)(y < nrb ? y : nrb - 1) * lp + c];
  double s = 0.0;
#pragma unroll
  for (int y = 0; y < kMaxRB; ++y)
    if (y < nrb) s += v[y];
  return s;
}

// Fixed-order sum of one double per thread over a 1024-thread workgroup:
// wave sums, then the 16 waves in order.  Every thread gets the total.
__device__ __forceinline__ double block_sum(double v, double *wsum) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int x = 0; x < kRowThreads / 64; ++x) s += wsum[x];
  __syncthreads();
  return s;
}

// Raw loads of four consecutive elements (p aligned to four elements), kept
// as loaded until raw_f64 turns them into doubles.
template <typename T> struct Quad;
template <> struct Quad<float> { float4 v; };
template <> struct Quad<uint16_t> { uint2 v; };  // bfloat16
template <> struct Quad<double> { double2 a, b; };
__device__ __forceinline__ void raw_load(const float *p, Quad<float> &q) { q.v = *(const float4 *)p; }
__device__ __forceinline__ void raw_load(const uint16_t *p, Quad<uint16_t> &q) { q.v = *(const uint2 *)p; }
__device__ __forceinline__ void raw_load(const double *p, Quad<double> &q) {
  q.a = *(const double2 *)p;
  q.b = *(const double2 *)(p + 2);
}
__device__ __forceinline__ void raw_f64(const Quad<float> &q, double (&o)[4]) {
  o[0] = q.v.x;
  o[1] = q.v.y;
  o[2] = q.v.z;
  o[3] = q.v.w;
}
__device__ __forceinline__ void raw_f64(const Quad<uint16_t> &q, double (&o)[4]) {
  o[0] = (double)__uint_as_float(q.v.x << 16);
  o[1] = (double)__uint_as_float(q.v.x & 0xFFFF0000u);
  o[2] = (double)__uint_as_float(q.v.y << 16);
  o[3] = (double)__uint_as_float(q.v.y & 0xFFFF0000u);
}
__device__ __forceinline__ void raw_f64(const Quad<double> &q, double (&o)[4]) {
  o[0] = q.a.x;
  o[1] = q.a.y;
  o[2] = q.b.x;
  o[3] = q.b.y;
}

// The partial dots of one workgroup: P[y * lp + c] for its kDotCols columns
// c0 .. (< cend) of one matrix M (type T, ld ldm, column c - cbase), rows of
// block y.  Every load (the column quads, then x) is issued before the first
// is used.
template <typename T>
__device__ __forceinline__ void dots_block(const T *__restrict__ M, int64_t ldm, int cbase, int c0,
                                           int cend, const double *__restrict__ x, int64_t m,
                                           double *__restrict__ P, int64_t lp,
                                           double (&red)[4][kDotCols]) {
  // four consecutive rows per thread (one 16- or 32-byte load per column);
  // a quad past m reads the last quad of the column (every leading
  // dimension is a multiple of four elements) and its terms are dropped
  const int64_t jq = (int64_t)blockIdx.y * kDotRows + 4 * threadIdx.x;
  const int64_t jb = jq < m ? jq : (m - 1) & ~(int64_t)3;
  Quad<T> raw[kDotCols];
#pragma unroll
  for (int c = 0; c < kDotCols; ++c) {
    const int cc = c0 + c < cend ? c0 + c : cend - 1;
    raw_load(M + (int64_t)(cc - cbase) * ldm + jb, raw[c]);
  }
  Quad<double> xq;
  raw_load(x + jb, xq);
  double xv[4];
  raw_f64(xq, xv);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // (a row block wholly inside m uses every term unconditionally, so no load
  // is moved under a condition)
  const bool full = (int64_t)(blockIdx.y + 1) * kDotRows <= m;
#pragma unroll
  for (int c = 0; c < kDotCols; ++c) {
    double mv[4];
    raw_f64(raw[c], mv);
    double a = 0.0;
    if (full) {
#pragma unroll
      for (int u = 0; u < 4; ++u) a = fma(mv[u], xv[u], a);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (jq + u < m) a = fma(mv[u], xv[u], a);
    }
    a = wave_sum(a);
    if (lane == 0) red[wave][c] = a;
  }
  __syncthreads();
  if (threadIdx.x < kDotCols && c0 + (int)threadIdx.x < cend) {
    const int c = threadIdx.x;
    P[(int64_t)blockIdx.y * lp + c0 + c] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
  }
}

// Number of column workgroups of k_dots: the columns of M1 and those of M2
// are never mixed in one workgroup.
inline int dots_col_blocks(int nfix, int kmax) {
  return (nfix + kDotCols - 1) / kDotCols + (kmax + kDotCols - 1) / kDotCols;
}

// P[y * lp + c] = sum over rows j of block y of M_c[j] * x[j] for c < ncols,
// ncols = nfix + t: column c < nfix is column c of M1 (type T1, ld ld1; the
// target B, or C for B = A), column c >= nfix is column c - nfix of M2 (FP64,
// ld ld2).  Workgroups x < ceil(nfix / 4) take four columns of M1 each, the
// rest four columns of M2.
template <typename T1>
__global__ __launch_bounds__(256) void k_dots(const T1 *__restrict__ M1, int64_t ld1, int nfix,
                                              const double *__restrict__ M2, int64_t ld2,
                                              const double *__restrict__ x, int64_t m,
                                              double *__restrict__ P, int64_t lp,
                                              const DevState *st, int64_t s_m2, int64_t s_x,
                                              int64_t s_p) {
  __shared__ double red[4][kDotCols];
  {  // problem blockIdx.z (M1 is shared)
    const int b = blockIdx.z;
    M2 += b * s_m2;
    x += b * s_x;
    P += b * s_p;
    st += b;
  }
  if (st->done || st->skip) return;
  const int ncols = nfix + st->t;
  const int nb1 = (nfix + kDotCols - 1) / kDotCols;
  if ((int)blockIdx.x < nb1) {
    dots_block(M1, ld1, 0, (int)blockIdx.x * kDotCols, nfix, x, m, P, lp, red);
  } else {
    const int c0 = nfix + ((int)blockIdx.x - nb1) * kDotCols;
    if (c0 >= ncols) return;
    dots_block(M2, ld2, nfix, c0, ncols, x, m, P, lp, red);
  }
}

// Loads of one round of a thread's row sum: M[j + s ld] for the columns
// s = s0 + 32 u (u < U), raw, all issued before any is used; a column
// s >= ns reads column ns - 1 instead, and is dropped by the caller (ns <= 0:
// nothing is read).
template <typename T, int U>
__device__ __forceinline__ void row_loads(const T *__restrict__ col0, int64_t ld, int s0, int ns,
                                          T (&raw)[U]) {
  if (ns <= 0) {  // (the same in the whole workgroup)
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u] = T(0);
    return;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int s = s0 + kRowGroups * u;
    raw[u] = col0[(int64_t)(s < ns ? s : ns - 1) * ld];
  }
}

// The row sum of one thread: sum over columns s = g, g + 32, ... < ns of
// M[j + s ld] * c[s], the first U terms from preloaded values, the rest
// (ns > 32 U) loaded in further rounds.
template <typename T, int U>
__device__ __forceinline__ double row_sum(const T *__restrict__ col0, int64_t ld, int g, int ns,
                                          const double (&pre)[U], const double *c) {
  double acc = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int s = g + kRowGroups * u;
    if (s < ns) acc = fma(pre[u], c[s], acc);
  }
  for (int s0 = g + kRowGroups * U; s0 < ns; s0 += kRowGroups * U) {
    T raw[U];
    row_loads(col0, ld, s0, ns, raw);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s0 + kRowGroups * u;
      if (s < ns) acc = fma(to_f64(raw[u]), c[s], acc);
    }
  }
  return acc;
}

// The first U values of a thread's row sum (columns g + 32 u < ns; the
// others 0).  The loads are unconditional (clamped columns), so they are all
// in flight together instead of each waited for inside its own branch.
template <typename T, int U>
__device__ __forceinline__ void row_convert(const T (&raw)[U], int g, int ns,
                                            double (&pre)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) pre[u] = g + kRowGroups * u < ns ? to_f64(raw[u]) : 0.0;
}
template <typename T, int U>
__device__ __forceinline__ void row_preload(const T *__restrict__ col0, int64_t ld, int g, int ns,
                                            double (&pre)[U]) {
  T raw[U];
  row_loads(col0, ld, g, ns, raw);
  row_convert(raw, g, ns, pre);
}

// The rows' sums over the 32 column groups, by wave 0: lanes 0..31 add groups
// 0..15 of their row, lanes 32..63 the rest.
__device__ __forceinline__ double row_total(const double (*red)[kRowRB + 1]) {
  const int r = threadIdx.x & (kRowRB - 1), x0 = (threadIdx.x >> 5) * (kRowGroups / 2);
  double s = 0.0;
#pragma unroll
  for (int x = 0; x < kRowGroups / 2; ++x) s += red[x0 + x][r];
  return s + __shfl_xor(s, 32, 64);
}

// out = v - Q c for this workgroup's 32 rows, c[s] = sum_y P[y * lp + s]
// (s < t); NORM: Pn[blockIdx.x] = sum of out^2 over its rows.
template <bool NORM, int UQ>
__global__ __launch_bounds__(1024) void k_rows_sub(const double *__restrict__ Q, int64_t ldq,
                                                   const double *__restrict__ v,
                                                   const double *__restrict__ P, int64_t lp,
                                                   int nrb, double *__restrict__ out,
                                                   double *__restrict__ Pn, int64_t m,
                                                   const DevState *st, int64_t s_q,
                                                   int64_t s_vec, int64_t s_p, int64_t s_pn) {
  extern __shared__ double cs[];  // t coefficients
  __shared__ double red[kRowGroups][kRowRB + 1];
  {  // problem blockIdx.z
    const int b = blockIdx.z;
    Q += b * s_q;
    v += b * s_vec;
    P += b * s_p;
    out += b * s_vec;
    if (NORM) Pn += b * s_pn;
    st += b;
  }
  if (st->done || st->skip) return;
  const int t = st->t;
  const int r = threadIdx.x & (kRowRB - 1), g = threadIdx.x / kRowRB;
  const int64_t j = (int64_t)blockIdx.x * kRowRB + r;
  const int64_t jc = j < m ? j : m - 1;
  // loads: this thread's first columns of Q, the base value, the coefficients
  double pre[UQ];
  row_preload(Q + jc, ldq, g, t, pre);
  const double vj = v[jc];
  for (int s = threadIdx.x; s < t; s += kRowThreads) cs[s] = psum(P, lp, nrb, s);
  __syncthreads();
  red[g][r] = row_sum(Q + jc, ldq, g, t, pre, cs);
  __syncthreads();
  if (threadIdx.x < 64) {  // wave 0: lanes 0..31 own the rows
    const double sum = row_total(red);
    double o = 0.0;
    if (threadIdx.x < kRowRB && j < m) {
      o = vj - sum;
      out[j] = o;
    }
    if constexpr (NORM) {
      const double sq = wave_sum(o * o);
      if (threadIdx.x == 0) Pn[blockIdx.x] = sq;
    }
  }
}

// ---- the slab form (S1, S2; see the file comment) ----

// Sum over each half of a wave (32 lanes), in lanes 31 and 63: four DPP steps
// leave a row's sum in its 16 lanes, one row broadcast adds row 0 to row 1
// and row 2 to row 3.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_step64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double half_total(double v) {
  v += dpp_step64<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
  v += dpp_step64<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
  v += dpp_step64<0x141, 0xF>(v);  // row_half_mirror
  v += dpp_step64<0x140, 0xF>(v);  // row_mirror
  v += dpp_step64<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  return v;
}

// P[s] = sum over the workgroup's 32 rows of x[u] * er for the columns
// s = g + 32 u < ns (x[u] = 0 beyond ns; er: this lane's row).
template <int U>
__device__ __forceinline__ void slab_dots(const double (&x)[U], double er, int g, int ns,
                                          double *__restrict__ P) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (kRowGroups * u >= ns) break;
    const double d = half_total(x[u] * er);
    const int s = g + kRowGroups * u;
    if ((threadIdx.x & 31) == 31 && s < ns) P[s] = d;
  }
}

// out[c] = sum over y < ng (in a fixed order) of P[y * lp + c], c < ne, by the
// 1024 threads of a workgroup: with few entries several threads share one,
// each adding a run of the partials, 16 in flight.  Ends with a barrier.
__device__ __forceinline__ void slab_sums(const double *__restrict__ P, int64_t lp, int ng, int ne,
                                          double *out, double *tmp) {
  int sh = 6;
  while (sh < 10 && (1 << sh) < ne) ++sh;
  const int width = 1 << sh, parts = kRowThreads >> sh;
  const int per = (ng + parts - 1) / parts;
  const int h = threadIdx.x >> sh, ci = threadIdx.x & (width - 1);
  const int y0 = h * per, y1 = y0 + per < ng ? y0 + per : ng;
  for (int c0 = 0; c0 < ne; c0 += width) {
    const int c = c0 + ci < ne ? c0 + ci : ne - 1;
    double a = 0.0;
    for (int y = y0; y < y1; y += 16) {
      double v[16];
#pragma unroll
      for (int x = 0; x < 16; ++x) v[x] = P[(int64_t)(y + x < y1 ? y + x : y1 - 1) * lp + c];
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (y + x < y1) a += v[x];
    }
    if (parts == 1) {
      if (c0 + ci < ne) out[c0 + ci] = a;
    } else {
      tmp[threadIdx.x] = a;
      __syncthreads();
      if ((int)threadIdx.x < width && c0 + ci < ne) {
        double b = 0.0;
        for (int x = 0; x < parts; ++x) b += tmp[x * width + ci];
        out[c0 + ci] = b;
      }
      __syncthreads();
    }
  }
  __syncthreads();
}

// S1: the next pick p from the streaming pass's per-workgroup winners (every
// workgroup reduces them by itself: 256 entries cost less than the pass's last
// workgroup doing it behind a device-wide arrival), then e1 = a - Q c1 for
// this workgroup's 32 rows; PART: P[blockIdx.x] = partials of Q^T e1
// (t <= 32 UQ).  Workgroup 0 writes the pick to the state, whose fields that
// the other workgroups read here (done, t) change only where none is left.
template <bool PART, int UQ>
__global__ __launch_bounds__(1024) void k_gs1(AView A, const float *__restrict__ wh, int64_t ldw,
                                              const ArgPart *__restrict__ part, int npart,
                                              const double *__restrict__ Q, int64_t ldq,
                                              double *__restrict__ e1, double *__restrict__ P,
                                              int64_t lp, int64_t m, DevState *st) {
  extern __shared__ double cs[];  // t coefficients
  __shared__ double red[kRowGroups][kRowRB + 1];
  __shared__ double er[kRowRB];
  __shared__ double bs[kRowThreads / 64];
  __shared__ int64_t bi[kRowThreads / 64];
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  if (st->done) {
    if (first) st->dec_pending = 0;  // the pass after the last pick has run
    return;
  }
  const int t = st->t;
  const int r = threadIdx.x & (kRowRB - 1), g = threadIdx.x / kRowRB;
  const int64_t j = (int64_t)blockIdx.x * kRowRB + r;
  const int64_t jc = j < m ? j : m - 1;
  double raw[UQ], pre[UQ];
  row_loads(Q + jc, ldq, g, t, raw);
  double best = -INFINITY;
  int64_t p = kNoIdx;
  for (int x = threadIdx.x; x < npart; x += kRowThreads) {
    const double sc = part[x].score;
    const int64_t i = part[x].idx;
    if (better(sc, i, best, p)) {
      best = sc;
      p = i;
    }
  }
  const int nw = npart < kRowThreads ? (npart + 63) >> 6 : kRowThreads / 64;
  if ((int)(threadIdx.x >> 6) < nw) {
    wave_argmax(best, p);
    if ((threadIdx.x & 63) == 0) {
      bs[threadIdx.x >> 6] = best;
      bi[threadIdx.x >> 6] = p;
    }
  }
  __syncthreads();
  best = bs[0];
  p = bi[0];
  for (int x = 1; x < nw; ++x)
    if (better(bs[x], bi[x], best, p)) {
      best = bs[x];
      p = bi[x];
    }
  if (first) {
    st->skip = 0;
    st->dec_pending = 0;
    if (p == kNoIdx) {
      st->p = -1;
      st->exhausted = 1;
      st->done = 1;
    } else {
      st->p = p;
    }
  }
  if (p == kNoIdx) return;
  double aj = 0.0;
  if (threadIdx.x < kRowRB) aj = col_scale(A, p) * (double)load_elem(A, p, jc);
  for (int s = threadIdx.x; s < t; s += kRowThreads) cs[s] = (double)wh[(int64_t)s * ldw + p];
  __syncthreads();
  row_convert(raw, g, t, pre);
  red[g][r] = row_sum(Q + jc, ldq, g, t, pre, cs);
  __syncthreads();
  if (threadIdx.x < 64) {
    const double sum = row_total(red);
    if (threadIdx.x < kRowRB) {
      const double o = aj - sum;
      if (j < m) e1[j] = o;
      if constexpr (PART) er[r] = j < m ? o : 0.0;
    }
  }
  if constexpr (PART) {
    __syncthreads();
    slab_dots(pre, er[r], g, t, P + (int64_t)blockIdx.x * lp);
  }
}

// S2: e2 = e1 - Q c2 with c2 the sums of S1's partials, the norm partial, and
// (explicit target) the partials [B^T e2 ; V^T e2] of this workgroup's rows.
template <typename TB, bool GRAM, int UQ, int UB>
__global__ __launch_bounds__(1024) void k_gs2(const double *__restrict__ Q, int64_t ldq,
                                              const double *__restrict__ V,
                                              const TB *__restrict__ B, int64_t ldb, int r,
                                              const double *__restrict__ e1,
                                              const double *__restrict__ P1, int64_t lp1,
                                              double *__restrict__ e2, double *__restrict__ Pn,
                                              double *__restrict__ P2, int64_t lp2, int64_t m,
                                              const DevState *st) {
  extern __shared__ double cs[];  // t coefficients
  __shared__ double red[kRowGroups][kRowRB + 1];
  __shared__ double tmp[kRowThreads];
  __shared__ double er[kRowRB];
  if (st->done || st->skip) return;
  const int t = st->t;
  const int rr = threadIdx.x & (kRowRB - 1), g = threadIdx.x / kRowRB;
  const int64_t j = (int64_t)blockIdx.x * kRowRB + rr;
  const int64_t jc = j < m ? j : m - 1;
  double qraw[UQ], vraw[UQ];
  TB braw[UB];
  row_loads(Q + jc, ldq, g, t, qraw);
  const double ej = e1[jc];
  if constexpr (!GRAM) {
    row_loads(B + jc, ldb, g, r, braw);
    row_loads(V + jc, ldq, g, t, vraw);
  }
  slab_sums(P1, lp1, (int)gridDim.x, t, cs, tmp);
  double pre[UQ];
  row_convert(qraw, g, t, pre);
  red[g][rr] = row_sum(Q + jc, ldq, g, t, pre, cs);
  __syncthreads();
  if (threadIdx.x < 64) {  // wave 0: lanes 0..31 own the rows
    const double sum = row_total(red);
    double o = 0.0;
    if (threadIdx.x < kRowRB) {
      if (j < m) {
        o = ej - sum;
        e2[j] = o;
      }
      er[rr] = o;
    }
    const double sq = wave_sum(o * o);
    if (threadIdx.x == 0) Pn[blockIdx.x] = sq;
  }
  if constexpr (!GRAM) {
    __syncthreads();
    const double e = er[rr];
    double *const P = P2 + (int64_t)blockIdx.x * lp2;
    double bpre[UB];
    row_convert(braw, g, r, bpre);
    slab_dots(bpre, e, g, r, P);
    row_convert(vraw, g, t, pre);
    slab_dots(pre, e, g, t, P + r);
  }
}

// Arguments of the last kernel of the step (see the file comment).
struct ZArgs {
  double *Q;         // basis (read: columns < t; written: column t)
  int64_t ldq;
  double *V;         // w history, ld ldq
  const double *e2;
  const double *P;   // K5 partials: [B^T e2 ; V^T e2], or [C e2 ; V^T e2]
  int64_t lp;
  int nrb;
  const double *Pn;  // K4 norm partials
  int npn;
  double *Pu;        // q . w partials (B = A)
  const void *B;     // explicit target (TB)
  int64_t ldb;
  int r;             // explicit target width (B = A: 0)
  int nfix;          // entries of P before the V^T e2 block (r, or m for B = A)
  double *q64;
  float *q32, *z32;
  const double *g0;
  uint8_t *mask;
  int64_t *idx;
  double *obj;
  int64_t m;
  int64_t s_q, s_vec, s_p, s_pn, s_q32, s_io;  // per-problem strides (see ChainArgs)
};

// TB: element type of the explicit target (float or bfloat16 bits); GRAM:
// B = A through C = A A^T (w comes from K5's partials of C e2); SLAB: the
// partials are S2's, one row of r + t per 32-row workgroup.
template <typename TB, bool GRAM, bool SLAB, int UQ, int UB>
__global__ __launch_bounds__(1024) void k_rows_z(ZArgs za, DevState *st) {
  extern __shared__ double sh[];  // upsilon (r) then c3 (t)
  __shared__ double tmp[SLAB ? kRowThreads : 1];
  __shared__ double redw[kRowGroups][kRowRB + 1];
  __shared__ double redz[kRowGroups][kRowRB + 1];
  __shared__ double wsum[kRowThreads / 64];
  __shared__ double wrow[kRowRB];
  {  // problem blockIdx.z (B, g0 and mask are shared)
    const int64_t b = blockIdx.z;
    za.Q += b * za.s_q;
    za.V += b * za.s_q;
    za.e2 += b * za.s_vec;
    za.q64 += b * za.s_vec;
    za.P += b * za.s_p;
    za.Pn += b * za.s_pn;
    if (za.Pu) za.Pu += b * za.s_pn;
    za.q32 += b * za.s_q32;
    za.z32 += b * za.s_q32;
    za.idx += b * za.s_io;
    za.obj += b * za.s_io;
    st += b;
  }
  if (st->done || st->skip) return;
  const int t = st->t;
  const int64_t p = st->p;
  const double thr = st->tau * za.g0[p];
  const int64_t m = za.m;
  const int r = GRAM ? 0 : za.r;
  const int rr = threadIdx.x & (kRowRB - 1), g = threadIdx.x / kRowRB;
  const int64_t j0 = (int64_t)blockIdx.x * kRowRB;
  const int64_t j = j0 + rr;
  const int64_t jc = j < m ? j : m - 1;
  // every load of the kernel at once: rows of B and Q (kept raw until the
  // row sums), e2, the norm partials, the coefficient partials
  TB braw[UB];
  double qraw[UQ];
  row_loads(za.Q + jc, za.ldq, g, t, qraw);
  if constexpr (!GRAM) row_loads((const TB *)za.B + jc, za.ldb, g, r, braw);
  const double e2j = za.e2[jc];
  // ||e2||^2 in a fixed order, by every wave (the same in every workgroup)
  double pn = 0.0;
  for (int x = threadIdx.x & 63; x < za.npn; x += 64) pn += za.Pn[x];
  double *ups = sh, *c3 = sh + r;
  if constexpr (SLAB) {
    slab_sums(za.P, za.lp, (int)gridDim.x, r + t, sh, tmp);
  } else {
    for (int c = threadIdx.x; c < r; c += kRowThreads) ups[c] = psum(za.P, za.lp, za.nrb, c);
    for (int s = threadIdx.x; s < t; s += kRowThreads) c3[s] = psum(za.P, za.lp, za.nrb, za.nfix + s);
  }
  if constexpr (GRAM)
    if (threadIdx.x < kRowRB) wrow[threadIdx.x] = psum(za.P, za.lp, za.nrb, jc);
  const double nrm2 = wave_sum(pn);
  __syncthreads();
  // Explicit target: the workgroup that arrives here last knows that all have
  // read the state, so it is the one that will change it; it arrives before
  // its sums, which hide the atomic.  (B = A needs every workgroup's q . w
  // partial, so there the last one to finish does.)
  constexpr int kRec = 64;  // the recording thread: wave 1's first
  uint32_t prev = 0;
  if constexpr (!GRAM)
    if (threadIdx.x == kRec)
      prev = __hip_atomic_fetch_add(&st->cnt[4], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // the basis check: a pick whose exact residual is at most tau * g0_p is
  // dropped (every workgroup takes the same decision from the same sum)
  if (!(isfinite(nrm2) && nrm2 > thr)) {
    const bool rec = GRAM ? blockIdx.x == 0 && threadIdx.x == 0
                          : threadIdx.x == kRec && prev == gridDim.x - 1;
    if (rec) {
      za.mask[p] = 2;
      st->skip = 1;
      st->n_reject += 1;
      st->enorm2 = nrm2;
      if constexpr (!GRAM) st->cnt[4] = 0;
    }
    return;
  }
  const double inv = 1.0 / sqrt(nrm2);
  for (int c = threadIdx.x; c < r; c += kRowThreads) ups[c] *= inv;
  for (int s = threadIdx.x; s < t; s += kRowThreads) c3[s] *= inv;
  __syncthreads();
  // w = B upsilon and Q c3 for this workgroup's rows
  double bpre[UB], qpre[UQ];
  if constexpr (!GRAM) {
    row_convert(braw, g, r, bpre);
    redw[g][rr] = row_sum((const TB *)za.B + jc, za.ldb, g, r, bpre, ups);
  }
  row_convert(qraw, g, t, qpre);
  redz[g][rr] = row_sum(za.Q + jc, za.ldq, g, t, qpre, c3);
  __syncthreads();
  if (threadIdx.x < 64) {
    double qw = 0.0, wj;
    const double qc = row_total(redz);
    if constexpr (GRAM) wj = wrow[rr] * inv;
    else wj = row_total(redw);
    if (threadIdx.x < kRowRB && j < m) {
      const double qv = e2j * inv;
      za.Q[(int64_t)t * za.ldq + j] = qv;
      za.q64[j] = qv;
      za.q32[j] = (float)qv;
      za.V[(int64_t)t * za.ldq + j] = wj;
      za.z32[j] = (float)(wj - qc);
      qw = qv * wj;
    }
    if constexpr (GRAM) {
      const double sq = wave_sum(qw);
      if (threadIdx.x == 0) za.Pu[blockIdx.x] = sq;
    }
  }
  double u2 = 0.0;
  bool rec;
  if constexpr (GRAM) {
    // the last workgroup records the pick: q . w over all workgroups
    // (visible after last_block_arrive)
    if (!last_block_arrive(&st->cnt[4])) return;
    double a = 0.0;
    for (int x = threadIdx.x; x < (int)gridDim.x; x += kRowThreads) a += za.Pu[x];
    u2 = block_sum(a, wsum);
    rec = threadIdx.x == 0;
  } else {
    if (threadIdx.x < kRec || threadIdx.x >= kRec + 64) return;
    double a = 0.0;
    for (int c = threadIdx.x - kRec; c < r; c += 64) a = fma(ups[c], ups[c], a);
    u2 = wave_sum(a);
    rec = threadIdx.x == kRec && prev == gridDim.x - 1;
  }
  if (rec) {
    const double F = st->F - u2;
    st->u2 = u2;
    st->enorm2 = nrm2;
    st->F = F;
    za.obj[t + 1] = F;
    za.idx[t] = p;
    za.mask[p] = 1;
    st->t = t + 1;
    st->dec_pending = 1;
    if (t + 1 >= st->k) st->done = 1;
    st->cnt[4] = 0;
  }
}

// ---------------------------------------------------------------------------
// The whole step of one small problem in one workgroup (blockIdx.x = the
// problem): for Algorithm 4's blocks, whose m, t and r are small, one
// workgroup per block does the six kernels' work with barriers in place of
// kernel boundaries, so a step of all blocks is one launch of nprob
// workgroups instead of six launches of thousands.  Same operations as
// K1-K6 (Gram-Schmidt with one re-orthogonalisation, the basis check,
// upsilon = B^T q, c3 = V^T q, w = B upsilon, z = w - Q c3, the pick's
// record); dot products are wave sums over the rows, row sums run over the
// columns in order, so every result has a fixed summation order.
constexpr int kBlkThreads = 1024;
constexpr int kBlkWaves = kBlkThreads / 64;
constexpr int kBlkMaxM = 2048;  // rows held in LDS

// sum over waves (in order) of one double per wave; every thread gets it
__device__ __forceinline__ double blk_sum(double v, double *wsum) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int x = 0; x < kBlkWaves; ++x) s += wsum[x];
  __syncthreads();
  return s;
}

// out[c] = sum_j M_c[j] x[j] for c < nc (M_c column c, ld ldm, element type
// T): wave w takes four columns at a time (w * 4 + 64 u ..), lanes stride
// the rows, sixteen loads in flight per lane.
template <typename T>
__device__ __forceinline__ void blk_dots(const T *__restrict__ M, int64_t ldm, int nc,
                                         const double *x, int64_t m, double *out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int c0 = wave * 4; c0 < nc; c0 += 4 * kBlkWaves) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t j0 = lane; j0 < m; j0 += 256) {
      double xv[4];
      T v[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t j = j0 + 64 * u;
        xv[u] = j < m ? x[j] : 0.0;
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
          const int c = c0 + cc < nc ? c0 + cc : nc - 1;
          v[cc][u] = M[(int64_t)c * ldm + (j < m ? j : m - 1)];
        }
      }
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[cc] = fma(to_f64(v[cc][u]), xv[u], acc[cc]);
    }
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
      const double a = wave_sum(acc[cc]);
      if (lane == 0 && c0 + cc < nc) out[c0 + cc] = a;
    }
  }
}

// sum over s < ns (in order) of M[j + s ldm] * c[s], sixteen loads in flight
template <typename T>
__device__ __forceinline__ double blk_row(const T *__restrict__ M, int64_t ldm, int ns, int64_t j,
                                          const double *c) {
  double acc = 0.0;
  int s = 0;
  for (; s + 16 <= ns; s += 16) {
    T v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = M[(int64_t)(s + u) * ldm + j];
#pragma unroll
    for (int u = 0; u < 16; ++u) acc = fma(to_f64(v[u]), c[s + u], acc);
  }
  for (; s < ns; ++s) acc = fma(to_f64(M[(int64_t)s * ldm + j]), c[s], acc);
  return acc;
}

template <typename TB>
__global__ __launch_bounds__(kBlkThreads) void k_chain_block(ChainArgs ca) {
  extern __shared__ double lds[];  // vec (m), coefficients (kmax + 1), upsilon (r)
  __shared__ double wsum[kBlkWaves];
  const int64_t b = blockIdx.x;
  DevState *st = ca.st + b;
  if (st->done || st->skip) return;
  const int t = st->t;
  const int64_t p = st->p;
  const int64_t m = ca.m;
  const int r = (int)ca.r;
  const double *Q = ca.Q + b * ca.s_q;
  double *Qw = ca.Q + b * ca.s_q;
  double *V = ca.V + b * ca.s_q;
  const double *a = ca.a + b * ca.s_vec;
  const TB *B = (const TB *)ca.B;
  double *vec = lds, *cf = lds + m, *ups = cf + (ca.kmax + 1);
  for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) vec[j] = a[j];
  __syncthreads();
  // Gram-Schmidt twice: vec <- vec - Q (Q^T vec)
  double nrm2 = 0.0;
  for (int pass = 0; pass < 2; ++pass) {
    blk_dots(Q, ca.ldq, t, vec, m, cf);
    __syncthreads();
    double sq = 0.0;
    for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) {
      const double e = vec[j] - blk_row(Q, ca.ldq, t, j, cf);
      vec[j] = e;
      sq = fma(e, e, sq);
    }
    __syncthreads();
    if (pass == 1) nrm2 = blk_sum(sq, wsum);
  }
  // the basis check (the same rule as the chain's K6)
  const double thr = st->tau * ca.g0[p];
  if (!(isfinite(nrm2) && nrm2 > thr)) {
    if (threadIdx.x == 0) {
      ca.mask[p] = 2;
      st->skip = 1;
      st->n_reject += 1;
      st->enorm2 = nrm2;
    }
    return;
  }
  const double inv = 1.0 / sqrt(nrm2);
  double *q64 = ca.q64 + b * ca.s_vec;
  float *q32 = ca.q32 + b * ca.s_q32;
  for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) {
    const double qv = vec[j] * inv;
    vec[j] = qv;
    Qw[(int64_t)t * ca.ldq + j] = qv;
    q64[j] = qv;
    q32[j] = (float)qv;
  }
  __syncthreads();
  // upsilon = B^T q, c3 = V^T q
  blk_dots(B, ca.ldb, r, vec, m, ups);
  blk_dots((const double *)V, ca.ldq, t, vec, m, cf);
  __syncthreads();
  double a2 = 0.0;
  for (int c = threadIdx.x; c < r; c += kBlkThreads) a2 = fma(ups[c], ups[c], a2);
  const double u2 = blk_sum(a2, wsum);
  // w = B upsilon, z = w - Q c3
  float *z32 = ca.z32 + b * ca.s_q32;
  for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) {
    const double wj = blk_row(B, ca.ldb, r, j, ups);
    const double qc = blk_row(Q, ca.ldq, t, j, cf);
    V[(int64_t)t * ca.ldq + j] = wj;
    z32[j] = (float)(wj - qc);
  }
  if (threadIdx.x == 0) {
    const double F = st->F - u2;
    st->u2 = u2;
    st->enorm2 = nrm2;
    st->F = F;
    ca.obj[b * ca.s_io + t + 1] = F;
    ca.idx[b * ca.s_io + t] = p;
    ca.mask[p] = 1;
    st->t = t + 1;
    st->dec_pending = 1;
    if (t + 1 >= st->k) st->done = 1;
  }
}

// The same for one problem with the history of omega (a small explicit target):
// the pick from the pass's winners, the column decoded here, c1 gathered.  One
// launch instead of the slab form's three, each of which spends most of its
// 5-8 us on its start, its first loads and its end.
template <typename TB>
__global__ __launch_bounds__(kBlkThreads) void k_chain_one(ChainArgs ca, AView A) {
  extern __shared__ double lds[];  // vec (m), coefficients (kmax + 1), upsilon (r)
  __shared__ double wsum[kBlkWaves];
  __shared__ double bs[kBlkWaves];
  __shared__ int64_t bi[kBlkWaves];
  DevState *st = ca.st;
  if (st->done) {
    if (threadIdx.x == 0) st->dec_pending = 0;  // the pass after the last pick has run
    return;
  }
  const int t = st->t;
  const int64_t m = ca.m;
  const int r = (int)ca.r;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double *Q = ca.Q;
  const TB *B = (const TB *)ca.B;
  double *vec = lds, *cf = lds + m, *ups = cf + (ca.kmax + 1);
  double best = -INFINITY;
  int64_t p = kNoIdx;
  for (int x = threadIdx.x; x < ca.npart; x += kBlkThreads) {
    const double sc = ca.part[x].score;
    const int64_t i = ca.part[x].idx;
    if (better(sc, i, best, p)) {
      best = sc;
      p = i;
    }
  }
  const int nw = ca.npart < kBlkThreads ? (ca.npart + 63) >> 6 : kBlkWaves;
  if (wave < nw) {
    wave_argmax(best, p);
    if (lane == 0) {
      bs[wave] = best;
      bi[wave] = p;
    }
  }
  __syncthreads();
  best = bs[0];
  p = bi[0];
  for (int x = 1; x < nw; ++x)
    if (better(bs[x], bi[x], best, p)) {
      best = bs[x];
      p = bi[x];
    }
  // (every thread has read the state)
  if (threadIdx.x == 0) {
    st->skip = 0;
    st->dec_pending = 0;
    st->p = p == kNoIdx ? -1 : p;
    if (p == kNoIdx) st->exhausted = st->done = 1;
  }
  if (p == kNoIdx) return;
  const double ps = col_scale(A, p);
  for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) vec[j] = ps * (double)load_elem(A, p, j);
  for (int s = threadIdx.x; s < t; s += kBlkThreads) cf[s] = (double)ca.wh[(int64_t)s * ca.ldw + p];
  __syncthreads();
  // vec <- vec - Q c1, then once more with c2 = Q^T vec
  double nrm2 = 0.0;
  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 1) {
      blk_dots(Q, ca.ldq, t, vec, m, cf);
      __syncthreads();
    }
    double sq = 0.0;
    for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) {
      const double e = vec[j] - blk_row(Q, ca.ldq, t, j, cf);
      vec[j] = e;
      sq = fma(e, e, sq);
    }
    __syncthreads();
    if (pass == 1) nrm2 = blk_sum(sq, wsum);
  }
  const double thr = st->tau * ca.g0[p];
  if (!(isfinite(nrm2) && nrm2 > thr)) {
    if (threadIdx.x == 0) {
      ca.mask[p] = 2;
      st->skip = 1;
      st->n_reject += 1;
      st->enorm2 = nrm2;
    }
    return;
  }
  const double inv = 1.0 / sqrt(nrm2);
  for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) {
    const double qv = vec[j] * inv;
    vec[j] = qv;
    ca.Q[(int64_t)t * ca.ldq + j] = qv;
    ca.q64[j] = qv;
    ca.q32[j] = (float)qv;
  }
  __syncthreads();
  blk_dots(B, ca.ldb, r, vec, m, ups);
  blk_dots((const double *)ca.V, ca.ldq, t, vec, m, cf);
  __syncthreads();
  for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) {
    const double wj = blk_row(B, ca.ldb, r, j, ups);
    const double qc = blk_row(Q, ca.ldq, t, j, cf);
    ca.V[(int64_t)t * ca.ldq + j] = wj;
    ca.z32[j] = (float)(wj - qc);
  }
  if (wave == kBlkWaves - 1) {
    double a2 = 0.0;
    for (int c = lane; c < r; c += 64) a2 = fma(ups[c], ups[c], a2);
    const double u2 = wave_sum(a2);
    if (lane == 0) {
      const double F = st->F - u2;
      st->u2 = u2;
      st->enorm2 = nrm2;
      st->F = F;
      ca.obj[t + 1] = F;
      ca.idx[t] = p;
      ca.mask[p] = 1;
      st->t = t + 1;
      st->dec_pending = 1;
      if (t + 1 >= st->k) st->done = 1;
    }
  }
}

// Gram-Schmidt of a small subset of A's columns, pick[0..k), in one workgroup:
// each column twice against the t kept before it, kept where its residual's
// squared norm is above tau of its own (norm2) as in the general kernels, which
// take four launches a column (18 us).  One CU reads Q's t columns four times
// for the next, so this serves m k <= 48 K: with the attempt at all columns at
// once before it, general kernels -> this: m 333, k 10 340 -> 228 us; 1024, 32
// about 740 -> 600; 700, 64 1365 -> 1240; but 1024, 64 1390 -> 1500 and 2048,
// 64 1550 -> 2490.  Columns t..k of Q are zero at the end.
__global__ __launch_bounds__(kBlkThreads) void k_gs_subset(AView A, const int64_t *__restrict__ pick,
                                                           int k, const double *__restrict__ norm2,
                                                           double tau, double *Q, int64_t ldq,
                                                           DevState *st) {
  extern __shared__ double lds[];  // vec (m), coefficients (k)
  __shared__ double wsum[kBlkWaves];
  const int64_t m = A.m;
  double *vec = lds, *cf = lds + m;
  int t = 0;
  for (int x = 0; x < k; ++x) {
    const int64_t p = pick[x];
    const double ps = col_scale(A, p);
    for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) vec[j] = ps * (double)load_elem(A, p, j);
    __syncthreads();
    double nrm2 = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
      blk_dots((const double *)Q, ldq, t, vec, m, cf);
      __syncthreads();
      double sq = 0.0;
      for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) {
        const double e = vec[j] - blk_row((const double *)Q, ldq, t, j, cf);
        vec[j] = e;
        sq = fma(e, e, sq);
      }
      __syncthreads();
      if (pass == 1) nrm2 = blk_sum(sq, wsum);
    }
    if (isfinite(nrm2) && nrm2 > tau * norm2[p]) {  // (the same in every thread)
      const double inv = 1.0 / sqrt(nrm2);
      for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) Q[(int64_t)t * ldq + j] = vec[j] * inv;
      ++t;
    }
    __syncthreads();  // the new column, for every wave's next dots
  }
  for (int x = t; x < k; ++x)
    for (int64_t j = threadIdx.x; j < m; j += kBlkThreads) Q[(int64_t)x * ldq + j] = 0.0;
  if (threadIdx.x == 0) {
    st->t = t;
    st->pos = k;
  }
}

bool gs_subset_fits(int64_t m, int k) { return m <= kBlkMaxM && k <= 256 && m * k <= 48 * 1024; }

hipError_t launch_gs_subset(const AView &A, const int64_t *pick, int k, const double *norm2,
                            double tau, double *Q, int64_t ldq, DevState *st, hipStream_t s) {
  hipLaunchKernelGGL(k_gs_subset, dim3(1), dim3(kBlkThreads), (size_t)(A.m + k) * sizeof(double), s, A,
                     pick, k, norm2, tau, Q, ldq, st);
  return hipGetLastError();
}

size_t chain_block_lds_bytes(int64_t m, int64_t r, int kmax) {
  return (size_t)(m + kmax + 1 + r) * sizeof(double);
}

bool chain_block_fits(int64_t m, int64_t r, int kmax, size_t lds_max) {
  return m <= kBlkMaxM && chain_block_lds_bytes(m, r, kmax) <= lds_max;
}

hipError_t launch_chain_block(const ChainArgs &ca, hipStream_t s) {
  const size_t lds = chain_block_lds_bytes(ca.m, ca.r, ca.kmax);
  const unsigned np = (unsigned)(ca.nprob > 0 ? ca.nprob : 1);
  if (ca.b_bf16)
    hipLaunchKernelGGL((k_chain_block<uint16_t>), dim3(np), dim3(kBlkThreads), lds, s, ca);
  else
    hipLaunchKernelGGL((k_chain_block<float>), dim3(np), dim3(kBlkThreads), lds, s, ca);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
int chain_row_blocks(int64_t m) { return (int)((m + kDotRows - 1) / kDotRows); }
int chain_row_groups(int64_t m) { return (int)((m + kRowRB - 1) / kRowRB); }

size_t chain_lds_bytes(int64_t r, int kmax) { return (size_t)(r + kmax + 1) * sizeof(double); }

bool chain_fits(int64_t m, int64_t r, int kmax, size_t lds_max) {
  return chain_row_blocks(m) <= kMaxRB && chain_lds_bytes(r, kmax) <= lds_max;
}

// The slab form holds one round of a thread's columns (t, r <= 32 kRowUMax), and
// every workgroup of a consumer reads all partials: m / 32 rows of t (S2) and
// of r + t (K6).  At 94 x 264 doubles (198 KB; m = 3001) S2 and K6 take 7.8 and
// 10.2 us against 4.4 + 4.6 + 4.4 + 10.2 us for K3, K4, K5 and K6; each further
// 100 KB costs them about 1 us, so the line lies near 400 KB.
constexpr int64_t kSlabBytes = 384 * 1024;
bool chain_slab_fits(int64_t m, int64_t r, int kmax) {
  return kmax <= kRowGroups * kRowUMax && r <= kRowGroups * kRowUMax &&
         (int64_t)chain_row_groups(m) * (r + kmax) * (int64_t)sizeof(double) <= kSlabBytes;
}

// One workgroup does the step of a small explicit target.  Its own work grows
// with m (r + 4 k), on one CU; the slab form's three launches cost about the same
// at any such size.  Per step with the pass, n = 5 000, slab form -> this: m 120,
// r 20, k 25: 27.7 -> 24.1 us; 333, 50, 25: 28.9 -> 26.4; 500, 20, 25: 29.8 ->
// 26.2; even at 512, 128, 25 (31.1 -> 31.5), and behind at k 60 (333, 50: 27.7 ->
// 29.4) and at 512, 128, 64 (29.5 -> 35.2).
static bool chain_one_fits(int64_t m, int64_t r, int kmax, bool gram) {
  return !gram && m <= 512 && r <= 64 && kmax <= 32;
}

// f(U) with U the smallest of 4, 8, 16 that holds n columns in one round
template <typename F>
static void with_row_u(int64_t n, F f) {
  if (n <= 4 * kRowGroups) f(std::integral_constant<int, 4>{});
  else if (n <= 8 * kRowGroups) f(std::integral_constant<int, 8>{});
  else f(std::integral_constant<int, kRowUMax>{});
}

hipError_t launch_chain(const ChainArgs &ca, hipStream_t s) {
  const int64_t m = ca.m;
  const int nrb = chain_row_blocks(m), nrg = chain_row_groups(m);
  if (nrb > kMaxRB) return hipErrorInvalidValue;
  const unsigned qdots = (unsigned)dots_col_blocks(0, ca.kmax);
  const size_t lds_t = (size_t)(ca.kmax + 1) * sizeof(double);
  const unsigned np = (unsigned)(ca.nprob > 0 ? ca.nprob : 1);
  if (ca.wh && chain_one_fits(m, ca.r, ca.kmax, ca.gram)) {
    const size_t lds = chain_block_lds_bytes(m, ca.r, ca.kmax);
    if (ca.b_bf16)
      hipLaunchKernelGGL((k_chain_one<uint16_t>), dim3(1), dim3(kBlkThreads), lds, s, ca, *ca.A);
    else
      hipLaunchKernelGGL((k_chain_one<float>), dim3(1), dim3(kBlkThreads), lds, s, ca, *ca.A);
    return hipGetLastError();
  }
  const dim3 gr(nrg, 1, np), br(kRowThreads);
  const bool bf = ca.b_bf16 && !ca.gram;
  // the slab form takes one problem with the history of omega; B = A keeps K5
  const bool slab = ca.wh && chain_slab_fits(m, ca.gram ? 0 : ca.r, ca.kmax);
  auto q_dots = [&](const double *x) {  // K1, K3: partials of Q^T x
    hipLaunchKernelGGL((k_dots<float>), dim3(qdots, nrb, np), dim3(256), 0, s,
                       (const float *)nullptr, (int64_t)0, 0, ca.Q, ca.ldq, x, m, ca.P, ca.lp,
                       ca.st, ca.s_q, ca.s_vec, ca.s_p);
  };
  with_row_u(ca.kmax, [&](auto uq) {
    constexpr int UQ = decltype(uq)::value;
    if (slab) {
      hipLaunchKernelGGL((k_gs1<true, UQ>), gr, br, lds_t, s, *ca.A, ca.wh, ca.ldw, ca.part,
                         ca.npart, ca.Q, ca.ldq, ca.e1, ca.P1, ca.lp1, m, ca.st);
      if (ca.gram)
        hipLaunchKernelGGL((k_gs2<float, true, UQ, 4>), gr, br, lds_t, s, ca.Q, ca.ldq, ca.V,
                           (const float *)nullptr, (int64_t)0, 0, ca.e1, ca.P1, ca.lp1, ca.e2,
                           ca.Pn, (double *)nullptr, (int64_t)0, m, ca.st);
      else
        with_row_u(ca.r, [&](auto ub) {
          constexpr int UB = decltype(ub)::value;
          if (bf)
            hipLaunchKernelGGL((k_gs2<uint16_t, false, UQ, UB>), gr, br, lds_t, s, ca.Q, ca.ldq,
                               ca.V, (const uint16_t *)ca.B, ca.ldb, (int)ca.r, ca.e1, ca.P1,
                               ca.lp1, ca.e2, ca.Pn, ca.P2, ca.lp, m, ca.st);
          else
            hipLaunchKernelGGL((k_gs2<float, false, UQ, UB>), gr, br, lds_t, s, ca.Q, ca.ldq, ca.V,
                               (const float *)ca.B, ca.ldb, (int)ca.r, ca.e1, ca.P1, ca.lp1, ca.e2,
                               ca.Pn, ca.P2, ca.lp, m, ca.st);
        });
      return;
    }
    if (ca.wh) {
      // S1 without partials: e1 = a - Q c1
      hipLaunchKernelGGL((k_gs1<false, UQ>), gr, br, lds_t, s, *ca.A, ca.wh, ca.ldw, ca.part,
                         ca.npart, ca.Q, ca.ldq, ca.e1, (double *)nullptr, (int64_t)0, m, ca.st);
    } else {
      q_dots(ca.a);  // K1: c1 partials
      // K2: e1 = a - Q c1
      hipLaunchKernelGGL((k_rows_sub<false, UQ>), gr, br, lds_t, s, ca.Q, ca.ldq, ca.a, ca.P, ca.lp,
                         nrb, ca.e1, (double *)nullptr, m, ca.st, ca.s_q, ca.s_vec, ca.s_p, ca.s_pn);
    }
    q_dots(ca.e1);  // K3: c2 partials
    // K4: e2 = e1 - Q c2, norm partials
    hipLaunchKernelGGL((k_rows_sub<true, UQ>), gr, br, lds_t, s, ca.Q, ca.ldq, ca.e1, ca.P, ca.lp,
                       nrb, ca.e2, ca.Pn, m, ca.st, ca.s_q, ca.s_vec, ca.s_p, ca.s_pn);
  });
  // K5: [B^T e2 ; V^T e2] partials (B = A: [C e2 ; V^T e2]); S2 formed them otherwise
  const int nfix = ca.gram ? (int)m : (int)ca.r;
  const bool zslab = slab && !ca.gram;
  if (!zslab) {
    const dim3 gd((unsigned)dots_col_blocks(nfix, ca.kmax), nrb, np);
    if (bf)
      hipLaunchKernelGGL((k_dots<uint16_t>), gd, dim3(256), 0, s, (const uint16_t *)ca.B, ca.ldb,
                         nfix, ca.V, ca.ldq, ca.e2, m, ca.P, ca.lp, ca.st, ca.s_q, ca.s_vec, ca.s_p);
    else
      hipLaunchKernelGGL((k_dots<float>), gd, dim3(256), 0, s, (const float *)ca.B, ca.ldb, nfix,
                         ca.V, ca.ldq, ca.e2, m, ca.P, ca.lp, ca.st, ca.s_q, ca.s_vec, ca.s_p);
  }
  // K6
  ZArgs za{};
  za.Q = ca.Q;
  za.ldq = ca.ldq;
  za.V = ca.V;
  za.e2 = ca.e2;
  za.P = zslab ? ca.P2 : ca.P;
  za.lp = ca.lp;
  za.nrb = nrb;
  za.Pn = ca.Pn;
  za.npn = nrg;
  za.Pu = ca.Pu;
  za.B = ca.B;
  za.ldb = ca.ldb;
  za.r = ca.gram ? 0 : (int)ca.r;
  za.nfix = nfix;
  za.q64 = ca.q64;
  za.q32 = ca.q32;
  za.z32 = ca.z32;
  za.g0 = ca.g0;
  za.mask = ca.mask;
  za.idx = ca.idx;
  za.obj = ca.obj;
  za.m = m;
  za.s_q = ca.s_q;
  za.s_vec = ca.s_vec;
  za.s_p = ca.s_p;
  za.s_pn = ca.s_pn;
  za.s_q32 = ca.s_q32;
  za.s_io = ca.s_io;
  const size_t lds_z = (size_t)(za.r + ca.kmax + 1) * sizeof(double);
  with_row_u(ca.kmax, [&](auto uq) {
    constexpr int UQ = decltype(uq)::value;
    if (ca.gram) {
      hipLaunchKernelGGL((k_rows_z<float, true, false, UQ, 4>), gr, br, lds_z, s, za, ca.st);
      return;
    }
    with_row_u(ca.r, [&](auto ub) {
      constexpr int UB = decltype(ub)::value;
      if (bf && slab)
        hipLaunchKernelGGL((k_rows_z<uint16_t, false, true, UQ, UB>), gr, br, lds_z, s, za, ca.st);
      else if (bf)
        hipLaunchKernelGGL((k_rows_z<uint16_t, false, false, UQ, UB>), gr, br, lds_z, s, za, ca.st);
      else if (slab)
        hipLaunchKernelGGL((k_rows_z<float, false, true, UQ, UB>), gr, br, lds_z, s, za, ca.st);
      else
        hipLaunchKernelGGL((k_rows_z<float, false, false, UQ, UB>), gr, br, lds_z, s, za, ca.st);
    });
  });
  return hipGetLastError();
}

}  // namespace gcss
