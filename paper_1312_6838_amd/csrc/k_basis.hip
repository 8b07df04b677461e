// Orthonormal FP64 basis of k given columns of A, all at once.
//
// A selection builds its basis one column at a time because each pick waits
// for the scores before it; the columns of a caller's subset are all known,
// so their basis needs no serial Gram-Schmidt (four launches and two
// reductions per column).  A subset of 100 columns at m = 1024 takes 0.19 ms
// with the error, against 2.06 ms column by column (MI355X).  Cholesky QR, in
// chunks of kBC columns:
//
//   S  = the chunk's columns, decoded                       (m x kBC)
//   S -= Q (Q^T S)              Q: the chunks before (none in the first)
//   R^T R = S^T S,  T = R^-1,  Y = S T                      (one workgroup: R, T)
//   Y -= Q (Q^T Y)
//   Q_chunk = Y (3/2 I - 1/2 Y^T Y)       one Newton step to orthonormality
//
// Rounding leaves Y^T Y = I + E with E about eps cond(S)^2; the Newton step
// takes the deviation to 3/8 E^2.  The result is used only where it is
// certified: every pivot above kPivotRel of its column's squared norm in A,
// every |E_ij| <= kDevMax (so ||E||^2 <= 2e-16 for 128 columns), Q^T Y as small.
// Where only the last two fail, but within kDevRefine (correlated columns, cond
// 1e3 .. 1e5: about 190 of 2100 us for 100 columns would be lost), the two steps
// on Y are done once more with Q's chunks as Y, certified by kDevRefined.
// Otherwise (dependent or nearly dependent columns) the flag says so, and the
// caller runs Gram-Schmidt, whose rule for dropping columns decides.  (The
// norm is that of the column as stored, as in that rule: what a chunk's S
// still holds of a column that depends on earlier chunks is rounding, or an
// exact remnant far below the rule's 1e-13, and against its own norm it would
// always pass.)
//
// All products are FP64 on the matrix cores (v_mfma_f64_16x16x4: lane l gives
// row l % 16 of the left and column l % 16 of the right operand at k = l / 16,
// register v of the result holds row l / 16 + 4 v, column l % 16), in 64 x 64
// tiles of four waves; sums over row splits have a fixed order.
#include "gcss_device.h"

namespace gcss {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kBC = 128;  // columns per chunk
constexpr int kBT = 64;   // tile edge
constexpr int kBK = 32;   // contraction chunk staged in LDS
constexpr double kPivotRel = 1e-8;
constexpr double kDevMax = 1e-10;
// a deviation of kDevRefine becomes 3/8 128 kDevRefine^2 = 1.2e-9 at most, which
// the second Newton step takes to 3/8 128 (1.5e-9)^2 = 1e-16
constexpr double kDevRefine = 5e-6;
constexpr double kDevRefined = 1.5e-9;

// v (a deviation) above `most` spoils the basis, above `ok` it wants refining
// (by whole waves: one atomic for each).
__device__ __forceinline__ void bs_check(double v, double ok, double most, int *flag) {
  const bool bad = !(fabs(v) <= most), fine = fabs(v) <= ok;
  const int code = (__ballot(bad) ? kBasisBad : 0) | (__ballot(!bad && !fine) ? kBasisRefine : 0);
  if (code && (threadIdx.x & 63) == 0) atomicOr(flag, code);
}

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// S[:, c] = column pick[c] of A (c < b; zero columns up to kBC), rows m..ldq zero.
__global__ __launch_bounds__(256) void k_bs_gather(AView A, const int64_t *__restrict__ pick, int b,
                                                   double *__restrict__ S, int64_t ldq,
                                                   int *__restrict__ flag) {
  const int c = blockIdx.y;
  if (flag && blockIdx.x == 0 && c == 0 && threadIdx.x == 0) *flag = 0;
  const int64_t p = c < b ? pick[c] : -1;
  const double sc = c < b ? col_scale(A, p) : 0.0;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < ldq) S[(int64_t)c * ldq + j] = c < b && j < A.m ? sc * (double)load_elem(A, p, j) : 0.0;
}

// Y = chunk of b columns of Q, rows m..ldq and columns b.. zero
__global__ __launch_bounds__(256) void k_bs_take(const double *__restrict__ Q, int64_t m, int b,
                                                 double *__restrict__ Y, int64_t ldq,
                                                 int *__restrict__ flag) {
  const int c = blockIdx.y;
  if (flag && blockIdx.x == 0 && c == 0 && threadIdx.x == 0) *flag = 0;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < ldq) Y[(int64_t)c * ldq + j] = c < b && j < m ? Q[(int64_t)c * ldq + j] : 0.0;
}

// Part[z][x][y] = X^T Y over the rows of split z for the 64 x 64 tile of
// columns 64 x.. of X (nx of them) and 64 y.. of Y.  Rows at or past m count
// as zero (Q's pads hold anything).  Grid (x tiles, y tiles, splits).
__global__ __launch_bounds__(256) void k_bs_tn(const double *__restrict__ X, int nx,
                                               const double *__restrict__ Y, int64_t ldq, int64_t m,
                                               int64_t rows, double *__restrict__ part) {
  constexpr int P = kBK + 2;  // LDS pitch (doubles): 16-byte reads of two k, 16 columns apart
  __shared__ __align__(16) double xs[kBT * P];
  __shared__ __align__(16) double ys[kBT * P];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.z * rows;
  const int64_t r1 = r0 + rows < m ? r0 + rows : m;
  const int x0 = blockIdx.x * kBT, y0 = blockIdx.y * kBT;
  // loader: 16 lanes x 2 rows per column, 16 columns at a time
  const int lr = 2 * (threadIdx.x & 15), lc = threadIdx.x >> 4;
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32, i16 = lane & 15, kg = lane >> 4;
  f64x4 acc[2][2] = {};
  for (int64_t rb = r0; rb < r1; rb += kBK) {
    double2 xv[4], yv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = lc + 16 * u;
      xv[u] = *(const double2 *)(X + (int64_t)(x0 + c < nx ? x0 + c : nx - 1) * ldq + rb + lr);
      yv[u] = *(const double2 *)(Y + (int64_t)(y0 + c) * ldq + rb + lr);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = lc + 16 * u;
      const bool a = rb + lr < r1, b = rb + lr + 1 < r1, ok = x0 + c < nx;
      *(double2 *)(xs + c * P + lr) = make_double2(a && ok ? xv[u].x : 0.0, b && ok ? xv[u].y : 0.0);
      *(double2 *)(ys + c * P + lr) = make_double2(a ? yv[u].x : 0.0, b ? yv[u].y : 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kBK / 8; ++s) {
      double2 xa[2], yb[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        xa[h] = *(const double2 *)(xs + (wi + 16 * h + i16) * P + 8 * s + 2 * kg);
        yb[h] = *(const double2 *)(ys + (wj + 16 * h + i16) * P + 8 * s + 2 * kg);
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          acc[a][b] = mfma64(xa[a].x, yb[b].x, acc[a][b]);
          acc[a][b] = mfma64(xa[a].y, yb[b].y, acc[a][b]);
        }
    }
    __syncthreads();
  }
  double *o = part + (((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * gridDim.y + blockIdx.y) * kBT * kBT;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        o[(wi + 16 * a + kg + 4 * v) * kBT + wj + 16 * b + i16] = acc[a][b][v];
}

// W (row-major, 64 ntx x kBC) = the sum over splits of the partial tiles.
// mode 0: W as it is; 1: W must be small (a second projection's
// coefficients); 2: W = 3/2 I - 1/2 sum, the sum being near I for the first b
// columns.  Modes 1 and 2 check the deviation.  Grid (elements / 256).
__global__ __launch_bounds__(256) void k_bs_reduce(const double *__restrict__ part, int ntx,
                                                   int nsplit, int mode, int b, double ok,
                                                   double most, double *__restrict__ W,
                                                   int *__restrict__ flag) {
  constexpr int nty = kBC / kBT;
  const int e = blockIdx.x * 256 + threadIdx.x;  // row-major element of W
  const int i = e / kBC, j = e % kBC;
  if (i >= ntx * kBT) return;
  const double *src = part + ((int64_t)(i / kBT) * nty + j / kBT) * kBT * kBT + (i % kBT) * kBT + j % kBT;
  const int64_t step = (int64_t)ntx * nty * kBT * kBT;
  double s = 0.0;
  for (int z0 = 0; z0 < nsplit; z0 += 8) {
    double v[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) v[z] = src[(z0 + z < nsplit ? z0 + z : nsplit - 1) * step];
#pragma unroll
    for (int z = 0; z < 8; ++z)
      if (z0 + z < nsplit) s += v[z];
  }
  if (mode == 2) {
    const double id = i == j ? 1.0 : 0.0;
    bs_check(i < b && j < b ? s - id : 0.0, ok, most, flag);
    W[e] = 1.5 * id - 0.5 * s;
  } else {
    if (mode == 1) bs_check(s, ok, most, flag);
    W[e] = s;
  }
}

// out = X W, or in - X W, for the 32 x 64 tile of rows 32 x.. and columns 64
// y..: X has kx columns, W is row-major with kBC columns.  Only columns < b and
// rows < m are written.  st: the state of a finished basis of k columns (last
// chunk; none of it where the flag is set, so that a pass over A for its error
// has nothing to do).  A FP64 matrix instruction takes 64 cycles of a SIMD, so the tile is
// kept low (twice the workgroups), and the next chunk's loads are in flight
// while this one is multiplied: 12.0 -> 7.5 us at m = 1024.
constexpr int kBR = 32;
__global__ __launch_bounds__(256) void k_bs_nn(const double *__restrict__ X, int kx,
                                               const double *__restrict__ W,
                                               const double *__restrict__ in, double *out,
                                               int64_t ldq, int64_t m, int b, DevState *st, int k,
                                               const int *__restrict__ flag) {
  constexpr int PX = kBR + 16, PW = kBT + 16;  // LDS pitches: four rows of 16 doubles, conflict-free
  __shared__ double xs[kBK * PX];  // [k][row]
  __shared__ double ws[kBK * PW];  // [k][column]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j0 = (int64_t)blockIdx.x * kBR;
  const int c0 = blockIdx.y * kBT;
  const int wi = (wave >> 1) * 16, wj = (wave & 1) * 32, i16 = lane & 15, kg = lane >> 4;
  const int xr = 2 * (threadIdx.x & 15), xk = threadIdx.x >> 4;  // loader of X: 32 rows x 16 at a time
  const int lr = 2 * (threadIdx.x & 31), lk = threadIdx.x >> 5;  // of W: 64 columns x 8 at a time
  f64x4 acc[2] = {};
  double2 xv[2], wv[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kk = k0 + xk + 16 * u;
      xv[u] = *(const double2 *)(X + (int64_t)(kk < kx ? kk : kx - 1) * ldq + j0 + xr);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int kk = k0 + lk + 8 * u;
      wv[u] = *(const double2 *)(W + (int64_t)(kk < kx ? kk : kx - 1) * kBC + c0 + lr);
    }
  };
  load(0);
  for (int k0 = 0; k0 < kx; k0 += kBK) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kk = xk + 16 * u;
      const bool ok = k0 + kk < kx;
      xs[kk * PX + xr] = ok && j0 + xr < m ? xv[u].x : 0.0;
      xs[kk * PX + xr + 1] = ok && j0 + xr + 1 < m ? xv[u].y : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int kk = lk + 8 * u;
      const bool ok = k0 + kk < kx;
      ws[kk * PW + lr] = ok ? wv[u].x : 0.0;
      ws[kk * PW + lr + 1] = ok ? wv[u].y : 0.0;
    }
    __syncthreads();
    if (k0 + kBK < kx) load(k0 + kBK);
#pragma unroll
    for (int s = 0; s < kBK / 4; ++s) {
      const double xa = xs[(4 * s + kg) * PX + wi + i16];
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[c] = mfma64(xa, ws[(4 * s + kg) * PW + wj + 16 * c + i16], acc[c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      // (register v holds row kg + 4 v of the tile, column i16)
      const int64_t j = j0 + wi + kg + 4 * v;
      const int col = c0 + wj + 16 * c + i16;
      if (j < m && col < b) {
        const int64_t o = (int64_t)col * ldq + j;
        out[o] = in ? in[o] - acc[c][v] : acc[c][v];
      }
    }
  if (st && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    st->t = *flag ? 0 : k;
    st->pos = k;
  }
}

// T = R^-1 (row-major kBC x kBC, upper; identity past b) with R^T R = the Gram
// matrix, by one workgroup with the matrix in LDS: L = R^T by
// panels of 16 (one wave factors and inverts the 16 x 16 diagonal block, the
// rows below are multiplied by that inverse, the trailing matrix is updated
// on the matrix cores), then L^-1 from the blocks' inverses by doubling
// (X21 = -X22 L21 X11 for 16, 32, 64).  A column-at-a-time factorisation
// would take two barriers and a root per column.  Panels and levels past b are
// left out (the identity stays): a subset that is handed to Gram-Schmidt has
// spent this for nothing.
constexpr int kCP = kBC + 2;  // LDS pitch
constexpr int kCThreads = 1024;

// tile (16 x 16) of C = sum over kk < K of A[i][k] B[k][j], A row-major at a
// (pitch kCP), B at b: BT ? B[k][j] = b[j][k] : b[k][j]
template <bool BT>
__device__ __forceinline__ f64x4 lds_mm(const double *a, const double *b, int K, f64x4 acc, double s) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kg = lane >> 4;
  for (int k = kg; k < K; k += 4)
    acc = mfma64(s * a[i16 * kCP + k], BT ? b[i16 * kCP + k] : b[k * kCP + i16], acc);
  return acc;
}
__device__ __forceinline__ f64x4 tile_load(const double *o) {
  const int lane = threadIdx.x & 63;
  f64x4 v;
#pragma unroll
  for (int x = 0; x < 4; ++x) v[x] = o[((lane >> 4) + 4 * x) * kCP + (lane & 15)];
  return v;
}
__device__ __forceinline__ void tile_store(double *o, const f64x4 &v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int x = 0; x < 4; ++x) o[((lane >> 4) + 4 * x) * kCP + (lane & 15)] = v[x];
}

// v of lane x (a constant), in scalar registers: shuffles (an LDS round trip
// per broadcast), FP64 roots and divisions made the kernel 175 us, now 63 us
__device__ __forceinline__ double lane_value(double v, int x) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), x),
                          __builtin_amdgcn_readlane(__double2loint(v), x));
}

__global__ __launch_bounds__(kCThreads) void k_bs_chol(const double *__restrict__ gram, int b,
                                                       const int64_t *__restrict__ pick,
                                                       const double *__restrict__ norm2,
                                                       double *__restrict__ T,
                                                       int *__restrict__ flag) {
  __shared__ double G[kBC * kCP];
  __shared__ double D[kBC * 16];  // inverses of the diagonal blocks, row-major 16 x 16 each
  __shared__ double g0[kBC];  // the columns' squared norms in A
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the Gram matrix, identity past b (gram and T may be one buffer)
#pragma unroll
  for (int u = 0; u < kBC * kBC / kCThreads; ++u) {
    const int e = threadIdx.x + u * kCThreads, i = e / kBC, j = e % kBC;
    double s = gram[e];
    if (i >= b || j >= b) s = i == j ? 1.0 : 0.0;
    G[i * kCP + j] = s;
  }
  if (threadIdx.x < kBC) g0[threadIdx.x] = (int)threadIdx.x < b ? norm2[pick[threadIdx.x]] : 1.0;
  __syncthreads();
  bool bad = false;
  int nb = 16;  // what of the matrix is worked on: 16, 32, 64 or 128
  while (nb < b) nb *= 2;
  for (int p = 0; p < nb; p += 16) {
    double *const d = D + p * 16;
    if (wave == 0) {
      // L of the diagonal block: lane i (of the first 16) holds row i
      const int i = lane & 15;
      double a[16], ri[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) a[c] = G[(p + i) * kCP + p + c];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const double piv = lane_value(a[c], c);
        const bool ok = piv > kPivotRel * g0[p + c];
        bad |= !ok;
        // piv^-1/2: two Newton steps on the hardware's estimate
        double r = __builtin_amdgcn_rsq(ok ? piv : 1.0);
        r = fma(0.5 * r, fma(-piv * r, r, 1.0), r);
        r = fma(0.5 * r, fma(-piv * r, r, 1.0), r);
        ri[c] = ok ? r : 0.0;
        a[c] *= ri[c];  // L[i][c] (rows above c hold the other triangle, unused)
#pragma unroll
        for (int x = c + 1; x < 16; ++x) a[x] = fma(-a[c], lane_value(a[c], x), a[x]);
      }
      // its inverse: lane i forms column i of L^-1 by forward substitution
      double v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        double s = r == i ? 1.0 : 0.0;
#pragma unroll
        for (int c = 0; c < r; ++c) s = fma(-lane_value(a[c], r), v[c], s);
        v[r] = s * ri[r];
      }
      if (lane < 16) {
#pragma unroll
        for (int r = 0; r < 16; ++r) d[r * 16 + i] = v[r];
      }
    }
    __syncthreads();
    // rows below: L21 = A21 L11^-T, one thread per (row, column), held until
    // every thread has read A21
    const int below = nb - p - 16;
    double lv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = threadIdx.x + u * kCThreads, i = e >> 4, c = e & 15;
      lv[u] = 0.0;
      if (i < below) {
        const double *row = G + (p + 16 + i) * kCP + p;
        double s = 0.0;
#pragma unroll
        for (int x = 0; x < 16; ++x) s = fma(row[x], d[c * 16 + x], s);
        lv[u] = s;
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = threadIdx.x + u * kCThreads, i = e >> 4, c = e & 15;
      if (i < below) G[(p + 16 + i) * kCP + p + c] = lv[u];
    }
    __syncthreads();
    // trailing update of the lower tiles: A22 -= L21 L21^T
    const int nt = below / 16;
    for (int t = wave; t < nt * (nt + 1) / 2; t += kCThreads / 64) {
      int ti = 0, rem = t;
      while (rem > ti) {
        rem -= ti + 1;
        ++ti;
      }
      const int tj = rem;
      double *o = G + (p + 16 + 16 * ti) * kCP + p + 16 + 16 * tj;
      const double *li = G + (p + 16 + 16 * ti) * kCP + p, *lj = G + (p + 16 + 16 * tj) * kCP + p;
      tile_store(o, lds_mm<true>(li, lj, 16, tile_load(o), -1.0));
    }
    __syncthreads();
  }
  if (wave == 0 && lane < 16 && bad) atomicOr(flag, kBasisBad);
  // the diagonal blocks' inverses into place (zero above their diagonals)
  for (int e = threadIdx.x; e < nb * 16; e += kCThreads) {
    const int p = e / 256 * 16, i = (e >> 4) & 15, c = e & 15;
    G[(p + i) * kCP + p + c] = c <= i ? D[e] : 0.0;
  }
  __syncthreads();
  // doubling: within blocks of 2s, X21 = -X22 (L21 X11); the product L21 X11
  // is kept in the block's upper right corner
  for (int s = 16; s < nb; s *= 2) {
    const int tp = (s / 16) * (s / 16), pairs = nb / (2 * s);
    for (int t = wave; t < pairs * tp; t += kCThreads / 64) {
      const int o = (t / tp) * 2 * s, ti = (t % tp) / (s / 16) * 16, tj = (t % tp) % (s / 16) * 16;
      const f64x4 z = {0.0, 0.0, 0.0, 0.0};
      tile_store(G + (o + ti) * kCP + o + s + tj,
                 lds_mm<false>(G + (o + s + ti) * kCP + o, G + o * kCP + o + tj, s, z, 1.0));
    }
    __syncthreads();
    for (int t = wave; t < pairs * tp; t += kCThreads / 64) {
      const int o = (t / tp) * 2 * s, ti = (t % tp) / (s / 16) * 16, tj = (t % tp) % (s / 16) * 16;
      const f64x4 z = {0.0, 0.0, 0.0, 0.0};
      tile_store(G + (o + s + ti) * kCP + o + tj,
                 lds_mm<false>(G + (o + s + ti) * kCP + o + s, G + o * kCP + o + s + tj, s, z, -1.0));
    }
    __syncthreads();
    // the corner back to zero (the next level multiplies whole blocks)
    for (int e = threadIdx.x; e < pairs * s * s; e += kCThreads) {
      const int o = e / (s * s) * 2 * s, i = e % (s * s) / s, c = e % s;
      G[(o + i) * kCP + o + s + c] = 0.0;
    }
    __syncthreads();
  }
  // T[k][j] = (L^-1)[j][k]
  for (int e = threadIdx.x; e < kBC * kBC; e += kCThreads) {
    const int kk = e / kBC, j = e % kBC;
    T[e] = kk <= j ? G[j * kCP + kk] : 0.0;
  }
}

}  // namespace

BasisPlan basis_plan(int64_t m, int64_t ldq, int kmax) {
  BasisPlan P{};
  // row splits of about 64 rows while that makes no more than 32
  P.nsplit = (int)(m / 64 < 1 ? 1 : m / 64 > 32 ? 32 : m / 64);
  P.rows = ((m + P.nsplit - 1) / P.nsplit + kBK - 1) / kBK * kBK;
  P.nsplit = (int)((m + P.rows - 1) / P.rows);
  const int ntx = (kmax + kBT - 1) / kBT;
  const int tiles = (ntx > 2 ? ntx : 2) * (kBC / kBT);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) / 256 * 256;
    return o;
  };
  P.S = take((size_t)ldq * kBC * 8);
  P.Y = take((size_t)ldq * kBC * 8);
  P.part = take((size_t)P.nsplit * tiles * kBT * kBT * 8);
  P.W = take((size_t)(ntx > 2 ? ntx : 2) * kBT * kBC * 8);
  P.bytes = off;
  return P;
}

hipError_t launch_basis(const BasisPlan &P, char *scr, const AView &A, const double *norm2,
                        const int64_t *pick, int k, double *Q, int64_t ldq, bool refine, DevState *st,
                        int *flag, hipStream_t s) {
  const int64_t m = A.m;
  double *S = (double *)(scr + P.S), *Y = (double *)(scr + P.Y), *part = (double *)(scr + P.part),
         *W = (double *)(scr + P.W);
  const unsigned nr = (unsigned)((m + kBR - 1) / kBR), ns = (unsigned)P.nsplit;
  const dim3 copy((unsigned)((ldq + 255) / 256), kBC);
  const double ok = refine ? kDevRefined : kDevMax, most = refine ? kDevRefined : kDevRefine;
  auto tn = [&](const double *X, int nx, const double *Z) {
    hipLaunchKernelGGL(k_bs_tn, dim3((unsigned)((nx + kBT - 1) / kBT), kBC / kBT, ns), dim3(256), 0, s,
                       X, nx, Z, ldq, m, P.rows, part);
  };
  auto reduce = [&](int nx, int mode, int b) {
    const int ntx = (nx + kBT - 1) / kBT;
    hipLaunchKernelGGL(k_bs_reduce, dim3((unsigned)(ntx * kBT * kBC / 256)), dim3(256), 0, s, part,
                       ntx, P.nsplit, mode, b, ok, most, W, flag);
  };
  auto nn = [&](const double *X, int kx, const double *in, double *out, int b, DevState *done) {
    hipLaunchKernelGGL(k_bs_nn, dim3(nr, kBC / kBT), dim3(256), 0, s, X, kx, W, in, out, ldq, m, b,
                       done, k, flag);
  };
  for (int t0 = 0; t0 < k; t0 += kBC) {
    const int b = k - t0 < kBC ? k - t0 : kBC;
    double *const Qc = Q + (int64_t)t0 * ldq;
    if (refine) {
      hipLaunchKernelGGL(k_bs_take, copy, dim3(256), 0, s, Qc, m, b, Y, ldq, t0 == 0 ? flag : nullptr);
    } else {
      hipLaunchKernelGGL(k_bs_gather, copy, dim3(256), 0, s, A, pick + t0, b, S, ldq,
                         t0 == 0 ? flag : nullptr);
      if (t0 > 0) {
        tn(Q, t0, S);
        reduce(t0, 0, b);
        nn(Q, t0, S, S, kBC, nullptr);
      }
      tn(S, kBC, S);
      reduce(kBC, 0, b);
      hipLaunchKernelGGL(k_bs_chol, dim3(1), dim3(kCThreads), 0, s, W, b, pick + t0, norm2, W, flag);
      nn(S, kBC, nullptr, Y, kBC, nullptr);
    }
    if (t0 > 0) {
      tn(Q, t0, Y);
      reduce(t0, 1, b);
      nn(Q, t0, Y, Y, kBC, nullptr);
    }
    tn(Y, kBC, Y);
    reduce(kBC, 2, b);
    nn(Y, kBC, nullptr, Qc, b, t0 + b == k ? st : nullptr);
    hipError_t e = hipGetLastError();
    if (e) return e;
  }
  return hipSuccess;
}

}  // namespace gcss
