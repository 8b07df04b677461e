// Reduced-precision storage of A: bfloat16 (round to nearest even) and OCP
// FP8 E4M3 (e4m3fn) with one binary32 scale per column.  One wavefront per
// column.  The encoders are written from the formats' definitions with
// exact scaling by powers of two and round-half-even (v_rndne_f32).
#include "gcss_device.h"

namespace gcss {

__device__ __forceinline__ uint16_t bf16_rne(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)(((u >> 16) & 0x8000u) | 0x7FC0u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// E4M3: bias 7, subnormal step 2^-9, largest finite 448 (S.1111.110).
__device__ __forceinline__ uint8_t fp8_rne_sat(float x) {
  const uint32_t u = __float_as_uint(x);
  const uint8_t sign = (uint8_t)((u >> 24) & 0x80u);
  const float ax = fabsf(x);
  if (ax != ax) return (uint8_t)(sign | 0x7Fu);
  if (ax >= 448.f) return (uint8_t)(sign | 0x7Eu);
  if (ax < 0.015625f) {  // below 2^-6: multiples of 2^-9 (code 8 is 2^-6 itself)
    const int c = (int)rintf(ax * 512.f);
    return (uint8_t)(sign | c);
  }
  int e = (int)((__float_as_uint(ax) >> 23) & 0xFFu) - 127;  // 2^e <= ax < 2^(e+1)
  float sc = ldexpf(ax, 3 - e);                                // in [8, 16)
  int q = (int)rintf(sc);
  if (q == 16) {
    q = 8;
    e += 1;
  }
  return (uint8_t)(sign | ((e + 7) << 3) | (q - 8));
}

__global__ __launch_bounds__(256) void k_quantize(const float *__restrict__ a, int64_t m,
                                                  int64_t n, int64_t lda, int dtype,
                                                  void *__restrict__ out, int64_t ldo,
                                                  float *__restrict__ scales) {
  const int lane = threadIdx.x & 63;
  const int64_t col = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= n) return;
  const float *src = a + col * lda;
  if (dtype == DT_BF16) {
    uint16_t *dst = (uint16_t *)out + col * ldo;
    for (int64_t j = lane; j < ldo; j += 64) dst[j] = j < m ? bf16_rne(src[j]) : (uint16_t)0;
    return;
  }
  float amax = 0.f;
  for (int64_t j = lane; j < m; j += 64) amax = fmaxf(amax, fabsf(src[j]));
  amax = wave_max(amax);
  const float s = amax > 0.f ? amax / 448.f : 1.f;
  if (lane == 0) scales[col] = s;
  uint8_t *dst = (uint8_t *)out + col * ldo;
  for (int64_t j = lane; j < ldo; j += 64) dst[j] = j < m ? fp8_rne_sat(src[j] / s) : (uint8_t)0;
}

// out[j + c*ldo] = the bfloat16 value in[j + c*ldi] as binary32 (exact),
// rows m..ldo-1 set to zero.  One wavefront per column.
__global__ __launch_bounds__(256) void k_bf16_to_f32(const uint16_t *__restrict__ in, int64_t m,
                                                     int64_t n, int64_t ldi,
                                                     float *__restrict__ out, int64_t ldo) {
  const int lane = threadIdx.x & 63;
  const int64_t col = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= n) return;
  const uint16_t *src = in + col * ldi;
  float *dst = out + col * ldo;
  for (int64_t j = lane; j < ldo; j += 64)
    dst[j] = j < m ? __uint_as_float((uint32_t)src[j] << 16) : 0.f;
}

hipError_t launch_bf16_to_f32(const void *in, int64_t m, int64_t n, int64_t ldi, float *out,
                              int64_t ldo, hipStream_t s) {
  hipLaunchKernelGGL(k_bf16_to_f32, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s,
                     (const uint16_t *)in, m, n, ldi, out, ldo);
  return hipGetLastError();
}

// The same conversions with 16-byte loads, one read of A and packed stores.
//
// Bound by memory: m n * (4 + output bytes), plus the pads of the output.
// The element-wise kernel above read FP8 columns twice with 4-byte loads,
// stored single bytes and spent ~30 vector instructions per element on a
// full division and the integer encoder: 697 us for 8192 x 32768 (1.9 TB/s).
// Here a column's values stay in registers between its maximum and its
// codes, and the quotient by the column's scale s is formed from r = 1 / s:
// q0 = x r, q = q0 + r (x - q0 s) with the residual exact by FMA, which is
// the correctly rounded x / s when r is correctly rounded (Markstein,
// "Computation of elementary functions on the IBM RISC System/6000", 1990)
// and no term underflows.  Columns whose scale lies in [2^-60, 2^60] meet
// that for every |x / s| >= 2^-11; below that any error leaves the code 0 (half
// of the smallest code is 2^-10).  Other columns (and infinities) divide.

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Four non-negative quotients (a NaN passes through) to E4M3 codes with the
// signs of x: v_cvt_pk_fp8_f32 rounds to nearest even; its input is clamped
// to 448, and a NaN's code is 0x7F.
__device__ __forceinline__ uint32_t fp8x4_rne_sat(const float (&q)[4], const f32x4_t &x) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(fminf(q[0], 448.f), fminf(q[1], 448.f), 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(fminf(q[2], 448.f), fminf(q[3], 448.f), w, true);
  uint32_t c = (uint32_t)w;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (q[e] != q[e]) c = (c & ~(0xFFu << (8 * e))) | (0x7Fu << (8 * e));
  // the top bytes of x[0..3], of which the sign bits
  const uint32_t lo = __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07030703u);
  const uint32_t hi = __builtin_amdgcn_perm(__float_as_uint(x[3]), __float_as_uint(x[2]), 0x07030703u);
  return c | (((lo & 0xFFFFu) | (hi << 16)) & 0x80808080u);
}

constexpr int kQuantV = 8;  // most 16-byte loads per thread that hold a column's part

// FP8: WPC waves of a 256-thread workgroup per column, V loads per thread
// (ldo <= 256 WPC V).
template <int WPC, int V>
__global__ __launch_bounds__(256) void k_quant_fp8(const float *__restrict__ a, int64_t m,
                                                   int64_t n, int64_t lda,
                                                   uint8_t *__restrict__ out, int64_t ldo,
                                                   float *__restrict__ scales) {
  __shared__ float red[4];
  const int wave = threadIdx.x >> 6;
  const int64_t col = (int64_t)blockIdx.x * (4 / WPC) + wave / WPC;
  const int tid = threadIdx.x % (64 * WPC);
  const bool live = col < n;  // (false only for whole waves, WPC = 1)
  const float *src = a + (live ? col : n - 1) * lda;
  f32x4_t v[V];
  float amax = 0.f;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int64_t j = 4 * (int64_t)(tid + 64 * WPC * u);
    // (a chunk past m reads the column's first one; a chunk that straddles
    // m ends inside lda, a multiple of four)
    v[u] = __builtin_nontemporal_load((const f32x4_t *)(src + (j < m ? j : 0)));
  }
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int64_t j = 4 * (int64_t)(tid + 64 * WPC * u);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[u][e] = j + e < m ? v[u][e] : 0.f;
      amax = fmaxf(amax, fabsf(v[u][e]));
    }
  }
  amax = wave_max(amax);
  if constexpr (WPC == 4) {
    if ((threadIdx.x & 63) == 0) red[wave] = amax;
    __syncthreads();
    amax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  }
  if (!live) return;
  const float s = amax > 0.f ? amax / 448.f : 1.f;  // (0 for a column of the smallest subnormals)
  if (tid == 0) scales[col] = s;
  uint32_t *dst = (uint32_t *)(out + col * ldo);
  const bool fast = s >= 0x1p-60f && s <= 0x1p60f;
  const float r = 1.f / s;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int64_t c = tid + 64 * WPC * u;
    if (4 * c < ldo) {
      uint32_t code = 0;
      if (fast) {
        float q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float ax = fabsf(v[u][e]);
          const float q0 = ax * r;
          q[e] = fmaf(fmaf(-q0, s, ax), r, q0);
        }
        code = fp8x4_rne_sat(q, v[u]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * c + e < m) code |= (uint32_t)fp8_rne_sat(v[u][e] / s) << (8 * e);
      }
      __builtin_nontemporal_store(code, dst + c);
    }
  }
}

// BF16: eight elements per thread, one 16-byte store; cpc = ldo / 8.
// NT: loads and stores bypass the caches.
template <bool NT>
__global__ __launch_bounds__(256) void k_quant_bf16(const float *__restrict__ a, int64_t m,
                                                    int64_t lda, uint16_t *__restrict__ out,
                                                    int64_t ldo, int64_t cpc, int64_t total) {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  auto load = [](const float *p) -> f32x4_t {
    if constexpr (NT) return __builtin_nontemporal_load((const f32x4_t *)p);
    else return *(const f32x4_t *)p;
  };
  for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < total; x += (int64_t)gridDim.x * 256) {
    // (a division in 64 bits takes several times the conversion's instructions)
    const int64_t col = total <= UINT32_MAX ? (int64_t)((uint32_t)x / (uint32_t)cpc) : x / cpc;
    const int64_t j = 8 * (x - col * cpc);
    const float *src = a + col * lda;
    f32x4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;  // (pads are not loaded)
    if (j < m) lo = load(src + j);
    if (j + 4 < m) hi = load(src + j + 4);
    u32x4_t o;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int e = 2 * w;
      const float x0 = e < 4 ? lo[e & 3] : hi[e & 3], x1 = e < 4 ? lo[(e & 3) + 1] : hi[(e & 3) + 1];
      const uint32_t b0 = j + e < m ? bf16_rne(x0) : 0u, b1 = j + e + 1 < m ? bf16_rne(x1) : 0u;
      o[w] = b0 | (b1 << 16);
    }
    u32x4_t *const dst = (u32x4_t *)(out + col * ldo + j);
    if constexpr (NT) __builtin_nontemporal_store(o, dst);
    else *dst = o;
  }
}

// The wide kernels need 16-byte aligned columns of A and whole packed words
// per output column; FP8 also a column that its waves' registers hold.  One
// wave per column keeps the maximum inside the wave, as far as its registers
// go (2048 rows); above that four waves share a column.  A wave issues its V
// loads whatever the column's length, so V is the smallest that holds it (with
// eight for all, columns of up to 128 rows were slower than element by element:
// m = 50, n = 120000 44 -> 56 us, with one 33 us).  The BF16 kernel bypasses the
// caches only where A and the output together exceed the last-level one (256
// MB): below it 2048 x 20000 takes 37 us against 42 so, and 64 x 200000 with 192
// rows of pads 30 against 35 (element by element 31); above it 8192 x 20000 159
// against 167 us.  (FP8 gains and loses a tenth either way.)
// Measured on MI355X, element-wise kernel -> these: FP8 8192 x 32768 697 ->
// 225 us (5.97 TB/s), FP8 1024 x 262144 614 -> 223 us, FP8 333 x 100003 77 ->
// 43 us; BF16 8192 x 32768 408 -> 261 us (6.2 TB/s), BF16 333 x 100003 42 ->
// 35 us.  Other shapes take the element-wise kernel.
hipError_t launch_quantize(const float *a, int64_t m, int64_t n, int64_t lda, int dtype,
                           void *out, int64_t ldo, float *scales, hipStream_t s) {
  const bool wide = lda % 4 == 0 && (uintptr_t)a % 16 == 0;
  if (dtype == DT_BF16 && wide && ldo % 8 == 0 && (uintptr_t)out % 16 == 0) {
    const int64_t cpc = ldo / 8, total = n * cpc;
    const int64_t blocks = (total + 255) / 256;
    const bool nt = n * (4 * m + 2 * ldo) > (int64_t)256 << 20;
    hipLaunchKernelGGL(nt ? k_quant_bf16<true> : k_quant_bf16<false>,
                       dim3((unsigned)(blocks < (1 << 20) ? blocks : (1 << 20))), dim3(256), 0, s, a, m,
                       lda, (uint16_t *)out, ldo, cpc, total);
  } else if (dtype == DT_FP8 && wide && ldo % 4 == 0 && (uintptr_t)out % 4 == 0 &&
             ldo <= 4 * kQuantV * 256) {
    auto run = [&](auto fn, int wpc) {
      hipLaunchKernelGGL(fn, dim3((unsigned)((n + 4 / wpc - 1) / (4 / wpc))), dim3(256), 0, s, a, m, n,
                         lda, (uint8_t *)out, ldo, scales);
    };
    if (ldo <= 256) run(k_quant_fp8<1, 1>, 1);
    else if (ldo <= 512) run(k_quant_fp8<1, 2>, 1);
    else if (ldo <= 1024) run(k_quant_fp8<1, 4>, 1);
    else if (ldo <= 2048) run(k_quant_fp8<1, kQuantV>, 1);
    else run(k_quant_fp8<4, kQuantV>, 4);
  } else {
    hipLaunchKernelGGL(k_quantize, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, a, m, n, lda,
                       dtype, out, ldo, scales);
  }
  return hipGetLastError();
}

}  // namespace gcss
