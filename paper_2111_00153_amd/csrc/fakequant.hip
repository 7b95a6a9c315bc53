// Quantization-aware-training helpers: the weight side of Alg. 1's loop body on the device.
//   forward   What = proj_S(W): every row projected onto the level set of its own scheme with its
//             own scaling factor (Eq. 1-4), written back as fp32 = rowscale * integer level --
//             bit for bit the value the packed inference path multiplies with;
//   backward  the straight-through estimator (Eq. 5): dW = dWhat, zero where the clip was active.
// Both are streaming kernels: 8 bytes per weight for the forward, 8 or 12 for the backward.  gfx950 only.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rmsmp_internal.h"

namespace rmsmp {

namespace {

constexpr int FQ_THREADS = 256;

// w/alpha limited to [-1, 1] (the clip of Section 3.1.1), one correctly rounded divide.
__device__ __forceinline__ float clip_ratio(float w, float alpha) {
  if (w < -alpha) return -1.0f;
  if (w > alpha) return 1.0f;
  return __fdiv_rn(w, alpha);
}

// The same with the reciprocal of alpha, correctly rounded, found once per row: q = w * (1 / alpha) is within 2 units in
// the last place, a fused residual w - q * alpha and one correction bring it within 1, a second one then gives the
// correctly rounded quotient (Markstein, IBM J. Res. Dev. 34, 1990): 5 operations where the divide takes 11.
// RANGE: alpha lies where none of this over- or underflows for any quotient that reaches a level other than
// 0; other rows divide.
struct RowScale {
  float alpha, inv, rowscale, Q;
  int scheme;
  bool range;
};
__device__ __forceinline__ RowScale row_scale(float alpha, int scheme) {
  RowScale s;
  s.alpha = alpha;
  s.scheme = scheme;
  s.Q = scheme == RMSMP_FIXED4 ? 7.0f : 127.0f;
  s.rowscale = scheme == RMSMP_POT4 ? __fmul_rn(alpha, 0.015625f) : __fdiv_rn(alpha, s.Q);
  s.range = alpha >= 0x1p-60f && alpha <= 0x1p60f;
  s.inv = s.range ? __fdiv_rn(1.0f, alpha) : 1.0f;
  return s;
}

// Fixed-m level of x in [-1, 1] as an integer in [-Q, Q], round half to even (Eq. 1-2).
__device__ __forceinline__ int fixed_int(float x, float Q) { return (int)rintf(__fmul_rn(x, Q)); }

// PoT-4 level of x in [-1, 1] as sign * 2^(6-k), k = 0..6, or 0 (Eq. 3-4).  The base-2 logarithm
// is rounded exactly: |x| = f * 2^e with f in [1, 2) rounds up iff f > sqrt(2), and the largest
// float below sqrt(2) has the fraction bits 0x3504f3.
__device__ __forceinline__ int pot4_int(float x) {
  const float a = fabsf(x);
  if (!(a > 0.0078125f)) return 0;  // at or below half of the smallest level, 2^-7
  const uint32_t bits = __float_as_uint(a);
  int e = (int)(bits >> 23) - 127;
  if ((bits & 0x7fffffu) > 0x3504f3u) e += 1;
  e = e > 0 ? 0 : e < -6 ? -6 : e;
  const int mag = 1 << (6 + e);
  return x < 0.0f ? -mag : mag;
}

template <bool RANGE>
__device__ __forceinline__ float project_one(float w, const RowScale& s) {
  float x;
  if (RANGE) {
    float q = __fmul_rn(w, s.inv);
    q = __fmaf_rn(__fmaf_rn(-q, s.alpha, w), s.inv, q);
    x = __fmaf_rn(__fmaf_rn(-q, s.alpha, w), s.inv, q);
    x = w < -s.alpha ? -1.0f : w > s.alpha ? 1.0f : x;
  } else {
    x = clip_ratio(w, s.alpha);
  }
  const int q = s.scheme == RMSMP_POT4 ? pot4_int(x) : fixed_int(x, s.Q);
  return __fmul_rn(s.rowscale, (float)q);
}
template <bool RANGE>
__device__ __forceinline__ float4 project_one(const float4& w, const RowScale& s) {
  return make_float4(project_one<RANGE>(w.x, s), project_one<RANGE>(w.y, s), project_one<RANGE>(w.z, s), project_one<RANGE>(w.w, s));
}
__device__ __forceinline__ float abs_max(float v) { return fabsf(v); }
__device__ __forceinline__ float abs_max(const float4& v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))); }

// max over the T threads of a row; every one gets the result.  red: an entry per wave of the work-group, all of whose threads
// come here.
template <int T>
__device__ __forceinline__ float row_max(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  if (T == 64) return v;
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  red += threadIdx.x / T * (T / 64);
  float m = red[0];
#pragma unroll
  for (int i = 1; i < T / 64; ++i) m = fmaxf(m, red[i]);
  return m;
}

// Results go past the caches: what these kernels write is as large as what they read, and nothing here reads it again
// (3072 x 768 out of the cache 7.3 -> 6.0 us, 4096 x 2000 15.7 -> 12.9; and the backward still finds W in the L2).
__device__ __forceinline__ void stream_out(float* p, float v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void stream_out(float4* p, const float4& v) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store((f4){v.x, v.y, v.z, v.w}, (f4*)p);
}

// A row is read once, all of it at a time, by T threads that hold NV elements (float, or float4 where rows are 16-byte
// aligned) each; T = 64: four rows per work-group, no barrier; T = 128: two.
// held_spread: a work-group's rows are eight apart, so that row r is read on XCD r % 8, whose L2 then has it when the backward, a
// work-group per row, reads it again (3072 x 768, clipped, projection and backward: 10.1 us with neighbouring rows).
constexpr int held_spread(int T, int NV) { return T == 128 || (T == 64 && NV > 2) ? 8 : 1; }
template <class V, int T, int NV>
__global__ __launch_bounds__(T < FQ_THREADS ? FQ_THREADS : T) void fake_quant_held_kernel(FakeQuantArgs a, int nv) {
  __shared__ float red[(T < FQ_THREADS ? FQ_THREADS : T) / 64];
  constexpr int ROWS = T < FQ_THREADS ? FQ_THREADS / T : 1;
  constexpr unsigned SPREAD = held_spread(T, NV);
  const int64_t row = (int64_t)(blockIdx.x / SPREAD) * (SPREAD * ROWS) + blockIdx.x % SPREAD + (ROWS > 1 ? SPREAD * __builtin_amdgcn_readfirstlane(threadIdx.x / T) : 0);
  if (T == 64 && row >= a.M) return;
  const int64_t r = row < a.M ? row : a.M - 1;  // (there is a barrier: past the last row that one's maximum once more)
  const V* w = (const V*)(a.W + r * a.K);
  V* out = (V*)(a.What + r * a.K);
  const int tid = threadIdx.x % T;
  V v[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) v[j] = tid + j * T < nv ? w[tid + j * T] : V{};
  const int scheme = a.scheme[r];
  float alpha;
  if (a.alpha) {
    alpha = a.alpha[r];
  } else {
    float m = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j) m = fmaxf(m, abs_max(v[j]));
    alpha = row_max<T>(m, red);
    if (alpha == 0.0f) alpha = 1.0f;
  }
  if (row >= a.M) return;
  if (a.alpha_out && tid == 0) a.alpha_out[r] = alpha;
  const RowScale s = row_scale(alpha, scheme);
  if (s.range) {
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (tid + j * T < nv) stream_out(out + tid + j * T, project_one<true>(v[j], s));
  } else {
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (tid + j * T < nv) out[tid + j * T] = project_one<false>(v[j], s);
  }
}

// One work-group per row, any K: read twice where the maximum is asked for.
template <class V>
__global__ __launch_bounds__(FQ_THREADS) void fake_quant_long_kernel(FakeQuantArgs a, int64_t nv) {
  __shared__ float red[FQ_THREADS / 64];
  const int64_t r = blockIdx.x;
  const V* w = (const V*)(a.W + r * a.K);
  V* out = (V*)(a.What + r * a.K);
  float alpha;
  if (a.alpha) {
    alpha = a.alpha[r];
  } else {
    float m = 0.0f;
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < nv; i += FQ_THREADS) m = fmaxf(m, abs_max(w[i]));
    alpha = row_max<FQ_THREADS>(m, red);
    if (alpha == 0.0f) alpha = 1.0f;
  }
  if (a.alpha_out && threadIdx.x == 0) a.alpha_out[r] = alpha;
  const RowScale s = row_scale(alpha, a.scheme[r]);
  if (s.range) {
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < nv; i += FQ_THREADS) stream_out(out + i, project_one<true>(w[i], s));
  } else {
    for (int64_t i = threadIdx.x; i < nv; i += FQ_THREADS) out[i] = project_one<false>(w[i], s);
  }
}

__device__ __forceinline__ float pass_unclipped(float g, float w, float alpha) { return fabsf(w) > alpha ? 0.0f : g; }
__device__ __forceinline__ float4 pass_unclipped(const float4& g, const float4& w, float alpha) {
  return make_float4(pass_unclipped(g.x, w.x, alpha), pass_unclipped(g.y, w.y, alpha), pass_unclipped(g.z, w.z, alpha), pass_unclipped(g.w, w.w, alpha));
}

constexpr int STE_COPY_U = 2;
// Nothing was clipped: the gradient passes unchanged (rows do not matter).
template <class V>
__global__ __launch_bounds__(FQ_THREADS) void ste_copy_kernel(const V* g, V* out, int64_t n) {
  constexpr int U = STE_COPY_U;
  const int64_t i0 = (int64_t)blockIdx.x * (FQ_THREADS * U) + threadIdx.x;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (i0 + u * FQ_THREADS < n) stream_out(out + i0 + u * FQ_THREADS, g[i0 + u * FQ_THREADS]);
}

// One work-group per row.
template <class V>
__global__ __launch_bounds__(FQ_THREADS) void ste_clipped_kernel(SteArgs a) {
  constexpr int E = sizeof(V) / sizeof(float);
  const int64_t r = blockIdx.x;
  const V* g = (const V*)(a.dWhat + r * a.K);
  const V* w = (const V*)(a.W + r * a.K);
  V* out = (V*)(a.dW + r * a.K);
  const float alpha = a.alpha[r];
  for (int64_t i = threadIdx.x; i < a.K / E; i += FQ_THREADS) {
    const V v = w[i];
    stream_out(out + i, pass_unclipped(g[i], v, alpha));
  }
}
// Short rows: a wave each.
template <class V>
__global__ __launch_bounds__(FQ_THREADS) void ste_clipped_short_kernel(SteArgs a) {
  constexpr int E = sizeof(V) / sizeof(float);
  const int64_t r = (int64_t)blockIdx.x * (FQ_THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  if (r >= a.M) return;
  const V* g = (const V*)(a.dWhat + r * a.K);
  const V* w = (const V*)(a.W + r * a.K);
  V* out = (V*)(a.dW + r * a.K);
  const float alpha = a.alpha[r];
  for (int i = threadIdx.x % 64; i < (int)a.K / E; i += 64) stream_out(out + i, pass_unclipped(g[i], w[i], alpha));
}

// Rows that are no multiple of 16 bytes (K >= 4), read 16 bytes at a time all the same: such a read touches at most two rows.
// The work-group's first row by one division, a thread's by counting on from there (magic, shift: / K below 2^31).
__global__ __launch_bounds__(FQ_THREADS) void ste_clipped_flat_kernel(SteArgs a, uint32_t magic, int shift) {
  constexpr int U = 4;
  const int64_t n = a.M * a.K, e0 = (int64_t)blockIdx.x * (FQ_THREADS * U * 4);
  const int64_t r0 = e0 / a.K;
  const uint32_t K = (uint32_t)a.K, first = (uint32_t)(e0 - r0 * a.K);
  const int64_t last = a.M - 1;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t at = (threadIdx.x + u * FQ_THREADS) * 4;
    const int64_t e = e0 + at;
    if (e >= n) break;
    const uint32_t dr = __umulhi(first + at, magic) >> shift;
    const uint32_t left = K - (first + at - dr * K);  // elements of row r from here on
    const int64_t r = r0 + dr;
    const float a0 = a.alpha[r], a1 = a.alpha[r < last ? r + 1 : r];
    if (e + 4 <= n) {
      const float4 g = *(const float4*)(a.dWhat + e), w = *(const float4*)(a.W + e);
      stream_out((float4*)(a.dW + e), make_float4(pass_unclipped(g.x, w.x, a0), pass_unclipped(g.y, w.y, left > 1 ? a0 : a1),
                                                  pass_unclipped(g.z, w.z, left > 2 ? a0 : a1), pass_unclipped(g.w, w.w, left > 3 ? a0 : a1)));
    } else {
      for (int i = 0; i < (int)(n - e); ++i) a.dW[e + i] = pass_unclipped(a.dWhat[e + i], a.W[e + i], left > (uint32_t)i ? a0 : a1);
    }
  }
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

template <class V, int T, int NV>
void held(const FakeQuantArgs& a, int nv, hipStream_t s) {
  constexpr int SPREAD = held_spread(T, NV), ROWS = (T < FQ_THREADS ? FQ_THREADS / T : 1) * SPREAD;
  hipLaunchKernelGGL((fake_quant_held_kernel<V, T, NV>), dim3((unsigned)((a.M + ROWS - 1) / ROWS * SPREAD)), dim3(T < FQ_THREADS ? FQ_THREADS : T), 0, s, a, nv);
}

// How many threads a row gets.  What bounds these calls besides the bytes is the number of waves that have to be launched, 12 000 of
// them for 3072 rows of 768 by work-groups of 256, a quarter of whose lanes have nothing to do: with rows enough to fill the
// chip a wave or two per row, with several elements a lane, take less.  us, tensors in the caches, row maximum found / alpha given, 256 threads per row (the kernel
// that had these rows before) against:
//   one wave      6000 x 600   9.1 / 7.3 -> 5.8 / 5.3    16384 x 201  14.5 / 9.8 -> 6.6 / 6.1    4096 x 301  6.1 / 4.6 -> 4.2 / 3.8
//   two waves     3072 x 768   5.8 / 4.8 -> 4.5 / 3.9     8192 x 1000 14.0 / 11.0 -> 10.4 / 10.3  2048 x 1200 5.4 / 4.1 -> 4.6 / 4.1
//                 4096 x 1536  9.0 / 7.4 -> 6.9 / 6.3     3072 x 769   6.1 / 4.6 -> 5.0 / 4.7
//   four waves, two elements a lane: 8192 x 1200 16.0 / 13.7 -> 13.6 / 13.5 (two waves 13.6 / 13.2), 16384 x 2048 38.9 / 38.7 -> 38.2 / 38.7 (two 41.5 / 41.5)
// Below: 1024 x 768 3.5 / 3.1 with 256 threads, 3.6 / 3.2 with two waves, 3.7 / 3.5 with one.  Work-groups of 1024 where rows are long, or few of
// them are all there is; rows longer than a work-group's registers hold are read twice.
template <class V>
void fake_quant_any(const FakeQuantArgs& a, int64_t nv, hipStream_t s) {
  constexpr bool ONE = sizeof(V) == sizeof(float);  // (rows that are no multiple of 16 bytes)
  const int n = (int)std::min<int64_t>(nv, 0x7fffffff);
  if (n <= 64) held<V, 64, 1>(a, n, s);
  else if (n <= 128 && a.M >= 2048) held<V, 64, 2>(a, n, s);
  else if (!ONE && n <= 192 && a.M >= 4096) held<V, 64, 3>(a, n, s);
  else if (ONE && n <= 256 && a.M >= 4096) held<V, 64, 4>(a, n, s);
  else if (ONE && n <= 512 && a.M >= 4096) held<V, 64, 8>(a, n, s);
  else if (n <= 256 && a.M >= 1280) held<V, 128, 2>(a, n, s);
  else if (n <= 512 && a.M >= 1280 && a.M < 8192) held<V, 128, 4>(a, n, s);
  else if (n <= 512 && a.M >= 8192) held<V, 256, 2>(a, n, s);
  else if (ONE && n <= 1024 && a.M >= 2048) held<V, 128, 8>(a, n, s);
  else if (n <= 256) held<V, 256, 1>(a, n, s);
  else if (n <= 1024) held<V, 256, 4>(a, n, s);
  else if (n <= 2048 && a.M >= 1024) held<V, 256, 8>(a, n, s);
  else if (n <= 2048) held<V, 1024, 2>(a, n, s);
  else if (n <= 4096 && a.M >= 1024) held<V, 256, 16>(a, n, s);
  else if (n <= 8192) held<V, 1024, 8>(a, n, s);
  else hipLaunchKernelGGL(fake_quant_long_kernel<V>, dim3((unsigned)a.M), dim3(FQ_THREADS), 0, s, a, nv);
}

int launch_fake_quant_rows(const FakeQuantArgs& a, void* stream) {
  if (a.M <= 0 || a.K <= 0) return 0;
  if (a.K % 4 == 0 && aligned16(a.W) && aligned16(a.What))
    fake_quant_any<float4>(a, a.K / 4, (hipStream_t)stream);
  else
    fake_quant_any<float>(a, a.K, (hipStream_t)stream);
  return (int)hipGetLastError();
}

template <class V>
void ste_any(const SteArgs& a, int64_t nv, hipStream_t s) {
  if (nv <= 64 || (nv <= 128 && a.M >= 2048))
    hipLaunchKernelGGL(ste_clipped_short_kernel<V>, dim3((unsigned)((a.M + 3) / 4)), dim3(FQ_THREADS), 0, s, a);
  else
    hipLaunchKernelGGL(ste_clipped_kernel<V>, dim3((unsigned)a.M), dim3(FQ_THREADS), 0, s, a);
}

int launch_ste_backward(const SteArgs& a, void* stream) {
  if (a.M <= 0 || a.K <= 0) return 0;
  hipStream_t s = (hipStream_t)stream;
  const bool aligned = aligned16(a.dWhat) && aligned16(a.dW);
  if (!a.alpha) {
    const int64_t n = a.M * a.K;
    const bool vec = aligned && n % 4 == 0;
    const int64_t nv = vec ? n / 4 : n, blocks = (nv + STE_COPY_U * FQ_THREADS - 1) / (STE_COPY_U * FQ_THREADS);
    if (blocks > 0x7fffffff) return (int)hipErrorInvalidValue;
    if (vec)
      hipLaunchKernelGGL(ste_copy_kernel<float4>, dim3((unsigned)blocks), dim3(FQ_THREADS), 0, s, (const float4*)a.dWhat, (float4*)a.dW, nv);
    else
      hipLaunchKernelGGL(ste_copy_kernel<float>, dim3((unsigned)blocks), dim3(FQ_THREADS), 0, s, a.dWhat, a.dW, nv);
  } else if (aligned && a.K % 4 == 0 && aligned16(a.W)) {
    ste_any<float4>(a, a.K / 4, s);
  } else if (aligned && aligned16(a.W) && a.K > 128 && a.K < ((int64_t)1 << 30) && a.M * a.K >= ((int64_t)1 << 22) &&
             a.M * a.K / (16 * FQ_THREADS) < 0x7fffffff) {
    // (8192 x 8191: 148 us, row by row 171; 1000 x 511, where this is too few work-groups: 3.1 and 2.7)
    const int shift = 31 - __builtin_clz((unsigned)a.K - 1);  // 2^shift < K <= 2^(shift + 1)
    const uint32_t magic = (uint32_t)((((unsigned __int128)1 << (32 + shift)) + (uint64_t)a.K - 1) / (uint64_t)a.K);
    const int64_t per = 16 * FQ_THREADS;
    hipLaunchKernelGGL(ste_clipped_flat_kernel, dim3((unsigned)((a.M * a.K + per - 1) / per)), dim3(FQ_THREADS), 0, s, a, magic, shift);
  } else {
    ste_any<float>(a, a.K, s);
  }
  return (int)hipGetLastError();
}

}  // namespace rmsmp
