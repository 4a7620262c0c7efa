// Row-wise kernels of the forward: embedding gather with the first RMSNorm,
// RMSNorm (optionally gathering rows) and the prefix-cache writer.
#include <type_traits>

#include "kernels.h"
#include "common.h"

namespace dllm {

namespace {

constexpr int kRowThreads = 256;

// store 4 consecutive values as one 8-byte (bf16) or 16-byte (fp32) access
__device__ __forceinline__ void store4(bf16_t* p, f32x4 v) {
  const uint32_t lo = uint32_t(f2bf(v.x)) | (uint32_t(f2bf(v.y)) << 16);
  const uint32_t hi = uint32_t(f2bf(v.z)) | (uint32_t(f2bf(v.w)) << 16);
  *reinterpret_cast<u32x2*>(p) = u32x2{lo, hi};
}
__device__ __forceinline__ void store4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }

constexpr int kNormChunks = 8;   // 16-byte chunks per thread held in registers: d <= 8192
// resid_rmsnorm: 1024 threads a row, so that each walks the partials of one or
// two chunks (512 rows of 8 parts, d 4096: a 265 us layer gains 1.3 us over 256
// threads a row, 1536 rows 4; up to d 2048 part of the threads have no chunk).
// The loads of 8, then 4, then 2 parts are in flight together: with 2 and 4
// parts loaded one after the other a launch took 11.5 us instead of 10.6 (1536
// rows, d 512), 9.8 instead of 9.3 (700 rows, d 1024), 13.3 instead of 13.0
// (512 rows, d 4096).
constexpr int kWideThreads = 1024;

// One workgroup per output row; the row stays in registers between the sum
// of squares (reduced in fp32 over 4 waves) and the scaled store.
template <typename T>
__global__ __launch_bounds__(kRowThreads) void rmsnorm_kernel(const float* __restrict__ x, int d, float eps,
                                                              const int32_t* __restrict__ pos, int n_pos, int seq,
                                                              T* __restrict__ out) {
  __shared__ float part[kRowThreads / kWave];
  const int r = blockIdx.x;
  const int src_row = pos ? (r / n_pos) * seq + min(max(pos[r % n_pos], 0), seq - 1) : r;
  const float* xr = x + size_t(src_row) * d;
  f32x4 v[kNormChunks];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < kNormChunks; ++j) {
    const int c = (threadIdx.x + j * kRowThreads) * 4;
    v[j] = c < d ? *reinterpret_cast<const f32x4*>(xr + c) : f32x4{0.f, 0.f, 0.f, 0.f};
    ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < kRowThreads / kWave; ++w) tot += part[w];
  const float inv = 1.0f / sqrtf(tot / float(d) + eps);
  T* o = out + size_t(r) * d;
#pragma unroll
  for (int j = 0; j < kNormChunks; ++j) {
    const int c = (threadIdx.x + j * kRowThreads) * 4;
    if (c < d) store4(o + c, v[j] * inv);
  }
}

// Embedding and the first layer's RMSNorm of one row: x[r] = emb[tok[r]],
// out[r] = x[r] / sqrt(mean(x[r]^2) + eps).  Two launches of 11 and 5 us for
// 512 rows of 4096 (2-byte loads) before.
template <typename T>
__global__ __launch_bounds__(kRowThreads) void embed_rmsnorm_kernel(const int32_t* __restrict__ tok,
                                                                    const T* __restrict__ emb, int d, int vocab,
                                                                    float eps, float* __restrict__ x,
                                                                    T* __restrict__ out, bool wide) {
  __shared__ float part[kRowThreads / kWave];
  const int r = blockIdx.x;
  const T* src = emb + size_t(min(max(tok[r], 0), vocab - 1)) * d;
  f32x4 v[kNormChunks];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < kNormChunks; ++j) {
    const int c = (threadIdx.x + j * kRowThreads) * 4;
    v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (c < d) {
      if (!wide) {   // an embedding that starts off a 16-byte boundary
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] = load_f(src + c + e);
      } else if constexpr (Elem<T>::bytes == 2) {
        const u32x2 w = *reinterpret_cast<const u32x2*>(src + c);
        v[j] = f32x4{bf2f(uint16_t(w.x)), bf2f(uint16_t(w.x >> 16)), bf2f(uint16_t(w.y)), bf2f(uint16_t(w.y >> 16))};
      } else {
        v[j] = *reinterpret_cast<const f32x4*>(src + c);
      }
      *reinterpret_cast<f32x4*>(x + size_t(r) * d + c) = v[j];
    }
    ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < kRowThreads / kWave; ++w) tot += part[w];
  const float inv = 1.0f / sqrtf(tot / float(d) + eps);
#pragma unroll
  for (int j = 0; j < kNormChunks; ++j) {
    const int c = (threadIdx.x + j * kRowThreads) * 4;
    if (c < d) store4(out + size_t(r) * d + c, v[j] * inv);
  }
}

// Residual update from split-K partial tiles fused with the RMSNorm that
// follows it: x[r] += part[0][r] + part[1][r] + ... (in this order), then
// out[r] = x[r] / sqrt(mean(x[r]^2) + eps).  With pos (the final norm): output
// row r reads row src(r) as in rmsnorm_kernel, and x, which nothing reads
// after it, is not written back.
template <typename T>
__global__ __launch_bounds__(kWideThreads) void resid_rmsnorm_kernel(const float* __restrict__ part, int splits, int np,
                                                                int M, float* __restrict__ x, int d, float eps,
                                                                const int32_t* __restrict__ pos, int n_pos, int seq,
                                                                T* __restrict__ out) {
  constexpr int THREADS = kWideThreads;
  constexpr int CH = kNormChunks * kRowThreads / THREADS;   // 16-byte chunks per thread: d <= 8192
  __shared__ float red[THREADS / kWave];
  const int r = blockIdx.x;
  const int sr = pos ? (r / n_pos) * seq + min(max(pos[r % n_pos], 0), seq - 1) : r;
  float* xr = x + size_t(sr) * d;
  auto pr = [&](int p, int c) { return *reinterpret_cast<const f32x4*>(part + (size_t(p) * M + sr) * np + c); };
  f32x4 v[CH];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int c = (threadIdx.x + j * THREADS) * 4;
    v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (c < d) {
      v[j] = *reinterpret_cast<const f32x4*>(xr + c);
      int p = 0;
      auto group = [&](auto n) {   // n parts, every load before the first sum, added in order
        constexpr int N = decltype(n)::value;
        f32x4 a[N];
#pragma unroll
        for (int q = 0; q < N; ++q) a[q] = pr(p + q, c);
#pragma unroll
        for (int q = 0; q < N; ++q) v[j] += a[q];
        p += N;
      };
      while (p + 8 <= splits) group(std::integral_constant<int, 8>{});
      if (p + 4 <= splits) group(std::integral_constant<int, 4>{});
      if (p + 2 <= splits) group(std::integral_constant<int, 2>{});
      if (p < splits) v[j] += pr(p, c);
      if (!pos) *reinterpret_cast<f32x4*>(xr + c) = v[j];
    }
    ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < THREADS / kWave; ++w) tot += red[w];
  const float inv = 1.0f / sqrtf(tot / float(d) + eps);
  T* o = out + size_t(r) * d;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int c = (threadIdx.x + j * THREADS) * 4;
    if (c < d) store4(o + c, v[j] * inv);
  }
}

// Copies one head's K rows and V^T columns into the cache: blocks 0 .. nk - 1
// of a head take its K rows as one run of 16-byte chunks, the rest kVtRows dims
// of V^T each, consecutive threads along the positions of a dim (a column of
// V^T per block, 2 bytes in every cache line, took 18 us for 512 positions of
// 32 heads of 128).
constexpr int kVtRows = 16;
constexpr int kCopyChunks = 4;   // 16-byte chunks of K per thread
template <typename T>
__global__ __launch_bounds__(kRowThreads) void kv_store_kernel(const T* __restrict__ k, const T* __restrict__ vt,
                                                               int seq, int hd, int vt_ld, T* __restrict__ ck,
                                                               T* __restrict__ cvt, int cap, int off, int nk,
                                                               bool wide) {
  const int h = blockIdx.x;
  if (int(blockIdx.y) < nk) {
    if (!wide) {   // a cache that starts off a 16-byte boundary
      for (int e = blockIdx.y * kRowThreads + threadIdx.x; e < seq * hd; e += nk * kRowThreads)
        ck[(size_t(h) * cap + off) * hd + e] = k[size_t(h) * seq * hd + e];
      return;
    }
    // head_dim rows are whole chunks, and so 16-byte aligned in both where the bases are
    const int n = seq * hd * int(sizeof(T)) / 16;
    const u32x4* src = reinterpret_cast<const u32x4*>(k + size_t(h) * seq * hd);
    u32x4* dst = reinterpret_cast<u32x4*>(ck + (size_t(h) * cap + off) * hd);
    const int c0 = blockIdx.y * kCopyChunks * kRowThreads + threadIdx.x;
    u32x4 v[kCopyChunks];
#pragma unroll
    for (int i = 0; i < kCopyChunks; ++i) v[i] = src[min(c0 + i * kRowThreads, n - 1)];
#pragma unroll
    for (int i = 0; i < kCopyChunks; ++i)
      if (c0 + i * kRowThreads < n) dst[c0 + i * kRowThreads] = v[i];
    return;
  }
  const int d0 = (blockIdx.y - nk) * kVtRows;   // head_dim is a multiple of kVtRows
  const T* src = vt + (size_t(h) * hd + d0) * vt_ld;
  T* dst = cvt + (size_t(h) * hd + d0) * cap + off;
  for (int s = threadIdx.x; s < seq; s += kRowThreads) {
    T v[kVtRows];
#pragma unroll
    for (int d = 0; d < kVtRows; ++d) v[d] = src[size_t(d) * vt_ld + s];
#pragma unroll
    for (int d = 0; d < kVtRows; ++d) dst[size_t(d) * cap + s] = v[d];
  }
}

}  // namespace

hipError_t embed_rmsnorm(int dtype, const int32_t* tok, int rows, const void* emb, int d, int vocab, float eps,
                         float* x, void* out, hipStream_t s) {
  if (d % 4 || d > kNormChunks * kRowThreads * 4) return hipErrorInvalidValue;
  const bool wide = reinterpret_cast<uintptr_t>(emb) % 16 == 0;
  if (dtype)
    hipLaunchKernelGGL(embed_rmsnorm_kernel<bf16_t>, dim3(rows), dim3(kRowThreads), 0, s, tok,
                       static_cast<const bf16_t*>(emb), d, vocab, eps, x, static_cast<bf16_t*>(out), wide);
  else
    hipLaunchKernelGGL(embed_rmsnorm_kernel<float>, dim3(rows), dim3(kRowThreads), 0, s, tok,
                       static_cast<const float*>(emb), d, vocab, eps, x, static_cast<float*>(out), wide);
  return hipGetLastError();
}

hipError_t rmsnorm(int dtype, const float* x, int d, float eps, int rows, const int32_t* pos, int n_pos, int seq,
                   void* out, hipStream_t s) {
  if (d % 4 || d > kNormChunks * kRowThreads * 4) return hipErrorInvalidValue;
  if (dtype)
    hipLaunchKernelGGL(rmsnorm_kernel<bf16_t>, dim3(rows), dim3(kRowThreads), 0, s, x, d, eps, pos, n_pos, seq,
                       static_cast<bf16_t*>(out));
  else
    hipLaunchKernelGGL(rmsnorm_kernel<float>, dim3(rows), dim3(kRowThreads), 0, s, x, d, eps, pos, n_pos, seq,
                       static_cast<float*>(out));
  return hipGetLastError();
}

hipError_t resid_rmsnorm(int dtype, const float* part, int splits, int np, int M, float* x, int d, float eps,
                         int rows, const int32_t* pos, int n_pos, int seq, void* out, hipStream_t s) {
  if (d % 4 || np % 4 || d > kNormChunks * kRowThreads * 4) return hipErrorInvalidValue;
  if (dtype)
    hipLaunchKernelGGL(resid_rmsnorm_kernel<bf16_t>, dim3(rows), dim3(kWideThreads), 0, s, part, splits, np, M, x, d,
                       eps, pos, n_pos, seq, static_cast<bf16_t*>(out));
  else
    hipLaunchKernelGGL(resid_rmsnorm_kernel<float>, dim3(rows), dim3(kWideThreads), 0, s, part, splits, np, M, x, d,
                       eps, pos, n_pos, seq, static_cast<float*>(out));
  return hipGetLastError();
}

hipError_t kv_store(int dtype, const void* k, const void* vt, int H, int seq, int hd, int vt_ld, void* ck,
                    void* cvt, int cap, int off, hipStream_t s) {
  const int nk = cdiv(cdiv(seq * hd * (dtype ? 2 : 4), 16), kCopyChunks * kRowThreads);
  if (hd % kVtRows) return hipErrorInvalidValue;
  const dim3 grid(H, nk + hd / kVtRows);
  const bool wide = (reinterpret_cast<uintptr_t>(ck) | reinterpret_cast<uintptr_t>(k)) % 16 == 0;
  if (dtype)
    hipLaunchKernelGGL(kv_store_kernel<bf16_t>, grid, dim3(kRowThreads), 0, s, static_cast<const bf16_t*>(k),
                       static_cast<const bf16_t*>(vt), seq, hd, vt_ld, static_cast<bf16_t*>(ck),
                       static_cast<bf16_t*>(cvt), cap, off, nk, wide);
  else
    hipLaunchKernelGGL(kv_store_kernel<float>, grid, dim3(kRowThreads), 0, s, static_cast<const float*>(k),
                       static_cast<const float*>(vt), seq, hd, vt_ld, static_cast<float*>(ck),
                       static_cast<float*>(cvt), cap, off, nk, wide);
  return hipGetLastError();
}

namespace {

// LM-head row t = c * n_lm + j reads position lm_pos[j] of sequence c: the
// shared sequence for c = 0, branch c-1's copy of the block for c >= 1 when
// the position lies in the block (else the shared row)
__global__ void packed_lm_rows_kernel(int S, int b0, int B, int R, const int32_t* __restrict__ lm_pos, int n_lm,
                                      int32_t* __restrict__ row, int32_t* __restrict__ src) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= R) return;
  const int c = t / n_lm;
  const int p = min(max(lm_pos[t - c * n_lm], 0), S - 1);
  row[t] = (c > 0 && p >= b0 && p < b0 + B) ? S + (c - 1) * B + (p - b0) : p;
  src[t] = p;
}

}  // namespace

hipError_t packed_lm_rows(int S, int b0, int B, int n_branch, const int32_t* lm_pos, int n_lm, int32_t* row,
                          int32_t* src, hipStream_t s) {
  const int R = (1 + n_branch) * n_lm;
  hipLaunchKernelGGL(packed_lm_rows_kernel, dim3(cdiv(R, 256)), dim3(256), 0, s, S, b0, B, R, lm_pos, n_lm, row,
                     src);
  return hipGetLastError();
}

}  // namespace dllm
