// Per-row kernels of the decode step: embedding gather fused with the first
// RMSNorm, RMSNorm of the residual stream, and the Q/K/V epilogue (rotary
// embedding, store of q, append of k/v to the shared prefix or to the row's
// paged tail).
#include "kernels.hpp"
#include "rownorm.hpp"

namespace rgd {

namespace {

constexpr int kNormThreads = 1024;

__global__ __launch_bounds__(256) void copy_rows_kernel(const uint32_t* src, size_t stride, uint32_t* dst, int words) {
  const uint32_t* s = (const uint32_t*)((const char*)src + blockIdx.x * stride);
  for (int i = threadIdx.x; i < words; i += 256) dst[(size_t)blockIdx.x * words + i] = s[i];
}

template <typename T>
__global__ __launch_bounds__(kNormThreads) void embed_rmsnorm_kernel(const int* tok, int tok_stride,
                                                                   const int* tok_map, const T* E, int d, int V,
                                                                   float* x, const float* g, float eps, T* xn) {
  const int r = blockIdx.x;
  const long long src = tok_map ? tok_map[r] : r;
  embed_norm_row(tok[src * tok_stride], E, d, V, g, eps, x + (long long)r * d, xn + (long long)r * d);
}

// Logistic readout of one residual row per workgroup (fixed reduction order).
__global__ __launch_bounds__(256) void residual_readout_kernel(const float* x, long long row0, long long stride,
                                                               int d, const float* w, float b, float* out) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  const float* xr = x + (row0 + r * stride) * d;
  float acc = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) acc = fmaf(xr[i], w[i], acc);
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) out[r] = 1.0f / (1.0f + expf(-(acc + b)));
}

template <typename T>
__global__ __launch_bounds__(kNormThreads) void residual_rmsnorm_kernel(float* x, const float* parts, int nparts,
                                                                      long long part_stride, const float* g,
                                                                      float eps, int d, T* xn) {
  const int r = blockIdx.x;
  float* xr = x + (long long)r * d;
  const float* pr = parts + (long long)r * d;
  float4 v[kChunks], gg[kChunks];
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int i = (threadIdx.x + c * blockDim.x) * 4;
    v[c] = gg[c] = float4{0.f, 0.f, 0.f, 0.f};
    if (i < d) {
      float4 q[kMaxSplitK];
#pragma unroll
      for (int p = 0; p < kMaxSplitK; ++p)
        if (p < nparts) q[p] = *(const float4*)(pr + p * part_stride + i);
      v[c] = *(const float4*)(xr + i);
      gg[c] = *(const float4*)(g + i);
#pragma unroll
      for (int p = 0; p < kMaxSplitK; ++p)
        if (p < nparts) {
          v[c].x += q[p].x;
          v[c].y += q[p].y;
          v[c].z += q[p].z;
          v[c].w += q[p].w;
        }
      if (nparts > 0) store4(xr + i, v[c]);
    }
  }
  norm_store(v, gg, d, eps, xn + (long long)r * d);
}

// One workgroup per (row, kRopeThreads groups of W neighbouring rotation pairs
// (j, j + D/2) of the fused q|k|v output), one group per thread.  The rotation
// of position pos, pair j is (cos, sin) = rope_cs[pos][j] (a table computed once
// on the host in fp64).
// NP >= nparts: the loads of all NP split partials (clamped to the last one,
// masked by a 0/1 factor) and of the rotation are issued before any of them is
// used, so the kernel waits for memory once (a partial or a table load used
// only under a condition is moved into a branch by the compiler, which then
// waits for it where the branches join, one memory round trip each).
constexpr int kRopeThreads = 256;
// W = 4 from this many rows (Hq + 2 Hkv = 48 heads of 128, bf16; W 1 / W 4):
// 2048 rows 45.3 / 27.6 us, 256 rows 10.0 / 8.5; 64 rows 5.0 / 5.1, where the
// memory round trip is all there is and the short workgroups spread wider.
constexpr int kRopeWideRows = 128;

template <typename T, int NP, int W>
__global__ __launch_bounds__(kRopeThreads) void qkv_rope_kernel(const float* parts, int nparts, long long part_stride,
                                                                Rows rows, int Hq, int Hkv, int D,
                                                                const float2* rope_cs, int max_pos, T* q,
                                                                KVLayout kv) {
  typedef float vec __attribute__((ext_vector_type(W)));
  typedef float vec2 __attribute__((ext_vector_type(2 * W)));
  const int r = blockIdx.x;
  const int half = D / 2, groups = half / W;  // threads per head
  const int item = blockIdx.y * kRopeThreads + threadIdx.x;
  const int h = item / groups, j = item % groups * W;
  if (h >= Hq + 2 * Hkv) return;
  const int pos = min(rows.prefill ? rows.base_pos[r] : rows.base_pos[r] + rows.t, max_pos);
  const int nqkv = (Hq + 2 * Hkv) * D;
  const float* pr = parts + (long long)r * nqkv + h * D + j;
  // columns j .. j + W - 1 and the same + D/2, summed over the splits in split
  // order (split-K partials are finite, so the 0/1 factor masks them exactly)
  vec a1[NP], a2[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const float* pp = pr + min(p, nparts - 1) * part_stride;
    a1[p] = *(const vec*)pp;
    a2[p] = *(const vec*)(pp + half);
  }
  const vec2 cs = *(const vec2*)(rope_cs + (long long)pos * half + j);
  const int b = rows.prompt[r];
  vec x1 = a1[0], x2 = a2[0];
#pragma unroll
  for (int p = 1; p < NP; ++p) {
    const float f = p < nparts ? 1.f : 0.f;
    x1 += a1[p] * f;
    x2 += a2[p] * f;
  }
  // q and k pairs (j, j + D/2) are rotated, v passes through (cos 1, sin 0)
  const float kq = h < Hq + Hkv ? 1.f : 0.f;
  float y1[W], y2[W];
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const float c = cs[2 * i] * kq + (1.f - kq), sn = cs[2 * i + 1] * kq;
    // one rounding order for every W: a row's bits do not depend on the launch
    y1[i] = fmaf(x1[i], c, -(x2[i] * sn));
    y2[i] = fmaf(x2[i], c, x1[i] * sn);
  }
  // destinations: the dims of a K head lie side by side, those of a V head
  // vstride apart
  const int ps = kv.page_size;
  const int page = rows.prefill ? 0 : rows.pages[(long long)r * rows.max_pages + rows.t / ps];
  const int slot = rows.prefill ? 0 : rows.t % ps;
  if (h < Hq + Hkv) {
    T* dst;
    if (h < Hq) dst = q + ((long long)r * Hq + h) * D;
    else if (rows.prefill) dst = (T*)kv.prefix_k + (((long long)b * Hkv + h - Hq) * kv.P + pos) * D;
    else dst = (T*)kv.pool_k + (((long long)page * Hkv + h - Hq) * ps + slot) * D;
    if constexpr (W == 4) {
      store4(dst + j, float4{y1[0], y1[1], y1[2], y1[3]});
      store4(dst + j + half, float4{y2[0], y2[1], y2[2], y2[3]});
    } else {
      store_f(dst + j, y1[0]);
      store_f(dst + j + half, y2[0]);
    }
  } else {
    const int hv = h - Hq - Hkv;
    const long long vstride = rows.prefill ? 64 : ps;
    T* vd = rows.prefill ? (T*)kv.prefix_v + (((long long)b * Hkv + hv) * (kv.VP / 64) + pos / 64) * D * 64 + pos % 64
                         : (T*)kv.pool_v + ((long long)page * Hkv + hv) * D * ps + slot;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      store_f(vd + (j + i) * vstride, y1[i]);
      store_f(vd + (j + half + i) * vstride, y2[i]);
    }
  }
}

template <typename T, int W>
void launch_rope(const float* parts, int nparts, long long part_stride, const Rows& rows, int Hq, int Hkv, int D,
                 const float* rope_cs, int max_pos, T* q, const KVLayout& kv, hipStream_t s) {
  const dim3 grid(rows.R, ((Hq + 2 * Hkv) * (D / 2 / W) + kRopeThreads - 1) / kRopeThreads);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kRopeThreads), 0, s, parts, nparts, part_stride, rows, Hq, Hkv, D,
                       (const float2*)rope_cs, max_pos, q, kv);
  };
  if (nparts == 1) run(qkv_rope_kernel<T, 1, W>);
  else if (nparts <= 4) run(qkv_rope_kernel<T, 4, W>);
  else if (nparts <= 8) run(qkv_rope_kernel<T, 8, W>);
  else run(qkv_rope_kernel<T, kMaxSplitK, W>);
}

}  // namespace

template <typename T>
hipError_t embed_rmsnorm(const int* tok, int tok_stride, const int* tok_map, int R, const T* E, int d, int V,
                         float* x, const float* g, float eps, T* xn, hipStream_t s) {
  if (d % 4 || d > kChunks * 4 * kNormThreads) return hipErrorInvalidValue;
  hipLaunchKernelGGL(embed_rmsnorm_kernel<T>, dim3(R), dim3(kNormThreads), 0, s, tok, tok_stride, tok_map, E, d,
                     V, x, g, eps, xn);
  return hipGetLastError();
}

hipError_t copy_rows(const void* src, size_t stride, void* dst, size_t bytes, int n, hipStream_t s) {
  if (bytes % 4 || stride % 4 || n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(copy_rows_kernel, dim3(n), dim3(256), 0, s, (const uint32_t*)src, stride, (uint32_t*)dst,
                     (int)(bytes / 4));
  return hipGetLastError();
}

hipError_t residual_readout(const float* x, long long row0, long long stride, int nrows, int d, const float* w,
                            float b, float* out, hipStream_t s) {
  if (nrows <= 0) return hipSuccess;
  hipLaunchKernelGGL(residual_readout_kernel, dim3(nrows), dim3(256), 0, s, x, row0, stride, d, w, b, out);
  return hipGetLastError();
}

template <typename T>
hipError_t residual_rmsnorm(float* x, const float* parts, int nparts, long long part_stride, const float* g,
                            float eps, int R, int d, T* xn, hipStream_t s) {
  if (d % 4 || d > kChunks * 4 * kNormThreads || nparts < 0 || nparts > kMaxSplitK) return hipErrorInvalidValue;
  hipLaunchKernelGGL(residual_rmsnorm_kernel<T>, dim3(R), dim3(kNormThreads), 0, s, x, parts, nparts, part_stride,
                     g, eps, d, xn);
  return hipGetLastError();
}

template <typename T>
hipError_t qkv_rope_store(const float* parts, int nparts, long long part_stride, const Rows& rows, int Hq,
                          int Hkv, int D, const float* rope_cs, int max_pos, T* q, const KVLayout& kv,
                          hipStream_t s) {
  if (D > 256 || (D & 1) || nparts < 1 || nparts > kMaxSplitK) return hipErrorInvalidValue;
  const uintptr_t at = (uintptr_t)parts | (uintptr_t)q | (uintptr_t)kv.prefix_k | (uintptr_t)kv.pool_k;
  if (rows.R >= kRopeWideRows && D % 8 == 0 && part_stride % 4 == 0 && at % 16 == 0)
    launch_rope<T, 4>(parts, nparts, part_stride, rows, Hq, Hkv, D, rope_cs, max_pos, q, kv, s);
  else
    launch_rope<T, 1>(parts, nparts, part_stride, rows, Hq, Hkv, D, rope_cs, max_pos, q, kv, s);
  return hipGetLastError();
}

template hipError_t embed_rmsnorm<float>(const int*, int, const int*, int, const float*, int, int, float*, const float*,
                                         float, float*, hipStream_t);
template hipError_t embed_rmsnorm<bf16_t>(const int*, int, const int*, int, const bf16_t*, int, int, float*, const float*,
                                          float, bf16_t*, hipStream_t);
template hipError_t residual_rmsnorm<float>(float*, const float*, int, long long, const float*, float, int, int,
                                            float*, hipStream_t);
template hipError_t residual_rmsnorm<bf16_t>(float*, const float*, int, long long, const float*, float, int, int,
                                             bf16_t*, hipStream_t);
template hipError_t qkv_rope_store<float>(const float*, int, long long, const Rows&, int, int, int, const float*, int, float*,
                                          const KVLayout&, hipStream_t);
template hipError_t qkv_rope_store<bf16_t>(const float*, int, long long, const Rows&, int, int, int, const float*, int,
                                           bf16_t*, const KVLayout&, hipStream_t);

}  // namespace rgd
