// fp32 GEMMs of small fp32 models: Y = X W^T with X [M][K] and W [N][K], both
// row-major and used in place.
//
// At these sizes (a step of 16 rows at d = 256 reads a few MB that stay in the
// caches) a GEMM is bound by latency: by its chain of memory round trips, not
// by bytes or operations.  One workgroup owns 16 MT rows x 16 NC columns; KW
// waves per column tile take one contiguous part of K each, request 16 bytes per
// lane of X and W several 16-k groups ahead and multiply on
// v_mfma_f32_16x16x4_f32 (full fp32), and the parts are added through LDS in
// part order.  Measured at 16 rows (one thread per output element / this): K
// 256 N 512 34 / 3.5 us, K 1024 N 256 128 / 6.0 us, SwiGLU K 256 N 1024 64 / 4.4
// us, LM head N 8192 66 / 6.6 us; at 1024 rows SwiGLU 1880 / 20.5 us.
// KW depends on K alone, so a row's arithmetic does not depend on the number of
// rows.
#include "gemm_common.hpp"
#include "kernels.hpp"

namespace rgd {

namespace {

// Any shape and alignment: one thread per output element.
template <int MODE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs a) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  const int m = blockIdx.y;
  const float* x = (const float*)a.x + (long long)m * a.ldx;
  const int K = a.K;
  const bool ok = n < a.N;
  const int nc = min(n, a.N - 1);
  float acc = 0.f, acc2 = 0.f;
  if (MODE == GEMM_SILU) {
    const float* wg = (const float*)a.seg[0].w + (long long)nc * K;
    const float* wu = (const float*)a.seg[1].w + (long long)nc * K;
    for (int k = 0; k < K; ++k) {
      acc += x[k] * wg[k];
      acc2 += x[k] * wu[k];
    }
    if (ok) ((float*)a.y)[(long long)m * a.ldy + n] = silu(acc) * acc2;
    return;
  }
  int si = 0;
  if (a.nseg > 1 && nc >= a.seg[1].n0) si = 1;
  if (a.nseg > 2 && nc >= a.seg[2].n0) si = 2;
  const float* w = (const float*)a.seg[si].w + (long long)(nc - a.seg[si].n0) * K;
  for (int k = 0; k < K; ++k) acc += x[k] * w[k];
  float* Y = (float*)a.y;
  if (MODE == GEMM_STORE) {
    if (ok) Y[(long long)m * a.ldy + n] = acc;
  } else {
    if (ok) Y[(long long)m * a.ldy + n] = acc;
    // 64 consecutive columns form one wave: its max is that tile's max
    const float v = wave_max(ok ? acc : -INFINITY);
    if ((threadIdx.x & 63) == 0 && ok) a.tilemax[(long long)m * a.ntiles + n / 64] = v;
  }
}


// 16-k group g of a row or column: this lane's four consecutive k, zero from
// `end` on (K, or the end of the wave's part).  The load is unconditional from a
// clamped address: behind a branch the groups would be waited for one by one.
RGD_DEV f32x4 load_k4(const float* p, int g, int kq, int K, int end) {
  const int k = g * 16 + kq * 4;
  const f32x4 v = *(const f32x4*)(p + min(k, K - 4));
  return k < end ? v : f32x4{0.f, 0.f, 0.f, 0.f};
}

template <int MODE, int MT, int NC, int KW>
__global__ __launch_bounds__(NC * KW * 64) void gemm_f32_mfma_kernel(GemmArgs a) {
  constexpr int NTH = NC * KW * 64, NB = MODE == GEMM_SILU ? 2 : 1, COLS = NC * 16, PITCH = COLS + 4;
  constexpr int U = MT == 1 ? 4 : 2;  // 16-k groups requested together
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), ct = wave % NC, kw = wave / NC;
  const int m0 = blockIdx.y * (MT * 16), n0 = blockIdx.x * COLS;
  const int K = a.K;

  const float* wp[NB];
  {
    const int n = min(n0 + ct * 16 + l16, a.N - 1);
    if (MODE == GEMM_SILU) {
      wp[0] = (const float*)a.seg[0].w + (long long)n * K;
      wp[NB - 1] = (const float*)a.seg[1].w + (long long)n * K;
    } else {
      int si = 0;
      if (a.nseg > 1 && n >= a.seg[1].n0) si = 1;
      if (a.nseg > 2 && n >= a.seg[2].n0) si = 2;
      const float* w = (const float*)(si == 0 ? a.seg[0].w : si == 1 ? a.seg[1].w : a.seg[2].w);
      wp[0] = w + (long long)(n - (si == 0 ? a.seg[0].n0 : si == 1 ? a.seg[1].n0 : a.seg[2].n0)) * K;
    }
  }
  const float* xp[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) xp[mt] = (const float*)a.x + (long long)min(m0 + mt * 16 + l16, a.M - 1) * a.ldx;

  f32x4 acc[MT][NB];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[mt][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int ng = (K + 15) / 16, g1 = (kw + 1) * ng / KW, end = min(g1 * 16, K);
  for (int g0 = kw * ng / KW; g0 < g1; g0 += U) {
    f32x4 x[U][MT], w[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int b = 0; b < NB; ++b) w[u][b] = load_k4(wp[b], g0 + u, kq, K, end);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) x[u][mt] = load_k4(xp[mt], g0 + u, kq, K, end);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            acc[mt][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][b][i], x[u][mt][i], acc[mt][b], 0, 0, 0);
  }

  // lane (l16, kq) holds row l16 of each row tile, columns 4 kq + {0..3}
  __shared__ __attribute__((aligned(16))) float red[KW][NB][MT * 16][PITCH];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int b = 0; b < NB; ++b) *(f32x4*)&red[kw][b][mt * 16 + l16][ct * 16 + kq * 4] = acc[mt][b];
  __syncthreads();
  for (int i = tid; i < MT * 16 * COLS; i += NTH) {
    const int r = i / COLS, c = i % COLS, m = m0 + r, n = n0 + c;
    float y[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      y[b] = red[0][b][r][c];
#pragma unroll
      for (int k = 1; k < KW; ++k) y[b] += red[k][b][r][c];
    }
    const bool ok = m < a.M && n < a.N;
    if (ok) ((float*)a.y)[(long long)m * a.ldy + n] = MODE == GEMM_SILU ? silu(y[0]) * y[NB - 1] : y[0];
    if (MODE == GEMM_LOGITS) {  // 64 columns: one wave per row
      const float v = wave_max(ok ? y[0] : -INFINITY);
      if (c == 0 && m < a.M) a.tilemax[(long long)m * a.ntiles + blockIdx.x] = v;
    }
  }
}

template <int MODE, int NC1, int NC4, int KW>
hipError_t launch_f32(const GemmArgs& a, hipStream_t s) {
  // up to 32 rows 16-row tiles and narrow workgroups (as many CUs as possible),
  // above them 64-row tiles
  if (a.M <= 32)
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<MODE, 1, NC1, KW>), dim3((a.N + 16 * NC1 - 1) / (16 * NC1), (a.M + 15) / 16),
                       dim3(NC1 * KW * 64), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<MODE, 4, NC4, KW>), dim3((a.N + 16 * NC4 - 1) / (16 * NC4), (a.M + 63) / 64),
                       dim3(NC4 * KW * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t gemm_f32(const GemmArgs& a, hipStream_t s) {
  // 16-byte loads along K need it and the row strides in whole float4s, aligned
  bool vec = a.K % 4 == 0 && a.ldx % 4 == 0 && (uintptr_t)a.x % 16 == 0;
  for (int i = 0; i < a.nseg; ++i) vec = vec && (uintptr_t)a.seg[i].w % 16 == 0;
  if (vec) {
    const bool deep = a.K > 512;
    switch (a.mode) {
      case GEMM_STORE: return deep ? launch_f32<GEMM_STORE, 1, 2, 8>(a, s) : launch_f32<GEMM_STORE, 1, 2, 4>(a, s);
      case GEMM_SILU: return deep ? launch_f32<GEMM_SILU, 1, 1, 8>(a, s) : launch_f32<GEMM_SILU, 1, 2, 4>(a, s);
      default: return launch_f32<GEMM_LOGITS, 4, 4, 4>(a, s);
    }
  }
  const dim3 grid((a.N + 255) / 256, a.M);
  switch (a.mode) {
    case GEMM_STORE:
      hipLaunchKernelGGL(gemm_f32_kernel<GEMM_STORE>, grid, dim3(256), 0, s, a); break;
    case GEMM_SILU:
      hipLaunchKernelGGL(gemm_f32_kernel<GEMM_SILU>, grid, dim3(256), 0, s, a); break;
    default:
      hipLaunchKernelGGL(gemm_f32_kernel<GEMM_LOGITS>, grid, dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace rgd
