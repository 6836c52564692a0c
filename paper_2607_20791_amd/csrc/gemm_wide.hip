// GEMMs of many rows (prefill chunks, wide decode steps): Y = X W^T with X
// [M][K] (bf16) and W in the packed panel layout of gemm.hip.
//
// With hundreds of rows the matrix units and the LDS bound the GEMM, not the
// weights' stream.  A workgroup of four waves, one per SIMD, owns 256 rows x
// 128 columns, each wave 128 x 64 of them: per 16 k it reads six fragments from
// LDS for eight 32x32x16 MFMAs (the 128-row tiles of gemm.hip read ten per
// sixteen smaller ones and kept the LDS busy all the time).  X and W of a 64-k
// step (48 KiB) are copied straight into one of three LDS slots without passing
// through registers, up to two steps ahead, with one barrier per step.  The
// operands are swapped (D^T = W X^T), so that a lane holds four consecutive
// columns of a row and stores 16 bytes at a time.
//
// A row's arithmetic is bit for bit that of the other tiles: two 32x32x16 MFMAs
// over the lower and the upper 16 of 32 k add up as one 16x16x32 does (checked
// on random inputs on gfx950, with either operand order), and the k order and
// the splits are the same.
//
// Measured on one MI355X at 2048 rows of random bf16 inputs (8B-class layer): SwiGLU
// 392-399 us, 1.21-1.23 PFLOP/s, down projection 201-216 us, 1.11-1.20 (1.3-1.38 on
// zeros, so part of the rest is power; a library product of 8192^3 reaches 1.36).  Eight waves of
// 64 x 64 (LDS traffic 176 instead of 144 KiB a step), 256-column tiles on two
// LDS slots, a fourth weight slot and a wave that touches the weights ahead
// were no faster.
#include <algorithm>

#include "gemm_common.hpp"
#include "kernels.hpp"

namespace rgd {

namespace {

constexpr int kBM = 256, kBN = 128;  // rows and columns of a workgroup's tile
constexpr int kXBytes = kBM * kStep * 2;  // X of one 64-k step in LDS

// 1 KiB from global memory to LDS, 16 bytes a lane: base + off (per lane) +
// OFF to lds + DST + OFF + 16 * lane.  No register is written; the compiler does not count it.
// (m0 is reserved: the compiler never holds a value there across statements, which
// its warning is about, but orders its own uses of m0 by the clobber.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int DST, int OFF>
RGD_DEV void dma16(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%4" ::"v"(off), "s"(base),
               "s"(lds), "n"(DST), "n"(OFF)
               : "m0", "scc");
}
#pragma clang diagnostic pop
template <int A, int B, typename F>
RGD_DEV void static_for(F&& f) {
  if constexpr (A < B) {
    f(std::integral_constant<int, A>{});
    static_for<A + 1, B>(f);
  }
}
template <int N>
RGD_DEV void dma_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

RGD_DEV f32x16 mfma32x32x16(const u32x4& a, const u32x4& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <int MODE, bool SUM, bool KEYS>
__global__ __launch_bounds__(256, 1) void gemm_wide_kernel(GemmArgs a) {
  constexpr int NT = 2, BN = kBN, SLOTS = 3;
  constexpr int PW = NT;                        // panels a wave copies per step (of 4 NT)
  constexpr int STAGE = kXBytes + BN * kStep * 2;
  constexpr int LOADS = 8 + 2 * PW;             // LDS copies per thread and step
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, kh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int gx = blockIdx.x, gy = blockIdx.y;
  xcd_order(gx, gy);
  const int m0 = gy * kBM;
  const int nst = a.K / kStep;
  const int split = blockIdx.z;
  const int st0 = SUM || MODE != GEMM_STORE ? 0 : int((long long)split * nst / a.splits);
  const int st1 = SUM || MODE != GEMM_STORE ? nst : int((long long)(split + 1) * nst / a.splits);
  const int nseg = MODE == GEMM_LOGITS ? min(4, (a.N - gx * 512 + 63) / 64) : SUM ? a.splits : 1;
  const int T = MODE == GEMM_LOGITS ? nseg * nst : st1 - st0;

  __shared__ __attribute__((aligned(1024))) unsigned char lds[SLOTS * STAGE];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // weights copied by this wave: panel slots wave * PW + i (slots [0, 2 NT) are
  // the columns of waves wn = 0, the others those of wn = 1)
  const char* wp[PW];
  int ngrp = 1, grp = 0;
  const int grp_wn = gx * 8 + wn * 4;  // LOGITS: 64-column groups of this wave's columns
  if (MODE == GEMM_LOGITS) {
    ngrp = (a.N + 63) / 64;
    grp = gx * 8 + (wave >> 1) * 4;
  } else {
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const int ps = wave * PW + i, half = ps / (2 * NT), j = ps % (2 * NT);
      int si = 0, p;
      if (MODE == GEMM_SILU) {
        si = j / NT;
        p = (gx * 2 + half) * NT + j % NT;
      } else {
        p = (gx * 2 + half) * 2 * NT + j;
        if (a.nseg > 1 && p * 16 >= a.seg[1].n0) si = 1;
        if (a.nseg > 2 && p * 16 >= a.seg[2].n0) si = 2;
      }
      const int lp = min(p - a.seg[si].n0 / 16, (a.seg[si].n + 15) / 16 - 1);
      wp[i] = (const char*)a.seg[si].w + ((long long)lp * nst + st0) * 2048;
    }
  }
  // X: copy i of wave w fills rows (4 i + w) * 8 .. + 7; lane l row l >> 3 of
  // them, chunk (l & 7), which holds chunk (l & 7) ^ swizzle of the row
  const char* X = (const char*)a.x + (long long)st0 * (kStep * 2);
  uint32_t xoff[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = (4 * i + wave) * 8 + (lane >> 3);
    xoff[i] = uint32_t(min(m0 + r, a.M - 1)) * uint32_t(a.ldx) * 2u + ((lane & 7) ^ xswz1(r & 15)) * 16;
  }
  const uint32_t lane16 = lane * 16;
  // The copies of one step (8 of X, then 2 per weight panel) are requested in
  // order; the cp_ values are the step's sources and LDS slot, and move on to the next
  // step after the last copy (staying at step T - 1).
  const char* cp_x = X;
  const char* cp_w[PW];
#pragma unroll
  for (int i = 0; i < PW; ++i)
    cp_w[i] = MODE == GEMM_LOGITS ? (const char*)a.seg[0].w + (long long)min(grp, ngrp - 1) * nst * 8192 + ((wave & 1) * PW + i) * 2048
                                  : wp[i];
  const uint32_t dst0 = lds0 + wave * 1024, dstw = wave * (PW * 2048 - 1024);
  uint32_t cp_dst = dst0;
  int cp_t = 0, cp_st = 0, cp_g = grp;
  auto copy = [&](auto c_) __attribute__((always_inline)) {
    constexpr int c = decltype(c_)::value;
    if constexpr (c < 8) {
      dma16<c * 4096, 0>(cp_x, xoff[c], cp_dst);
    } else {
      constexpr int i = (c - 8) >> 1, h = (c - 8) & 1;
      dma16<kXBytes + i * 2048, h * 1024>(cp_w[i], lane16, cp_dst + dstw);
    }
    if constexpr (c == LOADS - 1) {
      const bool on = cp_t + 1 < T;
      int dx = on ? 128 : 0;
      long long dw = on ? (MODE == GEMM_LOGITS ? 8192 : 2048) : 0;
      cp_t += on;
      if (MODE == GEMM_LOGITS) {
        cp_st += on;
        if (cp_st == nst) {  // the next 64 columns (groups follow each other; past the last it is read again)
          cp_st = 0;
          dx = -128 * (nst - 1);
          if (++cp_g >= ngrp) dw = -8192ll * (nst - 1);
        }
      }
      cp_x += dx;
#pragma unroll
      for (int i = 0; i < PW; ++i) cp_w[i] += dw;
      cp_dst = cp_dst == dst0 + (SLOTS - 1) * STAGE ? dst0 : cp_dst + STAGE;
    }
  };

  // fragments of 16-k sub-step s = 2 h + q2: row / column l32, k = 16 (2 q2 + kh) + 8 h
  const int xrow = (wm * 128 + l32) * 128, xsw = xswz1(l32 & 15);
  const int wrow = kXBytes + (wn * 2 * NT + (l32 >> 4)) * 2048 + (16 * kh + (l32 & 15)) * 16;
  int xo[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) xo[s] = xrow + ((2 * (2 * (s & 1) + kh) + (s >> 1)) ^ xsw) * 16;
  u32x4 xf[2][4], wf[2][NT];
  auto xfrag = [&](uint32_t base, int s, int mt) -> u32x4 { return *(const u32x4*)(lds + base + xo[s] + mt * 4096); };
  auto wfrag = [&](uint32_t base, int s, int j) -> u32x4 {
    return *(const u32x4*)(lds + base + wrow + j * 4096 + (s >> 1) * 1024 + (s & 1) * 512);
  };

  f32x16 acc[4][NT];
  f32x16 v[SUM ? 4 : 1][SUM ? NT : 1];
  const int mrow = m0 + wm * 128 + l32;  // + 32 mt
  // columns of value 4 g + i of tile j: col0(j) + 8 g + 4 kh + i
  auto col0 = [&](int j) { return gx * BN + (wn * NT + j) * 32; };
  auto zero = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[mt][j][i] = 0.f;
  };

  static_for<0, LOADS>(copy);
  static_for<0, LOADS>(copy);
  // SUM: the splits' sums are added in split order, as the consumer of separate
  // partials does, to the residual stream or to -0 (which adds exactly)
  if (SUM) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int m = min(mrow + mt * 32, a.M - 1);
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = min(col0(j) + 8 * g + 4 * kh, a.N - 4);
          f32x4 y = {-0.f, -0.f, -0.f, -0.f};
          if (a.accumulate) y = *(const f32x4*)((const float*)a.y + (long long)m * a.ldy + n);
#pragma unroll
          for (int i = 0; i < 4; ++i) v[mt][j][4 * g + i] = y[i];
        }
    }
  }
  zero();
  dma_wait_barrier<(SLOTS - 2) * LOADS>();
  static_for<0, 3>(copy);
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) xf[0][mt] = xfrag(0, 0, mt);
#pragma unroll
  for (int j = 0; j < NT; ++j) wf[0][j] = wfrag(0, 0, j);

  float rmax[4];
  unsigned long long rkey[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    rmax[mt] = -INFINITY;
    rkey[mt] = 0ull;
  }
  auto flush = [&](int seg, bool last) __attribute__((always_inline)) {
    if (SUM) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int j = 0; j < NT; ++j) v[SUM ? mt : 0][SUM ? j : 0] += acc[mt][j];
      zero();
      if (!last) return;
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int m = mrow + mt * 32;
      if (MODE == GEMM_SILU) {
#pragma unroll
        for (int j = 0; j < NT / 2; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int n = (gx * 2 + wn) * NT * 16 + j * 32 + 8 * g + 4 * kh;
            float y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = silu(acc[mt][j][4 * g + i]) * acc[mt][j + NT / 2][4 * g + i];
            if (m < a.M && n < a.N)
              *(u32x2*)((bf16_t*)a.y + (long long)m * a.ldy + n) = u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
          }
      } else {
        float* Y = (float*)a.y + (MODE == GEMM_STORE && !SUM ? (long long)split * a.split_stride : 0ll) + (long long)m * a.ldy;
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int n = (MODE == GEMM_LOGITS ? (grp_wn + seg) * 64 + j * 32 : col0(j)) + 8 * g + 4 * kh;
            f32x4 y;
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = SUM ? v[SUM ? mt : 0][SUM ? j : 0][4 * g + i] : acc[mt][j][4 * g + i];
            if (m < a.M && n < a.N) *(f32x4*)(Y + n) = y;
            if (MODE == GEMM_LOGITS) {
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const float z = n < a.N ? y[i] : -INFINITY;
                rmax[mt] = fmaxf(rmax[mt], z);
                if (KEYS) {
                  unsigned long long k = ((unsigned long long)ordered_u32(y[i]) << 32) |
                                         (unsigned long long)(0xFFFFFFFFu - uint32_t(n + i));
                  k = n < a.N ? k : 0ull;
                  rkey[mt] = k > rkey[mt] ? k : rkey[mt];
                }
              }
            }
          }
      }
    }
    if (MODE == GEMM_LOGITS) zero();
  };

  // One 64-k step from LDS slot `base`: four 16-k sub-steps of eight MFMAs; the
  // fragments of the next sub-step are read while one runs.  Before the last
  // sub-step this wave has read all of the step: one barrier there makes the
  // next step (copied by all waves) readable and this slot free, which the
  // copies of the step after the next two then fill, spread evenly up to the
  // third sub-step of the next step.
  uint32_t base = 0;
  auto step = [&]() __attribute__((always_inline)) {
    const uint32_t nbase = base == (SLOTS - 1) * STAGE ? 0 : base + STAGE;
    static_for<0, 32>([&](auto f_) __attribute__((always_inline)) {
      constexpr int s = decltype(f_)::value >> 3, u = decltype(f_)::value & 7, cur = s & 1, nxt = cur ^ 1;
      if constexpr (s == 3 && u == 0) dma_wait_barrier<(SLOTS - 2) * LOADS>();
      if constexpr (u < NT) wf[nxt][u] = s < 3 ? wfrag(base, s + 1, u) : wfrag(nbase, 0, u);
      if constexpr (u < 4) xf[nxt][u] = s < 3 ? xfrag(base, s + 1, u) : xfrag(nbase, 0, u);
      if constexpr (u % 3 == 1) copy(std::integral_constant<int, (3 * (s + 1)) % 12 + u / 3>{});
      acc[u & 3][u >> 2] = mfma32x32x16(wf[cur][u >> 2], xf[cur][u & 3], acc[u & 3][u >> 2]);
      __builtin_amdgcn_sched_barrier(0);
    });
    base = nbase;
  };
  int t = 0;
#pragma unroll 1
  for (int seg = 0; seg < nseg; ++seg) {
    const int end = MODE == GEMM_LOGITS ? (seg + 1) * nst : SUM ? int((long long)(seg + 1) * nst / a.splits) : T;
#pragma unroll 1
    for (; t < end; ++t) step();
    flush(seg, seg + 1 == nseg);
  }
  // no copy may be in flight when the LDS is used again or given back
  dma_wait_barrier<0>();

  if (MODE == GEMM_LOGITS) {
    // one maximum (and argmax key) per row over the workgroup's 512 columns
    float* red = (float*)lds;                                     // [2][256]
    unsigned long long* redk = (unsigned long long*)(lds + 4096);  // [2][256]
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      rmax[mt] = fmaxf(rmax[mt], __shfl_xor(rmax[mt], 32, 64));
      if (KEYS) {
        const unsigned long long k = __shfl_xor(rkey[mt], 32, 64);
        rkey[mt] = k > rkey[mt] ? k : rkey[mt];
      }
      if (kh == 0) {
        red[wn * kBM + wm * 128 + mt * 32 + l32] = rmax[mt];
        if (KEYS) redk[wn * kBM + wm * 128 + mt * 32 + l32] = rkey[mt];
      }
    }
    __syncthreads();
    const int m = m0 + tid;
    if (m < a.M) {
      a.tilemax[(long long)m * a.ntiles + gx] = fmaxf(red[tid], red[kBM + tid]);
      if (KEYS) {
        const unsigned long long k0 = redk[tid], k1 = redk[kBM + tid];
        a.tilekey[(long long)m * a.ntiles + gx] = k0 > k1 ? k0 : k1;
      }
    }
  }
}

}  // namespace

// Shapes that the wide tiles take.  X goes to LDS in 16-byte copies with 32-bit
// offsets and Y is stored 16 bytes at a time; rows at other addresses stay with
// gemm.hip's ordinary loads and stores.
bool gemm_wide_fits(const GemmArgs& a) {
  if (a.M <= kWideRows || (long long)a.M * a.ldx * 2 >= (1ll << 31)) return false;
  if ((uintptr_t)a.x % 16 || a.ldx % 8 || (uintptr_t)a.y % 16 || a.ldy % 4 || a.N % 4) return false;
  for (int i = 1; i < a.nseg && a.mode == GEMM_STORE; ++i)
    if (a.seg[i].n0 % kBN) return false;
  return true;
}

static long long rounds(long long workgroups) { return (workgroups + 255) / 256; }

// Whether they are faster than the 128-row tiles of gemm.hip.  Both run in rounds
// of 256 workgroups (one per CU), so the rounds decide, with the time of a wide
// workgroup over that of one of the others.  Measured with cold weights (us, 128-row
// tiles / wide):
// * LM head, 1.4 (K 1024) to 1.6 (K 4096) times: vocabulary 128256, K 4096, 129-256
//   rows (2 rounds against 1) 309 / 275, 257-384 (3 / 2) 437 / 467, 513-640 (5 / 3)
//   707 / 693; vocabulary 32768, 129-512 rows (1 / 1) 135 / 160-200; 513 (2 / 1) 250 / 199.
// * SwiGLU, 0.75 times: 4096 x 14336, 256 rows (1 / 1) 74 / 67, 512 (2 / 2) 138 / 110;
//   3072 x 10752, 257-384 rows (1 / 2) 62 / 76; 1024 x 3584 (16 steps) 24 / 14.
// * Projections from 129 to 256 rows where a split has 24 or more steps to run (in a
//   256-row decode step the down projection 41 against 44 us; the QKV projection
//   with its 16 steps per split takes 34 against 27 there, the O projection 23
//   against 20).
// * Projections above 256 rows, 0.85 times a 256-column workgroup: K 4096 QKV 257-384
//   rows (2 / 2) 46 / 41, 513-640 (2 / 3) 50 / 57.  Splits of at most 8 steps, whose 128-row
//   workgroups are 128 columns wide and share a CU: K 2048 QKV 257-384 rows 20 / 21,
//   448 23 / 21; K 1024 QKV 512 rows 9.3 / 11.2, 1024 14.0 / 12.6.
bool gemm_wide_wins(const GemmArgs& a) {
  const long long M = a.M, nb = (M + 127) / 128, wb = (M + kBM - 1) / kBM;
  auto cols = [&](int c) { return (long long)(a.N + c - 1) / c; };
  if (a.mode == GEMM_LOGITS) return (26600 + a.K) * rounds(cols(512) * wb) <= 20000 * rounds(cols(512) * nb);
  if (a.mode == GEMM_SILU) return 3 * rounds(cols(64) * wb) <= 4 * rounds(cols(128) * nb);
  const int steps = a.K / kStep / a.splits;
  if (M <= kBM) return steps >= 24;
  const long long w = rounds(cols(128) * wb * a.splits);
  if (steps > 8) return 17 * w <= 20 * rounds(cols(256) * nb * a.splits);
  return 6 * 256 * w <= 5 * std::max(256ll, cols(128) * nb * a.splits);
}

// Whether a projection's workgroups run their splits one after the other and
// add them, instead of one workgroup per split writing a partial output that
// the consumer adds: the fewer, longer workgroups against the partials' traffic.
// Costs in units of 0.01 us: 70 for a 64-k step of a tile and 700 for the start and
// end of a workgroup that runs all splits, 75 and 300 for one of a single split,
// rounds of 256 workgroups, and the partials written and read at 4.4 TB/s.
// Measured (us, one after the other / partials, with their read): K 1024 QKV 1024 rows
// 20.7 / 18.9, 2048 22.2 / 35.2; K 2048 QKV 385 rows 32.6 / 30.4, 512 33.1 / 34.6; K
// 4096 QKV 1024 rows 57 / 90, O 59 / 95; down (K 14336) 1024 167 / 160, 2048 194 / 347.
bool gemm_sums_splits(const GemmArgs& a) {
  if (a.mode != GEMM_STORE || a.splits == 1 || a.M <= kBM || !gemm_wide_fits(a)) return false;
  const long long tiles = (long long)((a.N + kBN - 1) / kBN) * ((a.M + kBM - 1) / kBM), nst = a.K / kStep;
  const long long one = rounds(tiles) * (70 * nst + 700);
  const long long parts = rounds(tiles * a.splits) * (75 * nst / a.splits + 300) + (long long)a.splits * a.M * a.N * 8 / 44000;
  return one < parts;
}

hipError_t gemm_wide(const GemmArgs& a, hipStream_t s) {
  const int rb = (a.M + kBM - 1) / kBM;
  if (a.mode == GEMM_LOGITS) {
    const dim3 grid((a.N + 511) / 512, rb);
    if (a.tilekey)
      hipLaunchKernelGGL((gemm_wide_kernel<GEMM_LOGITS, false, true>), grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((gemm_wide_kernel<GEMM_LOGITS, false, false>), grid, dim3(256), 0, s, a);
  } else if (a.mode == GEMM_SILU) {
    hipLaunchKernelGGL((gemm_wide_kernel<GEMM_SILU, false, false>), dim3((a.N + 63) / 64, rb), dim3(256), 0, s, a);
  } else if (a.summed) {
    hipLaunchKernelGGL((gemm_wide_kernel<GEMM_STORE, true, false>), dim3((a.N + 127) / 128, rb), dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((gemm_wide_kernel<GEMM_STORE, false, false>), dim3((a.N + 127) / 128, rb, a.splits), dim3(256), 0, s,
                       a);
  }
  return hipGetLastError();
}

}  // namespace rgd
