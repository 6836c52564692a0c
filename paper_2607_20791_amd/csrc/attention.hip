// Decode attention over a shared prompt KV plus per-row tails.
//
// The prompt KV of one prompt is read by every row (probe or branch) of that
// prompt.  bf16 path: the shared part is split over (prefix split, KV head,
// row block); a workgroup streams 64-position K/V tiles of its split through
// LDS once and all query vectors of the row block (rows x the G query heads of
// the KV head, up to RGD_ATTN_QV) consume them with MFMA.  Scores are computed
// transposed, S^T = K Q^T, with the K rows gathered so that each lane ends up
// holding eight consecutive positions of one query vector; those feed
// O^T += V^T P^T directly as the B operand, and the V cache is kept
// head-dim-major (transposed per KV head) so that V^T fragments are plain
// 16-byte reads.  Online softmax runs in the exp2 domain with a lazily moved
// exponent reference.  A second kernel attends each row's own paged tail (also
// on MFMA) and merges it with the prefix-split (o, log-sum-exp) partials in a
// fixed order.
//
// fp32 path: vector kernels of the same structure (prefix splits, then tail
// plus merge).
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace rgd {

namespace {

constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLog2e = 1.4426950408889634f;

RGD_DEV f32x4 mfma16x16x32(const u32x4& a, const u32x4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

RGD_DEV uint32_t pack2(float lo, float hi) { return pack_bf16x2(lo, hi); }

// 2^x on the hardware unit, without the denormal range fix-up of exp2f:
// results below 2^-126 flush to zero, far below what a softmax weight in
// bf16 or an fp32 sum of them can resolve.
RGD_DEV float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

// Exponent headroom of the lazy softmax rescale (log2 units).
constexpr float kLazy = 8.f;
// Exponent reference of a query vector with no visible position yet: finite,
// so that s*scale - kNoRef is huge for a visible score and -inf (never NaN)
// for a masked one.
constexpr float kNoRef = -3.0e38f;

#ifndef RGD_ATTN_NW
#define RGD_ATTN_NW 8
#endif
// Fragment reads in flight + 1 in the tile loop's register ring (measured at
// 64 rows: 5 and 7 alike, 3 slower by 0.3 us, 9 and 16 slower still).
#ifndef RGD_ATTN_RING
#define RGD_ATTN_RING 5
#endif

// Log-sum-exp of one split of a query vector: m its exponent reference (log2 units),
// `weights` the sum of its weights.  Only a split with no visible position (weight
// sum 0) is left out of the merge: a weight sum that is not a number, from a NaN among
// the scores, enters like any other and makes the output NaN.
RGD_DEV float split_lse(float m, float weights) { return weights != 0.f ? (m + __log2f(weights)) * kLn2 : -INFINITY; }
// The partials of a row's prefix splits are combined by these weights relative to the
// largest log-sum-exp (over their sum), added in split order; the sum of the weights
// is that of a butterfly over 64 lanes, lane k holding split k.  The kernel that walks
// over all splits does the same in one lane per query vector, from log-sum-exps read
// back from LDS, so both give the same bits.
RGD_DEV float split_weight(float lse, float mx) { return lse == -INFINITY ? 0.f : __expf(lse - mx); }
RGD_DEV float merged_lse(float mx, float den) { return den > 0.f ? mx + __logf(den) : -INFINITY; }
// A split's normalised output in bf16 (bounded by max|V|; the merged output is bf16 as
// well), a row of D values: dims 16 dt + 4 grp + {0..3} of a prefix kernel lane sit at
// (dt / 2) * 32 + grp * 8 + (dt % 2) * 4, so that a lane stores 16 bytes at a time
// and the four lanes of a query vector 64 side by side.
RGD_DEV int part_slot(int dim) { return (dim >> 5) * 32 + ((dim >> 2) & 3) * 8 + ((dim >> 4) & 1) * 4 + (dim & 3); }

// K tiles sit in LDS as unpadded 256-byte rows whose 16-byte chunks are
// XOR-swizzled: chunk c of row r is stored at chunk c ^ kswz(r).  A fragment
// read touches rows {0..3, 8..11, 16..19, 24..27} (+ a multiple of 4) of a
// 32-row half, and kswz maps those to distinct chunk positions, so the reads
// are free of bank conflicts.
RGD_DEV int kswz(int r) { return (r & 3) | ((r >> 1) & 12); }

// V^T tiles sit in LDS as unpadded 128-byte rows (64 positions of one head
// dimension) whose 16-byte chunks are XOR-swizzled: chunk c of row r is stored
// at chunk c ^ vswz(r).  A fragment read (16 consecutive rows, one chunk each)
// and a tile store (8 lanes per row) are then free of bank conflicts by the
// LDS conflict counter; a padded 144-byte pitch, conflict-free on paper, was
// measured 2-way conflicted on the fragment reads.
RGD_DEV int vswz(int r) { return (r >> 1) & 7; }

// Row of a 64-position tile that lane l16 supplies as the A operand of score
// block (h, e).  With this order the score MFMA leaves lane (q, grp) holding
// positions h*32 + grp*8 + e*4 + {0..3}, i.e. eight consecutive positions per
// 32-position half: exactly the B operand layout of the P V product, and the
// matching V^T fragment is one contiguous 16-byte read.
RGD_DEV int k_gather_row(int h, int e, int l16) { return h * 32 + (l16 >> 2) * 8 + e * 4 + (l16 & 3); }

// Shared-prefix attention: one workgroup per (prefix split, KV head, block of
// up to RGD_ATTN_QV query vectors of one prompt).  The row blocks of one
// (split, KV head) are Hkv * splits workgroups apart in dispatch order, a
// multiple of the 8 XCDs the dispatcher deals workgroups to in turn, so they
// share one XCD's L2 for their common tiles.  NW waves each own NQ MFMA column
// tiles of 16 query vectors, so each K / V^T fragment read from LDS feeds NQ
// MFMAs and each 64-position tile is fetched from HBM once for all rows of the
// prompt.  The tile loop is software-pipelined: tiles are fetched into
// registers one tile ahead and stored into a ring of three LDS buffers, and
// the scores of tile t+1 are computed (MFMA) while the softmax of tile t runs
// on the vector units.  One barrier per tile.
//
// WALK: one workgroup per (KV head, row block) walks over all splits, closes each
// at its end as a separate workgroup would and merges them at the end, in the lanes
// that hold them: the first split's partial from LDS, those of the next kWalkRegs and
// the last one from registers, the rest read back from memory.  Rows whose prefix ends with
// the walk are written out, those with positions left for the tail kernel leave their
// merged partial (fp32) and its log-sum-exp as partial 0.  With more than four heads per
// KV head the tail kernel merges those rows itself, from all their partials.  2048 rows,
// 32 heads, 4096 positions, first / second half: 84 / 225 us, against 155 / 310 split
// and 115 / 140 for the merge of the partials.
constexpr int kMaxWalkSplits = 40;
// partials that a walk keeps in registers (two waves per SIMD, which the LDS allows, have
// 256 each; the kernel then uses all of them)
#ifndef RGD_WALK_REGS
#define RGD_WALK_REGS 5
#endif
constexpr int kWalkRegs = RGD_WALK_REGS;
static_assert(kWalkRegs >= 1, "merged fp32 partials take the place of the bf16 partials of splits 0 and 1");
static_assert(kMaxWalkSplits <= 48, "the walk adds its weights as 16 sums of three");

template <int NW, int NQ, bool WALK>
__global__ __launch_bounds__(NW * 64) void attn_prefix_kernel(AttnArgs a, bf16_t* out) {
  constexpr int D = 128, TP = 64, NT = NW * 64, NB = 3;
  static_assert(NW * NQ * 16 == RGD_ATTN_QV, "a workgroup covers RGD_ATTN_QV query vectors");
  const int s = WALK ? 0 : blockIdx.x, g = blockIdx.y;
  // the row block comes with the arguments (walks: the last, longest ones first)
  const int4 rb = a.rblk[WALK ? gridDim.z - 1 - blockIdx.z : blockIdx.z];
  const int r0 = rb.x, nr = rb.y, b = rb.z, maxplen = rb.w;
  const int lo = s * a.split_len;
  const int hi = WALK ? prefix_part_end(maxplen, a.split_len) : min(lo + a.split_len, maxplen);
  const int G = a.Hq / a.Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, grp = lane >> 4;
  const int nq = nr * G;

  // B operand of the score MFMA: lane (q, grp) holds dims ks*32 + grp*8 + {0..7}
  u32x4 qf[NQ][4];
  bool vok[NQ];
  int vrow[NQ], vhead[NQ], vend[NQ];
  // Q fragments first (unconditional loads: a query vector past the block
  // reads row r0 and is zeroed), then the visible ends, whose loads then do
  // not hold up the Q loads
  int pl[NQ];
#pragma unroll
  for (int nt = 0; nt < NQ; ++nt) {
    const int v = wave * NQ * 16 + nt * 16 + l16;
    vok[nt] = v < nq;
    vrow[nt] = r0 + (vok[nt] ? v / G : 0);
    vhead[nt] = g * G + (vok[nt] ? v % G : 0);
    const bf16_t* qp = (const bf16_t*)a.q + ((long long)vrow[nt] * a.Hq + vhead[nt]) * D + grp * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qf[nt][ks] = *(const u32x4*)(qp + ks * 32);
    pl[nt] = a.rows.plen[vrow[nt]];
  }
  // the visible ends are formed after the prologue's barrier (their loads are
  // long back by then; waiting for them here would hold up the first tile)
  auto set_vend = [&]() {
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        if (!vok[nt]) qf[nt][ks] = u32x4{0u, 0u, 0u, 0u};
      vend[nt] = vok[nt] ? min(prefix_part_end(pl[nt], a.split_len), hi) : lo;
    }
  };
  const bool wave_active = (wave * NQ * 16) < nq;

  __shared__ __attribute__((aligned(16))) bf16_t k_lds[NB][TP * D];
  __shared__ __attribute__((aligned(16))) bf16_t v_lds[NB][D][TP];

  // this (prompt, KV head): K rows [P][D]; V in 64-position blocks [VP/64][D][64]
  const long long bg = (long long)b * a.Hkv + g;
  const bf16_t* kbase = (const bf16_t*)a.kv.prefix_k + bg * a.kv.P * D;
  const bf16_t* vbase = (const bf16_t*)a.kv.prefix_v + bg * a.kv.VP * D;
  const float scale = rsqrtf(float(D)) * kLog2e;

  // m: exponent reference (log2 units) of a query vector; kNoRef until some
  // position of it is visible.  lacc: running sum of its weights, produced by
  // the P V MFMA against an all-ones A operand (every element holds the sum,
  // taken over the same bf16 weights as the output).
  float m[NQ];
  f32x4 o[8][NQ], lacc[NQ];
#pragma unroll
  for (int nt = 0; nt < NQ; ++nt) {
    m[nt] = kNoRef;
    lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[dt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // WALK: log-sum-exps of the closed splits, their largest, and the first split's partials
  __shared__ float walk_lse[WALK ? kMaxWalkSplits : 1][WALK ? RGD_ATTN_QV : 1];
  __shared__ u32x4 walk_p0[WALK ? NQ * 4 * NT : 1];
  u32x4 walk_p[WALK ? kWalkRegs : 1][NQ][4];  // partials of the next kWalkRegs splits
  float wmx[NQ];
#pragma unroll
  for (int nt = 0; nt < NQ; ++nt) wmx[nt] = -INFINITY;
  const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};  // bf16 1.0 x 8

  // Register staging of the next tile.  Nothing reads these registers before
  // store_tile, so the loads stay in flight through a whole tile of compute;
  // zeroing of V past the range (whose cache contents are arbitrary) is done
  // at the store.
  constexpr int KSEG = TP * 16 / NT, VSEG = D * (TP / 8) / NT;  // 16-byte segments per thread
  u32x4 kreg[KSEG], vreg[VSEG];
  int vt0 = 0;
  // The loads are unconditional (a predicated load makes the compiler wait
  // for it where the branches join): K rows past the range read row hi - 1
  // (their scores are masked), V of the tile's 64-position block is in the
  // padded cache and is zeroed past the range at the store.
  auto load_tile = [&](int t0) {
    vt0 = t0;
    const bf16_t* vblk = vbase + (long long)(t0 / TP) * D * TP;
#pragma unroll
    for (int i = 0; i < KSEG; ++i) {
      const int seg = threadIdx.x + i * NT;
      const int pos = min(t0 + (seg >> 4), hi - 1);
      kreg[i] = *(const u32x4*)(kbase + (long long)pos * D + (seg & 15) * 8);
    }
#pragma unroll
    for (int i = 0; i < VSEG; ++i) {
      const int seg = threadIdx.x + i * NT;
      vreg[i] = *(const u32x4*)(vblk + (seg >> 3) * TP + (seg & 7) * 8);
    }
  };
  auto store_tile = [&](int buf) {
#pragma unroll
    for (int i = 0; i < KSEG; ++i) {
      const int seg = threadIdx.x + i * NT;
      const int row = seg >> 4;
      *(u32x4*)&k_lds[buf][row * D + (((seg & 15) ^ kswz(row)) * 8)] = kreg[i];
    }
    if (vt0 + TP <= hi) {
#pragma unroll
      for (int i = 0; i < VSEG; ++i) {
        const int seg = threadIdx.x + i * NT, row = seg >> 3;
        *(u32x4*)&v_lds[buf][row][((seg & 7) ^ vswz(row)) * 8] = vreg[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < VSEG; ++i) {
        const int seg = threadIdx.x + i * NT, row = seg >> 3;
        const int nv = hi - (vt0 + (seg & 7) * 8);  // valid positions of this segment
        u32x4 vv = vreg[i];
#pragma unroll
        for (int w = 0; w < 4; ++w) vv[w] &= nv >= 2 * w + 2 ? 0xFFFFFFFFu : (nv == 2 * w + 1 ? 0xFFFFu : 0u);
        *(u32x4*)&v_lds[buf][row][((seg & 7) ^ vswz(row)) * 8] = vv;
      }
    }
  };

  // The tile loop works on 32-position halves.  Scores of half hh of the tile
  // in buffer buf: sc[e][nt][i] is position hh*32 + grp*8 + e*4 + i.
  auto k_frag = [&](int buf, int hh, int e, int ks) -> u32x4 {
    const int row = k_gather_row(hh, e, l16);
    return *(const u32x4*)&k_lds[buf][row * D + (((ks * 4 + grp) ^ kswz(row)) * 8)];
  };
  // V^T fragment: lane (l16, grp) reads row dt*16 + l16 at positions hh*32 + grp*8 + {0..7}
  auto v_frag = [&](int buf, int dt, int hh) -> u32x4 {
    const int row = dt * 16 + l16;
    return *(const u32x4*)&v_lds[buf][row][((hh * 4 + grp) ^ vswz(row)) * 8];
  };
  auto scores = [&](int buf, int hh, f32x4 (&sc)[2][NQ]) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
#pragma unroll
      for (int nt = 0; nt < NQ; ++nt) sc[e][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const u32x4 ka = k_frag(buf, hh, e, ks);
#pragma unroll
        for (int nt = 0; nt < NQ; ++nt) sc[e][nt] = mfma16x16x32(ka, qf[nt][ks], sc[e][nt]);
      }
    }
  };

  // Masking, exponent arguments and the exponent reference of a half starting
  // at position p0; on return sc holds the base-2 exponents s*scale - m.
  // Positions past a query vector's end are masked (skipped when the half is
  // visible to every query vector of the wave).  Lazy rescaling: the
  // reference m of a query vector only moves when some score exceeds it by
  // more than kLazy, so weights stay below 2^kLazy and the accumulators are
  // rescaled on few halves.  The common path needs no cross-lane reduction:
  // each lane tests its own exponents (results of arithmetic, so their
  // maximum needs no NaN quieting), and only when some lane of the wave fails
  // are the raw maxima reduced over the four lane groups that share a query
  // vector.  A vector with no visible position yet has m = kNoRef: its
  // exponents are huge (a move) for visible scores and -inf for masked ones.
  auto prepare = [&](int p0, f32x4 (&sc)[2][NQ]) {
    bool full = true;
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt) full &= p0 + 32 <= vend[nt];
    if (!__all(full)) {
#pragma unroll
      for (int nt = 0; nt < NQ; ++nt)
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (p0 + grp * 8 + e * 4 + i >= vend[nt]) sc[e][nt][i] = -INFINITY;
    }
    f32x4 t[2][NQ];
    bool grow = false;
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt) {
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) t[e][nt][i] = fmaf(sc[e][nt][i], scale, -m[nt]);
      const float x = fmaxf(fmaxf(fmaxf(t[0][nt][0], t[0][nt][1]), fmaxf(t[0][nt][2], t[0][nt][3])),
                            fmaxf(fmaxf(t[1][nt][0], t[1][nt][1]), fmaxf(t[1][nt][2], t[1][nt][3])));
      grow |= x > kLazy;
    }
    if (__any(grow)) {
#pragma unroll
      for (int nt = 0; nt < NQ; ++nt) {
        float x = fmaxf(fmaxf(fmaxf(sc[0][nt][0], sc[0][nt][1]), fmaxf(sc[0][nt][2], sc[0][nt][3])),
                        fmaxf(fmaxf(sc[1][nt][0], sc[1][nt][1]), fmaxf(sc[1][nt][2], sc[1][nt][3]))) * scale;
        x = fmaxf(x, __shfl_xor(x, 16, 64));
        x = fmaxf(x, __shfl_xor(x, 32, 64));
        // only a query vector whose own maximum passed its reference by more
        // than kLazy moves: its arithmetic never depends on the other query
        // vectors of the wave (rows batched together give the same results)
        if (x > m[nt] + kLazy) {
          const float alpha = exp2_raw(m[nt] - x);  // 0 when moving from kNoRef
          lacc[nt] *= alpha;
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) o[dt][nt] *= alpha;
          m[nt] = x;
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) t[e][nt][i] = fmaf(sc[e][nt][i], scale, -x);
        }
      }
    }
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt) {
      sc[0][nt] = t[0][nt];
      sc[1][nt] = t[1][nt];
    }
  };

  // One straight-line stream per half: the scores of the following half
  // (buffer kb, half kh, into nxt), the exponentials of this half (cur)
  // interleaved with them, then this half's P V product (buffer vb, half vh).
  // The 16 fragment reads go through a register ring of RD slots, NQ MFMAs
  // each; the caller primes the ring before the half's softmax preparation so
  // that those reads overlap it, and every step ends in a scheduling barrier,
  // so that the reads stay RD - 1 steps ahead of their MFMAs as written (left
  // alone, the scheduler moves each read next to its use and the MFMAs wait
  // for LDS).  The two score blocks alternate, so consecutive score MFMAs are
  // independent.  After the last half kb holds stale data and nxt is simply
  // not used.
  constexpr int RD = RGD_ATTN_RING;  // fragment reads in flight + 1
  auto frag = [&](int kb, int kh, int vb, int vh, int f) -> u32x4 {
    return f < 8 ? k_frag(kb, kh, f & 1, f >> 1) : v_frag(vb, f - 8, vh);
  };
  auto prime = [&](int kb, int kh, int vb, int vh, u32x4 (&ring)[RD]) {
#pragma unroll
    for (int f = 0; f + 1 < RD; ++f) ring[f] = frag(kb, kh, vb, vh, f);
  };
  auto stream = [&](int kb, int kh, int vb, int vh, f32x4 (&cur)[2][NQ], f32x4 (&nxt)[2][NQ], u32x4 (&ring)[RD]) {
    float plo[NQ];
    uint32_t pw[NQ][4];  // packed weights, word 2e + (i >> 1)
#pragma unroll
    for (int f = 0; f < 16; ++f) {
      if (f + RD - 1 < 16) ring[(f + RD - 1) % RD] = frag(kb, kh, vb, vh, f + RD - 1);
      if (f < 8) {
        const int e = f & 1, ks = f >> 1;
        if (ks == 0) {
#pragma unroll
          for (int nt = 0; nt < NQ; ++nt) nxt[e][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int nt = 0; nt < NQ; ++nt) nxt[e][nt] = mfma16x16x32(ring[f % RD], qf[nt][ks], nxt[e][nt]);
        // step f exponentiates value i = f & 3 of block ce = f >> 2 of this
        // half; pairs are packed to bf16 as soon as both halves exist
        const int ce = f >> 2, i = f & 3;
#pragma unroll
        for (int nt = 0; nt < NQ; ++nt) {
          const float x = exp2_raw(cur[ce][nt][i]);
          if (i & 1) pw[nt][ce * 2 + (i >> 1)] = pack2(plo[nt], x);
          else plo[nt] = x;
        }
      } else {
        const int dt = f - 8;
#pragma unroll
        for (int nt = 0; nt < NQ; ++nt)
          o[dt][nt] = mfma16x16x32(ring[f % RD], u32x4{pw[nt][0], pw[nt][1], pw[nt][2], pw[nt][3]}, o[dt][nt]);
        if (dt == 7) {
#pragma unroll
          for (int n2 = 0; n2 < NQ; ++n2)
            lacc[n2] = mfma16x16x32(ones, u32x4{pw[n2][0], pw[n2][1], pw[n2][2], pw[n2][3]}, lacc[n2]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // the partial of the split just done: word pair dt % 2 of p[dt / 2]
  auto pack_split = [&](int nt, u32x4 (&p)[4]) __attribute__((always_inline)) {
    const float lt = lacc[nt][0], inv = lt > 0.f ? 1.0f / lt : 0.f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      p[dt >> 1][(dt & 1) * 2] = pack2(o[dt][nt][0] * inv, o[dt][nt][1] * inv);
      p[dt >> 1][(dt & 1) * 2 + 1] = pack2(o[dt][nt][2] * inv, o[dt][nt][3] * inv);
    }
  };
  auto part_at = [&](int sp, int nt) {
    return (bf16_t*)a.part_o + (((long long)sp * a.rows.R + vrow[nt]) * a.Hq + vhead[nt]) * D + grp * 8;
  };
  auto write_part = [&](int sp, int nt, const u32x4 (&p)[4]) __attribute__((always_inline)) {
    bf16_t* po = part_at(sp, nt);
#pragma unroll
    for (int j = 0; j < 4; ++j) *(u32x4*)(po + j * 32) = p[j];
    if (grp == 0) a.part_lse[((long long)sp * a.rows.R + vrow[nt]) * a.Hq + vhead[nt]] = split_lse(m[nt], lacc[nt][0]);
  };
  auto ends_here = [&](int nt) { return prefix_part_end(pl[nt], a.split_len) == pl[nt]; };
  auto merges = [&](int nt) { return G <= 4 || ends_here(nt); };
  auto lse_slot = [&](int nt) { return WALK ? (wave * NQ + nt) * 16 + l16 : 0; };
  auto p0_slot = [&](int nt, int j) { return WALK ? ((wave * NQ + nt) * 4 + j) * 64 + lane : 0; };
  // WALK: ends split sp, which is not the last
  auto close_split = [&](int sp) __attribute__((always_inline)) {
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt) {
      const float lse = split_lse(m[nt], lacc[nt][0]);
      u32x4 p[4];
      pack_split(nt, p);
      if (sp == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) walk_p0[p0_slot(nt, j)] = p[j];
      }
#pragma unroll
      for (int i = 0; i < (WALK ? kWalkRegs : 0); ++i)
        if (sp == 1 + i) {
#pragma unroll
          for (int j = 0; j < 4; ++j) walk_p[i][nt][j] = p[j];
        }
      if (vok[nt] && (sp > kWalkRegs || !merges(nt))) write_part(sp, nt, p);
      if (grp == 0) walk_lse[WALK ? sp : 0][lse_slot(nt)] = lse;
      wmx[nt] = fmaxf(wmx[nt], lse);
      m[nt] = kNoRef;
      lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) o[dt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  const int ntile = hi > lo ? (hi - lo + TP - 1) / TP : 0;
  // The loop is reached only through the prologue, whose first store waits for
  // every earlier load (the Q fragments included), so no wait for them is
  // needed inside the loop.
  const int tiles_split = a.split_len / TP;
  if (ntile > 0) {
    load_tile(lo);
    store_tile(0);
    if (ntile > 1) load_tile(lo + TP);
    __syncthreads();
    set_vend();
    f32x4 sa[2][NQ], sb[2][NQ];
    if (wave_active) scores(0, 0, sa);
    // tile t uses ring buffer t % NB; the loop is unrolled by NB so that every
    // buffer index is a constant (LDS offsets fold into the instructions)
    auto tile = [&](int t, auto cbc) {
      constexpr int cb = decltype(cbc)::value, nb = (cb + 1) % NB;
      const int t0 = lo + t * TP;
      if (t + 1 < ntile) {  // publish tile t+1
        store_tile(nb);
        if (t + 2 < ntile) load_tile(t0 + 2 * TP);
      }
      __syncthreads();
      if (wave_active) {
        u32x4 ring[RD];
        prime(cb, 1, cb, 0, ring);
        prepare(t0, sa);
        stream(cb, 1, cb, 0, sa, sb, ring);
        prime(nb, 0, cb, 1, ring);
        prepare(t0 + 32, sb);
        stream(nb, 0, cb, 1, sb, sa, ring);
        if (WALK && (t + 1) % tiles_split == 0 && t + 1 < ntile) close_split(t / tiles_split);  // uniform
      }
    };
    static_assert(NB == 3, "the tile loop is unrolled by the number of LDS tile buffers");
    for (int t = 0; t < ntile; t += NB) {
      tile(t, std::integral_constant<int, 0>{});
      if (t + 1 < ntile) tile(t + 1, std::integral_constant<int, 1>{});
      if (t + 2 < ntile) tile(t + 2, std::integral_constant<int, 2>{});
    }
  }

  if constexpr (!WALK) {
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt) {
      u32x4 p[4];
      pack_split(nt, p);
      if (vok[nt]) write_part(s, nt, p);
    }
  } else {
    const int ns = (ntile + tiles_split - 1) / tiles_split;
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt)
      if (grp == 0) walk_lse[ns - 1][lse_slot(nt)] = split_lse(m[nt], lacc[nt][0]);
    __syncthreads();
#pragma unroll
    for (int nt = 0; nt < NQ; ++nt) {
      if (!vok[nt]) continue;
      u32x4 pn[4];
      pack_split(nt, pn);
      if (!merges(nt)) {
        write_part(ns - 1, nt, pn);
        continue;
      }
      // (log-sum-exps come back from LDS: in registers, lse - max would be fused with the
      // product that lse ends in, unrounded)
      const float* lses = &walk_lse[0][lse_slot(nt)];
      const float mx = fmaxf(wmx[nt], lses[(ns - 1) * RGD_ATTN_QV]);
      auto weight = [&](int k) { return k < ns ? split_weight(lses[min(k, ns - 1) * RGD_ATTN_QV], mx) : 0.f; };
      // the sum over 64 lanes halved 32, 16, 8, 4, 2, 1 apart (kMaxWalkSplits <= 48)
      float d[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        d[k] = weight(k);
        if (ns > 32) d[k] += weight(k + 32);
        if (ns > 16) d[k] += weight(k + 16);
      }
#pragma unroll
      for (int h = 8; h > 0; h >>= 1)
#pragma unroll
        for (int k = 0; k < h; ++k) d[k] += d[k + h];
      const float inv = d[0] > 0.f ? 1.f / d[0] : 0.f;
      f32x4 y[8];
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) y[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
      auto add = [&](int k, const u32x4 (&p)[4]) __attribute__((always_inline)) {
        const float lse = lses[k * RGD_ATTN_QV], wk = split_weight(lse, mx) * inv;
        if (lse == -INFINITY) return;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
#pragma unroll
          for (int w = 0; w < 2; ++w) {
            const uint32_t x = p[dt >> 1][(dt & 1) * 2 + w];
            y[dt][2 * w] = fmaf(wk, __uint_as_float(x << 16), y[dt][2 * w]);
            y[dt][2 * w + 1] = fmaf(wk, __uint_as_float(x & 0xFFFF0000u), y[dt][2 * w + 1]);
          }
      };
      if (ns > 1) {
        u32x4 p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) p[j] = walk_p0[p0_slot(nt, j)];
        add(0, p);
      }
#pragma unroll
      for (int i = 0; i < kWalkRegs; ++i)
        if (1 + i < ns - 1) add(1 + i, walk_p[i][nt]);
      // four splits' loads at a time
      for (int k0 = 1 + kWalkRegs; k0 < ns - 1; k0 += 4) {
        u32x4 p[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j) p[u][j] = *(const u32x4*)(part_at(min(k0 + u, ns - 2), nt) + j * 32);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (k0 + u < ns - 1) add(k0 + u, p[u]);
      }
      add(ns - 1, pn);
      const long long idx = (long long)vrow[nt] * a.Hq + vhead[nt];
      if (ends_here(nt)) {
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
          *(u32x2*)(out + idx * D + dt * 16 + grp * 4) = u32x2{pack2(y[dt][0], y[dt][1]), pack2(y[dt][2], y[dt][3])};
      } else {
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) *(f32x4*)(a.part_o + idx * D + dt * 16 + grp * 4) = y[dt];
        if (grp == 0) a.part_lse[idx] = merged_lse(mx, d[0]);
      }
    }
  }
}

// fp32 attention of small decoders, on the vector units.  A step reads a few
// hundred KB that sit in the caches, so both kernels are bound by their chain of
// memory round trips and barriers: four lanes share a position's K row and hold
// all their loads of it at once, the first V block is requested before the
// softmax, and one wave does a head's softmax without workgroup barriers.
// Measured at 16 rows, 64 prefix positions, up to 32 tail positions (a loop over
// the row with one load at a time, block-wide reductions / this): prefix 27.1 /
// 6.8 us, tail and merge 10.8 / 7.4 us; 1024 prefill rows 55.9 / 11.7 us.
constexpr int kChunk = 256;      // positions per prefix split and per tail block
constexpr int kMaxSplits = 40;

// four floats of a caller's K or V, which need not be aligned to 16 bytes
typedef f32x4 f32x4_any __attribute__((aligned(4)));

// 8 consecutive elements starting at p
RGD_DEV void load8(const float* p, float* out) {
  const f32x4 a = *(const f32x4_any*)p, b = *(const f32x4_any*)(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[i] = a[i];
    out[4 + i] = b[i];
  }
}

// q . k for n <= kChunk positions and G <= 8 heads into sc[h][position]:
// position p by lanes 4 p .. 4 p + 3, lane j the float4s j, j + 4, .. of the row.
// k_row(p) gives the row of position p.
template <int D, typename F>
RGD_DEV void f32_scores(const float (&qs)[8][D], float (&sc)[8][kChunk], int n, int G, float scale, F k_row) {
  constexpr int NV = (D + 15) / 16;
  const int j = threadIdx.x & 3;
  for (int p0 = 0; p0 < n; p0 += 64) {
    const int p = p0 + (threadIdx.x >> 2);
    const float* kr = k_row(min(p, n - 1));
    f32x4 k[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) k[i] = *(const f32x4_any*)(kr + min(j * 4 + i * 16, D - 4));
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      if (h >= G) break;
      float dot = 0.f;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const f32x4 q = *(const f32x4*)&qs[h][min(j * 4 + i * 16, D - 4)];
        const float t = q[0] * k[i][0] + q[1] * k[i][1] + q[2] * k[i][2] + q[3] * k[i][3];
        dot += j * 4 + i * 16 < D ? t : 0.f;
      }
      dot += __shfl_xor(dot, 1, 64);
      dot += __shfl_xor(dot, 2, 64);
      if (j == 0) sc[h][p] = p < n ? dot * scale : -INFINITY;
    }
  }
}

// One head's block of n scores by one wave: the block's exponentials relative to
// the new running maximum replace them; m and l are the running maximum and
// sum (alpha: factor of what was summed before).
RGD_DEV void f32_softmax(float (&sc)[kChunk], int n, float& m, float& l, float& alpha) {
  const int lane = threadIdx.x & 63;
  float v[kChunk / 64], mx = m;
#pragma unroll
  for (int i = 0; i < kChunk / 64; ++i) {
    const int p = lane + 64 * i;
    v[i] = p < n ? sc[p] : -INFINITY;
    mx = fmaxf(mx, v[i]);
  }
  mx = wave_max(mx);
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < kChunk / 64; ++i) {
    const int p = lane + 64 * i;
    const float e = v[i] == -INFINITY ? 0.f : __expf(v[i] - mx);
    if (p < n) sc[p] = e;
    sum += e;
  }
  alpha = m == -INFINITY ? 0.f : __expf(m - mx);
  l = l * alpha + wave_sum(sum);
  m = mx;
}

// acc[h] += weights * V of dimension d over blocks of 8 positions part * 8,
// + 8 * parts, ..; the first block's values are given.  v_at(p) points at the
// values of positions p .. p + 7 (values past n are not used).
template <int PARTS, typename F>
RGD_DEV void f32_weighted(const float (&sc)[8][kChunk], int n, int G, int part, float (&v)[8], float (&acc)[8], F v_at) {
  for (int b0 = part * 8; b0 < n; b0 += PARTS * 8) {
    float nv[8];
    load8(v_at(min(b0 + PARTS * 8, (n - 1) & ~7)), nv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float ve = b0 + e < n ? v[e] : 0.f;
#pragma unroll
      for (int h = 0; h < 8; ++h)
        if (h < G) acc[h] += sc[h][min(b0 + e, n - 1)] * ve;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = nv[e];
  }
}

// One workgroup per (prefix split, KV head, row).
template <int D>
__global__ __launch_bounds__(256) void attn_prefix_f32_kernel(AttnArgs a) {
  constexpr int PARTS = 256 / D;
  const int c = blockIdx.x, g = blockIdx.y, r = blockIdx.z;
  const int G = a.Hq / a.Hkv, tid = threadIdx.x, wave = tid >> 6;
  __shared__ __attribute__((aligned(16))) float qs[8][D];
  __shared__ float sc[8][kChunk];
  __shared__ float accx[PARTS][8][D];
  __shared__ float ml[2][8];
  const int lo = c * a.split_len, n = min(a.split_len, a.rows.plen[r] - lo);
  const long long bg = (long long)a.rows.prompt[r] * a.Hkv + g;
  const float* kp = (const float*)a.kv.prefix_k + (bg * a.kv.P + lo) * D;
  const int d = tid % D, part = tid / D;
  // (split lengths are multiples of 64: lo starts a 64-position V block)
  const float* vp = (const float*)a.kv.prefix_v + (bg * (a.kv.VP / 64) + lo / 64) * D * 64 + (long long)d * 64;
  auto v_at = [&](int p) -> const float* { return vp + (long long)(p >> 6) * D * 64 + (p & 63); };
  for (int i = tid; i < G * D; i += 256) qs[i / D][i % D] = ((const float*)a.q)[((long long)r * a.Hq + g * G) * D + i];
  float v[8], acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (n > 0) load8(v_at(min(part * 8, (n - 1) & ~7)), v);
  __syncthreads();
  if (n > 0) f32_scores<D>(qs, sc, n, G, rsqrtf(float(D)), [&](int p) { return kp + (long long)p * D; });
  __syncthreads();
  for (int h = wave; h < G; h += 4) {
    float m = -INFINITY, l = 0.f, alpha;
    if (n > 0) f32_softmax(sc[h], n, m, l, alpha);
    ml[0][h] = m;
    ml[1][h] = l;
  }
  __syncthreads();
  if (n > 0) f32_weighted<PARTS>(sc, n, G, part, v, acc, v_at);
#pragma unroll
  for (int h = 0; h < 8; ++h)
    if (h < G) accx[part][h][d] = acc[h];
  __syncthreads();
  for (int i = tid; i < G * D; i += 256) {
    const int h = i / D, dd = i % D;
    float o = 0.f;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) o += accx[p][h][dd];
    const float l = ml[1][h];
    const long long idx = ((long long)c * a.rows.R + r) * a.Hq + g * G + h;
    a.part_o[idx * D + dd] = l > 0.f ? o / l : 0.f;
    if (dd == 0) a.part_lse[idx] = l > 0.f ? ml[0][h] + __logf(l) : -INFINITY;
  }
}

// Tail attention fused with the merge of all partials: one workgroup per
// (row, KV head) attends the row's own tail in blocks of kChunk positions, then
// merges the prefix-split partials of its heads with it in log-sum-exp form, in
// a fixed order.
template <int D>
__global__ __launch_bounds__(256) void attn_tail_combine_kernel(AttnArgs a, float* out) {
  constexpr int PARTS = 256 / D, kPre = 16;
  const int r = blockIdx.x, g = blockIdx.y;
  const int G = a.Hq / a.Hkv, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const long long R = a.rows.R;
  __shared__ __attribute__((aligned(16))) float qs[8][D];
  __shared__ float sc[8][kChunk];
  __shared__ float accx[PARTS][8][D];
  __shared__ float al[8], wts[8][kMaxSplits + 1];  // merge weights; column `splits` is the tail
  const int S = a.splits, n_all = a.tail_len;
  for (int i = tid; i < G * D; i += 256)
    qs[i / D][i % D] = ((const float*)a.q)[((long long)r * a.Hq + g * G) * D + i] * rsqrtf(float(D));
  // the prefix-split partials do not depend on the tail: request them now (first
  // 16 splits, 2 (head, dim) pairs per thread), from clamped addresses
  const long long pstep = R * a.Hq * D;
  const float* po = a.part_o + ((long long)r * a.Hq + g * G) * D;
  float pre[2][kPre];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int sp = 0; sp < kPre; ++sp) pre[k][sp] = po[min(tid + k * 256, G * D - 1) + min(sp, S - 1) * pstep];

  const int ps = a.kv.page_size;
  const int* pages = a.rows.pages ? a.rows.pages + (long long)r * a.rows.max_pages : nullptr;
  const int d = tid % D, part = tid / D;
  auto k_at = [&](int pos) -> const float* {
    return (const float*)a.kv.pool_k + (((long long)pages[pos / ps] * a.Hkv + g) * ps + pos % ps) * D;
  };
  // 8 positions from a multiple of 8 lie inside one page (pages hold a multiple of 8)
  auto v_at = [&](int pos) -> const float* {
    return (const float*)a.kv.pool_v + (((long long)pages[pos / ps] * a.Hkv + g) * D + d) * ps + pos % ps;
  };
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};  // heads wave and wave + 4
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < n_all; c0 += kChunk) {
    const int n = min(kChunk, n_all - c0);
    float v[8];
    load8(v_at(c0 + min(part * 8, (n - 1) & ~7)), v);
    __syncthreads();  // q is there; the block before is done with sc
    f32_scores<D>(qs, sc, n, G, 1.f, [&](int p) { return k_at(c0 + p); });
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int h = wave + 4 * k;
      if (h < G) {
        float alpha;
        f32_softmax(sc[h], n, m[k], l[k], alpha);
        if (lane == 0) al[h] = alpha;
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 8; ++h)
      if (h < G) acc[h] *= al[h];
    f32_weighted<PARTS>(sc, n, G, part, v, acc, [&](int p) { return v_at(c0 + p); });
  }
#pragma unroll
  for (int h = 0; h < 8; ++h)
    if (h < G) accx[part][h][d] = acc[h];
  // merge weights of heads wave and wave + 4: lane sp holds split sp
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int h = wave + 4 * k;
    if (h >= G) continue;
    const float ls = a.part_lse[(min(lane, S - 1) * R + r) * a.Hq + g * G + h];
    const float lse = lane < S ? ls : -INFINITY;
    const float lt = l[k] > 0.f ? m[k] + __logf(l[k]) : -INFINITY;
    const float M = wave_max(fmaxf(lse, lt));
    const float w = lse == -INFINITY ? 0.f : __expf(lse - M), wt = lt == -INFINITY ? 0.f : __expf(lt - M);
    const float den = wave_sum(w) + wt, inv = den > 0.f ? 1.0f / den : 0.f;
    if (lane < S) wts[h][lane] = w * inv;
    if (lane == 0) wts[h][S] = l[k] > 0.f ? wt * inv / l[k] : 0.f;  // applied to the unnormalised tail sum
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < (8 * D + 255) / 256; ++k) {
    const int i = tid + k * 256;
    if (i >= G * D) break;
    const int h = i / D, dd = i % D;
    float tail = 0.f;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) tail += accx[p][h][dd];
    float o = wts[h][S] * tail;
    if (k < 2) {
#pragma unroll
      for (int sp = 0; sp < kPre; ++sp)
        if (sp < S) o += wts[h][sp] * pre[k & 1][sp];
    }
#pragma unroll 4
    for (int sp = k < 2 ? kPre : 0; sp < S; ++sp) o += wts[h][sp] * po[i + sp * pstep];
    out[((long long)r * a.Hq + g * G) * D + i] = o;
  }
}

// Tail attention fused with the merge, bf16 caches: one workgroup per (row, KV
// head).  The row's 32-position tiles (the last positions of its prefix, then its
// paged tail) are dealt to four lanes of work in turn (tile t to lane t % 4), each
// attended with MFMA into a state of its own: the G query heads of the KV head
// form one 16-column tile, K and V^T fragments are loaded straight from the pages
// (K rows in the gathered order of the prefix kernel, so every lane ends up with
// eight consecutive positions).  The four states are merged through LDS in a fixed
// order, and a head's output is written by one wave.  The merge is in log-sum-exp
// form.  The prefix-split partials of heads 0 .. 3 are combined into one first (of
// the wave's first head while its first tile is loading), which leaves a two-term merge
// with the tail after the exchange; the partials of further heads (G > 4) and their
// tail are merged in one go, eight splits' loads at a time (64 rows of an 8193-position
// prompt, 16 splits, 8 query heads per KV head, 64 tail positions: 48.7 us with the
// prefix kernel, 53 one load at a time).
// NWV: waves per workgroup.  Four take one lane of work each: the shortest chain,
// for few (row, head) pairs.  One takes all four in turn: a workgroup's start and
// merge cost more than a tile, and with enough pairs to fill the chip fewer, longer
// waves pay them once instead of four times.  Attention stage of 256 rows x 8 KV heads
// over 1024-position prompts, four waves / one: tails of 4 positions 56.9 / 47.9 us,
// 64 59.8 / 55.6, 200 84.4 / 81.9 (4.2 less since one wave takes rows of one partial
// only and fewer registers: 78.2 to 74.0 in the attention entry point).  The states and their merge are the same, so the
// bits are too.
// GM: query heads per KV head at most (LDS).
// ROWS: all rows (0), or those of a list that a walk leaves, with the partials of
// the splits that a row's prefix reaches (1) or one merged fp32 partial (2).
constexpr int kMergeMaxSplits = 64;

template <int ROWS, int NWV, int GM>
__global__ __launch_bounds__(NWV * 64) void attn_tail_merge_kernel(AttnArgs a, bf16_t* out, const int* rowlist) {
  constexpr int D = 128, TT = 32;
  const int r = ROWS ? rowlist[blockIdx.x] : blockIdx.x, g = blockIdx.y;
  const int G = a.Hq / a.Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, grp = lane >> 4;
  const long long R = a.rows.R;
  const int ps = a.kv.page_size;
  const float scale = rsqrtf(float(D)) * kLog2e;

  __shared__ float w_m[4][GM], w_l[4][GM];
  __shared__ __attribute__((aligned(16))) float w_o[4][GM][D + 4];  // [lane of work][query][dim]

  // First requests: the row's visible prefix length and its first 64 tail
  // page numbers (lane i holds page i), so that tile addresses need no
  // further dependent load.  Without tail pages a valid int array stands in.
  const int n = a.tail_len;
  const int* prow = n > 0 ? a.rows.pages + (long long)r * a.rows.max_pages : a.rows.plen;
  const int plen = a.rows.plen[r];
  const int pg_reg = prow[n > 0 ? min(lane, a.rows.max_pages - 1) : 0];
  const int ps_ = a.kv.page_size;
  const bool pg_in_regs = (n + ps_ - 1) / ps_ <= 64;  // uniform
  auto page_at = [&](int pi) -> int {
    return pg_in_regs ? __shfl(pg_reg, pi, 64) : prow[min(pi, a.rows.max_pages - 1)];
  };
  const int prompt = a.rows.prompt[r];

  // The prefix-split partials and log-sum-exps do not depend on the tail:
  // request those of this wave's first head now so their latency overlaps the
  // tail attention (splits beyond kPrefetch are loaded by the combine).
  const int S = a.splits;
  constexpr bool kOne = NWV == 1 || ROWS == 2;  // one partial per head
  constexpr int kPrefetch = ROWS == 2 ? 2 : NWV == 1 ? 1 : 16;
  const long long pstep = R * a.Hq * D;
  // (Loads in this kernel are unconditional, from clamped addresses, and
  // masked afterwards: a predicated load makes the compiler wait for it where
  // the branches join, one memory round trip each.)
  // (a wave past the G heads loads head G-1's and does not use them)
  uint32_t pre[kPrefetch];  // bf16 pairs (ROWS 2: the two fp32 values)
  float pre_lse;
  {
    const int head = g * G + min(wave, G - 1);
    const long long i0 = ((long long)r * a.Hq + head) * D;
    if constexpr (ROWS == 2) {
      const u32x2 v = *(const u32x2*)(a.part_o + i0 + 2 * lane);
      pre[0] = v[0];
      pre[1] = v[1];
      pre_lse = a.part_lse[(long long)r * a.Hq + head];
    } else {
      const bf16_t* po = (const bf16_t*)a.part_o + i0 + part_slot(2 * lane);
#pragma unroll
      for (int k = 0; k < kPrefetch; ++k) pre[k] = *(const uint32_t*)(po + min(k, S - 1) * pstep);
      pre_lse = a.part_lse[((long long)min(lane, S - 1) * R + r) * a.Hq + head];
    }
  }

  u32x4 qf[4];
  {
    const bool ok = l16 < G;
    const bf16_t* qp = (const bf16_t*)a.q + ((long long)r * a.Hq + g * G + (ok ? l16 : 0)) * D + grp * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const u32x4 x = *(const u32x4*)(qp + ks * 32);
      qf[ks] = ok ? x : u32x4{0u, 0u, 0u, 0u};
    }
  }
  const int pe = prefix_part_end(plen, a.split_len);
  const int nsp = ROWS == 1 ? (pe + a.split_len - 1) / a.split_len : S;  // splits with a partial
  auto lane_of = [&](float v, int k) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k)); };
  // o += the split partials of a head by their weights (lane k holds split k's), in
  // split order; a split without positions is left out
  auto add_splits = [&](const bf16_t* po, float lses, float w, float inv, bool first, float& o0, float& o1) {
    auto add = [&](int k, uint32_t v) {
      if (lane_of(lses, k) == -INFINITY) return;  // uniform
      const float wk = lane_of(w, k) * inv;
      o0 = fmaf(wk, __uint_as_float(v << 16), o0);
      o1 = fmaf(wk, __uint_as_float(v & 0xFFFF0000u), o1);
    };
    if (first) {
#pragma unroll
      for (int k = 0; k < kPrefetch; ++k)
        if (k < nsp) add(k, pre[k]);
    }
    if (S == 1) {
      if (!first) add(0, *(const uint32_t*)po);
      return;
    }
    // eight splits' loads at a time
    for (int k0 = first ? kPrefetch : 0; k0 < nsp; k0 += 8) {
      uint32_t v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = *(const uint32_t*)(po + min(k0 + k, S - 1) * pstep);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k < nsp) add(k0 + k, v[k]);
    }
  };
  // maximum and sum over the lanes, which hold -inf and 0 from lane nsp on; up to four
  // lanes are read out, in the order of the butterfly
  auto lane_max = [&](float v) {
    if (S <= 4) return fmaxf(fmaxf(lane_of(v, 0), lane_of(v, 1)), fmaxf(lane_of(v, 2), lane_of(v, 3)));
    return wave_max(v);
  };
  auto lane_sum = [&](float v) {
    if (S <= 4) return (lane_of(v, 0) + lane_of(v, 2)) + (lane_of(v, 1) + lane_of(v, 3));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
  };
  // The prefix splits of one head combined into one partial (log-sum-exp
  // s_lse, normalised output s_o0 / s_o1 for dims 2*lane, 2*lane+1).  It needs no
  // tail data: the first head's is formed while the first tile's loads are in
  // flight.  Lane sp holds split sp's log-sum-exp.
  float s_lse = -INFINITY, s_o0 = 0.f, s_o1 = 0.f;
  auto combine_splits = [&](int head, float lses, bool first) {
    if (kOne || S == 1) {  // its weight is 1 (every lane holds its log-sum-exp)
      s_lse = lses;
      const long long i0 = ((long long)r * a.Hq + head) * D;
      if constexpr (ROWS == 2) {
        u32x2 v = {pre[0], pre[1]};
        if (!first) v = *(const u32x2*)(a.part_o + i0 + 2 * lane);
        s_o0 = __uint_as_float(v[0]);
        s_o1 = __uint_as_float(v[1]);
      } else {
        const uint32_t v = first ? pre[0] : *(const uint32_t*)((const bf16_t*)a.part_o + i0 + part_slot(2 * lane));
        s_o0 = __uint_as_float(v << 16);
        s_o1 = __uint_as_float(v & 0xFFFF0000u);
      }
      return;
    }
    lses = lane < nsp ? lses : -INFINITY;
    const float mx = lane_max(lses), w = split_weight(lses, mx), den = lane_sum(w);
    const float inv = den > 0.f ? 1.f / den : 0.f;
    s_lse = merged_lse(mx, den);
    s_o0 = s_o1 = 0.f;
    add_splits((const bf16_t*)a.part_o + ((long long)r * a.Hq + head) * D + part_slot(2 * lane), lses, w, inv, first, s_o0, s_o1);
  };
  bool combined = false;
  // the row's own positions: first its prefix positions the split kernel left
  // (fewer than 64 past a split boundary, read in place from the shared
  // prefix), then its paged tail; 32-position tiles of either, dealt to the
  // four waves in turn
  const int n_ovt = (plen - pe + TT - 1) / TT, n_all = n_ovt + (n + TT - 1) / TT;
  const long long bg = (long long)prompt * a.Hkv + g;
  const bf16_t* pk = (const bf16_t*)a.kv.prefix_k + bg * a.kv.P * D;
  const bf16_t* pv = (const bf16_t*)a.kv.prefix_v + bg * a.kv.VP * D;
#pragma unroll 1
  for (int w = wave; w < 4; w += NWV) {
    float m = -INFINITY, lsum = 0.f;
    f32x4 o[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int vt = w; vt < n_all; vt += 4) {
      const bool ov = vt < n_ovt;
      const int tb = ov ? pe + vt * TT : (vt - n_ovt) * TT;  // first position of the tile
      const int lim = ov ? plen : n;                          // positions < lim exist
      // every address of the tile first (page numbers come from registers),
      // then all its loads back to back
      int kp[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int pos = tb + k_gather_row(0, e, l16);
        kp[e] = pos < lim ? pos : tb;
      }
      // this lane's eight positions p0 .. p0+7 lie in one page (ps % 8 == 0) or
      // one 64-position block of the prefix V layout (p0 % 8 == 0)
      const int p0 = tb + grp * 8;
      const int nv = lim - p0;
      const int vp = nv > 0 ? p0 : tb;
      const int kpg0 = page_at(ov ? 0 : kp[0] / ps), kpg1 = page_at(ov ? 0 : kp[1] / ps);
      const int vpg = page_at(ov ? 0 : vp / ps);
      const bf16_t* kr[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int pg = e ? kpg1 : kpg0;
        kr[e] = ov ? pk + (long long)kp[e] * D + grp * 8
                   : (const bf16_t*)a.kv.pool_k + (((long long)pg * a.Hkv + g) * ps + kp[e] % ps) * D + grp * 8;
      }
      const bf16_t* vr = ov ? pv + ((long long)(vp / 64) * D + l16) * 64 + vp % 64
                            : (const bf16_t*)a.kv.pool_v + (((long long)vpg * a.Hkv + g) * D + l16) * ps + vp % ps;
      const long long vstep = ov ? 16LL * 64 : 16LL * ps;  // 16 head-dim rows
      u32x4 ka[2][4], va[8];
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) ka[e][ks] = *(const u32x4*)(kr[e] + ks * 32);  // past the end: masked scores
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) va[dt] = *(const u32x4*)(vr + dt * vstep);  // past the end: zeroed below
      if (!combined) {  // uniform: the first tile of the wave
        combine_splits(g * G + min(wave, G - 1), pre_lse, true);
        combined = true;
      }
      f32x4 sc[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        sc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) sc[e] = mfma16x16x32(ka[e][ks], qf[ks], sc[e]);
      }
      float x = -INFINITY;
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (p0 + e * 4 + i >= lim) sc[e][i] = -INFINITY;
          x = fmaxf(x, sc[e][i]);
        }
      x = fmaxf(x, __shfl_xor(x, 16, 64));
      x = fmaxf(x, __shfl_xor(x, 32, 64));
      x *= scale;
      if (x > m) {
        const float alpha = exp2_raw(m - x);
        lsum *= alpha;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) o[dt] *= alpha;
        m = x;
      }
      const float msub = m == -INFINITY ? INFINITY : m;
      float p[8];
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) p[e * 4 + i] = exp2_raw(fmaf(sc[e][i], scale, -msub));
#pragma unroll
      for (int i = 0; i < 8; ++i) lsum += p[i];
      const u32x4 pb = {pack2(p[0], p[1]), pack2(p[2], p[3]), pack2(p[4], p[5]), pack2(p[6], p[7])};
      if (nv < 8) {  // V past the row's end is arbitrary (unwritten slots): zero it
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            if (2 * w >= nv) va[dt][w] = 0u;
            else if (2 * w + 1 >= nv) va[dt][w] &= 0xFFFFu;
          }
      }
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) o[dt] = mfma16x16x32(va[dt], pb, o[dt]);
    }
    // tail state -> LDS (query q = l16, dims dt*16 + grp*4 + i)
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    if (l16 < GM) {
      if (grp == 0) {
        w_m[w][l16] = m;
        w_l[w][l16] = lsum;
      }
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) *(f32x4*)&w_o[w][l16][dt * 16 + grp * 4] = o[dt];
    }
  }
  if (!combined) combine_splits(g * G + min(wave, G - 1), pre_lse, true);
  __syncthreads();

  // merge: wave h handles query heads h, h + NWV, ...; lane holds dims 2*lane, 2*lane+1
  auto finish = [&](int h, float lses) {
    const int head = g * G + h;
    // tail state of this head (exp2 domain) from the four waves
    float tm = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) tm = fmaxf(tm, w_m[w][h]);
    float tl = 0.f, to0 = 0.f, to1 = 0.f;
    if (tm != -INFINITY) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float f = exp2_raw(w_m[w][h] - tm);
        tl += f * w_l[w][h];
        to0 += f * w_o[w][h][2 * lane];
        to1 += f * w_o[w][h][2 * lane + 1];
      }
    }
    const float tail_lse = tl > 0.f ? (tm + __log2f(tl)) * kLn2 : -INFINITY;
    if (kOne || h < 4) {  // the prefix splits are combined already: two partials left
      const float mx = fmaxf(s_lse, tail_lse);
      const float ws = s_lse == -INFINITY ? 0.f : __expf(s_lse - mx);
      const float wt = tail_lse == -INFINITY ? 0.f : __expf(tail_lse - mx);
      const float den = ws + wt;
      const float inv = den > 0.f ? 1.f / den : 0.f;
      const float ft = tl > 0.f ? wt * inv / tl : 0.f;  // applied to the unnormalised tail sum
      const float fs = ws * inv;
      *(uint32_t*)(out + ((long long)r * a.Hq + head) * D + 2 * lane) =
          pack_bf16x2(fs * s_o0 + ft * to0, fs * s_o1 + ft * to1);
      return;
    }
    const float ls = lane < nsp ? lses : -INFINITY;
    const float mx = fmaxf(lane_max(ls), tail_lse);
    const float w = split_weight(ls, mx), wt = split_weight(tail_lse, mx);
    const float den = lane_sum(w) + wt;
    const float inv = den > 0.f ? 1.f / den : 0.f;
    const float ft = tl > 0.f ? wt * inv / tl : 0.f;  // applied to the unnormalised tail sum
    float o0 = ft * to0, o1 = ft * to1;
    add_splits((const bf16_t*)a.part_o + ((long long)r * a.Hq + head) * D + part_slot(2 * lane), ls, w, inv, false, o0, o1);
    *(uint32_t*)(out + ((long long)r * a.Hq + head) * D + 2 * lane) = pack_bf16x2(o0, o1);
  };
  if (wave < G) finish(wave, 0.f);
  for (int h = wave + NWV; h < G; h += NWV) {  // further heads
    const int head = g * G + h;
    const float lses = a.part_lse[((long long)(ROWS == 2 ? 0 : min(lane, S - 1)) * R + r) * a.Hq + head];
    if (kOne || h < 4) combine_splits(head, lses, false);
    finish(h, lses);
  }
}

}  // namespace

hipError_t attn_prefix_bf16(const AttnArgs& a, bf16_t* out, hipStream_t s) {
  if (a.D != 128 || a.Hq / a.Hkv > RGD_ATTN_QV || a.split_len % 64 || a.kv.VP % 64) return hipErrorInvalidValue;
  if (a.walk && a.splits > kMaxWalkSplits) return hipErrorInvalidValue;
  if (a.splits <= 0 || a.nrblocks <= 0) return hipSuccess;
  if (!a.rblocks) return hipErrorInvalidValue;
  // one launch per kAttnInlineBlocks row blocks
  for (int c0 = 0; c0 < a.nrblocks; c0 += kAttnInlineBlocks) {
    AttnArgs b = a;
    const int n = std::min(kAttnInlineBlocks, a.nrblocks - c0);
    for (int i = 0; i < n; ++i) b.rblk[i] = a.rblocks[c0 + i];
    if (a.walk)
      hipLaunchKernelGGL((attn_prefix_kernel<RGD_ATTN_NW, RGD_ATTN_QV / 16 / RGD_ATTN_NW, true>),
                         dim3(1, a.Hkv, n), dim3(RGD_ATTN_NW * 64), 0, s, b, out);
    else
      hipLaunchKernelGGL((attn_prefix_kernel<RGD_ATTN_NW, RGD_ATTN_QV / 16 / RGD_ATTN_NW, false>),
                         dim3(a.splits, a.Hkv, n), dim3(RGD_ATTN_NW * 64), 0, s, b, out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// f<D>() for the head dimensions of fp32 models
template <typename F>
static hipError_t by_head_dim(int D, F f) {
  switch (D) {
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t attn_prefix_f32(const AttnArgs& a, hipStream_t s) {
  if (a.Hq / a.Hkv > 8 || a.split_len > kChunk || a.split_len % 64) return hipErrorInvalidValue;
  if (a.splits <= 0) return hipSuccess;
  return by_head_dim(a.D, [&](auto d) {
    hipLaunchKernelGGL(attn_prefix_f32_kernel<decltype(d)::value>, dim3(a.splits, a.Hkv, a.rows.R), dim3(256), 0, s, a);
  });
}

hipError_t attn_tail_combine_f32(const AttnArgs& a, float* out, hipStream_t s) {
  if (a.Hq / a.Hkv > 8 || (a.tail_len > 0 && !a.rows.pages) || (a.tail_len > 0 && a.kv.page_size % 8) || a.splits < 1 ||
      a.splits > kMaxSplits)
    return hipErrorInvalidValue;
  return by_head_dim(a.D, [&](auto d) {
    hipLaunchKernelGGL(attn_tail_combine_kernel<decltype(d)::value>, dim3(a.rows.R, a.Hkv), dim3(256), 0, s, a, out);
  });
}

hipError_t attn_tail_merge_bf16(const AttnArgs& a, bf16_t* out, hipStream_t s) {
  if (a.D != 128 || a.Hq / a.Hkv > 16 || a.splits > kMergeMaxSplits || a.splits < 1 ||
      (a.tail_len > 0 && (!a.rows.pages || a.kv.page_size % 8)))
    return hipErrorInvalidValue;
  const int rows = a.walk ? a.nleft : a.rows.R;  // after a walk only those with positions left
  if (rows < 1) return hipSuccess;
  // one wave per workgroup: enough pairs for eight waves on every CU, one partial
  // to merge per head (with 16 splits of an 8193-position prompt the serial loads of
  // four heads' partials cost more: 117 against 111 us)
  const int G = a.Hq / a.Hkv;
  const bool one = G <= 4 && (a.walk || a.splits == 1) && (long long)rows * a.Hkv >= 2048;
  const dim3 grid(rows, a.Hkv);
  if (a.walk) {
    if (one) hipLaunchKernelGGL((attn_tail_merge_kernel<2, 1, 4>), grid, dim3(64), 0, s, a, out, a.left);
    else if (G <= 4) hipLaunchKernelGGL((attn_tail_merge_kernel<2, 4, 4>), grid, dim3(256), 0, s, a, out, a.left);
    else hipLaunchKernelGGL((attn_tail_merge_kernel<1, 4, 16>), grid, dim3(256), 0, s, a, out, a.left);
  } else {
    if (one) hipLaunchKernelGGL((attn_tail_merge_kernel<0, 1, 4>), grid, dim3(64), 0, s, a, out, nullptr);
    else hipLaunchKernelGGL((attn_tail_merge_kernel<0, 4, 16>), grid, dim3(256), 0, s, a, out, nullptr);
  }
  return hipGetLastError();
}

}  // namespace rgd
