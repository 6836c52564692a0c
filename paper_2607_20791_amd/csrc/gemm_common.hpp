// Device helpers shared by the bf16 GEMM kernels.
#pragma once
#include <type_traits>

#include "common.hpp"

namespace rgd {
namespace {

RGD_DEV f32x4 mfma16x16x32(const u32x4& a, const u32x4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

RGD_DEV float silu(float g) { return g / (1.0f + __expf(-g)); }

constexpr int kStep = 64;  // k values per pipeline step

// Swizzle of the 16-byte chunks of an X row staged in LDS as 64 k values:
// chunk c of row r sits at c ^ xswz1(r).
RGD_DEV int xswz1(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// Workgroups are handed out in linear order (x fastest), round-robin over
// the chip's 8 XCDs, each with its own L2.  With several row blocks, the
// work is reordered so that the row blocks of one column group are 8 apart
// in that order: on one XCD at nearly the same time, so the later blocks'
// weight reads can hit the lines the first one brought into that L2.
RGD_DEV void xcd_order(int& gx, int& gy) {
  if (gridDim.y == 1) return;
  const int G = gridDim.x, Y = gridDim.y;
  const int lin = blockIdx.x + blockIdx.y * G;
  const int full = (G / 8) * 8;  // column groups in whole octets
  if (lin < full * Y) {
    gy = (lin / 8) % Y;
    gx = (lin / 8 / Y) * 8 + lin % 8;
  } else {
    const int rem = lin - full * Y, gr = G - full;
    gx = full + rem % gr;
    gy = rem / gr;
  }
}

}  // namespace
}  // namespace rgd
