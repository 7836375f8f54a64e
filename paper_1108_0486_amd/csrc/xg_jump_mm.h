// Jump-ahead on the matrix cores (gfx950).
//
// A member's x-part state S0 (r words) moves by T per word; T^J = g(T) with
// g = z^J mod P of degree below n.  With s_t, t = 0 .. n + r - 1, the words of
// S0's continuation (s_0 .. s_{r-1} is S0 itself), the jumped state's words are
//     y_j = xor over i < n of g_i s_{i + j},          j = 0 .. r - 1,
// i.e. over GF(2), bit b of them is the product of the r x (n + r) Toeplitz
// matrix G[j][t] = g_{t - j} with the column of the bits b of s.  Each product
// is a sum of zeros and ones taken modulo 2, so it runs exactly on the FP4
// matrix instructions (32 x 32 tiles, 64 values of t per instruction, 10 PFLOP/s
// dense): G's bits as FP4 1.0, the words' bits as FP4 0.5, sums of at most
// n / 2 in FP32, exact; y's bit is the sum's odd half.
//
// Layouts.  A 64-lane fragment gives lane l = 32 h + r row (or column) r and 32
// values of t (32 h .. 32 h + 31 of the block) in four registers.  The order of
// the 32 within a lane is free as long as both operands share it: register d
// holds t = 4 m + d in its m-th FP4, so that four masked shifts expand a word
// of 32 bits.  The bits b of a block of words come from a 32 x 32 bit transpose
// across the lanes of each half (word_bits).  Row r of G's tile mt in block c
// holds g's bits 64 c + 32 h - 32 mt - r .. + 31, so with q = 2 c + h - mt all
// fragments are the words g[32 q - r ..] (toeplitz_word), 32 of them per q.  Rows
// are numbered so that the result's words come out in order (row_word).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xg_device.h"

namespace xg {
namespace dev {

typedef int frag_t __attribute__((ext_vector_type(8)));   // four registers used (FP4)
typedef float tile_t __attribute__((ext_vector_type(16)));

// The 32 bits of w as FP4 values (0.5 for a set bit: 1, or 1.0: 2).
__device__ __forceinline__ uint4 half_bits(uint32_t w) {
  return make_uint4(w & 0x11111111u, (w >> 1) & 0x11111111u, (w >> 2) & 0x11111111u, (w >> 3) & 0x11111111u);
}
__device__ __forceinline__ uint4 one_bits(uint32_t w) {
  return make_uint4((w << 1) & 0x22222222u, w & 0x22222222u, (w >> 1) & 0x22222222u, (w >> 2) & 0x22222222u);
}

__device__ __forceinline__ frag_t frag(uint4 v) {
  return frag_t{(int)v.x, (int)v.y, (int)v.z, (int)v.w, 0, 0, 0, 0};
}

// acc += A B over 64 values of t, both operands FP4 (formats 4), no scales.
__device__ __forceinline__ tile_t mm_step(frag_t a, frag_t b, tile_t acc) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 4, 0, 0, 0, 0);
}

// Lane constants of word_bits.
struct TransposeLane {
  uint32_t sel16, sel8, keep4, keep2, keep1, rot4, rot2, rot1;
};

__device__ __forceinline__ TransposeLane transpose_lane(uint32_t lane) {
  TransposeLane k;
  // v_perm_b32 selectors (byte 0 .. 3: second operand, 4 .. 7: first operand)
  k.sel16 = lane & 16u ? 0x03020706u : 0x01000504u;
  k.sel8 = lane & 8u ? 0x07030501u : 0x02060004u;
  k.keep4 = lane & 4u ? 0xF0F0F0F0u : 0x0F0F0F0Fu;
  k.keep2 = lane & 2u ? 0xCCCCCCCCu : 0x33333333u;
  k.keep1 = lane & 1u ? 0xAAAAAAAAu : 0x55555555u;
  k.rot4 = lane & 4u ? 4u : 28u;
  k.rot2 = lane & 2u ? 2u : 30u;
  k.rot1 = lane & 1u ? 1u : 31u;
  return k;
}

// Bit kappa of the result on lane 32 h + b is bit b of v on lane 32 h + kappa:
// a 32 x 32 bit transpose in each half of the wavefront, by exchanging blocks
// of 16, 8, 4, 2 and 1 bits with the lane that differs in that bit.
__device__ __forceinline__ uint32_t word_bits(uint32_t v, const TransposeLane &k) {
  // 16: even rows of 16 lanes take the low halves of both rows, odd rows the high ones.
  const auto rows = __builtin_amdgcn_permlane16_swap(v, v, false, false);  // {even rows twice, odd rows twice}
  v = __builtin_amdgcn_perm(rows[0], rows[1], k.sel16);
  v = __builtin_amdgcn_perm(v, lane_xor<8>(v), k.sel8);
  uint32_t p = lane_xor<4>(v);
  v = select_bits(v, __builtin_amdgcn_alignbit(p, p, k.rot4), k.keep4);
  p = lane_xor<2>(v);
  v = select_bits(v, __builtin_amdgcn_alignbit(p, p, k.rot2), k.keep2);
  p = lane_xor<1>(v);
  return select_bits(v, __builtin_amdgcn_alignbit(p, p, k.rot1), k.keep1);
}

// Bits 32 q - r .. 32 q - r + 31 of a polynomial whose words are g[0 .. words),
// zero outside them.
__device__ __forceinline__ uint32_t toeplitz_word(const uint32_t *g, int words, int q, uint32_t r) {
  const uint32_t hi = q >= 0 && q < words ? g[q] : 0u;
  const uint32_t lo = q >= 1 && q <= words ? g[q - 1] : 0u;
  return r ? (hi << r) | (lo >> (32u - r)) : hi;
}

// The word of G's rows that row rho of a tile stands for.  A 32 x 32 result
// gives half h's lanes the rows 8 (i / 4) + 4 h + i % 4 in register i; with
// this order these are the words 16 h + i.
__device__ __forceinline__ constexpr uint32_t row_word(uint32_t rho) {
  return 16u * ((rho >> 2) & 1u) + 4u * (rho >> 3) + (rho & 3u);
}

// Bit 16 + i: the parity of the lane's sum in register i (an odd number of
// halves).  Adding 2^22, whose units are halves, leaves it in the lowest bit.
__device__ __forceinline__ uint32_t parities(const tile_t &acc) {
  uint32_t w = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) w = __builtin_amdgcn_alignbit(__float_as_uint(acc[i] + 0x1p22f), w, 1);
  return w;
}

// The words of two tiles: word w of a on lane w, of b on lane 32 + w.
__device__ __forceinline__ uint32_t tile_words(const tile_t &a, const tile_t &b, const TransposeLane &k) {
  const uint32_t wa = parities(a), wb = parities(b);
  const auto half = __builtin_amdgcn_permlane32_swap(wa, wb, false, false);  // {a, b of half 0}, {a, b of half 1}
  return word_bits((half[0] >> 16) | (half[1] & 0xFFFF0000u), k);
}

}  // namespace dev
}  // namespace xg
