// int4 codes as MFMA operands, shared by the kernels that scale group sums instead of weights: nibbles to bf16
// 128 + u, activations in the matching order, and the LDS layout of an activation block.
#pragma once
#include "qzo_device.hpp"

namespace qzo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Nibbles become bf16 by "and, or": 0x4300 | u is the bf16 pattern of 128 + u.  With mask and pattern in registers
// that the compiler cannot see into a pair is one instruction, with literals two.  Not inline asm: the wait states
// an MFMA needs after a vector instruction that wrote its operand are inserted for instructions that the compiler
// knows, not behind an asm block.
struct NibbleConsts { uint32_t mask, magic; };
__device__ __forceinline__ NibbleConsts nibble_constants() {
  NibbleConsts c;
  asm volatile("s_mov_b32 %0, 0x000f000f" : "=s"(c.mask));
  asm volatile("v_mov_b32 %0, 0x43004300" : "=v"(c.magic));
  return c;
}
// 8 nibbles of one dword -> the bf16 values 128 + u, in the order k = 0,4,1,5,2,6,3,7 (7 instructions)
__device__ __forceinline__ bf16x8 unpack8_biased(uint32_t w, NibbleConsts c) {
  union { bf16x8 v; uint32_t u[4]; } r;
  r.u[0] = (w & c.mask) | c.magic;
  r.u[1] = ((w >> 4) & c.mask) | c.magic;
  r.u[2] = ((w >> 8) & c.mask) | c.magic;
  r.u[3] = ((w >> 12) & c.mask) | c.magic;
  return r.v;
}
// the same in natural order (9 instructions): byte i of w and of w >> 4 become the low halves of a dword
__device__ __forceinline__ bf16x8 unpack8_natural(uint32_t w, NibbleConsts c) {
  const uint32_t o = w >> 4;
  union { bf16x8 v; uint32_t u[4]; } r;
  r.u[0] = (__builtin_amdgcn_perm(o, w, 0x0c040c00u) & c.mask) | c.magic;
  r.u[1] = (__builtin_amdgcn_perm(o, w, 0x0c050c01u) & c.mask) | c.magic;
  r.u[2] = (__builtin_amdgcn_perm(o, w, 0x0c060c02u) & c.mask) | c.magic;
  r.u[3] = (__builtin_amdgcn_perm(o, w, 0x0c070c03u) & c.mask) | c.magic;
  return r.v;
}
// The 16 levels of the published NormalFloat-4 code book (normal quantiles scaled to [-1, 1]).
__device__ const float NF4_LEVELS_DEV[16] = {
    -1.0f, -0.6961928009986877f, -0.5250730514526367f, -0.39491748809814453f,
    -0.28444138169288635f, -0.18477343022823334f, -0.09105003625154495f, 0.0f,
    0.07958029955625534f, 0.16093020141124725f, 0.24611230194568634f, 0.33791524171829224f,
    0.44070982933044434f, 0.5626170039176941f, 0.7229568362236023f, 1.0f};

// NormalFloat-4 weights of one block as MFMA operands: the 16 products scale * level, each rounded once to bf16 as the
// expanded matrix holds them, as byte tables (32 instructions per block); then 8 indices of one dword -> 8 products in
// natural order by byte permutations (26 instructions, 16 for a second table: the two bytes of the products are looked
// up for four indices at a time, eight entries per permutation, the half of the table chosen by bit 3).
// Levels rounded on their own, with the scale applied to the sums, need no table per block and pass, but a level's
// rounding is the same in every weight that has it: over activations of one sign the errors add up instead of averaging
// out (silu(g) g of 2048 / 8192 features: 9.6e-3 / 1.7e-2 in the hidden states, rounded products 6.4e-3 / 6.3e-3).
struct Nf4Table { uint32_t lo[4], hi[4]; };
__device__ __forceinline__ void nf4_table_part(Nf4Table& t, float s, int q) {      // entries 4 q .. 4 q + 3
  const uint32_t a = pack_bf16x2(s * NF4_LEVELS_DEV[4 * q], s * NF4_LEVELS_DEV[4 * q + 1]);
  const uint32_t b = pack_bf16x2(s * NF4_LEVELS_DEV[4 * q + 2], s * NF4_LEVELS_DEV[4 * q + 3]);
  t.lo[q] = __builtin_amdgcn_perm(b, a, 0x06040200u);
  t.hi[q] = __builtin_amdgcn_perm(b, a, 0x07050301u);
}
__device__ __forceinline__ Nf4Table nf4_table(float s) {
  Nf4Table t;
#pragma unroll
  for (int q = 0; q < 4; ++q) nf4_table_part(t, s, q);
  return t;
}
// Four indices: entry within a half of the table, and 0xff where bit 3 is set (permutation selectors 8 .. 11 return the
// top bit of a source's byte 1 or 3, eight times).
struct Nf4Select { uint32_t sel, upper; };
__device__ __forceinline__ uint32_t nf4_bytes(const uint32_t (&t)[4], Nf4Select s) {
  return (__builtin_amdgcn_perm(t[3], t[2], s.sel) & s.upper) | (__builtin_amdgcn_perm(t[1], t[0], s.sel) & ~s.upper);
}
// a: indices 0, 1, 4, 5 of a dword, b: 2, 3, 6, 7
__device__ __forceinline__ uint32_t nf4_entries_a(uint32_t w) { return __builtin_amdgcn_perm(w >> 4, w, 0x06020400u) & 0x07070707u; }
__device__ __forceinline__ uint32_t nf4_upper_a(uint32_t w) { return __builtin_amdgcn_perm(w << 8, w << 12, 0x0b090a08u); }
__device__ __forceinline__ uint32_t nf4_entries_b(uint32_t w) { return __builtin_amdgcn_perm(w >> 4, w, 0x07030501u) & 0x07070707u; }
__device__ __forceinline__ uint32_t nf4_upper_b(uint32_t w) { return __builtin_amdgcn_perm(w, w << 4, 0x0b090a08u); }
// high and low bytes of four products -> the first and the second two
__device__ __forceinline__ void nf4_merge(uint32_t high, uint32_t low, uint32_t& first, uint32_t& second) {
  first = __builtin_amdgcn_perm(high, low, 0x05010400u);
  second = __builtin_amdgcn_perm(high, low, 0x07030602u);
}
__device__ __forceinline__ bf16x8 unpack8_nf4(uint32_t w, const Nf4Table& t) {
  const Nf4Select a = {nf4_entries_a(w), nf4_upper_a(w)}, b = {nf4_entries_b(w), nf4_upper_b(w)};
  union { bf16x8 v; uint32_t u[4]; } r;
  nf4_merge(nf4_bytes(t.hi, a), nf4_bytes(t.lo, a), r.u[0], r.u[2]);
  nf4_merge(nf4_bytes(t.hi, b), nf4_bytes(t.lo, b), r.u[1], r.u[3]);
  return r.v;
}
// 8 consecutive bf16 (4 dwords) -> the same order 0,4,1,5,2,6,3,7
__device__ __forceinline__ u32x4 permute8(u32x4 x) {
  u32x4 r;
  r.x = __builtin_amdgcn_perm(x.z, x.x, 0x05040100u);    // (x0, x4): low halves of dwords 0 and 2
  r.y = __builtin_amdgcn_perm(x.z, x.x, 0x07060302u);    // (x1, x5): high halves
  r.z = __builtin_amdgcn_perm(x.w, x.y, 0x05040100u);    // (x2, x6)
  r.w = __builtin_amdgcn_perm(x.w, x.y, 0x07060302u);    // (x3, x7)
  return r;
}
// sum of 8 bf16 values in fp32
__device__ __forceinline__ float sum8_bf16(u32x4 x) {
  const uint32_t d[4] = {x.x, x.y, x.z, x.w};
  float lo = 0.0f, hi = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    lo += __uint_as_float(d[i] << 16);
    hi += __uint_as_float(d[i] & 0xffff0000u);
  }
  return lo + hi;
}

__device__ __forceinline__ uint32_t x_lds_off(uint32_t row, uint32_t chunk) {   // 256-byte rows, 16 chunks
  return row * 256u + ((chunk ^ (row & 15u)) << 4);
}

}  // namespace qzo
