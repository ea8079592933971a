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
// NormalFloat-4: 8 indices of one dword -> c * level in bf16, natural order (33 instructions: the two bytes of the 16
// levels are looked up for four indices at a time, eight entries per byte permutation, the half of the table chosen
// by bit 3).  The common factor c = 1 + 3580/8192, taken off again from the block's scale, is the one whose 16 products
// lie closest to bf16 numbers: 2-norm error of the level table 6.3e-4 (c = 1: 1.06e-3; products scale * level rounded
// to bf16, as the expanded matrix holds them: 1.6e-3).
constexpr float NF4_LEVEL_FACTOR = 1.0f + 3580.0f / 8192.0f;
struct Nf4Consts { uint32_t lo[4], hi[4]; };
__device__ __forceinline__ Nf4Consts nf4_constants() {
  return {{0x114180b8u, 0x000688d1u, 0xf9b56deau, 0xb8854f22u}, {0xbfbfbfbfu, 0x00bebebeu, 0x3e3e3e3du, 0x3f3f3f3fu}};
}
__device__ __forceinline__ void nf4_bytes(uint32_t x, const Nf4Consts& c, uint32_t& lo, uint32_t& hi) {
  const uint32_t sel = x & 0x07070707u, m = x & 0x08080808u, upper = (m << 5) - (m >> 3);    // 0xff where bit 3 is set
  lo = (__builtin_amdgcn_perm(c.lo[3], c.lo[2], sel) & upper) | (__builtin_amdgcn_perm(c.lo[1], c.lo[0], sel) & ~upper);
  hi = (__builtin_amdgcn_perm(c.hi[3], c.hi[2], sel) & upper) | (__builtin_amdgcn_perm(c.hi[1], c.hi[0], sel) & ~upper);
}
__device__ __forceinline__ bf16x8 unpack8_nf4(uint32_t w, const Nf4Consts& c) {
  uint32_t el, eh, ol, oh;                                // even and odd indices
  nf4_bytes(w & 0x0f0f0f0fu, c, el, eh);
  nf4_bytes((w >> 4) & 0x0f0f0f0fu, c, ol, oh);
  const uint32_t e0 = __builtin_amdgcn_perm(eh, el, 0x05010400u), e1 = __builtin_amdgcn_perm(eh, el, 0x07030602u);
  const uint32_t o0 = __builtin_amdgcn_perm(oh, ol, 0x05010400u), o1 = __builtin_amdgcn_perm(oh, ol, 0x07030602u);
  union { bf16x8 v; uint32_t u[4]; } r;
  r.u[0] = __builtin_amdgcn_perm(o0, e0, 0x05040100u);
  r.u[1] = __builtin_amdgcn_perm(o0, e0, 0x07060302u);
  r.u[2] = __builtin_amdgcn_perm(o1, e1, 0x05040100u);
  r.u[3] = __builtin_amdgcn_perm(o1, e1, 0x07060302u);
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
