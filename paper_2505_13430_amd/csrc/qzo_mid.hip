// Perturbed 4-bit linear for up to a few hundred tokens, zero-point int4 and NormalFloat-4:
//   Y[M,N] = X[M,K] * W_eff^T,  W_eff[n,k] = (s[n,k/128] + sigma*eps*z(row_base+n, k/128)) * (u[n,k] - zp[n,k/128])
// (paper Eq. 4-5), or (s[n,k/64] + sigma*eps*z(row_base+n, k/64)) * level[u[n,k]].  Above the few-token kernel's rows
// the weights are used by several token tiles, and a 256 x 256 output tile is still mostly padding and leaves most
// of the chip idle.
//
// A workgroup of eight wavefronts owns 256 output rows (32 per wavefront) and two or four tiles of 32 tokens.  As in
// the few-token kernel the nibbles enter the matrix unit as the exact integers 128 + u and the perturbed scale is
// applied to a group's fp32 sums, y += s_eff * P; the int4 weights are not rounded.  What the integers carry too much,
// s_eff (128 + zp) X with X the block sum of the activations (delivered by the kernel that wrote them), is taken off
// for two groups at a time by one fp32 MFMA per tile (32x32x2: its depth is the two groups), which costs no vector
// instruction and no broadcast reads.  A token tile lies in one pass of a stacked step and takes that pass's sign.
// Hidden states of one layer against 64 bits: 7.8e-3 (the tile kernel, whose weights are rounded to bf16) -> 6.4e-3.
//
// Everything a group needs comes by direct-to-LDS loads into a ring of three or four stages, requested two or three
// groups ahead (swizzled on the memory side, nothing passes through registers); one barrier per group.  Inside a group
// the instructions are dealt out behind the MFMAs by hand: unpacking behind the first tile's, a tile's rescaling
// behind the next one's, fragment reads four ahead.  The compiler's own order needed 256 registers and spilled.
//
// Work is split evenly whatever the shape: items (row block, token block) x pairs of groups are cut into one
// contiguous range per compute unit; an item that several ranges touch is summed by the reduction kernel in order.
//
// NormalFloat-4: the weights that enter the matrix unit are those of the expanded matrix, (s + sigma*eps*z) * level
// rounded once (hidden states equal to four digits).  The 16 products of a block are formed once per row and looked up
// by byte permutations (nf4_table, unpack8_nf4); a lane's half of a group's inputs is one block, so a lane holds one
// table per pass.  The sums need no rescaling and no correction.  A token block holds tiles of one pass, or half of
// its places for either (BOTH: a second table, and a second lookup behind the same selectors): about 310 or 470 vector
// instructions per group and wavefront with four tiles against 32 MFMAs, which bound it.
// Against expand-then-multiply, which writes and reads 2 bytes per weight and pass: 1 x 16 tokens at 7B widths
// 16.5 -> 4.2 ms per step, 1 x 57 17.1 -> 5.6 (wide layers beyond 64 tokens run in the tile kernel, nf4_tile_route).  Blocks of either kind in one launch (BOTH for the remainder only): 6-13 % slower, the second
// copy of the loop is more cold code per launch.
//
// What bounds the integer format: at 57 tokens per pass (4096 x 4096 .. 22016) a launch takes 16-43 us, of which about
// 10 us do not depend on the work (start of a kernel whose code and operands come from HBM, 15-30 MB of partial sums
// out); a group of four tiles takes 4200-5300 cycles with the matrix unit busy for 2300 and the LDS for 2700 of them.
// Whole steps of zero-point models at 7B widths against two passes of the few-token kernel: 1 x 33 tokens 7.24 -> 4.70 ms,
// 1 x 57 7.74 -> 5.00.  Beyond 64 tokens the tile kernel is the faster one (mid_route), but rounds the weights.
// Tried: one wavefront per SIMD with 64 rows each (half the LDS reads, but the accumulators move to AGPRs and every
// rescaling then pays two register moves: 15-25 % slower); K split between two halves of a workgroup (LDS merge
// instead of partial sums: more activation traffic, slower); activations and weights staged through registers
// (a wait for young activation loads waits for older weight loads, and four tiles spill: 25 % slower at four tiles);
// -(128 + zp) X as the initial accumulator (16 broadcast reads of the LDS per group: 5-8 % slower).
#include "qzo_device.hpp"
#include "qzo_kernels.hpp"
#include "qzo_nibble.hpp"
#include <algorithm>
#include <type_traits>

namespace qzo {

namespace {

// One stage of the LDS ring holds everything that a group needs: the activation block, the weights of the
// workgroup's rows, the block sums, scales and zero-points.
constexpr uint32_t MID_W = MID_ROWS * 64, MID_XS = 512, MID_S = 8 * 256;
template <int MT, bool NF4>
struct MidLds {
  static constexpr uint32_t X = MT * 8192, STAGE = X + MID_W + MID_XS + MID_S * (NF4 ? 1 : 2);
  static constexpr int S = MT == 4 ? 3 : 4;
  static constexpr uint32_t BYTES = STAGE * S;
  static constexpr int LOADS = MT + (NF4 ? 3 : 5);   // load instructions per wavefront and stage
  static_assert(BYTES <= 160 * 1024, "LDS of a compute unit");
};

#define QM_DTL(INSTR, RSRC, LDSADDR, VOFF)                                                   \
  asm volatile(QZO_SET_M0 INSTR " %1, %2, 0 offen lds" : : "s"(LDSADDR), "v"(VOFF), "s"(RSRC) : "memory", "m0")

// BOTH: NormalFloat-4, every token block holds tiles of both passes.
template <int MT, bool NF4, bool BOTH>
__global__ __launch_bounds__(512, 2) void mid_gemm_kernel(GemmArgs a, MidPlan mp, float* __restrict__ part) {
  mp.mt = MT; mp.both = BOTH ? 1u : 0u;            // known here
  typedef MidLds<MT, NF4> L;
  constexpr int S = L::S;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t lrow = lane & 31u, half = lane >> 5;     // MFMA operand: row, half of the group's inputs
  const uint32_t K = a.K, ngrp = K >> 7;
  const bool s_fp16 = a.s_fp16 != 0;
  const NibbleConsts nc = nibble_constants();
  constexpr uint32_t OUT_OF_RANGE = 0x80000000u;
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  auto rsrc = [](const void* p, uint64_t bytes) {
    return i32x4{(int)(uint32_t)(uintptr_t)p, (int)(uint32_t)((uintptr_t)p >> 32), (int)bytes, 0x00020000};
  };
  const i32x4 rx = rsrc(a.x, (uint64_t)mp.rows * K * 2), rw = rsrc(a.w, (uint64_t)a.N * (K >> 1));
  const i32x4 rs = rsrc(a.s, (uint64_t)a.N * ngrp * (NF4 ? 4 : 2)), rz = rsrc(NF4 ? a.s : a.zp, (uint64_t)a.N * ngrp);
  const i32x4 rxs = rsrc(a.xsum, (uint64_t)mp.rows * ngrp * 4);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // what a lane reads of a stage: two chunks of its weight row, fragment j of an activation tile
  const uint32_t wrd = L::X + wave * 2048u + lrow * 64u, wsw = (lrow >> 2) & 3u;
  const uint32_t wrd0 = wrd + (((2 * half) ^ wsw) << 4), wrd1 = wrd + (((2 * half + 1) ^ wsw) << 4);
  uint32_t xrd[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) xrd[j] = lrow * 256u + ((half * 8 + j) ^ (lrow & 15u)) * 16u;

  const uint32_t w = (mp.W & 7u) == 0 ? (blockIdx.x & 7u) * (mp.W >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  uint32_t i0 = w * mp.tot / mp.W;
  const uint32_t i1 = (w + 1) * mp.tot / mp.W;

  while (i0 < i1) {
    const uint32_t item = i0 / mp.U, u0 = i0 - item * mp.U, u1 = min(mp.U, u0 + (i1 - i0));
    const uint32_t slot = w - mid_range_of(item * mp.U, mp.W, mp.tot);
    const uint32_t rb = item / mp.Z, z = item - rb * mp.Z;
    i0 += u1 - u0;
    const uint32_t g0 = 2 * u0, g1 = min(ngrp, 2 * u1);
    const uint32_t nb = rb * MID_ROWS + wave * 32;
    const uint32_t n = min(nb + lrow, a.N - 1);             // the lane's row

    // loads: activations 4 rows of 256 bytes per instruction, weights 16 rows of 64 bytes, both swizzled on the
    // memory side (16-byte chunks; the LDS is filled in lane order)
    auto xrow_of = [&](uint32_t row) {             // (places without a tile: some row that exists)
      const MidTile k = mid_tile(mp, z, row >> 5);
      return min(k.pass, mp.T == mp.Tp ? 0u : 1u) * a.M + min(k.tile * 32 + (row & 31u), a.M - 1);
    };
    uint32_t xoff[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const uint32_t row = 4 * (i * 8 + wave) + (lane >> 4);
      xoff[i] = xrow_of(row) * K * 2 + (((lane & 15u) ^ (row & 15u)) << 4);
    }
    const uint32_t woff = (nb + (lane >> 2)) * (K >> 1) + ((lane & 3u) ^ ((lane >> 4) & 3u)) * 16, wstep = 16 * (K >> 1);
    const uint32_t soff = n * ngrp;
    const uint32_t xsoff = xrow_of(min((wave & 1u) * 64 + lane, MT * 32u - 1)) * 4u;
    // load instruction i of group g's stage
    auto load1 = [&](int i, uint32_t g, uint32_t stage) {
      const uint32_t base = lds0 + stage * L::STAGE, in = g < g1 ? 0u : OUT_OF_RANGE;
      if (i < MT)
        QM_DTL("buffer_load_dwordx4", rx, base + (i * 8 + wave) * 1024, xoff[i] + (in + g * 256));
      else if (i < MT + 2)
        QM_DTL("buffer_load_dwordx4", rw, base + L::X + wave * 2048 + (i - MT) * 1024, woff + (in + g * 64 + (i - MT) * wstep));
      else if (NF4 && i == MT + 2)       // the scales of the group's two blocks
        QM_DTL("buffer_load_dword", rs, base + L::X + MID_W + MID_XS + wave * 256, soff * 4 + (in + g * 4));
      else if (!NF4 && i == MT + 2)
        QM_DTL("buffer_load_dword", rxs, base + L::X + MID_W + (wave & 1u) * 256, xsoff + (in + g * mp.rows * 4));
      else if (!NF4 && i == MT + 3)
        QM_DTL("buffer_load_ushort", rs, base + L::X + MID_W + MID_XS + wave * 256, soff * 2 + (in + g * 2));
      else if (!NF4 && i == MT + 4)
        QM_DTL("buffer_load_ubyte", rz, base + L::X + MID_W + MID_XS + MID_S + wave * 256, soff + (in + g));
    };

    floatx16 y[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) y[m][r] = 0.0f;
    uint32_t zw[4];
    float z_even = 0.0f, z_odd = 0.0f;
    float xa[MT], bp = 0.0f, bm = 0.0f;                       // operands of the correction, see below
#pragma unroll
    for (int m = 0; m < MT; ++m) xa[m] = 0.0f;
#pragma unroll
    for (int i = 0; i < S - 1; ++i)
#pragma unroll
      for (int l = 0; l < L::LOADS; ++l) load1(l, g0 + i, i);
    uint32_t stage = 0;
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"((S - 2) * L::LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    // one group; integers: d = g % 2
    auto group = [&](uint32_t g, auto parity) {
      constexpr int d = decltype(parity)::value;
      const uint32_t to = stage == 0 ? S - 1 : stage - 1;     // the group before, which everyone has read
      const unsigned char* sb = lds + stage * L::STAGE;
      constexpr int R = 4;                  // fragments read ahead of their MFMA
      bf16x8 wf[8], wb[BOTH ? 8 : 1], xf[R];      // wb: the second pass's weights
      floatx16 p[2];
      auto xread = [&](int q) {
        xf[q % R] = *reinterpret_cast<const bf16x8*>(sb + xrd[q & 7] + (q >> 3) * 8192);
      };
      uint32_t wd[8];                       // the eight inputs that the lane's half feeds to k-step j
      {
        const u32x4 w0 = *reinterpret_cast<const u32x4*>(sb + wrd0), w1 = *reinterpret_cast<const u32x4*>(sb + wrd1);
        wd[0] = w0.x; wd[1] = w0.y; wd[2] = w0.z; wd[3] = w0.w;
        wd[4] = w1.x; wd[5] = w1.y; wd[6] = w1.z; wd[7] = w1.w;
      }
#pragma unroll
      for (int q = 0; q < R; ++q) xread(q);
      const uint32_t sbits = *reinterpret_cast<const uint32_t*>(sb + L::X + MID_W + MID_XS + wave * 256 + lane * 4);
      const uint32_t zbits = !NF4 ? *reinterpret_cast<const uint32_t*>(sb + L::X + MID_W + MID_XS + MID_S + wave * 256 + lane * 4) : 0u;
      float xs[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) xs[m] = NF4 ? 0.0f : *reinterpret_cast<const float*>(sb + L::X + MID_W + (m * 32 + lrow) * 4);
      // noise: a counter serves eight scales, a word two: two groups, or the two blocks of one NormalFloat-4 group
      const uint32_t pair = NF4 ? g : g >> 1;
      if ((NF4 || d == 0) && (g == g0 || (pair & 3u) == 0)) {
        const u32x4_t pw = philox4x32_10(a.row_base + n, pair >> 2, 0u, 0u, a.seed_lo, a.seed_hi);
        zw[0] = pw.x; zw[1] = pw.y; zw[2] = pw.z; zw[3] = pw.w;
      }
      if (NF4 || d == 0) {
        const uint32_t q = pair & 3u;
        normal_pair(q == 0 ? zw[0] : (q == 1 ? zw[1] : (q == 2 ? zw[2] : zw[3])), z_even, z_odd);
      }
      // perturbed scales of the two passes; for NormalFloat-4 those of the block that the lane's inputs lie in, and
      // without BOTH the first one is that of the token block's pass
      const bool second = NF4 && !BOTH && mid_tile(mp, z, 0).pass != 0;
      const float s0 = scale_to_f32(NF4 && half ? sbits >> 16 : sbits & 0xffffu, s_fp16);
      const float zn = (NF4 ? half != 0 : d != 0) ? z_odd : z_even;
      const float sp = __builtin_fmaf(second ? -a.eps_signed : a.eps_signed, zn, s0);
      const float sm = __builtin_fmaf(-a.eps_signed, zn, s0);
      Nf4Table tp, tm;
      if constexpr (NF4) tp = nf4_table(sp);
      if constexpr (BOTH) tm = nf4_table(sm);
      auto unpack = [&](int j) {
        if constexpr (NF4) wf[j] = unpack8_nf4(wd[j], tp);
        else wf[j] = unpack8_natural(wd[j], nc);
        if constexpr (BOTH) wb[j] = unpack8_nf4(wd[j], tm);
      };
      const float cz = -(128.0f + (float)(zbits & 0xffu));
      // correction operands: lanes of half k hold group k of a pair
      const bool mine = half == d;
#pragma unroll
      for (int m = 0; m < MT; ++m) xa[m] = mine ? xs[m] : (d == 0 ? 0.0f : xa[m]);
      bp = mine ? sp * cz : bp;
      bm = mine ? sm * cz : bm;
      // p[m % 2]: sums of tile m
      auto rescale = [&](int m, int r0, int cnt) {
        const float se = (z * MT + m) >= mp.Tp ? sm : sp;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (r >= r0 && r < r0 + cnt) y[m][r] = __builtin_fmaf(se, p[m & 1][r], y[m][r]);
      };
      unpack(0);
      __builtin_amdgcn_sched_barrier(0);
      // one slot per MFMA: what else the wavefront has to do is dealt out between them
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int q = m * 8 + j;
          const floatx16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
          if constexpr (NF4) y[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[q % R], BOTH && m >= MT / 2 ? wb[BOTH ? j : 0] : wf[j], y[m], 0, 0, 0);
          else p[m & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[q % R], wf[j], j == 0 ? zero : p[m & 1], 0, 0, 0);
          if (q + R < MT * 8) xread(q + R);
          if (m == 0 && j < 7) unpack(j + 1);
          if (!NF4 && m > 0 && j >= 1 && j <= 4) rescale(m - 1, (j - 1) * 4, 4);
          if (q >= 2 && q - 2 < L::LOADS) load1(q - 2, g + S - 1, to);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
      for (int l = MT * 8 - 2; l < L::LOADS; ++l) load1(l, g + S - 1, to);
      if (!NF4) rescale(MT - 1, 0, 16);
      stage = stage == S - 1 ? 0 : stage + 1;
      // the next group has landed (later ones may still be on their way), and everyone has read this one
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((S - 2) * L::LOADS) : "memory");
      __builtin_amdgcn_s_barrier();
    };
    if constexpr (NF4) {
      for (uint32_t g = g0; g < g1; ++g) group(g, std::integral_constant<int, 0>());
    } else for (uint32_t g = g0; g < g1; g += 2) {
      group(g, std::integral_constant<int, 0>());
      if (g + 1 < g1) group(g + 1, std::integral_constant<int, 1>());
      // the integers entered as 128 + u: y -= s_eff (128 + zp) X, two groups at a time on the fp32 matrix unit
#pragma unroll
      for (int m = 0; m < MT; ++m)
        y[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[m], (z * MT + m) >= mp.Tp ? bm : bp, y[m], 0, 0, 0);
    }

    // partial sums of this range
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(part, 0, (int)0x7fffffff, 0x00020000);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const MidTile k = mid_tile(mp, z, m);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t tok = k.tile * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        const uint32_t off = ((slot * mp.rows + k.pass * a.M + tok) * a.N + nb + lrow) * 4u;
        if (k.valid && tok < a.M && nb + lrow < a.N)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[m][r]), rp, (int)off, 0, WRITE_THROUGH);
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");        // loads past the end still write the LDS
}
#undef QM_DTL

// Block sums X[g][row] = sum of x[row, 128 g .. 128 g + 127]: 16 lanes a group.
__global__ __launch_bounds__(256) void block_sums_kernel(const u32x4* __restrict__ x, uint32_t rows, uint32_t K,
                                                         float* __restrict__ out) {
  const uint32_t c = blockIdx.x * 256 + threadIdx.x, cpr = K >> 3;
  const bool own = c < rows * cpr;
  float s = own ? sum8_bf16(x[c]) : 0.0f;
  s += __shfl_xor(s, 1, 64); s += __shfl_xor(s, 2, 64); s += __shfl_xor(s, 4, 64); s += __shfl_xor(s, 8, 64);
  if (own && (threadIdx.x & 15u) == 0) out[(c % cpr >> 4) * rows + c / cpr] = s;
}

}  // namespace

// Two token tiles per workgroup up to eleven tiles in all, four from there on: with four the workgroups read the
// weights half as often, with two their partial sums are half as large.  Inside the 7B step at 4096 x 4096 .. 22016
// (sum of the four linears of a layer with their reductions, two / four tiles): 4 tiles 135 / 140 us, 6 tiles
// 167 / 179, 10 tiles 227 / 230, 12 tiles 253 / 239, 16 tiles 326 / 289.  Fewer ranges than compute units (longer
// ranges, fewer partial sums) were slower at every size: 192 ranges +5 %, 128 +30 %.  NormalFloat-4, whose unpacking
// costs three times as much, takes four from four tiles on, as long as that leaves every compute unit two pairs of
// groups (steps with four / two: 7B widths 6 tiles 2.04 / 2.15 ms for eight layers, 16 tiles 3.07 / 3.73; d_model 1024
// 4 tiles 0.368 / 0.323 for four layers, 10 tiles 0.436 / 0.405; the smallest model of the tests 0.165 / 0.140).  With
// the limit, per linear, against four throughout: OPT-1.3B 4 tiles 0.97, 10 tiles 1.02, 16 tiles 0.99; a limit of one
// pair: the same but for 7B and 13B widths at 4 tiles (1.00 against 0.98).
MidPlan mid_plan(uint32_t M, uint32_t N, uint32_t K, bool dual, bool nf4) {
  MidPlan p = {};
  const uint32_t Tp = (M + 31) / 32, T = dual ? 2 * Tp : Tp;
  p.rows = dual ? 2 * M : M; p.T = T; p.Tp = Tp;
  p.U = ((K >> 7) + 1) / 2;
  const uint32_t blocks = (N + MID_ROWS - 1) / MID_ROWS, cus = gemm_workgroups(1u << 20, 1u << 20);
  p.mt = T >= (nf4 ? 4u : 12u) && (!nf4 || blocks * ((T + 3) / 4) * p.U >= 2 * cus) ? 4 : 2;
  p.Z = (T + p.mt - 1) / p.mt;
  p.both = nf4 && dual && Tp % p.mt != 0;
  p.tot = blocks * p.Z * p.U;
  p.W = std::min(p.tot, cus);
  const uint32_t shortest = p.tot / p.W;
  p.slots = std::min(p.U, (p.U + shortest - 1) / shortest + 1);   // no item is touched by more ranges than that
  return p;
}
uint64_t mid_ws_floats(uint32_t M, uint32_t N, uint32_t K, bool dual, bool nf4) {
  const MidPlan p = mid_plan(M, N, K, dual, nf4);
  return (uint64_t)p.slots * p.rows * N;
}
// 32-bit byte offsets into the operands and the partial sums, 32-bit products in the ranges' arithmetic
bool mid_fits(uint32_t M, uint32_t N, uint32_t K, bool dual, bool nf4) {
  const MidPlan p = mid_plan(M, N, K, dual, nf4);
  return (uint64_t)p.slots * p.rows * N * 4 < (1ull << 31) && (uint64_t)p.rows * K * 2 < (1ull << 31) &&
         ((uint64_t)N + MID_ROWS) * (K >> 1) < (1ull << 31) &&
         ((uint64_t)N / MID_ROWS + 1) * p.Z * p.U * (p.W + 1) < (1ull << 32);
}

template <int MT, bool NF4, bool BOTH>
static hipError_t mid_launch(const GemmArgs& a, const MidPlan& mp, float* ws, hipStream_t st) {
  static bool ready = false;
  constexpr uint32_t L = MidLds<MT, NF4>::BYTES;
  if (!ready) {
    hipError_t e = hipFuncSetAttribute((const void*)mid_gemm_kernel<MT, NF4, BOTH>, hipFuncAttributeMaxDynamicSharedMemorySize, L);
    if (e != hipSuccess) return e;
    ready = true;
  }
  mid_gemm_kernel<MT, NF4, BOTH><<<mp.W, 512, L, st>>>(a, mp, ws);
  return hipGetLastError();
}
template <bool NF4, bool BOTH>
static hipError_t mid_launch_mt(const GemmArgs& a, const MidPlan& mp, float* ws, hipStream_t st) {
  return mp.mt == 2 ? mid_launch<2, NF4, BOTH>(a, mp, ws, st) : mid_launch<4, NF4, BOTH>(a, mp, ws, st);
}

hipError_t launch_block_sums(const void* x, uint32_t rows, uint32_t K, float* out, hipStream_t st) {
  block_sums_kernel<<<(rows * (K >> 3) + 255) / 256, 256, 0, st>>>((const u32x4*)x, rows, K, out);
  return hipGetLastError();
}

hipError_t launch_mid_gemm(const GemmArgs& a, float* ws, hipStream_t st) {
  if (a.M == 0 || a.N == 0) return hipSuccess;
  const MidPlan p = mid_plan(a.M, a.N, a.K, a.dual != 0, a.nf4 != 0);
  if (!ws || (!a.nf4 && (!a.xsum || !a.zp)) || !mid_fits(a.M, a.N, a.K, a.dual != 0, a.nf4 != 0)) return hipErrorInvalidValue;
  hipError_t e = !a.nf4 ? mid_launch_mt<false, false>(a, p, ws, st)
                        : (p.both ? mid_launch_mt<true, true>(a, p, ws, st) : mid_launch_mt<true, false>(a, p, ws, st));
  if (e != hipSuccess) return e;
  return launch_mid_reduce(a, ws, p, st);
}

}  // namespace qzo
