// Perturbed W4A16 linear for few tokens inside a model (up to 64 per pass, both passes of a step in one launch): the
// product of the few-token kernel (qzo_skinny.hip) bit for bit - 0x4300 | u as the bf16 value 128 + u, group sums
// P by MFMA, y += s_eff (P - (128 + zp) X) in fp32 - for activations that their producer has laid out for it (XPack) and
// whose block sums X it has delivered.
//
// A workgroup of W wavefronts owns 32 W output rows and one K slice; W (4 to 12 with one token tile, 4 to 8 with two) is the one whose
// rounds of a workgroup per compute unit take the least time: at 16 tokens one round for every linear of the 7B shape.  With four tiles
// W is 6, and 22016 rows take two rounds (115 x 4 workgroups).  The slice's activations come by direct-to-LDS loads in the order in which the MFMA wants them
// (1 KB a load, no permutation, no address arithmetic in the loop), weights two rounds (four groups) ahead into registers;
// everyone's first round is requested before anyone's second, or the youngest wavefront's first weights queue behind all of the
// oldest one's.  The arguments of the first loads arrive in registers (read from memory: 1.2 us); the noise of the eight groups
// is drawn while the first loads are on their way, either half of a wavefront half of the variates.  With one token tile the K
// loop holds no barrier: a wavefront waits for its own weights only.  With more tiles the activations are a ring of six (two
// tiles) or four (four) groups, refilled by loads dealt out behind the MFMAs.  One wavefront serves the tokens of both passes: a weight is unpacked once for a step;
// where a launch of 33 to 64 tokens would be short of workgroups, one of two tiles serves each pass (few_launch_wide).
//
// Bound, 1 x 16 tokens of the 7B shape, one launch of 12288 / 22016 / 4096 rows (25 / 45 / 23 MB): 7.2 / 10.1 / 8.2 us from its
// first instruction to its last (before: 12.3 / 17.1 / 12.9), of which reading alone takes some 3.5 / 6.5 / 3.5 whatever the
// pattern (128 bytes of eight rows, 512 of two, linear: 8.4 us a launch of 45 MB, all included); eight groups of 850 cycles
// behind the first loads and 1400 cycles of stores are what does not overlap.  Step 2.67 -> 2.26 ms (another board
// 2.71 -> 2.39).
// Four tiles (57 tokens), workgroups of 192 rows: a group takes 2000 cycles (two wavefronts on a SIMD, 1024 of MFMAs each), 2950
// with the six loads of 1 KB that refill the ring, whatever places they take; then 4400 cycles of stores: 22 / 40 / 20 MB of partial sums
// at the rate of the last-level cache.  12288 / 22016 / 4096 rows 17.4 / 33.7 / 17.9 us; refills in a row and the barrier at the head of a
// group, 256 rows: 3600 cycles a group, a step of 4.43 ms for 4.10.  The weights are builtin loads, whose waits the compiler counts without
// the refills (asm): before the third round's weights are stored (group 3) it waits until 4 loads are out where 16 could be, before the
// fourth's (group 5) for all of them, the last group's activations among them.
// Tried: all four rounds of weights requested at once (everything arrives, then everything is computed: 10.0 / 13.7 / 9.9 us);
// activations of the later groups behind the first weights (no difference).
#include "qzo_device.hpp"
#include "qzo_kernels.hpp"
#include "qzo_nibble.hpp"
#include <algorithm>
#include <type_traits>

namespace qzo {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// LDS: a ring of XS groups of activations, the slice's block sums, 4 KB per wavefront in which a round of weights (two
// groups of 32 rows) turns from "a lane per 16 bytes of a line" to "a lane per row".
template <int MT>
struct FewLds {
  static constexpr int XS = MT == 1 ? 8 : (MT == 2 ? 6 : 4), W = MT == 1 ? 12 : (MT == 2 ? 8 : 6);      // W: most wavefronts
  static constexpr uint32_t GROUP = MT * 8192u, SUMS = XS * GROUP, WT = SUMS + 8 * MT * 128u;
  static constexpr uint32_t bytes(uint32_t waves) { return WT + waves * 4096u; }
  static_assert(WT + W * 4096u <= 160 * 1024, "LDS of a compute unit");
};

#define QF_DTL(RSRC, LDSADDR, VOFF)                                                          \
  asm volatile(QZO_SET_M0 "buffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(LDSADDR), "v"(VOFF), "s"(RSRC) : "memory", "m0")

// What a wavefront needs later than its first loads.
struct FewRest { uint32_t row_base, seed_lo, seed_hi; float eps_signed; };

// Passes of a launch: one, both in a wavefront (the first half of its tile rows is the +eps pass, the second half the -eps pass), or
// both, a workgroup for each (the tiles of the two passes behind each other in every group of x).
enum { ONE_PASS, BOTH_PASSES, PASS_EACH };

// MT tiles of 32 token rows.
template <int MT, int PASSES, bool ZP>
__global__ __launch_bounds__(FewLds<MT>::W * 64) void few_gemm_kernel(const void* x, const void* w, const void* s, const float* xsum,
    uint32_t N, uint32_t K, uint32_t per, uint32_t packed, float* part, const void* zp, FewRest a) {
  const uint32_t M = packed & 0xffu, W = (packed >> 8) & 0xfu;        // tokens of a pass, wavefronts
  const bool s_fp16 = (packed >> 12 & 1u) != 0;
  typedef FewLds<MT> L;
  constexpr int XS = L::XS;
  constexpr bool DUAL = PASSES == BOTH_PASSES, EACH = PASSES == PASS_EACH;
  uint32_t pass = 0, slice = blockIdx.y, block = blockIdx.x;
  if (EACH) {         // unit u of both passes: neighbours on one XCD, equal shares for the XCDs
    const uint32_t blocks = packed >> 16, u = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7u);
    pass = (blockIdx.x >> 3) & 1u; slice = u / blocks; block = u - slice * blocks;
  }
  constexpr uint32_t ROWS = 32 * MT, TPP = DUAL ? ROWS / 2 : ROWS;
  constexpr uint32_t ROWS_X = EACH ? 2 * ROWS : ROWS, GROUP_X = ROWS_X * 256;      // of a group in memory
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t lrow = lane & 31u, half = lane >> 5;     // MFMA operand: row of the wavefront, half of the k-step
  const uint32_t lr = lane >> 3, lc = lane & 7u;          // weight loads: row within an instruction's 8, 16-byte chunk
  const uint32_t ngrp = K >> 7;
  const uint32_t g0 = slice * per, g1 = min(g0 + per, ngrp);
  if (EACH && g0 >= ngrp) return;
  const uint32_t nb = (block * W + wave) * 32, n_own = nb + lrow;
  const uint32_t n = min(n_own, N - 1);
  const NibbleConsts nc = nibble_constants();
  constexpr uint32_t OUT_OF_RANGE = 0x80000000u;
  const i32x4 rx = {(int)(uint32_t)(uintptr_t)x, (int)(uint32_t)((uintptr_t)x >> 32), (int)(ngrp * GROUP_X), 0x00020000};
  const i32x4 rxs = {(int)(uint32_t)(uintptr_t)xsum, (int)(uint32_t)((uintptr_t)xsum >> 32), (int)(ngrp * ROWS_X * 4), 0x00020000};
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(w), 0, (int)((uint64_t)N * (K >> 1)), 0x00020000);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(s), 0, (int)((uint64_t)N * ngrp * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(ZP ? zp : s), 0, (int)((uint64_t)N * ngrp), 0x00020000);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
  unsigned char* const wtw = lds + L::WT + wave * 4096u;
  const uint32_t woff = (nb + lr) * (K >> 1) + lc * 16, wstep = 8 * (K >> 1), soff = n * ngrp;

  // y[m][4 b + c]: weight row n, tile row 32 m + 8 b + 4 half + c
  floatx16 y[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) y[m][r] = 0.0f;

  for (uint32_t gb = g0; gb < g1; gb += 8) {
    const uint32_t cnt = min(g1 - gb, 8u);
    if (gb != g0) __syncthreads();                  // the groups before have been read
    asm volatile("" ::: "memory");
    // First what the first two groups need: weights, activations, block sums, scales; behind it the other activations
    // and the second round of weights, which are on their way while the first groups are computed.  The wait for the
    // scales is one for everything before them, that for the second round of weights one for all activations.
    u32x4 wq[2][4];                                 // round r (groups gb + 2 r and the next) in r % 2: rows 8 i + lr, chunk lc
    auto wload = [&](int r) __attribute__((always_inline)) {
      const uint32_t wo = woff + (2u * r < cnt ? (gb + 2 * r) * 64u : OUT_OF_RANGE);
#pragma unroll
      for (int i = 0; i < 4; ++i) wq[r & 1][i] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(wo + i * wstep), 0, 0);
    };
    auto xload = [&](uint32_t first, uint32_t last) __attribute__((always_inline)) {
      for (uint32_t q = first * MT * 8 + wave; q < min(last, cnt) * MT * 8; q += W)
        QF_DTL(rx, lds0 + q * 1024, gb * GROUP_X + (EACH ? q / (MT * 8) + pass : 0u) * L::GROUP + q * 1024 + lane * 16);
    };
    xload(0, XS);
    if (wave < MT)
      QF_DTL(rxs, lds0 + L::SUMS + wave * 1024,
             gb * (ROWS_X * 4) + (EACH ? (wave * 1024 + lane * 16) / (ROWS * 4) + pass : 0u) * (ROWS * 4) + wave * 1024 + lane * 16);
    u32x4 sv;
    if (((ngrp | gb) & 1u) == 0) {
      sv = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)((soff + gb) * 2), 0, 0);
    } else {
      uint32_t h[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        h[j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)((soff + gb) * 2), 2 * j, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) sv[j] = h[2 * j] | (h[2 * j + 1] << 16);
    }
    uint32_t zv[2] = {0, 0};
    if (ZP && ((ngrp | gb) & 3u) == 0) {
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rz, (int)(soff + gb), 0, 0);
      zv[0] = v.x; zv[1] = v.y;
    } else if (ZP) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        zv[j >> 2] |= (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rz, (int)(soff + gb), j, 0) << (8 * (j & 3));
    }
    asm volatile("" ::: "memory");
    wload(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    wload(1);
    asm volatile("" ::: "memory");
    // noise of groups gb .. gb + 7 of the lane's row, by way of the wavefront's LDS: a counter serves eight groups, a
    // lane draws the variates of its half of them
    float z[8];
    {
      uint32_t* const zb = reinterpret_cast<uint32_t*>(wtw);          // [group of two counters][row]
      const uint32_t first = gb & 7u;
      uint32_t row_id = a.row_base, seed_lo = a.seed_lo, seed_hi = a.seed_hi;
      asm volatile("" : "+s"(row_id), "+s"(seed_lo), "+s"(seed_hi));       // (waited for here, not before the first loads)
      row_id += n;
      for (uint32_t c = 0; c < (first + cnt > 8 ? 2u : 1u); ++c) {
        const u32x4_t pw = philox4x32_10(row_id, (gb >> 3) + c, 0u, 0u, seed_lo, seed_hi);
        float v[4];
        normal_pair(half ? pw.z : pw.x, v[0], v[1]);
        normal_pair(half ? pw.w : pw.y, v[2], v[3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) zb[(c * 8 + half * 4 + i) * 32 + lrow] = __float_as_uint(v[i]);
      }
#pragma unroll
      for (int d = 0; d < 8; ++d) z[d] = __uint_as_float(zb[(first + d) * 32 + lrow]);
      asm volatile("" ::: "memory");                // read before the weights take the place
    }
    // a round to the wavefront's LDS buffer: row r, chunk c at 128 r + 16 (c ^ r % 8)
    auto wstore = [&](auto R_) __attribute__((always_inline)) {
      constexpr int r = decltype(R_)::value;
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(wtw + (8 * i + lr) * 128 + ((lc ^ lr) << 4)) = wq[r & 1][i];
      if (r < 2) wload(r + 2);
    };
    uint32_t wd[2][8];                              // the lane's 64 nibbles of a group
    auto wread = [&](auto D_) __attribute__((always_inline)) {
      constexpr int d = decltype(D_)::value;
      const uint32_t c0 = 4 * (d & 1) + 2 * half;
      const u32x4 w0 = *reinterpret_cast<const u32x4*>(wtw + lrow * 128 + ((c0 ^ (lrow & 7u)) << 4));
      const u32x4 w1 = *reinterpret_cast<const u32x4*>(wtw + lrow * 128 + (((c0 + 1) ^ (lrow & 7u)) << 4));
#pragma unroll
      for (int i = 0; i < 4; ++i) { wd[d & 1][i] = w0[i]; wd[d & 1][4 + i] = w1[i]; }
    };
    // the scales have landed, and with them everything requested before them
    asm volatile("" : "+v"(sv));
    __syncthreads();
    wstore(std::integral_constant<int, 0>());
    wread(std::integral_constant<int, 0>());

    // Group d and those behind it (nested, so that a wait for weights counts the weight loads that were issued in between and not the
    // least of several paths; the refills, in asm, it does not count and waits for).  Its last tile is rescaled behind the next group's first MFMAs, its first fragments are read
    // behind the last ones of the group before; the barrier of the ring stands in its second half, where nobody waits for
    // operands (at the head of a group, with everything begun and ended there: 3300 cycles a group of four tiles).
    constexpr int R = 4;                            // fragments read ahead of their MFMA
    // (One tile: three wavefronts a SIMD, and 135 registers too many.  Four with zero-points: 46 too many, which went to scratch memory
    // by the counter that the ring's waits count; without, steps of six layers of 7B widths, 33 / 64 tokens 1.045 / 1.113 -> 0.784 / 0.861
    // ms, five of 13B 1.439 / 1.529 -> 1.015 / 1.102; the plain kernel 0.960 / 1.056, 1.103 / 1.211.)
    constexpr bool LATE = MT > 1 && !(MT == 4 && ZP);
    bf16x8 xf[R], wf[8];
    floatx16 p[2];                                  // sums of the tile at work and of the one before
    float4 xg[4];                                   // block sums of the latter's, then the former's tile rows
    float se_last_p = 0.0f, se_last_m = 0.0f, cz_last = 0.0f;
    auto rescale = [&](int i, int m, int b, float se_p, float se_m, float cz) __attribute__((always_inline)) {
      const float se = DUAL && 2 * m + (b >= 2) >= MT ? se_m : se_p;
      const float4 x = xg[b];
      const floatx16& q = p[i];
      y[m][4 * b + 0] = __builtin_fmaf(se, __builtin_fmaf(cz, x.x, q[4 * b + 0]), y[m][4 * b + 0]);
      y[m][4 * b + 1] = __builtin_fmaf(se, __builtin_fmaf(cz, x.y, q[4 * b + 1]), y[m][4 * b + 1]);
      y[m][4 * b + 2] = __builtin_fmaf(se, __builtin_fmaf(cz, x.z, q[4 * b + 2]), y[m][4 * b + 2]);
      y[m][4 * b + 3] = __builtin_fmaf(se, __builtin_fmaf(cz, x.w, q[4 * b + 3]), y[m][4 * b + 3]);
    };
#pragma unroll
    for (int q = 0; q < R; ++q) xf[q] = *reinterpret_cast<const bf16x8*>(lds + q * 1024 + lane * 16);
    auto group = [&](auto&& self, auto D_) __attribute__((always_inline)) -> void {
      constexpr int d = decltype(D_)::value, Q = MT * 8;
      // the ring: group d + 1 has landed (those behind it may be on their way), everyone has read group d - 1, whose place
      // is refilled, a load behind every other MFMA
      constexpr bool wait = d + 1 >= XS && d < 7, refill = d >= 1 && d - 1 + XS < 8;
      constexpr int NR = (Q + (MT == 4 ? L::W : 4) - 1) / (MT == 4 ? L::W : 4), BAR = Q - 2 * NR;       // NR: loads of a wavefront
      static_assert(XS == 8 || BAR >= 0, "slots for the loads");
      const uint32_t refill_off = d - 1 + XS < (int)cnt ? (gb + d - 1 + XS) * GROUP_X + pass * L::GROUP + lane * 16 : OUT_OF_RANGE;
      const unsigned char* const xb = lds + (d % XS) * L::GROUP + lane * 16;
      const unsigned char* const xb_next = lds + ((d + 1) % XS) * L::GROUP + lane * 16;
      const float* const sums = reinterpret_cast<const float*>(lds + L::SUMS) + d * ROWS + 4 * half;
      const float eps = EACH && pass ? -a.eps_signed : a.eps_signed;
      const float s0 = scale_to_f32((d & 1) ? sv[d >> 1] >> 16 : sv[d >> 1] & 0xffffu, s_fp16);
      const float se_p = __builtin_fmaf(eps, z[d], s0), se_m = __builtin_fmaf(-eps, z[d], s0);
      const float cz = ZP ? -(128.0f + (float)((zv[d >> 2] >> (8 * (d & 3))) & 0xffu)) : -136.0f;
      wf[0] = unpack8_biased(wd[d & 1][0], nc);
      __builtin_amdgcn_sched_barrier(0);
      // one slot per MFMA: what else the wavefront has to do is dealt out behind them
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < 8; ++j) {               // k-step j: inputs 64 half + 8 j .. + 7 of the group
          const int q = m * 8 + j, i = (d * MT + m) & 1;
          const floatx16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
          p[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[q % R], wf[j], j == 0 ? zero : p[i], 0, 0, 0);
          // the next round's weights take the place of this one's, whose last group is in registers
          if constexpr ((d & 1) && d < 7)
            if (q == Q / 2) wstore(std::integral_constant<int, (d + 1) / 2>());
          if (q == BAR && (wait || refill)) {
            if (wait) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(MT == 4 && d < 6 ? NR : 0) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
          }
          if (refill && q > BAR && ((q - BAR) & 1)) {
            const uint32_t c = wave + ((q - BAR) >> 1) * W, r = c < (uint32_t)Q ? c : wave;      // (past the end: its first one again)
            QF_DTL(rx, lds0 + ((d + XS - 1) % XS) * L::GROUP + r * 1024, refill_off + r * 1024);
          }
          if (q + R < Q) xf[q % R] = *reinterpret_cast<const bf16x8*>(xb + (q + R) * 1024);
          else if (d < 7) xf[q % R] = *reinterpret_cast<const bf16x8*>(xb_next + (q + R - Q) * 1024);
          if (m == 0 && j < 7) wf[j + 1] = unpack8_biased(wd[d & 1][j + 1], nc);
          if (j >= 1 && j <= 4 && m > 0) rescale(i ^ 1, m - 1, j - 1, se_p, se_m, cz);
          if (LATE && j >= 1 && j <= 4 && m == 0 && d > 0) rescale(i ^ 1, MT - 1, j - 1, se_last_p, se_last_m, cz_last);
          if (j >= 4) xg[j - 4] = *reinterpret_cast<const float4*>(sums + m * 32 + 8 * (j - 4));
          if constexpr (d < 7)
            if (q == Q - 2) wread(std::integral_constant<int, d + 1>());
          __builtin_amdgcn_sched_barrier(0);
        }
      if (!LATE) {
#pragma unroll
        for (int b = 0; b < 4; ++b) rescale((d * MT + MT - 1) & 1, MT - 1, b, se_p, se_m, cz);
      }
      if (d < 7 && d + 1 < (int)cnt) {
        se_last_p = se_p; se_last_m = se_m; cz_last = cz;
        if constexpr (d < 7) self(self, std::integral_constant<int, d + 1>());
      } else if (LATE) {
#pragma unroll
        for (int b = 0; b < 4; ++b) rescale((d * MT + MT - 1) & 1, MT - 1, b, se_p, se_m, cz);
      }
    };
    group(group, std::integral_constant<int, 0>());
    __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): loads that nobody waited for would be waited for above
  }

  // partial sums of this slice
  const uint32_t rows = PASSES == ONE_PASS ? M : 2 * M;
  const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(part, 0, (int)((uint64_t)(slice + 1) * rows * N * 4), 0x00020000);
  if (n_own < N) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t tr = 32 * m + 8 * (r >> 2) + 4 * half + (r & 3), tok = tr % TPP;
        const uint32_t off = ((slice * rows + (tr / TPP + pass) * M + tok) * N + n_own) * 4u;
        if (tok < M) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[m][r]), rp, (int)off, 0, WRITE_THROUGH);
      }
  }
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");        // loads past the end still write the LDS
}
#undef QF_DTL

template <int MT, int PASSES, bool ZP>
hipError_t few_prepare() {
  return hipFuncSetAttribute((const void*)few_gemm_kernel<MT, PASSES, ZP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             FewLds<MT>::bytes(FewLds<MT>::W));
}
// Wavefronts per workgroup: the least time, rounds of a workgroup per compute unit, each (start and stores) + W.  Four tiles: six, as the
// refills of the ring are dealt out.
struct FewPlan { uint32_t waves, blocks, rounds; };
template <int MT>
FewPlan few_plan(uint32_t N, uint32_t slices) {
  const uint32_t tiles = (N + 31) / 32, cus = gemm_workgroups(1u << 20, 1u << 20);
  FewPlan best = {};
  for (uint32_t w = MT == 4 ? FewLds<MT>::W : 4; w <= FewLds<MT>::W; ++w) {
    const uint32_t blocks = (tiles + w - 1) / w, rounds = (uint32_t)(((uint64_t)blocks * slices + cus - 1) / cus);
    if (!best.waves || (uint64_t)rounds * (4 + w) < (uint64_t)best.rounds * (4 + best.waves)) best = {w, blocks, rounds};
  }
  return best;
}
template <int MT, int PASSES>
hipError_t few_launch(const GemmArgs& a, const FewPlan& p, float* ws, uint32_t ks, uint32_t per, hipStream_t st) {
  const uint32_t w = p.waves, blocks = p.blocks;
  const dim3 grid = PASSES == PASS_EACH ? dim3((blocks * ks + 7) / 8 * 16) : dim3(blocks, ks);
  const FewRest r = {a.row_base, a.seed_lo, a.seed_hi, a.eps_signed};
  const uint32_t packed = a.M | (w << 8) | (a.s_fp16 ? 1u << 12 : 0u) | (PASSES == PASS_EACH ? blocks << 16 : 0u);
  if (a.zp)
    few_gemm_kernel<MT, PASSES, true><<<grid, w * 64, FewLds<MT>::bytes(w), st>>>(a.x, a.w, a.s, a.xsum, a.N, a.K, per, packed, ws, a.zp, r);
  else
    few_gemm_kernel<MT, PASSES, false><<<grid, w * 64, FewLds<MT>::bytes(w), st>>>(a.x, a.w, a.s, a.xsum, a.N, a.K, per, packed, ws, nullptr, r);
  return hipGetLastError();
}
template <int MT, int PASSES>
hipError_t few_launch(const GemmArgs& a, float* ws, uint32_t ks, uint32_t per, hipStream_t st) {
  return few_launch<MT, PASSES>(a, few_plan<MT>(a.N, ks), ws, ks, per, st);
}
// Both passes of 33 to 64 tokens.  A workgroup for each pass has half the work, but unpacks every weight a second time; its
// launch is the faster one where it takes no more rounds (both launches' times, us, 64 tokens: 1024 x 1024 11.4 -> 5.8, 6144 x 2048 14.7 ->
// 11.6, 2048 x 8192 14.4 -> 13.8 and 16384 x 4096 34.0 -> 27.3; one round more: 12288 x 4096 20.1 -> 22.9, 11264 x 2048 15.0 ->
// 17.8, 22016 x 4096 36.5 -> 37.4, 15360 x 5120 35.6 -> 33.2).
hipError_t few_launch_wide(const GemmArgs& a, float* ws, uint32_t ks, uint32_t per, hipStream_t st) {
  const FewPlan both = few_plan<4>(a.N, ks), each = few_plan<2>(a.N, 2 * ks);
  if (each.rounds <= both.rounds && each.blocks < 65536u) return few_launch<2, PASS_EACH>(a, each, ws, ks, per, st);
  return few_launch<4, BOTH_PASSES>(a, both, ws, ks, per, st);
}

}  // namespace

hipError_t launch_few_gemm(const GemmArgs& a, float* ws, uint32_t ks, uint32_t per, hipStream_t st) {
  static bool ready = false;
  if (!ready) {
    hipError_t e = few_prepare<1, BOTH_PASSES, false>();
    if (e == hipSuccess) e = few_prepare<1, BOTH_PASSES, true>();
    if (e == hipSuccess) e = few_prepare<1, ONE_PASS, false>();
    if (e == hipSuccess) e = few_prepare<1, ONE_PASS, true>();
    if (e == hipSuccess) e = few_prepare<2, BOTH_PASSES, false>();
    if (e == hipSuccess) e = few_prepare<2, BOTH_PASSES, true>();
    if (e == hipSuccess) e = few_prepare<2, ONE_PASS, false>();
    if (e == hipSuccess) e = few_prepare<2, ONE_PASS, true>();
    if (e == hipSuccess) e = few_prepare<4, BOTH_PASSES, false>();
    if (e == hipSuccess) e = few_prepare<4, BOTH_PASSES, true>();
    if (e == hipSuccess) e = few_prepare<2, PASS_EACH, false>();
    if (e == hipSuccess) e = few_prepare<2, PASS_EACH, true>();
    if (e != hipSuccess) return e;
    ready = true;
  }
  if (!a.xsum || a.xp.M != a.M || a.xp.rows != few_pack(a.M, a.dual != 0).rows) return hipErrorInvalidValue;
  switch (a.xp.rows >> 5) {
    case 1: return a.dual ? few_launch<1, BOTH_PASSES>(a, ws, ks, per, st) : few_launch<1, ONE_PASS>(a, ws, ks, per, st);
    case 2: return a.dual ? few_launch<2, BOTH_PASSES>(a, ws, ks, per, st) : few_launch<2, ONE_PASS>(a, ws, ks, per, st);
    case 4: return a.dual ? few_launch_wide(a, ws, ks, per, st) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qzo
