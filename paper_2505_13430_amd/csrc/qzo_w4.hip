// W4A16 group-dequant GEMM with the Q-SPSA perturbation fused into the weight operand (paper Eq. 4-5):
//   Y[M,N] = X[M,K] * W_eff^T,  W_eff[n,k] = (s[n,k/128] + sigma*eps*z(row_base+n, k/128)) * (u[n,k] - zp),
// bf16 MFMA (v_mfma_f32_32x32x16_bf16) with fp32 accumulation; a weight is formed in fp32 and rounded to bf16 once.
//
// A workgroup of four wavefronts, one per SIMD, owns 32 MT tokens x 256 features (MT = 1 .. 8), a wavefront all its
// tokens and 64 of the features: 2 MT accumulator tiles, in AGPRs from MT = 5 on.  A wavefront unpacks the weights that
// it multiplies, in registers, one k-step ahead of the MFMAs: they pass through the LDS as nibbles (8 KB a k-tile, read
// by their wavefront only, no barrier), not as 32 KB of bf16 that eight wavefronts stored and fetched between barriers.
// What the LDS carries per k-tile of 256 x 256 outputs falls from 256 to 170 KB, and no weight is converted twice.
// Everything comes from memory by direct-to-LDS loads (swizzled on the memory side): activations into a ring of three
// stages, two k-tiles ahead, weights and scales into two slots of a group each, two k-tiles ahead.  One barrier per
// k-tile, in front of its last k-step, whose operands are in registers by then.
// A lone wavefront issues an instruction every four cycles, so an MFMA of 32 cycles leaves seven places: fragment reads,
// loads and the conversion (eight pieces per dword) are dealt out behind the MFMAs in source order, held by scheduling
// fences.  With the conversion in four pieces behind every other MFMA, all loads at the head of a k-tile and the next
// k-step's conversion sunk behind the noise's branch by the compiler a k-tile took 1.73 us, as it stands 1.58.
//
// The noise is drawn by one lane per row (64 rows, 64 lanes): a Philox counter serves eight groups, a Box-Muller pair
// two, one exchange between the wavefront's halves hands the perturbed scales to both.
//
// Per k-tile at MT = 8 on a full chip, against the kernel this one replaces (eight wavefronts in alternating phases,
// weight tile in the LDS), same board: 1.79 -> 1.58 us (1203 -> 1358 TFLOP/s), with zero-points 1.95 -> 1.64.  Counters
// (8192 x 12288 x 4096): 2990 cycles a k-tile at 1.66 GHz, 2048 of them MFMAs; wavefronts wait 31 % of them.  Timing-only
// variants (board with 1.69): loads not issued 1.59; noise left out -0.02 to -0.05; fragment reads left out -0.08.
// Lower tiles serve the sizes whose rounds of 256-token tiles are badly filled (w4_plan): steps at 7B widths, before ->
// after: 4 x 33 tokens 9.4 -> 6.6 ms, 8 x 200 with zero-points 45.2 -> 39.4, 16 x 64 28.2 -> 25.8; OPT-1.3B 16 x 256
// 21.8 -> 19.4; one linear 2048 x 11008 x 4096, both signs, 0.432 -> 0.336; the tests' smallest model 0.180 -> 0.119.  With a
// unit's first three k-tiles loaded ahead of the stores of the one before, the time around a k-loop fell from 6.4 to 3.8 us.
// The rotary embedding rides on the epilogue (rows in an order that gives a lane both features of a pair).  NormalFloat-4
// takes 6 % more per k-tile than int4 (products of a level by byte permutations): 4 x 100 tokens 21.7 -> 14.8 ms.
// The noise's instructions as straight-line pieces behind the MFMAs: 1.609 against 1.612 us a k-tile, not kept.
// Outputs are the same bit for bit whatever MT: every one sums the same k-steps in the same order.
#include "qzo_gemm_tile.hpp"
#include "qzo_nibble.hpp"
#include <algorithm>
#include <cstddef>
#include <type_traits>

namespace qzo {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

enum : int { W4_INT4 = 0, W4_ZP = 1, W4_NF4 = 2 };

// LDS: three stages of activations (a k-tile of 32 MT rows of 128 bytes), two slots of packed weights (a group of 256
// rows: 64 bytes each) with their scales and zero-points (a dword each).
template <int MT, int FMT>
struct W4Lds {
  static constexpr bool ZP = FMT == W4_ZP;
  static constexpr uint32_t X = MT * 4096u, W0 = 3 * X, W = 256 * 64, S = 256 * 4, SLOT = W + S * (ZP ? 2 : 1);
  static constexpr uint32_t RED = W0 + 2 * SLOT, BYTES = RED + 2048;      // RED: a double per thread (sum of squares)
  static constexpr int NW = ZP ? 6 : 5;            // load instructions per wavefront for a group's weights
  static_assert(BYTES <= 160 * 1024, "LDS of a compute unit");
};

#define Q4_DTL(INSTR, RSRC, LDSADDR, VOFF, SOFF)                                             \
  asm volatile(QZO_SET_M0 INSTR " %1, %2, %3 offen lds"                                      \
               : : "s"(LDSADDR), "v"(VOFF), "s"(RSRC), "s"(SOFF) : "memory", "m0")

#define Q4_INLINE __attribute__((always_inline))
template <int V>
using Int = std::integral_constant<int, V>;

// What a wavefront needs later than its first loads.  (Those want x .. zp, which arrive in registers; an argument read from
// memory takes 1.2 us.)
struct W4Rest {
  void* y;
  const void *resid, *bias;
  float *partials, *split_ws;
  const float* rope;
  uint32_t rope_S, ldy, row_base, seed_lo, seed_hi;
  float eps_signed;
};
struct W4Args {
  const void *x, *w, *s;
  uint32_t M, N, K, second_row, kt_per, packed;
  const void* zp;
  W4Rest rest;
};
// The rest, read where it is asked for: left to itself the compiler reads all of it first and waits.
typedef const __attribute__((address_space(4))) W4Rest* W4RestPtr;
__device__ __forceinline__ W4RestPtr w4_rest() {
  auto p = (const __attribute__((address_space(4))) unsigned char*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(W4Args, rest);
  asm volatile("" : "+s"(p));
  return (W4RestPtr)p;
}
// packed: epilogue flags, fp16 scales, heads of 128, workgroups, K slices.  No K slices (0): all of K, and kt_per holds the
// launch's feature tiles in its place (w4_columns), so that the arguments of the first loads fit the registers.
__host__ __device__ constexpr uint32_t w4_pack(uint32_t epi, bool s_fp16, bool rope128, uint32_t wgs, uint32_t ksplit) {
  return epi | (s_fp16 ? 64u : 0u) | (rope128 ? 128u : 0u) | (wgs << 8) | (ksplit << 20);
}

__host__ __device__ constexpr uint32_t w4_columns(uint32_t first_n, uint32_t tiles_n) { return first_n | (tiles_n << 16); }

template <int MT, int FMT>
__global__ __launch_bounds__(256, 1) void w4_gemm_kernel(const void* x, const void* w, const void* s, uint32_t M, uint32_t N, uint32_t K,
                                                         uint32_t second_row, uint32_t kt_per_or_columns, uint32_t packed, const void* zp,
                                                         W4Rest) {
  typedef W4Lds<MT, FMT> L;
  constexpr bool ZP = FMT == W4_ZP, NF4 = FMT == W4_NF4;
  constexpr int SLOTS = 2 * MT;                    // MFMAs of a k-step
  // A byte offset beyond every buffer (each is below 2^31 bytes), and an index of scales whose byte offset (times 1, 2 or
  // 4: zero-points, scales, pairs of NormalFloat-4 scales) is beyond theirs (at most N K / 32 < 2^27 bytes, and a group's
  // offset on top of it does not wrap).
  constexpr uint32_t OUT_OF_RANGE = 0x80000000u, SCALE_OUT_OF_RANGE = OUT_OF_RANGE >> 2, SCALE_BYTES = NF4 ? 4 : 2;
  static_assert((uint64_t)SCALE_OUT_OF_RANGE * SCALE_BYTES + (1u << 27) < (1ull << 32) && SCALE_OUT_OF_RANGE >= (1u << 27));
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t lrow = lane & 31u, half = lane >> 5;
  const uint32_t G = K >> 7, epi = packed & 63u, wgs = (packed >> 8) & 0xfffu, ksplit = packed >> 20;
  const uint32_t kt_per = ksplit ? kt_per_or_columns : K / BK, first_n = ksplit ? 0u : kt_per_or_columns & 0xffffu;
  const bool swiglu = (epi & EPI_SWIGLU) != 0, rope = (epi & EPI_ROPE) != 0, s_fp16 = (packed & 64u) != 0;
  const bool rope128 = (packed & 128u) != 0;
  const uint32_t tiles_n = ksplit ? (N + 255u) >> 8 : kt_per_or_columns >> 16, tiles_per_pass = (M + 32 * MT - 1) / (32 * MT);
  TileWalk walk = tile_walk_of(second_row ? 2 * tiles_per_pass : tiles_per_pass, ksplit ? tiles_n * ksplit : tiles_n, wgs);
  uint32_t tile_m, tile_n;
  if (!tile_walk_get(walk, tile_m, tile_n)) {
    if ((epi & EPI_SUMSQ) && threadIdx.x == 0) w4_rest()->partials[blockIdx.x] = 0.0f;
    return;
  }

  auto rsrc = [](const void* q, uint64_t bytes) {
    return i32x4{(int)(uint32_t)(uintptr_t)q, (int)(uint32_t)((uintptr_t)q >> 32), (int)bytes, 0x00020000};
  };
  const uint32_t rows_all = second_row ? second_row + M : M;
  const i32x4 rx = rsrc(x, (uint64_t)rows_all * K * 2), rw = rsrc(w, (uint64_t)N * (K >> 1));
  const i32x4 rs = rsrc(s, (uint64_t)N * G * SCALE_BYTES), rz = rsrc(ZP ? zp : s, (uint64_t)N * G);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // a unit of work: K slice kslice of output tile (tile_m, tile_n), k-tiles kt0 .. kt0 + 2 ng - 1
  uint32_t kslice, kt0, ng, row0, row_last, own, noise_row, pass;
  uint32_t xo[MT], wo[4], so;
  float eps;
  auto point = [&]() Q4_INLINE {
    kslice = ksplit > 1 ? tile_n / tiles_n : 0u;
    tile_n = first_n + tile_n - kslice * tiles_n;
    kt0 = kslice * kt_per;
    ng = min(kt_per, K / BK - kt0) >> 1;
    pass = tile_m >= tiles_per_pass ? 1u : 0u;
    row0 = pass * second_row + (tile_m - pass * tiles_per_pass) * (32 * MT);
    row_last = pass * second_row + M - 1;
    // fused SwiGLU: a wavefront's rows are 32 gate rows and the 32 up rows of the same features; rotary embedding of
    // heads of 128 (N % 256 == 0): 32 features and their partners 64 further on
    auto wrow = [&](uint32_t r) Q4_INLINE {
      if (rope128) return tile_n * 256u + (r >> 7) * 128u + ((r >> 6) & 1u) * 32u + ((r >> 5) & 1u) * 64u + (r & 31u);
      return swiglu ? ((r >> 5) & 1u) * (N >> 1) + tile_n * 128u + (r >> 6) * 32u + (r & 31u)
                    : min(tile_n * 256u + r, N - 1);
    };
    // a load instruction fills 1 KB of LDS in lane order: 8 rows of 128 bytes of activations, 16 rows of 64 bytes of
    // weights; the swizzles of their 16-byte chunks are applied on the memory side
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const uint32_t row = 8 * (4 * i + wave) + (lane >> 3);
      xo[i] = min(row0 + row, row_last) * K * 2 + (((lane & 7u) ^ ((row >> 1) & 7u)) << 4) + kt0 * (BK * 2);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      wo[q] = wrow(wave * 64 + 16 * q + (lane >> 2)) * (K >> 1) + (((lane & 3u) ^ ((lane >> 4) & 3u)) << 4) + kt0 * (BK / 2);
    own = wrow(wave * 64 + lane);
    so = own * G + (kt0 >> 1);
  };
  auto load_x = [&](int i, uint32_t kt, uint32_t stage) Q4_INLINE {
    Q4_DTL("buffer_load_dwordx4", rx, lds0 + stage + (4 * i + wave) * 1024, xo[i], kt * (BK * 2));
  };
  auto load_w = [&](int q, uint32_t g, uint32_t slot) Q4_INLINE {
    const uint32_t base = lds0 + L::W0 + slot;
    if (q < 4) Q4_DTL("buffer_load_dwordx4", rw, base + wave * 4096 + q * 1024, wo[q], g * 64);
    else if (q == 4 && NF4) Q4_DTL("buffer_load_dword", rs, base + L::W + wave * 256, so * SCALE_BYTES, g * SCALE_BYTES);    // of two blocks
    else if (q == 4) Q4_DTL("buffer_load_ushort", rs, base + L::W + wave * 256, so * SCALE_BYTES, g * SCALE_BYTES);
    else Q4_DTL("buffer_load_ubyte", rz, base + L::W + L::S + wave * 256, so, g);
  };
  auto request_first = [&]() Q4_INLINE {       // groups 0 and 1, k-tiles 0, 1 and 2, in the order the k-loop goes on with
#pragma unroll
    for (int q = 0; q < L::NW; ++q) load_w(q, 0u, 0u);
#pragma unroll
    for (int i = 0; i < MT; ++i) load_x(i, 0u, 0u);
    if (ng < 2) {
#pragma unroll
      for (int q = 0; q < 4; ++q) wo[q] = OUT_OF_RANGE;
      so = SCALE_OUT_OF_RANGE;
    }
#pragma unroll
    for (int q = 0; q < L::NW; ++q) load_w(q, 1u, L::SLOT);
#pragma unroll
    for (int i = 0; i < MT; ++i) load_x(i, 1u, L::X);
    if (ng < 2) {
#pragma unroll
      for (int i = 0; i < MT; ++i) xo[i] = OUT_OF_RANGE;
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) load_x(i, 2u, 2 * L::X);
  };

  // fragment addresses: activations: row lrow (+ 32 i), chunk of k-step ks; weights: row lrow (+ 32 j), the dwords of
  // chunk c that hold the eight inputs of the lane's half of k-steps 2 c and 2 c + 1
  uint32_t xrd[4], wrd[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) xrd[ks] = lrow * 128u + (((uint32_t)(ks * 2 + half) ^ ((lrow >> 1) & 7u)) << 4);
#pragma unroll
  for (int c = 0; c < 4; ++c) wrd[c] = L::W0 + wave * 4096 + lrow * 64u + (((uint32_t)c ^ ((lrow >> 2) & 3u)) << 4) + half * 4;

  floatx16 acc[MT][2];
  bf16x8 fx[2][MT], fw[2][2];
  uint32_t raw[2][8];                               // nibbles of the group: [feature tile][k-step of the group]
  float se[2], m8[2];                               // per feature tile: operands of the conversion
  float z_even = 0.0f, z_odd = 0.0f;
  uint32_t zw0 = 0, zw1 = 0, zw2 = 0, zw3 = 0, sbits = 0, zbits = 0;
  const floatx16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

  auto read_raw = [&](int c, uint32_t slot) Q4_INLINE {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t* q = reinterpret_cast<const uint32_t*>(lds + (wrd[c] + slot) + j * 2048);
      raw[j][2 * c] = q[0];
      raw[j][2 * c + 1] = q[2];
    }
  };
  auto read_scale = [&](uint32_t slot) Q4_INLINE {
    sbits = *reinterpret_cast<const uint32_t*>(lds + L::W0 + slot + L::W + wave * 256 + lane * 4);
    if (ZP) zbits = *reinterpret_cast<const uint32_t*>(lds + L::W0 + slot + L::W + L::S + wave * 256 + lane * 4);
  };
  // noise of the lane's own row: a counter serves eight scales, a word two: those of two groups, or of the two blocks of
  // a NormalFloat-4 group g
  uint32_t row_base, seed_lo, seed_hi;
  float eps_signed;
  auto noise = [&](uint32_t g, bool first) Q4_INLINE {
    const uint32_t pair = NF4 ? g : g >> 1;
    if (first || ((pair & 3u) == 0 && (NF4 || (g & 1u) == 0))) {
      const u32x4_t w = philox4x32_10(noise_row, pair >> 2, 0u, 0u, seed_lo, seed_hi);
      zw0 = w.x; zw1 = w.y; zw2 = w.z; zw3 = w.w;
    }
    if (NF4 || (g & 1u) == 0) {
      const uint32_t q = pair & 3u, w0 = zw0, w1 = zw1, w2 = zw2, w3 = zw3;
      float even, odd;
      normal_pair(q == 0 ? w0 : (q == 1 ? w1 : (q == 2 ? w2 : w3)), even, odd);
      z_even = even; z_odd = odd;
    }
  };
  // the lane's row is row lane of the wavefront's 64: one exchange between the halves gives every lane its two tiles'
  // n: the group, of a NormalFloat-4 group the block
  auto new_scale = [&](uint32_t n) Q4_INLINE {
    const float even = z_even, odd = z_odd;
    const float s = __builtin_fmaf(eps, (n & 1u) ? odd : even, scale_to_f32(NF4 && (n & 1u) ? sbits >> 16 : sbits & 0xffffu, s_fp16));
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    const float s0 = __uint_as_float(r[0]), s1 = __uint_as_float(r[1]);
    if (ZP) {
      const float nz = -(float)(zbits & 0xffu);
      const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(nz), __float_as_uint(nz), false, false);
      se[0] = s0; se[1] = s1;
      m8[0] = __uint_as_float(q[0]); m8[1] = __uint_as_float(q[1]);
    } else if (NF4) {
      se[0] = s0; se[1] = s1;
    } else {
      se[0] = 512.0f * s0; se[1] = 512.0f * s1;
      m8[0] = -8.0f * s0; m8[1] = -8.0f * s1;
    }
  };
  // Conversion of a dword of nibbles in eight pieces.  A byte holding a nibble u read as an fp8 E4M3 pattern is exactly
  // u * 2^-9: fma(u 2^-9, 512 se, -8 se) is (u-8)*se with one rounding; with zero-points fma(u 2^-9, 512, -zp) is the
  // integer u - zp and its product with se is rounded once.
  typedef float f2 __attribute__((ext_vector_type(2)));
  union Frag { bf16x8 v; uint32_t u[4]; };
  f2 cl, ch;
  uint32_t clo, chi;
  float ce0, ce1;
  Frag cf;
  auto weight = [&](float u, int j) Q4_INLINE {
    return ZP ? __builtin_fmaf(u, 512.0f, m8[j]) * se[j] : __builtin_fmaf(u, se[j], m8[j]);
  };
  // NormalFloat-4: products of scale and level, rounded, in tables per feature tile (this k-tile's and the next one's); a
  // dword's eight are looked up by byte permutations (unpack8_nf4)
  Nf4Table tab[NF4 ? 2 : 1], tab_next[NF4 ? 2 : 1];
  Nf4Select sel;
  uint32_t nf_a = 0, nf_b = 0;
  auto next_table = [&](int piece) Q4_INLINE { if constexpr (NF4) nf4_table_part(tab_next[piece >> 2], se[piece >> 2], piece & 3); };
  auto use_table = [&]() Q4_INLINE { if constexpr (NF4) { tab[0] = tab_next[0]; tab[1] = tab_next[1]; } };
  auto convert = [&](int buf, int piece, int kk) Q4_INLINE {
    const int j = piece >> 3;
    if constexpr (NF4) {
      const uint32_t w = raw[j][kk];
      const Nf4Table& t = tab[j];
      switch (piece & 7) {
        case 0: sel.sel = nf4_entries_a(w); break;
        case 1: sel.upper = nf4_upper_a(w); break;
        case 2: nf_a = nf4_bytes(t.lo, sel); break;
        case 3: nf_b = nf4_bytes(t.hi, sel); break;
        case 4: nf4_merge(nf_b, nf_a, cf.u[0], cf.u[2]); sel.sel = nf4_entries_b(w); break;
        case 5: sel.upper = nf4_upper_b(w); break;
        case 6: nf_a = nf4_bytes(t.lo, sel); break;
        default: nf_b = nf4_bytes(t.hi, sel); nf4_merge(nf_b, nf_a, cf.u[1], cf.u[3]); fw[buf][j] = cf.v;
      }
      return;
    }
    switch (piece & 7) {
      case 0: clo = raw[j][kk] & 0x0f0f0f0fu; chi = (raw[j][kk] >> 4) & 0x0f0f0f0fu; break;
      case 1: cl = __builtin_amdgcn_cvt_pk_f32_fp8(clo, false); ch = __builtin_amdgcn_cvt_pk_f32_fp8(chi, false); break;
      case 2: ce0 = weight(cl.x, j); ce1 = weight(ch.x, j); break;
      case 3: cf.u[0] = pack_bf16x2(ce0, ce1); ce0 = weight(cl.y, j); ce1 = weight(ch.y, j); break;
      case 4: cf.u[1] = pack_bf16x2(ce0, ce1); cl = __builtin_amdgcn_cvt_pk_f32_fp8(clo, true); break;
      case 5: ch = __builtin_amdgcn_cvt_pk_f32_fp8(chi, true); ce0 = weight(cl.x, j); ce1 = weight(ch.x, j); break;
      case 6: cf.u[2] = pack_bf16x2(ce0, ce1); ce0 = weight(cl.y, j); ce1 = weight(ch.y, j); break;
      default: cf.u[3] = pack_bf16x2(ce0, ce1); fw[buf][j] = cf.v;
    }
  };
  auto read_x = [&](int buf, int i, int ks, uint32_t stage) Q4_INLINE {
    fx[buf][i] = *reinterpret_cast<const bf16x8*>(lds + (xrd[ks] + stage) + i * 4096);
  };

  uint32_t st_cur = 0, st_next = L::X, st_load = 2 * L::X;      // stages of k-tiles t, t + 1, t + 2
  // k-step S of k-tile D of a group: its MFMAs with, dealt out between them, the fragment reads and the conversion for
  // the next k-step, and a share of the loads: from the barrier before step 3 of a k-tile to the next barrier those of
  // the k-tile after the next one and, once per group, of the weights of the group after the next one.
  constexpr int ODD = 1;
  auto loads = [&](auto E_, int first, int count, uint32_t g, uint32_t slot, uint32_t stage) Q4_INLINE {
    constexpr int E = decltype(E_)::value;          // k-tile of its group that the loads are issued for
#pragma unroll
    for (int n = 0; n < MT + L::NW; ++n)
      if (n >= first && n < first + count) {
        if (E == ODD && n < L::NW) load_w(n, g + 2, slot);
        else if (n < MT + (E == ODD ? L::NW : 0)) load_x(n - (E == ODD ? L::NW : 0), 2 * g + E + 2, stage);
      }
  };
  // START: the unit's first group: its accumulators start from zero, its third k-tile is on its way already.
  auto step = [&](auto S_, auto D_, auto START_, uint32_t g, uint32_t slot) Q4_INLINE {
    constexpr int S = decltype(S_)::value, D = decltype(D_)::value;
    constexpr bool START = decltype(START_)::value != 0, FIRST = START && D == 0 && S == 0;
    constexpr int buf = S & 1, nb = buf ^ 1, ks = (S + 1) & 3, kk = (D * 4 + S + 1) & 7;
    // load slots: steps 3, 0, 1, 2 in this order; E: the k-tile whose list they belong to
    constexpr int E = S == 3 ? D ^ 1 : D, NL = MT + (E ? L::NW : 0), Q = (S + 1) & 3;
    const uint32_t stage = S == 3 ? st_next : st_cur, lg = S == 3 && D ? g + 1 : g;
#pragma unroll
    for (int m = 0; m < SLOTS; ++m) {
      const int i = m >> 1, j = m & 1;
      if (FIRST) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[buf][j], fx[buf][i], zero16, 0, 0, 0);
      else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[buf][j], fx[buf][i], acc[i][j], 0, 0, 0);
      // S = 2: denser, the barrier that follows waits for them
      if (S == 2 ? m < MT : (m & 1) == 0) read_x(nb, S == 2 ? m : m >> 1, ks, stage);
      const int l0 = (Q * SLOTS + m) * NL / (4 * SLOTS), l1 = (Q * SLOTS + m + 1) * NL / (4 * SLOTS);
      if (!(START && D == 0 && S < 3)) loads(Int<E>(), l0, l1 - l0, lg, slot, S == 3 ? st_cur : st_load);
#pragma unroll
      for (int c = m * 16 / SLOTS; c < (m + 1) * 16 / SLOTS; ++c) convert(nb, c, kk);
      if (NF4 && S < 2) {
#pragma unroll
        for (int c = m * 4 / SLOTS; c < (m + 1) * 4 / SLOTS; ++c) next_table(S * 4 + c);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // keeps the conversion here (single uses behind a branch would be moved there, with no MFMA to hide behind)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      u32x4 pin = __builtin_bit_cast(u32x4, fw[nb][j]);
      asm volatile("" : "+v"(pin));
      fw[nb][j] = __builtin_bit_cast(bf16x8, pin);
    }
  };
  // Ends a k-tile: all but the LEFT loads issued last have landed, as far as this wavefront's go, and everyone is past
  // its fragment reads.  In a unit's first group the stores of the epilogue before may be among the youngest.
  uint32_t stores = 0;                              // of the last epilogue, issued behind the unit's first loads
  auto sync = [&](auto LEFT_, auto START_) Q4_INLINE {
    constexpr int LEFT = decltype(LEFT_)::value;
    if (decltype(START_)::value && stores == 4 * MT)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(std::min(63, LEFT + 4 * MT)) : "memory");
    else if (decltype(START_)::value && stores == 2 * MT)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(std::min(63, LEFT + 2 * MT)) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(LEFT) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto next_stage = [&]() Q4_INLINE {
    const uint32_t o = st_cur;
    st_cur = st_next; st_next = st_load; st_load = o;
  };
  auto group = [&](uint32_t g, auto START_) Q4_INLINE {
    const uint32_t slot = (g & 1u) ? L::SLOT : 0u, other = L::SLOT - slot, gb = (kt0 >> 1) + g;
    if (g + 2 >= ng) {
#pragma unroll
      for (int q = 0; q < 4; ++q) wo[q] = OUT_OF_RANGE;
      so = SCALE_OUT_OF_RANGE;
    }
    read_raw(2, slot); read_raw(3, slot);
    if (NF4) new_scale(1u);                         // of the second block, for k-tile 1
    step(Int<0>(), Int<0>(), START_, g, slot);
    step(Int<1>(), Int<0>(), START_, g, slot);
    noise(gb + 1, false);
    __builtin_amdgcn_sched_barrier(0);
    step(Int<2>(), Int<0>(), START_, g, slot);
    sync(Int<MT>(), START_);
    if (NF4) { use_table(); read_scale(other); }
    step(Int<3>(), Int<0>(), START_, g, slot);
    next_stage();
    read_raw(0, other); read_raw(1, other);
    if (NF4) new_scale(0u);
    else read_scale(other);
    step(Int<0>(), Int<1>(), START_, g, slot);
    step(Int<1>(), Int<1>(), START_, g, slot);
    step(Int<2>(), Int<1>(), START_, g, slot);
    sync(Int<MT + L::NW>(), START_);
    if (NF4) use_table();
    else new_scale(gb + 1);
    if (g + 2 >= ng) {
#pragma unroll
      for (int i = 0; i < MT; ++i) xo[i] = OUT_OF_RANGE;
    }
    step(Int<3>(), Int<1>(), START_, g, slot);
    next_stage();
  };

  // sum of squares: unit by unit in double, in the LDS (no register is held over the k-loop): fp32 sums that go on over all
  // units lose up to 1.5e-5 where the terms are alike.  One linear 2048 x 11008 x 4096, both signs, against such sums:
  // 0.337 against 0.336 ms (two runs of either differ by 0.4 %); with a wavefront's sum taken per unit 1.2 % more.
  double* const ssq_units = reinterpret_cast<double*>(lds + L::RED) + t;
  if (epi & EPI_SUMSQ) *ssq_units = 0.0;

  point();
  request_first();
  {
    const W4RestPtr a = w4_rest();
    row_base = a->row_base; seed_lo = a->seed_lo; seed_hi = a->seed_hi; eps_signed = a->eps_signed;
  }
  for (;;) {
    noise_row = row_base + own;
    eps = pass ? -eps_signed : eps_signed;
    sync(Int<2 * MT + L::NW>(), Int<1>());          // the first group's weights and the first k-tile have landed
    st_cur = 0; st_next = L::X; st_load = 2 * L::X;
    read_raw(0, 0u); read_raw(1, 0u); read_scale(0u);
#pragma unroll
    for (int i = 0; i < MT; ++i) read_x(0, i, 0, 0u);
    noise(kt0 >> 1, true);
    new_scale(NF4 ? 0u : kt0 >> 1);
    if (NF4) {
#pragma unroll
      for (int c = 0; c < 8; ++c) next_table(c);
      use_table();
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) convert(0, c, 0);
    __builtin_amdgcn_sched_barrier(0);
    group(0u, Int<1>());
    for (uint32_t g = 1; g < ng; ++g) group(g, Int<0>());

    const uint32_t r0 = row0, m0 = row0 + lrow, m_last = row_last, n0 = tile_n * 256u + wave * 64u, slice = kslice;
    const uint32_t done_n = tile_n;
    tile_walk_next(walk);
    const bool more = tile_walk_get(walk, tile_m, tile_n);
    if (more) {                 // every wavefront is past the barrier that ended the last k-tile
      point();
      request_first();
    }
    const W4RestPtr a = w4_rest();
    // output rows and features of a lane: token row0 + 32 i + lrow, features 8 b + 4 half + c of feature tile j; after
    // QZO swap of two register groups a lane owns eight consecutive features
    const uint32_t ldy = a->ldy ? a->ldy : N, NO = swiglu ? N >> 1 : N;
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
        a->y, 0, (int)(((uint64_t)(rows_all - 1) * (swiglu ? NO : ldy) + NO) * 2), 0x00020000);
    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
// accumulators are read out one piece at a time (left to itself the compiler copies all of them to vector registers)
#define Q4_ACC(I, J, R, DST)                                                                 \
  do {                                                                                       \
    if constexpr (MT >= 5) asm("v_accvgpr_read_b32 %0, %1" : "=v"(DST) : "a"(acc[I][J][R])); \
    else DST = acc[I][J][R];                                                                 \
  } while (0)
#define Q4_SWAP8(LO, HI)                                                                     \
  do {                                                                                       \
    _Pragma("unroll") for (int c_ = 0; c_ < 4; ++c_) {                                       \
      const auto r_ = __builtin_amdgcn_permlane32_swap(__float_as_uint((LO)[c_]),            \
                                                       __float_as_uint((HI)[c_]), false, false); \
      (LO)[c_] = __uint_as_float(r_[0]);                                                     \
      (HI)[c_] = __uint_as_float(r_[1]);                                                     \
    }                                                                                        \
  } while (0)
    if (ksplit > 1) {
      // this slice's fp32 sums, [slice][rows][N]; the epilogue proper runs in the reduction
      const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
          a->split_ws + ((uint64_t)slice * rows_all + r0) * N, 0, (int)((m_last - r0 + 1) * N * 4), 0x00020000);
#pragma unroll
      for (int u = 0; u < 4 * MT; ++u) {
        const int i = u >> 2, j = (u >> 1) & 1, bp = u & 1;
        float v[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) Q4_ACC(i, j, 4 * (2 * bp + h) + c, v[h][c]);
        Q4_SWAP8(v[0], v[1]);
        const uint32_t m = m0 + i * 32, n = n0 + j * 32 + (2u * bp + half) * 8u;
        const uint32_t o = m <= m_last && n < N ? ((m - r0) * N + n) * 4u : OUT_OF_RANGE;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(v[h][0]), __float_as_uint(v[h][1]), __float_as_uint(v[h][2]),
                                                       __float_as_uint(v[h][3])}, rp, (int)(o + 16 * h), 0, 0);
        if (u & 1) __builtin_amdgcn_sched_barrier(0);
      }
      stores = 1;
    } else if (swiglu) {
      // y[m, f] = silu(gate) * up, f = 128 tile_n + 32 wave + 8 b + 4 half + c; y is [rows, N/2]
#pragma unroll
      for (int u = 0; u < 2 * MT; ++u) {
        const int i = u >> 1, bp = u & 1;
        float v[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            float gt, up;
            Q4_ACC(i, 0, 4 * (2 * bp + h) + c, gt);
            Q4_ACC(i, 1, 4 * (2 * bp + h) + c, up);
            v[h][c] = gt * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * gt)) * up;
          }
        Q4_SWAP8(v[0], v[1]);
        const uint32_t m = m0 + i * 32, f = done_n * 128u + wave * 32u + (2u * bp + half) * 8u;
        const u32x4 out = {pack_bf16x2(v[0][0], v[0][1]), pack_bf16x2(v[0][2], v[0][3]),
                           pack_bf16x2(v[1][0], v[1][1]), pack_bf16x2(v[1][2], v[1][3])};
        __builtin_amdgcn_raw_buffer_store_b128(out, ry, (int)(m <= m_last ? (m * NO + f) * 2u : OUT_OF_RANGE), 0, 0);
        if (u & 1) __builtin_amdgcn_sched_barrier(0);
      }
      stores = 2 * MT;
    } else if (rope) {
      // qkv [rows, 3d] with the rotary embedding on its q and k thirds: the wavefront's two feature tiles hold feature f
      // and feature f + dh/2 of a head for the same token.  An output is rounded to bf16 first (what a separate pass
      // would read), rotated in fp32 at its position and rounded again.
      const uint32_t hd = rope128 ? 64u : 32u;
      const uint32_t na = (rope128 ? done_n * 256u + (wave >> 1) * 128u + (wave & 1u) * 32u : n0) + half * 8u;
      const bool rotate = na < (N / 3u) * 2u;            // a wavefront's columns lie within one third of qkv
      const float2* table = reinterpret_cast<const float2*>(a->rope) + (rope128 ? (wave & 1u) * 32u : 0u) + half * 8u;
      const uint32_t pass_row0 = m0 >= second_row ? second_row : 0u;
      // the (cos, sin) values of a step are requested AHEAD steps before they are used
      auto table_of = [&](int u) Q4_INLINE {
        const uint32_t pos = (min(m0 + (u >> 1) * 32, m_last) - pass_row0) % a->rope_S;
        return reinterpret_cast<const float4*>(table + (uint64_t)pos * hd + (u & 1) * 16u);
      };
      constexpr int AHEAD = NF4 && MT == 8 ? 2 : 4;        // (registers)
      float4 tn[AHEAD][4] = {};
      if (rotate) {
#pragma unroll
        for (int u = 0; u < AHEAD && u < 2 * MT; ++u)
#pragma unroll
          for (int q = 0; q < 4; ++q) tn[u][q] = table_of(u)[q];
      }
#pragma unroll
      for (int u = 0; u < 2 * MT; ++u) {
        const int i = u >> 1, bp = u & 1;
        float4 cs[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) cs[q] = tn[u % AHEAD][q];
        if (rotate && u + AHEAD < 2 * MT) {
#pragma unroll
          for (int q = 0; q < 4; ++q) tn[u % AHEAD][q] = table_of(u + AHEAD)[q];
        }
        float va[2][4], vb[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            Q4_ACC(i, 0, 4 * (2 * bp + h) + c, va[h][c]);
            Q4_ACC(i, 1, 4 * (2 * bp + h) + c, vb[h][c]);
          }
        Q4_SWAP8(va[0], va[1]);
        Q4_SWAP8(vb[0], vb[1]);
        u32x4 oa = {pack_bf16x2(va[0][0], va[0][1]), pack_bf16x2(va[0][2], va[0][3]),
                    pack_bf16x2(va[1][0], va[1][1]), pack_bf16x2(va[1][2], va[1][3])};
        u32x4 ob = {pack_bf16x2(vb[0][0], vb[0][1]), pack_bf16x2(vb[0][2], vb[0][3]),
                    pack_bf16x2(vb[1][0], vb[1][1]), pack_bf16x2(vb[1][2], vb[1][3])};
        if (rotate) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {                    // cs[q]: (cos, sin) of pairs 2 q and 2 q + 1
            const float a0 = __uint_as_float(oa[q] << 16), a1 = __uint_as_float(oa[q] & 0xffff0000u);
            const float b0 = __uint_as_float(ob[q] << 16), b1 = __uint_as_float(ob[q] & 0xffff0000u);
            oa[q] = pack_bf16x2(a0 * cs[q].x - b0 * cs[q].y, a1 * cs[q].z - b1 * cs[q].w);
            ob[q] = pack_bf16x2(b0 * cs[q].x + a0 * cs[q].y, b1 * cs[q].z + a1 * cs[q].w);
          }
        }
        const uint32_t m = m0 + i * 32, n = na + bp * 16u;
        const bool inside = m <= m_last && n < N;
        const uint32_t o = (m * N + n) * 2u;
        __builtin_amdgcn_raw_buffer_store_b128(oa, ry, (int)(inside ? o : OUT_OF_RANGE), 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(ob, ry, (int)(inside ? o + hd * 2u : OUT_OF_RANGE), 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      stores = 4 * MT;
    } else {
      const bool with_resid = (epi & EPI_RESIDUAL) != 0, with_bias = (epi & EPI_BIAS) != 0;
      const __amdgpu_buffer_rsrc_t rr_ = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<void*>(with_resid ? a->resid : a->y), 0, (int)(((uint64_t)(rows_all - 1) * ldy + N) * 2), 0x00020000);
      auto at = [&](int u) Q4_INLINE {
        const uint32_t m = m0 + (u >> 2) * 32, n = n0 + ((u >> 1) & 1) * 32 + (2u * (u & 1) + half) * 8u;
        return m <= m_last && n < N ? (m * ldy + n) * 2u : OUT_OF_RANGE;
      };
      // residuals are requested AHEAD pieces before they are used: a few memory latencies per tile, not one per piece
      constexpr int AHEAD = NF4 && MT == 8 ? 8 : 12;
      u32x4 rr[AHEAD];
      uint4 bb[4];
      if (with_resid) {
#pragma unroll
        for (int u = 0; u < AHEAD && u < 4 * MT; ++u) rr[u] = __builtin_amdgcn_raw_buffer_load_b128(rr_, (int)at(u), 0, 0);
      }
      if (with_bias) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          bb[c] = *reinterpret_cast<const uint4*>((const bf16_t*)a->bias + min(n0 + (c >> 1) * 32 + (2u * (c & 1) + half) * 8u, N - 8));
      }
      auto add8 = [&](float (&v)[2][4], u32x4 w) Q4_INLINE {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[q >> 1][2 * (q & 1)] += __uint_as_float(w[q] << 16);
          v[q >> 1][2 * (q & 1) + 1] += __uint_as_float(w[q] & 0xffff0000u);
        }
      };
      float ssq[2] = {0.0f, 0.0f};                  // per feature tile
#pragma unroll
      for (int u = 0; u < 4 * MT; ++u) {
        const int i = u >> 2, j = (u >> 1) & 1, bp = u & 1;
        float v[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < 4; ++c) Q4_ACC(i, j, 4 * (2 * bp + h) + c, v[h][c]);
        Q4_SWAP8(v[0], v[1]);
        const uint32_t o = at(u);
        if (with_bias) add8(v, u32x4{bb[u & 3].x, bb[u & 3].y, bb[u & 3].z, bb[u & 3].w});
        if (with_resid) {
          add8(v, rr[u % AHEAD]);
          if (u + AHEAD < 4 * MT) rr[u % AHEAD] = __builtin_amdgcn_raw_buffer_load_b128(rr_, (int)at(u + AHEAD), 0, 0);
        }
        if (epi & EPI_RELU) {
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[h][c] = fmaxf(v[h][c], 0.0f);
        }
        const u32x4 out = {pack_bf16x2(v[0][0], v[0][1]), pack_bf16x2(v[0][2], v[0][3]),
                           pack_bf16x2(v[1][0], v[1][1]), pack_bf16x2(v[1][2], v[1][3])};
        __builtin_amdgcn_raw_buffer_store_b128(out, ry, (int)o, 0, 0);
        if ((epi & EPI_SUMSQ) && o != OUT_OF_RANGE) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float q0 = __uint_as_float(out[q] << 16), q1 = __uint_as_float(out[q] & 0xffff0000u);
            ssq[j] = __builtin_fmaf(q0, q0, ssq[j]);
            ssq[j] = __builtin_fmaf(q1, q1, ssq[j]);
          }
        }
        if (u & 1) __builtin_amdgcn_sched_barrier(0);
      }
      stores = 4 * MT;
      if (epi & EPI_SUMSQ) *ssq_units += (double)(ssq[0] + ssq[1]);
    }
#undef Q4_SWAP8
#undef Q4_ACC
    if (!more) break;
  }
  if (epi & EPI_SUMSQ) {
    const float sum = wave_sum((float)*ssq_units);
    float* red = reinterpret_cast<float*>(lds + L::RED);
    __syncthreads();
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    if (t == 0) w4_rest()->partials[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
  }
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");         // loads past the end still write the LDS
}
#undef Q4_DTL

// The LDS limits of all instantiations are set together: a size that is captured into a graph may be the first of its
// tile height.
template <int MT, int FMT>
hipError_t w4_prepare() {
  hipError_t e = hipFuncSetAttribute((const void*)w4_gemm_kernel<MT, FMT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     W4Lds<MT, FMT>::BYTES);
  if constexpr (MT > 1) return e != hipSuccess ? e : w4_prepare<MT - 1, FMT>();
  return e;
}
// W4Args lists the kernel's parameters: where each one begins, by its type's alignment, and the last one's place.
template <class F>
struct LastParameter;
template <class... P>
struct LastParameter<void (*)(P...)> {
  static constexpr size_t place() {
    size_t begin = 0, end = 0;
    ((begin = (end + alignof(P) - 1) / alignof(P) * alignof(P), end = begin + sizeof(P)), ...);
    return begin;
  }
};
static_assert(LastParameter<decltype(&w4_gemm_kernel<8, W4_INT4>)>::place() == offsetof(W4Args, rest) &&
              sizeof(W4Args) - offsetof(W4Args, rest) == sizeof(W4Rest), "w4_rest() reads the last parameter");
template <int MT>
void w4_launch(const GemmArgs& a, const W4Plan& p, hipStream_t st) {
  const W4Rest r = {a.y, a.resid, a.bias, a.partials, a.split_ws, a.rope, a.rope_S, a.ldy, a.row_base, a.seed_lo, a.seed_hi, a.eps_signed};
  const uint32_t packed = w4_pack(a.epi, a.s_fp16 != 0, (a.epi & EPI_ROPE) && a.rope_dh == 128, p.wgs, p.count_n ? 0u : p.ksplit);
  const uint32_t kt_per = p.count_n ? w4_columns(p.first_n, p.count_n) : p.kt_per;
#define Q4_LAUNCH(FMT) \
  w4_gemm_kernel<MT, FMT><<<p.wgs, 256, W4Lds<MT, FMT>::BYTES, st>>>(a.x, a.w, a.s, a.M, a.N, a.K, p.second_row, kt_per, packed, a.zp, r)
  if (a.nf4) Q4_LAUNCH(W4_NF4);
  else if (a.zp) Q4_LAUNCH(W4_ZP);
  else Q4_LAUNCH(W4_INT4);
#undef Q4_LAUNCH
}

}  // namespace

namespace {

W4Plan w4_plan_of(uint32_t cus, uint32_t M, uint32_t second_row, uint32_t tiles_n, uint32_t K, uint32_t ksplit, uint32_t kt_per, uint32_t mt) {
  W4Plan p = {};
  p.mt = mt;
  p.ksplit = ksplit; p.kt_per = ksplit > 1 ? kt_per : K / BK;
  p.second_row = second_row;
  p.tiles_n = tiles_n;
  p.tiles_per_pass = (M + 32 * mt - 1) / (32 * mt);
  p.tiles_m = second_row ? 2 * p.tiles_per_pass : p.tiles_per_pass;
  const uint64_t places = ((uint64_t)p.tiles_m * p.tiles_n * ksplit + 7) / 8 * 8;     // an equal share for every XCD
  p.wgs = (uint32_t)std::min<uint64_t>(places, cus);
  p.rounds = (uint32_t)((places + cus - 1) / cus);
  p.last = (uint32_t)(places - (uint64_t)(p.rounds - 1) * cus);
  return p;
}
// A round lasts as long as one unit, K_TILE us per k-tile on a full chip and 1.5 + 0.9 mt us around the k-loop (repeated
// launches, N = 8192, K from 2048 to 16384, one round each); the matrix unit alone accounts for 0.13 us per tile of 32 tokens,
// what does not shrink with the tile is the conversion of its 256 weight rows.
double w4_time(const W4Plan& p) {
  static const double K_TILE[9] = {0, 0.58, 0.71, 0.83, 0.95, 1.11, 1.26, 1.42, 1.58};
  return p.rounds * (p.kt_per * K_TILE[p.mt] + 1.5 + 0.9 * p.mt);
}

}  // namespace

// Height of the output tiles: the one whose rounds of units take the least time.
W4Plan w4_plan(uint32_t M, uint32_t second_row, uint32_t N, uint32_t K, uint32_t ksplit, uint32_t kt_per,
               uint32_t most_parts, uint32_t height) {
  const uint32_t cus = gemm_workgroups(1u << 20, 1u << 20);
  W4Plan best = {};
  double best_time = 0.0;
  for (uint32_t mt = height ? height : 8; mt > 0; --mt) {
    const W4Plan p = w4_plan_of(cus, M, second_row, (N + BN - 1) / BN, K, ksplit, kt_per, mt);
    if (most_parts && p.wgs > most_parts && mt < 8) continue;
    const double time = w4_time(p);
    if (!best.mt || time < 0.98 * best_time) { best = p; best_time = time; }
    if (height) break;
  }
  return best;
}

// A last round that one height fills badly: whole rounds of one height, the other feature tiles in tiles of another height,
// two launches (5 us for the second).  A last round filled to a share f takes 0.7 + 0.3 f of a whole one (the clock rises, and
// workgroups do not end together): with that the ratio of both sides is foretold to 0.02, without it 0.05 to 0.1 too low.
// Two heights over one, both passes, int4 / NormalFloat-4 / zero-points: 22016 x 4096 400 tokens 0.92 / 0.93 / 0.93, 450 tokens
// 0.93 / 0.86 / 0.87, 260 0.95 / 0.95 / 0.96; 27648 x 5120 800 tokens 0.90 / 0.87 / 0.89, 1200 0.94 / 0.91 / 0.91; 11008 x 4096 1000
// tokens 0.97 / 0.97 / 0.95.  Where less than GAIN is foretold the measured ratios reach 1.0 (12288 x 4096 1000 tokens 0.96 /
// 0.98 / 0.99 at 0.93 are the worst beyond it).  Not in tiles of 32: a tail of them was foretold at 0.94 and measured 1.03.
bool w4_two_heights(const W4Plan& one, uint32_t M, uint32_t K, W4Plan* head, W4Plan* tail) {
  constexpr double TWO_LAUNCHES = 5.0, GAIN = 0.95;
  constexpr uint32_t MOST_ROUNDS = 8, LEAST = 2;      // (beyond eight rounds the last one is too small a part)
  if (one.ksplit > 1 || one.rounds < 2 || one.rounds > MOST_ROUNDS || one.tiles_n >= 65536u) return false;
  const uint32_t cus = gemm_workgroups(1u << 20, 1u << 20);
  auto time = [cus](const W4Plan& p) {
    const double part = p.last < cus ? 0.7 + 0.3 * p.last / cus : 1.0;
    return w4_time(p) * (p.rounds - 1 + part) / p.rounds;
  };
  double best = GAIN * time(one);
  bool found = false;
  for (uint32_t mt = 8; mt >= LEAST; --mt) {
    const W4Plan p = w4_plan_of(cus, M, one.second_row, one.tiles_n, K, 1, 0, mt);
    for (uint32_t whole = p.rounds - 1, tries = 3; whole > 0 && tries > 0; --whole, --tries) {
      const uint32_t n1 = (uint32_t)std::min<uint64_t>((uint64_t)whole * cus / p.tiles_m, one.tiles_n);
      if (n1 == 0 || n1 == one.tiles_n) continue;
      W4Plan h = w4_plan_of(cus, M, one.second_row, n1, K, 1, 0, mt);
      h.count_n = n1;
      const double t1 = time(h) + TWO_LAUNCHES;
      if (t1 >= best) continue;
      for (uint32_t m2 = 8; m2 >= LEAST; --m2) {
        W4Plan t = w4_plan_of(cus, M, one.second_row, one.tiles_n - n1, K, 1, 0, m2);
        if (m2 == mt || t1 + time(t) >= best) continue;
        t.first_n = n1; t.count_n = t.tiles_n;
        best = t1 + time(t);
        *head = h; *tail = t;
        found = true;
      }
    }
  }
  return found;
}

hipError_t launch_w4(const GemmArgs& a, const W4Plan& p, hipStream_t st) {
  W4Plan head, tail;
  // (a sum of squares has a place per workgroup of one launch)
  if ((a.epi & EPI_SUMSQ) || !w4_two_heights(p, a.M, a.K, &head, &tail)) return launch_w4_tiles(a, p, st);
  const hipError_t e = launch_w4_tiles(a, head, st);
  return e != hipSuccess ? e : launch_w4_tiles(a, tail, st);
}

hipError_t launch_w4_tiles(const GemmArgs& a, const W4Plan& p, hipStream_t st) {
  static bool ready = false;
  if (!ready) {
    hipError_t e = w4_prepare<8, W4_INT4>();
    if (e == hipSuccess) e = w4_prepare<8, W4_ZP>();
    if (e == hipSuccess) e = w4_prepare<8, W4_NF4>();
    if (e != hipSuccess) return e;
    ready = true;
  }
  if ((a.epi & EPI_SUMSQ) && p.wgs > a.n_partials) return hipErrorInvalidValue;
  if (a.epi >= 64u || p.wgs >= 4096u || p.ksplit >= 4096u) return hipErrorInvalidValue;        // w4_pack
  switch (p.mt) {
    case 1: w4_launch<1>(a, p, st); break;
    case 2: w4_launch<2>(a, p, st); break;
    case 3: w4_launch<3>(a, p, st); break;
    case 4: w4_launch<4>(a, p, st); break;
    case 5: w4_launch<5>(a, p, st); break;
    case 6: w4_launch<6>(a, p, st); break;
    case 7: w4_launch<7>(a, p, st); break;
    case 8: w4_launch<8>(a, p, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace qzo
