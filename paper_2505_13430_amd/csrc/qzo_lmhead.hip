// lm_head with the cross-entropy folded in, for few rows: per row and 64 vocabulary columns (max, sum exp(l - max)) and the
// target's logit, as the 256 x 256 tile kernel's epilogue writes them, bit for bit (same k-steps in the same order, same
// order inside a slice).
//
// With few rows the product is bound by reading the matrix (262 MB at 32000 x 4096), and 256 x 256 tiles are few: 125 of
// them occupy half of the chip and spend 1.6 us per k-tile on rows that do not exist.  Here a workgroup of two
// wavefronts owns 32 MT rows x 128 columns, a wavefront 64 of the columns; both operands come by direct-to-LDS
// loads into a ring of four stages, three k-tiles ahead, which keeps 40-60 KB per workgroup in flight.
#include "qzo_gemm_tile.hpp"
#include <type_traits>

namespace qzo {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

#define QH_DTL(RSRC, LDSADDR, VOFF, SOFF)                                                    \
  asm volatile(QZO_SET_M0 "buffer_load_dwordx4 %1, %2, %3 offen lds"                         \
               : : "s"(LDSADDR), "v"(VOFF), "s"(RSRC), "s"(SOFF) : "memory", "m0")

template <int MT>
struct HeadLds {
  static constexpr uint32_t X = MT * 4096u, W = 128 * 128, STAGE = X + W;
  static constexpr int S = 4, LOADS = 8 + 2 * MT;          // load instructions per wavefront and k-tile
  static constexpr uint32_t BYTES = S * STAGE;
  static_assert(BYTES <= 160 * 1024, "LDS of a compute unit");
};

template <int MT>
__global__ __launch_bounds__(128, 1) void lmhead_kernel(CeArgs c) {
  typedef HeadLds<MT> L;
  constexpr uint32_t OUT_OF_RANGE = 0x80000000u;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t lrow = lane & 31u, half = lane >> 5;
  const uint32_t K = c.K, nkt = K / BK, m0 = blockIdx.y * (32 * MT), n0 = blockIdx.x * 128 + wave * 64;
  auto rsrc = [](const void* q, uint64_t bytes) {
    return i32x4{(int)(uint32_t)(uintptr_t)q, (int)(uint32_t)((uintptr_t)q >> 32), (int)bytes, 0x00020000};
  };
  const i32x4 rx = rsrc(c.x, (uint64_t)c.M * K * 2), rw = rsrc(c.w, (uint64_t)c.V * K * 2);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // a load instruction fills 8 rows of 128 bytes, swizzled on the memory side: the wavefront's own 64 rows of the matrix,
  // and every other one of the workgroup's instructions for the activations
  uint32_t wo[8], xo[2 * MT];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t row = 8 * i + (lane >> 3);
    wo[i] = min(n0 + row, c.V - 1) * K * 2 + (((lane & 7u) ^ ((row >> 1) & 7u)) << 4);
  }
#pragma unroll
  for (int i = 0; i < 2 * MT; ++i) {
    const uint32_t row = 8 * (2 * i + wave) + (lane >> 3);
    xo[i] = min(m0 + row, c.M - 1) * K * 2 + (((lane & 7u) ^ ((row >> 1) & 7u)) << 4);
  }
  auto load = [&](uint32_t kt, uint32_t stage) __attribute__((always_inline)) {
    const uint32_t base = lds0 + stage * L::STAGE, in = kt < nkt ? 0u : OUT_OF_RANGE;
#pragma unroll
    for (int i = 0; i < 8; ++i) QH_DTL(rw, base + L::X + wave * 8192 + i * 1024, wo[i] + in, kt * (BK * 2));
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) QH_DTL(rx, base + (2 * i + wave) * 1024, xo[i] + in, kt * (BK * 2));
  };
  uint32_t rd[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) rd[ks] = lrow * 128u + (((uint32_t)(ks * 2 + half) ^ ((lrow >> 1) & 7u)) << 4);

  floatx16 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
#pragma unroll
  for (int s = 0; s < L::S - 1; ++s) load(s, s);
  uint32_t stage = 0;
  for (uint32_t kt = 0; kt < nkt; ++kt) {
    // this k-tile has landed (two later ones may be on their way), and everyone has read the one before
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((L::S - 2) * L::LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    load(kt + L::S - 1, stage == 0 ? L::S - 1 : stage - 1);
    const unsigned char* sb = lds + stage * L::STAGE;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      bf16x8 fw[2], fx[MT];
#pragma unroll
      for (int j = 0; j < 2; ++j) fw[j] = *reinterpret_cast<const bf16x8*>(sb + L::X + wave * 8192 + j * 4096 + rd[ks]);
#pragma unroll
      for (int i = 0; i < MT; ++i) fx[i] = *reinterpret_cast<const bf16x8*>(sb + i * 4096 + rd[ks]);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[j], fx[i], acc[i][j], 0, 0, 0);
    }
    stage = stage == L::S - 1 ? 0 : stage + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");        // loads past the end still write the LDS

  // acc[i][j][4 b + q]: row m0 + 32 i + lrow, column n0 + 32 j + 8 b + 4 half + q
  const uint32_t slice = n0 >> 6;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const uint32_t m = m0 + i * 32 + lrow;
    const bool has_target = m < c.M && (m % c.S) != c.S - 1;
    const uint32_t target = has_target ? (uint32_t)c.tok[(m % c.tok_rows) + 1] : 0xffffffffu;
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t n = n0 + 4 * half + j * 32 + (r >> 2) * 8 + (r & 3);
        if (n < c.V) mx = fmaxf(mx, acc[i][j][r]);
        if (n == target) c.tgt[m] = acc[i][j][r];
      }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float sum = 0.0f;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t n = n0 + 4 * half + j * 32 + (r >> 2) * 8 + (r & 3);
        if (n < c.V) sum += expf(acc[i][j][r] - mx);
      }
    sum += __shfl_xor(sum, 32, 64);
    if (m < c.M && half == 0 && slice < c.n_slices)
      reinterpret_cast<float2*>(c.part)[(uint64_t)m * c.n_slices + slice] = make_float2(mx, sum);
  }
}
#undef QH_DTL

template <int MT>
hipError_t head_attr() {
  return hipFuncSetAttribute((const void*)lmhead_kernel<MT>, hipFuncAttributeMaxDynamicSharedMemorySize, HeadLds<MT>::BYTES);
}
template <int MT>
void head_launch(const CeArgs& c, hipStream_t st) {
  // all n_slices slices of a row are written, those beyond the vocabulary as empty ones
  lmhead_kernel<MT><<<dim3(c.n_slices / 2, (c.M + 32 * MT - 1) / (32 * MT)), 128, HeadLds<MT>::BYTES, st>>>(c);
}

}  // namespace

// One tile of rows, or all workgroups on the chip at once (two per compute unit with mt = 1 only, by their LDS).  A step of
// one layer, tile kernel -> this one with mt = 1 / 2 / 4 (us, matrix not in the caches; 32000 x 4096 unless stated): 32 rows
// 235 -> 205 / 209 / 218; 64 rows 261 -> 246 / 235 / 244; 114 rows 299 -> 348 / 319 / 280; 240 rows 335 -> 514 / 420 / 371;
// 50272 x 2048 with 32 rows 179 -> 159 / 169 / 183, 114 rows 211 -> 273 / 237 / 221; 1024 x 256 with 512 rows
// 80 -> 65 / 68 / 76.
uint32_t lmhead_rows_mt(const CeArgs& c) {
  const uint32_t cus = gemm_workgroups(1u << 20, 1u << 20);
  for (uint32_t mt = 1; mt <= 4; mt *= 2) {
    const uint64_t tiles = (c.M + 32 * mt - 1) / (32 * mt), wgs = tiles * (c.n_slices / 2);
    if (wgs <= cus || (mt == 1 && tiles == 1 && wgs <= 2 * cus)) return mt;
  }
  return 0;
}

hipError_t launch_lmhead_rows(const CeArgs& c, uint32_t mt, hipStream_t st) {
  static bool ready = false;
  if (!ready) {
    hipError_t e = head_attr<1>();
    if (e == hipSuccess) e = head_attr<2>();
    if (e == hipSuccess) e = head_attr<4>();
    if (e != hipSuccess) return e;
    ready = true;
  }
  if (mt == 1) head_launch<1>(c, st);
  else if (mt == 2) head_launch<2>(c, st);
  else head_launch<4>(c, st);
  return hipGetLastError();
}

}  // namespace qzo
