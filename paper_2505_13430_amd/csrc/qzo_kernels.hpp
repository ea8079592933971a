// Host-side launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "../../include/qzo.h"

namespace qzo {

// One run of consecutive rows with the same number of groups per row, inside
// one decoder layer's slice of the scale arena.
struct UpdSeg {
  uint32_t off;        // first scale, relative to the layer's slice
  uint32_t rows, G;    // rows x G scales
  uint32_t row_base;   // noise row id of its first row, relative to the layer
  uint32_t first_wg;   // first workgroup (of 256 units) serving this segment
};
struct UpdPlan {
  UpdSeg seg[4];
  uint32_t n_seg;
  uint32_t wgs_per_layer;
  uint32_t n_layers;
  uint64_t layer_stride;     // scales per layer
  uint32_t rows_per_layer;
  uint32_t fp16;             // storage type of the arena: 0 bf16, 1 fp16
};

// Epilogue selection of the GEMM.
enum : uint32_t {
  EPI_BIAS = 1u,       // + bias[n]
  EPI_RESIDUAL = 2u,   // y = resid[m,n] + acc
  EPI_RELU = 4u,
  EPI_SUMSQ = 8u,      // per-workgroup sum of bf16(y)^2 into partials
  EPI_SWIGLU = 16u,    // W is [gate rows | up rows] (N = 2F): y[M,F] = silu(gate) * up
  EPI_ROPE = 32u,      // not where K is split: y is qkv [M, 3d] of heads of 64 or 128 features; the rotary embedding
                       // is applied to the q and k thirds on the way out (rope, rope_S); with heads of 128 the rows
                       // of an expanded W must be in ROW_ORDER_ROPE128 order (the fused kernel takes them so by itself)
};

// Activations as the few-token kernel inside a model (qzo_few.hip) takes them, written so by the kernel that makes them:
// tile rows in whole tiles of 32, the +eps pass's from row 0 on, the -eps pass's from row tpp on; for a group of 128
// features and a tile, 8 KB in the order of the MFMA's operand: [k-step][half * 32 + row] of 16 bytes, the eight inputs
// 64 half + 8 k-step .. + 7 in the order 0,4,1,5,2,6,3,7 that the nibbles are unpacked in.  Rows beyond a pass's tokens
// are never written (what they hold reaches no output).  Block sums beside it: fp32 [K/128][rows].
struct XPack {
  uint32_t M, tpp, rows;       // tokens of a pass; tile rows of a pass, of all passes (0: plain row-major)
  __host__ __device__ uint32_t tile_row(uint32_t m) const { return m < M ? m : tpp + m - M; }
  // byte offset of features 8 c .. 8 c + 7 of row m
  __host__ __device__ uint32_t chunk(uint32_t m, uint32_t c) const {
    const uint32_t r = tile_row(m);
    return ((c >> 4) * (rows >> 5) + (r >> 5)) * 8192u + (c & 7u) * 1024u + (((c >> 3) & 1u) * 32u + (r & 31u)) * 16u;
  }
};
inline XPack few_pack(uint32_t M, bool dual) {
  const uint32_t tpp = dual && M <= 16 ? 16u : (M + 31) / 32 * 32;
  return {M, tpp, dual ? 2 * tpp : tpp};
}
struct NextNorm {
  const void *gain, *bias;     // bias: LayerNorm, null: RMSNorm
  float eps;
  void* out;                   // bf16 [rows, N]
  float* xsum;                 // nullable: block sums of out, [N/128][rows]
  XPack pack;                  // of out and xsum
  bool done;                   // set by the launcher that took it over
};
// The attention that reads a qkv projection next: a slice reduction may leave its slices to it.
struct NextAttention {
  uint32_t batch, seq, heads, dh;
  const float* part;           // set by the launcher that left them: fp32 [slices][batch * seq][3 heads dh]
  uint32_t slices;
};
struct GemmArgs {
  const void* x;        // bf16 [M,K]
  const void* w;        // packed int4 [N,K/2] (W4) or bf16 [N,K] (dense)
  const void* s;        // bf16 [N,K/128] (W4) or fp16 [N] per-channel scales (codebook)
  const void* cb;       // fp16 [65536,8] codebook (codebook only)
  const void* zp;       // uint8 [N,K/128] zero-points (int4 only; null = symmetric, zero-point 8)
  const void* bias;     // bf16 [N] or null
  const void* resid;    // bf16 [M,N] or null
  void* y;              // bf16 [M,N]
  float* partials;      // EPI_SUMSQ: one float per workgroup
  uint32_t n_partials;  // EPI_SUMSQ, fused int4 kernel: how many of them there is room for
  float* skinny_ws;     // fp32 scratch of skinny_ws_floats(rows, N, K) floats: enables the few-token path (M <= 64)
  float* mid_ws;        // fp32 scratch of mid_ws_floats(M, N, K, dual) floats: enables mid_gemm_kernel
  float* split_ws;      // fp32 scratch of tile_split_ws_floats(M, N, K) floats: enables split-K of the int4 tile kernel
  uint32_t most_slices; // fused int4 kernel: K slices that split_ws has room for (0: as many as tile_ksplit takes)
  uint32_t ksplit, kt_per;   // set by the launcher: K slices and k-tiles per slice
  const float* rope;    // EPI_ROPE: (cos, sin) of [rope_S positions][dh/2 pairs]; row m sits at position m % rope_S
  uint32_t rope_S, rope_dh;
  uint32_t dual;        // both passes of a step stacked: x, y, resid hold 2 M rows; rows [0,M) use +eps_signed,
                        // [M,2M) -eps_signed
  uint32_t flip_row;    // tile kernels: first row of the second pass (0: one pass), whose rows take -eps_signed; set by
                        // the launcher of the fused kernel, by the caller of the plain bf16 GEMM (a multiple of 256)
  uint64_t w_flip;      // plain bf16 GEMM with flip_row: bytes from w to the matrix of the second pass
  uint32_t M, N, K;
  uint32_t ldy;         // row stride of y and resid in elements when the call covers a column block of a wider
                        // matrix (0: N); plain epilogues only (bias, residual, ReLU)
  uint32_t row_base;
  uint32_t seed_lo, seed_hi;
  float eps_signed;
  uint32_t epi;
  uint32_t s_fp16;      // int4 formats: s holds fp16 instead of bf16
  uint32_t nf4;         // mid_gemm_kernel and the fused kernel: w holds NormalFloat-4 indices, s bf16 [N,K/64], no block sums
  // few_gemm_kernel and mid_gemm_kernel: block sums X[g][row] = sum of x[row, 128 g .. 128 g + 127] (fp32, [K/128][rows], rows = M or
  // 2 M when dual, or xp.rows), delivered by the kernel that wrote x, and the same for the output y of the K-slice reduction
  // ([N_out/128][rows], rows as before or yp.rows, N_out % 128 == 0; null: not wanted).  skinny_gemm_kernel sums its blocks itself.
  const float* xsum;
  float* xsum_out;
  XPack xp, yp;               // layout of x and xsum, of the reduction's y and xsum_out
  // The norm that reads y next (null: none wanted): a slice reduction norms the rows it completes (NextNorm::done).
  struct NextNorm* next;
  struct NextAttention* next_attention;      // (null: y is wanted)
};
hipError_t launch_w4a16_gemm(const GemmArgs& a, hipStream_t st);
// Output tiles of the fused kernel: 32 mt tokens x 256 features, each in one pass of a stacked step; units of work are
// (output tile, K slice of kt_per k-tiles).  M: tokens of a pass; second_row: first row of the second pass (0: one pass).
struct W4Plan {
  uint32_t mt, tiles_m, tiles_per_pass, tiles_n, ksplit, kt_per;
  uint32_t second_row;
  uint32_t wgs, rounds;              // persistent workgroups, units of the busiest one
  uint32_t last;                     // units of the last round
  uint32_t first_n, count_n;         // a launch of some feature tiles only: the first, how many (0: all of them)
};
// most_parts (0: no limit): room for one partial sum of squares per workgroup; never refused when it holds one per
// 256 x 256 tile, rounded up to a multiple of 8.  height (0: by the rule): mt.
W4Plan w4_plan(uint32_t M, uint32_t second_row, uint32_t N, uint32_t K, uint32_t ksplit, uint32_t kt_per, uint32_t most_parts,
               uint32_t height = 0);
hipError_t launch_w4_tiles(const GemmArgs& a, const W4Plan& p, hipStream_t st);
// The plan p of a.M, a.N, a.K, or two launches of different heights where they are faster; same results bit for bit.
bool w4_two_heights(const W4Plan& p, uint32_t M, uint32_t K, W4Plan* head, W4Plan* tail);
hipError_t launch_w4(const GemmArgs& a, const W4Plan& p, hipStream_t st);
// Order of the rows of an expanded (bf16) weight matrix: natural; the fused-SwiGLU consumer's tile order;
// the fused-RoPE consumer's order for heads of 128 features (within every 256 rows, so that a lane of the
// GEMM holds feature i and feature i + 64 of a head).
enum : int { ROW_ORDER_NATURAL = 0, ROW_ORDER_SWIGLU = 1, ROW_ORDER_ROPE128 = 2 };
// Few-token path (M <= 64): weights streamed once, K split over workgroups, partial sums in ws.
constexpr uint32_t SKINNY_MAX_M = 64;
constexpr uint32_t STACK_TILE_MAX_M = 4096;  // tile kernel: the two passes share a launch up to this many tokens per pass
constexpr uint32_t SKINNY_MAX_M_DUAL = 32;   // per sign, when both perturbed passes share one launch
uint32_t skinny_ksplit(uint32_t N, uint32_t K);
uint64_t skinny_ws_floats(uint32_t rows, uint32_t N, uint32_t K);      // rows = M, or 2 M in dual mode
bool skinny_fits(uint32_t rows, uint32_t N, uint32_t K);
uint32_t skinny_reduce_blocks(uint32_t M, uint32_t N, uint32_t epi);   // EPI_SUMSQ partial count
hipError_t launch_skinny_gemm(const GemmArgs& a, float* ws, hipStream_t st);
// Its product for packed activations (a.xp), ks slices of per groups.
hipError_t launch_few_gemm(const GemmArgs& a, float* ws, uint32_t ks, uint32_t per, hipStream_t st);
// Adds K-slice partial sums part[slice][M][N] in slice order and applies a's epilogue.
hipError_t launch_partial_reduce(const GemmArgs& a, const float* part, uint32_t ksplit, hipStream_t st);
// Some dozen to a few hundred tokens per pass (mid_gemm_kernel): items (block of MID_ROWS output rows, block of mt token
// tiles) x U pairs of groups of K are cut into W equal contiguous ranges, one per workgroup; an item that
// several ranges touch has one partial sum per range, in range order.
// The token tiles of both passes are counted through, and a place of a token block holds one of them; a NormalFloat-4
// block that would hold tiles of both passes (Tp % mt != 0) has half of its places for either (both = 1), so that which
// pass a place belongs to is known when its kernel is compiled.  Either way ceil(T / mt) blocks.
constexpr uint32_t MID_ROWS = 256;
struct MidPlan {
  uint32_t mt, Z, U, W, tot;           // Z: token blocks per row block; U: pairs of groups of K; tot = items * U
  uint32_t T, Tp, rows, slots;         // token tiles of 32 (all, of one pass), rows of x, most slices of an item
  uint32_t both;
};
MidPlan mid_plan(uint32_t M, uint32_t N, uint32_t K, bool dual, bool nf4);
uint64_t mid_ws_floats(uint32_t M, uint32_t N, uint32_t K, bool dual, bool nf4);
bool mid_fits(uint32_t M, uint32_t N, uint32_t K, bool dual, bool nf4);
struct MidTile { uint32_t pass, tile, valid; };      // tile: within its pass
// Place m of token block z.
__host__ __device__ inline MidTile mid_tile(const MidPlan& p, uint32_t z, uint32_t m) {
  if (p.both) {
    const uint32_t half = p.mt >> 1, pass = m >= half ? 1u : 0u, tile = z * half + m - pass * half;
    return {pass, tile, tile < p.Tp ? 1u : 0u};
  }
  const uint32_t ti = z * p.mt + m, pass = ti >= p.Tp ? 1u : 0u;
  return {pass, ti - pass * p.Tp, ti < p.T ? 1u : 0u};
}
__host__ __device__ inline uint32_t mid_block_of(const MidPlan& p, uint32_t pass, uint32_t tile) {
  return p.both ? tile / (p.mt >> 1) : (pass * p.Tp + tile) / p.mt;
}
// Range that holds unit i: ranges are [w tot / W, (w+1) tot / W).
__host__ __device__ inline uint32_t mid_range_of(uint32_t i, uint32_t W, uint32_t tot) { return ((i + 1) * W - 1) / tot; }
__host__ __device__ inline uint32_t mid_slices(const MidPlan& p, uint32_t item) {
  return mid_range_of((item + 1) * p.U - 1, p.W, p.tot) - mid_range_of(item * p.U, p.W, p.tot) + 1;
}
hipError_t launch_block_sums(const void* x, uint32_t rows, uint32_t K, float* out, hipStream_t st);
hipError_t launch_mid_gemm(const GemmArgs& a, float* ws, hipStream_t st);
hipError_t launch_mid_reduce(const GemmArgs& a, const float* part, const MidPlan& mp, hipStream_t st);
// Split-K of the int4 tile kernel when an M x N output has too few 256 x 256 tiles for the chip:
// number of K slices (1: none) and k-tiles per slice.
uint32_t tile_ksplit(uint32_t M, uint32_t N, uint32_t K, uint32_t* kt_per);
// Column split of a launch whose output tiles are a little more than whole rounds of the chip: the first
// tile_tail_cols(...) columns (whole rounds, ordinary launch) and the rest (at most half a round of tiles,
// cut along K so that they fill the chip); 0: no split.  Plain epilogues only.
uint32_t tile_tail_cols(uint32_t M, uint32_t N, uint32_t K, uint32_t epi);
// Estimated time (us) of launch_bf16_gemm with split_ws given: see there.
double bf16_gemm_estimate(uint32_t M, uint32_t N, uint32_t K, uint32_t epi);
uint64_t tile_split_ws_floats(uint32_t M, uint32_t N, uint32_t K);
// Stacked passes of M tokens each: K slices and column tails are those of a launch whose second pass starts on a multiple
// of 256 rows, in which every tile of 256 tokens lies in one pass.
inline uint32_t stacked_cut_rows(uint32_t M) { return (M + 255u) / 256u * 256u + M; }
// w = uint16 codes [N,K/8]; cb and s as above; N % 8 == 0, K % 128 == 0.
hipError_t launch_codebook_gemm(const GemmArgs& a, hipStream_t st);
// pipe: 0 / 1 = operand tiles staged through registers (compiler's / explicit issue order),
// 2 = loaded from memory straight into the LDS.
hipError_t launch_bf16_gemm(const GemmArgs& a, int pipe, hipStream_t st);
// The plain bf16 GEMM with one wavefront per SIMD and deferred output stores (no split-K): what
// launch_bf16_gemm(pipe = 2) runs when the output tiles fill the chip.
hipError_t launch_bf16_gemm_wide(const GemmArgs& a, hipStream_t st);
constexpr int PLAIN_GEMM_PIPE = 2;     // the route the models take: 3 % faster than 1 on a full step
// One linear's perturbed weights written out as bf16 [N,K] (rows in the GEMM's tile order
// when the consumer fuses SwiGLU), for launch_bf16_gemm.
hipError_t launch_expand_codebook(const void* codes, const void* cb, const void* c_fp16, uint32_t N,
                                  uint32_t K, uint32_t row_base, uint32_t seed_lo, uint32_t seed_hi,
                                  float eps_signed, int swiglu, void* out_bf16, hipStream_t st);
// NormalFloat-4 blocks of 64: se_scratch receives the perturbed scales, fp32 [N, K/64].
hipError_t launch_expand_nf4(const void* q, const void* s_bf16, uint32_t N, uint32_t K, uint32_t row_base,
                             uint32_t seed_lo, uint32_t seed_hi, float eps_signed, int swiglu,
                             float* se_scratch, void* out_bf16, hipStream_t st);
// int4 groups of 128 (zp: uint8 [N, K/128] or null = 8; g_idx: int32 [K] group of each column, or
// null = k / 128): se_scratch fp32 [N, K/128].
hipError_t launch_expand_int4(const void* q, const void* s_bf16, const void* zp, const int32_t* g_idx,
                              uint32_t N, uint32_t K, uint32_t row_base, uint32_t seed_lo, uint32_t seed_hi, float eps_signed,
                              int swiglu, float* se_scratch, void* out_bf16, hipStream_t st);
// Inside a model the perturbed scales of every linear are written by one launch per pass (fp32, laid
// out like the scale arena) and the expansions read them from there.
hipError_t launch_perturbed_scales_all(const void* arena, const UpdPlan& plan, uint32_t seed_lo, uint32_t seed_hi,
                                       float eps_signed, float* se_all, hipStream_t st);
hipError_t launch_expand_int4_from(const void* q, const float* se, const void* zp, const int32_t* g_idx,
                                   uint32_t N, uint32_t K, int swiglu, void* out_bf16, hipStream_t st);
hipError_t launch_expand_nf4_from(const void* q, const float* se, uint32_t N, uint32_t K, int swiglu,
                                  void* out_bf16, hipStream_t st);
// Stacked passes (NormalFloat-4): the same launch over the model leaves z itself, and an expansion reads its linear's
// scales s and z and writes both passes' matrices, +eps at out_bf16 and -eps N*K elements further on.
hipError_t launch_scale_noise_all(const void* arena, const UpdPlan& plan, uint32_t seed_lo, uint32_t seed_hi,
                                  float* z_all, hipStream_t st);
hipError_t launch_expand_nf4_pair(const void* q, const void* s_bf16, const float* z, float eps, uint32_t N, uint32_t K,
                                  int order, void* out_bf16, hipStream_t st);
// Tokens from which a forward of its own (passes not stacked) never cuts K of an int4 qkv or gate/up linear [N,K], whose
// epilogues (rotary embedding, SwiGLU) then ride on the tile kernel.  The line is where the chip is filled without K
// slices; at 7B widths 2800-2960 tokens, 10 to 12 token tiles.
inline uint32_t whole_k_min_m(uint32_t N, uint32_t K) {
  return 2300u + (uint32_t)(3.3e10 / ((double)N * (double)K));
}
// The codebook format is always expanded inside a model: its fused kernel is 45 % slower than the
// plain GEMM and cannot split K.
constexpr uint32_t EXPAND_MIN_M_CODEBOOK = 1;
hipError_t launch_channel_update(void* c_fp16, uint32_t n, uint32_t row_base, uint32_t seed_lo,
                                 uint32_t seed_hi, float eta, float d_clipped,
                                 const qzo_step_result* res, hipStream_t st);
// One 16-bit tensor of the model table inside the flat vector of un-quantized parameters.
struct DenseSeg {
  uint64_t first8;     // first entry / 8
  void* out;           // the tensor (device), written by the perturbation
  uint32_t fmt;        // 0: bf16, 1: fp16
  uint32_t pad;
};
hipError_t launch_dense_perturb(const float* master, const DenseSeg* segs_dev, uint32_t n_seg,
                                uint64_t n_dense, uint32_t seed_lo, uint32_t seed_hi, float eps_signed,
                                hipStream_t st);
hipError_t launch_dense_update(float* master, uint64_t n_dense, uint32_t seed_lo, uint32_t seed_hi,
                               float eta, float d_clipped, const qzo_step_result* res, hipStream_t st);
uint32_t gemm_workgroups(uint32_t M, uint32_t N);

// lm_head GEMM with the cross-entropy folded into the epilogue: for every row
// m and every 64-column slice it writes (max, sum exp(l - max)) and, where the
// target column falls in the slice, the target logit.
struct CeArgs {
  const void* x;        // bf16 [M,K]  final hidden states
  const void* w;        // bf16 [V,K]  lm_head
  const int32_t* tok;   // [B,S]; row m takes its target from tok[(m % tok_rows) + 1]
  uint32_t tok_rows;    // B*S (M is a multiple of it: the same batch may be stacked twice)
  float* part;          // [M, n_slices, 2]
  float* tgt;           // [M]
  uint32_t M, V, K, S;
  uint32_t n_slices;    // ceil(V/256)*4
};
hipError_t launch_lmhead_ce(const CeArgs& a, hipStream_t st);
// The kernel for few rows: tiles of 32 mt (1, 2, 4) rows x 128 columns; mt, or 0 where the tile kernel is the faster one.
uint32_t lmhead_rows_mt(const CeArgs& c);
hipError_t launch_lmhead_rows(const CeArgs& c, uint32_t mt, hipStream_t st);
hipError_t launch_mfma_rate(float* sink, uint32_t workgroups, uint32_t iters, int random_operands,
                            hipStream_t st);
// Behind the last forward of a step: d and its clipping into res (null: not wanted).  loss_plus: where an earlier forward
// left the other pass's loss, when n_pass = 1.
struct StepTail {
  qzo_step_result* res;
  float eps, clip;
  const float* loss_plus;
};
// Mean losses of n_pass passes of M rows each (pass p from row p * stride on) into loss_out[p].
hipError_t launch_ce_reduce(const float* part, const float* tgt, uint32_t M, uint32_t stride, uint32_t n_pass, uint32_t S,
                            uint32_t n_slices, float* rowloss, float* loss_out, const StepTail& tail, hipStream_t st);

hipError_t launch_sum_partials(const float* partials, uint32_t n, float* out, hipStream_t st);

// rope (nullable): receives the table of rotary angles, (cos, sin) of [S positions][dh/2 pairs].
// pass_stride: rows per pass of a stacked forward (M for a single pass); rows m % pass_stride >= tok_rows get zeros.
hipError_t launch_embed(const int32_t* tok, uint32_t tok_rows, uint32_t pass_stride, const void* tok_emb,
                        const void* pos_emb, uint32_t M, uint32_t S, uint32_t d, void* h, float* rope, uint32_t dh,
                        float theta, hipStream_t st);
// xsum_t (nullable, d % 128 == 0): receives the block sums of the output, [d/128][M] fp32 (see GemmArgs::xsum); with it
// pack: layout of the output and the sums
hipError_t launch_rmsnorm(const void* x, const void* gain, uint32_t M, uint32_t d, float eps,
                          void* y, hipStream_t st, float* xsum_t = nullptr, const XPack& pack = XPack{});
hipError_t launch_layernorm(const void* x, const void* gain, const void* bias, uint32_t M,
                            uint32_t d, float eps, void* y, hipStream_t st, float* xsum_t = nullptr,
                            const XPack& pack = XPack{});
hipError_t launch_rope(void* qkv, const float* table, uint32_t M, uint32_t S, uint32_t pass_stride, uint32_t d,
                       uint32_t n_heads, hipStream_t st);
// rope (nullable): the (cos, sin) table; with it the kernel rotates q and k itself (qkv holds them unrotated).
constexpr uint32_t ATTENTION_ROPE_MAX_S = 256;   // up to this sequence length the models let it do so
hipError_t launch_attention(const void* qkv, uint32_t B, uint32_t S, uint32_t n_heads,
                            uint32_t dh, void* out, const float* rope, hipStream_t st, const float* part = nullptr,
                            uint32_t slices = 0, const XPack& pack = XPack{}, float* xsum = nullptr);
// pack: layout of out, xsum receives its block sums (heads of 128, at most 128 positions).
// Whether it takes the projection's K slices in qkv's place (with rope).
bool attention_adds_slices(uint32_t B, uint32_t S, uint32_t n_heads, uint32_t dh, uint32_t slices);
hipError_t launch_scale_update(void* arena, const UpdPlan& plan, uint32_t seed_lo,
                               uint32_t seed_hi, float eta, float d_clipped,
                               const qzo_step_result* res, hipStream_t st);
hipError_t launch_rtn_quantize(const float* w, uint32_t N, uint32_t K, void* q, void* s,
                               hipStream_t st);
hipError_t launch_rtn_quantize_asym(const float* w, uint32_t N, uint32_t K, bool s_fp16, void* q, void* zp,
                                    void* s, hipStream_t st);
hipError_t launch_debug_normals(uint32_t seed_lo, uint32_t seed_hi, uint32_t stream_id,
                                uint32_t row0, uint32_t n_rows, uint32_t G, float* out,
                                hipStream_t st);
hipError_t launch_debug_philox(uint32_t seed_lo, uint32_t seed_hi, const uint32_t* ctr,
                               uint32_t n, uint32_t* out, hipStream_t st);
hipError_t launch_debug_normal_pairs(const uint32_t* words, uint32_t n, float* out,
                                     hipStream_t st);
hipError_t launch_repack_kmajor(const void* qweight, const void* qzeros, const void* scales,
                                uint32_t N, uint32_t K, uint32_t zero_add, bool s_fp16, void* q_out,
                                void* zp_out, void* s_out, hipStream_t st);
hipError_t launch_debug_dequant(const void* q, const void* s, const void* zp, bool s_fp16, uint32_t row_base,
                                uint32_t N, uint32_t K, uint32_t seed_lo, uint32_t seed_hi, float eps_signed,
                                void* w_eff, hipStream_t st);

}  // namespace qzo
