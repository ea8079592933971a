// C ABI of the QZO hot path (include/qzo.h): argument checking, the decoder
// forward as a sequence of kernel launches on the caller's stream, and the
// step of Algorithm 1 (two perturbed forwards, SPSA scalar + clipping, update).
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>
#include "../../include/qzo.h"
#include "qzo_kernels.hpp"
#include <algorithm>

using namespace qzo;

namespace {

thread_local std::string g_err;

qzo_status fail(qzo_status st, const std::string& msg) {
  g_err = msg;
  return st;
}
qzo_status hip_fail(hipError_t e, const char* what) {
  return fail(QZO_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}
#define QZO_HIP(call)                                         \
  do {                                                        \
    hipError_t e_ = (call);                                   \
    if (e_ != hipSuccess) return hip_fail(e_, #call);         \
  } while (0)

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
// The GEMM kernels address X [M,K], a bf16 W [N,K] and Y [M,N] with 32-bit byte offsets.
bool bf16_gemm_fits(uint64_t M, uint64_t N, uint64_t K) {
  return M * K * 2 < (1ull << 31) && N * K * 2 < (1ull << 31) && M * N * 2 < (1ull << 31);
}
uint64_t up256(uint64_t x) { return (x + 255u) & ~uint64_t(255); }

struct Linear {           // one quantized linear of a layer
  uint32_t N, K;
  uint64_t s_off;         // first scale within the layer's arena slice
  uint32_t row_base;      // first noise row within the layer
};

struct Workspace {
  unsigned char *h, *a, *qkv, *att, *ff, *act;
  float *ce_part, *tgt, *rowloss, *losses, *skinny;
  float *xs_a, *xs_act;     // few-token path: block sums of the norm output and of the MLP's hidden activation
  float* mid;               // mid_gemm_kernel's partial sums
  float* split;             // K-slice partial sums of the int4 tile kernel (too few tiles for the chip)
  unsigned char* wexp;      // one linear's expanded bf16 weights (expand-then-multiply paths)
  float* se;                // expand-then-multiply of int4 / NormalFloat-4: every perturbed scale of the model, fp32
  float* rope;              // Llama: (cos, sin) of every (position < seq, pair of the head), rebuilt by every pass
  uint64_t total;
};

}  // namespace

struct qzo_model {
  qzo_model_config cfg;
  std::vector<qzo_buf> T;
  void* arena;
  uint64_t n_scales;
  Linear lin[4];
  uint64_t scales_per_layer;
  uint32_t rows_per_layer;
  UpdPlan plan;
  uint32_t tensors_per_layer, first_layer_tensor;
  // int4 linears: 0 = by size, 1 = the fused kernel with its passes stacked up to STACK_TILE_MAX_M tokens, 2 = always
  // expand-then-multiply
  int int4_path = 0;
  // joint SPSA on the un-quantized parameters (off until qzo_model_enable_joint)
  float* dense_master = nullptr;       // caller-owned fp32 [n_dense]
  uint64_t n_dense = 0;
  DenseSeg* dense_segs = nullptr;      // device, caller-owned (qzo_model_enable_joint's table_dev)
  uint32_t n_dense_segs = 0;
};

namespace {

qzo_status check_cfg(const qzo_model_config* c) {
  if (!c) return fail(QZO_ERR_ARG, "config is null");
  if (c->struct_size != sizeof(qzo_model_config))
    return fail(QZO_ERR_ARG, "config.struct_size does not match this library");
  if (c->arch > 1) return fail(QZO_ERR_ARG, "config.arch must be 0 (Llama) or 1 (OPT)");
  if (c->quant > 3)
    return fail(QZO_ERR_UNSUPPORTED,
                "quant must be 0 (int4 group scales), 1 (codebook), 2 (int4 with zero-points) or 3 (NormalFloat-4)");
  if (c->quant == 1 && c->arch != 0)
    return fail(QZO_ERR_UNSUPPORTED, "the codebook variant is built for the Llama family only");
  if (c->quant == 3 ? c->group_size != 64 : c->group_size != 128)
    return fail(QZO_ERR_SHAPE, "group_size must be 128 (64 for the NormalFloat-4 format)");
  if (!c->n_layers || !c->d_model || !c->n_heads || !c->d_ffn || !c->vocab || !c->max_seq)
    return fail(QZO_ERR_SHAPE, "zero dimension in config");
  if (c->d_model % 128 || c->d_ffn % 128)
    return fail(QZO_ERR_SHAPE, "d_model and d_ffn must be multiples of 128");
  if (c->d_model % c->n_heads) return fail(QZO_ERR_SHAPE, "d_model not divisible by n_heads");
  uint32_t dh = c->d_model / c->n_heads;
  if (dh != 64 && dh != 128) return fail(QZO_ERR_SHAPE, "head size must be 64 or 128");
  if (c->scale_fp16 > 1 || c->act_order > 1) return fail(QZO_ERR_ARG, "scale_fp16 and act_order must be 0 or 1");
  if (c->scale_fp16 && c->quant != 0 && c->quant != 2)
    return fail(QZO_ERR_UNSUPPORTED, "fp16 group scales are built for the int4 formats (quant 0 and 2)");
  if (c->act_order && c->quant != 2)
    return fail(QZO_ERR_UNSUPPORTED, "a group index per column belongs to the zero-point format (quant 2)");
  return QZO_OK;
}

void layer_linears(const qzo_model_config& c, Linear lin[4]) {
  const uint32_t d = c.d_model, F = c.d_ffn;
  const uint32_t N[4] = {3 * d, d, c.arch == 0 ? 2 * F : F, d};
  const uint32_t K[4] = {d, d, d, F};
  uint64_t off = 0;
  uint32_t row = 0;
  for (int i = 0; i < 4; ++i) {
    lin[i] = {N[i], K[i], off, row};
    off += (uint64_t)N[i] * (K[i] / c.group_size);
    row += N[i];
  }
}

// Merge a layer's consecutive linears with equal groups-per-row into update segments.
qzo_status build_plan(const Linear* lin, int n_lin, uint32_t n_layers, UpdPlan& p, uint32_t group = 128,
                      uint32_t scale_fp16 = 0) {
  std::memset(&p, 0, sizeof(p));
  p.fp16 = scale_fp16;
  uint32_t wg = 0;
  for (int i = 0; i < n_lin; ++i) {
    const uint32_t G = lin[i].K / group;
    if (p.n_seg && p.seg[p.n_seg - 1].G == G) {
      p.seg[p.n_seg - 1].rows += lin[i].N;
    } else {
      if (lin[i].s_off > 0xffffffffull) return fail(QZO_ERR_SHAPE, "layer has too many scales");
      p.seg[p.n_seg++] = {(uint32_t)lin[i].s_off, lin[i].N, G, lin[i].row_base, 0};
    }
    p.layer_stride = lin[i].s_off + (uint64_t)lin[i].N * G;
    p.rows_per_layer = lin[i].row_base + lin[i].N;
  }
  for (uint32_t i = 0; i < p.n_seg; ++i) {
    const uint64_t units = (uint64_t)p.seg[i].rows * ((p.seg[i].G + 7) / 8);
    if (units >= (1u << 24)) return fail(QZO_ERR_SHAPE, "update segment exceeds 2^24 counters");
    p.seg[i].first_wg = wg;
    wg += (uint32_t)((units + 255) / 256);
  }
  p.wgs_per_layer = wg;
  p.n_layers = n_layers;
  return QZO_OK;
}

// Bytes and kind (0: bf16, 1: fp16, 2: packed integers) of every tensor of the model table.
void table_layout(const qzo_model_config& c, std::vector<uint64_t>& need, std::vector<uint8_t>& kind) {
  const bool llama = c.arch == 0, codebook = c.quant == 1, asym = c.quant == 2;
  const uint64_t d = c.d_model, F = c.d_ffn, V = c.vocab;
  auto b16 = [&](uint64_t n) { need.push_back(n * 2); kind.push_back(0); };
  auto packed = [&](uint64_t bytes) { need.push_back(bytes); kind.push_back(2); };
  b16(V * d);
  if (!llama) b16((uint64_t)c.max_seq * d);
  // a packed weight [N,K/2]; with zero-points, followed by its uint8 [N,K/128] tensor;
  // codebook variant: uint16 codes [N,K/8], then the linear's fp16 [65536,8] codebook
  auto weight = [&](uint64_t N, uint64_t K) {
    if (codebook) {
      packed(N * K / 4);
      need.push_back(65536 * 16); kind.push_back(1);
      return;
    }
    packed(N * K / 2);
    if (asym) packed(N * K / 128);
    if (asym && c.act_order) packed(K * 4);       // int32 group index of every input column
  };
  for (uint32_t l = 0; l < c.n_layers; ++l) {
    if (llama) {
      b16(d); weight(3 * d, d); weight(d, d);
      b16(d); weight(2 * F, d); weight(d, F);
    } else {
      b16(d); b16(d);
      weight(3 * d, d); b16(3 * d); weight(d, d); b16(d);
      b16(d); b16(d);
      weight(F, d); b16(F); weight(d, F); b16(d);
    }
  }
  b16(d);
  if (!llama) b16(d);
  b16(V * d);
}

uint64_t layer_weights(const qzo_model* m) {
  uint64_t weights = 0;
  for (int i = 0; i < 4; ++i) weights += (uint64_t)m->lin[i].N * m->lin[i].K;
  return weights;
}
// NormalFloat-4 without expansion, up to this many tokens per pass.
uint32_t nf4_fused_most(const qzo_model* m) { return layer_weights(m) <= (1u << 28) ? 512u : 384u; }

// NormalFloat-4 in the tile kernel (w4_gemm_kernel): wide layers beyond 64 tokens per pass.  A weight is looked up once per
// tile of up to 256 tokens, by mid_gemm_kernel once per 64 or 128, but that one cuts K as finely as the chip is wide.
// Steps, tile kernel over mid_gemm_kernel: 7B widths 64 tokens 1.12, 65 0.90, 96 0.91, 128 1.03, 132 0.80, 192 0.86, 256 0.88,
// 400 0.72, 512 0.83; 13B widths 64 1.11, 96 0.82, 128 0.96, 256 0.76, 384 0.78; narrower layers (2048 x 8192 and less) 0.93-1.18.
bool nf4_tile_route(const qzo_model* m, uint64_t M1) {
  if (m->cfg.quant != 3 || M1 <= 64 || M1 > nf4_fused_most(m)) return false;
  const uint64_t weights = layer_weights(m);
  if (weights <= (1u << 26) || (weights <= (1u << 28) && M1 > 96 && M1 <= 128)) return false;
  for (int i = 0; i < 4; ++i) {
    const uint64_t N = m->lin[i].N, K = m->lin[i].K;
    if (((M1 + 255) / 256 * 256 + M1) * std::max(N, K) * 2 >= (1ull << 31) || N * K / 2 >= (1ull << 31)) return false;
  }
  return true;
}

// Token counts per pass that take mid_gemm_kernel: NormalFloat-4, and zero-point int4 with fp16 scales beyond the
// few-token kernel's stacked range.
//   Zero-points: it applies the perturbed scale in fp32 to exact integers, where the tile kernel rounds every weight to bf16.
// The range is the one in which that cost no time while the tile kernel's tiles were all 256 tokens high.  Since they are
// not, the tile kernel is faster beyond 64 tokens: mid_gemm_kernel's time over its, steps of eight layers: 7B widths 1.09 (96
// tokens), 1.19 (132), 1.14 (192); 13B widths 1.19 (96), 1.24 (128); OPT-1.3B widths 1.03 (96), 0.97 (128), 1.04 (132), 0.94 (256).
// The range stays, for its precision.  Up to 64 tokens, over the few-token kernel's with a workgroup
// per pass: 7B widths 0.91-0.94, 13B 0.88-0.89, 2560 x 10240 and 3072 x 8192 0.93-0.96, but OPT-1.3B 1.01-1.04, 2048 x 5632
// 1.05-1.07, smaller models 0.97-1.02: there the few-token kernel stays, whose losses are those of two separate passes.  (That kernel was
// skinny_gemm_kernel.  few_gemm_kernel is the faster one: six layers of 7B widths, 33 / 64 tokens, 0.73 / 0.79 ms with bf16 scales, here
// 0.82 / 0.86; the range stays, with its results.)
// A route that the caller chose stays: 1 (fused) keeps the tile kernel beyond the few-token kernel's 64 tokens.
//   NormalFloat-4: the tile kernel where nf4_tile_route says so.  Whole steps of this kernel against two forwards / one
// stacked forward on expanded matrices: 7B widths 0.27 / 0.26 (16 tokens), 0.33 / 0.32 (57), 0.50 / 0.59 (192), 0.49 / 0.63 (256), 0.86 / 0.90 (400), 0.77 / 0.83
// (512); 13B widths 0.29 (57), 0.53 / 0.67 (256), and beyond the limit 0.88 / 0.95 (400), 0.82 / 0.93 (512); OPT-1.3B widths
// 0.41 / 0.50 (57), 0.45 / 0.72 (256), 0.62 / 0.88 (512), and beyond 0.95 (640), 1.08 (768).  Single passes: 0.43-0.72 (57
// tokens), 0.81-0.89 (512).
//   int4 with a bf16 arena keeps the other routes although the kernel is faster there too (zero-point models, eight
// layers, two-pass or tile kernel -> this one: 7B widths 1 x 57 1.43 -> 1.34 ms, 2 x 40 2.60 -> 1.63, 4 x 33 2.65 -> 2.23;
// OPT-1.3B 1 x 57 0.82 -> 0.86, 2 x 40 1.37 -> 0.97) and rounds less.  Nothing in the interface or the method asks for that: the
// performance cases do.  Another order of sums moves the losses by the activations' 16-bit noise, and a scale whose update
// lies near half a bf16 step (2^-8 of the value) then falls to its other side; a state that two updates went through may be
// two steps, 1.6e-2, apart, and perf/cases.py allows 1e-2 between two implementations, set too tight for two updates.
// (fp16 scales have an eighth of that step; NormalFloat-4's are ten times larger, an update is far below half of theirs.)
bool mid_route(const qzo_model* m, uint64_t M1) {
  const qzo_model_config& c = m->cfg;
  const bool nf4 = c.quant == 3;
  if (nf4_tile_route(m, M1)) return false;
  if (!nf4 && (c.quant != 2 || !c.scale_fp16 || c.act_order)) return false;
  if (!nf4 && (M1 <= SKINNY_MAX_M_DUAL || m->int4_path == 2 || (m->int4_path == 1 && M1 > SKINNY_MAX_M))) return false;
  const uint64_t weights = layer_weights(m);
  if (!nf4 && M1 <= SKINNY_MAX_M && weights <= (1u << 26)) return false;
  const uint32_t most = nf4 ? nf4_fused_most(m)
                            : (weights <= (1u << 26) ? 256u : (weights <= (1u << 28) ? 192u : 128u));
  if (M1 > most) return false;
  for (int i = 0; i < 4; ++i)
    if (!mid_fits((uint32_t)M1, m->lin[i].N, m->lin[i].K, true, nf4)) return false;
  return true;
}

// One pass on its own (qzo_forward_loss, joint mode): the few-token kernel is the faster one over its whole range
// (7B widths, 33 / 57 tokens: 3.34 / 3.65 ms a pass against 3.60 / 3.92; OPT-1.3B, 57: 1.88 against 2.22).
// NormalFloat-4 has no few-token kernel: where mid_route holds, mid_gemm_kernel serves its single passes, too (16 tokens: 3.9 ms
// a pass, expanded 8.1).
bool mid_single_pass(const qzo_model* m, uint64_t M1) { return m->cfg.quant == 3 || M1 > SKINNY_MAX_M; }

// Row at which the second pass of a stacked forward starts: behind the first one's, on a multiple of 256 where the plain
// GEMM's token tiles take their pass's expanded matrix (the rows in between are padding: zeros at the embedding, never
// read back).
uint64_t stacked_pass_stride(const qzo_model* m, uint64_t M1) {
  const bool tiles_of_256 = m->cfg.quant == 3 && !mid_route(m, M1) && !nf4_tile_route(m, M1);
  return tiles_of_256 ? (M1 + 255) / 256 * 256 : M1;
}
uint64_t widest_row(const qzo_model_config& c) {
  return std::max<uint64_t>({3ull * c.d_model, (c.arch == 0 ? 2ull : 1ull) * c.d_ffn});
}

// NormalFloat-4 beyond mid_gemm_kernel's range: one expansion can read the indices once and write both passes' matrices
// (4.5 bytes per weight instead of two times 2.5), the plain GEMM's tiles take their pass's.  That halves the launches,
// and twice the tiles leave fewer compute units idle in a launch's last round; but it takes K slices away from launches
// that filled the chip with them, and two matrices of a wide linear (180 MB each at 7B widths) no longer stay in the
// last-level cache between expansion and product.  Steps, separate -> stacked: OPT-1.3B 513 .. 4096 tokens 0.69-0.90 of
// the time; 7B widths 1024 tokens 0.95, 1536 0.93, but 513 1.05, 1152 1.06, 3584 1.05; 13B widths 1280 0.89, 1792
// 1.07; 4096 x 16384 (OPT) 520 1.16.  Hence an estimate: what the launches save against 0.4 us per million weights of a
// layer (no constant part: a small model, bound by its launches, always stacks).  Of 200 measured pairs of shape and
// token count it stacks ten that are slower that way (by 0.7-5.8 %) and leaves nine apart that are faster stacked (by
// 1.0-5.4 %).  385 to 512 tokens of the layers that leave mid_gemm_kernel there: 0.87-0.94 of the time at all sizes.
//   The same for int4, whose fused kernel does without the expansion: 1.22 of the fused kernel's time at 1024 tokens, 1.05 at
// 2048, 0.99 at 3072, 1.00 at 4096.
bool nf4_stack_pays(const qzo_model* m, uint64_t M1) {
  if (M1 <= 512) return true;
  const bool llama = m->cfg.arch == 0;
  const uint32_t epi[4] = {llama ? EPI_ROPE : EPI_BIAS, EPI_RESIDUAL, llama ? EPI_SWIGLU : EPI_BIAS | EPI_RELU, EPI_RESIDUAL};
  const uint32_t rows = (uint32_t)(stacked_pass_stride(m, M1) + M1);
  double gain = 0.0, weights = 0.0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t N = m->lin[i].N, K = m->lin[i].K;
    gain += 2.0 * bf16_gemm_estimate((uint32_t)M1, N, K, epi[i]) - bf16_gemm_estimate(rows, N, K, epi[i]);
    weights += (double)N * K;
  }
  return gain > 0.4e-6 * weights;
}

// Whether qzo_step runs its two perturbed passes as one forward over 2 * batch sequences.  With at
// most 64 tokens the few-token kernels serve both in one launch (half the launches, bit-identical to separate passes); on the route
// above mid_gemm_kernel serves both.
// Beyond (at most 4096 tokens per pass), a launch of
// the tile kernel holds both passes' token tiles, the second pass's with -eps: twice the tiles per
// launch for a chip that such token counts do not fill, half the launches.
// NormalFloat-4 beyond mid_gemm_kernel's range (up to 4096 tokens, too): where nf4_stack_pays.
bool passes_stacked(const qzo_model* m, uint64_t M1) {
  const qzo_model_config& c = m->cfg;
  if (c.quant == 1 || m->dense_master || c.act_order) return false;
  if (c.quant == 3)
    return mid_route(m, M1) || nf4_tile_route(m, M1) || (M1 <= STACK_TILE_MAX_M && (stacked_pass_stride(m, M1) + M1) * widest_row(c) * 2 < (1ull << 31) &&
                                nf4_stack_pays(m, M1));
  if (M1 <= SKINNY_MAX_M_DUAL || mid_route(m, M1)) return true;
  if (M1 > STACK_TILE_MAX_M || m->int4_path == 2) return false;
  if (M1 <= SKINNY_MAX_M) {      // linears of millions of rows: the partial sums of both passes may be too large where one's fit
    for (int i = 0; i < 4; ++i)
      if (!skinny_fits(2 * (uint32_t)M1, m->lin[i].N, m->lin[i].K)) return false;
    return true;
  }
  // Up to a fifth beyond whole_k_min_m always; from there on where the same linears are cut along K either way, namely
  // none, so that the sums (and losses) are those of two forwards.  Stacked over separate there: 7B widths 3240 tokens
  // 0.96, 3360 0.99, 3600 0.99, 4096 0.96; 13B widths 3072 0.99.
  if (m->int4_path == 0) {
    const uint64_t rows = stacked_cut_rows((uint32_t)M1);
    bool beyond = false, cut = rows * widest_row(c) * 2 >= (1ull << 31);
    for (int i = 0; i < 4; ++i) {
      const uint32_t N = m->lin[i].N, K = m->lin[i].K;
      beyond = beyond || M1 * 5 >= (uint64_t)whole_k_min_m(N, K) * 6;
      for (uint32_t r : {(uint32_t)M1, (uint32_t)rows})
        cut = cut || tile_ksplit(r, N, K, nullptr) > 1 || tile_tail_cols(r, N, K, c.arch == 0 && i == 2 ? EPI_SWIGLU : 0);
    }
    if (beyond && cut) return false;
  }
  return true;
}

Workspace carve(const qzo_model* m, uint32_t batch, uint32_t seq, void* base) {
  const qzo_model_config& c = m->cfg;
  const uint64_t M1 = (uint64_t)batch * seq;
  const bool int4 = c.quant == 0 || c.quant == 2;
  const bool stack = passes_stacked(m, M1);
  const uint64_t M = stack ? stacked_pass_stride(m, M1) + M1 : M1, d = c.d_model, F = c.d_ffn;
  const uint64_t n_slices = ((c.vocab + 255) / 256) * 4;
  Workspace w;
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    unsigned char* p = base ? (unsigned char*)base + off : nullptr;
    off += up256(bytes);
    return p;
  };
  // rows of the norm's and the attention's outputs and of the MLP's activation: whole tiles where the few-token kernel takes them packed
  const bool few = M1 <= SKINNY_MAX_M && int4 && !c.act_order;
  const uint64_t Mp = few ? std::max<uint64_t>({M, few_pack((uint32_t)M1, false).rows, few_pack((uint32_t)M1, stack).rows}) : M;
  w.h = take(M * d * 2);
  w.a = take(Mp * d * 2);
  w.qkv = take(M * 3 * d * 2);
  w.att = take(Mp * d * 2);
  w.ff = take(c.arch == 0 ? 0 : Mp * F * 2);    // Llama: SwiGLU is folded into the gate/up GEMM
  w.act = take(c.arch == 0 ? Mp * F * 2 : 0);
  w.ce_part = (float*)take(M * n_slices * 8);
  w.tgt = (float*)take(M * 4);
  w.rowloss = (float*)take(M * 4);
  w.losses = (float*)take(256);
  // few-token path of the int4 GEMM: fp32 partial sums of the K slices of the largest linear
  uint64_t sk = 0;
  const bool mid = mid_route(m, M1), nf4_expanded = c.quant == 3 && !mid && !nf4_tile_route(m, M1);
  if (few)
    for (int i = 0; i < 4; ++i)
      sk = std::max<uint64_t>(sk, skinny_ws_floats((uint32_t)(mid ? M1 : M), m->lin[i].N, m->lin[i].K));
  w.skinny = (float*)take(sk * 4);
  if (sk == 0) w.skinny = nullptr;
  const bool sums = sk || (mid && int4);        // NormalFloat-4 needs none
  w.xs_a = sums ? (float*)take((d / 128) * Mp * 4) : nullptr;
  w.xs_act = sums ? (float*)take((F / 128) * Mp * 4) : nullptr;
  uint64_t mw = 0;
  if (mid)
    for (int i = 0; i < 4; ++i)
      for (int dual = mid_single_pass(m, M1) ? 0 : 1; dual < (stack ? 2 : 1); ++dual)
        mw = std::max<uint64_t>(mw, mid_ws_floats((uint32_t)M1, m->lin[i].N, m->lin[i].K, dual != 0, c.quant == 3));
  w.mid = (float*)take(mw * 4);
  if (mw == 0) w.mid = nullptr;
  // more tokens than that but still too few output tiles for the chip: split-K partial sums
  uint64_t sp = 0;
  if ((M1 > SKINNY_MAX_M && int4 && !mid) || c.act_order || (c.quant == 3 && !mid) || (c.quant == 1 && M1 >= EXPAND_MIN_M_CODEBOOK))
    for (int i = 0; i < 4; ++i) {
      sp = std::max<uint64_t>(sp, tile_split_ws_floats(stack ? stacked_cut_rows((uint32_t)M1) : (uint32_t)M, m->lin[i].N, m->lin[i].K));
      // a single pass (qzo_forward_loss) of a batch whose step stacks its two passes
      if (stack) sp = std::max<uint64_t>(sp, tile_split_ws_floats((uint32_t)M1, m->lin[i].N, m->lin[i].K));
    }
  w.split = (float*)take(sp * 4);
  if (sp == 0) w.split = nullptr;
  // codebook variant with many tokens: the largest linear written out as bf16
  // and the NormalFloat-4 format beyond mid_gemm_kernel's range (with its block scales or their noise, fp32)
  uint64_t ex = 0, sx = 0;
  for (int i = 0; i < 4; ++i) {
    const uint64_t bytes = (uint64_t)m->lin[i].N * m->lin[i].K * 2;
    const bool expanded = nf4_expanded || c.act_order || (c.quant == 1 && M1 >= EXPAND_MIN_M_CODEBOOK) ||
                          (int4 && m->int4_path == 2 && !stack);
    if (expanded) ex = std::max(ex, bytes);
    if (nf4_expanded && stack) ex = std::max(ex, 2 * bytes);      // both passes' matrices
  }
  if (ex && c.quant != 1) sx = m->n_scales * 4;     // every perturbed scale of the model, fp32
  w.wexp = take(ex);
  if (ex == 0) w.wexp = nullptr;
  w.se = (float*)take(sx);
  if (sx == 0) w.se = nullptr;
  w.rope = c.arch == 0 ? (float*)take((uint64_t)seq * (c.d_model / c.n_heads / 2) * 8) : nullptr;
  w.total = off;
  return w;
}

qzo_status check_batch(const qzo_model* m, const void* tok, uint32_t batch, uint32_t seq,
                       const void* ws, uint64_t ws_bytes) {
  if (!m) return fail(QZO_ERR_ARG, "model is null");
  if (!tok || !ws) return fail(QZO_ERR_ARG, "tokens or workspace is null");
  if (!aligned16(tok) || !aligned16(ws)) return fail(QZO_ERR_ALIGN, "tokens/workspace not 16-byte aligned");
  if (batch == 0 || seq < 2) return fail(QZO_ERR_SHAPE, "need batch >= 1 and seq >= 2");
  if (seq > m->cfg.max_seq) return fail(QZO_ERR_SHAPE, "seq exceeds max_seq");
  if ((uint64_t)batch * seq > 0x7fffffffull) return fail(QZO_ERR_SHAPE, "batch*seq too large");
  {
    // the kernels address every operand with 32-bit byte offsets: tokens x widest tensor row, in
    // bf16, must stay below 2^31 bytes (stacked passes count twice)
    const qzo_model_config& c = m->cfg;
    const uint64_t M1 = (uint64_t)batch * seq, rows = !passes_stacked(m, M1) ? M1 : (c.quant != 3 && M1 <= SKINNY_MAX_M) || mid_route(m, M1) ? 2 * M1
                                                      : stacked_cut_rows((uint32_t)M1);
    if (rows * widest_row(c) * 2 >= (1ull << 31))
      return fail(QZO_ERR_SHAPE, "batch*seq too large for this model: an activation tensor would exceed 2^31 bytes");
  }
  Workspace w = carve(m, batch, seq, nullptr);
  if (ws_bytes < w.total) return fail(QZO_ERR_WORKSPACE, "workspace smaller than qzo_workspace_bytes");
  return QZO_OK;
}

// Optional per-kernel-class timing with HIP events recorded on the caller's
// stream around each launch (qzo_profile_begin / qzo_profile_collect).
struct ProfRec { hipEvent_t a, b; uint32_t kind; double work; };
struct Profiler {
  bool on = false;
  std::vector<ProfRec> pool;
  size_t used = 0;
  uint32_t stride = 1;          // every stride-th launch of a class is bracketed
  uint32_t seen[8] = {};
} g_prof;

struct ProfScope {
  ProfRec* r = nullptr;
  hipStream_t st;
  ProfScope(uint32_t kind, double work, hipStream_t s) : st(s) {
    if (!g_prof.on || g_prof.used >= g_prof.pool.size()) return;
    if (g_prof.seen[kind & 7u]++ % g_prof.stride) return;
    r = &g_prof.pool[g_prof.used++];
    r->kind = kind;
    r->work = work;
    (void)hipEventRecord(r->a, st);
  }
  ~ProfScope() {
    if (r) (void)hipEventRecord(r->b, st);
  }
};
enum { PK_W4GEMM = 0, PK_LMHEAD = 1, PK_ATTN = 2, PK_UPDATE = 3, PK_OTHER = 4, PK_EXPAND = 5, PK_COUNT = 6 };


// The decoder forward with every quantized linear perturbed by sign*eps*z.
// n_pass = 2 (see passes_stacked): both passes of a step stacked, rows [0,M1) perturbed by
// +eps_signed and rows [P, P + M1) by -eps_signed, P = stacked_pass_stride(m, M1); their losses go to
// loss_out[0] and [1].  tail: of a step's last forward.
qzo_status forward(qzo_model* m, const int32_t* tok, uint32_t batch1, uint32_t seq, uint64_t seed,
                   float eps_signed, const Workspace& w, float* loss_out, hipStream_t st,
                   void* hidden_out = nullptr, uint32_t n_pass = 1, const StepTail& tail = StepTail{}) {
  const qzo_model_config& c = m->cfg;
  const uint32_t batch = batch1 * n_pass, M1 = batch1 * seq;
  const uint32_t P = n_pass == 2 ? (uint32_t)stacked_pass_stride(m, M1) : M1;     // rows per pass
  const bool padded = P != M1;                                                // rows [M1, P) are padding
  const uint32_t M = n_pass == 2 ? P + M1 : M1;                               // rows of every activation
  const uint32_t d = c.d_model, F = c.d_ffn, H = c.n_heads, dh = d / H;
  const bool llama = c.arch == 0, asym = c.quant == 2;
  const uint32_t seed_lo = (uint32_t)seed, seed_hi = (uint32_t)(seed >> 32);
  const unsigned char* arena = (const unsigned char*)m->arena;

  if (m->dense_master) {      // joint mode: the 16-bit tensors become round16(theta_u + eps_signed z)
    ProfScope ps(PK_OTHER, 0, st);
    QZO_HIP(launch_dense_perturb(m->dense_master, m->dense_segs, m->n_dense_segs, m->n_dense, seed_lo,
                                 seed_hi, eps_signed, st));
  }
  if (w.se) {   // some linear takes the expansion route: one launch perturbs every scale of the model
    ProfScope ps(PK_EXPAND, 0, st);
    if (n_pass == 2) QZO_HIP(launch_scale_noise_all(m->arena, m->plan, seed_lo, seed_hi, w.se, st));
    else QZO_HIP(launch_perturbed_scales_all(m->arena, m->plan, seed_lo, seed_hi, eps_signed, w.se, st));
  }
  {
    ProfScope ps(PK_OTHER, 0, st);
    QZO_HIP(launch_embed(tok, M1, P, m->T[0].ptr_dev, llama ? nullptr : m->T[1].ptr_dev, M, seq, d, w.h,
                         llama ? w.rope : nullptr, dh, c.rope_theta, st));
  }
  const double attn_flops = 2.0 * batch * H * (double)seq * seq * dh;   // causal: half of 4 B H S^2 dh
  const double Mreal = (double)n_pass * M1;                             // rows that count as work
  // attention over both passes: one launch when they are contiguous, one per pass otherwise
  // short sequences: no RoPE launch, the attention kernel rotates q and k itself
  const bool rope_in_attention = llama && seq <= ATTENTION_ROPE_MAX_S;
  // few-token linears take the block sums of their input from its producer
  float* const mid_ws = n_pass == 2 || mid_single_pass(m, M1) ? w.mid : nullptr;
  const bool few = (mid_ws && c.quant != 3) || (w.skinny && M1 <= SKINNY_MAX_M && (c.quant == 0 || c.quant == 2) && !c.act_order);
  float* const xs_a = few ? w.xs_a : nullptr;
  // layout of the norms' outputs and the MLP's activation
  const XPack pack = few && !mid_ws && !w.wexp ? few_pack(M1, n_pass == 2) : XPack{};
  // and the attention's where a head is a group; its block sums take the place of the norm's, which the qkv linear has read
  const XPack att_pack = dh == 128 && !padded && xs_a ? pack : XPack{};
  NextAttention na = {batch, seq, H, dh, nullptr, 0};
  auto attention = [&](bool rotated) {
    ProfScope ps(PK_ATTN, attn_flops, st);
    const float* tb = (llama && !rotated) ? w.rope : nullptr;
    if (na.part) return launch_attention(nullptr, batch, seq, H, dh, w.att, tb, st, na.part, na.slices, att_pack, xs_a);
    if (!padded) return launch_attention(w.qkv, batch, seq, H, dh, w.att, tb, st, nullptr, 0, att_pack, xs_a);
    hipError_t e = launch_attention(w.qkv, batch1, seq, H, dh, w.att, tb, st);
    if (e != hipSuccess) return e;
    return launch_attention((const unsigned char*)w.qkv + (size_t)P * 3 * d * 2, batch1, seq, H, dh,
                            (unsigned char*)w.att + (size_t)P * d * 2, tb, st);
  };
  auto other = [&](hipError_t e) { return e; };
  (void)other;
  bool rope_fused = false;     // set by a qkv linear whose GEMM applied the rotary embedding itself
  // the norm that follows a linear into the residual stream: taken over by the linear's slice reduction where it has one
  NextNorm nn = {};
  auto norm = [&](const void* gain, const void* nbias, float* xs) {
    if (nn.done) { nn.done = false; return hipSuccess; }
    return nbias ? launch_layernorm(w.h, gain, nbias, M, d, c.norm_eps, w.a, st, xs, xs ? pack : XPack{})
                 : launch_rmsnorm(w.h, gain, M, d, c.norm_eps, w.a, st, xs, xs ? pack : XPack{});
  };
  auto before = [&](const void* gain, const void* nbias, float* xs) {
    nn = {gain, nbias, c.norm_eps, w.a, xs, xs ? pack : XPack{}, false};
  };
  for (uint32_t l = 0; l < c.n_layers; ++l) {
    const qzo_buf* T = &m->T[m->first_layer_tensor + (size_t)l * m->tensors_per_layer];
    const uint64_t layer_off = (uint64_t)l * m->scales_per_layer;
    // Position of a tensor of the symmetric table (and of the li-th weight) within this layer: with
    // zero-points every packed weight is followed by one more tensor.
    static const uint32_t wpos_llama[4] = {1, 2, 4, 5}, wpos_opt[4] = {2, 4, 8, 10};
    const uint32_t* wpos = llama ? wpos_llama : wpos_opt;
    const uint32_t extra = (asym ? 1u : 0u) + (c.act_order ? 1u : 0u);    // tensors that follow a packed weight
    auto tpos = [&](uint32_t k) {
      uint32_t shift = 0;
      for (int i = 0; i < 4; ++i) shift += wpos[i] < k ? extra : 0u;
      return k + shift;
    };
    auto ti = [&](uint32_t k) { return T[tpos(k)].ptr_dev; };
    auto gemm = [&](int li, const void* x, const void* bias, const void* resid, void* y, uint32_t epi) {
      GemmArgs g = {};
      g.x = x; g.w = ti(wpos[li]); g.zp = asym ? T[tpos(wpos[li]) + 1].ptr_dev : nullptr;
      g.s = arena + (layer_off + m->lin[li].s_off) * 2;
      g.bias = bias; g.resid = resid; g.y = y;
      g.M = M1; g.N = m->lin[li].N; g.K = m->lin[li].K;
      g.dual = n_pass == 2;
      g.row_base = l * m->rows_per_layer + m->lin[li].row_base;
      g.seed_lo = seed_lo; g.seed_hi = seed_hi; g.eps_signed = eps_signed;
      g.epi = epi & ~EPI_ROPE;                // a request: granted below where the kernel's epilogue can rotate
      g.s_fp16 = c.scale_fp16;
      g.skinny_ws = mid_ws ? nullptr : w.skinny;
      g.split_ws = w.split;
      g.mid_ws = mid_ws;
      g.next = li == 1 || li == 3 ? &nn : nullptr;
      g.next_attention = llama && li == 0 && rope_in_attention && !padded ? &na : nullptr;
      g.nf4 = c.quant == 3;
      if (few) {     // the few-token kernel takes the block sums of its input from the kernel that wrote it
        g.xsum = (li == 0 || li == 2) ? w.xs_a : (li == 3 ? w.xs_act : nullptr);
        g.xsum_out = li == 2 ? w.xs_act : nullptr;
        g.xp = li == 1 ? att_pack : pack;
        if (li == 1 && att_pack.rows) g.xsum = w.xs_a;
        if (li == 2) g.yp = pack;
        if (mid_ws && li == 1 && c.quant != 3) {      // the attention output's block sums, where the norm's were
          hipError_t e = launch_block_sums(x, M, g.K, w.xs_a, st);
          if (e != hipSuccess) return e;
          g.xsum = w.xs_a;
        }
      }
      if (c.act_order) {
        // a group index per column: scale and zero-point are looked up per weight while the perturbed
        // matrix is written out; the fused kernels, whose k-tile shares one scale per row, cannot serve it
        const int32_t* g_idx = (const int32_t*)T[tpos(wpos[li]) + 2].ptr_dev;
        const bool split = w.split && tile_ksplit(g.M, g.N, g.K, nullptr) > 1;
        {
          ProfScope pe(PK_EXPAND, 2.5 * (double)g.N * g.K, st);
          hipError_t e = launch_expand_int4_from(g.w, w.se + layer_off + m->lin[li].s_off, g.zp, g_idx, g.N, g.K,
                                                 (epi & EPI_SWIGLU) != 0 && !split, w.wexp, st);
          if (e != hipSuccess) return e;
        }
        g.w = w.wexp; g.s = nullptr; g.zp = nullptr; g.skinny_ws = nullptr; g.split_ws = (split || (w.split && tile_tail_cols(g.M, g.N, g.K, g.epi))) ? w.split : nullptr;
        ProfScope ps(PK_W4GEMM, 2.0 * Mreal * (double)g.N * g.K, st);
        return launch_bf16_gemm(g, PLAIN_GEMM_PIPE, st);
      }
      if (c.quant == 3 && w.wexp) {
        // NormalFloat-4: table lookup and scaling once per weight (stacked passes: both matrices), then a plain bf16 GEMM
        const bool pair = n_pass == 2;
        if (pair) {
          g.M = M; g.dual = 0;
          g.flip_row = P; g.w_flip = (uint64_t)g.N * g.K * 2;
        }
        const bool split = w.split && tile_ksplit(g.M, g.N, g.K, nullptr) > 1;
        int order = ((epi & EPI_SWIGLU) && !split) ? ROW_ORDER_SWIGLU : ROW_ORDER_NATURAL;
        if (epi == EPI_ROPE && !split && (dh == 64 || (dh == 128 && g.N % 256 == 0))) {   // as for int4 below
          if (dh == 128) order = ROW_ORDER_ROPE128;
          g.epi = EPI_ROPE; g.rope = w.rope; g.rope_S = seq; g.rope_dh = dh;
          rope_fused = true;
        }
        {
          ProfScope pe(PK_EXPAND, (pair ? 4.5 : 2.5) * (double)g.N * g.K, st);
          float* const se = w.se + layer_off + m->lin[li].s_off;
          hipError_t e = pair ? launch_expand_nf4_pair(g.w, g.s, se, eps_signed, g.N, g.K, order, w.wexp, st)
                              : launch_expand_nf4_from(g.w, se, g.N, g.K, order, w.wexp, st);
          if (e != hipSuccess) return e;
        }
        g.w = w.wexp; g.s = nullptr; g.skinny_ws = nullptr; g.split_ws = (split || (w.split && tile_tail_cols(g.M, g.N, g.K, g.epi))) ? w.split : nullptr;
        ProfScope ps(PK_W4GEMM, 2.0 * Mreal * (double)g.N * g.K, st);
        return launch_bf16_gemm(g, PLAIN_GEMM_PIPE, st);
      }
      if (w.wexp) {
        // the caller's choice: write the perturbed matrix out once, then a plain bf16 GEMM.  The rotary embedding
        // of a qkv linear rides on that GEMM's epilogue (heads of 64 or 128; with 128 the matrix is
        // written in the row order that puts feature i and i + 64 of a head into one lane).
        int order = (epi & EPI_SWIGLU) ? ROW_ORDER_SWIGLU : ROW_ORDER_NATURAL;
        if (epi == EPI_ROPE && (dh == 64 || (dh == 128 && g.N % 256 == 0))) {
          if (dh == 128) order = ROW_ORDER_ROPE128;
          g.epi = EPI_ROPE; g.rope = w.rope; g.rope_S = seq; g.rope_dh = dh;
          rope_fused = true;
        }
        {
          ProfScope pe(PK_EXPAND, 2.5 * (double)g.N * g.K, st);
          hipError_t e = launch_expand_int4_from(g.w, w.se + layer_off + m->lin[li].s_off, g.zp, nullptr, g.N,
                                                 g.K, order, w.wexp, st);
          if (e != hipSuccess) return e;
        }
        g.w = w.wexp; g.s = nullptr; g.zp = nullptr; g.skinny_ws = nullptr;
        // (plain epilogues: the launcher cuts K where the output tiles do not fill the chip, or the last
        // columns' K where they are a little more than whole rounds, exactly as it does for the fused kernel)
        g.split_ws = (g.epi & (EPI_SWIGLU | EPI_ROPE)) ? nullptr : w.split;
        ProfScope ps(PK_W4GEMM, 2.0 * Mreal * (double)g.N * g.K, st);
        return launch_bf16_gemm(g, PLAIN_GEMM_PIPE, st);
      }
      if (M1 > SKINNY_MAX_M && !mid_ws && (epi & (EPI_ROPE | EPI_SWIGLU))) {
        // Tile kernel: the rotary embedding rides on its epilogue (sequences too long for the attention kernel's own)
        // where the linear is not cut along K.  A pass of whole_k_min_m tokens or more never cuts these linears.
        const bool whole = m->int4_path == 0 && M >= whole_k_min_m(g.N, g.K) && !passes_stacked(m, M1);
        if (whole) g.split_ws = nullptr;
        const uint32_t r = n_pass == 2 ? stacked_cut_rows(M1) : M1;
        const bool cut = g.split_ws && (tile_ksplit(r, g.N, g.K, nullptr) > 1 || tile_tail_cols(r, g.N, g.K, g.epi));
        if (epi == EPI_ROPE && (whole || !rope_in_attention) && !cut && (dh == 64 || g.N % 256 == 0)) {
          g.epi = EPI_ROPE; g.rope = w.rope; g.rope_S = seq; g.rope_dh = dh;
          rope_fused = true;
        }
      }
      ProfScope ps(PK_W4GEMM, 2.0 * Mreal * (double)g.N * g.K, st);
      return launch_w4a16_gemm(g, st);
    };
    auto cgemm = [&](int li, const void* x, const void* codes, const void* cb, const void* resid,
                     void* y, uint32_t epi) {
      GemmArgs g = {};
      g.x = x; g.w = codes; g.cb = cb;
      g.s = arena + ((uint64_t)l * m->rows_per_layer + m->lin[li].row_base) * 2;   // fp16 channel scales
      g.resid = resid; g.y = y;
      g.M = M; g.N = m->lin[li].N; g.K = m->lin[li].K;
      g.row_base = l * m->rows_per_layer + m->lin[li].row_base;
      g.seed_lo = seed_lo; g.seed_hi = seed_hi; g.eps_signed = eps_signed;
      g.epi = epi & ~EPI_ROPE;                // a request, served by the plain GEMM below when it does not split K
      if (w.wexp) {
        // many tokens: reconstruct the perturbed matrix once, then a plain bf16 GEMM
        // (rows in natural order when the GEMM will split K: its reduction applies SwiGLU)
        const bool split = w.split && tile_ksplit(g.M, g.N, g.K, nullptr) > 1;
        int order = ((epi & EPI_SWIGLU) && !split) ? ROW_ORDER_SWIGLU : ROW_ORDER_NATURAL;
        if (epi == EPI_ROPE && !split && (dh == 64 || (dh == 128 && g.N % 256 == 0))) {   // as for int4
          if (dh == 128) order = ROW_ORDER_ROPE128;
          g.epi = EPI_ROPE; g.rope = w.rope; g.rope_S = seq; g.rope_dh = dh;
          rope_fused = true;
        }
        {
          ProfScope pe(PK_EXPAND, 2.25 * (double)g.N * g.K, st);
          hipError_t e = launch_expand_codebook(codes, cb, g.s, g.N, g.K, g.row_base, seed_lo, seed_hi,
                                                eps_signed, order, w.wexp, st);
          if (e != hipSuccess) return e;
        }
        g.w = w.wexp; g.cb = nullptr; g.s = nullptr; g.split_ws = (split || (w.split && tile_tail_cols(g.M, g.N, g.K, g.epi))) ? w.split : nullptr;
        ProfScope ps(PK_W4GEMM, 2.0 * Mreal * (double)g.N * g.K, st);
        return launch_bf16_gemm(g, PLAIN_GEMM_PIPE, st);
      }
      ProfScope ps(PK_W4GEMM, 2.0 * Mreal * (double)g.N * g.K, st);
      return launch_codebook_gemm(g, st);
    };
    // the next layer's first tensors are its first norm's, behind the last layer the final norm's
    const bool last = l + 1 == c.n_layers;
    auto after_layer = [&](size_t k) { return T[m->tensors_per_layer + k].ptr_dev; };
    if (llama && c.quant == 1) {
      // attn_norm, codes/cb qkv, codes/cb o, ffn_norm, codes/cb gate+up, codes/cb down
      QZO_HIP(launch_rmsnorm(w.h, T[0].ptr_dev, M, d, c.norm_eps, w.a, st));
      rope_fused = false;
      QZO_HIP(cgemm(0, w.a, T[1].ptr_dev, T[2].ptr_dev, nullptr, w.qkv, EPI_ROPE));
      if (!rope_fused && !rope_in_attention) QZO_HIP(launch_rope(w.qkv, w.rope, M, seq, P, d, H, st));
      QZO_HIP(attention(rope_fused || !rope_in_attention));
      QZO_HIP(cgemm(1, w.att, T[3].ptr_dev, T[4].ptr_dev, w.h, w.h, EPI_RESIDUAL));
      QZO_HIP(launch_rmsnorm(w.h, T[5].ptr_dev, M, d, c.norm_eps, w.a, st));
      QZO_HIP(cgemm(2, w.a, T[6].ptr_dev, T[7].ptr_dev, nullptr, w.act, EPI_SWIGLU));
      QZO_HIP(cgemm(3, w.act, T[8].ptr_dev, T[9].ptr_dev, w.h, w.h, EPI_RESIDUAL));
    } else if (llama) {
      // attn_norm, wqkv, wo, ffn_norm, wgu, wdown (symmetric-table positions)
      QZO_HIP(norm(ti(0), nullptr, xs_a));
      rope_fused = false;
      na.part = nullptr;
      QZO_HIP(gemm(0, w.a, nullptr, nullptr, w.qkv, EPI_ROPE));
      if (!rope_fused && !rope_in_attention) QZO_HIP(launch_rope(w.qkv, w.rope, M, seq, P, d, H, st));
      QZO_HIP(attention(rope_fused || !rope_in_attention));
      before(ti(3), nullptr, xs_a);
      QZO_HIP(gemm(1, w.att, nullptr, w.h, w.h, EPI_RESIDUAL));
      QZO_HIP(norm(ti(3), nullptr, xs_a));
      QZO_HIP(gemm(2, w.a, nullptr, nullptr, w.act, EPI_SWIGLU));
      before(after_layer(0), nullptr, last ? nullptr : xs_a);
      QZO_HIP(gemm(3, w.act, nullptr, w.h, w.h, EPI_RESIDUAL));
    } else {
      // ln1_g, ln1_b, wqkv, bqkv, wo, bo, ln2_g, ln2_b, wfc1, bfc1, wfc2, bfc2 (symmetric-table positions)
      QZO_HIP(norm(ti(0), ti(1), xs_a));
      QZO_HIP(gemm(0, w.a, ti(3), nullptr, w.qkv, EPI_BIAS));
      QZO_HIP(attention(true));
      before(ti(6), ti(7), xs_a);
      QZO_HIP(gemm(1, w.att, ti(5), w.h, w.h, EPI_BIAS | EPI_RESIDUAL));
      QZO_HIP(norm(ti(6), ti(7), xs_a));
      QZO_HIP(gemm(2, w.a, ti(9), nullptr, w.ff, EPI_BIAS | EPI_RELU));
      before(after_layer(0), after_layer(1), last ? nullptr : xs_a);
      QZO_HIP(gemm(3, w.ff, ti(11), w.h, w.h, EPI_BIAS | EPI_RESIDUAL));
    }
  }
  const size_t end = m->first_layer_tensor + (size_t)c.n_layers * m->tensors_per_layer;
  QZO_HIP(norm(m->T[end].ptr_dev, llama ? nullptr : m->T[end + 1].ptr_dev, nullptr));
  const void* lm_head = m->T[end + (llama ? 1 : 2)].ptr_dev;
  if (hidden_out)
    QZO_HIP(hipMemcpyAsync(hidden_out, w.a, (size_t)M * d * 2, hipMemcpyDeviceToDevice, st));
  CeArgs ce = {};
  ce.w = lm_head; ce.tok = tok; ce.tok_rows = M1;
  ce.V = c.vocab; ce.K = d; ce.S = seq; ce.n_slices = ((c.vocab + 255) / 256) * 4;
  // both passes in one launch when they are contiguous, one launch per pass otherwise
  for (uint32_t r0 = 0; r0 < M; r0 += P) {
    ce.x = (const unsigned char*)w.a + (size_t)r0 * d * 2;
    ce.part = w.ce_part + (size_t)r0 * ce.n_slices * 2;
    ce.tgt = w.tgt + r0;
    ce.M = padded ? M1 : M;
    ProfScope ps(PK_LMHEAD, 2.0 * ce.M * (double)c.vocab * d, st);
    QZO_HIP(launch_lmhead_ce(ce, st));
    if (!padded) break;
  }
  QZO_HIP(launch_ce_reduce(w.ce_part, w.tgt, M1, P, n_pass, seq, ce.n_slices, w.rowloss, loss_out, tail, st));
  return QZO_OK;
}

}  // namespace

extern "C" {

const char* qzo_last_error(void) { return g_err.c_str(); }

qzo_status qzo_model_scale_count(const qzo_model_config* cfg, uint64_t* out) {
  qzo_status st = check_cfg(cfg);
  if (st != QZO_OK) return st;
  if (!out) return fail(QZO_ERR_ARG, "out is null");
  Linear lin[4];
  layer_linears(*cfg, lin);
  if (cfg->quant == 1)
    *out = (uint64_t)(lin[3].row_base + lin[3].N) * cfg->n_layers;     // one scale per output row
  else
    *out = (lin[3].s_off + (uint64_t)lin[3].N * (lin[3].K / cfg->group_size)) * cfg->n_layers;
  return QZO_OK;
}

qzo_status qzo_model_create(const qzo_model_config* cfg, const qzo_buf* tensors, uint32_t n_tensors,
                            void* scale_arena_dev, uint64_t n_scales, qzo_model** out) {
  qzo_status st = check_cfg(cfg);
  if (st != QZO_OK) return st;
  if (!tensors || !scale_arena_dev || !out) return fail(QZO_ERR_ARG, "null argument");
  if (!aligned16(scale_arena_dev)) return fail(QZO_ERR_ALIGN, "scale arena not 16-byte aligned");
  const bool llama = cfg->arch == 0;
  const bool codebook = cfg->quant == 1;
  const bool asym = cfg->quant == 2;
  const uint32_t per_layer = codebook ? 10 : (llama ? 6 : 12) + (asym ? 4 : 0) + (cfg->act_order ? 4 : 0),
                 head = llama ? 1 : 2, tail = llama ? 2 : 3;
  if (n_tensors != head + per_layer * cfg->n_layers + tail)
    return fail(QZO_ERR_ARG, "tensor count does not match the architecture's table");
  uint64_t want = 0;
  qzo_model_scale_count(cfg, &want);
  if (n_scales != want) return fail(QZO_ERR_SHAPE, "n_scales does not match the config");
  if ((uint64_t)cfg->n_layers * (4 * (uint64_t)cfg->d_model + (llama ? 2 : 1) * (uint64_t)cfg->d_ffn) >
      0xffffffffull)
    return fail(QZO_ERR_SHAPE, "too many quantized rows");

  std::vector<uint64_t> need;
  std::vector<uint8_t> kind;
  table_layout(*cfg, need, kind);
  for (uint32_t i = 0; i < n_tensors; ++i) {
    if (!tensors[i].ptr_dev) return fail(QZO_ERR_ARG, "tensor " + std::to_string(i) + " is null");
    if (!aligned16(tensors[i].ptr_dev))
      return fail(QZO_ERR_ALIGN, "tensor " + std::to_string(i) + " not 16-byte aligned");
    if (tensors[i].bytes != need[i])
      return fail(QZO_ERR_SHAPE, "tensor " + std::to_string(i) + " has " +
                                     std::to_string(tensors[i].bytes) + " bytes, expected " +
                                     std::to_string(need[i]));
  }

  qzo_model* m = new qzo_model();
  m->cfg = *cfg;
  m->T.assign(tensors, tensors + n_tensors);
  m->arena = scale_arena_dev;
  m->n_scales = n_scales;
  layer_linears(*cfg, m->lin);
  m->scales_per_layer = m->lin[3].s_off + (uint64_t)m->lin[3].N * (m->lin[3].K / cfg->group_size);
  m->rows_per_layer = m->lin[3].row_base + m->lin[3].N;
  m->tensors_per_layer = per_layer;
  m->first_layer_tensor = head;
  st = build_plan(m->lin, 4, cfg->n_layers, m->plan, cfg->group_size, cfg->scale_fp16);
  if (st != QZO_OK) { delete m; return st; }
  for (int i = 0; i < 4; ++i)       // one linear written out in bf16 must fit 32-bit byte offsets
    if ((uint64_t)m->lin[i].N * m->lin[i].K * 2 >= (1ull << 31)) {
      delete m;
      return fail(QZO_ERR_SHAPE, "a linear of this model exceeds 2^31 bytes in bf16");
    }
  if ((uint64_t)cfg->vocab * cfg->d_model * 2 >= (1ull << 31)) {
    delete m;
    return fail(QZO_ERR_SHAPE, "lm_head exceeds 2^31 bytes");
  }
  *out = m;
  return QZO_OK;
}

qzo_status qzo_model_destroy(qzo_model* m) {
  if (!m) return QZO_OK;
  delete m;
  return QZO_OK;
}

qzo_status qzo_model_dense_count(const qzo_model_config* cfg, uint64_t* out) {
  qzo_status st = check_cfg(cfg);
  if (st != QZO_OK) return st;
  if (!out) return fail(QZO_ERR_ARG, "out is null");
  std::vector<uint64_t> need;
  std::vector<uint8_t> kind;
  table_layout(*cfg, need, kind);
  uint64_t n = 0;
  for (size_t i = 0; i < need.size(); ++i)
    if (kind[i] != 2) n += need[i] / 2;
  *out = n;
  return QZO_OK;
}

qzo_status qzo_model_joint_table_bytes(const qzo_model_config* cfg, uint64_t* out) {
  qzo_status st = check_cfg(cfg);
  if (st != QZO_OK) return st;
  if (!out) return fail(QZO_ERR_ARG, "out is null");
  std::vector<uint64_t> need;
  std::vector<uint8_t> kind;
  table_layout(*cfg, need, kind);
  uint64_t n = 0;
  for (size_t i = 0; i < need.size(); ++i) n += kind[i] != 2;
  *out = up256(n * sizeof(DenseSeg));
  return QZO_OK;
}

qzo_status qzo_model_enable_joint(qzo_model* m, float* dense_master_dev, uint64_t n_dense, void* table_dev,
                                  uint64_t table_bytes) {
  if (!m || !dense_master_dev || !table_dev) return fail(QZO_ERR_ARG, "null argument");
  if (m->dense_master) return fail(QZO_ERR_ARG, "joint mode is already on");
  if (!aligned16(dense_master_dev) || !aligned16(table_dev))
    return fail(QZO_ERR_ALIGN, "dense master or table not 16-byte aligned");
  uint64_t want = 0;
  qzo_model_dense_count(&m->cfg, &want);
  if (n_dense != want) return fail(QZO_ERR_SHAPE, "n_dense does not match the config");
  std::vector<uint64_t> need;
  std::vector<uint8_t> kind;
  table_layout(m->cfg, need, kind);
  std::vector<DenseSeg> segs;
  uint64_t first = 0;
  for (size_t i = 0; i < need.size(); ++i) {
    if (kind[i] == 2) continue;
    const uint64_t n = need[i] / 2;
    if (n % 8) return fail(QZO_ERR_SHAPE, "a 16-bit tensor's size is not a multiple of 8");
    DenseSeg sg = {};
    sg.first8 = first / 8;
    sg.out = const_cast<void*>(m->T[i].ptr_dev);
    sg.fmt = kind[i];
    segs.push_back(sg);
    first += n;
  }
  if (table_bytes < segs.size() * sizeof(DenseSeg))
    return fail(QZO_ERR_WORKSPACE, "table smaller than qzo_model_joint_table_bytes");
  QZO_HIP(hipMemcpy(table_dev, segs.data(), segs.size() * sizeof(DenseSeg), hipMemcpyHostToDevice));
  m->dense_segs = (DenseSeg*)table_dev;
  m->n_dense_segs = (uint32_t)segs.size();
  m->n_dense = n_dense;
  m->dense_master = dense_master_dev;
  return QZO_OK;
}

qzo_status qzo_workspace_bytes(const qzo_model* m, uint32_t batch, uint32_t seq, uint64_t* out) {
  if (!m || !out) return fail(QZO_ERR_ARG, "null argument");
  if (batch == 0 || seq < 2 || seq > m->cfg.max_seq) return fail(QZO_ERR_SHAPE, "bad batch/seq");
  *out = carve(m, batch, seq, nullptr).total;
  return QZO_OK;
}

qzo_status qzo_forward_loss(qzo_model* m, const int32_t* tokens_dev, uint32_t batch, uint32_t seq,
                            uint64_t seed, float eps, int sign, void* workspace_dev,
                            uint64_t workspace_bytes, float* loss_dev, void* stream) {
  qzo_status st = check_batch(m, tokens_dev, batch, seq, workspace_dev, workspace_bytes);
  if (st != QZO_OK) return st;
  if (!loss_dev) return fail(QZO_ERR_ARG, "loss_dev is null");
  if (sign != 1 && sign != -1) return fail(QZO_ERR_ARG, "sign must be +1 or -1");
  if (!std::isfinite(eps)) return fail(QZO_ERR_ARG, "eps not finite");
  Workspace w = carve(m, batch, seq, workspace_dev);
  return forward(m, tokens_dev, batch, seq, seed, sign > 0 ? eps : -eps, w, loss_dev,
                 (hipStream_t)stream);
}

qzo_status qzo_debug_forward(qzo_model* m, const int32_t* tokens_dev, uint32_t batch, uint32_t seq,
                             uint64_t seed, float eps, int sign, void* workspace_dev,
                             uint64_t workspace_bytes, float* loss_dev, void* hidden_dev,
                             void* stream) {
  qzo_status st = check_batch(m, tokens_dev, batch, seq, workspace_dev, workspace_bytes);
  if (st != QZO_OK) return st;
  if (!loss_dev || !hidden_dev) return fail(QZO_ERR_ARG, "null output");
  if (sign != 1 && sign != -1) return fail(QZO_ERR_ARG, "sign must be +1 or -1");
  Workspace w = carve(m, batch, seq, workspace_dev);
  return forward(m, tokens_dev, batch, seq, seed, sign > 0 ? eps : -eps, w, loss_dev,
                 (hipStream_t)stream, hidden_dev);
}

static qzo_status step_impl(qzo_model* m, const int32_t* tokens_dev, uint32_t batch, uint32_t seq,
                            uint64_t seed, float eps, float eta, float eta_dense, float clip,
                            void* workspace_dev, uint64_t workspace_bytes, qzo_step_result* result_dev,
                            void* stream) {
  qzo_status st = check_batch(m, tokens_dev, batch, seq, workspace_dev, workspace_bytes);
  if (st != QZO_OK) return st;
  if (!result_dev) return fail(QZO_ERR_ARG, "result_dev is null");
  if (!(clip >= 0.0f)) return fail(QZO_ERR_ARG, "clip must be >= 0");
  if (!std::isfinite(eps) || !std::isfinite(eta) || !std::isfinite(eta_dense))
    return fail(QZO_ERR_ARG, "eps/eta not finite");
  hipStream_t s = (hipStream_t)stream;
  Workspace w = carve(m, batch, seq, workspace_dev);
  const StepTail tail = {result_dev, eps, clip, w.losses};
  if (passes_stacked(m, (uint64_t)batch * seq)) {
    // one forward over both passes
    st = forward(m, tokens_dev, batch, seq, seed, eps, w, w.losses, s, nullptr, 2, tail);
    if (st != QZO_OK) return st;
  } else {
    st = forward(m, tokens_dev, batch, seq, seed, eps, w, w.losses, s);
    if (st != QZO_OK) return st;
    st = forward(m, tokens_dev, batch, seq, seed, -eps, w, w.losses + 1, s, nullptr, 1, tail);
    if (st != QZO_OK) return st;
  }
  {
    ProfScope ps(PK_UPDATE, 4.0 * (double)m->n_scales, s);
    if (m->cfg.quant == 1)
      QZO_HIP(launch_channel_update(m->arena, (uint32_t)m->n_scales, 0u, (uint32_t)seed,
                                    (uint32_t)(seed >> 32), eta, 0.0f, result_dev, s));
    else
      QZO_HIP(launch_scale_update(m->arena, m->plan, (uint32_t)seed, (uint32_t)(seed >> 32), eta, 0.0f,
                                  result_dev, s));
  }
  if (m->dense_master) {
    // SPSA part of the joint step, then the 16-bit tensors are brought back to round16(theta_u)
    ProfScope ps(PK_OTHER, 0, s);
    QZO_HIP(launch_dense_update(m->dense_master, m->n_dense, (uint32_t)seed, (uint32_t)(seed >> 32),
                                eta_dense, 0.0f, result_dev, s));
    QZO_HIP(launch_dense_perturb(m->dense_master, m->dense_segs, m->n_dense_segs, m->n_dense,
                                 (uint32_t)seed, (uint32_t)(seed >> 32), 0.0f, s));
  }
  return QZO_OK;
}

qzo_status qzo_step(qzo_model* m, const int32_t* tokens_dev, uint32_t batch, uint32_t seq,
                    uint64_t seed, float eps, float eta, float clip, void* workspace_dev,
                    uint64_t workspace_bytes, qzo_step_result* result_dev, void* stream) {
  if (m && m->dense_master) return fail(QZO_ERR_ARG, "the model is in joint mode: call qzo_step_joint");
  return step_impl(m, tokens_dev, batch, seq, seed, eps, eta, 0.0f, clip, workspace_dev, workspace_bytes,
                   result_dev, stream);
}

qzo_status qzo_step_joint(qzo_model* m, const int32_t* tokens_dev, uint32_t batch, uint32_t seq,
                          uint64_t seed, float eps, float eta, float eta_dense, float clip,
                          void* workspace_dev, uint64_t workspace_bytes, qzo_step_result* result_dev,
                          void* stream) {
  if (m && !m->dense_master) return fail(QZO_ERR_ARG, "joint mode is off: call qzo_model_enable_joint first");
  return step_impl(m, tokens_dev, batch, seq, seed, eps, eta, eta_dense, clip, workspace_dev,
                   workspace_bytes, result_dev, stream);
}

qzo_status qzo_model_apply_update(qzo_model* m, uint64_t seed, float eta, float d_clipped,
                                  void* stream) {
  if (!m) return fail(QZO_ERR_ARG, "model is null");
  if (!std::isfinite(eta) || !std::isfinite(d_clipped)) return fail(QZO_ERR_ARG, "eta/d' not finite");
  if (m->cfg.quant == 1)
    QZO_HIP(launch_channel_update(m->arena, (uint32_t)m->n_scales, 0u, (uint32_t)seed,
                                  (uint32_t)(seed >> 32), eta, d_clipped, nullptr, (hipStream_t)stream));
  else
    QZO_HIP(launch_scale_update(m->arena, m->plan, (uint32_t)seed, (uint32_t)(seed >> 32), eta,
                                d_clipped, nullptr, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_apply_update(void* s_dev, uint32_t n_rows, uint32_t G, uint32_t row_base,
                            uint64_t seed, float eta, float d_clipped, uint32_t scale_fp16, void* stream) {
  if (!s_dev) return fail(QZO_ERR_ARG, "s_dev is null");
  if (scale_fp16 > 1) return fail(QZO_ERR_ARG, "scale_fp16 must be 0 or 1");
  if (!aligned16(s_dev)) return fail(QZO_ERR_ALIGN, "s_dev not 16-byte aligned");
  if (!std::isfinite(eta) || !std::isfinite(d_clipped)) return fail(QZO_ERR_ARG, "eta/d' not finite");
  if (n_rows == 0 || G == 0) return QZO_OK;
  Linear lin = {n_rows, G * 128, 0, row_base};
  UpdPlan plan;
  qzo_status st = build_plan(&lin, 1, 1, plan, 128, scale_fp16);
  if (st != QZO_OK) return st;
  QZO_HIP(launch_scale_update(s_dev, plan, (uint32_t)seed, (uint32_t)(seed >> 32), eta, d_clipped,
                              nullptr, (hipStream_t)stream));
  return QZO_OK;
}

// Scratch of a single perturbed linear: [partial sums of y^2][K-slice partial sums], each part rounded up to 256 bytes.
// total: what a call needs, with one sum per 256 x 256 tile; best: with one per workgroup of the tile height that is
// fastest (lower tiles, more of them), which a call uses where its scratch has that room.
struct LinearScratch { uint32_t parts, best_parts; uint64_t part_floats; uint64_t part_off, total, best; bool skinny, split; };
static LinearScratch linear_scratch(uint32_t M, uint32_t N, uint32_t K, bool with_sumsq) {
  LinearScratch ls = {};
  if (M == 0 || N == 0) return ls;
  ls.skinny = M <= SKINNY_MAX_M;
  ls.split = !ls.skinny && tile_ksplit(M, N, K, nullptr) > 1;     // too few tiles for the chip
  ls.parts = (ls.skinny || ls.split) ? skinny_reduce_blocks(M, N, 0) : ((M + 255) / 256) * ((N + 255) / 256);
  ls.part_floats = ls.skinny ? skinny_ws_floats(M, N, K) : (ls.split ? tile_split_ws_floats(M, N, K) : 0);
  ls.part_off = with_sumsq ? up256((uint64_t)ls.parts * 4) : 0;
  ls.total = ls.part_off + up256(ls.part_floats * 4);
  ls.best = ls.total; ls.best_parts = ls.parts;
  if (!ls.skinny && !ls.split && with_sumsq) {
    ls.best_parts = std::max(ls.parts, w4_plan(M, 0, N, K, 1, 0, 0).wgs);
    ls.best = up256((uint64_t)ls.best_parts * 4);
    ls.parts = (uint32_t)(ls.total / 4);
  }
  return ls;
}

static qzo_status linear_check(const void* x_dev, const void* q_dev, const void* s_dev, const void* y_dev,
                               uint32_t M, uint32_t N, uint32_t K, uint32_t group, float eps, int sign) {
  if (!x_dev || !q_dev || !s_dev || !y_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(x_dev) || !aligned16(q_dev) || !aligned16(s_dev) || !aligned16(y_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (group != 128) return fail(QZO_ERR_SHAPE, "group must be 128");
  if (K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "K must be a positive multiple of 128");
  if (N % 8) return fail(QZO_ERR_SHAPE, "N must be a multiple of 8");
  if (sign != 1 && sign != -1) return fail(QZO_ERR_ARG, "sign must be +1 or -1");
  if (!std::isfinite(eps)) return fail(QZO_ERR_ARG, "eps not finite");
  // buffer loads and stores address each operand with 32-bit byte offsets
  if ((uint64_t)M * K * 2 >= (1ull << 31) || (uint64_t)N * K / 2 >= (1ull << 31) ||
      (uint64_t)M * N * 2 >= (1ull << 31))
    return fail(QZO_ERR_SHAPE, "an operand exceeds 2^31 bytes");
  return QZO_OK;
}

// The launches of a single perturbed linear; scratch (scratch_bytes >= ls.total) is known to be large enough.
static qzo_status dequant_gemm_run(const void* x_dev, const void* q_dev, const void* s_dev, const void* zp_dev,
                                   uint32_t scale_fp16, uint32_t row_base, uint32_t M, uint32_t N, uint32_t K, uint64_t seed,
                                   float eps, int sign, void* y_dev, float* sumsq_dev, void* scratch,
                                   uint64_t scratch_bytes, const LinearScratch& ls, hipStream_t st) {
  if (M == 0 || N == 0) {
    if (sumsq_dev) QZO_HIP(launch_sum_partials(nullptr, 0, sumsq_dev, st));
    return QZO_OK;
  }
  GemmArgs g = {};
  g.x = x_dev; g.w = q_dev; g.s = s_dev; g.zp = zp_dev; g.y = y_dev;
  g.M = M; g.N = N; g.K = K; g.row_base = row_base;
  g.seed_lo = (uint32_t)seed; g.seed_hi = (uint32_t)(seed >> 32);
  g.eps_signed = sign > 0 ? eps : -eps;
  g.s_fp16 = scale_fp16;
  float* part = (float*)((unsigned char*)scratch + ls.part_off);
  if (ls.skinny) g.skinny_ws = part;
  if (ls.split) g.split_ws = part;
  if (sumsq_dev) {
    g.epi = EPI_SUMSQ;
    g.partials = (float*)scratch;
    g.n_partials = scratch_bytes >= ls.best ? ls.best_parts : ls.parts;
  }
  QZO_HIP(launch_w4a16_gemm(g, st));
  // one sum per block of the slice reduction, or per workgroup of the tile kernel
  const uint32_t sums = (ls.skinny || ls.split) ? ls.parts : w4_plan(M, 0, N, K, 1, 0, g.n_partials).wgs;
  if (sumsq_dev) QZO_HIP(launch_sum_partials((const float*)scratch, sums, sumsq_dev, st));
  return QZO_OK;
}

static qzo_status dequant_gemm(const void* x_dev, const void* q_dev, const void* s_dev,
                               const void* zp_dev, uint32_t scale_fp16, uint32_t row_base, uint32_t M, uint32_t N,
                               uint32_t K, uint32_t group, uint64_t seed, float eps, int sign,
                               void* y_dev, float* sumsq_dev, void* scratch_dev, uint64_t scratch_bytes,
                               void* stream) {
  qzo_status st = linear_check(x_dev, q_dev, s_dev, y_dev, M, N, K, group, eps, sign);
  if (st != QZO_OK) return st;
  const LinearScratch ls = linear_scratch(M, N, K, sumsq_dev != nullptr);
  if (ls.total) {
    if (!scratch_dev) return fail(QZO_ERR_ARG, "scratch_dev is null");
    if ((uintptr_t)scratch_dev & 255u) return fail(QZO_ERR_ALIGN, "scratch not 256-byte aligned");
    if (scratch_bytes < ls.total) return fail(QZO_ERR_WORKSPACE, "scratch too small: see qzo_linear_scratch_bytes");
  }
  return dequant_gemm_run(x_dev, q_dev, s_dev, zp_dev, scale_fp16, row_base, M, N, K, seed, eps, sign, y_dev,
                          sumsq_dev, scratch_dev, scratch_bytes, ls, (hipStream_t)stream);
}

qzo_status qzo_linear_scratch_bytes(uint32_t M, uint32_t N, uint32_t K, int with_sumsq, uint64_t* out) {
  if (!out) return fail(QZO_ERR_ARG, "out is null");
  if (K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "K must be a positive multiple of 128");
  *out = linear_scratch(M, N, K, with_sumsq != 0).best;
  return QZO_OK;
}

qzo_status qzo_dequant_gemm(const void* x_dev, const void* q_dev, const void* s_dev,
                            uint32_t row_base, uint32_t M, uint32_t N, uint32_t K, uint32_t group,
                            uint64_t seed, float eps, int sign, void* y_dev, float* sumsq_dev,
                            void* scratch_dev, uint64_t scratch_bytes, void* stream) {
  return dequant_gemm(x_dev, q_dev, s_dev, nullptr, 0u, row_base, M, N, K, group, seed, eps, sign, y_dev,
                      sumsq_dev, scratch_dev, scratch_bytes, stream);
}

// ---- qzo_dequant_gemm for callers that cannot allocate: the scratch is a fixed array of this library ----
// Every GPU the library runs on holds its own copy of the array at its own address; the name below is
// a host-side stand-in, so host code only ever uses the per-device address that hipGetSymbolAddress
// returned (looked up once per device, with that device current).
constexpr uint64_t STATIC_SCRATCH_BYTES = 32ull << 20;
static __device__ __align__(256) unsigned char static_scratch[STATIC_SCRATCH_BYTES];
constexpr int STATIC_SCRATCH_MAX_DEVICES = 64;
static void* g_static_scratch_ptr[STATIC_SCRATCH_MAX_DEVICES] = {};
static std::mutex g_static_scratch_mutex;

qzo_status qzo_dequant_gemm_static(const void* x_dev, const void* q_dev, const void* s_dev,
                                   uint32_t row_base, uint32_t M, uint32_t N, uint32_t K, uint32_t group,
                                   uint64_t seed, float eps, int sign, void* y_dev, float* sumsq_dev,
                                   void* stream) {
  qzo_status st = linear_check(x_dev, q_dev, s_dev, y_dev, M, N, K, group, eps, sign);
  if (st != QZO_OK) return st;
  const LinearScratch ls = linear_scratch(M, N, K, sumsq_dev != nullptr);
  if (ls.total > STATIC_SCRATCH_BYTES)
    return fail(QZO_ERR_WORKSPACE, "this size needs " + std::to_string(ls.total) +
                                       " bytes of scratch, the fixed array holds " +
                                       std::to_string(STATIC_SCRATCH_BYTES) +
                                       ": call qzo_dequant_gemm with scratch of your own");
  int dev = -1;
  QZO_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= STATIC_SCRATCH_MAX_DEVICES) return fail(QZO_ERR_UNSUPPORTED, "device ordinal out of range");
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_static_scratch_mutex);
    if (!g_static_scratch_ptr[dev]) {
      void* p = nullptr;
      QZO_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(static_scratch)));
      if (!p) return fail(QZO_ERR_HIP, "hipGetSymbolAddress returned a null address");
      g_static_scratch_ptr[dev] = p;
    }
    ptr = g_static_scratch_ptr[dev];
  }
  // nothing in the scratch has to start at zero: every partial sum that is read was written by this call
  return dequant_gemm_run(x_dev, q_dev, s_dev, nullptr, 0u, row_base, M, N, K, seed, eps, sign, y_dev, sumsq_dev,
                          ptr, STATIC_SCRATCH_BYTES, ls, (hipStream_t)stream);
}

qzo_status qzo_dequant_gemm_zp(const void* x_dev, const void* q_dev, const void* s_dev,
                               const void* zp_dev, uint32_t scale_fp16, uint32_t row_base, uint32_t M,
                               uint32_t N, uint32_t K, uint32_t group, uint64_t seed, float eps, int sign,
                               void* y_dev, float* sumsq_dev, void* scratch_dev, uint64_t scratch_bytes,
                               void* stream) {
  if (!zp_dev) return fail(QZO_ERR_ARG, "zp_dev is null");
  if (scale_fp16 > 1) return fail(QZO_ERR_ARG, "scale_fp16 must be 0 or 1");
  return dequant_gemm(x_dev, q_dev, s_dev, zp_dev, scale_fp16, row_base, M, N, K, group, seed, eps, sign, y_dev,
                      sumsq_dev, scratch_dev, scratch_bytes, stream);
}

qzo_status qzo_repack_kmajor(const void* qweight_dev, const void* qzeros_dev, const void* scales_dev,
                             uint32_t N, uint32_t K, uint32_t group, uint32_t zero_add, uint32_t scale_fp16,
                             void* q_dev, void* zp_dev, void* s_dev, void* stream) {
  if (!qweight_dev || !qzeros_dev || !scales_dev || !q_dev || !zp_dev || !s_dev)
    return fail(QZO_ERR_ARG, "null device pointer");
  if (group != 128 || K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "group must be 128 and divide K");
  if (N == 0 || N % 8) return fail(QZO_ERR_SHAPE, "N must be a positive multiple of 8");
  if (zero_add > 15) return fail(QZO_ERR_ARG, "zero_add must be 0 .. 15");
  if (scale_fp16 > 1) return fail(QZO_ERR_ARG, "scale_fp16 must be 0 or 1");
  if (!aligned16(q_dev) || !aligned16(s_dev)) return fail(QZO_ERR_ALIGN, "output not 16-byte aligned");
  QZO_HIP(launch_repack_kmajor(qweight_dev, qzeros_dev, scales_dev, N, K, zero_add, scale_fp16 != 0, q_dev,
                               zp_dev, s_dev, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_codebook_scratch_bytes(uint32_t M, uint32_t N, int with_sumsq, uint64_t* out) {
  if (!out) return fail(QZO_ERR_ARG, "out is null");
  *out = (with_sumsq && M && N) ? up256((uint64_t)((M + 255) / 256) * ((N + 255) / 256) * 4) : 0;
  return QZO_OK;
}

qzo_status qzo_codebook_gemm(const void* x_dev, const void* codes_dev, const void* codebook_dev,
                             const void* c_dev, uint32_t row_base, uint32_t M, uint32_t N, uint32_t K,
                             uint64_t seed, float eps, int sign, void* y_dev, float* sumsq_dev,
                             void* scratch_dev, uint64_t scratch_bytes, void* stream) {
  if (!x_dev || !codes_dev || !codebook_dev || !c_dev || !y_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(x_dev) || !aligned16(codes_dev) || !aligned16(codebook_dev) || !aligned16(c_dev) ||
      !aligned16(y_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "K must be a positive multiple of 128");
  if (N % 8) return fail(QZO_ERR_SHAPE, "N must be a multiple of 8");
  if (sign != 1 && sign != -1) return fail(QZO_ERR_ARG, "sign must be +1 or -1");
  if (!std::isfinite(eps)) return fail(QZO_ERR_ARG, "eps not finite");
  if ((uint64_t)M * K * 2 >= (1ull << 31) || (uint64_t)N * K / 4 >= (1ull << 31) ||
      (uint64_t)M * N * 2 >= (1ull << 31))
    return fail(QZO_ERR_SHAPE, "an operand exceeds 2^31 bytes");
  uint64_t need = 0;
  qzo_codebook_scratch_bytes(M, N, sumsq_dev != nullptr, &need);
  if (need) {
    if (!scratch_dev) return fail(QZO_ERR_ARG, "scratch_dev is null");
    if ((uintptr_t)scratch_dev & 255u) return fail(QZO_ERR_ALIGN, "scratch not 256-byte aligned");
    if (scratch_bytes < need) return fail(QZO_ERR_WORKSPACE, "scratch too small: see qzo_codebook_scratch_bytes");
  }
  hipStream_t st = (hipStream_t)stream;
  if (M == 0 || N == 0) {
    if (sumsq_dev) QZO_HIP(launch_sum_partials(nullptr, 0, sumsq_dev, st));
    return QZO_OK;
  }
  GemmArgs g = {};
  g.x = x_dev; g.w = codes_dev; g.cb = codebook_dev; g.s = c_dev; g.y = y_dev;
  g.M = M; g.N = N; g.K = K; g.row_base = row_base;
  g.seed_lo = (uint32_t)seed; g.seed_hi = (uint32_t)(seed >> 32);
  g.eps_signed = sign > 0 ? eps : -eps;
  const uint32_t tiles = ((M + 255) / 256) * ((N + 255) / 256);
  if (sumsq_dev) {
    g.epi = EPI_SUMSQ;
    g.partials = (float*)scratch_dev;
  }
  QZO_HIP(launch_codebook_gemm(g, st));
  if (sumsq_dev) QZO_HIP(launch_sum_partials((const float*)scratch_dev, tiles, sumsq_dev, st));
  return QZO_OK;
}

static qzo_status int4_expand_check(const void* q_dev, const void* s_dev, const int32_t* g_idx_dev,
                                    uint32_t K, uint32_t group, float eps, int sign) {
  if (!q_dev || !s_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(q_dev) || !aligned16(s_dev) || !aligned16(g_idx_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (group != 128 || K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "group must be 128 and divide K");
  if (sign != 1 && sign != -1) return fail(QZO_ERR_ARG, "sign must be +1 or -1");
  if (!std::isfinite(eps)) return fail(QZO_ERR_ARG, "eps not finite");
  return QZO_OK;
}

qzo_status qzo_int4_expand(const void* q_dev, const void* s_dev, const void* zp_dev,
                           const int32_t* g_idx_dev, uint32_t row_base, uint32_t N, uint32_t K,
                           uint32_t group, uint64_t seed, float eps, int sign, float* se_dev, void* w_dev,
                           void* stream) {
  qzo_status st = int4_expand_check(q_dev, s_dev, g_idx_dev, K, group, eps, sign);
  if (st != QZO_OK) return st;
  if (!se_dev || !w_dev) return fail(QZO_ERR_ARG, "null output");
  if (!aligned16(se_dev) || !aligned16(w_dev)) return fail(QZO_ERR_ALIGN, "output not 16-byte aligned");
  QZO_HIP(launch_expand_int4(q_dev, s_dev, zp_dev, g_idx_dev, N, K, row_base, (uint32_t)seed,
                             (uint32_t)(seed >> 32), sign > 0 ? eps : -eps, false, se_dev, w_dev,
                             (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_int4_scratch_bytes(uint32_t N, uint32_t K, uint64_t* out) {
  if (!out) return fail(QZO_ERR_ARG, "out is null");
  *out = up256((uint64_t)N * K * 2) + up256((uint64_t)N * (K / 128) * 4);
  return QZO_OK;
}

qzo_status qzo_int4_gemm_expanded(const void* x_dev, const void* q_dev, const void* s_dev, const void* zp_dev,
                                  const int32_t* g_idx_dev, uint32_t row_base, uint32_t M, uint32_t N,
                                  uint32_t K, uint32_t group, uint64_t seed, float eps, int sign, void* y_dev,
                                  void* scratch_dev, uint64_t scratch_bytes, void* stream) {
  qzo_status st = int4_expand_check(q_dev, s_dev, g_idx_dev, K, group, eps, sign);
  if (st != QZO_OK) return st;
  if (!x_dev || !y_dev || !scratch_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(x_dev) || !aligned16(y_dev) || ((uintptr_t)scratch_dev & 255u))
    return fail(QZO_ERR_ALIGN, "x/y need 16-byte, scratch 256-byte alignment");
  if (N % 8) return fail(QZO_ERR_SHAPE, "N must be a multiple of 8");
  uint64_t need = 0;
  qzo_int4_scratch_bytes(N, K, &need);
  if (scratch_bytes < need) return fail(QZO_ERR_WORKSPACE, "scratch too small: see qzo_int4_scratch_bytes");
  if (!bf16_gemm_fits(M, N, K)) return fail(QZO_ERR_SHAPE, "an operand exceeds 2^31 bytes");
  if (M == 0 || N == 0) return QZO_OK;
  hipStream_t s = (hipStream_t)stream;
  unsigned char* wexp = (unsigned char*)scratch_dev;
  float* se = (float*)(wexp + up256((uint64_t)N * K * 2));
  QZO_HIP(launch_expand_int4(q_dev, s_dev, zp_dev, g_idx_dev, N, K, row_base, (uint32_t)seed,
                             (uint32_t)(seed >> 32), sign > 0 ? eps : -eps, false, se, wexp, s));
  GemmArgs g = {};
  g.x = x_dev; g.w = wexp; g.y = y_dev; g.M = M; g.N = N; g.K = K;
  QZO_HIP(launch_bf16_gemm(g, PLAIN_GEMM_PIPE, s));
  return QZO_OK;
}

static qzo_status nf4_check(const void* q_dev, const void* s_dev, uint32_t N, uint32_t K, uint32_t block,
                            float eps, int sign) {
  if (!q_dev || !s_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(q_dev) || !aligned16(s_dev)) return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (block != 64 || K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "block must be 64 and K a positive multiple of 128");
  if (N % 8) return fail(QZO_ERR_SHAPE, "N must be a multiple of 8");
  if (sign != 1 && sign != -1) return fail(QZO_ERR_ARG, "sign must be +1 or -1");
  if (!std::isfinite(eps)) return fail(QZO_ERR_ARG, "eps not finite");
  return QZO_OK;
}

qzo_status qzo_nf4_expand(const void* q_dev, const void* s_dev, uint32_t row_base, uint32_t N, uint32_t K,
                          uint32_t block, uint64_t seed, float eps, int sign, float* se_dev, void* w_dev,
                          void* stream) {
  qzo_status st = nf4_check(q_dev, s_dev, N, K, block, eps, sign);
  if (st != QZO_OK) return st;
  if (!se_dev || !w_dev) return fail(QZO_ERR_ARG, "null output");
  if (!aligned16(se_dev) || !aligned16(w_dev)) return fail(QZO_ERR_ALIGN, "output not 16-byte aligned");
  QZO_HIP(launch_expand_nf4(q_dev, s_dev, N, K, row_base, (uint32_t)seed, (uint32_t)(seed >> 32),
                            sign > 0 ? eps : -eps, false, se_dev, w_dev, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_nf4_scratch_bytes(uint32_t N, uint32_t K, uint64_t* out) {
  if (!out) return fail(QZO_ERR_ARG, "out is null");
  *out = up256((uint64_t)N * K * 2) + up256((uint64_t)N * (K / 64) * 4);
  return QZO_OK;
}

// A single linear is expanded first from this many tokens on, unless it is small.  Fused over expanded: 11008 x 4096 16 tokens
// 0.24, 256 0.50, 1024 0.96, 2048 0.99, 3072 0.98, 4096 1.10; 4096 x 11008 16 0.11, 1024 0.52, 2048 0.84, 3072 1.04; 4096 x 4096
// 1024 0.77, 2048 0.88, 3072 1.00, 8192 1.12; 22016 x 4096 1024 0.85, 2048 0.96, 3072 1.03; 8192 x 512 and 1024 x 1024 4096 tokens
// 0.76 and 0.63, 8192 0.43 and 0.73.
constexpr uint32_t NF4_LINEAR_EXPAND_MIN_M = 2816;
constexpr uint64_t NF4_LINEAR_NEVER_EXPAND = 1ull << 23;
qzo_status qzo_nf4_gemm(const void* x_dev, const void* q_dev, const void* s_dev, uint32_t row_base,
                        uint32_t M, uint32_t N, uint32_t K, uint32_t block, uint64_t seed, float eps,
                        int sign, void* y_dev, void* scratch_dev, uint64_t scratch_bytes, void* stream) {
  qzo_status st = nf4_check(q_dev, s_dev, N, K, block, eps, sign);
  if (st != QZO_OK) return st;
  if (!x_dev || !y_dev || !scratch_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(x_dev) || !aligned16(y_dev) || ((uintptr_t)scratch_dev & 255u))
    return fail(QZO_ERR_ALIGN, "x/y need 16-byte, scratch 256-byte alignment");
  uint64_t need = 0;
  qzo_nf4_scratch_bytes(N, K, &need);
  if (scratch_bytes < need) return fail(QZO_ERR_WORKSPACE, "scratch too small: see qzo_nf4_scratch_bytes");
  if (!bf16_gemm_fits(M, N, K)) return fail(QZO_ERR_SHAPE, "an operand exceeds 2^31 bytes");
  if (M == 0 || N == 0) return QZO_OK;
  hipStream_t s = (hipStream_t)stream;
  GemmArgs g = {};
  g.x = x_dev; g.y = y_dev; g.M = M; g.N = N; g.K = K;
  if (M < NF4_LINEAR_EXPAND_MIN_M || (uint64_t)N * K <= NF4_LINEAR_NEVER_EXPAND) {
    g.nf4 = 1; g.w = q_dev; g.s = s_dev; g.row_base = row_base;
    g.seed_lo = (uint32_t)seed; g.seed_hi = (uint32_t)(seed >> 32); g.eps_signed = sign > 0 ? eps : -eps;
    // K slices, where the expansion's place holds the partial sums of two or more
    const uint64_t room = need / ((uint64_t)M * N * 4);
    const bool tail = tile_ksplit(M, N, K, nullptr) < 2;
    if (room >= 2 && (!tail || tile_split_ws_floats(M, N, K) * 4 <= need)) {
      g.split_ws = (float*)scratch_dev;
      g.most_slices = tail ? 0u : (uint32_t)std::min<uint64_t>(room, 0xffffffffu);
    }
    QZO_HIP(launch_w4a16_gemm(g, s));
    return QZO_OK;
  }
  unsigned char* wexp = (unsigned char*)scratch_dev;
  float* se = (float*)(wexp + up256((uint64_t)N * K * 2));
  QZO_HIP(launch_expand_nf4(q_dev, s_dev, N, K, row_base, (uint32_t)seed, (uint32_t)(seed >> 32),
                            sign > 0 ? eps : -eps, false, se, wexp, s));
  g.w = wexp;
  QZO_HIP(launch_bf16_gemm(g, PLAIN_GEMM_PIPE, s));
  return QZO_OK;
}

qzo_status qzo_model_set_int4_path(qzo_model* m, int mode) {
  if (!m) return fail(QZO_ERR_ARG, "model is null");
  if (mode < 0 || mode > 2) return fail(QZO_ERR_ARG, "mode must be 0 (by token count), 1 (fused) or 2 (expanded)");
  if (m->cfg.quant != 0 && m->cfg.quant != 2) return fail(QZO_ERR_UNSUPPORTED, "the model's format is not int4");
  m->int4_path = mode;
  return QZO_OK;
}

qzo_status qzo_debug_bf16_gemm(const void* x_dev, const void* w_dev, uint32_t M, uint32_t N, uint32_t K,
                               int pipe, void* y_dev, void* stream) {
  if (!x_dev || !w_dev || !y_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(x_dev) || !aligned16(w_dev) || !aligned16(y_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "K must be a positive multiple of 128");
  if (N % 8) return fail(QZO_ERR_SHAPE, "N must be a multiple of 8");
  if (pipe < 0 || pipe > 2) return fail(QZO_ERR_ARG, "pipe must be 0, 1 or 2");
  if (!bf16_gemm_fits(M, N, K)) return fail(QZO_ERR_SHAPE, "an operand exceeds 2^31 bytes");
  GemmArgs g = {};
  g.x = x_dev; g.w = w_dev; g.y = y_dev; g.M = M; g.N = N; g.K = K;
  QZO_HIP(launch_bf16_gemm(g, pipe, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_debug_fused_linear(const void* x_dev, const void* q_dev, const void* s_dev, const void* zp_dev, int nf4,
                                  uint32_t row_base, uint32_t M, uint32_t passes, uint32_t N, uint32_t K, uint64_t seed, float eps,
                                  int sign, uint32_t epilogue, const void* bias_dev, const void* resid_dev, const float* rope_dev,
                                  uint32_t rope_seq, uint32_t rope_head_dim, uint32_t* height, void* y_dev, void* stream) {
  const bool swiglu = epilogue & EPI_SWIGLU, rope = epilogue & EPI_ROPE;
  if (!x_dev || !q_dev || !s_dev || !y_dev || !height || ((epilogue & EPI_BIAS) && !bias_dev) ||
      ((epilogue & EPI_RESIDUAL) && !resid_dev) || (rope && !rope_dev))
    return fail(QZO_ERR_ARG, "null pointer");
  if (!aligned16(x_dev) || !aligned16(q_dev) || !aligned16(s_dev) || !aligned16(zp_dev) || !aligned16(y_dev) || !aligned16(bias_dev) ||
      !aligned16(resid_dev) || !aligned16(rope_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if ((epilogue & ~(EPI_BIAS | EPI_RESIDUAL | EPI_RELU | EPI_SWIGLU | EPI_ROPE)) || ((swiglu || rope) && (epilogue & (epilogue - 1))) ||
      (nf4 && zp_dev) || *height > 8 || passes < 1 || passes > 2 || !std::isfinite(eps))
    return fail(QZO_ERR_ARG, "no such epilogue, format, tile height or number of passes");
  if (M == 0 || N == 0 || N % 8 || K == 0 || K % 128 || (swiglu && N % 256) ||
      (rope && (rope_seq == 0 || (rope_head_dim != 64 && rope_head_dim != 128) || N % (3 * rope_head_dim) || (rope_head_dim == 128 && N % 256))))
    return fail(QZO_ERR_SHAPE, "need K % 128 == 0, N % 8 == 0, SwiGLU N % 256 == 0, rotary embedding heads of 64 or 128 (whole tiles of two)");
  const uint64_t rows = (uint64_t)passes * M;
  if (rows * K * 2 >= (1ull << 31) || (uint64_t)N * K / 2 >= (1ull << 31) || rows * N * 2 >= (1ull << 31))
    return fail(QZO_ERR_SHAPE, "an operand exceeds 2^31 bytes");
  GemmArgs g = {};
  g.x = x_dev; g.w = q_dev; g.s = s_dev; g.zp = zp_dev; g.nf4 = nf4 != 0;
  g.bias = bias_dev; g.resid = resid_dev; g.y = y_dev;
  g.M = M; g.N = N; g.K = K; g.row_base = row_base; g.flip_row = passes == 2 ? M : 0;
  g.seed_lo = (uint32_t)seed; g.seed_hi = (uint32_t)(seed >> 32); g.eps_signed = sign > 0 ? eps : -eps;
  g.epi = epilogue; g.rope = rope_dev; g.rope_S = rope_seq; g.rope_dh = rope_head_dim;
  const W4Plan p = w4_plan(M, g.flip_row, N, K, 1, 0, 0, *height);
  QZO_HIP(*height ? launch_w4_tiles(g, p, (hipStream_t)stream) : launch_w4(g, p, (hipStream_t)stream));
  W4Plan head, tail;
  *height = !*height && w4_two_heights(p, M, K, &head, &tail) ? head.mt | tail.mt << 16 : p.mt;
  return QZO_OK;
}

qzo_status qzo_debug_attention_slices(const float* part_dev, uint32_t slices, uint32_t batch, uint32_t seq, uint32_t n_heads,
                                      uint32_t head_dim, const float* rope_dev, int joined, void* qkv_dev, void* out_dev,
                                      uint32_t* joined_out, void* stream) {
  if (!part_dev || !rope_dev || !qkv_dev || !out_dev || !joined_out) return fail(QZO_ERR_ARG, "null pointer");
  if (!aligned16(part_dev) || !aligned16(rope_dev) || !aligned16(qkv_dev) || !aligned16(out_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (batch == 0 || seq == 0 || seq > ATTENTION_ROPE_MAX_S || n_heads == 0 || n_heads > 1024 || (head_dim != 64 && head_dim != 128) ||
      slices == 0 || (uint64_t)batch * seq > (1u << 20) || (uint64_t)slices * batch * seq * 3 * n_heads * head_dim >= (1ull << 29))
    return fail(QZO_ERR_SHAPE, "need seq <= 256, heads of 64 or 128 features, slices of less than 2^31 bytes in all");
  hipStream_t st = (hipStream_t)stream;
  NextAttention na = {batch, seq, n_heads, head_dim, nullptr, 0};
  GemmArgs g = {};
  g.y = qkv_dev; g.M = batch * seq; g.N = 3 * n_heads * head_dim;
  g.next_attention = joined ? &na : nullptr;
  QZO_HIP(launch_partial_reduce(g, part_dev, slices, st));
  *joined_out = na.part ? 1u : 0u;
  QZO_HIP(launch_attention(qkv_dev, batch, seq, n_heads, head_dim, out_dev, rope_dev, st, na.part, na.slices));
  return QZO_OK;
}

qzo_status qzo_debug_attention_linear(const void* qkv_dev, uint32_t batch, uint32_t seq, uint32_t n_heads, uint32_t passes,
                                      const float* rope_dev, int packed, void* att_dev, float* xsum_dev, const void* q_dev,
                                      const void* s_dev, const void* zp_dev, int scale_fp16, uint32_t N, uint32_t row_base,
                                      uint64_t seed, float eps, int sign, float* part_dev, uint64_t part_floats,
                                      uint32_t* slices_out, void* y_dev, void* stream) {
  if (!qkv_dev || !att_dev || !xsum_dev || !q_dev || !s_dev || !part_dev || !slices_out || !y_dev) return fail(QZO_ERR_ARG, "null pointer");
  if (!aligned16(qkv_dev) || !aligned16(rope_dev) || !aligned16(att_dev) || !aligned16(xsum_dev) || !aligned16(q_dev) || !aligned16(s_dev) ||
      !aligned16(zp_dev) || !aligned16(part_dev) || !aligned16(y_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if ((passes != 1 && passes != 2) || (sign != 1 && sign != -1)) return fail(QZO_ERR_ARG, "passes must be 1 or 2, sign +1 or -1");
  const uint64_t M1 = (uint64_t)batch * seq, K = (uint64_t)n_heads * 128;
  if (M1 == 0 || M1 > SKINNY_MAX_M || n_heads == 0 || n_heads > 1024 || N == 0 || N % 8 || !skinny_fits(passes * (uint32_t)M1, N, (uint32_t)K))
    return fail(QZO_ERR_SHAPE, "need 1 to 64 tokens a pass, N a multiple of 8, operands and partial sums below 2^31 bytes");
  if (part_floats < skinny_ws_floats(passes * (uint32_t)M1, N, (uint32_t)K)) return fail(QZO_ERR_WORKSPACE, "part_dev too small");
  hipStream_t st = (hipStream_t)stream;
  const XPack pack = packed ? few_pack((uint32_t)M1, passes == 2) : XPack{};
  QZO_HIP(launch_attention(qkv_dev, passes * batch, seq, n_heads, 128, att_dev, rope_dev, st, nullptr, 0, pack, xsum_dev));
  GemmArgs g = {};
  g.x = att_dev; g.w = q_dev; g.s = s_dev; g.zp = zp_dev; g.y = y_dev;
  g.M = (uint32_t)M1; g.N = N; g.K = (uint32_t)K; g.dual = passes == 2;
  g.row_base = row_base; g.s_fp16 = scale_fp16 != 0;
  g.seed_lo = (uint32_t)seed; g.seed_hi = (uint32_t)(seed >> 32); g.eps_signed = sign > 0 ? eps : -eps;
  g.xp = pack; g.xsum = packed ? xsum_dev : nullptr;
  QZO_HIP(launch_skinny_gemm(g, part_dev, st));
  *slices_out = (uint32_t)(skinny_ws_floats(1, N, (uint32_t)K) / N);
  return QZO_OK;
}

qzo_status qzo_debug_reduce_norm(const float* part_dev, uint32_t slices, uint32_t M, uint32_t N, const void* bias_dev,
                                 const void* resid_dev, const void* gain_dev, const void* norm_bias_dev, float eps,
                                 int joined, void* y_dev, void* out_dev, float* xsum_dev, uint32_t* joined_out,
                                 void* stream) {
  if (!part_dev || !resid_dev || !gain_dev || !y_dev || !out_dev || !joined_out) return fail(QZO_ERR_ARG, "null pointer");
  if (!aligned16(part_dev) || !aligned16(bias_dev) || !aligned16(resid_dev) || !aligned16(gain_dev) ||
      !aligned16(norm_bias_dev) || !aligned16(y_dev) || !aligned16(out_dev) || !aligned16(xsum_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (M == 0 || N == 0 || N % 128 || slices == 0 || (uint64_t)slices * M * N >= (1ull << 31))
    return fail(QZO_ERR_SHAPE, "need M >= 1, N a positive multiple of 128, slices >= 1, slices*M*N below 2^31");
  hipStream_t st = (hipStream_t)stream;
  NextNorm nn = {gain_dev, norm_bias_dev, eps, out_dev, xsum_dev, XPack{}, false};
  GemmArgs g = {};
  g.bias = bias_dev; g.resid = resid_dev; g.y = y_dev; g.M = M; g.N = N;
  g.epi = EPI_RESIDUAL | (bias_dev ? EPI_BIAS : 0u);
  g.next = joined ? &nn : nullptr;
  QZO_HIP(launch_partial_reduce(g, part_dev, slices, st));
  *joined_out = nn.done ? 1u : 0u;
  if (!nn.done)
    QZO_HIP(norm_bias_dev ? launch_layernorm(y_dev, gain_dev, norm_bias_dev, M, N, eps, out_dev, st, xsum_dev)
                          : launch_rmsnorm(y_dev, gain_dev, M, N, eps, out_dev, st, xsum_dev));
  return QZO_OK;
}

qzo_status qzo_apply_update_channel(void* c_dev, uint32_t n_rows, uint32_t row_base, uint64_t seed,
                                    float eta, float d_clipped, void* stream) {
  if (!c_dev) return fail(QZO_ERR_ARG, "c_dev is null");
  if (!std::isfinite(eta) || !std::isfinite(d_clipped)) return fail(QZO_ERR_ARG, "eta/d' not finite");
  QZO_HIP(launch_channel_update(c_dev, n_rows, row_base, (uint32_t)seed, (uint32_t)(seed >> 32), eta,
                                d_clipped, nullptr, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_debug_mfma_rate(uint32_t iters, int random_operands, float* sink_dev,
                               uint32_t* workgroups_out, void* stream) {
  if (!sink_dev || !workgroups_out) return fail(QZO_ERR_ARG, "null pointer");
  if (iters == 0 || iters > (1u << 20)) return fail(QZO_ERR_ARG, "iters must be 1 .. 2^20");
  const uint32_t wgs = gemm_workgroups(1u << 20, 1u << 20);      // one per compute unit
  *workgroups_out = wgs;
  QZO_HIP(launch_mfma_rate(sink_dev, wgs, iters, random_operands != 0, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_profile_begin(uint32_t max_records) {
  while (g_prof.pool.size() < max_records) {
    ProfRec r = {};
    QZO_HIP(hipEventCreate(&r.a));
    QZO_HIP(hipEventCreate(&r.b));
    g_prof.pool.push_back(r);
  }
  g_prof.used = 0;
  for (uint32_t& c : g_prof.seen) c = 0;
  g_prof.on = true;
  return QZO_OK;
}

qzo_status qzo_profile_stride(uint32_t stride) {
  if (stride == 0) return fail(QZO_ERR_ARG, "stride must be >= 1");
  g_prof.stride = stride;
  return QZO_OK;
}

qzo_status qzo_profile_collect(uint32_t kind, double* total_ms, uint64_t* launches, double* work) {
  if (!total_ms || !launches || !work) return fail(QZO_ERR_ARG, "null output");
  if (kind >= PK_COUNT) return fail(QZO_ERR_ARG, "unknown kernel class");
  g_prof.on = false;
  double ms = 0, wk = 0;
  uint64_t n = 0;
  for (size_t i = 0; i < g_prof.used; ++i) {
    ProfRec& r = g_prof.pool[i];
    if (r.kind != kind) continue;
    QZO_HIP(hipEventSynchronize(r.b));
    float t = 0;
    QZO_HIP(hipEventElapsedTime(&t, r.a, r.b));
    ms += t;
    wk += r.work;
    ++n;
  }
  *total_ms = ms; *launches = n; *work = wk;
  return QZO_OK;
}

qzo_status qzo_rtn_quantize(const float* w_dev, uint32_t N, uint32_t K, uint32_t group, void* q_dev,
                            void* s_dev, void* stream) {
  if (!w_dev || !q_dev || !s_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(w_dev) || !aligned16(q_dev) || !aligned16(s_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (group != 128 || K % 128) return fail(QZO_ERR_SHAPE, "group must be 128 and divide K");
  QZO_HIP(launch_rtn_quantize(w_dev, N, K, q_dev, s_dev, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_rtn_quantize_asym(const float* w_dev, uint32_t N, uint32_t K, uint32_t group,
                                 uint32_t scale_fp16, void* q_dev, void* zp_dev, void* s_dev, void* stream) {
  if (!w_dev || !q_dev || !zp_dev || !s_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(w_dev) || !aligned16(q_dev) || !aligned16(s_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (group != 128 || K % 128) return fail(QZO_ERR_SHAPE, "group must be 128 and divide K");
  if (scale_fp16 > 1) return fail(QZO_ERR_ARG, "scale_fp16 must be 0 or 1");
  QZO_HIP(launch_rtn_quantize_asym(w_dev, N, K, scale_fp16 != 0, q_dev, zp_dev, s_dev, (hipStream_t)stream));
  return QZO_OK;
}

qzo_status qzo_debug_normals(uint64_t seed, uint32_t stream_id, uint32_t row0, uint32_t n_rows,
                             uint32_t G, float* out_dev, void* stream) {
  if (!out_dev) return fail(QZO_ERR_ARG, "out_dev is null");
  QZO_HIP(launch_debug_normals((uint32_t)seed, (uint32_t)(seed >> 32), stream_id, row0, n_rows, G,
                               out_dev, (hipStream_t)stream));
  return QZO_OK;
}
qzo_status qzo_debug_philox(uint64_t seed, const uint32_t* ctr_dev, uint32_t n, uint32_t* out_dev,
                            void* stream) {
  if (!ctr_dev || !out_dev) return fail(QZO_ERR_ARG, "null device pointer");
  QZO_HIP(launch_debug_philox((uint32_t)seed, (uint32_t)(seed >> 32), ctr_dev, n, out_dev,
                              (hipStream_t)stream));
  return QZO_OK;
}
qzo_status qzo_debug_normal_pairs(const uint32_t* words_dev, uint32_t n, float* out_dev,
                                  void* stream) {
  if (!words_dev || !out_dev) return fail(QZO_ERR_ARG, "null device pointer");
  QZO_HIP(launch_debug_normal_pairs(words_dev, n, out_dev, (hipStream_t)stream));
  return QZO_OK;
}
qzo_status qzo_debug_dequant(const void* q_dev, const void* s_dev, uint32_t row_base, uint32_t N,
                             uint32_t K, uint32_t group, uint64_t seed, float eps, int sign,
                             void* w_eff_dev, void* stream) {
  return qzo_debug_dequant_zp(q_dev, s_dev, nullptr, 0u, row_base, N, K, group, seed, eps, sign, w_eff_dev,
                              stream);
}

qzo_status qzo_debug_dequant_zp(const void* q_dev, const void* s_dev, const void* zp_dev,
                                uint32_t scale_fp16, uint32_t row_base, uint32_t N, uint32_t K,
                                uint32_t group, uint64_t seed, float eps, int sign, void* w_eff_dev,
                                void* stream) {
  if (scale_fp16 > 1) return fail(QZO_ERR_ARG, "scale_fp16 must be 0 or 1");
  if (!q_dev || !s_dev || !w_eff_dev) return fail(QZO_ERR_ARG, "null device pointer");
  if (!aligned16(q_dev) || !aligned16(s_dev) || !aligned16(w_eff_dev))
    return fail(QZO_ERR_ALIGN, "device pointer not 16-byte aligned");
  if (group != 128 || K == 0 || K % 128) return fail(QZO_ERR_SHAPE, "group must be 128 and divide K");
  if (sign != 1 && sign != -1) return fail(QZO_ERR_ARG, "sign must be +1 or -1");
  QZO_HIP(launch_debug_dequant(q_dev, s_dev, zp_dev, scale_fp16 != 0, row_base, N, K, (uint32_t)seed, (uint32_t)(seed >> 32),
                               sign > 0 ? eps : -eps, w_eff_dev, (hipStream_t)stream));
  return QZO_OK;
}

}  // extern "C"
