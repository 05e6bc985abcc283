// Internal declarations shared by the host API and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/moe_lrc.h"
#include "layout.h"

namespace lrc {

// Device-visible description of one expert: where its packed projections live.
struct ExpertDesc {
  const uint32_t* codes[3];
  const uint32_t* meta[3];
  const _Float16* af[3];      // packed A factor (null if none); a pair held at 3 bits: the code dwords of its units
  const _Float16* bf[3];      // packed B factor; at 3 bits: the metadata of its units
  const uint32_t* afm[3];     // pairs held at 3 bits (layout.h): metadata of the A units ...
  const uint32_t* bfc[3];     // ... and code dwords of the B units
  float lambda[3];            // power-of-two pre-scale folded into the metadata
  float inv_lambda[3];
  float xa_scale[3];          // what (in A) is multiplied by: lambda, over the power-of-two factors folded into a
                              // 3-bit pair's operands
  int32_t rank[3];            // rank of each projection's factor pair (0: none); a prefix of the factor sections
  int32_t has_factors;
  int32_t q3;                 // bit m: projection m's pair is held at 3 bits
};

// Byte offsets of the sections of an expert's two blobs (weights: codes+meta; factors: A+B).
struct BlobLayout {
  MatLayout mat[3];
  size_t off_codes[3], off_meta[3], off_af[3], off_bf[3];
  size_t w_bytes, f_bytes;
};

struct Workspace {       // carved out of the caller's buffer; all offsets 256-byte aligned
  size_t topk_idx, topk_w, counts, offsets, comp_counts, row_pair, pair_row;
  size_t y_rows, xh, xh_sh, h, p13, p2, y_part, sh_y_part, sh_h, sh_y, plan, plan2, tok_exp, row_exp, row_exp_sh;
  size_t cmp_index, cmp_list, total;
};

}  // namespace lrc

struct moe_lrc_stack;

struct moe_lrc_layer {
  moe_lrc_config cfg;
  int device;
  moe_lrc_stack* pool = nullptr;       // pooled residency: the stack whose slot pool serves this layer
  int pool_index = -1;                 // ... and the layer's place in it
  size_t dev_w_base = 0;               // device pointer of expert e's weights: d_w + w_off[e] - dev_w_base (pooled
                                       // residency keeps only the shared experts on the device)
  int n_cu = 0;                        // compute units of `device`
  lrc::BlobLayout routed, shared;
  int n_total;                         // E + S
  uint8_t* d_w = nullptr;              // device: weight blobs (resident) or slot pool (staged)
  uint8_t* d_f = nullptr;              // device: factor blobs / slots
  uint8_t* h_w = nullptr;              // pinned host pool (staged only)
  uint8_t* h_f = nullptr;
  std::vector<size_t> w_off, f_off;    // per-expert offsets into the pools
  lrc::ExpertDesc* d_desc = nullptr;
  std::vector<lrc::ExpertDesc> h_desc;
  uint64_t desc_gen = 1;               // counts what writes h_desc and d_desc outside a stack's steps
  uint16_t* d_wg = nullptr;
  float* d_bias = nullptr;
  double* d_logits = nullptr;          // [max_tokens][E] gate logits of the routing paths that go through memory (many experts)
  bool gate_set = false, has_bias = false;
  std::vector<uint8_t> mat_set;        // [n_total*3]
  std::vector<int> mat_rank;           // [n_total*3] rank of each projection's factor pair (Section 3.1: may differ)
  std::vector<uint8_t> mat_q3;         // [n_total*3] 1: the pair is held at 3 bits (layout.h), in the projection's own
                                       // factor sections, and dequantized by the kernels that consume it
  std::vector<float> mat_inv_mu;       // [n_total*3] 1 / (the power-of-two factors folded into a 3-bit pair's operands)
  int live13 = 0, live2 = 0;           // 16-column tiles of the A factors of W1 and W3, and of W2, over all experts
  int n_q3 = 0;                        // projections held at 3 bits (0: the launches take the kernels without that path)
  size_t f_total = 0;                  // bytes of d_f (and of h_f)
  int32_t* d_perm = nullptr;           // block counters of the grouping of many pairs by several blocks (kPermuteScratchInts)
  int32_t* d_stat = nullptr;           // [2 + 2E]: active, comp-active, counts, comp counts
  int32_t* h_stat = nullptr;           // pinned mirror
  hipStream_t side = nullptr;
  hipEvent_t ev_t0 = nullptr, ev_t1 = nullptr;   // bracket the staged copies on the side stream
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;   // shared experts on the side stream (resident mode)
  moe_lrc_stats stats{};
  bool stats_valid = false;
  int ksplit13 = 1, ksplit2 = 1;
  bool profile = false, profile_valid = false;
  hipEvent_t marks[MOE_LRC_N_STAGES + 1] = {};   // stage i runs between marks[i] and marks[i+1]
};

namespace lrc {

int set_error(int code, const std::string& msg);
// returns MOE_LRC_EHIP (with the call's text and HIP's message as the last error) if a HIP call fails
#define LRC_HIP(expr)                                                                       \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return lrc::set_error(MOE_LRC_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)
Workspace plan_workspace(const moe_lrc_layer* L, int T);

// ---- kernel launchers (each returns hipError_t of the launch) ------------------------------
// tok_exp (may be null): receives every token's pre-scale exponent (ffn_common.h)
// guess: a second layer of the same hidden size whose gate is applied to the same tokens (layer == null: none)
struct RouteGuess { const moe_lrc_layer* layer; int32_t* idx; float* w; };
hipError_t launch_route(const moe_lrc_layer* L, const void* x, int T, int32_t* idx, float* w,
                        _Float16* xh /*may be null*/, int32_t* tok_exp, hipStream_t s, const RouteGuess& guess = RouteGuess{nullptr, nullptr, nullptr});
// Batches whose routing is tiled on the fp64 matrix cores instead of one block per token: at least 128
// tiles of 16 tokens x 16 experts and 2^26 products.  Whole call, one block per token -> tiled, us.  Above the line no
// shape measured loses: H = 2048, E = 128: T = 256 24.3 -> 17.4, 512 30.7 -> 22.9; E = 64: 512 18.5 -> 16.9,
// 2048 45 -> 37; H = 4096, E = 8: 2048 29.1 -> 22.2, 4096 56 -> 26; H = 1216, E = 60: 1001 24.3 -> 15.5.  The two cross
// below it, at no one product of the sizes (a block per token fills the chip in steps of T, a tile takes H in
// series): H = 2048, E = 128: T = 128 13.8 -> 15.2, 160 23.9 -> 15.5, 255 24.4 -> 17.6; E = 64: 256 14.9 -> 14.7,
// 511 18.6 -> 17.1; H = 4096, E = 8: 1024 15.9 -> 20.2, 1400 22.2 -> 20.8, 2047 29.1 -> 22.6; E = 32: 512 16.9 -> 21.2,
// 700 24.8 -> 22.0; H = 5120, E = 16: 512 24.9 -> 23.3, 1800 94 -> 25; H = 512, E = 120: 128 10.7 -> 13.6,
// 1000 25.6 -> 15.7.  The line is on the safe side of all of these.
inline bool tiled_gate(int T, int E, int H) {
  return ((T + 15) / 16) * ((E + 15) / 16) >= 128 && (long long)T * E * H >= (1 << 26);
}
hipError_t launch_permute(const moe_lrc_layer* L, const int32_t* idx, int T, int32_t* counts,
                          int32_t* offsets, int32_t* row_pair, int32_t* pair_row,
                          int32_t* comp_counts, hipStream_t s);
struct PlanSpec;   // plan.h
struct FfnTables;
// the grouping of the pairs by expert run inside the preparing launch (few pairs): the routing
// kernel's indices in, the five arrays of moe_lrc_permute out
struct PermuteArgs { const int32_t* idx; int32_t *counts, *offsets, *row_pair, *pair_row, *comp_counts; int P; };
constexpr int kFusedPermuteMaxPairs = 1024;
// the routing of a token or two run inside the preparing launch as well (forward only): gate
// [E][H] bf16 and bias (or null) in, the outputs of moe_lrc_route and the tokens' pre-scale exponents out
struct RouteArgs { const uint16_t* wg; const float* bias; int32_t* idx; float* w; int32_t* tok_exp; int renorm; };
constexpr int kFusedRoutePairs = 16;      // (token, expert) gate products: one per wavefront of a block (always grouped by ballots, group_small)
// above this many pairs several blocks group them (two launches); their counters live in the layer
constexpr int kPermuteOneBlockPairs = 8192, kPermuteMaxBlocks = 64;
constexpr int kPermuteScratchInts = kPermuteMaxBlocks * 2 * 256 + 64;
// The routed rows that take the rank-r term (Section 3.2: the Top-n pairs), compacted per expert in
// row order by the preparing launch for the grouped (in A) kernels, which then touch only those
// rows.  Expert e's compact rows are offsets[e] .. offsets[e] + (its number of such rows) - 1, i.e.
// the front of its own row range: list [T * k] names the routed row of each compact row, index
// [T * k] the compact row of each routed row (-1 for a row without the term).
struct CompactArgs { int32_t *index, *list; };
// The last rows of the operand-order buffers, which the decode flavour stages in place of rows past
// an expert's last one (decode_index.h, staged_row), are kept at zero by one block of the preparing
// launch: those of its own output and, if given, of the buffer `h` (h_rt rows, Fp columns) that the
// fused projection writes next.
struct ZeroRowsArgs { uint4* h; int h_rt, Fp; };
// fp16 copy of the activations in operand order, every row times its power-of-two pre-scale
// (ffn_common.h; exponents to row_exp, taken from tok_exp per token if given): one row per routed
// pair (row_pair given) or one per token (row_pair null); with `stat`, one more block counts the
// per-expert rows
struct FfnArgs;
// xa13: the arguments of the expert-FFN launches that follow, when their fused W1|W3 projection takes
// the decode flavour and wants (x A1 | x A3) made by further blocks of this launch; else null
hipError_t launch_convert_x(const moe_lrc_layer* L, const void* x_bf16, int T, _Float16* xg, int rt,
                            const int32_t* offsets, const int32_t* row_pair, int32_t* stat,
                            const FfnTables* tables /* or null */, const FfnArgs* xa13,
                            const int32_t* tok_exp /* or null */, int32_t* row_exp,
                            const PermuteArgs* perm /* or null: offsets and row_pair are ready */,
                            const CompactArgs* cmp /* or null */, const RouteArgs* route /* or null: perm->idx is ready */,
                            const ZeroRowsArgs& zr,
                            hipStream_t s, int32_t* host_stat = nullptr /* pinned: a copy of `stat` for the host */);
// The preparing launch: threads of a block, and blocks side by side (grid.y) per 16 rows: a block covers 1024 columns in one
// go (two 8-column units per thread), and there are no more blocks than CUs.
constexpr int kPrepThreads = 1024;
inline int prep_columns(int hidden, int rows, int n_cu) {
  const int row_blocks = (rows + 15) / 16, most = n_cu / (row_blocks > 1 ? row_blocks : 1), want = hidden / (16 * (kPrepThreads / 16));
  return want < 1 || most < 1 ? 1 : want < most ? want : most;
}
// (x A1 | x A3) of every expert for every token instead of for the routed rows: it then waits neither for the routing
// nor for the grouping.  Up to 64 tokens in passes of 16 side by side, or of 32 where the grid has no more (xa_tokens_pass); ranks
// whose fragments are one per wavefront of the kernel that copies them.  xa_by_tokens is the part of the rule that does
// not depend on where the factors are: what is computed grows with factor tiles x experts x passes, and a CU holds one block of
// this launch, so only while these blocks leave a quarter of the CUs to the others and no block has a second pass; with more
// experts than 32, or than eight to a slot of the Top-k, most of it is not used.  Whole forward, by rows -> by tokens, us:
// 8 experts, Top-2, 2048 x 1024, T = 64, rank 64 (128 blocks) 55.4 -> 53.0, rank 128 (256) 54.0 -> 57.2; rank 128, T = 16 (128) 48.9 -> 47.5; 16
// experts, rank 32 (128) 52.5 -> 49.8, rank 64 (256) 53.9 -> 57.1; 8 experts, Top-1, 4096 x 1024, rank 64, T = 48 (192) 52.1 -> 50.7, T = 64
// (256) 53.0 -> 56.9; two passes of 32: hidden 1024, T = 64, rank 8 50.5 -> 52.9; 64 experts, Top-8, rank 16, T = 16 (128) 78.4 -> 79.5.
constexpr int kXaTokens = 64, kXaTokensRank = 128, kXaTokensExperts = 32;
LRC_HD int xa_tokens_pass(int T, int columns) { return 16 * columns >= T ? 16 : 32; }
inline bool xa_by_tokens(const moe_lrc_config& c, int T, int n_cu) {
  const int columns = prep_columns(c.hidden, T * c.top_k, n_cu), pass = xa_tokens_pass(T, columns), passes = (T + pass - 1) / pass;
  return c.rank > 0 && c.rank <= kXaTokensRank && c.top_n > 0 && T <= kXaTokens && c.n_experts <= kXaTokensExperts &&
         c.n_experts <= 8 * c.top_k && passes <= columns && 4 * passes * (2 * ((c.rank + 15) / 16) * c.n_experts) <= 3 * n_cu;
}
inline size_t xa_tokens_bytes(const moe_lrc_config& c, int T) {
  return (size_t(c.n_experts) * T + 1) * ((c.rank + 31) / 32) * 128;
}

constexpr int kMaxKBlocks = 8;    // most K-blocks the decode W2 kernel splits into
// blocks (per K-block) of a decode launch that shares its blocks out by a table: `target` (the
// device's CUs over the K-blocks), or enough for ceil(NT / 32) blocks per expert that can be active
inline int plan_blocks(int n_exp, int pairs, int NT, int target) {
  const int active = n_exp < pairs ? n_exp : pairs, base = (NT + 31) / 32;
  return active * base > target ? active * base : target;
}

constexpr int kActPadRows = 32;   // rows past the last one that a 32-row staging pass may read

struct FfnArgs {
  const ExpertDesc* desc;     // device array, already offset to the first expert of this launch
  int n_exp;                  // experts in this launch (grid.y)
  int bits, group, rank, rpad;
  int H, F, top_k, top_n, T;
  const int32_t* offsets;     // [n_exp+1] or null: shared experts, rows e*T .. e*T+T-1
  const int32_t* row_pair;    // null for shared experts (row -> token = row % T)
  const int32_t* comp_rows;   // [n_exp] rows that take the rank-r term (written by the prep kernel), or null
  const _Float16* xh;         // gathered activations in operand order, x_rt rows (routed: one per pair)
  _Float16* h;                // SwiGLU output in operand order, h_rt rows
  int x_rt, h_rt;
  float* p13;                 // (x A1 | x A3), fp16 [rows][2 * ls * 32] (ffn_common.h, KArgs::p)
  int p_tokens;               // ... or [n_exp][p_tokens tokens][2 * ls * 32] and a row of zeros (KArgs::p_tokens)
  int32_t* row_tok;           // ... then also [rows]: KArgs::row_tok, written by the preparing launch
  float* p2;                  // (h A2), fp16 [rows][ls * 32]; decode flavour: one per W2 K-block
  int n_shared;               // shared experts that the layer runs beside these
  float* ha;                  // decode flavour of both projections: room for ha_bytes of (h A2) part sums (decode_ha_bytes)
  size_t ha_bytes;
  void* y_rows;               // [rows][H] bf16
  float* y_part;              // fp32 partial outputs of the W2 K-blocks (decode flavour), or null
  int32_t *plan, *plan2;      // routed experts: the block or chunk tables (plan.h) of W1|W3 and of W2
  const void* x_tokens;       // the bf16 tokens [T][H] (routed launches)
  int xa13_here;              // decode flavour of W1|W3: (x A1 | x A3) is made by a launch of its own in front of the
                              // FFN kernel (staged layers: the factors arrive after the preparing launch) instead
                              // of by further blocks of the preparing launch
  int keep_partials;          // decode flavour, W2 split into K-blocks: leave the fp32 partial sums in y_part for
                              // the combine instead of adding them into y_rows
  int live13, live2;          // 16-column factor tiles that hold a pair's columns: those of W1 and W3, those of W2, summed
                              // over the experts
  int ksplit13, ksplit2;      // most K-blocks of the staged (in A) products (what p13 and p2 have room for)
  int total_rows;
  int n_cu;                   // compute units of the device (the launches size their grids to fill them)
  int q3;                     // some factor pair of the layer is held at 3 bits: the launches take the kernels that
                              // can dequantize such pairs
  const PermuteArgs* perm;    // forward with few pairs: the preparing launch groups the pairs itself (else null)
  const int32_t *cmp_index, *cmp_list;   // CompactArgs of this call (null: none made)
  int32_t* row_exp;           // per input row (routed: per routed row; shared: per token): pre-scale exponent
  const int32_t* tok_exp;     // per token, from the routing kernel, or null
  hipEvent_t* marks;          // null, or 4 events recorded after xa13, w13, xa2, w2
};
hipError_t launch_expert_ffn(const FfnArgs& a, hipStream_t s);
// K-blocks the decode flavour splits W2 into (1: none); the W2 output of a launch is y_rows, or with
// keep_partials that many fp32 partial sums [kb][rows][H] in y_part
int decode_w2_kblocks(const FfnArgs& a);
size_t decode_ha_bytes(const FfnArgs& a);   // what the part sums of (h A2) take of ha_bytes (0: that form is not taken)
// bit 0: the fused W1|W3 projection takes the grouped GEMM (else the decode flavour, up to this many expected rows per expert), bit 1: W2 does
constexpr int kDecodeMaxRows13 = 40;
int expert_ffn_path(const FfnArgs& a);
// once per device, before the first launch: lets the FFN kernels use the whole LDS of a CU
hipError_t ffn_init_device();
hipError_t decode_init_device();
// the tables (plan.h) that launch_expert_ffn(a) will read: to be made by launch_convert_x
FfnTables expert_ffn_tables(const FfnArgs& a);
// y_part != null: the expert outputs are the sums over `kblocks` fp32 partial sums [kb][T*k][H]
// (the decode flavour's W2 K-blocks) instead of the bf16 rows y_rows
// residual != null: out = residual + (the weighted sum), rounded once
hipError_t launch_combine(const moe_lrc_layer* L, const void* y_rows, const float* y_part, int kblocks, const float* w,
                          const int32_t* pair_row, const void* y_shared, const void* residual, int T, void* out,
                          hipStream_t s);
// ---- host API internals shared with the layer stack (stack.hip) ----
const BlobLayout& blob_of(const moe_lrc_layer* L, int expert);
void factor_section_bytes(const moe_lrc_layer* L, int e, int mat, size_t& a_bytes, size_t& b_bytes);
void set_factor_ptrs(const moe_lrc_layer* L, int e, int mat, ExpertDesc& d, const uint8_t* a_base, const uint8_t* b_base);
void fill_algorithmic_stats(moe_lrc_layer* L, const int32_t* stat);
// moe_lrc_forward after its argument checks; residual as in launch_combine
int forward_impl(moe_lrc_layer* L, const void* x, int T, void* out, void* ws, hipStream_t s, const void* residual);
// pooled residency (stack.hip).  pool_begin, before the preparing launch: *ahead if the FFN kernels may be
// launched before the host knows the counts; pool_counts_written:
// right after the preparing launch, which has written the counts to L->h_stat; pool_stage: waits for them,
// brings the experts that received rows into slots of the stack's pool, points the layer's expert table at
// them and makes `s` wait for the copies; *complete if everything was in place already
RouteGuess pool_guess(const moe_lrc_layer* L);
int pool_begin(moe_lrc_layer* L, bool* ahead);
int pool_counts_written(moe_lrc_layer* L, hipStream_t s);
int pool_stage(moe_lrc_layer* L, int T, hipStream_t s, bool* complete);
hipError_t launch_debug_unpack(const uint32_t* packed, const MatLayout& m, uint8_t* codes_dev,
                               hipStream_t s);
}  // namespace lrc
