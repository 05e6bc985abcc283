// Weighted combine (Section 2.1: y = sum_{i in TopK} w_i E_i(x)), the fp16 activation copy with the
// per-call expert statistics, and the unpack hook that reads the private packed layout back.
#include <algorithm>

#include "decode_index.h"
#include "internal.h"
#include "permute_body.h"
#include "plan.h"
#include "route_body.h"
#include "unpack.h"
#include "xa_rows.h"

namespace lrc {

namespace {

__device__ inline float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ inline float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ inline uint32_t pack_bf16(float a, float b) {
  uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  ua += 0x7fffu + ((ua >> 16) & 1u);
  ub += 0x7fffu + ((ub >> 16) & 1u);
  return (ua >> 16) | (ub & 0xffff0000u);
}

// out[t] = sum_j w[t][j] * y_rows[pair_row[t*k+j]] + sum_s y_shared[s*T+t]; slots in order j = 0..k-1,
// then the shared experts: a fixed order, so two runs give identical bits.  With y_part, row R's
// output is the sum over the K-blocks kb = 0.. of y_part[kb][R] (fp32, in that order) instead of
// the bf16 row y_rows[R].
// PARTS: the rows come as K-block parts (y_part); else as bf16 rows (y_rows).
template <bool PARTS>
__global__ __launch_bounds__(256) void combine_kernel(const uint16_t* __restrict__ y_rows,
                                                      const float* __restrict__ y_part, int kblocks, size_t kb_stride,
                                                      const float* __restrict__ w,
                                                      const int32_t* __restrict__ pair_row,
                                                      const uint16_t* __restrict__ y_shared,
                                                      const uint16_t* __restrict__ residual, int T, int H,
                                                      int top_k, int n_shared, uint16_t* __restrict__ out) {
  // (grid.y walks the 8-column chunks of a row in steps of the block size: few tokens still make many blocks)
  const int t = blockIdx.x;
  for (int ch = blockIdx.y * 256 + threadIdx.x; ch < H / 8; ch += 256 * gridDim.y) {
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int j = 0; j < top_k; ++j) {
      const int row = pair_row[t * top_k + j];
      const float wj = w[t * top_k + j];
      if constexpr (PARTS) {
        // every K-block's part is requested before the first is added; the additions keep the
        // order kb = 0, 1, ...
        float4 pl[kMaxKBlocks], ph[kMaxKBlocks];
#pragma unroll
        for (int kb = 0; kb < kMaxKBlocks; ++kb) {
          if (kb < kblocks) {
            const float4* s2 = reinterpret_cast<const float4*>(y_part + kb * kb_stride + size_t(row) * H) + 2 * ch;
            pl[kb] = s2[0]; ph[kb] = s2[1];
          }
        }
        float4 lo = pl[0], hi = ph[0];
#pragma unroll
        for (int kb = 1; kb < kMaxKBlocks; ++kb) {
          if (kb >= kblocks) break;
          const float4 a = pl[kb], b = ph[kb];
          lo.x += a.x; lo.y += a.y; lo.z += a.z; lo.w += a.w;
          hi.x += b.x; hi.y += b.y; hi.z += b.z; hi.w += b.w;
        }
        acc[0] = fmaf(wj, lo.x, acc[0]); acc[1] = fmaf(wj, lo.y, acc[1]); acc[2] = fmaf(wj, lo.z, acc[2]); acc[3] = fmaf(wj, lo.w, acc[3]);
        acc[4] = fmaf(wj, hi.x, acc[4]); acc[5] = fmaf(wj, hi.y, acc[5]); acc[6] = fmaf(wj, hi.z, acc[6]); acc[7] = fmaf(wj, hi.w, acc[7]);
      } else {
        const uint4 v = reinterpret_cast<const uint4*>(y_rows + size_t(row) * H)[ch];
        const uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[2 * i] = fmaf(wj, bf16_lo(a[i]), acc[2 * i]);
          acc[2 * i + 1] = fmaf(wj, bf16_hi(a[i]), acc[2 * i + 1]);
        }
      }
    }
    for (int s = 0; s < n_shared; ++s) {
      const uint4 v = reinterpret_cast<const uint4*>(y_shared + (size_t(s) * T + t) * H)[ch];
      const uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] += bf16_lo(a[i]);
        acc[2 * i + 1] += bf16_hi(a[i]);
      }
    }
    if (residual != nullptr) {                 // a stack of layers: out = x + layer(x)
      const uint4 v = reinterpret_cast<const uint4*>(residual + size_t(t) * H)[ch];
      const uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] += bf16_lo(a[i]);
        acc[2 * i + 1] += bf16_hi(a[i]);
      }
    }
    reinterpret_cast<uint4*>(out + size_t(t) * H)[ch] =
        make_uint4(pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3]), pack_bf16(acc[4], acc[5]),
                   pack_bf16(acc[6], acc[7]));
  }
}

// ceil(rows/16) blocks write the fp16 copy of sixteen rows' tokens in operand order (the layout
// the FFN kernels stage from, see act_unit in ffn_common.h): row R of the routed rows is the token
// of pair row_pair[R]; without row_pair, row R is token R.  Thread (row r = t % 16, column lane
// t / 16) converts the 16-byte units t / 16, t / 16 + 64, ... of its row: a wavefront reads 64
// contiguous bytes of each of its rows and writes runs of 256 bytes (sixteen rows of one unit).
// The blocks in front of those count, one wavefront per expert, the routed rows and the rows that take
// the rank-r term (what the router-guided transfer must bring in): stat = [-, -, rows[E], comp rows[E]].
// (and compact the latter for the grouped (in A) kernels, CompactArgs).  They are first because one of them is the longest
// chain of a large batch: an expert that nearly every token takes has its rows counted one batch after the other (Qwen3 shape,
// T = 4096, 4096 rows on one expert: launch 80 -> 50 us with the counting in front and eight batches requested together,
// and without a pass over the rows for their exponents, which the routing leaves).
// Then one block makes the tables of the FFN launches (plan.h), and xa_tiles * E further
// blocks compute (x A1 | x A3) for the decode flavour of the fused projection from the bf16 tokens
// (xa_rows.h), so that no launch of its own stands between this one and the W1|W3 kernel.
// Where that is done for every token and expert (KArgs::p_tokens) those blocks run beside the grouping instead of
// after it, and the row blocks leave, per routed row, which token's result it takes (row_tok).
// Bound: the longest chain of dependent loads (grouping, then the tokens or the tables; tokens and factors,
// then a sum over the wavefronts); Mixtral shape T = 64 17.2 -> 11.2 us, T = 1 15.3 -> 11.8, since neither waits for the other
// and the tables are made without 64-bit divisions from counts read once.
// At most this many blocks for the passes of (x A1 | x A3) beyond the experts' first ones.  Whole forward, us, with 0 / 32 / 64 / 128 / 256: Qwen3
// shape T = 64 87.2 / 86.2 / 86.1 / 86.2 / 86.1, T = 128 145.9 / 139.8 / 134.5 / 134.4 / 134.4, T = 256 263 / 243 / 236 / 230 / 230, rank 64
// T = 64 94.7 / 99.6 / 96.4 / 96.3 / 96.3, T = 128 151.5 / 166.1 / 155.7 / 149.2 / 145.3; Mixtral rank 64 T = 160 271.6 / 268.7 / 266.7 / 265.6 /
// 265.9; where no expert has more than 32 rows the same with any of them, while up to four blocks a tile, one a pass, cost 16 experts, rank 64,
// Top-1, T = 100 37.8 -> 50.6, 32 experts, Top-4, T = 128 51.9 -> 64.7.
constexpr int kMorePassBlocks = 128;
constexpr int kStatAhead = 8;              // batches of 64 rows whose pairs a counting wavefront asks for together
// With a token or two every block first routes them itself (route.wg != null).
// With few pairs, every block first groups the pairs by expert itself (perm.idx != null) instead of a launch of its own
// doing it beforehand: by ballots, into its LDS (group_small; the first of the last blocks writes the results out), or, of more pairs and
// experts, by the body of the permute kernel, writing the same values from every block; offsets and row_pair are then this block's
// own writes, read back after a barrier (hence no __restrict__ on them).
struct SmallRows {                         // grouped by this block, in its LDS
  const SmallGroup& sg;
  const int32_t* tok_exp;                  // null: the block has routed the tokens itself
  int top_k;
  __device__ int offset(int e) const { return sg.offset[e]; }
  __device__ int pair(int row) const { return sg.pair[row]; }
  __device__ int exponent(int pair, int) const { return tok_exp ? tok_exp[pair / top_k] : sg.tok_exp[pair / top_k]; }
};

// The launch's blocks in order: `stat` that count, row blocks x columns, `plan` for the tables, factor tiles x passes of
// (x A1 | x A3) and `more` for the passes that only some experts have, then `columns` that keep the zero rows.
struct PrepGrid {
  int stat, row_blocks, columns, plan, tiles, passes, more;
  LRC_HD int rows_at() const { return stat; }
  LRC_HD int plan_at() const { return stat + row_blocks * columns; }
  LRC_HD int xa_at() const { return plan_at() + plan; }
  LRC_HD int zero_at() const { return xa_at() + tiles * passes + more; }
  LRC_HD int blocks() const { return zero_at() + columns; }
};
// The passes of a factor tile run on one XCD (block b runs on XCD b % 8), whose L2 then holds the tile.
__device__ inline void xa_block(const PrepGrid& g, int i, int& tile, int& pass) {
  if (g.tiles % 8 == 0) {
    const int j = i / (8 * g.passes), in = i - j * 8 * g.passes;
    pass = in >> 3; tile = 8 * j + (in & 7);
  } else {
    pass = i / g.tiles; tile = i - pass * g.tiles;
  }
}

// What a block does once the pairs are grouped: its role by its index (XA: some have (x A1 | x A3) to make).
template <bool XA, class Rows>
__device__ inline void prep_roles(const Rows& grouped, const uint16_t* __restrict__ x, int rows, int H, uint4* __restrict__ xg, int rt, bool routed, int E,
                                  int top_k, int top_n, int32_t* __restrict__ stat, const FfnTables& tables, const PrepGrid& g, const ffn::KArgs& xa,
                                  bool have_exp, int32_t* __restrict__ row_exp, const CompactArgs& cmp, const ZeroRowsArgs& zr,
                                  int32_t* __restrict__ host_stat, int32_t* __restrict__ row_tok, ffn::float4_t (*red)[64], uint32_t* row_max) {
  constexpr int kWavesPerBlock = kPrepThreads / 64, kColLanes = kPrepThreads / 16;
  const int block = blockIdx.x;
  if (block >= g.zero_at()) {                                               // the zero rows
    const int n = (block - g.zero_at()) * kPrepThreads + threadIdx.x, step = kPrepThreads * g.columns;
    const int xu = (H + kTileK - 1) / kTileK * (kTileK / 8);               // 16-byte units per row
    for (int i = n; i < xu * dec::kZeroRows; i += step)
      xg[size_t(i / dec::kZeroRows) * rt + rt - dec::kZeroRows + i % dec::kZeroRows] = make_uint4(0, 0, 0, 0);
    if (zr.h != nullptr)
      for (int i = n; i < zr.Fp / 8 * dec::kZeroRows; i += step)
        zr.h[size_t(i / dec::kZeroRows) * zr.h_rt + zr.h_rt - dec::kZeroRows + i % dec::kZeroRows] = make_uint4(0, 0, 0, 0);
    return;
  }
  if constexpr (XA) {
    if (block >= g.xa_at()) {                                               // of the routed rows
      // Every tile has a block for its expert's first pass of 32 rows, which takes the others too where the launch has no blocks for them;
      // these deal out the passes beyond the first of the experts that have any (an expert with many rows must not be one block's chain
      // of passes, nor every tile have blocks for rows that only a few experts have: each block groups the pairs and takes a CU).
      constexpr int kOnly = 1 << 20;
      const int per = g.tiles / E, i = block - g.xa_at();
      if (i < g.tiles) {
        const int e = i / per;
        ffn::xa_rows_body<true, true, kWavesPerBlock>(xa, grouped, x, i - e * per, e, 0, 0, g.more > 0 ? kOnly : 1, red);
        return;
      }
      const auto offset = [&](int e) { return grouped.offset(e); };
      int e, pass;
      for (int item = i - g.tiles; further_pass(offset, E, item / per, threadIdx.x & 63, e, pass); item += g.more) {
        if (item >= g.more) __syncthreads();           // (the item before this one is done with the sums)
        ffn::xa_rows_body<true, true, kWavesPerBlock>(xa, grouped, x, item % per, e, 0, pass, kOnly, red);
      }
      return;
    }
  }
  if (block >= g.plan_at()) {                                               // the tables of the FFN launches (plan.h)
    const auto offset = [&](int e) { return grouped.offset(e); };
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (part < 2) make_plan(offset, E, part == 0 ? tables.plan[0] : tables.plan[1], part == 0 ? PlanSpec{0, 0, 0, nullptr} : tables.plan[0], lane);
    else if (part < 4) make_chunks(offset, E, part == 2 ? tables.chunk[0] : tables.chunk[1], lane);
    return;
  }
  if (block < g.rows_at()) {
    const int e = block * kWavesPerBlock + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (e >= E) return;
    const int b = grouped.offset(e), n = grouped.offset(e + 1) - b;
    // the expert's rows that take the rank-r term, counted and (for the grouped (in A) kernels,
    // CompactArgs) compacted in row order by ballot
    int comp = 0;
    for (int r0 = 0; r0 < n; r0 += 64 * kStatAhead) {
      int pair[kStatAhead];
#pragma unroll
      for (int u = 0; u < kStatAhead; ++u) pair[u] = grouped.pair(b + min(r0 + 64 * u + lane, n - 1));
#pragma unroll
      for (int u = 0; u < kStatAhead; ++u) {
        if (r0 + 64 * u >= n) break;
        const int r = r0 + 64 * u + lane;
        const bool f = r < n && pair[u] % top_k < top_n;
        const unsigned long long m = __ballot(f);
        if (cmp.index != nullptr) {
          const int at = b + comp + __popcll(m & ((1ull << lane) - 1ull));
          if (r < n) cmp.index[b + r] = f ? at : -1;
          if (f) cmp.list[at] = b + r;
        }
        comp += __popcll(m);
      }
    }
    if (lane == 0) { stat[2 + e] = n; stat[2 + E + e] = comp; }
    if (lane == 0 && host_stat != nullptr) { host_stat[2 + e] = n; host_stat[2 + E + e] = comp; }
    return;
  }
  const int at = block - g.rows_at(), column = at % g.columns;
  const int R = at / g.columns * 16 + (threadIdx.x & 15);
  const int pair = routed && R < rows ? grouped.pair(R) : 0, t = routed ? pair / top_k : R < rows ? R : 0;
  const uint4* xrow = reinterpret_cast<const uint4*>(x + size_t(t) * H);
  // The row's power-of-two pre-scale (ffn_common.h): from the routing kernel's per-token exponents,
  // or, without them, from a pass of this block over its sixteen rows.
  int se = 0;
  if (have_exp) {
    se = grouped.exponent(pair, R);
  } else {
    if (threadIdx.x < 16) row_max[threadIdx.x] = 0;
    __syncthreads();
    uint32_t m = 0;
    if (R < rows)
      for (int k8 = threadIdx.x >> 4; k8 < H / 8; k8 += kColLanes) {
        const uint4 v = xrow[k8];
        const uint32_t in[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) m = max(m, max(in[i] & 0x7fffu, (in[i] >> 16) & 0x7fffu));
      }
    atomicMax(&row_max[threadIdx.x & 15], m);
    __syncthreads();
    se = ffn::row_exponent(row_max[threadIdx.x & 15]);
  }
  if (R >= rows) return;
  if (column == 0 && (threadIdx.x >> 4) == 0) {
    row_exp[R] = se;
    if (row_tok != nullptr) row_tok[R] = pair - t * top_k < top_n ? t : -1;
  }
  const float sc = ffn::pow2i(se);
  // (the columns are split when there are few rows, so that the launch still fills the chip)
  // (two adjacent units per thread: a wavefront reads 128 contiguous bytes of each of its rows; H / 8 is even)
  for (int k8p = 2 * (column * kColLanes + (threadIdx.x >> 4)); k8p < H / 8; k8p += 2 * kColLanes * g.columns) {
    const uint4 vv[2] = {xrow[k8p], xrow[k8p + 1]};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k8 = k8p + u, ks = k8 >> 5, q = (k8 >> 3) & 3, s = k8 & 7;
      xg[size_t((ks * 8 + s) * 4 + q) * rt + R] = __builtin_bit_cast(uint4, ffn::scaled_unit(vv[u], sc));
    }
  }
}

// FULL: with the blocks of (x A1 | x A3) and the grouping, whose registers leave a CU one block.  Without either (batches beyond the decode
// flavour) the launch is the gather, many rounds of blocks, and a CU holds two
// (47 registers instead of 106).  Qwen3 shape, T = 4096: 52 -> 43 us (134 MB written); Mixtral, T = 2048: 20 -> 17.
template <bool FULL>
__global__ __launch_bounds__(kPrepThreads, FULL ? 4 : 8) void prep_kernel(const uint16_t* __restrict__ x, int rows, int H,
                                                   uint4* __restrict__ xg, int rt,
                                                   const int32_t* offsets,
                                                   const int32_t* row_pair, int E, int top_k,
                                                   int top_n, int32_t* __restrict__ stat, FfnTables tables, PrepGrid g, ffn::KArgs xa,
                                                   const int32_t* tok_exp, int32_t* __restrict__ row_exp,
                                                   PermuteArgs perm, CompactArgs cmp, RouteArgs route, ZeroRowsArgs zr,
                                                   int32_t* __restrict__ host_stat, int32_t* __restrict__ row_tok) {
  __shared__ uint32_t row_max[16];
  const bool routed = row_pair != nullptr;
  if constexpr (!FULL) {
    prep_roles<false>(ffn::GroupedRows{offsets, row_pair, tok_exp, row_exp, top_k}, x, rows, H, xg, rt, routed, E, top_k, top_n, stat, tables, g, xa,
                      tok_exp != nullptr, row_exp, cmp, zr, host_stat, row_tok, nullptr, row_max);
    return;
  } else {
    __shared__ ffn::float4_t red[2 * kPrepThreads / 64][64];
    __shared__ SmallGroup sg;
    constexpr int kWavesPerBlock = kPrepThreads / 64;
    const int block = blockIdx.x;
    if (xa.p_tokens > 0 && block >= g.xa_at() && block < g.zero_at()) {
      // (x A1 | x A3) of all tokens: nothing to wait for
      int tile, p;
      xa_block(g, block - g.xa_at(), tile, p);
      const int pass = xa_tokens_pass(xa.p_tokens, g.columns), per = g.tiles / E, e = tile / per;
      ffn::xa_tokens_body<kWavesPerBlock>(xa, x, route.wg != nullptr ? nullptr : tok_exp, tile - e * per, e, pass * p, pass == 32, red);
      return;
    }
    auto roles = [&](const auto& grouped, bool have_exp) {
      prep_roles<true>(grouped, x, rows, H, xg, rt, routed, E, top_k, top_n, stat, tables, g, xa, have_exp, row_exp, cmp, zr, host_stat, row_tok, red, row_max);
    };
    static_assert(kFusedRoutePairs <= kSmallExperts, "the pairs that this launch routes itself are grouped by ballots");
    if (perm.idx != nullptr && (route.wg != nullptr || group_small_fits(perm.P, E))) {
      const bool out = block == g.zero_at();     // the block that writes the results
      const PermuteOut o{perm.counts, perm.offsets, perm.row_pair, perm.pair_row, perm.comp_counts};
      if (route.wg != nullptr) {
        // a token or two: every block routes them itself (route_body.h) instead of a launch of its own doing it beforehand
        route_small_body(reinterpret_cast<double*>(&red[0][0]), sg.idx, sg.tok_exp, x, route, perm.P / top_k, H, E, top_k, out);
        __syncthreads();
        group_small(sg, [&](int i) { return sg.idx[i]; }, perm.P, E, top_k, top_n, out, o);
      } else {
        group_small(sg, [&](int i) { return perm.idx[i]; }, perm.P, E, top_k, top_n, out, o);
      }
      roles(SmallRows{sg, route.wg != nullptr ? nullptr : tok_exp, top_k}, true);
      return;
    }
    if (perm.idx != nullptr) {
      PermuteLds& pl = *reinterpret_cast<PermuteLds*>(&red[0][0]);     // (the reduction buffer is not in use yet)
      static_assert(sizeof(PermuteLds) <= sizeof(red), "the permutation tables must fit the reduction buffer");
      permute_body(pl, perm.idx, perm.P, E, top_k, top_n, perm.counts, perm.offsets, perm.row_pair, perm.pair_row, perm.comp_counts);
      __syncthreads();
    }
    roles(ffn::GroupedRows{offsets, row_pair, tok_exp, row_exp, top_k}, tok_exp != nullptr);
  }
}

// One wavefront per packed tile: runs the same field extraction as the FFN kernels and writes the
// integer codes back as one byte each.
template <int BITS>
__global__ __launch_bounds__(64) void unpack_kernel(const uint32_t* __restrict__ packed, int K, int N,
                                                    int KS, uint8_t* __restrict__ codes) {
  const int tile = blockIdx.x, NT = N / kTileN, ks = tile / NT, nt = tile % NT, lane = threadIdx.x;
  uint32_t w[2 * BITS];
  load_codes<BITS>(packed + size_t(tile) * kWave * 2 * BITS, lane, w);
  const int n = nt * kTileN + (lane & 15), kbase = ks * kTileK + (lane >> 4) * kLaneK;
#pragma unroll
  for (int pi = 0; pi < 32; ++pi) {
    const uint32_t f = Extract<BITS>::field(w, pi);
    const int k = kbase + 2 * pi;
    if (k < K) codes[size_t(k) * N + n] = (uint8_t)field_code<BITS>(f & 0xffffu, pi);
    if (k + 1 < K) codes[size_t(k + 1) * N + n] = (uint8_t)field_code<BITS>(f >> 16, pi);
  }
}

}  // namespace

hipError_t launch_combine(const moe_lrc_layer* L, const void* y_rows, const float* y_part, int kblocks, const float* w,
                          const int32_t* pair_row, const void* y_shared, const void* residual, int T, void* out,
                          hipStream_t s) {
  const moe_lrc_config& c = L->cfg;
  // enough blocks for the chip when there are few tokens: up to one per 256 chunks of 8 columns
  const int gy = std::max(1, std::min((c.hidden / 8 + 255) / 256, (2 * L->n_cu + T - 1) / T));
  auto kernel = y_part != nullptr ? combine_kernel<true> : combine_kernel<false>;
  hipLaunchKernelGGL(kernel, dim3(T, gy), dim3(256), 0, s, (const uint16_t*)y_rows, y_part, kblocks,
                     size_t(T) * c.top_k * c.hidden, w, pair_row,
                     (const uint16_t*)y_shared, (const uint16_t*)residual, T, c.hidden, c.top_k, c.n_shared, (uint16_t*)out);
  return hipGetLastError();
}

hipError_t launch_convert_x(const moe_lrc_layer* L, const void* x_bf16, int T, _Float16* xg, int rt,
                            const int32_t* offsets, const int32_t* row_pair, int32_t* stat,
                            const FfnTables* tables, const FfnArgs* xa13, const int32_t* tok_exp, int32_t* row_exp,
                            const PermuteArgs* perm, const CompactArgs* cmp, const RouteArgs* route, const ZeroRowsArgs& zr,
                            hipStream_t s, int32_t* host_stat) {
  const moe_lrc_config& c = L->cfg;
  const int rows = row_pair ? T * c.top_k : T;
  const int row_blocks = (rows + 15) / 16, ky = prep_columns(c.hidden, rows, L->n_cu);
  const FfnTables t = tables ? *tables : FfnTables{};
  const int plan_block = t.plan[0].plan || t.plan[1].plan || t.chunk[0].table || t.chunk[1].table ? 1 : 0;
  // (x A1 | x A3) of the decode flavour: 16-column tiles of both factors
  ffn::KArgs xa{};
  int xa_tiles = 0;
  if (xa13 && xa13->rank > 0 && xa13->top_n > 0 && row_pair) {
    const FfnArgs& f = *xa13;
    xa.desc = f.desc; xa.offsets = f.offsets; xa.row_pair = f.row_pair; xa.top_k = f.top_k; xa.top_n = f.top_n;
    xa.rank = f.rank; xa.ls = (f.rank + 31) / 32; xa.K = f.H; xa.p = f.p13; xa.total_rows = f.total_rows;
    xa.kb_steps = (f.H + kTileK - 1) / kTileK;
    xa.tok_exp = tok_exp; xa.row_exp = row_exp;
    xa.rpad = f.rpad; xa.n_exp = f.n_exp; xa.p_tokens = f.p_tokens;
    xa_tiles = 2 * f.rpad / 16;
  }
  const int stat_blocks = stat ? (c.n_experts + kPrepThreads / 64 - 1) / (kPrepThreads / 64) : 0;
  PrepGrid g{stat_blocks, row_blocks, ky, plan_block, xa_tiles * c.n_experts, 1, 0};
  if (xa.p_tokens > 0) {
    const int pass = xa_tokens_pass(xa.p_tokens, ky);
    g.passes = (xa.p_tokens + pass - 1) / pass;
  } else if (xa_tiles > 0 && T > 32) {
    // (experts with more than 32 rows have at most rows / 32 passes beyond their first ones)
    g.more = std::min(kMorePassBlocks, xa_tiles * (rows / 32));
  }
  const int cmp_block = (cmp && row_pair && stat) ? 1 : 0;     // (the compaction rides the per-expert counting)
  const bool full = xa_tiles > 0 || perm != nullptr;
  hipLaunchKernelGGL(full ? prep_kernel<true> : prep_kernel<false>, dim3(g.blocks()),
                     dim3(kPrepThreads), 0, s, (const uint16_t*)x_bf16, rows, c.hidden, reinterpret_cast<uint4*>(xg), rt, offsets,
                     row_pair, c.n_experts, c.top_k, c.top_n, stat, t, g, xa, tok_exp, row_exp,
                     perm ? *perm : PermuteArgs{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0},
                     cmp_block ? *cmp : CompactArgs{nullptr, nullptr},
                     (route && perm) ? *route : RouteArgs{nullptr, nullptr, nullptr, nullptr, nullptr, 0}, zr, host_stat,
                     xa_tiles > 0 && xa.p_tokens > 0 ? xa13->row_tok : nullptr);
  return hipGetLastError();
}

hipError_t launch_debug_unpack(const uint32_t* packed, const MatLayout& m, uint8_t* codes_dev,
                               hipStream_t s) {
  const dim3 grid(m.NT * m.KS), block(64);
  switch (m.bits) {
    case 2: hipLaunchKernelGGL(unpack_kernel<2>, grid, block, 0, s, packed, m.K, m.N, m.KS, codes_dev); break;
    case 3: hipLaunchKernelGGL(unpack_kernel<3>, grid, block, 0, s, packed, m.K, m.N, m.KS, codes_dev); break;
    case 4: hipLaunchKernelGGL(unpack_kernel<4>, grid, block, 0, s, packed, m.K, m.N, m.KS, codes_dev); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace lrc
