// Grouping of the (token, slot) pairs by expert: the body of the permute kernel, also run by every
// block of the launch that prepares the activations when there are few pairs (no launch of its own
// then).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.h"

namespace lrc {

constexpr int kMaxExperts = 256;
constexpr int kPermWaves = 16;
struct PermuteLds {
  int32_t hist[kPermWaves][kMaxExperts];
  int32_t comp[kMaxExperts];
  int32_t total[kMaxExperts];
};

// One workgroup of 16 wavefronts (1024 threads).  Wavefront w owns a contiguous run of pair ids, so
// pair order (= token order) is kept by walking the run in order and ranking equal experts inside
// each 64-pair step with ballots; per-(wavefront, expert) counters in LDS carry the positions.
// Ends with every result written (by this block) but not yet fenced: callers that read them back
// follow with __syncthreads().
// (idx carries no __restrict__: the caller may have written it itself just before)
__device__ inline void permute_body(PermuteLds& L, const int32_t* idx, int P, int E, int top_k, int top_n,
                                    int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                    int32_t* __restrict__ row_pair, int32_t* __restrict__ pair_row,
                                    int32_t* __restrict__ comp_counts) {
  auto& hist = L.hist;
  auto& comp = L.comp;
  auto& total = L.total;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < kPermWaves * kMaxExperts; i += 1024) (&hist[0][0])[i] = 0;
  for (int i = threadIdx.x; i < kMaxExperts; i += 1024) comp[i] = 0;
  __syncthreads();

  const int per_wave = ((P + kPermWaves - 1) / kPermWaves + 63) / 64 * 64;
  const int begin = wave * per_wave, end = min(P, begin + per_wave);
  for (int i = begin + lane; i < end; i += 64) {
    const int e = min(max(idx[i], 0), E - 1);     // out-of-range ids cannot leave the LDS tables
    atomicAdd(&hist[wave][e], 1);
    if (i % top_k < top_n) atomicAdd(&comp[e], 1);
  }
  __syncthreads();

  if (threadIdx.x < E) {
    int run = 0;
    for (int wv = 0; wv < kPermWaves; ++wv) {
      const int c = hist[wv][threadIdx.x];
      hist[wv][threadIdx.x] = run;
      run += c;
    }
    total[threadIdx.x] = run;
    counts[threadIdx.x] = run;
    comp_counts[threadIdx.x] = comp[threadIdx.x];
  }
  __syncthreads();
  if (threadIdx.x < E) {
    int off = 0;
    for (int e = 0; e < (int)threadIdx.x; ++e) off += total[e];
    offsets[threadIdx.x] = off;
    if ((int)threadIdx.x == E - 1) offsets[E] = off + total[threadIdx.x];
    for (int wv = 0; wv < kPermWaves; ++wv) hist[wv][threadIdx.x] += off;
  }
  __syncthreads();

  int nbits = 0;
  while ((1 << nbits) < E) ++nbits;
  for (int base = begin; base < end; base += 64) {
    const int i = base + lane;
    const bool valid = i < end;
    const int e = valid ? min(max(idx[i], 0), E - 1) : 0;
    unsigned long long same = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
      const bool bit = (e >> b) & 1;
      const unsigned long long bb = __ballot(valid && bit);
      same &= bit ? bb : ~bb;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1ull));
    const int cnt = __popcll(same);
    int pos = 0;
    if (valid) pos = hist[wave][e] + rank;
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) hist[wave][e] = pos + cnt;
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      row_pair[pos] = i;
      pair_row[i] = pos;
    }
  }
}

// The same for few pairs and experts by ballots alone (where group_small_fits): every wavefront groups all pairs for itself, without a
// barrier or a read back of what it has stored, and leaves the offsets and the rows' pairs in the block's LDS (all wavefronts write
// the same values there).  idx may be in LDS.  With `out` wavefront 0 writes the five arrays of the permute kernel.
// Every block of the launch that prepares the activations does this first, so its length counts once a round of blocks: two ballots and
// their counts per 64 pairs and expert, against the five barriers and the LDS tables of the kernel's body.  Whole forward, the body ->
// ballots, us, hidden 1024, by (steps of 64 pairs) x experts, no factors / rank 128: 2 30.7 -> 29.5 / 38.7 -> 38.0, 8 30.8 -> 29.4 / 37.0 -> 35.6, 9
// 1.2 less / 1.2 less, 12 0.9 less / 0.6 less with one step, 0.4 less / 0.1 more with two or more; 14 0.7 less / 0.4 more, 16 0.3 less / 1.9
// more with 16 experts, 24 34.2 -> 33.4 / 42.9 -> 43.4, 32 37.9 -> 39.9 / 55.0 -> 65.6 with 32 experts.
constexpr int kSmallPairs = 256, kSmallExperts = 16;      // (what it can take: the experts of a token that the launch routes itself)
LRC_HD bool group_small_fits(int P, int E) { return P <= kSmallPairs && (P + 63) / 64 * E <= 12; }
struct SmallGroup {
  int32_t offset[kSmallExperts + 1];
  int32_t pair[kSmallPairs];             // pair of every row
  int32_t idx[64];                       // the experts and exponents of the tokens that the block has routed itself
  int32_t tok_exp[64];
};
struct PermuteOut { int32_t *counts, *offsets, *row_pair, *pair_row, *comp_counts; };
template <class Idx>
__device__ inline void group_small(SmallGroup& sg, const Idx& idx, int P, int E, int top_k, int top_n, bool out, const PermuteOut& o) {
  constexpr int kPer = kSmallPairs / 64;
  const int lane = threadIdx.x & 63, steps = (P + 63) / 64;
  const unsigned long long below = (1ull << lane) - 1ull;
  int e[kPer], pos[kPer];
  unsigned long long comp[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    e[j] = -1; pos[j] = 0; comp[j] = 0;
    if (j >= steps) continue;
    const int i = lane + 64 * j;
    if (i < P) e[j] = min(max(idx(i), 0), E - 1);             // out-of-range ids cannot leave the tables
    comp[j] = __ballot(i < P && i % top_k < top_n);
  }
  int at = 0, my_first = 0, my_count = 0, my_comp = 0;
  for (int x = 0; x < E; ++x) {
    const int first = at;
    int n_comp = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (j >= steps) continue;
      const unsigned long long m = __ballot(e[j] == x);
      if (e[j] == x) pos[j] = at + __popcll(m & below);
      at += __popcll(m);
      n_comp += __popcll(m & comp[j]);
    }
    if (lane == x) { my_first = first; my_count = at - first; my_comp = n_comp; }
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (e[j] >= 0) sg.pair[pos[j]] = lane + 64 * j;
  if (lane < E) sg.offset[lane] = my_first;
  if (lane == 0) sg.offset[E] = P;
  if (out && threadIdx.x < 64) {
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (e[j] >= 0) { o.row_pair[pos[j]] = lane + 64 * j; o.pair_row[lane + 64 * j] = pos[j]; }
    if (lane < E) { o.counts[lane] = my_count; o.offsets[lane] = my_first; o.comp_counts[lane] = my_comp; }
    if (lane == 0) o.offsets[E] = P;
  }
  __builtin_amdgcn_wave_barrier();
}

}  // namespace lrc
