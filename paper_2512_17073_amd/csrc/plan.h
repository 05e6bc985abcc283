// Sharing a decode launch's blocks out among the experts that have rows.
//
// With a fixed number of blocks per expert, experts without rows leave CUs idle and experts with
// several 32-row passes finish last.  One wavefront (part of the launch that prepares the
// activations) writes, for every block of the later launch, which expert it serves: each expert with
// rows gets `base` blocks (enough for 32 n-tiles per block), the rest of `target` blocks go by
// weight (the number of 32-row passes the expert's rows need: every pass streams its weights
// again), dealt by the running sum of the weights.  Entry i of the table (PlanEntry, 32 bytes, read by block i with one scalar
// load): expert (or -1: the block exits), the block's n-tiles, first row and number of rows of the expert, and where the
// part sums of (h A2) go and how many there are.  What takes a division is done here, a lane per entry, and not by every wavefront
// of the launches that read the table.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "decode_index.h"
#include "wave.h"

namespace lrc {

struct PlanSpec { int B, NT, target; int32_t* plan; };     // B entries for a projection of NT n-tiles; plan == null: no table wanted
// own: the block's place among the part sums of its expert (ha_slot); slots: ha_slots of the expert's blocks in the other table
struct PlanEntry { int32_t e, t0, t1, r0, cnt, own, slots, pad; };
constexpr int kPlanEntryInts = 8;
LRC_HD PlanEntry plan_entry(int e, int b, int G, int NT, int r0, int cnt, int slots) {
  PlanEntry p{e, 0, 0, r0, cnt, 0, slots, 0};
  dec::block_tiles(b, G, NT, p.t0, p.t1);
  p.own = dec::ha_slot(b, p.t0, G, NT);
  return p;
}

// One table's shares: as many blocks as fill the chip (`target`), more only if the experts with rows need
// them; the rest of the grid exits at once.  Every expert gets its fewest blocks (a block owns at most
// 32 n-tiles) or its share by weight of all the blocks, whichever is more (the shares by weight are then
// scaled down to what is left): its blocks start where the fewest blocks of the experts before it and their part of
// the rest end.  (Also called on the host, for tests.)
LRC_HD int plan_least(const PlanSpec& p) { return (p.NT + 31) / 32; }
LRC_HD int plan_total(const PlanSpec& p, int n_active) {
  const int least = n_active * plan_least(p), want = p.target > least ? p.target : least;
  return p.B < want ? p.B : want;
}
// ... an expert's claim on the blocks beyond the fewest ...
LRC_HD int plan_claim(int total, int weight, int wsum, int least) {
  const int claim = int(uint32_t(total * weight) / uint32_t(wsum > 1 ? wsum : 1)) - least;
  return claim > 0 ? claim : 0;
}
// ... and what `claims` of all the `over` claims get of the `extra` blocks
LRC_HD int plan_part(int extra, int claims, int over) { return over > 0 ? int(uint32_t(extra * claims) / uint32_t(over)) : 0; }

// other: the spec of the table whose blocks leave part sums for this table's (null: none).
// The rest of the preparing launch is short, so this chain sets its length: the experts' rows are read once, 64
// experts to a register, and nothing is divided in 64 bits (blocks times passes: below 2^31 for any launch of
// this flavour, whose experts have 128 rows at most on average).
// offset(e): first row of expert e, of E that of all rows.
template <class Offset>
__device__ inline void make_plan(const Offset& offset, int E, const PlanSpec sp, const PlanSpec other, int lane) {
  if (sp.plan == nullptr) return;
  int32_t* __restrict__ plan = sp.plan;
  constexpr int kChunks = 4;                   // (at most 256 experts)
  const unsigned long long below = (1ull << lane) - 1ull;
  int cnt[kChunks], r0[kChunks], weight[kChunks];
  unsigned long long active[kChunks];
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    const int e = min(64 * i + lane, E - 1);
    r0[i] = cnt[i] = 0;
    if (64 * i >= E) continue;
    r0[i] = offset(e);
    cnt[i] = offset(e + 1);
  }
  int n_active = 0, wsum = 0;
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    cnt[i] = 64 * i + lane < E ? cnt[i] - r0[i] : 0;
    // what an expert's rows cost: every 32-row pass streams the expert's weights again
    weight[i] = (cnt[i] + 31) / 32;
    active[i] = __ballot(cnt[i] > 0);
    n_active += __popcll(active[i]);
    if (64 * i < E) wsum += lane_value(wave_scan(weight[i]), 63);
  }
  // One table's shares: blocks [lo, hi) of the experts of every chunk; returns the blocks used.
  auto shares = [&](const PlanSpec& p, int (&lo)[kChunks], int (&hi)[kChunks]) {
    const int base = plan_least(p), total = plan_total(p, n_active), extra = total - n_active * base;
    int claim[kChunks], incl[kChunks], over = 0, act = 0;    // claims on the blocks beyond the fewest, summed up to here
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      if (64 * i >= E) continue;
      claim[i] = plan_claim(total, weight[i], wsum, cnt[i] > 0 ? base : 0);
      incl[i] = over + wave_scan(claim[i]);
      over = lane_value(incl[i], 63);
    }
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      lo[i] = hi[i] = 0;
      if (64 * i >= E) continue;
      const int first = (act + __popcll(active[i] & below)) * base;
      if (cnt[i] > 0) {
        lo[i] = first + plan_part(extra, incl[i] - claim[i], over);
        hi[i] = first + base + plan_part(extra, incl[i], over);
      }
      act += __popcll(active[i]);
    }
    return n_active > 0 ? n_active * base + (over > 0 ? extra : 0) : 0;
  };
  const int B = sp.B;
  int lo[kChunks], hi[kChunks], olo[kChunks], ohi[kChunks], slots[kChunks] = {0, 0, 0, 0};
  const int used = shares(sp, lo, hi);
  if (other.plan != nullptr) {
    shares(other, olo, ohi);
#pragma unroll
    for (int i = 0; i < kChunks; ++i) slots[i] = dec::ha_slots(ohi[i] - olo[i], other.NT);
  }
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    if (64 * i >= E) continue;
    if (__popcll(active[i]) <= 8) {
      // few experts with many blocks each: the whole wavefront writes one expert's entries after the other's
      for (unsigned long long todo = active[i]; todo; todo &= todo - 1) {
        const int j = __ffsll(todo) - 1;
        const int lo_j = lane_value(lo[i], j), G_j = lane_value(hi[i], j) - lo_j, hi_j = min(lo_j + G_j, B);
        const int r0_j = lane_value(r0[i], j), cnt_j = lane_value(cnt[i], j), slots_j = lane_value(slots[i], j);
        for (int b = lo_j + lane; b < hi_j; b += 64)
          reinterpret_cast<PlanEntry*>(plan)[b] = plan_entry(64 * i + j, b - lo_j, G_j, sp.NT, r0_j, cnt_j, slots_j);
      }
    } else if (cnt[i] > 0) {
      // many experts with few blocks each: every lane writes its own expert's entries
      for (int b = lo[i]; b < hi[i] && b < B; ++b)
        reinterpret_cast<PlanEntry*>(plan)[b] = plan_entry(64 * i + lane, b - lo[i], hi[i] - lo[i], sp.NT, r0[i], cnt[i], slots[i]);
    }
  }
  for (int b = used + lane; b < B; b += 64) reinterpret_cast<PlanEntry*>(plan)[b] = PlanEntry{-1, 0, 0, 0, 0, 0, 0, 0};
}

// The grouped GEMM's work items: chunks of kChunkRows rows of one expert.  Item i of a launch reads entry i (expert, or -1: nothing
// to do; the expert's first row and number of rows; the chunk's first row within them) with one scalar load, instead of counting
// every expert's chunks in every block.  By expert, or (by_length) the whole chunks of all experts first, then the experts' last
// chunks, those with more row pairs (32 rows) before those with fewer, so that short blocks fill the end of a launch that is a few
// rounds of blocks.  W2 alone in this order, whole layer (us): Mixtral shape T = 700 660 -> 647, 1024 902 -> 843, 2048 1565 -> 1548, DeepSeek
// T = 512 and Qwen3 T = 4096 unchanged.  W1|W3 too: Qwen3 T = 1500 285 -> 278, 4096 553 -> 547; not where an expert's weights are
// far beyond the L2, which its last chunk then reads once more (Mixtral T = 700 647 -> 668, 2048 1498 -> 1513), nor below 64 rows
// an expert, whose chunks are nearly alike (DeepSeek T = 512 198 -> 202).
constexpr int kChunkRows = 128;
struct ChunkEntry { int32_t e, r0, cnt, r; };
constexpr int kChunkEntryInts = 4;
struct ChunkSpec { int items; bool by_length; int32_t* table; };       // table == null: none wanted
LRC_HD int chunk_count(int rows) { return (rows + kChunkRows - 1) / kChunkRows; }
LRC_HD int chunk_tail_pairs(int rows) { return (rows % kChunkRows + 31) / 32; }       // row pairs of the last, partly filled chunk (0: none)
// most items of a launch: every expert but the whole chunks' has at most one partly filled chunk; a multiple of 8 for the XCD order
LRC_HD int chunk_items(int total_rows, int n_exp) { return (total_rows / kChunkRows + n_exp + 7) / 8 * 8; }

template <class Offset>
__device__ inline void make_chunks(const Offset& offset, int E, const ChunkSpec sp, int lane) {
  if (sp.table == nullptr) return;
  ChunkEntry* table = reinterpret_cast<ChunkEntry*>(sp.table);
  constexpr int kChunks = 4;                   // (at most 256 experts)
  const unsigned long long below = (1ull << lane) - 1ull;
  int r0[kChunks], cnt[kChunks];
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    r0[i] = cnt[i] = 0;
    if (64 * i >= E) continue;
    const int e = min(64 * i + lane, E - 1);
    r0[i] = offset(e);
    cnt[i] = offset(e + 1);
  }
  int base = 0;
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    if (64 * i >= E) continue;
    cnt[i] = 64 * i + lane < E ? cnt[i] - r0[i] : 0;
    const int n = sp.by_length ? cnt[i] / kChunkRows : chunk_count(cnt[i]);
    const int incl = wave_scan(n), first = base + incl - n;
    for (int j = 0; j < n; ++j)
      if (first + j < sp.items) table[first + j] = ChunkEntry{64 * i + lane, r0[i], cnt[i], j * kChunkRows};
    base += lane_value(incl, 63);
  }
  if (sp.by_length)
    for (int rp = kChunkRows / 32; rp > 0; --rp)
#pragma unroll
      for (int i = 0; i < kChunks; ++i) {
        if (64 * i >= E) continue;
        const bool mine = chunk_tail_pairs(cnt[i]) == rp;
        const unsigned long long m = __ballot(mine);
        const int at = base + __popcll(m & below);
        if (mine && at < sp.items) table[at] = ChunkEntry{64 * i + lane, r0[i], cnt[i], cnt[i] / kChunkRows * kChunkRows};
        base += __popcll(m);
      }
  for (int i = base + lane; i < sp.items; i += 64) table[i] = ChunkEntry{-1, 0, 0, 0};
}

// The n-th pass of 32 rows beyond the experts' first ones, counted over the experts in order: its expert, and the pass within it (from 1).
template <class Offset>
__device__ inline bool further_pass(const Offset& offset, int E, int n, int lane, int& e, int& pass) {
  for (int g = 0, base = 0; g < E; g += 64) {
    const int x = min(g + lane, E - 1), cnt = g + lane < E ? offset(x + 1) - offset(x) : 0;
    const int more = max((cnt + 31) / 32 - 1, 0), incl = wave_scan(more), total = lane_value(incl, 63);
    if (n < base + total) {
      const int first = __ffsll(__ballot(base + incl > n)) - 1;
      e = g + first;
      pass = 1 + n - base - lane_value(incl - more, first);
      return true;
    }
    base += total;
  }
  return false;
}

// What the preparing launch makes for the FFN launches: per projection (W1|W3, W2) the one table its flavour reads.
struct FfnTables { PlanSpec plan[2]; ChunkSpec chunk[2]; };

}  // namespace lrc
