// Sharing a decode launch's blocks out among the experts that have rows.
//
// With a fixed number of blocks per expert, experts without rows leave CUs idle and experts with
// several 32-row passes finish last.  One wavefront (part of the launch that prepares the
// activations) writes, for every block of the later launch, which expert it serves: each expert with
// rows gets `base` blocks (enough for 32 n-tiles per block), the rest of `target` blocks go by
// weight (the number of 32-row passes the expert's rows need: every pass streams its weights
// again), dealt by the running sum of the weights.  Entry i of the table (PlanEntry, 32 bytes, read by block i with one scalar
// load): expert (or -1: the block exits), index of the block within the expert, blocks of the expert,
// first row and number of rows of the expert.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lrc {

struct PlanSpec { int B, NT, target; int32_t* plan; };     // B entries for a projection of NT n-tiles; plan == null: no table wanted
struct PlanEntry { int32_t e, b, G, r0, cnt, slots, pad0, pad1; };     // slots: ha_slots of the expert's blocks in the other table
constexpr int kPlanEntryInts = 8;

// other: the spec of the table whose blocks leave part sums for this table's (null: none)
__device__ inline void make_plan(const int32_t* __restrict__ offsets, int E, const PlanSpec sp, const PlanSpec other, int lane) {
  if (sp.plan == nullptr) return;
  int32_t* __restrict__ plan = sp.plan;
  // what an expert's rows cost: every 32-row pass streams the expert's weights again
  auto weight = [](int cnt) { return (cnt + 31) / 32; };
  auto scan = [&](int v) {
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt *= 2) {
      const int t = __shfl_up(v, dlt);
      if (lane >= dlt) v += t;
    }
    return v;
  };
  auto rows_of = [&](int e) { return e < E ? offsets[e + 1] - offsets[e] : 0; };
  int n_active = 0, wsum = 0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int cnt = rows_of(e0 + lane);
    n_active += __popcll(__ballot(cnt > 0));
    wsum += __shfl(scan(weight(cnt)), 63);
  }
  // One table's shares: as many blocks as fill the chip (`target`), more only if the experts with rows need
  // them; the rest of the grid exits at once.  Every expert gets its fewest blocks (a block owns at most
  // 32 n-tiles) or its share by weight of all the blocks, whichever is more (the shares by weight are then
  // scaled down to what is left).
  struct Shares {
    int base, total, over, w_before, act_before;
    long long extra;
  };
  auto want_of = [&](const Shares& h, int cnt) {     // an expert's claim on the blocks beyond the fewest
    const int want = wsum > 0 ? int((long long)h.total * weight(cnt) / wsum) : 0;
    return max(0, want - (cnt > 0 ? h.base : 0));
  };
  auto shares = [&](const PlanSpec& p) {
    Shares h{};
    h.base = (p.NT + 31) / 32;
    h.total = min(p.B, max(p.target, n_active * h.base));
    h.extra = h.total - n_active * h.base;
    for (int e0 = 0; e0 < E; e0 += 64) h.over += __shfl(scan(want_of(h, rows_of(e0 + lane))), 63);
    return h;
  };
  // the blocks [lo, hi) of this lane's expert, 64 experts at a time
  auto step = [&](Shares& h, int cnt, int& lo, int& hi) {
    const int act = cnt > 0 ? 1 : 0, ai = scan(act), w = want_of(h, cnt), wi = scan(w);
    lo = hi = 0;
    if (act) {
      lo = (h.act_before + ai - 1) * h.base + (h.over > 0 ? int(h.extra * (h.w_before + wi - w) / h.over) : 0);
      hi = (h.act_before + ai) * h.base + (h.over > 0 ? int(h.extra * (h.w_before + wi) / h.over) : 0);
    }
    h.act_before += __shfl(ai, 63); h.w_before += __shfl(wi, 63);
  };
  const int B = sp.B;
  Shares mine = shares(sp), theirs{};
  if (other.plan != nullptr) theirs = shares(other);
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int e = e0 + lane, cnt = rows_of(e), r0 = e < E ? offsets[e] : 0;
    int lo, hi, olo = 0, ohi = 0;
    step(mine, cnt, lo, hi);
    if (other.plan != nullptr) step(theirs, cnt, olo, ohi);
    const int slots = min(ohi - olo, other.NT);
    const unsigned long long with_rows = __ballot(cnt > 0);
    if (__popcll(with_rows) <= 8) {
      // few experts with many blocks each: the whole wavefront writes one expert's entries after the other's
      for (unsigned long long todo = with_rows; todo; todo &= todo - 1) {
        const int j = __ffsll(todo) - 1;
        const int lo_j = __shfl(lo, j), G_j = __shfl(hi, j) - lo_j, hi_j = min(lo_j + G_j, B);
        const int r0_j = __shfl(r0, j), cnt_j = __shfl(cnt, j), slots_j = __shfl(slots, j);
        for (int i = lo_j + lane; i < hi_j; i += 64)
          reinterpret_cast<PlanEntry*>(plan)[i] = PlanEntry{e0 + j, i - lo_j, G_j, r0_j, cnt_j, slots_j, 0, 0};
      }
    } else if (cnt > 0) {
      // many experts with few blocks each: every lane writes its own expert's entries
      for (int i = lo; i < hi && i < B; ++i) reinterpret_cast<PlanEntry*>(plan)[i] = PlanEntry{e, i - lo, hi - lo, r0, cnt, slots, 0, 0};
    }
  }
  const int used = n_active > 0 ? n_active * mine.base + (mine.over > 0 ? int(mine.extra) : 0) : 0;
  for (int i = used + lane; i < B; i += 64) reinterpret_cast<PlanEntry*>(plan)[i] = PlanEntry{-1, 0, 1, 0, 0, 0, 0, 0};
}

}  // namespace lrc
