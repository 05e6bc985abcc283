// The shares of the decode launches' blocks (csrc/plan.h) for many row counts: consecutive, enough for every expert with rows,
// within the grid; the 32-bit quotients against 64-bit ones; and what W2 takes of the part sums of (h A2) against what the
// blocks of the fused projection leave, and against the room that is kept for them.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../paper_2512_17073_amd/csrc/internal.h"
#include "../paper_2512_17073_amd/csrc/plan.h"

using namespace lrc;

#define REQUIRE(cond, ...) do { if (!(cond)) { printf(__VA_ARGS__); printf("\n"); exit(1); } } while (0)

// blocks of every expert: the sums that the device takes over lanes, taken in order
static std::vector<std::pair<int, int>> shares(const PlanSpec& p, const std::vector<int>& cnt, int* used) {
  int n_active = 0, wsum = 0, over = 0;
  for (int c : cnt) { n_active += c > 0; wsum += (c + 31) / 32; }
  const int least = plan_least(p), total = plan_total(p, n_active), extra = total - n_active * least;
  REQUIRE(extra >= 0, "fewer blocks than the experts need");
  std::vector<int> claim, before;
  for (int c : cnt) {
    const int w = (c + 31) / 32;
    claim.push_back(plan_claim(total, w, wsum, c > 0 ? least : 0));
    const long long exact = wsum ? (long long)total * w / wsum - (c > 0 ? least : 0) : 0;
    REQUIRE(claim.back() == (exact > 0 ? exact : 0), "claim %d, in 64 bits %lld", claim.back(), exact);
    before.push_back(over);
    over += claim.back();
  }
  std::vector<std::pair<int, int>> out;
  int act = 0;
  for (size_t e = 0; e < cnt.size(); ++e) {
    const int lo = plan_part(extra, before[e], over), hi = plan_part(extra, before[e] + claim[e], over);
    REQUIRE(over == 0 || (lo == (long long)extra * before[e] / over && hi == (long long)extra * (before[e] + claim[e]) / over), "part of the rest");
    out.push_back(cnt[e] > 0 ? std::make_pair(act * least + lo, (act + 1) * least + hi) : std::make_pair(0, 0));
    act += cnt[e] > 0;
  }
  *used = n_active ? n_active * least + (over > 0 ? extra : 0) : 0;
  return out;
}

int main() {
  std::mt19937 rng(5);
  auto upto = [&](int n) { return int(rng() % unsigned(n)) + 1; };
  for (int round = 0; round < 20000; ++round) {
    const int E = round % 7 == 0 ? 256 : upto(64), k = upto(E < 16 ? E : 16), T = upto(round % 3 ? 64 : 128 * E / k > 0 ? 128 * E / k : 1);
    const int H = 64 * upto(round % 5 ? 64 : 256), F = 64 * upto(round % 5 ? 64 : 1024), kb = upto(kMaxKBlocks), n_cu = 256;
    // rows: every token picks k experts, from all of them or from a few
    const int few = std::max(k, round % 2 ? E : upto(E));
    std::vector<int> cnt(E, 0);
    for (int t = 0; t < T; ++t)
      for (int j = 0, e = int(rng() % unsigned(few)); j < k; ++j) ++cnt[(e + j) % few];
    const int P = T * k, NT13 = F / kTileN, NT2 = H / kTileN, target2 = (n_cu + kb - 1) / kb;
    const PlanSpec p13{plan_blocks(E, P, NT13, n_cu), NT13, n_cu, nullptr}, p2{plan_blocks(E, P, NT2, target2), NT2, target2, nullptr};
    for (const PlanSpec& p : {p13, p2}) {
      int used = 0, next = 0;
      const auto s = shares(p, cnt, &used);
      for (int e = 0; e < E; ++e) {
        if (!cnt[e]) continue;
        const int G = s[e].second - s[e].first;
        REQUIRE(s[e].first == next, "expert %d starts at block %d, not %d", e, s[e].first, next);
        REQUIRE(G >= plan_least(p) && (p.NT + G - 1) / G <= 32, "expert %d: %d blocks for %d n-tiles", e, G, p.NT);
        // (what W2's blocks of the expert add up is what as many fused blocks leave: every one with an n-tile, one each)
        int left = 0;
        for (int b = 0; b < G; ++b) {
          int t0, t1;
          dec::block_tiles(b, G, p.NT, t0, t1);
          if (t0 == t1) continue;
          REQUIRE(dec::ha_slot(b, t0, G, p.NT) < dec::ha_slots(G, p.NT), "block %d of %d", b, G);
          ++left;
        }
        REQUIRE(left == dec::ha_slots(G, p.NT), "%d parts left, %d taken", left, dec::ha_slots(G, p.NT));
        REQUIRE(dec::ha_slots(G, p.NT) <= dec::ha_slots(p.B, p.NT), "more parts than there is room for");
        next = s[e].second;
      }
      REQUIRE(used <= p.B && next == used, "%d blocks used of %d, %d dealt", used, p.B, next);
    }
  }
  return 0;
}
