// The cut of the offline half's dense fp64 products (csrc/gemm_cut.h), over sizes from one chunk up: every chunk of the reduction
// in one part of its row block, the parts numbered from 0 without a gap, and no more of them than there is room for; small products
// in one block per CU at most, none of them with chunks of two row blocks, large ones in as many as the chip holds.  And the room
// that a factors call keeps: not above 64 MB where a place for every part of a cut of three blocks per CU is below.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_2512_17073_amd/csrc/gemm_cut.h"

using namespace lrc;

#define REQUIRE(cond, ...) do { if (!(cond)) { printf(__VA_ARGS__); printf("\n"); exit(1); } } while (0)

static void check_cut(int M, int Nc, int Kd, int max_parts) {
  const GemmCut c = gemm_cut(M, Nc, Kd, max_parts);
  REQUIRE(c.gy * kGemmRows >= M && c.chunks * kGemmK >= Kd && c.gx * 16 * c.ct >= Nc && c.per_block > 0 && c.parts > 0, "%d x %d x %d: not covered", M, Nc, Kd);
  REQUIRE(max_parts == 0 || (!c.shared && c.parts <= max_parts), "%d x %d x %d: %d parts of at most %d", M, Nc, Kd, c.parts, max_parts);
  const long long chunks = (long long)c.gx * c.gy * c.chunks;
  if (max_parts == 0 && chunks <= 8192 && c.gx * c.gy <= 256) REQUIRE(!c.shared && c.gx * c.blocks() <= 256, "%d x %d x %d: %d blocks", M, Nc, Kd, c.gx * c.blocks());
  if (max_parts == 0 && chunks > 8192 && c.gx * c.gy < 330) REQUIRE(c.gx * c.blocks() > 400 && c.gx * c.blocks() <= 512 + c.gx, "%d x %d x %d: %d blocks", M, Nc, Kd, c.gx * c.blocks());
  std::vector<int> next_chunk(c.gy, 0), next_part(c.gy, 0);
  for (int b = 0; b < c.blocks(); ++b) {
    const long long hi = c.end(b);
    REQUIRE(c.begin(b) < hi, "%d x %d x %d: block %d of %d has nothing to do", M, Nc, Kd, b, c.blocks());
    for (long long at = c.begin(b); at < hi;) {
      const int y = int(at / c.chunks), first = int(at - (long long)y * c.chunks), last = int(std::min<long long>(c.chunks, first + (hi - at)));
      REQUIRE(y < c.gy && first == next_chunk[y] && last > first, "%d x %d x %d: block %d takes chunks %d..%d of row block %d, %d is next", M, Nc, Kd, b, first, last, y, next_chunk[y]);
      REQUIRE(c.part_of(b, y) == next_part[y] && next_part[y] < c.parts, "%d x %d x %d: part %d of row block %d, %d is next of %d", M, Nc, Kd, c.part_of(b, y), y, next_part[y], c.parts);
      next_chunk[y] = last;
      ++next_part[y];
      at += last - first;
    }
  }
  for (int y = 0; y < c.gy; ++y)
    REQUIRE(next_chunk[y] == c.chunks && next_part[y] == c.parts_of(y), "%d x %d x %d: row block %d ends at chunk %d of %d, part %d of %d", M, Nc, Kd, y, next_chunk[y], c.chunks, next_part[y], c.parts_of(y));
}

// ... three blocks per CU, row blocks alike, a place for every part
static size_t all_parts(int M, int Nc, int Kd) {
  const int ct = std::min(4, (Nc + 15) / 16), gx = (Nc + 16 * ct - 1) / (16 * ct), gy = (M + 127) / 128;
  const int parts = std::max(1, std::min({std::max(1, 768 / (gx * gy)), 512, Kd / 64}));
  const int k_per = ((Kd + parts - 1) / parts + 31) / 32 * 32;
  return size_t((Kd + k_per - 1) / k_per) * M * Nc;
}

int main() {
  std::mt19937 rng(11);
  auto upto = [&](int n) { return int(rng() % unsigned(n)) + 1; };
  for (int round = 0; round < 20000; ++round) {
    const int M = upto(round % 4 ? 6000 : 140000), Nc = upto(round % 5 ? 96 : 1088), Kd = upto(round % 3 ? 9000 : 100);
    check_cut(M, Nc, Kd, 0);
    check_cut(std::min(Nc, 96), std::min(Nc, 96), Kd, kGramParts);
  }
  const int sizes[] = {300, 512, 700, 1024, 1408, 2048, 2944, 4096, 6000, 8192, 11008, 14336, 20000, 28672, 40000, 50000, 57344, 70000, 98304, 110000, 131072};
  int below = 0;
  for (int K : sizes)
    for (int N : sizes)
      for (int r : {1, 8, 16, 24, 32, 48, 64, 88, 128, 256}) {
        const int l = r + 8;
        if (l > std::min(K, N) || (long long)K * N > 1500000000LL) continue;
        const size_t was = size_t(K) * l + 2 * size_t(N) * l + std::max({all_parts(K, l, N), all_parts(N, l, K), all_parts(l, l, K), all_parts(l, l, N), all_parts(K, r, l)});
        const size_t is = size_t(K) * l + size_t(N) * l + factors_room(K, N, r, l, l <= 96);
        if (was * 8 > size_t(64) << 20) continue;
        ++below;
        REQUIRE(is * 8 <= size_t(64) << 20, "%d x %d, rank %d: %.1f MB, %.1f before", K, N, r, is / 131072.0, was / 131072.0);
      }
  REQUIRE(below > 500, "%d shapes", below);
  return 0;
}
