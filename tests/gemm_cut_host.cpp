// The cut of the offline half's dense fp64 products (csrc/gemm_cut.h), over sizes from one chunk up: every chunk of the reduction
// in one part of its row block, the parts numbered from 0 without a gap, and no more of them than there is room for; small products
// in one block per CU at most, none of them with chunks of two row blocks, large ones in as many as the chip holds.
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

int main() {
  std::mt19937 rng(11);
  auto upto = [&](int n) { return int(rng() % unsigned(n)) + 1; };
  for (int round = 0; round < 20000; ++round) {
    const int M = upto(round % 4 ? 6000 : 140000), Nc = upto(round % 5 ? 96 : 1088), Kd = upto(round % 3 ? 9000 : 100);
    check_cut(M, Nc, Kd, 0);
    check_cut(std::min(Nc, 96), std::min(Nc, 96), Kd, kGramParts);
  }
  return 0;
}
