// How the offline half's dense fp64 products are cut into blocks, and the room that a factors call keeps for their parts.
#pragma once
#include <stddef.h>

#include <algorithm>

#include "layout.h"

namespace lrc {

constexpr int kGemmRows = 128, kGemmK = 32, kGemmBlocks = 512;       // rows of a block, of the reduction in a chunk, blocks that fill the chip

// How a product is cut (gemm_cut).  The blocks of a column group (ct tiles of 16 columns) share out the chunks of all row blocks in order,
// `per_block` each, whatever row block they belong to, so that every block has the same work: part z of row block y is that of the
// z-th block that has chunks of it (at most `parts`).  Or (shared == false) row blocks are cut alike, into `parts` of per_block chunks,
// the last one shorter.
struct GemmCut {
  int ct, gx, gy, chunks, parts, per_block;           // chunks: of one row block
  bool shared;
  LRC_HD int first_block(int y) const { return int((long long)y * chunks / per_block); }                       // shared: that has chunks of row block y
  LRC_HD int parts_of(int y) const { return shared ? first_block(y + 1) - first_block(y) + ((long long)(y + 1) * chunks % per_block != 0) : parts; }
  LRC_HD int part_of(int block, int y) const { return shared ? block - first_block(y) : block % parts; }
  // A block's chunks, counted over all row blocks: begin .. end - 1.
  LRC_HD long long begin(int block) const { return shared ? (long long)block * per_block : (long long)(block / parts) * chunks + block % parts * per_block; }
  LRC_HD long long end(int block) const {
    const long long last = shared ? (long long)gy * chunks : (long long)(block / parts + 1) * chunks, at = begin(block) + per_block;
    return at < last ? at : last;
  }
  LRC_HD int blocks() const { return shared ? int(((long long)gy * chunks + per_block - 1) / per_block) : gy * parts; }
};

// Small products take a block per CU at most, of whole chunks of one row block, row blocks cut alike: a second block on some of the
// CUs is as long as on all of them, and a block with chunks of two row blocks pays its start and its end twice.  (At least four
// chunks each where that leaves 128 blocks: fewer parts to add.)  All products of a call, cut for 512 blocks -> so, us: 4096 x 700 with
// 16 columns 168 -> 139, 768 x 2916 145 -> 120, 1500 x 3000 with 64 297 -> 242, 3008 x 739 with 24 190 -> 160, 16384 x 2048 368 -> 325,
// 2048 x 2944 with 40 238 -> 203, 512 x 768 the same; at the line, 8192 chunks (8192 x 4096 with 56 columns) 700 -> 692, 8000 (4096 x 8000
// with 40) 536 -> 543, with 16 338 -> 312; above, 11008 (4096 x 11008 with 24) 549 -> 629, 14336 with 40 840 -> 895.
// Larger ones take kGemmBlocks blocks of equal work, unless the row blocks by themselves are three quarters of these or all, or more
// than twice as many.  Whole call, cut -> not cut, us: 300 row blocks (38400 x 1024, 16 columns) 734 -> 761, 390 867 -> 858, 450
// 930 -> 906, 500 1005 -> 1002, 520 1014 -> 1075, 800 1361 -> 1425; with 40 columns (x 512) 300 1205 -> 1196, 390 1325 -> 1311, 450
// 1397 -> 1368, 520 1490 -> 1506, 700 1718 -> 1682.
// max_parts > 0 (a Gram matrix whose parts the factorisation adds up itself: at most kGramParts of them, all in flight at once
// there): row blocks cut alike, two chunks each at least.
constexpr int kGramParts = 32, kOneEachChunks = 8192, kCus = 256;
inline GemmCut gemm_cut(int M, int Nc, int Kd, int max_parts = 0) {
  GemmCut c;
  c.ct = std::min(4, (Nc + 15) / 16);
  c.gx = (Nc + 16 * c.ct - 1) / (16 * c.ct);
  c.gy = (M + kGemmRows - 1) / kGemmRows;
  c.chunks = (Kd + kGemmK - 1) / kGemmK;
  c.parts = 1;
  const long long all = (long long)c.gy * c.chunks, rows = (long long)c.gx * c.gy, blocks = std::max(1, kGemmBlocks / c.gx);
  const bool one_each = max_parts == 0 && rows <= kCus && all * c.gx <= kOneEachChunks;
  c.shared = max_parts == 0 && !one_each && (c.gy < blocks * 3 / 4 || (c.gy > blocks && c.gy < 2 * blocks));
  if (c.shared) {
    c.per_block = int((all + blocks - 1) / blocks);
    for (int y = 0; y < c.gy; ++y) c.parts = std::max(c.parts, c.parts_of(y));
    return c;
  }
  if (max_parts > 0) {
    c.parts = std::max(1, std::min(max_parts, Kd / 64));
  } else if (one_each) {
    const int least = int(std::max(2LL, std::min(4LL, all / 128)));
    c.parts = std::max(1, std::min(kCus / int(rows), c.chunks / least));
  }
  c.per_block = (c.chunks + c.parts - 1) / c.parts;
  c.parts = (c.chunks + c.per_block - 1) / c.per_block;
  return c;
}

// Room for a product's parts, in doubles: all but the first, which lies where the product will be; of a Gram matrix all of them.
inline size_t gemm_part_doubles(int M, int Nc, int Kd) { return size_t(gemm_cut(M, Nc, Kd).parts - 1) * M * Nc; }
inline size_t gram_part_doubles(int l, int Kd) { return size_t(gemm_cut(l, l, Kd, kGramParts).parts) * l * l; }

// What a factors call of a K x N matrix with l columns keeps beside its two panels, in doubles: N x l for Bm, or its orthonormalised copy, and
// (small: l columns fit one block's LDS) the parts of a Gram matrix behind it; the parts of all other products, which are done when
// that is written, lie in the same place.  (An allocation above 64 MB costs a call 280 us more than one below: with a place of their own for
// all parts 70000 x 512, rank 32, took 1800 us instead of 1520, 131072 x 256 2150 instead of 1810.)
inline size_t factors_room(int K, int N, int rank, int l, bool small) {
  const size_t panel = size_t(N) * l, gram = small ? std::max(gram_part_doubles(l, K), gram_part_doubles(l, N)) : gemm_part_doubles(l, l, K);
  return std::max({panel + (small ? gram : 0), gram, gemm_part_doubles(K, l, N), gemm_part_doubles(N, l, K), gemm_part_doubles(K, rank, l)});
}

}  // namespace lrc
