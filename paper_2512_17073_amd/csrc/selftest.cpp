// Host-only self-check of the decode-flavour FFN kernels' index arithmetic (no device needed).
// The kernels form every buffer offset and LDS address through the functions of decode_index.h;
// this file walks the same functions for every block, wavefront, lane and step of a launch and
// checks each result against the size of what it addresses, and that the blocks and wavefronts
// together read every packed tile of the expert exactly once per pass.
#include <cstdio>
#include <string>
#include <vector>

#include <cmath>
#include <cstring>

#include "decode_index.h"
#include "factor_q3.h"
#include "ffn_common.h"
#include "internal.h"
#include "pack.h"

namespace lrc {

namespace {

using namespace dec;

struct Shape {
  int K, N, bits, group, ls_max, LSm[2], r0, cnt, total_rows, G, kblocks;
  bool dual;
};

#define SELF_FAIL(...)                                 \
  do {                                                 \
    char buf_[512];                                    \
    std::snprintf(buf_, sizeof buf_, __VA_ARGS__);     \
    return std::string(buf_);                          \
  } while (0)

// "" if every index of one launch shape is in range, else the first violation
std::string check_shape(const Shape& sh) {
  const int Kp = padded_k(sh.K), KS = Kp / kTileK, NT = sh.N / kTileN, Gr = Kp / sh.group;
  int gs = 0;
  while ((1 << gs) < sh.group) ++gs;
  const uint32_t code_bytes = uint32_t(KS) * NT * (kWave * 2 * sh.bits * 4), meta_bytes = uint32_t(Gr) * NT * kTileN * 4;
  const int rt = sh.total_rows + kActPadRows;                       // rows of the operand-order activation buffers
  const size_t in_units = size_t(rt) * Kp / 8;
  const int kb_steps = (KS + sh.kblocks - 1) / sh.kblocks;
  const int MT = sh.cnt <= 16 ? 1 : 2, NP = sh.dual ? 2 : 1;
  const int pitch = NP * sh.ls_max * 32;
  for (int kb = 0; kb < sh.kblocks; ++kb) {
    const int ks_lo = kb * kb_steps, KSl = std::min(KS, ks_lo + kb_steps) - ks_lo;
    if (KSl <= 0) SELF_FAIL("K-block %d of %d has no k-step", kb, sh.kblocks);
    const bool lowrank = sh.LSm[0] > 0 || sh.LSm[1] > 0;
    const int LS = lowrank ? std::max(sh.LSm[0], sh.LSm[1]) : 0;
    std::vector<int> seen(size_t(KSl) * NT * 2, 0), seen_lr(size_t(std::max(LS, 1)) * NT * 2, 0);
    for (int b = 0; b < sh.G; ++b) {
      int t0, t1;
      block_tiles(b, sh.G, NT, t0, t1);
      const int nt_b = t1 - t0;
      if (nt_b == 0) continue;
      if (nt_b > max_block_tiles(MT)) SELF_FAIL("block %d of %d owns %d n-tiles (at most %d)", b, sh.G, nt_b, max_block_tiles(MT));
      const int units = block_units(nt_b, sh.dual), kwl = waves_per_unit_log2(units), kw = 1 << kwl, groups = kWaves / kw;
      if ((kw > 1 && units * kw > kWaves) || (kw < kWaves && units * kw * 2 <= kWaves))
        SELF_FAIL("%d wavefronts per unit for %d units", kw, units);
      if (units > groups * unit_slots(sh.dual, MT)) SELF_FAIL("%d units do not fit %d wavefront groups", units, groups);
      const StepPlan sp = step_plan(KSl, MT);
      const int p_frags = NP * LS * MT;
      const bool p_late = p_frags * 64 > kSpareUnits;
      if (p_frags * 64 > (p_late ? kLdsUnits : kSpareUnits)) SELF_FAIL("%d (in A) fragments exceed their LDS region", p_frags);
      if (kw > 1 && ((kWaves * MT) * kStreams) * 64 > kLdsUnits) SELF_FAIL("reduction buffer exceeds LDS");
      for (int r = 0; r < sh.cnt; r += 16 * MT) {
        // staging: LDS units and global units
        for (int ph = 0; ph < sp.n_ph; ++ph) {
          const int nk = std::min(sp.KP, KSl - ph * sp.KP);
          for (int wave = 0; wave < kWaves; ++wave)
            for (int mt = 0; mt < MT; ++mt)
              for (int kl = wave >> 3; kl < nk; kl += 2)
                for (int lane = 0; lane < 64; ++lane) {
                  const int q = lane >> 4, rowl = lane & 15, s = wave & 7;
                  const int ks = ks_lo + ph * sp.KP + kl, k8 = ks * 32 + staged_group(ks, q, sh.K) * 8 + s;
                  if (k8 >= sh.K / 8) SELF_FAIL("staging reads unit %d of a row of %d", k8, sh.K / 8);
                  if (ks * 32 + q * 8 + s < sh.K / 8 && k8 != ks * 32 + q * 8 + s) SELF_FAIL("staging of k-step %d, group %d reads unit %d", ks, q, k8);
                  if (act_frag_unit(mt, kl, s, sp.KP) + 64 > kLdsUnits) SELF_FAIL("staged fragment (mt %d, kl %d, s %d) leaves LDS", mt, kl, s);
                  const int row = staged_row(sh.r0 + r, r, mt, rowl, sh.cnt, rt);
                  if (row < 0 || row >= rt) SELF_FAIL("staging reads row %d of %d", row, rt);
                  if (r + 16 * mt + rowl < sh.cnt ? row != sh.r0 + r + 16 * mt + rowl : row < sh.total_rows + kActPadRows - kZeroRows)
                    SELF_FAIL("staging reads row %d for row %d of an expert with %d rows at %d", row, r + 16 * mt + rowl, sh.cnt, sh.r0);
                  const size_t u = ffn::act_unit(k8, row, rt);
                  if (u >= in_units) SELF_FAIL("staging reads unit %zu of %zu (row %d of %d)", u, in_units, row, rt);
                }
        }
        // (in A) fragments
        for (int f = 0; f < p_frags; ++f) {
          const int mt = f % MT, g = f / MT, st = g % LS, m = g / LS;
          if (p_frag_unit(m, st, mt, LS, MT) + 64 > (p_late ? kLdsUnits : kSpareUnits)) SELF_FAIL("(in A) fragment %d leaves its LDS region", f);
          for (int lane = 0; lane < 64; ++lane) {
            const int q = lane >> 4, c = lane & 15;
            const int row = sh.r0 + std::min(r + 16 * mt + c, sh.cnt - 1);
            const size_t h = size_t(row) * pitch + m * sh.ls_max * 32 + 32 * st + 8 * q;
            if (h + 8 > size_t(sh.total_rows) * pitch) SELF_FAIL("(in A) copy reads half %zu of %zu", h, size_t(sh.total_rows) * pitch);
          }
        }
        // the steps of every wavefront (the kernel fetches RING steps past the last one)
        if (r > 0) continue;                  // (the steps do not depend on the pass)
        for (int wave = 0; wave < kWaves; ++wave) {
          const int grp = wave / kw, kwi = wave % kw, own = own_units(grp, groups, units, sh.dual);
          const int gps = kTileK >> gs, tb = kWave * 2 * sh.bits * 4;
          const Strides strides = walk_strides(kwl, sh.bits, NT, gps);
          for (int ph = 0; ph < sp.n_ph; ++ph)
            for (int ts = 0; ts < own; ++ts) {
              const int unit = grp + ts * groups, first = ks_lo + ph * sp.KP, len = phase_steps(sp, ph, KSl), tile0 = stream_tile(t0, unit, 0, sh.dual);
              if (unit >= units || len <= 0 || len > sp.KP) SELF_FAIL("segment of unit %d of %d, %d steps", unit, units, len);
              Walk at = walk_start(first, len, tile0, kwi, kwl, sh.bits, NT, gps, strides);
              // (the kernel fetches a turn of the ring past the last own step: the last one again)
              for (int k = 0; k < at.n + 2 * kRing; ++k, walk_on(at, strides)) {
                const int st = std::min(at.n > 0 ? (std::min(k, at.n - 1) << kwl) + kwi : len - 1, len - 1), ks = first + st;
                if (k < at.n && (k << kwl) + kwi >= len) SELF_FAIL("own step %d of a segment of %d", k, len);
                for (int m = 0; m < kStreams; ++m) {
                  const int tile = stream_tile(t0, unit, m, sh.dual), next_tile = sh.dual ? 0 : m;
                  const bool ok = tile < t1;
                  const uint32_t code = at.code + next_tile * tb, meta = at.meta + next_tile * (kTileN * 4);
                  if (ok && k < at.n) ++seen[(size_t(ks - ks_lo) * NT + tile) * 2 + (sh.dual ? m : 0)];
                  for (int lane = 0; lane < 64; ++lane) {
                    const LaneOffsets o = lane_offsets(lane, sh.bits, NT, gs, ok);
                    const uint32_t q = lane >> 4, c = lane & 15, w1 = sh.bits == 3 ? 8 : 16;
                    if (!ok) {
                      if (o.code0 < kNoTile || o.code1 < kNoTile || o.meta < kNoTile || code_bytes > kNoTile || meta_bytes > kNoTile) SELF_FAIL("a stream without a tile reads inside its resource");
                      if (((uint64_t(o.code1) + code + 16) >> 32) != 0 || ((uint64_t(o.meta) + meta + 4) >> 32) != 0) SELF_FAIL("an offset past every resource wraps round");
                      continue;
                    }
                    if (code + o.code0 != (uint32_t(ks) * NT + tile) * tb + lane * 16) SELF_FAIL("code offset does not address tile (%d, %d)", ks, tile);
                    if (code + o.code0 + 16 > code_bytes) SELF_FAIL("code load at %u + 16 > %u", code + o.code0, code_bytes);
                    if (sh.bits > 2 && code + o.code1 + w1 > (uint32_t(ks) * NT + tile + 1) * tb) SELF_FAIL("second code load at %u leaves tile (%d, %d)", code + o.code1, ks, tile);
                    if (meta + o.meta != ((uint32_t(ks) * gps + ((q * kLaneK) >> gs)) * NT + tile) * (kTileN * 4) + c * 4 || meta + o.meta + 4 > meta_bytes)
                      SELF_FAIL("metadata load at %u of %u", meta + o.meta, meta_bytes);
                  }
                }
              }
            }
          // rank steps, by turns of the ring (the first turn is fetched whether it holds a step or not)
          const int turns = own > 0 ? rank_turns(sh.dual, LS, kwi, kwl) : 0;
          for (int t = 0; t < std::max(turns, 1); ++t)
            for (int i = 0; i < kRing; ++i)
              for (int m = 0; m < kStreams; ++m) {
                const int ts = rank_slot_unit(sh.dual, i), st = rank_slot_step(sh.dual, t, i, kwi, kwl);
                const int tile = stream_tile(t0, grp + ts * groups, m, sh.dual), LSq = lowrank ? sh.LSm[sh.dual ? m : 0] : 0;
                const bool ok = ts < own && tile < t1;
                const uint32_t bf_size = uint32_t(NT) * LSq * 1024, bm_size = uint32_t(NT / 4) * LSq * 128, bc_size = uint32_t(NT) * LSq * 256;
                if (ok && st < LSq) ++seen_lr[(size_t(st) * NT + tile) * 2 + (sh.dual ? m : 0)];
                for (int lane = 0; lane < 64; ++lane) {
                  const uint32_t q = lane >> 4, c = lane & 15;
                  const RankOffsets o = rank_offsets(st, tile, ok, lane, NT, false), oq = rank_offsets(st, tile, ok, lane, NT, true);
                  if (ok && st < LSq) {
                    if (o.bf != (uint32_t(st) * NT + tile) * 1024 + lane * 16 || o.bf + 16 > bf_size) SELF_FAIL("rank step %d reads the B factor at %u of %u", st, o.bf, bf_size);
                    if (oq.bf != ((uint32_t(st) * (NT / 4) + tile / 4) * 4 + q) * 32 + (c & 1) * 16 || oq.bf + 16 > bm_size)
                      SELF_FAIL("rank step %d: metadata of a 3-bit unit at %u of %u", st, oq.bf, bm_size);
                    if (oq.bc != (uint32_t(st) * NT + tile) * 256 + lane * 4 || oq.bc + 4 > bc_size) SELF_FAIL("rank step %d: codes of a 3-bit unit at %u of %u", st, oq.bc, bc_size);
                  } else if (o.bf < bf_size || oq.bf < bm_size || oq.bc < bc_size) {
                    SELF_FAIL("rank step %d of stream %d reads inside a resource it should not", st, m);
                  }
                }
              }
        }
      }
    }
    // every packed tile of the K-block exactly once (both streams of a dual launch)
    for (int ks = 0; ks < KSl; ++ks)
      for (int t = 0; t < NT; ++t)
        for (int m = 0; m < (sh.dual ? 2 : 1); ++m)
          if (seen[(size_t(ks) * NT + t) * 2 + m] != 1)
            SELF_FAIL("K-block %d: tile (k-step %d, n-tile %d, stream %d) read %d times", kb, ks, t, m, seen[(size_t(ks) * NT + t) * 2 + m]);
    for (int st = 0; st < LS; ++st)
      for (int t = 0; t < NT; ++t)
        for (int m = 0; m < (sh.dual ? 2 : 1); ++m) {
          const int want = st < sh.LSm[sh.dual ? m : 0] ? 1 : 0;
          if (seen_lr[(size_t(st) * NT + t) * 2 + m] != want)
            SELF_FAIL("rank step %d n-tile %d stream %d read %d times (want %d)", st, t, m, seen_lr[(size_t(st) * NT + t) * 2 + m], want);
        }
  }
  return "";
}

// (h A2) made by the fused launch: every block's operand reads, its copy of them in LDS, and the part sums it
// leaves for the K-blocks of W2
std::string check_h_a2(int F, int rank2, const Shape& sh, int kblocks) {
  const int NT = F / kTileN, ht = (rank2 + 15) / 16, slots = ha_slots(sh.G, NT);
  std::vector<int> left(slots, 0), taken(slots, 0);
  for (int b = 0; b < sh.G; ++b) {
    int t0, t1;
    block_tiles(b, sh.G, NT, t0, t1);
    if (t0 == t1) continue;
    const int slot = ha_slot(b, t0, sh.G, NT);
    if (slot < 0 || slot >= slots) SELF_FAIL("block %d of %d leaves its sums in place %d of %d", b, sh.G, slot, slots);
    ++left[slot];
    if (ha_part(slot, sh.total_rows, sh.r0 + sh.cnt - 1, 16 * ht - 4) + 4 > size_t(slots) * sh.total_rows * kHaRank)
      SELF_FAIL("block %d stores past its part sums", b);
    const int u0 = t0 / 2, n_u = (t1 - 1) / 2 - u0 + 1, g0 = t0 / 4, n_q = ((t1 - 1) / 4 - g0) / 4 + 1;
    for (int rt = 0; rt < ht; ++rt)
      for (int tile = t0; tile < t1; ++tile) {
        if ((tile / 4 - g0) / 4 >= n_q) SELF_FAIL("n-tile %d: its metadata is not among the copied groups", tile);
        for (int lane = 0; lane < 64; ++lane) {
          const uint32_t at = ha_operand(rt, tile, lane, F);
          // (packed: [factor tile][unit of 32 inputs][lane][8 inputs])
          const int q = lane >> 4, c = lane & 15, unit = at / (2 * kWave), l = at / 2 % kWave, f = 32 * (unit - rt * (F / 32)) + 8 * (l >> 4) + 4 * (at & 1);
          if (unit / (F / 32) != rt || (l & 15) != c || f != 16 * tile + 4 * q) SELF_FAIL("operand of n-tile %d, lane %d reads input %d", tile, lane, f);
          const uint32_t own = at - (rt * (F / 32 - n_u) + u0) * (kWave * 2);
          if (own / (2 * kWave) != uint32_t(rt * n_u + tile / 2 - u0) || own >= uint32_t(n_u * ht * kWave * 2)) SELF_FAIL("operand of n-tile %d, lane %d: outside its copy", tile, lane);
        }
      }
  }
  for (int kb = 0; kb < kblocks; ++kb) {
    int lo, hi;
    ha_share(kb, kblocks, slots, lo, hi);
    for (int s = lo; s < hi; ++s) ++taken[s];
  }
  for (int s = 0; s < slots; ++s)
    if (left[s] != 1 || taken[s] != 1) SELF_FAIL("part sum %d of %d left %d and taken %d times", s, slots, left[s], taken[s]);
  return "";
}

}  // namespace

}  // namespace lrc

using namespace lrc;

extern "C" int moe_lrc_selftest_decode_index(int hidden, int ffn, int bits, int group, int layer_rank, int rank1,
                                             int rank3, int rank2, int first_row, int rows, int total_rows,
                                             int blocks_w13, int blocks_w2, int kblocks_w2) {
  if (hidden <= 0 || ffn <= 0 || hidden % 64 || ffn % 64 || bits < 2 || bits > 4 ||
      (group != 64 && group != 128 && group != 256) || layer_rank < 0 || layer_rank > 1024 || rank1 < 0 ||
      rank3 < 0 || rank2 < 0 || rank1 > layer_rank || rank3 > layer_rank || rank2 > layer_rank || rows < 1 ||
      first_row < 0 || first_row + rows > total_rows || blocks_w13 < 1 || blocks_w2 < 1 || kblocks_w2 < 1 ||
      kblocks_w2 > kMaxKBlocks)
    return set_error(MOE_LRC_EINVAL, "selftest_decode_index: argument out of range");
  const int ls = (layer_rank + 31) / 32;
  Shape a{hidden, ffn, bits, group, ls, {(rank1 + 31) / 32, (rank3 + 31) / 32}, first_row, rows, total_rows, blocks_w13, 1, true};
  std::string err = check_shape(a);
  if (!err.empty()) return set_error(MOE_LRC_ESHAPE, "selftest_decode_index (W1|W3): " + err);
  Shape b{ffn, hidden, bits, group, ls, {(rank2 + 31) / 32, (rank2 + 31) / 32}, first_row, rows, total_rows, blocks_w2, kblocks_w2, false};
  err = check_shape(b);
  if (!err.empty()) return set_error(MOE_LRC_ESHAPE, "selftest_decode_index (W2): " + err);
  if (rank2 > 0 && layer_rank <= kHaRank) err = check_h_a2(ffn, rank2, a, kblocks_w2);
  if (!err.empty()) return set_error(MOE_LRC_ESHAPE, "selftest_decode_index (h A2): " + err);
  return MOE_LRC_OK;
}

namespace {
// one half of a packed fp16 FMA as the device computes it: exact product and sum, one rounding
float half_fma(uint16_t f, uint16_t s, uint16_t c) {
  auto h = [](uint16_t b) { _Float16 v; std::memcpy(&v, &b, 2); return (double)v; };
  return (float)(_Float16)std::fma(h(f), h(s), h(c));
}
uint32_t q3_field_rt(uint32_t v, int i) {
  return i == 0 ? ffn::q3_field<0>(v) : i == 1 ? ffn::q3_field<1>(v) : i == 2 ? ffn::q3_field<2>(v) : ffn::q3_field<3>(v);
}
}  // namespace

extern "C" int moe_lrc_selftest_factor_pair(int K, int N, int rank, const uint8_t* a_codes, const uint16_t* a_scale,
                                          const uint16_t* a_zero, const uint8_t* b_codes, const uint16_t* b_scale,
                                          const uint16_t* b_zero, float* A_out, float* B_out) {
  if (!a_codes || !a_scale || !a_zero || !b_codes || !b_scale || !b_zero || !A_out || !B_out)
    return set_error(MOE_LRC_EINVAL, "selftest_factor_pair: null argument");
  if (K <= 0 || N <= 0 || K % 64 || N % 64 || rank <= 0 || rank > 1024 || rank % 8)
    return set_error(MOE_LRC_ESHAPE, "selftest_factor_pair: K and N must be multiples of 64, rank a multiple of 8 in 8..1024");
  std::vector<uint8_t> abuf(q3_a_bytes(K, rank)), bbuf(q3_b_bytes(N, rank));
  const float mu_a = pack_factor_a_q3(K, rank, a_codes, a_scale, a_zero, abuf.data());
  const float mu_b = pack_factor_b_q3(N, rank, b_codes, b_scale, b_zero, bbuf.data());
  if (mu_a == 0.f || mu_b == 0.f) return set_error(MOE_LRC_EINVAL, "selftest_factor_pair: code out of range (3 bits)");
  // A: the reads of the (in A) kernels: unit (tile, kk), lane (q, c); codes dword, metadata dword of (tile, kk / 2, c)
  const int k32 = K / 32, g64 = K / 64, NT = N / 16, NG = N / 64;
  const uint32_t* acw = reinterpret_cast<const uint32_t*>(abuf.data());
  const uint32_t* amw = reinterpret_cast<const uint32_t*>(abuf.data() + q3_a_codes_bytes(K, rank));
  for (int tile = 0; tile < (rank + 15) / 16; ++tile)
    for (int kk = 0; kk < k32; ++kk)
      for (int lane = 0; lane < 64; ++lane) {
        const int q = lane >> 4, c = lane & 15, rho = 16 * tile + c;
        const uint32_t codes = acw[(size_t(tile) * k32 + kk) * 64 + lane], meta = amw[(size_t(tile) * g64 + (kk >> 1)) * 16 + c];
        for (int j = 0; j < 8; ++j) {
          const uint32_t f = q3_field_rt(codes, j >> 1);
          const float v = half_fma(uint16_t(j & 1 ? f >> 16 : f), uint16_t(meta), uint16_t(meta >> 16)) / mu_a;
          if (rho < rank) A_out[size_t(32 * kk + 8 * q + j) * rank + rho] = v;
          else if (v != 0.f) return set_error(MOE_LRC_ESHAPE, "selftest_factor_pair: a column of A past the rank is not zero");
        }
      }
  // B: the reads of the FFN kernels' rank steps: unit (st, nt), lane (q, c); codes dword, 32 bytes of
  // metadata of (st, nt / 4, q): eight scale halves, then eight offset halves
  const uint32_t* bcw = reinterpret_cast<const uint32_t*>(bbuf.data());
  const uint16_t* bmh = reinterpret_cast<const uint16_t*>(bbuf.data() + q3_b_codes_bytes(N, rank));
  for (int st = 0; st < (rank + 31) / 32; ++st)
    for (int nt = 0; nt < NT; ++nt)
      for (int lane = 0; lane < 64; ++lane) {
        const int q = lane >> 4, c = lane & 15;
        const uint32_t codes = bcw[(size_t(st) * NT + nt) * 64 + lane];
        const uint16_t* mh = bmh + ((size_t(st) * NG + nt / 4) * 4 + q) * 16;
        for (int j = 0; j < 8; ++j) {
          const uint32_t f = q3_field_rt(codes, j >> 1);
          const float v = half_fma(uint16_t(j & 1 ? f >> 16 : f), mh[j], mh[8 + j]) / mu_b;
          const int rho = 32 * st + 8 * q + j;
          if (rho < rank) B_out[size_t(rho) * N + nt * 16 + c] = v;
          else if (v != 0.f) return set_error(MOE_LRC_ESHAPE, "selftest_factor_pair: a row of B past the rank is not zero");
        }
      }
  return MOE_LRC_OK;
}
