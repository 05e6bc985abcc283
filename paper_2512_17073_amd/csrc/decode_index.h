// Index arithmetic of the decode-flavour FFN kernels (ffn_decode.hip), as plain integer functions
// that compile for the device and for the host.  The kernels call them; moe_lrc_selftest_decode_index
// (host only) sweeps shapes, ranks and block shares through the same functions and checks every
// offset against the size of the buffer resource or LDS region it addresses.
#pragma once
#include <stdint.h>

#include "layout.h"

namespace lrc {
namespace dec {

constexpr int kWaves = 16;            // wavefronts of a block
constexpr int kLdsUnits = 8192;       // 16-byte units of staged activations (128 KB)
constexpr int kSpareUnits = 2048;     // 16-byte units behind them (32 KB): (in A) fragments of small ranks
constexpr int kRing = 2;              // ring slots of a wavefront (each holds one k-step of two streams)
constexpr int kStreams = 2;           // streams of a slot: (W1, W3) tiles of one n-tile, or two n-tiles of W2

// A block's n-tiles: block b of the G that share an expert owns tiles [t0, t1).  (G * NT stays far below 2^31: both are at
// most a few thousand times the 32 n-tiles of a block.)
LRC_HD void block_tiles(int b, int G, int NT, int& t0, int& t1) {
  t0 = (int)(uint32_t(b) * uint32_t(NT) / uint32_t(G));
  t1 = (int)(uint32_t(b + 1) * uint32_t(NT) / uint32_t(G));
}

// Work units of a block: an n-tile of both projections (DUAL) or a pair of adjacent n-tiles (W2).
LRC_HD int block_units(int nt_b, bool dual) { return dual ? nt_b : (nt_b + 1) / 2; }
// Unit slots a wavefront visits one after the other.
LRC_HD int unit_slots(bool dual, int mt) { (void)mt; return dual ? 2 : 1; }
// n-tiles a block can own
LRC_HD int max_block_tiles(int mt) { (void)mt; return 32; }

// Wavefronts that share one unit, each taking every kw-th k-step: the largest power of two kw with units * kw <= 16, at least 1.
LRC_HD int waves_per_unit_log2(int units) { return units <= 1 ? 4 : units > 8 ? 0 : __builtin_clz(uint32_t(units - 1)) - 28; }

// n-tile of stream m of unit u (block-relative unit index): DUAL: tile t0 + u for both streams;
// W2: tiles t0 + 2u and t0 + 2u + 1.
LRC_HD int stream_tile(int t0, int u, int m, bool dual) { return dual ? t0 + u : t0 + 2 * u + m; }

// A wavefront walks segments: (phase ph, own unit ts), ph = 0 .. n_ph - 1 over the k-steps of a staging phase, then ph = n_ph
// over the rank steps.  Own step `si` of a segment is its step si * kw + kwi; a segment is walked in whole turns of the
// ring, so that ring slots are indexed statically, and while a turn is multiplied the next turn, of the same segment or
// of the one after it, is fetched.  No step is walked that only pads: a segment's turns follow from its own length.
struct StepPlan {
  int KP;        // k-steps per phase (16 with one row tile, 8 with two)
  int n_ph;      // phases of this K-block
};
LRC_HD StepPlan step_plan(int KSl, int mt) {
  StepPlan p;
  p.KP = (kLdsUnits / 512) / mt;
  p.n_ph = (KSl + p.KP - 1) / p.KP;
  return p;
}
// Units of a wavefront of group grp (0, 1 or 2: units grp and grp + groups).
LRC_HD int own_units(int grp, int groups, int units, bool dual) { return (grp < units ? 1 : 0) + (dual && grp + groups < units ? 1 : 0); }

struct Segment {
  int unit;      // block-relative unit
  int base;      // absolute k-step of its first step (k-steps)
  int len;       // steps, shared by kw wavefronts
  bool lr;       // rank steps of the B factor (else k-steps of packed codes)
};
// own: units of the wavefront (own_units); beyond the last segment (ph > n_ph, or no rank steps) the length is zero
LRC_HD Segment segment(int ph, int ts, int own, const StepPlan& p, int grp, int groups, int ks_lo, int KSl, int LS) {
  Segment s;
  const int left = KSl - ph * p.KP;
  s.unit = grp + ts * groups;
  s.base = ks_lo + ph * p.KP;
  s.lr = ph >= p.n_ph;
  s.len = ts >= own ? 0 : ph < p.n_ph ? (left < p.KP ? left : p.KP) : ph == p.n_ph ? LS : 0;
  return s;
}
// ... and own steps that are walked, whole turns of the ring.
LRC_HD int segment_steps(int len, int kw_log2) { return ((len + (kRing << kw_log2) - 1) >> (kw_log2 + 1)) * kRing; }
static_assert(kRing == 2, "the shift above");

// What own step si of a segment reads (k-share kwi of 1 << kw_log2).
struct StepRef {
  bool reg;      // a k-step of packed codes (else a rank step, or nothing)
  bool lr;       // a rank step of the B factor
  int unit;      // block-relative unit
  int ks;        // absolute k-step (reg)
  int st;        // step within the segment: k-step within the phase (reg), rank step (lr)
};
LRC_HD StepRef step_ref(const Segment& s, int si, int kwi, int kw_log2) {
  StepRef r;
  r.unit = s.unit;
  r.st = (si << kw_log2) + kwi;
  r.ks = s.base + r.st;
  r.reg = !s.lr && r.st < s.len;
  r.lr = s.lr && r.st < s.len;
  return r;
}

// Byte offsets of a lane's loads of one stream of a step (the hardware range-checks offset + size
// against the resource; a step that reads nothing gets an offset at the end of every resource).
// q3: the stream's factor pair is held at 3 bits (layout.h).  A rank step then reads, through `bf`,
// the lane's half of the 32 bytes of metadata of (rank step, group of four n-tiles, lane group) from
// a resource of (NT / 4) * LS * 128 bytes, and through `bc` the unit's code dword from a resource of
// NT * LS * 256 bytes; `bc` of any other step lies past every resource.
struct LaneOffsets { uint32_t code0, code1, meta, bf, bc; };
LRC_HD LaneOffsets lane_offsets(const StepRef& r, int tile, bool tile_ok, int lane, int bits, int NT, int group_shift,
                                uint32_t code_bytes, uint32_t meta_bytes, uint32_t bf_bytes_max, bool q3 = false) {
  const uint32_t tdw = kWave * 2 * bits, q = lane >> 4, c = lane & 15;
  const uint32_t gps = kTileK >> group_shift;
  const uint32_t meta_lane = ((q * kLaneK) >> group_shift) * (uint32_t(NT) * kTileN * 4) + c * 4;
  LaneOffsets o;
  const bool ok = r.reg && tile_ok, lr = r.lr && tile_ok;
  const uint32_t past = code_bytes > bf_bytes_max ? code_bytes : bf_bytes_max;
  const uint32_t tile_base = (uint32_t(r.ks) * NT + tile) * (tdw * 4);
  o.code0 = (ok ? tile_base : past) + lane * 16;
  o.code1 = (ok ? tile_base : code_bytes) + 1024 + lane * (bits == 3 ? 8 : 16);
  o.meta = (ok ? (uint32_t(r.ks) * gps * NT + tile) * (kTileN * 4) : meta_bytes) + meta_lane;
  // (selects on wave-uniform conditions rather than branches: the loads of a step stay in one block)
  const bool lq = q3 && lr;
  const uint32_t unit = uint32_t(r.st) * NT + tile, group4 = uint32_t(r.st) * (NT / 4) + (tile >> 2);
  o.bf = (lq ? group4 * 128 : lr ? unit * 1024 : past) + (lq ? q * 32 + (c & 1) * 16 : lane * 16);
  o.bc = (lq ? unit * 256 : 0xfffffe00u) + lane * 4;
  return o;
}

// Row of the operand-order activation buffer (in_rt rows) that lane row `rowl` of row tile mt stages
// in the pass that starts at the expert's row r (rin: that row's index in the buffer).  Past the
// expert's last row the MFMA columns are never stored: they read the buffer's last 16 rows, which
// the preparing launch keeps at zero (multiplying zeros costs the matrix cores the least).
constexpr int kZeroRows = 16;
LRC_HD int staged_row(int rin, int r, int mt, int rowl, int cnt, int in_rt) {
  return r + 16 * mt + rowl < cnt ? rin + 16 * mt + rowl : in_rt - kZeroRows + rowl;
}

// Lane group (64 inputs) of k-step ks that lane group q stages: its own, or past K (a multiple of 64) the k-step's last one below
// it (the padded weights there are exact zeros, any finite value will do).
LRC_HD int staged_group(int ks, int q, int K) { const int left = K / kLaneK - 4 * ks; return q < left ? q : left - 1; }

// (h A2) of the fused projection's own columns, left by every block for the W2 launch (ranks up to kHaRank):
// a 16-column factor tile rt of A2 meets the 16 columns of n-tile `tile` as the operand of a 16x16x16
// product, so lane (q, c) reads inputs 16 tile + 4 q .. + 3 of column 16 rt + c: half (q % 2) of the packed
// unit (tile / 2) of lane (2 (tile % 2) + q / 2, c).  Index of that half in units of four values.
constexpr int kHaRank = 32;                // (one rank step: the part sums of a row are 128 bytes)
LRC_HD uint32_t ha_operand(int rt, int tile, int lane, int F) {
  const int q = lane >> 4, c = lane & 15;
  return ((uint32_t(rt) * (F / 32) + tile / 2) * kWave + (2 * (tile & 1) + (q >> 1)) * 16 + c) * 2 + (q & 1);
}
// Part sums an expert's G blocks leave (blocks past the NT-th own no tile), and the place of block b's.
LRC_HD int ha_slots(int G, int NT) { return G < NT ? G : NT; }
LRC_HD int ha_slot(int b, int t0, int G, int NT) { return G <= NT ? b : t0; }
// The part sums K-block kb of kblocks takes: [lo, hi).
LRC_HD void ha_share(int kb, int kblocks, int slots, int& lo, int& hi) { lo = kb * slots / kblocks; hi = (kb + 1) * slots / kblocks; }
LRC_HD size_t ha_part(int slot, int total_rows, int row, int col) { return (size_t(slot) * total_rows + row) * kHaRank + col; }

// LDS unit of staged activation fragment (row tile mt, k-step kl of the phase, sub-step s).
LRC_HD int act_frag_unit(int mt, int kl, int s, int KP) { return ((mt * KP + kl) * 8 + s) * 64; }
// LDS unit (relative to the fragment region) of (in A) fragment (stream m, rank step st, row tile mt).
LRC_HD int p_frag_unit(int m, int st, int mt, int LS, int MT) { return ((m * LS + st) * MT + mt) * 64; }


}  // namespace dec
}  // namespace lrc
