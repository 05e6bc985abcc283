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

// A block's n-tiles: block b of the G that share an expert owns tiles [t0, t1).  (G * NT is at most 2^27: a projection has at most
// 4096 n-tiles, the wider of a layer's two sizes being 65536 at most, and a launch at most 256 experts times 128 blocks.)
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

// A wavefront walks segments: (phase ph, own unit ts), the k-steps of a staging phase.  Its own step k of a segment is step
// (k << kw_log2) + kwi; a segment is walked in whole turns of the ring, so that ring slots are indexed statically, and while
// a turn is multiplied the next turn, of the same segment or of the one after it, is fetched.  The rank steps of the units follow.
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
LRC_HD int phase_steps(const StepPlan& p, int ph, int KSl) { return KSl - ph * p.KP < p.KP ? KSl - ph * p.KP : p.KP; }
// Own steps of a segment of len steps.
LRC_HD int own_steps(int len, int kwi, int kw_log2) { return len > kwi ? (len - kwi + (1 << kw_log2) - 1) >> kw_log2 : 0; }

// Where the own steps of a segment lie: byte offsets (wave-uniform) of n-tile `tile`'s codes and metadata at the first and at the last
// of them.  From one to the next both move by a fixed stride and stop at the last: what is fetched beyond it is not multiplied.  A
// wavefront without a step of its own in the segment stays at the segment's last step.
struct Walk {
  uint32_t code, meta, code_last, meta_last;
  int n;         // own steps
};
struct Strides { uint32_t code, meta; };
LRC_HD Strides walk_strides(int kw_log2, int bits, int NT, int gps) {
  return Strides{uint32_t(NT << kw_log2) * (kWave * 2 * bits * 4), uint32_t((NT * gps) << kw_log2) * (kTileN * 4)};
}
// first: absolute k-step of the segment's first step
LRC_HD Walk walk_start(int first, int len, int tile, int kwi, int kw_log2, int bits, int NT, int gps, const Strides& st) {
  Walk w;
  w.n = own_steps(len, kwi, kw_log2);
  const uint32_t ks = first + (kwi < len ? kwi : len - 1), more = w.n > 1 ? w.n - 1 : 0;
  w.code = (ks * NT + tile) * (kWave * 2 * bits * 4);
  w.meta = (ks * gps * NT + tile) * (kTileN * 4);
  w.code_last = w.code + more * st.code;
  w.meta_last = w.meta + more * st.meta;
  return w;
}
LRC_HD void walk_on(Walk& w, const Strides& st) {
  w.code = w.code + st.code < w.code_last ? w.code + st.code : w.code_last;
  w.meta = w.meta + st.meta < w.meta_last ? w.meta + st.meta : w.meta_last;
}
// A lane's part of the offsets of a k-step's loads: the first 16 bytes of its codes, the rest, its metadata.  A stream without a tile
// adds kNoTile, which lies past every resource (the hardware then reads zeros without touching memory).
constexpr uint32_t kNoTile = 0x80000000u;
struct LaneOffsets { uint32_t code0, code1, meta; };
LRC_HD LaneOffsets lane_offsets(int lane, int bits, int NT, int group_shift, bool tile_ok) {
  const uint32_t q = lane >> 4, c = lane & 15, past = tile_ok ? 0u : kNoTile;
  return LaneOffsets{past + lane * 16, past + 1024 + lane * (bits == 3 ? 8 : 16), past + ((q * kLaneK) >> group_shift) * (uint32_t(NT) * kTileN * 4) + c * 4};
}
// The rank steps of a wavefront come in turns of the ring, too: turn t brings, in slot i, rank_slot_step of own unit rank_slot_unit (both
// own units' steps side by side in the fused projection, two steps of the one unit of W2).
LRC_HD int rank_slot_unit(bool dual, int i) { return dual ? i : 0; }
LRC_HD int rank_slot_step(bool dual, int t, int i, int kwi, int kw_log2) { return kwi + ((dual ? t : kRing * t + i) << kw_log2); }
// Turns of a wavefront that has a unit, of LS rank steps (0: none of its own).
LRC_HD int rank_turns(bool dual, int LS, int kwi, int kw_log2) { const int n = own_steps(LS, kwi, kw_log2); return dual ? n : (n + kRing - 1) / kRing; }

// Byte offsets of a lane's loads of rank step st of one stream (range-checked: a step past the stream's own rank, or without a tile,
// lies past the resource): the B factor's unit; or, of a pair held at 3 bits (layout.h), through `bf` the lane's half of the 32
// bytes of metadata of (rank step, group of four n-tiles, lane group) from a resource of (NT / 4) * LS * 128 bytes, and through `bc` the
// unit's code dword from a resource of NT * LS * 256 bytes.
struct RankOffsets { uint32_t bf, bc; };
LRC_HD RankOffsets rank_offsets(int st, int tile, bool ok, int lane, int NT, bool q3) {
  const uint32_t q = lane >> 4, c = lane & 15, unit = uint32_t(st) * NT + tile, group4 = uint32_t(st) * (NT / 4) + (tile >> 2);
  RankOffsets o;
  o.bf = ok ? (q3 ? group4 * 128 + q * 32 + (c & 1) * 16 : unit * 1024 + lane * 16) : kNoTile;
  o.bc = ok ? unit * 256 + lane * 4 : kNoTile;
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
