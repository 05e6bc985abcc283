// Decode flavour of the expert FFN (Sections 2.3 and 3.2): few rows per expert, so the layer is a
// stream of packed weights and the job is to keep HBM busy.
//
//   - one block of 16 wavefronts per CU.  For routed experts every block reads which expert it
//     serves, which share of the expert's n-tiles and where the expert's rows are from one 32-byte
//     entry of a table the preparing launch has made (plan.h): experts without rows get no blocks,
//     experts whose rows need several 32-row passes get more;
//   - the activations of the expert (up to 32 rows) are staged into 128 KB of LDS once per phase of
//     16 (or 8) k-steps by direct global -> LDS copies, issued together with the first packed tiles
//     and the (in A) fragments: one memory round trip before the first multiply;
//   - a ring slot of a wavefront holds one k-step of two streams: the W1 and W3 tiles of one n-tile
//     in the fused kernel, two adjacent n-tiles in the W2 kernel.  An activation fragment read from
//     LDS meets both streams;
//   - each wavefront streams its packed tiles HBM -> registers with buffer loads through a ring of
//     register slots walked by straight-line code: a load past the end of the resource returns
//     zeros, so refills are unconditional and the number of loads in flight is static;
//   - codes are unpacked in registers (unpack.h) straight into MFMA A-operands; the rank-r term is
//     ceil(r / 32) more steps per stream on the B factor's fp16 units against (in A), which
//     the launches before have left in global memory; the rank is the projection's own (Section 3.1
//     allocates a rank per expert matrix): a stream with fewer rank steps reads zeros past its factor;
//   - (h A2) of ranks up to 32 is made at the end of the fused projection's blocks, from the h they hold in
//     registers: each block's columns are a share of its long K, and the W2 blocks add the shares of
//     their K-block up while their activations arrive, where that is less than a launch between the two costs, which
//     reads h and A2 again (ha_room).  Larger ranks and many rows over few experts keep that launch;
//   - a long K (W2) is split into K-blocks (grid.z) of one or two phases whose fp32 partial outputs
//     the combine (or reduce_kernel, for the stand-alone call) adds in a fixed order.
#include <algorithm>
#include <type_traits>

#include "decode_index.h"
#include "factor_q3.h"
#include "ffn_common.h"
#include "plan.h"
#include "xa_rows.h"

namespace lrc {

namespace {

using namespace ffn;
using namespace dec;


// One expert's share of a block: MT = row tiles per pass (1 when the expert has at most 16 rows).
// (A pass of 32 rows can be put on v_mfma_f32_32x32x16_f16, which has the same peak rate as the
// 16x16x32 shape used here and needs half as many instructions, by swapping 16-lane rows between the
// two streams' registers; measured, the four swaps per sub-step cost this kernel more than the two
// matrix instructions save.)
// Q3: some factor pair of the layer is held at 3 bits (layout.h): a rank step of such a pair brings
// the unit's code dword in the slot's metadata register and the lane's half of the unit's metadata in
// its first four code registers, and is dequantized into the fp16 unit before it is used.
// HA: (h A2) is left by the fused projection's blocks and added up by those of W2 (KArgs::ha).
// A pass's start is what a launch of short streams consists of: with one k-step to multiply, this kernel took 14 us, most of them
// in five dependent reads of the expert's table entry, 64-bit divisions, and code that every wavefront ran once.  So: one level
// of loads from the block's entry to the expert's (all of it read at once, into scalar registers), the activations requested
// before its pointers have arrived, no division, and one copy of the code that multiplies and fetches (a straight-line
// kilobyte that runs once costs 0.2 us of instruction fetch beside its issue).
template <int BITS, bool DUAL, int MT, bool Q3, bool HA>
__device__ __forceinline__ void decode_body(const KArgs& a, uint4* xs, const PlanEntry& pe) {
  constexpr int NS = kStreams;
  constexpr int TS = DUAL ? 2 : 1;
  constexpr int NC = Extract<BITS>::kClasses;
  constexpr int RING = kRing;
  const int e = pe.e, r0 = pe.r0, cnt = pe.cnt, t0 = pe.t0, t1 = pe.t1;
  const int th = threadIdx.x, lane = th & 63;
  const int wave = __builtin_amdgcn_readfirstlane(th >> 6);
  const int q = lane >> 4, c = lane & 15;
  // the expert's table entry: everything this block needs of it, requested together
  const ConstDesc d = const_desc(a.desc + e);
  const int has_factors = d->has_factors, q3 = d->q3, rank2 = d->rank[2];
  const int comp = *const_i32((a.comp_rows ? a.comp_rows : &a.desc->q3) + (a.comp_rows ? e : 0));
  const uint32_t* codes[NS] = {d->codes[DUAL ? 0 : 2], d->codes[DUAL ? 1 : 2]};
  const uint32_t* metas[NS] = {d->meta[DUAL ? 0 : 2], d->meta[DUAL ? 1 : 2]};
  const int ranks[NS] = {d->rank[DUAL ? 0 : 2], d->rank[DUAL ? 1 : 2]};
  const float lam[2] = {d->inv_lambda[DUAL ? 0 : 2], d->inv_lambda[DUAL ? 1 : 2]};
  // (x A1 | x A3) kept per token (ranks up to kXaTokensRank: its fragments are at most one per wavefront): the token
  // of the row whose part of a fragment this lane copies, on its way while the expert's table entry is read
  int token = -1;
  if constexpr (DUAL) {
    if (a.p_tokens > 0) token = a.row_tok[r0 + min(16 * (wave % MT) + c, cnt - 1)];
  }

  // how the block's units are dealt to the 16 wavefronts
  const int nt_b = t1 - t0;
  const int units = block_units(nt_b, DUAL);
  const int kwl = waves_per_unit_log2(units), kw = 1 << kwl;
  const int groups = kWaves >> kwl, grp = wave >> kwl, kwi = wave & (kw - 1), own = own_units(grp, groups, units, DUAL);

  // this block's K-block: k-steps ks_lo .. ks_lo + KSl - 1
  const int kb = blockIdx.z, ks_lo = kb * a.kb_steps, KSl = min(a.KS, ks_lo + a.kb_steps) - ks_lo;
  const StepPlan sp = step_plan(KSl, MT);
  const int KP = sp.KP;
  const uint32_t code_bytes = uint32_t(a.KS) * a.NT * (kWave * 2 * BITS * 4), meta_bytes = uint32_t(a.G) * a.NT * kTileN * 4;

  // (what a later pass or phase forms again is formed there, not kept in registers from the start of the block)
  auto again = [](int v) { asm volatile("" : "+s"(v)); return v; };
  // A phase is MT * nk * 8 fragments of 64 units (16 rows x 4 column groups of one MFMA sub-step);
  // four 256-byte runs of the operand-order buffer become 1 KB of LDS, lane-linear.  Rows past the
  // expert's last one read the zero rows at the end of the buffer (staged_row): their output
  // columns are never stored.  The copy is asynchronous and takes no registers: each lane's 16 bytes go from
  // global memory straight to LDS (wave-uniform LDS base + 16 * lane), counted by vmcnt.  A lane's address is a
  // wave-uniform base (k-step, sub-step) plus a 32-bit offset (column group, row) that is the same for every k-step but one
  // that K ends in.
  auto stage_issue = [&](const auto& A, int r, int ph, int nk) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    // first input row of this pass (shared experts all read the token rows 0..T-1)
    const int rin = ((DUAL && !A.offsets) ? 0 : r0) + r;
    const int s = wave & 7;                  // fragment (mt, kl, s): wavefront w takes s = w % 8, kl = w / 8, w / 8 + 2, ...
    const size_t step = size_t(A.in_rt) * 32 * 16;       // bytes of a k-step
    uint32_t row[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) row[mt] = uint32_t(staged_row(rin, r, mt, ln & 15, cnt, A.in_rt)) * 16u;
    for (int kl = wave >> 3; kl < nk; kl += 2) {
      const int ks = ks_lo + ph * KP + kl;
      const uint8_t* base = reinterpret_cast<const uint8_t*>(A.in) + ks * step + size_t(s * 4) * (uint32_t(A.in_rt) * 16u);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, 0xffffffffu, 0x00020000);
      const uint32_t group = uint32_t(staged_group(ks, ln >> 4, A.K)) * (uint32_t(A.in_rt) * 16u);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rs, reinterpret_cast<__attribute__((address_space(3))) void*>(reinterpret_cast<uintptr_t>(xs + act_frag_unit(mt, kl, s, KP))), 16,
            int(group + row[mt]), 0, 0, 0);
    }
  };
  // (h A2) from the part sums of the fused projection's blocks: TPO threads share four columns of a row.
  // The first kHaFirst parts are requested before anything else of the pass, the sums go
  // to LDS as the fragments p_issue would copy.
  constexpr int TPO = 8 / MT, kHaFirst = BITS == 4 ? 2 : 4;
  constexpr bool joined = HA && !DUAL;      // (its fragments always fit behind the activations)
  float4_t part[kHaFirst];
  int pair_of_row = 0, ha_lo = 0, ha_hi = 0;
  int hj = 0, hcol = 0, hrow = 0;
  auto part_issue = [&](int r) {
    const KernArgs ka = kern_args();
    int ht_ = th;
    asm volatile("" : "+v"(ht_));
    hj = ht_ & (TPO - 1); hcol = (ht_ / TPO) & 7; hrow = ht_ / (8 * TPO);
    const int row = r0 + min(r + hrow, cnt - 1);
    ha_share(kb, gridDim.z, pe.slots, ha_lo, ha_hi);
#pragma unroll
    for (int i = 0; i < kHaFirst; ++i)
      part[i] = *reinterpret_cast<const float4_t*>(ka->ha + ha_part(max(min(ha_lo + hj + i * TPO, ha_hi - 1), 0), ka->total_rows, row, 4 * hcol));
    pair_of_row = ka->row_pair[row];
  };
  int row_se[MT];                             // the rows' exponents for the end of the pass
  auto exp_issue = [&](const auto& A, int r) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) row_se[mt] = A.row_exp[(A.offsets ? r0 : 0) + min(r + 16 * mt + c, cnt - 1)];
  };
  // (the first pass's, on their way before the table entry's fields are used)
  if constexpr (joined) part_issue(0);
  stage_issue(a, 0, 0, min(KP, KSl));
  __builtin_amdgcn_sched_barrier(0);

  // The rank-r term rides the same stream (B-factor units in place of packed codes, against (in A)
  // instead of the activations).  With K-blocks, every K-block meets the part of (in A) summed over
  // its own k-steps (the term is linear in it).  Each stream has the rank of its own projection; a
  // resource of the size its rank fills makes later steps read zeros.
  const bool lowrank = a.rank > 0 && a.row_pair != nullptr && has_factors != 0 && comp > 0;
  int LSm[NS];
#pragma unroll
  for (int m = 0; m < NS; ++m) LSm[m] = lowrank ? int(uint32_t(min(ranks[m], a.rank) + 31) / 32) : 0;
  const int LS = max(LSm[0], LSm[1]);
  // 16-column tiles of (h A2) that this launch makes (fused projection) or adds up (W2)
  const int ht = HA && lowrank ? int(uint32_t(min(rank2, a.rank) + 15) / 16) : 0;

  __amdgpu_buffer_rsrc_t code_rs[NS], meta_rs[NS];
  bool q3m[NS];
#pragma unroll
  for (int m = 0; m < NS; ++m) {
    q3m[m] = Q3 && ((q3 >> (DUAL ? m : 2)) & 1) != 0;
    code_rs[m] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(codes[m]), 0, code_bytes, 0x00020000);
    meta_rs[m] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(metas[m]), 0, meta_bytes, 0x00020000);
  }
  // (in A) fragments: [projection][rank step][row tile][lane].  Up to 32 of them sit behind the staged
  // activations from the start of a pass; more (ranks above 256) take the place of the activations
  // after the last k-step.
  // (the two streams of the W2 kernel are tiles of one projection: they meet the same fragments)
  constexpr int NP = DUAL ? 2 : 1;
  const int p_frags = NP * LS * MT;
  const bool p_late = p_frags * 64 > kSpareUnits;
  uint4* p_lds = p_late ? xs : xs + kLdsUnits;
  const int pitch = NP * a.ls * 32;                  // halves per row of (in A): [A1 | A3], or A2
  // The fused projection's own columns of A2: the packed units (32 inputs each) u0 .. u0 + n_u - 1 of every
  // factor tile (3-bit pair: their code dwords, then the metadata of the n_q x 4 groups of 64 inputs from g0
  // on) are copied behind those fragments at the start of the first pass, where they fit; else read when used.
  const bool q3_a2 = Q3 && ((q3 >> 2) & 1) != 0;
  const int u0 = t0 / 2, n_u = (t1 - 1) / 2 - u0 + 1, g0 = t0 / 4, n_q = ((t1 - 1) / 4 - g0) / 4 + 1;
  const bool a2_early = HA && DUAL && ht > 0 && !p_late && p_frags * 64 + (q3_a2 ? (n_u + n_q) * 16 : n_u * 64) * ht <= kSpareUnits;
  // Copies to LDS of 16 (or 4) bytes a lane, byte offset `at` from a wave-uniform base.  (By a buffer resource: with a global_load_lds in flight
  // the compiler waits for every load at the next barrier.  Rows of this flavour are at most 128 an expert on average: `at` is below 2^27.)
  auto copy16 = [](const void* from, int at, uint4* to) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(from), 0, 0xffffffffu, 0x00020000),
        reinterpret_cast<__attribute__((address_space(3))) void*>(reinterpret_cast<uintptr_t>(to)), 16, at, 0, 0, 0);
  };
  auto copy4 = [](const void* from, int at, uint4* to) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(from), 0, 0xffffffffu, 0x00020000),
        reinterpret_cast<__attribute__((address_space(3))) void*>(reinterpret_cast<uintptr_t>(to)), 4, at, 0, 0, 0);
  };

  // (in A) of a pass's rows: fp16 row-major in global memory, already multiplied by the
  // projection's power-of-two pre-scale and zero for rows without the term.  Fragment
  // (m, st, mt): lane (q, c) copies columns 32 st + 8 q .. + 7 of row 16 mt + c.  A row past the
  // expert's last one is clamped to a valid row (its output column is never stored).
  auto p_issue = [&](const auto& A, int r) {
    const _Float16* P = reinterpret_cast<const _Float16*>(A.p) + size_t(kb) * A.total_rows * pitch;
    for (int f = wave; f < p_frags; f += kWaves) {
      const int mt = f % MT, g = f / MT, m = g >= LS ? 1 : 0, st = g - m * LS;
      const int row = r0 + min(r + 16 * mt + c, cnt - 1);
      copy16(P, (row * pitch + m * A.ls * 32 + 32 * st + 8 * q) * 2, p_lds + p_frag_unit(m, st, mt, LS, MT));
    }
  };
  // ... or kept per token (the projection's rows of every token, p_tokens > 0)
  auto p_issue_tokens = [&](const auto& A, int r) {
    if (wave >= p_frags) return;
    const int mt = wave % MT, g = wave / MT, m = g >= LS ? 1 : 0, st = g - m * LS, pr = r + 16 * mt + c;
    if (r > 0) token = A.row_tok[r0 + min(pr, cnt - 1)];
    // (rows without the term read the row of zeros)
    const int row = pr < cnt && token >= 0 ? e * A.p_tokens + token : A.n_exp * A.p_tokens;
    copy16(A.p, (row * pitch + m * A.ls * 32 + 32 * st + 8 * q) * 2, p_lds + p_frag_unit(m, st, mt, LS, MT));
  };
  auto p_start = [&](const auto& A, int r) {
    if (p_late || joined) return;
    if (DUAL && A.p_tokens > 0) p_issue_tokens(A, r);
    else p_issue(A, r);
  };
  auto p_join = [&](int r) {
    if (LS == 0) return;                     // (ranks up to kHaRank: one rank step)
    const KernArgs ka = kern_args();
    const int row = r0 + min(r + hrow, cnt - 1), col = 4 * hcol;
    const bool take = r + hrow < cnt && pair_of_row % ka->top_k < ka->top_n;
    const float lam2 = const_desc(ka->desc + e)->xa_scale[2];
    float4_t sum = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kHaFirst; ++i)
      if (ha_lo + hj + i * TPO < ha_hi) sum += part[i];
    for (int sl = ha_lo + hj + kHaFirst * TPO; sl < ha_hi; sl += TPO)
      sum += *reinterpret_cast<const float4_t*>(ka->ha + ha_part(sl, ka->total_rows, row, col));
#pragma unroll
    for (int dlt = 1; dlt < TPO; dlt *= 2)
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] += __shfl_xor(sum[i], dlt);
    if (hj == 0) {
      half4_t v = half4_t{0, 0, 0, 0};
      if (take && col < 16 * ht) v = half4_t{to_f16_sat(sum[0] * lam2), to_f16_sat(sum[1] * lam2), to_f16_sat(sum[2] * lam2), to_f16_sat(sum[3] * lam2)};
      reinterpret_cast<half4_t*>(p_lds + p_frag_unit(0, 0, hrow >> 4, LS, MT) + (hcol >> 1) * 16 + (hrow & 15))[hcol & 1] = v;
    }
  };

  // The own steps of the wavefront's segments are fetched a turn of the ring ahead of their use: wave-uniform offsets that move by a
  // stride, beside lane offsets that stay (a scalar instruction of each of the sixteen wavefronts goes through the one scalar unit
  // of the CU: sixty a step, with the offsets formed anew, were a good part of a step; about 25 now.  W2 alone, before and with this:
  // Mixtral T = 64 48 -> 46 us, T = 13 at 3 bits 52 -> 46, T = 1 17.1 -> 16.2; W1|W3 at T = 13, 3 bits 87 -> 81).
  // The same loads bring the first turn of rank steps at the end: other resources and lane offsets, no branch between two
  // kinds of loads, behind which the compiler's waits would be for all of them.
  const int gps = kTileK >> a.group_shift;
  const Strides strides = walk_strides(kwl, BITS, a.NT, gps);
  constexpr int NLO = DUAL && !Q3 ? 1 : NS;    // W1 and W3 are laid out alike: one set of offsets serves both (registers: the kernel is at its 128)
  struct Source {
    Walk at;                                  // of the next fetch
    Strides by;
    uint32_t code2, meta2;                    // W2: from the first stream's tile to the second's
    LaneOffsets lo[NLO];
    __amdgpu_buffer_rsrc_t code[NS], meta[NS];
  } src;
  auto fetch = [&](Slot<BITS, NS>& sl) {
#pragma unroll
    for (int m = 0; m < NS; ++m) {
      const uint32_t code = src.at.code + (m > 0 && !DUAL ? src.code2 : 0), meta = src.at.meta + (m > 0 && !DUAL ? src.meta2 : 0);
      const LaneOffsets& lo = src.lo[m < NLO ? m : 0];
      const u32x4 v0 = __builtin_amdgcn_raw_buffer_load_b128(src.code[m], lo.code0, code, 0);
      sl.cw[m][0] = v0[0]; sl.cw[m][1] = v0[1]; sl.cw[m][2] = v0[2]; sl.cw[m][3] = v0[3];
      if constexpr (BITS == 3) {
        const u32x2 v1 = __builtin_amdgcn_raw_buffer_load_b64(src.code[m], lo.code1, code, 0);
        sl.cw[m][4] = v1[0]; sl.cw[m][5] = v1[1];
      } else if constexpr (BITS == 4) {
        // (code1 by the instruction's own offset, a register less of the kernel's 128.  A rank step reads the next unit's 16 bytes with it and
        // leaves them)
        const u32x4 v1 = __builtin_amdgcn_raw_buffer_load_b128(src.code[m], lo.code0 + 1024, code, 0);
        sl.cw[m][4] = v1[0]; sl.cw[m][5] = v1[1]; sl.cw[m][6] = v1[2]; sl.cw[m][7] = v1[3];
      }
      sl.mw[m] = __builtin_amdgcn_raw_buffer_load_b32(src.meta[m], lo.meta, meta, 0);
    }
    walk_on(src.at, src.by);
  };
  // fetches from here on: the steps of (phase ph, own unit ts), or nothing
  auto fetch_from = [&](int ph, int ts, bool some) {
    const int tile = stream_tile(again(t0), again(grp) + ts * groups, 0, DUAL);
    src.by = strides;
    src.at = walk_start(again(ks_lo) + ph * KP, some ? phase_steps(sp, ph, KSl) : 1, some ? tile : 0, again(kwi), kwl, BITS, a.NT, gps, strides);
    src.code2 = kWave * 2 * BITS * 4; src.meta2 = kTileN * 4;
#pragma unroll
    for (int m = 0; m < NS; ++m) {
      if (m < NLO) src.lo[m] = lane_offsets(lane, BITS, a.NT, a.group_shift, some && (DUAL ? tile : tile + m) < t1);
      src.code[m] = code_rs[m]; src.meta[m] = meta_rs[m];
    }
  };
  // The B factor of stream m's projection, of the size its rank fills (3-bit pair: the B section's metadata, 128 bytes per rank step and
  // group of four n-tiles, and the code dwords of its units; no bytes of these for an fp16 pair: every read gives zero).  Read from
  // the table again where it is used: it would not fit the scalar registers through the k-steps.
  auto rank_rsrc = [&](int m, __amdgpu_buffer_rsrc_t& bf, __amdgpu_buffer_rsrc_t& bc) {
    const KernArgs ka = kern_args();
    const ConstDesc dd = const_desc(ka->desc + e);
    const int mat = DUAL ? m : 2, NT = ka->NT;
    bf = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(dd->bf[mat]), 0, q3m[m] ? uint32_t(NT / 4) * LSm[m] * 128 : uint32_t(NT) * LSm[m] * 1024, 0x00020000);
    if constexpr (Q3) bc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(dd->bfc[mat]), 0, q3m[m] ? uint32_t(NT) * LSm[m] * 256 : 0u, 0x00020000);
  };
  // Offsets of slot i of rank turn t (a stream past its own rank, or without a unit, reads nothing: past its resource)
  auto rank_at = [&](int t, int i, int m, int ln) {
    const int ts = rank_slot_unit(DUAL, i), tile = stream_tile(again(t0), again(grp) + ts * groups, m, DUAL);
    return rank_offsets(rank_slot_step(DUAL, t, i, again(kwi), kwl), tile, ts < own && tile < t1, ln, a.NT, Q3 && q3m[m]);
  };
  // ... the first turn, by the fetch that ends the k-steps: slot i from here on
  auto fetch_rank_from = [&](int i) {
    int ln = lane;
    asm volatile("" : "+v"(ln));              // (the offsets are made here, not kept in registers through the k-steps)
    src.by = Strides{0, 0};
    src.at = Walk{0, 0, 0, 0, 0};
    src.code2 = src.meta2 = 0;
#pragma unroll
    for (int m = 0; m < NS; ++m) {
      if (m < NLO) {
        const RankOffsets o = rank_at(0, i, m, ln);
        src.lo[m] = LaneOffsets{o.bf, kNoTile, Q3 ? o.bc : kNoTile};
      }
      if (i == 0) {
        if constexpr (Q3) rank_rsrc(m, src.code[m], src.meta[m]);
        else rank_rsrc(m, src.code[m], src.code[m]);
      }
    }
  };
  // ... and slot i of a turn beyond the first
  auto fetch_rank = [&](Slot<BITS, NS>& sl, int t, int i) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int m = 0; m < NS; ++m) {
      const RankOffsets o = rank_at(t, i, m, ln);
      const u32x4 v0 = __builtin_amdgcn_raw_buffer_load_b128(src.code[m], o.bf, 0, 0);
      sl.cw[m][0] = v0[0]; sl.cw[m][1] = v0[1]; sl.cw[m][2] = v0[2]; sl.cw[m][3] = v0[3];
      if constexpr (Q3) sl.mw[m] = __builtin_amdgcn_raw_buffer_load_b32(src.meta[m], o.bc, 0, 0);
    }
  };
  Slot<BITS, NS> ring[RING];
  static_assert(RING == 2 && TS <= RING, "a rank turn's slots: a unit each, or two steps of one unit");

  // ---- start of the first pass: the copies that are left ----
  p_start(a, 0);
  if (a2_early) {
    uint4* dst = p_lds + p_frags * 64;
    for (int f = wave; f < n_u * ht; f += kWaves) {      // (ht: 1 or 2)
      const int rt = f >= n_u ? 1 : 0, unit = (rt * (a.N / 32) + u0 + f - rt * n_u) * kWave + lane;
      if (q3_a2) copy4(d->af[2], unit * 4, dst + f * 16);
      else copy16(d->af[2], unit * 16, dst + f * 64);
    }
    if (q3_a2)
      for (int f = wave; f < n_q * ht; f += kWaves) {
        const int rt = f >= n_q ? 1 : 0, g = min(g0 + 4 * (f - rt * n_q) + q, a.N / 64 - 1);
        copy4(d->afm[2], ((rt * (a.N / 64) + g) * 16 + c) * 4, dst + (n_u * ht + f) * 16);
      }
  }
  __builtin_amdgcn_sched_barrier(0);
  constexpr int kAheadLoads = RING * NS * (BITS == 2 ? 2 : 3);

  for (int r = 0; r < cnt; r += 16 * MT) {
    // every pass computes all MT row tiles (a last pass with fewer rows computes columns nobody stores)
    if (r > 0) {
      __syncthreads();                        // everyone is done with the previous pass's LDS
      const KernArgs ka = kern_args();
      const int ra = again(r);
      if constexpr (joined) part_issue(ra);
      stage_issue(*ka, ra, 0, min(KP, KSl));
      p_start(*ka, ra);
    }
    // The first turn of the ring and the rows' exponents, requested last, stay in flight over the wait for the copies to LDS: in one place
    // for all passes, for registers that two places load are moved where the two meet, behind a wait for all loads (16 of the 24
    // kernels had one), and spill: scalar spills W1|W3 at 2 bits with part sums 171 -> 120, with 3-bit pairs 308 -> 188, vector spills at 4
    // bits 3 to 11 registers -> 0.  Whole forward, Mixtral shape T = 64: 143.9 -> 140.5 us on one card, 132.6 -> 131.7 on another, at 4
    // bits 194.1 -> 191.6; T = 1, T = 13 at 3 bits, Qwen3 T = 64 the same.
    fetch_from(0, 0, own > 0);
#pragma unroll
    for (int i = 0; i < RING; ++i) fetch(ring[i]);
    __builtin_amdgcn_sched_barrier(0);
    exp_issue(*kern_args(), again(r));
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (joined) p_join(again(r));
    wait_loads_barrier_but<kAheadLoads + MT>();

    float4_t acc[TS][MT][NS];
#pragma unroll
    for (int ts = 0; ts < TS; ++ts)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int m = 0; m < NS; ++m) acc[ts][mt][m] = float4_t{0.f, 0.f, 0.f, 0.f};
    // a rank step of one unit: the slot holds B-factor units, which meet (in A) as they are
    auto compute_lr = [&](const Slot<BITS, NS>& cur, int st, float4_t (&ac)[MT][NS]) {
#pragma unroll
      for (int m = 0; m < NS; ++m) {
        if (st >= LSm[m]) continue;
        half8_t bfrag = __builtin_bit_cast(half8_t, make_uint4(cur.cw[m][0], cur.cw[m][1], cur.cw[m][2], cur.cw[m][3]));
        if constexpr (Q3) {
          if (q3m[m]) {
            const uint32_t mine[4] = {cur.cw[m][0], cur.cw[m][1], cur.cw[m][2], cur.cw[m][3]};
            bfrag = q3_unit_b(cur.mw[m], mine, (c & 1) != 0);
          }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const half8_t pf = __builtin_bit_cast(half8_t, p_lds[p_frag_unit(DUAL ? m : 0, st, mt, LS, MT) + lane]);
          ac[mt][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bfrag, pf, ac[mt][m], 0, 0, 0);
        }
      }
    };
    // a k-step of packed codes of one unit
    auto compute = [&](const Slot<BITS, NS>& cur, int kl, float4_t (&ac)[MT][NS]) {
      const uint4* xk = xs + size_t(kl) * 8 * 64 + lane;
      uint32_t s2[NS][NC], c2[NS];
#pragma unroll
      for (int m = 0; m < NS; ++m) {
        s2[m][0] = (cur.mw[m] & 0xffffu) | (cur.mw[m] << 16);
        c2[m] = (cur.mw[m] >> 16) | (cur.mw[m] & 0xffff0000u);
        constexpr uint32_t step = Extract<BITS>::kStepBits == 2 ? 0x44004400u : 0x48004800u;   // 4.0 or 8.0
#pragma unroll
        for (int p = 1; p < NC; ++p) s2[m][p] = pk_mul(s2[m][p - 1], step);
      }
      // One sub-step: 32 rows of both weight tiles are unpacked into MFMA operands while the
      // activation fragments wait in registers.  Where the registers allow (XB == 2) the fragments of
      // sub-step s + 1 are requested from LDS before sub-step s is unpacked; the reads and the waits
      // are written out, because the compiler would move each read down to its use.
      constexpr int XB = (MT == 1 || BITS == 2) ? 2 : 1;
      half8_t xf[XB][MT];
      uint32_t xaddr[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xaddr[mt] = uint32_t(reinterpret_cast<uintptr_t>(xk)) + mt * KP * 8 * 1024;
      if constexpr (XB == 2) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) xf[0][mt] = lds_read16<0>(xaddr[mt]);
      }
      auto substep = [&](auto S) {
        constexpr int s = decltype(S)::value;
        if constexpr (XB == 2) {
          if constexpr (s < 7) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xf[(s + 1) & 1][mt] = lds_read16<(s + 1) * 1024>(xaddr[mt]);
          }
        } else {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) xf[0][mt] = __builtin_bit_cast(half8_t, xk[(size_t(mt) * KP * 8 + s) * 64]);
        }
        half8_t wf[NS];
#pragma unroll
        for (int m = 0; m < NS; ++m) {
          uint32_t v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            v[j] = pk_fma(Extract<BITS>::field(cur.cw[m], 4 * s + j), s2[m][Extract<BITS>::cls(4 * s + j)], c2[m]);
          wf[m] = __builtin_bit_cast(half8_t, make_uint4(v[0], v[1], v[2], v[3]));
        }
        if constexpr (XB == 2) {
          // the fragments of this sub-step are older than the MT reads just issued
          if constexpr (MT == 1) lds_wait<(s < 7 ? 1 : 0)>(xf[s & 1][0]);
          else lds_wait<(s < 7 ? 2 : 0)>(xf[s & 1][0], xf[s & 1][MT - 1]);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int m = 0; m < NS; ++m)
            ac[mt][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[m], xf[XB == 2 ? (s & 1) : 0][mt], ac[mt][m], 0, 0, 0);
      };
      substep(std::integral_constant<int, 0>{}); substep(std::integral_constant<int, 1>{});
      substep(std::integral_constant<int, 2>{}); substep(std::integral_constant<int, 3>{});
      substep(std::integral_constant<int, 4>{}); substep(std::integral_constant<int, 5>{});
      substep(std::integral_constant<int, 6>{}); substep(std::integral_constant<int, 7>{});
    };

#pragma unroll 1
    for (int ph = 0; ph < sp.n_ph; ++ph) {
      if (ph > 0) {
        __syncthreads();                      // everyone is done with the previous phase
        stage_issue(*kern_args(), again(r), ph, min(KP, KSl - ph * KP));
        wait_loads_barrier();
      }
      const int n = own_steps(phase_steps(sp, ph, KSl), kwi, kwl);
#pragma unroll
      for (int ts = 0; ts < TS; ++ts) {
        if (ts >= own) continue;
        // the segment after this one: the next unit's or the next phase's; after the last one the first turn of rank steps
        const int nts = ts + 1 < own ? ts + 1 : 0, nph = nts > 0 ? ph : ph + 1;
        const bool last = nph == sp.n_ph;
        // slot i of the ring: consumed, then refilled a turn ahead (without an own step, one turn to refill it)
#pragma unroll 1
        for (int si = 0; si < n || si == 0; si += RING) {
          const bool over = si + RING >= n;
          if (over && !last) fetch_from(nph, nts, true);
#pragma unroll
          for (int i = 0; i < RING; ++i) {
            if (si + i < n) compute(ring[i], ((si + i) << kwl) + kwi, acc[ts]);
            if (over && last) fetch_rank_from(i);
            fetch(ring[i]);
          }
        }
      }
    }
    if (LS > 0) {                             // the rank steps (none unless this block adds the term)
      if (p_late) {                           // many of them: their (in A) fragments replace the activations
        __syncthreads();
        p_issue(*kern_args(), again(r));
        wait_loads_barrier();
      }
      // The last fetch of the k-steps has brought the first turn, one slot is refilled while the other's step is on its way.  (Requests
      // after the first turn's products had nothing in flight beside them: a memory round trip more a unit and pass.  Whole forward,
      // Mixtral shape, so -> with this, us: rank 64 T = 8 118.4 -> 116.0, T = 160 281.3 -> 279.9; rank 128 T = 8 123 -> 120, T = 64
      // 161.3 -> 159.9; 3 bits with 3-bit pairs, rank 64, T = 8 145.3 -> 138.4, T = 160 326 -> 316.6; rank 32 the same.)
      const int turns = own > 0 ? rank_turns(DUAL, LS, kwi, kwl) : 0;
      auto slot_lr = [&](int t, int i) {
        const int ts = rank_slot_unit(DUAL, i), st = rank_slot_step(DUAL, t, i, kwi, kwl);
        if (ts < own && st < LS) compute_lr(ring[i], st, acc[ts]);
      };
      int t = 0;
#pragma unroll 1
      for (; t + 1 < turns; ++t)
#pragma unroll
        for (int i = 0; i < RING; ++i) {
          slot_lr(t, i);
          fetch_rank(ring[i], t + 1, i);
        }
#pragma unroll
      for (int i = 0; i < RING; ++i) slot_lr(t, i);
    }

    // ---- wavefronts that shared a unit add up their partial sums through LDS ----
    if (kw > 1) {
      float4_t* red = reinterpret_cast<float4_t*>(xs);
      __syncthreads();
      if (kwi != 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int m = 0; m < NS; ++m) red[((wave * MT + mt) * NS + m) * 64 + lane] = acc[0][mt][m];
      }
      __syncthreads();
      if (kwi == 0) {
        for (int j = 1; j < kw; ++j)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int m = 0; m < NS; ++m) acc[0][mt][m] += red[(((wave + j) * MT + mt) * NS + m) * 64 + lane];
      }
    }
    const KernArgs ka = kern_args();          // (what the end of a pass needs is read again: it would not fit the scalar registers until here)
    int ln = lane, tn = th, hn = ht, gn = grp;
    asm volatile("" : "+v"(ln), "+v"(tn), "+s"(hn), "+s"(gn));    // (addresses and conditions are made here, not kept in registers through the pass)
    if (!(HA && DUAL) && kwi != 0) continue;  // (the next pass starts with a barrier every wavefront reaches)
    // ---- epilogue: lane holds output columns 16*tile + 4*q .. +3 of token column c ----
    half4_t hs[TS][MT];                       // (this wavefront's h, for (h A2): zero without a unit)
#pragma unroll
    for (int ts = 0; ts < TS; ++ts)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) hs[ts][mt] = half4_t{0, 0, 0, 0};
    const int mine = kwi == 0 ? own : 0;
#pragma unroll
    for (int ts = 0; ts < TS; ++ts) {
      const int unit = gn + ts * groups;
      if (ts >= mine) continue;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int row = r + 16 * mt + c;
        if constexpr (DUAL) {
          // (a column without a row: its inputs are zeros, its (in A) some row's; nothing of it is stored)
          const int se = row_se[mt];          // the row's inputs were scaled by 2^se
          const int tile = t0 + unit;
          const float dn = pow2i(-se), up = pow2i(2 * se);
          const float i1 = lam[0] * dn, i3 = lam[1] * dn;
          half4_t hv;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float g = acc[ts][mt][0][i] * i1, u = acc[ts][mt][1][i] * i3;
            hv[i] = to_f16_sat(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u * up);
          }
          // h in operand order for the W2 kernel: columns f .. f+3 are half of one 16-byte unit
          const int f = tile * kTileN + 4 * q;
          if (row < cnt) *reinterpret_cast<half4_t*>(reinterpret_cast<_Float16*>(ka->out) + act_unit(f >> 3, r0 + row, ka->out_rt) * 8 + (f & 7)) = hv;
          hs[ts][mt] = hv;
        } else {
          if (row >= cnt) continue;
          const float i2 = lam[0] * pow2i(-2 * row_se[mt]);       // (h was stored times 2^(2 se))
#pragma unroll
          for (int m = 0; m < NS; ++m) {
            const int tile = t0 + 2 * unit + m;
            if (tile >= t1) continue;
            const size_t o = size_t(r0 + row) * ka->N + tile * kTileN + 4 * q;
            if (ka->partial != nullptr) {          // K-blocks: fp32 partial sums, added up by the combine or by reduce_kernel
              *reinterpret_cast<float4_t*>(ka->partial + size_t(kb) * ka->total_rows * ka->N + o) = acc[ts][mt][m] * i2;
            } else {
              uint2 yv;
              yv.x = f32x2_to_bf16x2(acc[ts][mt][m][0] * i2, acc[ts][mt][m][1] * i2);
              yv.y = f32x2_to_bf16x2(acc[ts][mt][m][2] * i2, acc[ts][mt][m][3] * i2);
              *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(ka->out) + o) = yv;
            }
          }
        }
      }
    }
    // (h A2) over the block's columns: the wavefronts' sums meet in LDS, in group order
    if (HA && DUAL && hn > 0) {
      float4_t* red = reinterpret_cast<float4_t*>(xs);
      __syncthreads();                       // (everyone is done with the activations and the fragments)
      if (kwi == 0) {
        // (the four columns of h a lane holds are its share of a 16x16x16 product's operand; not unrolled: what a
        // block runs once is fetched from memory while the wavefront waits)
#pragma unroll 1
        for (int rt = 0; rt < hn; ++rt) {
          uint2 w[TS];
#pragma unroll
          for (int ts = 0; ts < TS; ++ts) {
            const int tile = min(t0 + gn + ts * groups, t1 - 1);       // (without a unit: h is zero)
            const uint32_t at = ha_operand(rt, tile, ln, ka->N);
            if (a2_early) {
              const uint32_t own = at - (rt * (ka->N / 32 - n_u) + u0) * (kWave * 2);
              if (q3_a2) {
                const uint32_t* codes = reinterpret_cast<const uint32_t*>(p_lds + p_frags * 64);
                w[ts] = make_uint2(codes[own >> 1], codes[n_u * hn * kWave + (rt * n_q * 4 + tile / 4 - g0) * 16 + (ln & 15)]);
              } else {
                w[ts] = reinterpret_cast<const uint2*>(p_lds + p_frags * 64)[own];
              }
            } else if (q3_a2) {                // 3-bit pair: the unit's code dword and its metadata
              w[ts] = make_uint2(as_global<uint32_t>(uniform_ptr(ka->desc[e].af[2]))[at >> 1],
                                 as_global<uint32_t>(uniform_ptr(ka->desc[e].afm[2]))[(rt * (ka->N / 64) + tile / 4) * 16 + (ln & 15)]);
            } else {
              w[ts] = __builtin_bit_cast(uint2, as_global<u32x2>(uniform_ptr(ka->desc[e].af[2]))[at]);
            }
          }
          float4_t sum[MT];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) sum[mt] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ts = 0; ts < TS; ++ts) {
            if (q3_a2) w[ts] = q3_half_unit_a(w[ts].x, w[ts].y, (ln & 16) != 0);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) sum[mt] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4_t, w[ts]), hs[ts][mt], sum[mt], 0, 0, 0);
          }
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) red[((gn * hn + rt) * MT + mt) * 64 + ln] = sum[mt];
        }
      }
      __syncthreads();
      const int slot = pe.own, used = min(groups, units);
      for (int i = tn; i < hn * MT * 64; i += 64 * kWaves) {
        float4_t sum = float4_t{0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < used; j += 8) {    // (eight reads in flight)
          float4_t v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = red[min(j + u, used - 1) * hn * MT * 64 + i];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (j + u < used) sum += v[u];
        }
        const int row = r + 16 * ((i >> 6) % MT) + (i & 15), rt = (i >> 6) / MT;
        if (row < cnt)
          *reinterpret_cast<float4_t*>(ka->ha + ha_part(slot, ka->total_rows, r0 + row, 16 * rt + 4 * ((i >> 4) & 3))) = sum;
      }
    }
  }
}

template <int BITS, bool DUAL, bool Q3, bool HA>
__global__ __launch_bounds__(64 * kWaves, 4) void qgemm_decode_kernel(KArgs a) {
  extern __shared__ uint4 xs[];
  PlanEntry pe;
  if (a.plan != nullptr) {                   // shares by table (plan.h): one 32-byte entry per block
    const auto* src = reinterpret_cast<const __attribute__((address_space(4))) PlanEntry*>(reinterpret_cast<uintptr_t>(a.plan)) + blockIdx.x;
    pe.e = src->e; pe.t0 = src->t0; pe.t1 = src->t1; pe.r0 = src->r0; pe.cnt = src->cnt; pe.own = src->own; pe.slots = src->slots;
    if (pe.e < 0) return;
  } else {
    const int e = blockIdx.y, r0 = a.offsets ? a.offsets[e] : e * a.T;
    pe = plan_entry(e, blockIdx.x, gridDim.x, a.NT, r0, a.offsets ? a.offsets[e + 1] - r0 : a.T, 0);
  }
  if (pe.cnt == 0 || pe.t0 == pe.t1) return;
  if (pe.cnt <= 16) decode_body<BITS, DUAL, 1, Q3, HA>(a, xs, pe);
  else decode_body<BITS, DUAL, 2, Q3, HA>(a, xs, pe);
}

template <bool DUAL>
__global__ __launch_bounds__(1024) void xa_rows_kernel(KArgs a) {
  __shared__ float4_t red[32][64];
  xa_rows_body<DUAL, false, 16>(a, GroupedRows{a.offsets, a.row_pair, a.tok_exp, a.row_exp, a.top_k}, nullptr, blockIdx.x, blockIdx.y, blockIdx.z, 0, 1, red);
}

// (x A1 | x A3) from the bf16 tokens in a launch of its own: the same body, block size and summation
// order as the blocks of the preparing launch that normally do this, so that a layer whose factors
// arrive late (staged residency) gets the same bits.
__global__ __launch_bounds__(1024) void xa13_tokens_kernel(KArgs a, const uint16_t* __restrict__ x_bf16) {
  __shared__ float4_t red[32][64];
  xa_rows_body<true, true, 16>(a, GroupedRows{a.offsets, a.row_pair, a.tok_exp, a.row_exp, a.top_k}, x_bf16, blockIdx.x, blockIdx.y, 0, 0, 1, red);
}

// y_rows[R][n] = bf16(sum over K-blocks of partial[kb][R][n]), K-blocks in order (deterministic).
__global__ __launch_bounds__(256) void reduce_kernel(const float* __restrict__ partial, int kblocks, size_t stride,
                                                     size_t units, uint2* __restrict__ y) {
  const size_t u = size_t(blockIdx.x) * 256 + threadIdx.x;       // one unit = 4 outputs
  if (u >= units) return;
  float4_t sum = *reinterpret_cast<const float4_t*>(partial + u * 4);
  for (int kb = 1; kb < kblocks; ++kb) sum += *reinterpret_cast<const float4_t*>(partial + kb * stride + u * 4);
  uint2 v;
  v.x = f32x2_to_bf16x2(sum[0], sum[1]);
  v.y = f32x2_to_bf16x2(sum[2], sum[3]);
  y[u] = v;
}

// Bytes of the part sums of (h A2) where the fused launch leaves them for W2 (0: xa_rows_kernel makes (h A2) in between): both
// projections on this flavour, ranks up to 32, room for the parts, and few enough of them.  Every W2 block reads the parts of its
// rows, `slots` of 128 bytes a row: 100 KB cost it about 2 us, the launch in between 3 and 0.25 more per pass of 32 rows and 1000
// inputs (the FFN width).  The host does not know the counts: the parts are bounded for tokens that select half as many
// experts as they can (96 KB), and for tokens that all select the same (320 KB), each plus what the passes of the launch
// would cost.  Whole forward, launch in between -> part sums, us, in bounds: Mixtral T = 1 64.4 -> 60.9, T = 64 151.8 -> 146.3 (all
// tokens alike 124.0 -> 118.8), T = 160 289.8 -> 285.0; Qwen3 T = 16 72.6 -> 69.3, T = 64 103.4 -> 100.9; hidden 256, FFN 512, 8 experts,
// Top-2, T = 16 42.4 -> 40.3; 16 experts, Top-2, 2048 x 1024, T = 32 54.8 -> 51.9 (all tokens alike 50.7 -> 53.6).  Out of them: 4 experts, Top-1, 1536 x 896, T = 100 53 -> 63; 32 experts, Top-4, 2048 x 1408, T = 64, all tokens alike
// 105 -> 112; Qwen3 T = 256 311 -> 315.  At rank 64, with twice the parts and the sums of two steps, most shapes lose (Mixtral
// T = 32 138.9 -> 140.2, T = 160 299.5 -> 304.6, Qwen3 T = 128 172 -> 179).  Beside shared experts the launch in between is free, the side
// stream fills it: DeepSeek shape T = 1 80.5 -> 82.8 (without them T = 64 105.9 -> 101.2).
size_t ha_room(const FfnArgs& f) {
  if (f.offsets == nullptr || f.plan == nullptr || f.ha == nullptr || f.rank <= 0 || f.top_n <= 0 || f.rank > dec::kHaRank || f.n_shared > 0) return 0;
  const int NT = f.F / kTileN, pairs = f.T * f.top_k, kb = decode_w2_kblocks(f);
  const size_t room = size_t(ha_slots(plan_blocks(f.n_exp, pairs, NT, f.n_cu), NT)) * f.total_rows * kHaRank * 4;
  // `experts` of them share the pairs and the blocks of the fused launch: KB of parts that a W2 block reads, within `limit` or not
  auto within = [&](int experts, int limit) {
    const int rows = std::min(f.T, (pairs + experts - 1) / experts), passes = (rows + 31) / 32;
    const int slots = std::min(std::max(f.n_cu / experts, (NT + 31) / 32), NT);
    return slots * (rows <= 16 ? 16 : 32 * passes) / (8 * kb) <= limit + f.F * passes / 80;
  };
  return room <= f.ha_bytes && within(std::max(f.top_k, std::min(f.n_exp, pairs) / 2), 96) && within(f.top_k, 320) ? room : 0;
}

template <int BITS>
hipError_t launch_bits(const FfnArgs& f, hipStream_t s, int which) {
  int gs = 0;
  while ((1 << gs) < f.group) ++gs;
  KArgs a{};
  a.desc = f.desc; a.offsets = f.offsets; a.row_pair = f.row_pair; a.comp_rows = f.comp_rows;
  a.row_exp = f.row_exp; a.tok_exp = f.tok_exp;
  a.group_shift = gs; a.top_k = f.top_k; a.top_n = f.top_n; a.T = f.T;
  a.rank = f.rank; a.rpad = f.rpad; a.ls = (f.rank + 31) / 32; a.total_rows = f.total_rows;
  const bool comp = f.rank > 0 && f.top_n > 0 && f.row_pair != nullptr;
  // shared experts (no routing): a (blocks per expert x experts) grid; the blocks of the experts
  // together should cover the CUs, and a block takes at most 32 n-tiles
  auto blocks_per_expert = [&](int NT, int kblocks) {
    int g = (f.n_cu + f.n_exp * kblocks - 1) / (f.n_exp * kblocks);
    g = std::max(g, (NT + 31) / 32);
    return std::min(g, NT);
  };
  // activations + the (in A) fragments of small ranks
  const size_t lds = size_t(kLdsUnits + kSpareUnits) * 16;
  // routed experts: the blocks are shared out among the experts that have rows by the tables the
  // launch that prepared the activations has left (plan.h)
  const bool by_table = f.offsets != nullptr && f.plan != nullptr;
  const int pairs = f.T * f.top_k;
  // (the kernels that can dequantize 3-bit factor pairs, where the layer holds any)
  const bool q3 = comp && f.q3;
  // (h A2) made by the fused launch's blocks themselves
  const bool ha = comp && which == 3 && ha_room(f) > 0;
  a.ha = ha ? f.ha : nullptr;
  auto pick = [&](auto DUAL_) {
    constexpr bool DUAL = decltype(DUAL_)::value;
    if (ha) return q3 ? qgemm_decode_kernel<BITS, DUAL, true, true> : qgemm_decode_kernel<BITS, DUAL, false, true>;
    return q3 ? qgemm_decode_kernel<BITS, DUAL, true, false> : qgemm_decode_kernel<BITS, DUAL, false, false>;
  };
  auto k13 = pick(std::true_type{}), k2 = pick(std::false_type{});

  if (which & 1) {
    // W1 | W3 with the SwiGLU epilogue
    a.in = f.xh; a.out = f.h; a.K = f.H; a.N = f.F; a.NT = f.F / kTileN;
    a.in_rt = f.x_rt; a.out_rt = f.h_rt;
    a.KS = padded_k(f.H) / kTileK; a.G = padded_k(f.H) / f.group;
    a.p = f.p13; a.p_tokens = f.p_tokens; a.row_tok = f.row_tok; a.n_exp = f.n_exp;
    a.kb_steps = a.KS; a.partial = nullptr;
    // ((x A1 | x A3) has been made by the launch that prepared the activations, unless it is asked for here)
    if (comp && f.xa13_here)
      hipLaunchKernelGGL(xa13_tokens_kernel, dim3(2 * a.rpad / 16, f.n_exp), dim3(1024), 0, s, a, (const uint16_t*)f.x_tokens);
    if (f.marks) (void)hipEventRecord(f.marks[0], s);
    if (by_table) {
      a.plan = f.plan;
      hipLaunchKernelGGL(k13, dim3(plan_blocks(f.n_exp, pairs, a.NT, f.n_cu), 1, 1), dim3(64 * kWaves), lds, s, a);
      a.plan = nullptr;
    } else {
      hipLaunchKernelGGL(k13, dim3(blocks_per_expert(a.NT, 1), f.n_exp, 1), dim3(64 * kWaves), lds, s, a);
    }
    if (f.marks) (void)hipEventRecord(f.marks[1], s);
  }
  if (which & 2) {
    // W2
    a.in = f.h; a.out = f.y_rows; a.K = f.F; a.N = f.H; a.NT = f.H / kTileN;
    a.in_rt = f.h_rt; a.out_rt = 0;
    a.KS = padded_k(f.F) / kTileK; a.G = padded_k(f.F) / f.group;
    a.p = f.p2; a.p_tokens = 0;
    // a long K (many phases of staged activations) is split into K-blocks of one 16-k-step phase each;
    // their fp32 partial outputs are added by the combine, or by reduce_kernel when y_rows is wanted.
    // The rank-r term is linear in (h A2): every K-block adds B2 times the part of (h A2) over its own
    // k-steps, so (h A2) needs no sum over the K-blocks either.
    const int kblocks = decode_w2_kblocks(f);
    a.kb_steps = (a.KS + kblocks - 1) / kblocks;
    a.partial = kblocks > 1 ? f.y_part : nullptr;
    if (comp && !ha) hipLaunchKernelGGL(xa_rows_kernel<false>, dim3(a.rpad / 16, f.n_exp, kblocks), dim3(1024), 0, s, a);
    if (f.marks) (void)hipEventRecord(f.marks[2], s);
    if (by_table) {
      a.plan = f.plan2;                      // (every K-block uses the same shares)
      const int B = plan_blocks(f.n_exp, pairs, a.NT, (f.n_cu + kblocks - 1) / kblocks);
      hipLaunchKernelGGL(k2, dim3(B, 1, kblocks), dim3(64 * kWaves), lds, s, a);
      a.plan = nullptr;
    } else {
      hipLaunchKernelGGL(k2, dim3(blocks_per_expert(a.NT, kblocks), f.n_exp, kblocks), dim3(64 * kWaves), lds, s, a);
    }
    if (kblocks > 1 && !f.keep_partials) {
      const size_t units = size_t(f.total_rows) * f.H / 4;
      hipLaunchKernelGGL(reduce_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, s, f.y_part, kblocks,
                         size_t(f.total_rows) * f.H, units, reinterpret_cast<uint2*>(f.y_rows));
    }
    if (f.marks) (void)hipEventRecord(f.marks[3], s);
  }
  return hipGetLastError();
}

}  // namespace

size_t decode_ha_bytes(const FfnArgs& f) { return expert_ffn_path(f) == 0 ? ha_room(f) : 0; }

// K-blocks of the decode flavour's W2 launch: one 16-k-step phase each, at most kMaxKBlocks
int decode_w2_kblocks(const FfnArgs& f) {
  const int KS2 = padded_k(f.F) / kTileK;
  return f.y_part ? std::min(kMaxKBlocks, (KS2 + 15) / 16) : 1;
}

void decode_plan_specs(const FfnArgs& f, int which, PlanSpec& p13, PlanSpec& p2) {
  const int pairs = f.T * f.top_k, NT13 = f.F / kTileN, NT2 = f.H / kTileN;
  if (which & 1) p13 = PlanSpec{plan_blocks(f.n_exp, pairs, NT13, f.n_cu), NT13, f.n_cu, f.plan};
  if (which & 2) {
    const int kb2 = decode_w2_kblocks(f);
    const int target2 = (f.n_cu + kb2 - 1) / kb2;
    p2 = PlanSpec{plan_blocks(f.n_exp, pairs, NT2, target2), NT2, target2, f.plan2};
  }
}

template <int BITS> static hipError_t decode_init_bits() {
  const void* fns[8] = {
      reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, true, false, false>), reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, false, false, false>),
      reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, true, true, false>), reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, false, true, false>),
      reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, true, false, true>), reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, false, false, true>),
      reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, true, true, true>), reinterpret_cast<const void*>(&qgemm_decode_kernel<BITS, false, true, true>)};
  for (const void* fn : fns) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (kLdsUnits + kSpareUnits) * 16);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t decode_init_device() {
  // 128 KB of activations + 32 KB of (in A) fragments = all 160 KB of a CU
  hipError_t e = decode_init_bits<2>();
  if (e == hipSuccess) e = decode_init_bits<3>();
  if (e == hipSuccess) e = decode_init_bits<4>();
  return e;
}

hipError_t launch_decode_ffn(const FfnArgs& f, hipStream_t s, int which) {
  switch (f.bits) {
    case 2: return launch_bits<2>(f, s, which);
    case 3: return launch_bits<3>(f, s, which);
    case 4: return launch_bits<4>(f, s, which);
  }
  return hipErrorInvalidValue;
}

}  // namespace lrc
