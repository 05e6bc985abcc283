// Expert FFN on grouped rows (Sections 2.3 and 3.2), many-rows flavour (prefill):
//   g = x D1 + c (x A1) B1,  u = x D3 + c (x A3) B3,  h = silu(g) * u,  y = h D2 + c (h A2) B2
// with D = Qinv(Q(W)) unpacked from the bit-packed codes inside the wavefront's registers and
// c = 1 only for rows that hold a Top-n (token, expert) pair.
//
// With hundreds of rows per expert the work is a grouped GEMM and the matrix cores are the bound.
// Kernel design (gfx950):
//   - a block of 4 wavefronts owns 128 rows of one expert x 128 output columns (of both W1 and W3 in
//     the fused kernel; 128 or 256 columns of W2); a wavefront owns two n-tiles (16 columns each; four
//     of W2) for all 128 rows, so a tile of weights unpacked once in registers (unpack.h) feeds all
//     the rows.  Two blocks share a CU (80 KB of LDS and one wavefront per SIMD each): what a block
//     waits for on its own (its first loads, the barriers, its epilogue) is time the other one
//     multiplies in.  With one block of 8 wavefronts per CU that time was lost: the fused launch took
//     272 us and W2 194 on the Qwen3 shape at T = 4096 (8 and 3 k-steps per block), 248 and 150 so;
//     a long K (Mixtral, 16 and 56 k-steps) gains 2 %;
//   - the products run on v_mfma_f32_32x32x16_f16 (the same peak rate as the 16x16x32 shape, half
//     as many MFMA and LDS-read instructions per flop): two streams of 16 output columns that meet
//     the same activations (W1 and W3 of one n-tile, or two n-tiles of W2) become the 32 rows of one
//     A operand by a swap of 16-lane rows between their registers, which puts the same inputs of both
//     streams side by side; the activations are staged as fragments of 32 rows;
//   - the packed weights never touch LDS: each wavefront loads its tiles HBM -> registers, the next
//     k-step's into the registers of the current one as soon as its last code is unpacked (a second
//     set of registers does not fit beside 128 accumulators at 3 and 4 bits; at 4 bits the fused kernel and the one
//     with four n-tiles of W2 per wavefront spill 92 to 100 bytes per lane as it is), chunks of fewer rows into a second
//     set a whole k-step ahead (a dword of every line of the next k-step's tiles requested ahead, for the L2, was
//     slower instead of faster on full chunks: Mixtral shape T = 2048 1555 -> 1606 us);
//   - the activations of half a k-step (128 rows x 128 columns, 32 KB, MFMA operand order) are
//     double-buffered in LDS: the copy of the next half goes from memory straight to LDS (no
//     registers) while the current one is multiplied; one barrier per half;
//   - the rank-r term is extra steps: the B factor's 32-wide units take the place of the codes and
//     meet (in A), which xa_kernel (or xa_tile_kernel and xa_join_kernel) has left in global memory; its first fragments are
//     copied into LDS at the start.
// Experts with few rows (decode) take the other flavour, ffn_decode.hip.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "decode_index.h"
#include "factor_q3.h"
#include "ffn_common.h"
#include "plan.h"

namespace lrc {

namespace {

using namespace ffn;

constexpr int kByLengthRows = 64;         // rows an expert from which W1|W3 takes the chunks by length (plan.h)
constexpr int kGemmWaves = 4;             // wavefronts per block of the grouped GEMM (two blocks per CU)
constexpr int kBM = 128;                  // rows of an expert per block
constexpr int kHalfUnits = kBM / 16 * 4 * 64;   // 16-byte units of half a k-step of activations (32 KB)
constexpr int kGemmLdsUnits = 5120;       // LDS of a grouped-GEMM block: 80 KB, half of a CU's
struct Chunk { int e, r0, cnt, r; };
// Work item `item` of an (in A) launch -> (expert, first row of its chunk of ROWS compact rows): the items enumerate the chunks of the
// experts in order.  (How many compact rows an expert has is counted by the launch that makes the tables of plan.h, so these
// items are found here.)  64 experts at a time, read together: every lane counts the chunks of one expert, a prefix sum
// over the wavefront finds the one that holds the item (every wavefront of the block does the same).
template <int ROWS>
__device__ inline bool find_chunk(const KArgs& a, int item, Chunk& c) {
  constexpr int kGroups = 4;                // (at most 256 experts)
  const int lane = threadIdx.x & 63;
  int r0[kGroups], cnt[kGroups];
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    r0[g] = cnt[g] = 0;
    if (64 * g >= a.n_exp) continue;
    const int e = min(64 * g + lane, a.n_exp - 1);
    r0[g] = a.offsets[e]; cnt[g] = a.comp_rows[e];
  }
  int base = 0;
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    if (64 * g >= a.n_exp) continue;
    const int n = 64 * g + lane < a.n_exp ? (cnt[g] + ROWS - 1) / ROWS : 0, incl = wave_scan(n), total = lane_value(incl, 63);
    if (item < base + total) {
      const int first = __ffsll(__ballot(base + incl > item)) - 1;
      c.e = 64 * g + first;
      c.r0 = lane_value(r0[g], first); c.cnt = lane_value(cnt[g], first);
      c.r = (item - base - lane_value(incl - n, first)) * ROWS;
      return true;
    }
    base += total;
  }
  return false;
}

static_assert(kBM == kChunkRows, "the chunk tables' rows");

typedef float float16_t __attribute__((ext_vector_type(16)));
constexpr int kRP = kBM / 32;             // 32-row fragments ("row pairs") of a chunk

// fn(std::integral_constant<int, 0>{}) ... fn(std::integral_constant<int, N - 1>{})
template <int... I, class Fn> __device__ inline void static_for_impl(std::integer_sequence<int, I...>, Fn&& fn) {
  (fn(std::integral_constant<int, I>{}), ...);
}
template <int N, class Fn> __device__ inline void static_for(Fn&& fn) { static_for_impl(std::make_integer_sequence<int, N>{}, fn); }

// Half a k-step (sub-steps 4 half .. 4 half + 3) as fragments for the 32x32x16 products: fragment (row
// pair rp, sub-step s, operand p) at unit ((rp * 4 + s % 4) * 2 + p) * 64; lane l holds, of row
// 32 rp + l % 32, the 8 inputs of lane group q = p + 2 (l / 32) of sub-step s.  (After the row swap,
// operand p of a sub-step holds in lanes 0..31 the weights of lane group q = p and in lanes 32..63
// those of q = p + 2.)  Wavefront w of the block's four copies the fragments of sub-step 4 half + w.
// Only the first rp_n row pairs are copied (the others hold no rows of the expert and are not read).
// A lane's address is a wave-uniform base (k-step, sub-step, operand, first row of the chunk) plus a
// 32-bit offset that is the same for every k-step: `full` for the row pairs before the last one
// (512 bytes apart), `last` for the last one, whose rows past the chunk's last one read the zero rows
// at the end of the buffer (see staged_row).
struct StageOffsets { uint32_t full, last; };
__device__ inline StageOffsets stage_offsets(const KArgs& a, int rin, int rows, int rp_n, int lane) {
  const int n = lane & 31, R = 32 * (rp_n - 1) + n;
  const uint32_t q2 = (lane >> 5) ? 2u * uint32_t(a.in_rt) : 0u;      // lane group q = p + 2 (l / 32)
  return {(q2 + uint32_t(n)) * 16u, (q2 + uint32_t(R < rows ? R : a.in_rt - dec::kZeroRows + (n & 15) - rin)) * 16u};
}
template <int RPN>
__device__ inline void stage_half(const KArgs& a, uint4* buf, int ks, int half, int rin, const StageOffsets& so, int wave, int lane) {
  const int s = 4 * half + wave;
  const uint32_t group = uint32_t(a.in_rt) * 16u;       // bytes of one lane group's units
  const uint8_t* base = reinterpret_cast<const uint8_t*>(a.in) + (size_t(ks) * 8 + s) * 4 * group + size_t(rin) * 16;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, 0xffffffffu, 0x00020000);
  const int qv = a.K / kLaneK - 4 * ks;                 // lane groups of this k-step that lie below K
  static_for<2>([&](auto P) {
    constexpr int p = decltype(P)::value;
    // K is a multiple of 64: past it the padded weights are exact zeros and any finite activation will
    // do; lanes that would read there take a lane group below K instead
    uint32_t back = (p + 2 < qv || lane < 32) ? 0u : 2u * group;
    asm volatile("" : "+v"(back));                      // (made here, not kept in registers for every case)
    const int soff = p < qv ? int(p * group) : 0;
    const int full = int(so.full - back), last = int(so.last - back);
    static_for<RPN>([&](auto Rp) {
      constexpr int rp = decltype(Rp)::value;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, reinterpret_cast<__attribute__((address_space(3))) void*>(reinterpret_cast<uintptr_t>(buf + ((rp * 4 + wave) * 2 + p) * 64)), 16,
          rp == RPN - 1 ? last : full, rp == RPN - 1 ? soff : soff + rp * 512, 0, 0);   // (an immediate offset would move the LDS address too)
    });
  });
}

// (in A) fragments of a rank step for the 32x32x16 products: V variants per rank step (4 fused, 2
// for W2).  Variant v, lane l (half h = l / 32) holds the 8 rank indices of group `grp` of
// projection m's (in A).  The fused projections meet different (in A): the A operand of variant v
// keeps W1's columns in input half h = v & 1 and W3's in the other, so the fragment holds A1's part
// where W1 sits and A3's where W3 sits.
__device__ inline void rank_frag_source(int v, int lane, bool dual, int& m, int& grp) {
  const int h = lane >> 5;
  if (dual) { m = h ^ (v & 1); grp = (v >> 1) + 2 * h; }
  else { m = 0; grp = v + 2 * h; }
}

// Codes and metadata of one k-step of a wavefront's two n-tiles.
template <int BITS, int NM, int NTW> struct Slot2 { Slot<BITS, NM> t[NTW]; };

// Q3: some factor pair of the layer is held at 3 bits (layout.h): the rank steps of such a pair fetch
// the unit's code dword and the lane's half of the unit's metadata with loads of their own, one rank
// step ahead (the k-loop is that of the plain kernel), and dequantize them into the
// fp16 unit before it is used.
template <int BITS, bool DUAL, int NTW, bool Q3 = false>
__global__ __launch_bounds__(64 * kGemmWaves, 2) void qgemm_tile_kernel(KArgs a) {
  extern __shared__ uint4 xs[];           // two halves of a k-step of activations, then (in A) fragments
  constexpr int WAVES = kGemmWaves;
  constexpr int NM = DUAL ? 2 : 1;
  constexpr int kNTW = NTW;                              // n-tiles per wavefront
  constexpr int DW = 2 * BITS;
  constexpr int NC = Extract<BITS>::kClasses;
  Chunk ch;
  int item = blockIdx.y, bx = blockIdx.x;
  if (a.by_xcd) {                          // block b runs on XCD b % 8: chunk 8 i + b % 8, its column blocks one after the other
                                           // (the launch has a multiple of 8 chunks)
    const int b = blockIdx.y * gridDim.x + blockIdx.x, j = b >> 3, round = j / (int)gridDim.x;
    bx = j - round * (int)gridDim.x;
    item = 8 * round + (b & 7);
  }
  if (a.plan != nullptr) {                 // (one scalar load: the preparing launch has made the table)
    const auto* at = reinterpret_cast<const __attribute__((address_space(4))) ChunkEntry*>(reinterpret_cast<uintptr_t>(a.plan)) + item;
    ch.e = at->e; ch.r0 = at->r0; ch.cnt = at->cnt; ch.r = at->r;
    if (ch.e < 0) return;
  } else {                                 // shared experts: every one has the same rows
    const int per = (a.T + kBM - 1) / kBM;
    ch.e = item / per; ch.r = (item - ch.e * per) * kBM; ch.r0 = ch.e * a.T; ch.cnt = a.T;
    if (ch.e >= a.n_exp) return;
  }
  const int e = ch.e, r0 = ch.r0, cnt = ch.cnt, r = ch.r;
  // the expert's table entry: everything of it that the block needs, requested together
  const ConstDesc d = const_desc(a.desc + e);
  const int has_factors = d->has_factors, q3 = d->q3;
  const int comp = *const_i32((a.comp_rows ? a.comp_rows : &a.desc->q3) + (a.comp_rows ? e : 0));
  const int th = threadIdx.x, lane = th & 63;
  const int wave = __builtin_amdgcn_readfirstlane(th >> 6);
  const int q = lane >> 4, c = lane & 15;
  const int tdw = kWave * DW;
  const int tile0 = (bx * WAVES + wave) * kNTW;

  const int code_bytes = a.KS * a.NT * tdw * 4, meta_bytes = a.G * a.NT * kTileN * 4;
  const uint32_t* codes[NM];
  const uint32_t* metas[NM];
  const _Float16* bfs[NM];
  int ranks[NM];
  float lam[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const int mat = DUAL ? m : 2;
    codes[m] = d->codes[mat]; metas[m] = d->meta[mat]; bfs[m] = d->bf[mat]; ranks[m] = d->rank[mat]; lam[m] = d->inv_lambda[mat];
  }
  const bool lowrank = a.rank > 0 && has_factors != 0 && a.row_pair != nullptr && comp > 0;
  // every projection has the rank of its own factor pair (Section 3.1): the expert runs the rank
  // steps of the larger one, a resource of the size its rank fills makes the other read zeros
  int LSm[NM];
  __amdgpu_buffer_rsrc_t code_rs[NM], meta_rs[NM], bf_rs[NM];
  bool q3m[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    LSm[m] = lowrank ? int(uint32_t(min(ranks[m], a.rank) + 31) / 32) : 0;
    q3m[m] = Q3 && ((q3 >> (DUAL ? m : 2)) & 1) != 0;
    code_rs[m] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(codes[m]), 0, code_bytes, 0x00020000);
    meta_rs[m] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(metas[m]), 0, meta_bytes, 0x00020000);
    // (a 3-bit pair's rank steps read zeros here and fetch their units themselves)
    bf_rs[m] = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(bfs[m]), 0, q3m[m] ? 0 : a.NT * LSm[m] * 1024, 0x00020000);
  }
  const int LS = max(LSm[0], LSm[NM - 1]);
  const int gps = kTileK >> a.group_shift;               // groups per k-step
  const int meta_lane = ((q * kLaneK) >> a.group_shift) * (a.NT * kTileN * 4) + c * 4;

  // The packed tiles of a k-step: one 32-bit lane offset per kind of load, everything else scalar.
  // (An n-tile past the last one is clamped: its columns are never stored.)
  // (kFetchLoads: the loads of one fetch, which the wait in the middle of a k-step with two slots leaves in flight.)
  constexpr int kCodeLoads = BITS == 2 ? 1 : 2, kTileLoads = kCodeLoads + 1;    // of a tile: codes, then a dword of metadata
  constexpr int kFetchLoads = kNTW * NM * kTileLoads;
  const int lane16 = lane * 16, lane1 = 1024 + lane * (BITS == 3 ? 8 : 16);
  auto fetch = [&](int step, Slot2<BITS, NM, kNTW>& sl) {
#pragma unroll
    for (int t = 0; t < kNTW; ++t) {
      const int tile = min(tile0 + t, a.NT - 1);
      const int tile_off = (step * a.NT + tile) * (tdw * 4), meta_off = (step * gps * a.NT + tile) * (kTileN * 4);
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        Slot<BITS, NM>& s1 = sl.t[t];
        static_for<kTileLoads>([&](auto I) {               // (one load each)
          constexpr int i = decltype(I)::value;
          if constexpr (i == kCodeLoads) {
            s1.mw[m] = __builtin_amdgcn_raw_buffer_load_b32(meta_rs[m], meta_lane, meta_off, 0);
          } else if constexpr (i == 1 && BITS == 3) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(code_rs[m], lane1, tile_off, 0);
            s1.cw[m][4] = v[0]; s1.cw[m][5] = v[1];
          } else {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(code_rs[m], i == 0 ? lane16 : lane1, tile_off, 0);
            s1.cw[m][4 * i] = v[0]; s1.cw[m][4 * i + 1] = v[1]; s1.cw[m][4 * i + 2] = v[2]; s1.cw[m][4 * i + 3] = v[3];
          }
        });
      }
    }
  };
  // The B-factor units of a rank step: range-checked lane offsets, so that a stream past its own rank
  // (and one whose pair is held at 3 bits) reads zeros.
  auto fetch_rank = [&](int st, Slot2<BITS, NM, kNTW>& sl) {
#pragma unroll
    for (int t = 0; t < kNTW; ++t) {
      int unit = st * a.NT + min(tile0 + t, a.NT - 1);
      asm volatile("" : "+s"(unit));       // (the offsets are made here, not kept in registers through the k-steps)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const u32x4 v0 = __builtin_amdgcn_raw_buffer_load_b128(bf_rs[m], unit * 1024 + lane16, 0, 0);
        Slot<BITS, NM>& s1 = sl.t[t];
        s1.cw[m][0] = v0[0]; s1.cw[m][1] = v0[1]; s1.cw[m][2] = v0[2]; s1.cw[m][3] = v0[3];
      }
    }
  };

  // first input row of this chunk (shared experts all read the token rows 0..T-1)
  const int rin = ((DUAL && !a.offsets) ? 0 : r0) + r;

  // Streams (16 output columns that meet the same activations) are paired into the 32 rows of an A
  // operand: (W1, W3) of n-tile j in the fused kernel, n-tiles 2j and 2j + 1 otherwise.
  constexpr int NPAIR = kNTW * NM / 2;
  // acc[j][rp]: the 32 x 32 result of pair j and row pair rp; register i of lane l holds, of row
  // 32 rp + l % 32, stream i / 8, column 8 ((i / 4) % 2) + 4 (l / 32) + i % 4 of the stream's n-tile
  float16_t acc[NPAIR][kRP];
  auto clear = [&](auto FROM_) {             // (those of row pairs FROM ..: unused ones are cleared after the k-steps, and take no registers in them)
#pragma unroll
    for (int j = 0; j < NPAIR; ++j)
#pragma unroll
      for (int rp = decltype(FROM_)::value; rp < kRP; ++rp)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[j][rp][i] = 0.f;
  };
  clear(std::integral_constant<int, 0>{});
  const int rp_n = min(kRP, (cnt - r + 31) >> 5);         // row pairs that hold rows of this expert

  // the two streams of pair j: (tile slot, projection)
  auto pair_stream = [](int j, int side, int& t, int& m) {
    if constexpr (DUAL) { t = j; m = side; }
    else { t = 2 * j + side; m = 0; }
  };

  // Half a k-step (four sub-steps) for a chunk with RPN row pairs that hold rows.  A sub-step (32
  // inputs per lane group) has F = 2 RPN fragments of activations, operand p major; fragment g of the
  // half's 4 F is read from LDS kPF fragments ahead of its two MFMAs (one per pair), and the weights
  // of the next sub-step are unpacked, a piece per fragment, behind the MFMAs of the current one, so
  // that the matrix pipe, the LDS reads and the unpacking run side by side within a wavefront.
  constexpr int kPF = BITS == 2 ? 2 : 1;   // (1 to 4 measure alike; 3 and 4 bits need the registers)
  uint32_t sc[kNTW][NM][NC];               // the slot's metadata, one dword per field class
  uint32_t v[NPAIR][2][4];                 // operand registers of the next sub-step, before the swap
  constexpr int PIECES = NPAIR * 4;
  // Row pairs up to which the next k-step's tiles have a slot of their own.  At 4 bits one: with two the registers run out
  // (whole layer, second slot up to two / one row pairs, us: Mixtral shape T = 200 369 / 354, DeepSeek shape
  // T = 512 220 / 210, 700 248 / 236, Qwen3 shape T = 4096 575 / 565; with none 352, 206, 234 and 577).
  constexpr int kTwoSlots = BITS == 4 ? 1 : 3;
  auto unpack_piece = [&](const Slot2<BITS, NM, kNTW>& sl, int s, int piece) {
    const int j = piece / 4, i = piece % 4;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      int t, m;
      pair_stream(j, side, t, m);
      v[j][side][i] = dequant(Extract<BITS>::field(sl.t[t].cw[m], 4 * s + i), sc[t][m][Extract<BITS>::cls(4 * s + i)]);
    }
  };
  auto compute = [&](auto RPN_, auto HALF_, Slot2<BITS, NM, kNTW>& sl, auto&& request) {
    constexpr int RPN = decltype(RPN_)::value, HALF = decltype(HALF_)::value;
    constexpr int F = 2 * RPN, G = 4 * F;
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>(xs + lane));
    // LDS byte offset of fragment g of the half: sub-step g / F, operand (g % F) / RPN, row pair (g % F) % RPN
    auto frag_off = [](int g) constexpr { return HALF * kHalfUnits * 16 + (g / F) * 2048 + ((g % F) % RPN) * 8192 + ((g % F) / RPN) * 1024; };
    half8_t xf[kPF + 1];
    static_for<(kPF < G ? kPF : G)>([&](auto g) { xf[g] = lds_read16<frag_off(g)>(base); });
    if constexpr (HALF == 0) {             // the slot's metadata and its first sub-step
#pragma unroll
      for (int t = 0; t < kNTW; ++t)
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          sc[t][m][0] = sl.t[t].mw[m];
#pragma unroll
          for (int p = 1; p < NC; ++p) sc[t][m][p] = meta_class<BITS>(sc[t][m][p - 1]);
        }
      static_for<PIECES>([&](auto pc) { unpack_piece(sl, 0, pc); });
    }
    static_for<4>([&](auto S) {
      constexpr int sl4 = decltype(S)::value, s = 4 * HALF + sl4;
      // rows of 16 lanes swapped between the two streams of a pair: operand 0 = lane groups q = 0, 2
      // of both streams side by side, operand 1 = q = 1, 3
      uint32_t A[2][NPAIR][4];
#pragma unroll
      for (int j = 0; j < NPAIR; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const auto sw = __builtin_amdgcn_permlane16_swap(v[j][0][i], v[j][1][i], false, false);
          A[0][j][i] = sw[0]; A[1][j][i] = sw[1];
        }
      if constexpr (s == 7) request();     // (every code of the slot has been unpacked: the next k-step's take its registers)
      __builtin_amdgcn_sched_barrier(0);
      static_for<F>([&](auto Fi) {
        constexpr int f = decltype(Fi)::value, g = sl4 * F + f, p = f / RPN, rp = f % RPN;
        if constexpr (g + kPF < G) xf[(g + kPF) % (kPF + 1)] = lds_read16<frag_off(g + kPF)>(base);
        lds_wait<(G - 1 - g < kPF ? G - 1 - g : kPF)>(xf[g % (kPF + 1)]);
#pragma unroll
        for (int j = 0; j < NPAIR; ++j) {
          const half8_t av = __builtin_bit_cast(half8_t, make_uint4(A[p][j][0], A[p][j][1], A[p][j][2], A[p][j][3]));
          acc[j][rp] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, xf[g % (kPF + 1)], acc[j][rp], 0, 0, 0);
        }
        if constexpr (s < 7) {
#pragma unroll
          for (int pc = PIECES * f / F; pc < PIECES * (f + 1) / F; ++pc) unpack_piece(sl, s + 1, pc);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };

  // ---- prologue: the first half k-step of activations, the first tiles, and the (in A) fragments of
  //      the first rank steps.  (in A) of the chunk's rows is fp16 row-major in global memory
  //      (xa_kernel has scaled it and zeroed the rows without the term); fragment (rank step st,
  //      variant v, row pair rp) sits at unit ((st * V + v) * 4 + rp) * 64 of its region
  //      (rank_frag_source).  The 16 KB behind the activations hold kRankFirst rank steps: ranks up
  //      to 32 (fused) or 64; later ones take the place of the activations, kRankChunk at a time.
  constexpr int V = DUAL ? 4 : 2;
  constexpr int kRankFirst = (kGemmLdsUnits - 2 * kHalfUnits) / (V * kRP * 64), kRankChunk = 2 * kHalfUnits / (V * kRP * 64);
  auto stage_rank = [&](uint4* region, int c0, int c1) {
    const _Float16* P = reinterpret_cast<const _Float16*>(a.p);
    const int pitch = NM * a.ls * 32;                                // halves per row
    for (int f = wave; f < (c1 - c0) * V * kRP; f += WAVES) {
      const int rp = f % kRP, g = f / kRP, vi = g % V, sl = g / V;
      int m, grp;
      rank_frag_source(vi, lane, DUAL, m, grp);
      const int row = min(r0 + r + 32 * rp + (lane & 31), a.total_rows - 1);
      const _Float16* src = P + size_t(row) * pitch + m * a.ls * 32 + 32 * (c0 + sl) + 8 * grp;
      __builtin_amdgcn_global_load_lds(
          reinterpret_cast<const __attribute__((address_space(1))) void*>(reinterpret_cast<uintptr_t>(src)),
          reinterpret_cast<__attribute__((address_space(3))) void*>(reinterpret_cast<uintptr_t>(region + ((size_t(sl) * V + vi) * kRP + rp) * 64)), 16, 0, 0);
    }
  };
  const StageOffsets so = stage_offsets(a, rin, cnt - r, rp_n, lane);
  // (the activations need nothing of the expert's table entry)
  if (rp_n == 4) stage_half<4>(a, xs, 0, 0, rin, so, wave, lane);
  else if (rp_n == 3) stage_half<3>(a, xs, 0, 0, rin, so, wave, lane);
  else if (rp_n == 2) stage_half<2>(a, xs, 0, 0, rin, so, wave, lane);
  else stage_half<1>(a, xs, 0, 0, rin, so, wave, lane);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int m = 0; m < NM; ++m) asm volatile("" : "+s"(lam[m]));       // (read here, with the rest: not again in front of the k-steps, whose waits count loads)
  Slot2<BITS, NM, kNTW> cur;
  fetch(0, cur);
  if (LS > 0) stage_rank(xs + 2 * kHalfUnits, 0, min(LS, kRankFirst));
  wait_loads_barrier();

  // ---- the k-steps, in halves: while one half of the activations is multiplied, the next half is
  //      copied into the other half of the buffer (free since the last barrier); the next k-step's
  //      tiles are requested at the start of a k-step.  One copy of the loop per number of row pairs,
  //      so that every count is static.
  const int steps = a.KS;
  auto k_loop = [&](auto RPN_) {
    constexpr int RPN = decltype(RPN_)::value;
    // Up to kTwoSlots row pairs leave registers for a second slot: the next k-step's tiles are requested a whole k-step ahead
    // instead of an eighth (which a cold weight's latency exceeds by far), and the wait in the middle of
    // the k-step leaves them in flight.
    if constexpr (RPN <= kTwoSlots) {
      Slot2<BITS, NM, kNTW> nxt;
      auto one = [&](int step, Slot2<BITS, NM, kNTW>& now, Slot2<BITS, NM, kNTW>& then) {
        stage_half<RPN>(a, xs + kHalfUnits, step, 1, rin, so, wave, lane);
        __builtin_amdgcn_sched_barrier(0);               // (in this order: the wait below counts from the last)
        fetch(min(step + 1, steps - 1), then);
        __builtin_amdgcn_sched_barrier(0);
        compute(RPN_, std::integral_constant<int, 0>{}, now, [] {});
        wait_loads_barrier_but<kFetchLoads>();
        if (step + 1 < steps) stage_half<RPN>(a, xs, step + 1, 0, rin, so, wave, lane);
        __builtin_amdgcn_sched_barrier(0);
        compute(RPN_, std::integral_constant<int, 1>{}, now, [] {});
        wait_loads_barrier();
      };
      for (int step = 0; step < steps; step += 2) {
        one(step, cur, nxt);
        if (step + 1 < steps) one(step + 1, nxt, cur);
      }
      return;
    }
    for (int step = 0; step < steps; ++step) {
      stage_half<RPN>(a, xs + kHalfUnits, step, 1, rin, so, wave, lane);
      __builtin_amdgcn_sched_barrier(0);
      compute(RPN_, std::integral_constant<int, 0>{}, cur, [] {});
      wait_loads_barrier();
      if (step + 1 < steps) stage_half<RPN>(a, xs, step + 1, 0, rin, so, wave, lane);
      __builtin_amdgcn_sched_barrier(0);
      compute(RPN_, std::integral_constant<int, 1>{}, cur, [&] {
        if (step + 1 < steps) fetch(step + 1, cur);
      });
      wait_loads_barrier();
    }
  };
  if (rp_n == 4) k_loop(std::integral_constant<int, 4>{});
  else if (rp_n == 3) { k_loop(std::integral_constant<int, 3>{}); clear(std::integral_constant<int, 3>{}); }
  else if (rp_n == 2) { k_loop(std::integral_constant<int, 2>{}); clear(std::integral_constant<int, 2>{}); }
  else { k_loop(std::integral_constant<int, 1>{}); clear(std::integral_constant<int, 1>{}); }

  // ---- rank steps ----
  // 3-bit pairs: the code dword and the lane's half of the metadata (layout.h) of every stream's unit
  // of one rank step; zeros for fp16 pairs, past the stream's own rank and past the last n-tile
  struct QUnits { uint32_t codes[kNTW][NM]; uint32_t meta[kNTW][NM][4]; };
  auto q_load = [&](int st, QUnits& qu) {
#pragma unroll
    for (int t = 0; t < kNTW; ++t)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        qu.codes[t][m] = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) qu.meta[t][m][i] = 0;
        if constexpr (Q3) {
          const int tile = tile0 + t;
          if (q3m[m] && st < LSm[m] && tile < a.NT) {
            const int mat = DUAL ? m : 2;
            qu.codes[t][m] = uniform_ptr(d->bfc[mat])[(size_t(st) * a.NT + tile) * kWave + lane];
            const uint4 v = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint8_t*>(uniform_ptr(d->bf[mat])) +
                                                            ((size_t(st) * (a.NT / 4) + (tile >> 2)) * 4 + q) * 32 + (c & 1) * 16);
            qu.meta[t][m][0] = v.x; qu.meta[t][m][1] = v.y; qu.meta[t][m][2] = v.z; qu.meta[t][m][3] = v.w;
          }
        }
      }
  };
  QUnits qnext;
  if (LS > 0) fetch_rank(0, cur);
  for (int c0 = 0, c1; c0 < LS; c0 = c1) {
    c1 = min(LS, c0 == 0 ? kRankFirst : c0 + kRankChunk);
    const uint4* region = c0 == 0 ? xs + 2 * kHalfUnits : xs;
    q_load(c0, qnext);
    if (c0 > 0) {
      __syncthreads();                       // (everyone is done with what the buffer held)
      stage_rank(xs, c0, c1);
      wait_loads_barrier();
    }
    // the fp16 B-factor unit of stream (t, m) of a rank step: from the slot, or rebuilt from a 3-bit unit
    auto b_unit = [&](const Slot2<BITS, NM, kNTW>& cur, const QUnits& qu, int t, int m, uint32_t (&u)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) u[i] = cur.t[t].cw[m][i];
      if constexpr (Q3) {
        if (q3m[m]) {
          const uint32_t own[4] = {qu.meta[t][m][0], qu.meta[t][m][1], qu.meta[t][m][2], qu.meta[t][m][3]};
          const uint4 v = __builtin_bit_cast(uint4, q3_unit_b(qu.codes[t][m], own, (c & 1) != 0));
          u[0] = v.x; u[1] = v.y; u[2] = v.z; u[3] = v.w;
        }
      }
    };
    auto rank_step = [&](const Slot2<BITS, NM, kNTW>& cur, const QUnits& qu, int st) {
#pragma unroll
      for (int j = 0; j < NPAIR; ++j) {
        // the B-factor units of the pair's two streams, 16-lane rows swapped: r0 = rank groups 0 and 2
        // of both streams side by side, r1 = groups 1 and 3 (a stream past its own rank holds zeros)
        int t0s, m0s, t1s, m1s;
        pair_stream(j, 0, t0s, m0s);
        pair_stream(j, 1, t1s, m1s);
        uint32_t u0[4], u1[4], r0v[4], r1v[4];
        b_unit(cur, qu, t0s, m0s, u0);
        b_unit(cur, qu, t1s, m1s, u1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const auto sw = __builtin_amdgcn_permlane16_swap(u0[i], u1[i], false, false);
          r0v[i] = sw[0]; r1v[i] = sw[1];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
          uint32_t av[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (DUAL) {
              // W1 and W3 meet different (in A): W1's columns keep one half of the inputs, W3's the
              // other (lane rows 0, 3 or 1, 2), zero elsewhere
              const bool keep = (v & 1) ? (q == 1 || q == 2) : (q == 0 || q == 3);
              av[i] = keep ? (v < 2 ? r0v[i] : r1v[i]) : 0u;
            } else {
              av[i] = v == 0 ? r0v[i] : r1v[i];
            }
          }
          const half8_t avh = __builtin_bit_cast(half8_t, make_uint4(av[0], av[1], av[2], av[3]));
#pragma unroll
          for (int rp = 0; rp < kRP; ++rp)
            if (rp < rp_n) {
              const half8_t pf = __builtin_bit_cast(half8_t, region[((size_t(st - c0) * V + v) * kRP + rp) * 64 + lane]);
              acc[j][rp] = __builtin_amdgcn_mfma_f32_32x32x16_f16(avh, pf, acc[j][rp], 0, 0, 0);
            }
        }
      }
    };
    for (int st = c0; st < c1; ++st) {
      const QUnits qcur = qnext;
      q_load(st + 1 < c1 ? st + 1 : LS, qnext);   // (LS: nothing to fetch)
      Slot2<BITS, NM, kNTW> nxt;
      fetch_rank(st + 1, nxt);
      rank_step(cur, qcur, st);
      cur = nxt;
    }
  }

  // ---- epilogue: lane l holds, of row 32 rp + l % 32, columns 8 g + 4 (l / 32) .. + 3 (g = 0, 1) of
  //      both streams of every pair ----
  const int hh = lane >> 5;
  if constexpr (DUAL) {
#pragma unroll
    for (int j = 0; j < NPAIR; ++j)
#pragma unroll
      for (int rp = 0; rp < kRP; ++rp) {
        const int row = r + 32 * rp + (lane & 31), tile = tile0 + j;
        if (rp >= rp_n || row >= cnt || tile >= a.NT) continue;
        const int se = a.row_exp[(a.offsets ? r0 : 0) + row];        // the row's inputs were scaled by 2^se
        const float dn = pow2i(-se), up = pow2i(2 * se);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          half4_t hv;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float gg = acc[j][rp][4 * g + i] * (lam[0] * dn), uu = acc[j][rp][8 + 4 * g + i] * (lam[NM - 1] * dn);
            hv[i] = to_f16_sat(gg * __builtin_amdgcn_rcpf(1.0f + __expf(-gg)) * uu * up);
          }
          // h in operand order for the W2 kernel: columns f .. f+3 are half of one 16-byte unit
          const int f = tile * kTileN + 8 * g + 4 * hh;
          *reinterpret_cast<half4_t*>(reinterpret_cast<_Float16*>(a.out) + act_unit(f >> 3, r0 + row, a.out_rt) * 8 + (f & 7)) = hv;
        }
      }
  } else {
    // y_rows is row-major: a lane's four columns would be an 8-byte store per row (32 rows per
    // instruction).  The wavefront turns its 128 x (16 kNTW) results round in its own part of the
    // activation buffer and stores whole 16-byte pieces of 32 kNTW contiguous bytes per row.
    constexpr int kPitch = 16 * kNTW * 2 + 16;                       // bytes per row in LDS
    static_assert(kGemmWaves * kBM * kPitch <= kGemmLdsUnits * 16, "the results of a block must fit its LDS");
    __syncthreads();                                                 // (everyone is done with the buffer and the (in A) fragments)
    uint8_t* mine = reinterpret_cast<uint8_t*>(xs) + wave * (kBM * kPitch);
#pragma unroll
    for (int rp = 0; rp < kRP; ++rp) {
      const int row = r + 32 * rp + (lane & 31);
      if (rp >= rp_n) continue;
      const int se = a.row_exp[(a.offsets ? r0 : 0) + min(row, cnt - 1)];
      const float l2 = lam[0] * pow2i(-2 * se);
#pragma unroll
      for (int j = 0; j < NPAIR; ++j)
#pragma unroll
        for (int side = 0; side < 2; ++side)
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            uint2 yv;
            yv.x = f32x2_to_bf16x2(acc[j][rp][8 * side + 4 * g] * l2, acc[j][rp][8 * side + 4 * g + 1] * l2);
            yv.y = f32x2_to_bf16x2(acc[j][rp][8 * side + 4 * g + 2] * l2, acc[j][rp][8 * side + 4 * g + 3] * l2);
            *reinterpret_cast<uint2*>(mine + (32 * rp + (lane & 31)) * kPitch + ((2 * j + side) * 16 + 8 * g + 4 * hh) * 2) = yv;
          }
    }
    constexpr int kPieces = 2 * kNTW;                                // 16-byte pieces per row
    const int piece = lane % kPieces;
    if (tile0 + piece / 2 < a.NT)
      for (int i = lane / kPieces; i < min(kBM, cnt - r); i += 64 / kPieces)
        *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(a.out) + size_t(r0 + r + i) * a.N + tile0 * kTileN + 8 * piece) =
            *reinterpret_cast<const uint4*>(mine + i * kPitch + 16 * piece);
  }
}

// (in A)[row][rho], fp16 row-major [routed row][NM * ls * 32 columns] ([A1 | A3] in the fused case, each
// padded to a multiple of 32), multiplied by the projection's power-of-two pre-scale, zero for rows
// without the rank-r term and in the padding columns.
// Only the rows that take the term are computed: the items run over 16 MT of the compact rows that the
// preparing launch has made of them (CompactArgs: the front of every expert's row range), and every
// sum goes to its routed row.  Blocks past the items write the zero rows.
// The product is skinny (16 to 128 columns) and its operands are in cache, so it is bound by latency:
// a block of 16 wavefronts takes 16 MT rows x at most T 16-column factor tiles (grid.y: groups of T
// tiles), the wavefronts share K and read both operands straight into registers, three or four units of 32
// inputs ahead; their sums meet in LDS, in wavefront
// order.  Qwen3 T = 4096: 30 + 22 us for the two products, DeepSeek T = 512: 12 + 10; with the two launches below
// 43 + 37 and 16 + 16.  Where those are faster instead: xa_staged.
// Q3: some factor pair of the layer is held at 3 bits (layout.h); such a pair's units are fetched as
// (codes, metadata) dwords and dequantized.
constexpr int kXaWaves = 16, kXaTiles = 4;
constexpr int kXaZeroUnits = 8192;         // 16-byte units a zeroing block looks after
template <bool DUAL, int T, int MT, bool Q3>
__global__ __launch_bounds__(64 * kXaWaves) void xa_kernel(KArgs a, int items, bool uneven, const int32_t* __restrict__ comp_index,
                                                           const uint16_t* __restrict__ x_bf16, _Float16* __restrict__ P) {
  constexpr int NM = DUAL ? 2 : 1;
  constexpr int kAhead = T * MT == 8 ? 3 : 4;     // units in flight (registers)
  __shared__ float4_t red[kXaWaves][MT][64];
  const int th = threadIdx.x, lane = th & 63;
  const int pitch = NM * a.ls * 32;
  if ((int)blockIdx.x >= items) {                        // rows without the term
    if (blockIdx.y != 0) return;
    const int per_row = pitch / 8;
    const size_t u0 = size_t((int)blockIdx.x - items) * kXaZeroUnits, end = size_t(a.total_rows) * per_row;
    for (size_t u = u0 + th; u < u0 + kXaZeroUnits && u < end; u += 64 * kXaWaves)
      if (comp_index[u / per_row] < 0) reinterpret_cast<uint4*>(P)[u] = make_uint4(0, 0, 0, 0);
    return;
  }
  Chunk ch;
  if (!find_chunk<16 * MT>(a, blockIdx.x, ch)) return;
  const int e = __builtin_amdgcn_readfirstlane(ch.e), r0 = __builtin_amdgcn_readfirstlane(ch.r0);
  const int cnt = __builtin_amdgcn_readfirstlane(ch.cnt), r = __builtin_amdgcn_readfirstlane(ch.r);
  const ConstDesc d = const_desc(a.desc + e);
  if (!d->has_factors) return;
  const int wave = __builtin_amdgcn_readfirstlane(th >> 6);
  const int q = lane >> 4, c = lane & 15;
  // The chunk's rows are compact rows: row_list names the routed row of each (past the last one: the
  // last one again, its sums are not stored).  The fused projections read the rows' bf16 tokens (whole
  // lines; the compact rows of the operand-order buffer are 16-byte pieces of lines shared with rows
  // that do not take the term) and scale them as the preparing launch does, W2 reads h.
  int R[MT];
  const u32x4* xrow[MT];
  float xs2[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    R[mt] = a.row_list[r0 + min(r + 16 * mt + c, cnt - 1)];
    xrow[mt] = DUAL ? reinterpret_cast<const u32x4*>(x_bf16 + size_t(a.row_pair[R[mt]] / a.top_k) * a.K) : nullptr;
    xs2[mt] = DUAL ? pow2i(a.row_exp[R[mt]]) : 1.f;
  }
  const int rt = a.rpad / 16, tiles = NM * rt;
  // zeros in 16 columns of the chunk's rows
  const int R_first = R[0], R_last = R[MT - 1];
  auto zero_tile = [=](int m, int tl, int mt) {
    if (r + 16 * mt + c < cnt)
      *reinterpret_cast<half4_t*>(P + size_t(mt ? R_last : R_first) * pitch + m * a.ls * 32 + 16 * tl + 4 * q) = half4_t{0, 0, 0, 0};
  };
  // the padding columns of a rank that is an odd number of tiles
  auto zero_padding = [=] {
    if ((rt & 1) && blockIdx.y == 0 && wave >= 2 && wave < 2 + MT * NM) zero_tile((wave - 2) / MT, rt, (wave - 2) % MT);
  };
  // Ranks that differ (Section 3.1): a block all of whose tiles lie past their projection's own rank leaves here
  // (largest rank 1024, every pair at 16, Qwen3 T = 4096: (x A) 674 -> 174 us, (h A2) 210 -> 75).
  if (uneven) {
    bool some = false;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int tile = blockIdx.y * T + t, m = tile / rt;
      some |= tile < tiles && 16 * (tile - m * rt) < __builtin_amdgcn_readfirstlane(d->rank[DUAL ? min(m, 1) : 2]);
    }
    if (!some) {
      // (the FFN kernel reads the columns of the rank steps its expert runs, those of the expert's larger pair)
      const int rank_e = max(__builtin_amdgcn_readfirstlane(d->rank[DUAL ? 0 : 2]), __builtin_amdgcn_readfirstlane(d->rank[DUAL ? 1 : 2]));
      const int tile = blockIdx.y * T + wave / MT, m = tile / rt, tl = tile - m * rt;
      if (wave < T * MT && tile < tiles && 16 * tl < (rank_e + 31) / 32 * 32) zero_tile(m, tl, wave % MT);
      zero_padding();
      return;
    }
  }
  // factor tile t of this block: 16 columns of projection m.  (The loads are unconditional: what a tile past
  // the projection's own rank or past the last one reads lies inside the factor sections, and its
  // products are dropped.)
  GlobalPtr<uint32_t> af[T];
  GlobalPtr<uint32_t> am[T];                 // 3-bit pairs: the tile's metadata, [group of 64 inputs][16 columns]
  bool q3t[T], valid[T];
  float scale[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int tile = min(blockIdx.y * T + t, tiles - 1), m = tile / rt, tl = tile - m * rt, mat = DUAL ? m : 2;
    valid[t] = 16 * tl < __builtin_amdgcn_readfirstlane(d->rank[mat]);
    q3t[t] = Q3 && __builtin_amdgcn_readfirstlane((d->q3 >> mat) & 1) != 0;
    scale[t] = d->xa_scale[mat];
    af[t] = as_global<uint32_t>(uniform_ptr(d->af[mat])) + size_t(tl) * (a.K / 32) * kWave * (q3t[t] ? 1 : 4);
    am[t] = q3t[t] ? as_global<uint32_t>(uniform_ptr(d->afm[mat])) + size_t(valid[t] ? tl : 0) * (a.K / 64) * 16 + c : nullptr;
  }
  float4_t acc[T][MT];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = float4_t{0.f, 0.f, 0.f, 0.f};

  // Unit kk: inputs 32 kk + 8 q + j of lane group q.  Wavefront w takes a contiguous run of units.
  struct Ops { u32x4 x[MT], w[T]; uint32_t mw[T]; };
  const u32x4* in_units = reinterpret_cast<const u32x4*>(a.in);
  const int units = a.K / 32, per = (units + kXaWaves - 1) / kXaWaves, k_lo = wave * per, k_hi = min(units, k_lo + per);
  auto load = [&](int kk_, Ops& o) {
    const int kk = max(0, min(kk_, k_hi - 1));
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) o.x[mt] = DUAL ? xrow[mt][4 * kk + q] : in_units[act_unit(4 * kk + q, R[mt], a.in_rt)];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      o.mw[t] = 0;
      if (Q3 && q3t[t]) {
        o.w[t] = u32x4{af[t][kk * kWave + lane], 0, 0, 0};
        o.mw[t] = am[t][(kk >> 1) * 16];
      } else {
        o.w[t] = reinterpret_cast<GlobalPtr<u32x4>>(af[t])[kk * kWave + lane];
      }
    }
  };
  auto multiply = [&](const Ops& o) {
    half8_t x[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if constexpr (DUAL) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[mt][2 * i] = (_Float16)(__uint_as_float(o.x[mt][i] << 16) * xs2[mt]);
          x[mt][2 * i + 1] = (_Float16)(__uint_as_float(o.x[mt][i] & 0xffff0000u) * xs2[mt]);
        }
      } else {
        x[mt] = __builtin_bit_cast(half8_t, o.x[mt]);
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      half8_t w = Q3 && q3t[t] ? q3_unit_a(o.w[t][0], o.mw[t]) : __builtin_bit_cast(half8_t, o.w[t]);
      if (!valid[t]) w = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w, x[mt], acc[t][mt], 0, 0, 0);
    }
  };
  Ops ring[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) load(k_lo + i, ring[i]);
  for (int k0 = k_lo; k0 < k_hi; k0 += kAhead)
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      if (k0 + i < k_hi) multiply(ring[i]);
      load(k0 + i + kAhead, ring[i]);
    }

  // the wavefronts' sums, one factor tile at a time: lane (q, c) holds columns 4 q .. + 3 of row 16 mt + c
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int tile = blockIdx.y * T + t, m = tile / rt;
    if (tile >= tiles) continue;
    if (t > 0) __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[wave][mt][lane] = acc[t][mt];
    __syncthreads();
    if (wave < MT) {
      float4_t sum = red[0][wave][lane];
#pragma unroll
      for (int w = 1; w < kXaWaves; ++w) sum += red[w][wave][lane];
      sum *= scale[t];
      if (r + 16 * wave + c < cnt)
        *reinterpret_cast<half4_t*>(P + size_t(wave ? R_last : R_first) * pitch + m * a.ls * 32 + 16 * (tile - m * rt) + 4 * q) =
            half4_t{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
    }
  }
  zero_padding();
}

// The same product for many factor tiles or a long K, in two launches: with 128 rows staged through LDS,
// eight row tiles meet every fragment of the factors, and the rows are read once per 32 factor tiles (the
// kernel above reads the factors once per 16 or 32 rows and the rows once per four tiles).  Which of the
// two a product takes: xa_staged below.
// xa_tile_kernel: K-block sums in fp32, [K-block][compact row][NM * ls * 32 columns], already multiplied by
// the projection's pre-scale.  A block of 8 wavefronts takes 128 compact rows and at most 8 NT factor tiles,
// wavefront w tiles w, w + 8, ...; the k-steps of activations are double-buffered in LDS; grid.x splits K so
// that the launch fills the chip, grid.z walks groups of 8 NT tiles.  Tiles past their projection's own rank are
// neither read, multiplied nor stored, and a block without a tile that counts leaves at once.
// xa_join_kernel: adds the K-blocks in order and writes every routed row of an expert: fp16 sums, and zeros
// for the rows without the term and between a projection's rank and the rank steps its expert runs.
constexpr int kXtWaves = 8;
constexpr int kXtRowTiles = kBM / 16;
constexpr int kXtStepUnits = kXtRowTiles * 8 * 64;       // 16-byte units of a k-step of activations (64 KB)

// Copy of the activations of k-step ks for the 128 rows of a chunk into `buf`, as 64 fragments (row tile
// mt, sub-step s) of 64 units: wavefront w copies the fragments with s = w, each lane its own 16 bytes from
// global memory straight to LDS; R[mt] is this lane's input row of row tile mt.  A column past the end is
// clamped to a valid unit (the factor units that meet it are zeros).
__device__ inline void stage_step_rows(const KArgs& a, uint4* buf, int ks, const int (&R)[kXtRowTiles], int mt_n, int wave, int lane) {
  const uint4* in_units = reinterpret_cast<const uint4*>(a.in);
  const int q = lane >> 4, s = wave;
  const int k8 = min(ks * 32 + q * 8 + s, a.K / 8 - 1);
#pragma unroll
  for (int mt = 0; mt < kXtRowTiles; ++mt)
    if (mt < mt_n)        // (row tiles past the chunk's last row are not read)
      __builtin_amdgcn_global_load_lds(
          reinterpret_cast<const __attribute__((address_space(1))) void*>(reinterpret_cast<uintptr_t>(in_units + act_unit(k8, R[mt], a.in_rt))),
          reinterpret_cast<__attribute__((address_space(3))) void*>(reinterpret_cast<uintptr_t>(buf + (mt * 8 + s) * 64)), 16, 0, 0);
}

template <bool DUAL, int NT, bool Q3>
__global__ __launch_bounds__(64 * kXtWaves, 2) void xa_tile_kernel(KArgs a) {
  extern __shared__ uint4 xs[];
  constexpr int NM = DUAL ? 2 : 1;
  constexpr bool kAhead = NT <= 2;                       // registers for the factor units of a whole k-step ahead
  Chunk ch;
  if (!find_chunk<kBM>(a, blockIdx.y, ch)) return;
  const int e = __builtin_amdgcn_readfirstlane(ch.e), r0 = __builtin_amdgcn_readfirstlane(ch.r0);
  const int cnt = __builtin_amdgcn_readfirstlane(ch.cnt), r = __builtin_amdgcn_readfirstlane(ch.r);
  const ConstDesc d = const_desc(a.desc + e);
  if (!d->has_factors) return;
  const int th = threadIdx.x, lane = th & 63;
  const int wave = __builtin_amdgcn_readfirstlane(th >> 6);
  const int q = lane >> 4, c = lane & 15;
  const int mt_n = min(kXtRowTiles, (cnt - r + 15) >> 4);
  const int rt = a.rpad / 16, tiles = NM * rt;           // 16-column factor tiles in all
  const int pitch = NM * a.ls * 32;
  // K-block blockIdx.x
  const int steps_all = (a.K + kTileK - 1) / kTileK;
  const int per = (steps_all + gridDim.x - 1) / gridDim.x;
  const int step_lo = blockIdx.x * per, steps = min(steps_all, step_lo + per);

  // A fragment of activations (k-step ks, sub-step s) holds, in lane (q, row), the columns
  // 256 ks + 64 q + 8 s + j: the factor unit that meets it is the one with those K rows, unit
  // (8 ks + 2 q + s / 4, tile) of the packed factor, lane (s % 4, c) of it.
  GlobalPtr<half8_t> af[NT];
  GlobalPtr<uint32_t> am[NT];                // 3-bit pairs: the tile's metadata, [group of 64 inputs][16 columns]
  bool q3t[NT], valid[NT];
  const int z0 = blockIdx.z * (kXtWaves * NT), z1 = min(tiles, z0 + kXtWaves * NT);
  bool some = false;                         // a tile of this block lies below its projection's rank
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const int first = max(z0 - m * rt, 0);
    some |= first < min(rt, z1 - m * rt) && 16 * first < __builtin_amdgcn_readfirstlane(d->rank[DUAL ? m : 2]);
  }
  if (!some) return;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int tile = z0 + wave + t * kXtWaves;
    af[t] = nullptr; am[t] = nullptr; q3t[t] = false; valid[t] = false;
    if (tile < tiles) {
      const int m = tile / rt, tl = tile - m * rt, mat = DUAL ? m : 2;
      valid[t] = 16 * tl < __builtin_amdgcn_readfirstlane(d->rank[mat]);
      q3t[t] = Q3 && __builtin_amdgcn_readfirstlane((d->q3 >> mat) & 1) != 0;
      if (q3t[t]) {
        af[t] = reinterpret_cast<GlobalPtr<half8_t>>(as_global<uint32_t>(uniform_ptr(d->af[mat])) + size_t(tl) * (a.K / 32) * kWave + c);
        am[t] = as_global<uint32_t>(uniform_ptr(d->afm[mat])) + size_t(tl) * (a.K / 64) * 16 + c;
      } else {
        af[t] = as_global<half8_t>(uniform_ptr(d->af[mat])) + size_t(tl) * (a.K / 32) * kWave + c;
      }
    }
  }
  // The chunk's rows are compact rows: row_list names the routed row whose activations each one reads.  A
  // row past the expert's last compact row reads one of the zero rows at the end of the buffer (its
  // results are never stored).
  int Rm[kXtRowTiles];
#pragma unroll
  for (int mt = 0; mt < kXtRowTiles; ++mt)
    Rm[mt] = r + 16 * mt + c < cnt ? a.row_list[r0 + r + 16 * mt + c] : a.in_rt - dec::kZeroRows + c;
  float4_t acc[NT][kXtRowTiles];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int mt = 0; mt < kXtRowTiles; ++mt) acc[t][mt] = float4_t{0.f, 0.f, 0.f, 0.f};

  // the factor units of sub-step s of k-step `step` for this lane (zero past K)
  auto load_unit = [&](int step, int s, int t) {
    const int kk = step * 8 + 2 * q + (s >> 2);          // this lane's 32-row unit of the factor
    u32x4 v = u32x4{0, 0, 0, 0};
    if (valid[t] && kk * 32 < a.K) {
      if (Q3 && q3t[t]) v[0] = reinterpret_cast<GlobalPtr<uint32_t>>(af[t])[size_t(kk) * kWave + (s & 3) * 16];
      else v = __builtin_bit_cast(u32x4, af[t][size_t(kk) * kWave + (s & 3) * 16]);
    }
    return v;
  };
  // 3-bit pairs: a lane's eight units of a k-step lie in one group of 64 inputs (rows 256 step + 64 q ..):
  // one dword of metadata per k-step and tile
  auto load_meta = [&](int step, int t) {
    uint32_t mv = 0;
    if (Q3 && q3t[t] && valid[t] && (step * 4 + q) * 64 < a.K) mv = am[t][(step * 4 + q) * 16];
    return mv;
  };
  // the operand of a fetched unit (a unit that was not fetched is all zeros in either format)
  auto operand = [&](const u32x4& v, uint32_t mv, int t) {
    if (Q3 && q3t[t]) return q3_unit_a(v[0], mv);
    return __builtin_bit_cast(half8_t, v);
  };
  u32x4 wnext[kAhead ? 8 : 1][NT];
  uint32_t mnext[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) mnext[t] = load_meta(step_lo, t);
  if constexpr (kAhead) {
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int t = 0; t < NT; ++t) wnext[s][t] = load_unit(step_lo, s, t);
  }
  stage_step_rows(a, xs + (step_lo & 1) * kXtStepUnits, step_lo, Rm, mt_n, wave, lane);
  wait_loads_barrier();
  for (int step = step_lo; step < steps; ++step) {
    stage_step_rows(a, xs + ((step + 1) & 1) * kXtStepUnits, step + 1, Rm, mt_n, wave, lane);
    const uint4* buf = xs + (step & 1) * kXtStepUnits;
    half8_t wcur[kAhead ? 8 : 1][NT];
    uint32_t mcur[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) { mcur[t] = mnext[t]; mnext[t] = load_meta(step + 1, t); }
    if constexpr (kAhead) {                  // this step's units have arrived; ask for the next step's
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) wcur[s][t] = operand(wnext[s][t], mcur[t], t);
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) wnext[s][t] = load_unit(step + 1, s, t);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      half8_t wf[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if constexpr (kAhead) wf[t] = wcur[s][t];
        else wf[t] = operand(load_unit(step, s, t), mcur[t], t);
      }
#pragma unroll
      for (int mt = 0; mt < kXtRowTiles; ++mt)
        if (mt < mt_n) {
          const half8_t xf = __builtin_bit_cast(half8_t, buf[(mt * 8 + s) * 64 + lane]);
#pragma unroll
          for (int t = 0; t < NT; ++t)
            if (valid[t]) acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[t], xf, acc[t][mt], 0, 0, 0);
        }
    }
    // the copy of the next step has landed; everyone is done with this step's half of LDS
    wait_loads_barrier();
  }

  // lane holds columns 16 tile + 4 q .. + 3 of row 16 mt + c
  float* part = a.partial + size_t(blockIdx.x) * a.total_rows * pitch;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (!valid[t]) continue;
    const int tile = z0 + wave + t * kXtWaves, m = tile / rt, tl = tile - m * rt;
    const float lam = d->xa_scale[DUAL ? m : 2];
#pragma unroll
    for (int mt = 0; mt < kXtRowTiles; ++mt) {
      const int row = r + 16 * mt + c;
      if (mt >= mt_n || row >= cnt) continue;
      *reinterpret_cast<float4_t*>(part + size_t(r0 + row) * pitch + m * a.ls * 32 + 16 * tl + 4 * q) = acc[t][mt] * lam;
    }
  }
}

// One thread: four columns of a routed row.
__global__ __launch_bounds__(256) void xa_join_kernel(KArgs a, int kblocks, int nm, bool uneven, const int32_t* __restrict__ comp_index,
                                                      _Float16* __restrict__ P) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  const int ls32 = a.ls * 32, pitch = nm * ls32, per_row = pitch / 4;
  if (i >= size_t(a.total_rows) * per_row) return;
  const int row = int(i / per_row), col = int(i - size_t(row) * per_row) * 4;
  const int m = col / ls32, cm = col - m * ls32;         // projection, column of its (in A)
  const int ci = comp_index[row];                        // the row's place among those with the term (-1: none)
  int rank = a.rpad;
  if (uneven) {
    int e = 0;                                           // the expert of the row: the last one with offsets[e] <= row
    for (int step = 128; step > 0; step /= 2)
      if (e + step < a.n_exp && a.offsets[e + step] <= row) e += step;
    const int32_t* ranks = a.desc[e].rank;
    const int rank_e = nm == 2 ? max(ranks[0], ranks[1]) : ranks[2];
    if (cm / 32 * 32 >= rank_e) return;                  // a rank step this expert does not run
    rank = ranks[nm == 2 ? m : 2];
  }
  float4_t sum = float4_t{0.f, 0.f, 0.f, 0.f};
  if (ci >= 0 && cm / 16 * 16 < rank) {
    const float4_t* part = reinterpret_cast<const float4_t*>(a.partial + size_t(ci) * pitch + col);
    const size_t kb4 = size_t(a.total_rows) * per_row;
    sum = part[0];
    for (int kb = 1; kb < kblocks; ++kb) sum += part[kb * kb4];
  }
  *reinterpret_cast<half4_t*>(P + size_t(row) * pitch + col) = half4_t{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
}

// Whether a product takes the two launches.  What the one launch takes grows with the factor tiles times K; past
// about 20480 the staged rows win (us, one launch / two):
//   fused, K = 4096: rank 16 (8192) T = 1024 17 / 25, 4096 22 / 37; rank 32 (16384) 23 / 25 and 28 / 38;
//     rank 64 (32768) 28 / 27 and 47 / 42; rank 256 49 / 45 and 112 / 87; rank 1024 138 / 91 and 389 / 253
//   fused, K = 2048, 128 experts, T = 4096: rank 32 (8192) 41 / 46; rank 128 (32768) 94 / 70; rank 1024 663 / 358
//   W2, K = 14336, T = 2048: rank 16 (14336) 45 / 50; rank 64 (57344) 66 / 54; rank 256 132 / 84
//   W2, K = 768, T = 4096: rank 128 (6144) 38 / 45; rank 256 (12288) 63 / 55; rank 512 108 / 79
// (below the line the two launches still win here and there: K = 4096, rank 32, T = 256: 24 / 19; K = 1408, rank 128,
// T = 1024: 31 / 23.)  With ranks that differ the tiles that hold columns count, averaged over the experts, but at
// least a fifth of the grid, whose blocks without such tiles are not free (largest rank 1024, the others 16,
// K = 1216, T = 2048: 93 / 44).  3-bit pairs, two tiles per block: the two launches past 8192 unless the rows are few,
// tiles times K times rows at most 4e7 (rank 64, K = 4096, T = 1024 22 / 32, 2048 37 / 34, 4096 55 / 52; rank 256,
// K = 768, T = 4096 91 / 59).
bool xa_staged(const FfnArgs& f, bool dual) {
  const long long K = dual ? f.H : f.F, tiles = (dual ? 2 : 1) * f.rpad / 16;
  const long long cost5 = std::max<long long>(5 * (dual ? f.live13 : f.live2), tiles * f.n_exp) * K / f.n_exp;     // 5 x tiles x K
  if (f.q3) return cost5 > 5 * 8192 && cost5 * f.T * f.top_n > 5 * 40000000LL;
  return cost5 > 5 * 20480;
}

// Whether the column blocks of a chunk run on one XCD, whose L2 then holds the chunk's rows once for all of them: where the weights that
// the chunk meets (`mats` matrices of an expert) fit half of that L2.  Otherwise neighbouring blocks share columns of
// weights, not rows.  Whole layer, columns dealt over the XCDs -> one XCD (us): Qwen3 shape T = 4096 (1.4 and 0.7 MB) 615 -> 600,
// DeepSeek T = 512 (1.8 and 0.9 MB) 200 -> 195; Mixtral T = 2048 (51 and 26 MB) 1540 -> 1578.  Above the line it is no one thing:
// W1|W3 alone of hidden = FFN = 3072 at 4 bits (10.6 MB), T = 1024 199 -> 221, T = 2048 343 -> 332; 4096 x 7168 at 3 bits (26 MB),
// T = 2048 780 -> 793; hidden = FFN = 2048 at 3 bits (3.7 MB) 311 -> 301.
// Routed experts only: shared experts are few chunks, which would leave XCDs without work, and run beside the routed ones.  64 routed experts
// (Top-1) and one shared, 2048 x 1408, columns dealt / one XCD: T = 128 144 / 156, 256 132 / 144, 768 155 / 155, 1500 171 / 185.
bool gemm_by_xcd(const FfnArgs& f, int mats) {
  return f.offsets != nullptr && (long long)mats * f.H * f.F * (8 * f.bits + 256 / f.group) / 64 <= 2 << 20;     // bits / 8 + 4 / group bytes a weight
}

template <int BITS>
hipError_t launch_bits(const FfnArgs& f, hipStream_t s, int which) {
  int gs = 0;
  while ((1 << gs) < f.group) ++gs;
  KArgs a{};
  a.desc = f.desc; a.offsets = f.offsets; a.row_pair = f.row_pair; a.comp_rows = f.comp_rows; a.n_exp = f.n_exp;
  a.row_exp = f.row_exp; a.tok_exp = f.tok_exp;
  a.group_shift = gs; a.top_k = f.top_k; a.top_n = f.top_n; a.T = f.T;
  a.rank = f.rank; a.rpad = f.rpad; a.ls = (f.rank + 31) / 32; a.total_rows = f.total_rows;
  const bool comp = f.rank > 0 && f.top_n > 0 && f.row_pair != nullptr;
  const int items_n = f.offsets ? chunk_items(f.total_rows, f.n_exp) : f.n_exp * ((f.T + kBM - 1) / kBM);
  auto items = [&] { return items_n; };
  const size_t glds = size_t(kGemmLdsUnits) * 16;

  // (in A) of the rows that take the term (T * top_n in all), zeros for the others
  auto xa = [&](auto DUAL_, float* buf) {
    constexpr bool DUAL = decltype(DUAL_)::value;
    constexpr int nm = DUAL ? 2 : 1;
    const int tiles = nm * f.rpad / 16;
    a.p = buf;
    KArgs ax = a;
    ax.row_list = f.cmp_list;
    const bool uneven = (DUAL ? f.live13 : f.live2) < (long long)f.n_exp * tiles;    // (ranks that differ)
    if (xa_staged(f, DUAL)) {
      const int steps = (a.K + kTileK - 1) / kTileK, ksplit = DUAL ? f.ksplit13 : f.ksplit2;
      const int per_kb = (steps + ksplit - 1) / ksplit, kblocks = (steps + per_kb - 1) / per_kb;     // no K-block without a k-step
      const int pitch = nm * a.ls * 32, per_wave = (tiles + kXtWaves - 1) / kXtWaves;               // factor tiles per wavefront
      ax.partial = buf + (size_t(f.total_rows) * pitch / 2 + 63) / 64 * 64;                         // (behind the fp16 result)
      auto tile = [&](auto kernel, int nt) {
        hipLaunchKernelGGL(kernel, dim3(kblocks, f.T * f.top_n / kBM + f.n_exp, (tiles + kXtWaves * nt - 1) / (kXtWaves * nt)), dim3(64 * kXtWaves),
                           size_t(2) * kXtStepUnits * 16, s, ax);
      };
      if (per_wave <= 2) f.q3 ? tile(xa_tile_kernel<DUAL, 2, true>, 2) : tile(xa_tile_kernel<DUAL, 2, false>, 2);
      else f.q3 ? tile(xa_tile_kernel<DUAL, 4, true>, 4) : tile(xa_tile_kernel<DUAL, 4, false>, 4);
      const size_t groups = size_t(f.total_rows) * pitch / 4;
      hipLaunchKernelGGL(xa_join_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, ax, kblocks, nm, uneven, f.cmp_index,
                         reinterpret_cast<_Float16*>(buf));
      return;
    }
    // 32 rows per block share the factor units it reads; 16 when that makes too few blocks: W2's longer
    // K wants more of them (K = 4096, rank 64, 2048 rows with the term: 28 us with 32 rows, 36 with 16; W2 with
    // K = 14336 88 and 67)
    // (3-bit pairs: two tiles per block; with four, the dequantized operands do not fit the registers, 9 to 41 of them
    // spilled: rank 64, K = 4096, T = 1024: 64 us with four tiles, 22 with two)
    const int per = tiles <= 2 ? tiles : f.q3 ? 2 : kXaTiles, gy = (tiles + per - 1) / per;
    const bool wide = f.T * f.top_n / 32 * gy >= (DUAL ? f.n_cu / 4 : f.n_cu);
    const int xitems = f.T * f.top_n / (wide ? 32 : 16) + f.n_exp;
    const size_t units = size_t(f.total_rows) * nm * a.ls * 4;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(xitems + unsigned((units + kXaZeroUnits - 1) / kXaZeroUnits), gy), dim3(64 * kXaWaves), 0, s, ax,
                         xitems, uneven, f.cmp_index, (const uint16_t*)f.x_tokens, reinterpret_cast<_Float16*>(buf));
    };
    auto pick = [&](auto T_) {
      constexpr int T = decltype(T_)::value;
      if constexpr (T <= 2) {
        if (f.q3) return wide ? go(xa_kernel<DUAL, T, 2, true>) : go(xa_kernel<DUAL, T, 1, true>);
      }
      wide ? go(xa_kernel<DUAL, T, 2, false>) : go(xa_kernel<DUAL, T, 1, false>);
    };
    if (per == kXaTiles) pick(std::integral_constant<int, kXaTiles>{});
    else if (per == 2) pick(std::integral_constant<int, 2>{});
    else if constexpr (!DUAL) pick(std::integral_constant<int, 1>{});
  };
  if (which & 1) {
  // W1 | W3 with the SwiGLU epilogue
  a.in = f.xh; a.out = f.h; a.K = f.H; a.N = f.F; a.NT = f.F / kTileN;
  a.in_rt = f.x_rt; a.out_rt = f.h_rt;
  a.KS = padded_k(f.H) / kTileK; a.G = padded_k(f.H) / f.group;
  if (comp) xa(std::true_type{}, f.p13);
  a.by_xcd = gemm_by_xcd(f, 2);
  a.plan = f.offsets ? f.plan : nullptr;
  if (f.marks) (void)hipEventRecord(f.marks[0], s);
  if (comp && f.q3) hipLaunchKernelGGL((qgemm_tile_kernel<BITS, true, 2, true>), dim3((a.NT + 2 * kGemmWaves - 1) / (2 * kGemmWaves), items()), dim3(64 * kGemmWaves), glds, s, a);
  else hipLaunchKernelGGL((qgemm_tile_kernel<BITS, true, 2>), dim3((a.NT + 2 * kGemmWaves - 1) / (2 * kGemmWaves), items()), dim3(64 * kGemmWaves), glds, s, a);
  if (f.marks) (void)hipEventRecord(f.marks[1], s);
  }
  if (which & 2) {
  // W2
  a.in = f.h; a.out = f.y_rows; a.K = f.F; a.N = f.H; a.NT = f.H / kTileN;
  a.in_rt = f.h_rt; a.out_rt = 0;
  a.KS = padded_k(f.F) / kTileK; a.G = padded_k(f.F) / f.group;
  if (comp) xa(std::false_type{}, f.p2);
  a.by_xcd = gemm_by_xcd(f, 1);
  a.plan = f.offsets ? f.plan2 : nullptr;
  if (f.marks) (void)hipEventRecord(f.marks[2], s);
  // Four n-tiles per wavefront use a fragment of activations twice as often as two (with two the LDS reads are the
  // bound), but make blocks twice as large: two only while four make fewer blocks than there are CUs.  Whole layer, four / two
  // (us): Mixtral shape T = 1024 (320 blocks of four) 840 / 874, 1500 (432) 1167 / 1197, 2048 (576) 1420 / 1461; 700 (240) 650 / 646;
  // DeepSeek T = 512 (768) 187 / 196; Qwen3 T = 1500 (1264) 283 / 286, 4096 (2560) 532 / 565.  At 4 bits, where four spill: Mixtral
  // T = 850 (272) 723 / 727, 960 (304) 802 / 850, 2048 1521 / 1541; DeepSeek T = 512 207 / 212; Qwen3 T = 1500 287 / 301; 3072 x 3072,
  // 8 experts, T = 1050 (240) 205 / 202, 1400 (300) 259 / 264.  The one loss beyond the line: 2048 x 1408, 16 experts, T = 1600 (264) 142 / 140.
  // (expected number of chunks: about half of the experts end with a partly filled one)
  const int chunks = std::max(1, f.offsets ? f.total_rows / kBM + (f.n_exp + 1) / 2 : f.n_exp * ((f.T + kBM - 1) / kBM));
  const bool q3 = comp && f.q3;
  if (chunks * ((a.NT + 4 * kGemmWaves - 1) / (4 * kGemmWaves)) >= f.n_cu) {
    if (q3) hipLaunchKernelGGL((qgemm_tile_kernel<BITS, false, 4, true>), dim3((a.NT + 4 * kGemmWaves - 1) / (4 * kGemmWaves), items()), dim3(64 * kGemmWaves), glds, s, a);
    else hipLaunchKernelGGL((qgemm_tile_kernel<BITS, false, 4>), dim3((a.NT + 4 * kGemmWaves - 1) / (4 * kGemmWaves), items()), dim3(64 * kGemmWaves), glds, s, a);
  } else {
    if (q3) hipLaunchKernelGGL((qgemm_tile_kernel<BITS, false, 2, true>), dim3((a.NT + 2 * kGemmWaves - 1) / (2 * kGemmWaves), items()), dim3(64 * kGemmWaves), glds, s, a);
    else hipLaunchKernelGGL((qgemm_tile_kernel<BITS, false, 2>), dim3((a.NT + 2 * kGemmWaves - 1) / (2 * kGemmWaves), items()), dim3(64 * kGemmWaves), glds, s, a);
  }
  if (f.marks) (void)hipEventRecord(f.marks[3], s);
  }
  return hipGetLastError();
}

}  // namespace

// Which flavour a projection takes (measured on Mixtral, DeepSeek and Qwen3 shapes): the decode
// flavour up to 24 rows per expert; beyond that the grouped GEMM as soon as it is efficient: the
// fused W1|W3 from about 40 rows per expert on, W2 (whose grid has few column blocks) once its grid
// of (128-row chunk, 256 columns) blocks covers the 256 CUs.
// bit 0: W1|W3 takes the decode flavour, bit 1: W2 does
static int decode_parts(const FfnArgs& f) {
  // expected rows per expert under uniform routing decides the flavour of each projection
  const int rows = f.offsets ? (f.T * f.top_k + f.n_exp - 1) / f.n_exp : f.T;
  const int chunks = f.offsets ? f.total_rows / kBM + (f.n_exp + 1) / 2 : f.n_exp * ((f.T + kBM - 1) / kBM);
  const bool w2_grid_full = chunks * ((f.H / kTileN + 15) / 16) >= f.n_cu;
  const bool d13 = rows <= kDecodeMaxRows13;
  // (beyond 128 rows per expert the decode flavour would stream the weights five times or more)
  const bool d2 = rows <= 24 || (!w2_grid_full && rows <= 128);
  return (d13 ? 1 : 0) | (d2 ? 2 : 0);
}

template <int BITS> static hipError_t tile_init_bits() {
  const void* fns[6] = {reinterpret_cast<const void*>(&qgemm_tile_kernel<BITS, true, 2>),
                        reinterpret_cast<const void*>(&qgemm_tile_kernel<BITS, false, 4>),
                        reinterpret_cast<const void*>(&qgemm_tile_kernel<BITS, false, 2>),
                        reinterpret_cast<const void*>(&qgemm_tile_kernel<BITS, true, 2, true>),
                        reinterpret_cast<const void*>(&qgemm_tile_kernel<BITS, false, 4, true>),
                        reinterpret_cast<const void*>(&qgemm_tile_kernel<BITS, false, 2, true>)};
  for (const void* fn : fns) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLdsUnits * 16);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t ffn_init_device() {
  const void* fns[8] = {reinterpret_cast<const void*>(&xa_tile_kernel<true, 2, false>), reinterpret_cast<const void*>(&xa_tile_kernel<false, 2, false>),
                        reinterpret_cast<const void*>(&xa_tile_kernel<true, 4, false>), reinterpret_cast<const void*>(&xa_tile_kernel<false, 4, false>),
                        reinterpret_cast<const void*>(&xa_tile_kernel<true, 2, true>), reinterpret_cast<const void*>(&xa_tile_kernel<false, 2, true>),
                        reinterpret_cast<const void*>(&xa_tile_kernel<true, 4, true>), reinterpret_cast<const void*>(&xa_tile_kernel<false, 4, true>)};
  for (const void* fn : fns) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kXtStepUnits * 16);
    if (e != hipSuccess) return e;
  }
  hipError_t e = tile_init_bits<2>();
  if (e == hipSuccess) e = tile_init_bits<3>();
  if (e == hipSuccess) e = tile_init_bits<4>();
  if (e == hipSuccess) e = decode_init_device();
  return e;
}

int expert_ffn_path(const FfnArgs& f) { return 3 & ~decode_parts(f); }

FfnTables expert_ffn_tables(const FfnArgs& f) {
  FfnTables t{};
  if (f.offsets == nullptr) return t;
  const int dp = decode_parts(f), items = chunk_items(f.total_rows, f.n_exp);
  decode_plan_specs(f, dp, t.plan[0], t.plan[1]);
  // (the order of the chunks: plan.h)
  if (!(dp & 1)) t.chunk[0] = ChunkSpec{items, gemm_by_xcd(f, 2) && f.total_rows >= kByLengthRows * f.n_exp, f.plan};
  if (!(dp & 2)) t.chunk[1] = ChunkSpec{items, true, f.plan2};
  return t;
}

hipError_t launch_expert_ffn(const FfnArgs& f, hipStream_t s) {
  auto tile = [&](int which) {
    switch (f.bits) {
      case 2: return launch_bits<2>(f, s, which);
      case 3: return launch_bits<3>(f, s, which);
      case 4: return launch_bits<4>(f, s, which);
    }
    return hipErrorInvalidValue;
  };
  const int dp = decode_parts(f);
  if (dp == 3) return launch_decode_ffn(f, s, 3);
  hipError_t e = (dp & 1) ? launch_decode_ffn(f, s, 1) : tile(1);
  if (e != hipSuccess) return e;
  return (dp & 2) ? launch_decode_ffn(f, s, 2) : tile(2);
}

}  // namespace lrc
