// (in A) for the rows of the decode flavour: the body shared by xa_rows_kernel (ffn_decode.hip) and
// by the launch that prepares the activations (misc.hip), which runs it for the fused W1|W3
// projections in further blocks.
#pragma once
#include <type_traits>

#include "factor_q3.h"
#include "ffn_common.h"

namespace lrc {
namespace ffn {

constexpr int kXaBatch = 4;     // factor and activation units requested together (8 spill in a 1024-thread block)

// (in A)[row][rho] for the rows of the decode flavour, finished in one launch:
//   P[row][m * ls * 32 + rho] = fp16(lambda_m * sum_k in[row][k] * A_m[k][rho]) for rows that take the
// rank-r term, 0 for the other rows of an expert that has such rows; lambda_m is the projection's
// power-of-two pre-scale.  grid = (16-column tiles of [A1 | A3] or of A2, the last of an odd
// number writing the padding to ls * 32 columns; experts); the NW wavefronts of a block split K and add their parts through LDS in a
// fixed order.  A tile past the projection's own rank writes zeros (the FFN kernel reads the columns
// of every rank step its expert runs).  TOKENS: the rows are read from the bf16 tokens through
// row_pair (the launch that prepares the activations runs this body in further blocks); otherwise
// from the fp16 operand-order buffer.
// Rows: where the grouping is read from: offset(e), pair(row), and the exponent of a row's token, exponent(pair, row).
// (Nothing is read of the factors of an expert without a row that takes the term, whose rows get zeros: in staged
// residency they were not brought in.)
// Bound: the chain of dependent loads, so the expert's table entry is read at once into scalar registers.
struct GroupedRows {                       // written by an earlier launch, or by this block
  const int32_t *offsets, *row_pair, *tok_exp, *row_exp;
  int top_k;
  __device__ int offset(int e) const { return offsets[e]; }
  __device__ int pair(int row) const { return row_pair[row]; }
  __device__ int exponent(int pair, int row) const { return tok_exp ? tok_exp[pair / top_k] : row_exp[row]; }
};
// Eight bf16 values times a power of two, rounded to fp16 (two to an instruction).
__device__ inline half8_t scaled_unit(const uint4& v, float scale) {
  typedef float float2_t __attribute__((ext_vector_type(2)));
  const uint32_t in[4] = {v.x, v.y, v.z, v.w};
  uint32_t o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float2_t f = float2_t{__uint_as_float(in[i] << 16) * scale, __uint_as_float(in[i] & 0xffff0000u) * scale};
    o[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, half2_t));
  }
  return __builtin_bit_cast(half8_t, make_uint4(o[0], o[1], o[2], o[3]));
}
// The block takes every `passes`-th pass of 32 rows.
template <bool DUAL, bool TOKENS, int NW, class Rows>
__device__ __forceinline__ void xa_rows_body(const KArgs& a, const Rows& rows, const uint16_t* __restrict__ x_bf16, int tile, int e, int kb,
                                             int pass, int passes, float4_t (*red)[64] /* [2 * NW][64] */) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c = lane & 15, q = lane >> 4;
  const int first = rows.offset(e), next = rows.offset(e + 1);
  const ConstDesc d = const_desc(a.desc + e);
  const int tpm = a.rpad / 16;                     // 16-column tiles per projection; the last one of an odd number also
                                                   // writes the zeros that pad it to ls * 32 columns
  const int m = tile / tpm, tl = tile - m * tpm, mat = DUAL ? m : 2;
  const int pitch = (DUAL ? 2 : 1) * a.ls * 32;
  const int has_factors = d->has_factors, q3_bits = d->q3, rank_m = d->rank[mat];
  const float lam = d->xa_scale[mat];
  // a pair held at 3 bits (layout.h): one dword of codes per lane and unit, one of metadata per
  // (tile, group of 64 inputs, column), dequantized here
  const GlobalPtr<u32x4> af = as_global<u32x4>(d->af[mat]);
  const GlobalPtr<uint32_t> aq = as_global<uint32_t>(d->af[mat]), am = as_global<uint32_t>(d->afm[mat]);
  const int r0 = __builtin_amdgcn_readfirstlane(first), cnt = __builtin_amdgcn_readfirstlane(next) - r0;
  if (cnt == 0 || !has_factors) return;
  const bool q3 = ((q3_bits >> mat) & 1) != 0;
  const bool live = 16 * tl < min(rank_m, a.rank);
  const bool pad = (tpm & 1) && tl == tpm - 1;
  const int g64 = a.K / 64;
  // this block's K-block (grid.z K-blocks of kb_steps k-steps each; one when kb_steps covers K): the
  // FFN kernel's K-block kb applies the B factor to the part of (in A) summed over its own k-steps
  const int k32 = a.K / 32, kb_lo = min(k32, kb * a.kb_steps * 8), kb_hi = min(k32, (kb + 1) * a.kb_steps * 8);
  const int per = (kb_hi - kb_lo + NW - 1) / NW;
  const int kk0 = kb_lo + wave * per, kk1 = min(kb_hi, kk0 + per);
  _Float16* P = reinterpret_cast<_Float16*>(const_cast<float*>(a.p)) + size_t(kb) * a.total_rows * pitch;
  const uint4* src = reinterpret_cast<const uint4*>(a.in);       // operand order: unit (k8, row)
  // Two row tiles share every load of the factor; all loads of a batch are issued before the first
  // is awaited (unconditional loads from clamped addresses, not multiplied where they do not count).
  for (int r = 32 * pass; r < cnt; r += 32 * passes) {
    bool flagged[2];
    int pair[2];
    const uint4* xrow[2];
    float xs2[2] = {1.f, 1.f};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int row = min(r + 16 * t + c, cnt - 1);
      pair[t] = rows.pair(r0 + row);
      flagged[t] = r + 16 * t + c < cnt && (pair[t] % a.top_k) < a.top_n;
      xrow[t] = TOKENS ? reinterpret_cast<const uint4*>(x_bf16 + size_t(pair[t] / a.top_k) * a.K) : nullptr;
      // the row's power-of-two pre-scale (the fp16 operand-order buffer holds the rows already scaled)
      if constexpr (TOKENS) xs2[t] = pow2i(rows.exponent(pair[t], r0 + row));
    }
    const bool any0 = __ballot(flagged[0]) != 0ull, any1 = __ballot(flagged[1]) != 0ull;   // block-uniform
    float4_t acc[2] = {float4_t{0.f, 0.f, 0.f, 0.f}, float4_t{0.f, 0.f, 0.f, 0.f}};
    if (live && (any0 || any1)) {
      // (with rows in the first row tile only, twice as many units are in flight: the second tile's registers are free)
      auto k_loop = [&](auto Q3_, auto TWO_) {
      constexpr bool Q3 = decltype(Q3_)::value, TWO = decltype(TWO_)::value;
      constexpr int NB = TWO ? kXaBatch : 2 * kXaBatch, NT = TWO ? 2 : 1;
      for (int kk = kk0; kk < kk1; kk += NB) {
        u32x4 wf[NB];
        uint4 xv[NT][NB];
        uint32_t cq[NB], mq[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          const int ku = max(min(kk + u, kk1 - 1), 0);
          if constexpr (Q3) {
            cq[u] = aq[(size_t(tl) * k32 + ku) * kWave + lane];
            mq[u] = am[(size_t(tl) * g64 + (ku >> 1)) * 16 + c];
          } else {
            wf[u] = af[(size_t(tl) * k32 + ku) * kWave + lane];
          }
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            if constexpr (TOKENS) xv[t][u] = xrow[t][4 * ku + q];
            else xv[t][u] = src[act_unit(4 * ku + q, r0 + min(r + 16 * t + c, cnt - 1), a.in_rt)];
          }
        }
        asm volatile("" ::: "memory");         // (none of them is moved behind the tests below)
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          if (kk + u >= kk1) break;            // (a step past this wavefront's share)
          const half8_t w = Q3 ? q3_unit_a(cq[u], mq[u]) : __builtin_bit_cast(half8_t, wf[u]);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            half8_t xf = TOKENS ? scaled_unit(xv[t][u], xs2[t]) : __builtin_bit_cast(half8_t, xv[t][u]);
            if (!flagged[t]) xf = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w, xf, acc[t], 0, 0, 0);
          }
        }
      }
      };
      if (q3) { if (any1) k_loop(std::true_type{}, std::true_type{}); else k_loop(std::true_type{}, std::false_type{}); }
      else { if (any1) k_loop(std::false_type{}, std::true_type{}); else k_loop(std::false_type{}, std::false_type{}); }
      red[wave][lane] = acc[0];
      red[NW + wave][lane] = acc[1];
      __syncthreads();
    }
    // wavefront t: lane (q, c) holds columns 16 tl + 4 q .. + 3 of row r + 16 t + c
    if (wave < 2) {
      const int row = r + 16 * wave + c;
      const bool take = wave == 0 ? flagged[0] : flagged[1];
      half4_t v = half4_t{0, 0, 0, 0};
      if (live && (any0 || any1)) {
        float4_t sum = red[wave * NW][lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += red[wave * NW + w][lane];
        if (take) v = half4_t{to_f16_sat(sum[0] * lam), to_f16_sat(sum[1] * lam), to_f16_sat(sum[2] * lam), to_f16_sat(sum[3] * lam)};
      }
      if (row < cnt) {
        _Float16* at = P + size_t(r0 + row) * pitch + m * a.ls * 32 + 16 * tl + 4 * q;
        *reinterpret_cast<half4_t*>(at) = v;
        if (pad) *reinterpret_cast<half4_t*>(at + 16) = half4_t{0, 0, 0, 0};
      }
    }
    if (r + 32 * passes < cnt) __syncthreads();
  }
}

// The same for every token, whatever it is routed to (p_tokens > 0): P[e][token][m * ls * 32 + rho], so that it
// needs neither the routing nor the grouping.  grid = (16-column tiles of [A1 | A3]; experts; passes of 32 tokens, or
// of 16 (`wide` false), from token r0 on).  tok_exp: the tokens' exponents, or null: taken from the rows here.  Per row the
// same products in the same order as above: the same bits.
template <int NW, int BATCH = kXaBatch>
__device__ __forceinline__ void xa_tokens_body(const KArgs& a, const uint16_t* __restrict__ x_bf16, const int32_t* tok_exp, int tile, int e,
                                               int r0, bool wide, float4_t (*red)[64] /* [2 * NW][64] */) {
  const ConstDesc d = const_desc(a.desc + e);
  const int lane = threadIdx.x & 63, c = lane & 15, q = lane >> 4, T = a.p_tokens;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rt = a.rpad / 16, m = tile / rt, tl = tile - m * rt, pitch = 2 * a.ls * 32;
  const int has_factors = d->has_factors, rank_m = d->rank[m], q3_bits = d->q3;
  const float lam = d->xa_scale[m];
  const GlobalPtr<half8_t> af = as_global<half8_t>(d->af[m]);
  const GlobalPtr<uint32_t> aq = as_global<uint32_t>(d->af[m]), am = as_global<uint32_t>(d->afm[m]);
  _Float16* P = reinterpret_cast<_Float16*>(const_cast<float*>(a.p));
  _Float16* col = P + m * a.ls * 32 + 16 * tl + 4 * q;               // this lane's four columns
  const bool pad = (rt & 1) && tl == rt - 1;                         // ... and the padding columns behind the last tile
  auto store = [&](size_t row, half4_t v) {
    *reinterpret_cast<half4_t*>(col + row * pitch) = v;
    if (pad) *reinterpret_cast<half4_t*>(col + row * pitch + 16) = half4_t{0, 0, 0, 0};
  };
  if (e == 0 && r0 == 0 && wave == NW - 1 && c == 0) store(size_t(a.n_exp) * T, half4_t{0, 0, 0, 0});     // the row of zeros
  if (!has_factors || r0 >= T) return;
  const bool live = 16 * tl < min(rank_m, a.rank);
  const bool q3 = ((q3_bits >> m) & 1) != 0;
  const int k32 = a.K / 32, g64 = a.K / 64, per = (k32 + NW - 1) / NW, kk0 = min(k32, wave * per), kk1 = min(k32, kk0 + per);
  float4_t acc[2] = {float4_t{0.f, 0.f, 0.f, 0.f}, float4_t{0.f, 0.f, 0.f, 0.f}};
  if (live) {
    const uint4* xrow[2];
    float xs2[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) xrow[t] = reinterpret_cast<const uint4*>(x_bf16 + size_t(min(r0 + 16 * t + c, T - 1)) * a.K);
    if (tok_exp != nullptr) {
#pragma unroll
      for (int t = 0; t < 2; ++t) xs2[t] = pow2i(tok_exp[min(r0 + 16 * t + c, T - 1)]);
    }
    // the rows' exponents from the rows themselves; `first`: the first units, which are multiplied next, are in hand
    auto exponents = [&](auto NT_, auto NB_, const auto& first) {
      constexpr int NT = decltype(NT_)::value, NB = decltype(NB_)::value;
      uint32_t* peak = reinterpret_cast<uint32_t*>(red);           // [NW][2][16]
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        uint32_t mx = 0;
        auto take = [&](const uint4& v) {
          const uint32_t in[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) mx = max(mx, max(in[i] & 0x7fffu, (in[i] >> 16) & 0x7fffu));
        };
#pragma unroll
        for (int u = 0; u < NB; ++u)
          if (kk0 + u < kk1) take(first[t][u]);
        for (int kk = kk0 + NB; kk < kk1; ++kk) take(xrow[t][4 * kk + q]);
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, 16));
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, 32));
        if (q == 0) peak[(wave * 2 + t) * 16 + c] = mx;
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        uint32_t mx = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) mx = max(mx, peak[(w * 2 + t) * 16 + c]);
        xs2[t] = pow2i(row_exponent(mx));
      }
      __syncthreads();
    };
    auto k_loop = [&](auto Q3_, auto TWO_) {
      constexpr bool Q3 = decltype(Q3_)::value, TWO = decltype(TWO_)::value;
      constexpr int NB = TWO ? BATCH : 2 * BATCH, NT = TWO ? 2 : 1;
      half8_t wf[NB];
      uint4 xv[NT][NB];
      uint32_t cq[NB], mq[NB];
      auto request = [&](int kk) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          const int ku = max(min(kk + u, kk1 - 1), 0);
          if constexpr (Q3) {
            cq[u] = aq[(size_t(tl) * k32 + ku) * kWave + lane];
            mq[u] = am[(size_t(tl) * g64 + (ku >> 1)) * 16 + c];
          } else {
            wf[u] = af[(size_t(tl) * k32 + ku) * kWave + lane];
          }
#pragma unroll
          for (int t = 0; t < NT; ++t) xv[t][u] = xrow[t][4 * ku + q];
        }
        asm volatile("" ::: "memory");         // (none of them is moved behind the tests below)
      };
      request(kk0);
      if (tok_exp == nullptr) exponents(std::integral_constant<int, NT>{}, std::integral_constant<int, NB>{}, xv);
      for (int kk = kk0; kk < kk1; kk += NB) {
        if (kk > kk0) request(kk);
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          if (kk + u >= kk1) break;            // (a step past this wavefront's share)
          if constexpr (Q3) wf[u] = q3_unit_a(cq[u], mq[u]);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const half8_t xf = scaled_unit(xv[t][u], xs2[t]);
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[u], xf, acc[t], 0, 0, 0);
          }
        }
      }
    };
    const bool two = wide && r0 + 16 < T;
    if (q3) { if (two) k_loop(std::true_type{}, std::true_type{}); else k_loop(std::true_type{}, std::false_type{}); }
    else { if (two) k_loop(std::false_type{}, std::true_type{}); else k_loop(std::false_type{}, std::false_type{}); }
    red[wave][lane] = acc[0];
    red[NW + wave][lane] = acc[1];
    __syncthreads();
  }
  // wavefront t: lane (q, c) columns 16 tl + 4 q .. + 3 of token r0 + 16 t + c
  if (wave < (wide ? 2 : 1) && r0 + 16 * wave + c < T) {
    half4_t v = half4_t{0, 0, 0, 0};
    if (live) {
      float4_t sum = red[wave * NW][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += red[wave * NW + w][lane];
      v = half4_t{to_f16_sat(sum[0] * lam), to_f16_sat(sum[1] * lam), to_f16_sat(sum[2] * lam), to_f16_sat(sum[3] * lam)};
    }
    store(size_t(e) * T + r0 + 16 * wave + c, v);
  }
}

}  // namespace ffn
}  // namespace lrc
