// Device-side pieces of the routing (Section 2.1: w = softmax(G(x)), Top-k) shared by the routing
// kernels and by the launch that prepares the activations, which routes a handful of tokens itself.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace lrc {

__device__ inline double bf16_to_double(uint32_t bits16) {
  return (double)__uint_as_float(bits16 << 16);
}

// The value of lane ^ OFF, in pairs: fn(v, other) over both gives what a butterfly by shuffles gives, inside the vector
// registers (a shuffle goes through the LDS unit: about 100 cycles a step against 20).
template <int OFF> __device__ inline void lane_pair(uint32_t v, uint32_t& a, uint32_t& b) {
  static_assert(OFF == 32 || OFF == 16 || OFF == 8 || OFF == 4 || OFF == 2 || OFF == 1, "a power of two below 64");
  if constexpr (OFF >= 16) {               // halves or rows of 16 lanes swapped: own and other, in lane order
    const auto r = OFF == 32 ? __builtin_amdgcn_permlane32_swap(v, v, false, false) : __builtin_amdgcn_permlane16_swap(v, v, false, false);
    a = r[0]; b = r[1];
  } else {
    a = v;
    if constexpr (OFF == 8) b = __builtin_amdgcn_update_dpp(0, int(v), 0x128, 0xf, 0xf, true);            // row_ror 8
    else if constexpr (OFF == 4) {         // banks 0 and 2 of a row from 4 lanes up, 1 and 3 from 4 lanes down
      b = __builtin_amdgcn_update_dpp(0, int(v), 0x104, 0xf, 0x5, false);
      b = __builtin_amdgcn_update_dpp(int(b), int(v), 0x114, 0xf, 0xa, false);
    } else b = __builtin_amdgcn_update_dpp(0, int(v), OFF == 2 ? 0x4e : 0xb1, 0xf, 0xf, true);            // quad_perm
  }
}
template <int OFF, class Fn> __device__ inline double lane_step(double v, Fn&& fn) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  uint32_t la, lb, ha, hb;
  lane_pair<OFF>(uint32_t(u), la, lb);
  lane_pair<OFF>(uint32_t(u >> 32), ha, hb);
  return fn(__builtin_bit_cast(double, (uint64_t(ha) << 32) | la), __builtin_bit_cast(double, (uint64_t(hb) << 32) | lb));
}
template <class Fn> __device__ inline double wave_reduce(double v, Fn&& fn) {
  v = lane_step<32>(v, fn); v = lane_step<16>(v, fn); v = lane_step<8>(v, fn);
  v = lane_step<4>(v, fn); v = lane_step<2>(v, fn); return lane_step<1>(v, fn);
}
__device__ inline double wave_sum(double v) { return wave_reduce(v, [](double a, double b) { return a + b; }); }
__device__ inline double wave_max(double v) { return wave_reduce(v, [](double a, double b) { return fmax(a, b); }); }

// Top-k of one token's logits (value descending, ties to the lower index), and
// the softmax weights of the selected experts (Section 2.1), by one wavefront: lane holds the
// logits of experts lane, lane + 64, lane + 128, lane + 192.
// Bound: the serial chain of top_k selections.  One is a wave maximum of the values alone; who holds it is read from
// ballots, and the exponentials and quotients wait until lane j holds the j-th value, so that all are taken at once
// (Top-8 of 128, T = 4096: 17.0 -> 10.3 us, shuffles with the index beside the value and an exponential per selection before;
// Top-6 of 64, T = 512: 8.3 -> 6.0).
__device__ inline void select_topk(const double (&v)[4], int lane, int E, int top_k, int renorm,
                                   int32_t* __restrict__ idx_t, float* __restrict__ w_t, int32_t* idx_l = nullptr) {
  uint32_t taken = 0;
#pragma unroll
  for (int m = 0; m < 4; ++m)
    if (lane + 64 * m >= E) taken |= 1u << m;
  double vmax = 0.0, my_v = 0.0;
  int my_idx = 0;
  for (int j = 0; j < top_k; ++j) {
    double bv = 0.0;
    int bm = -1;                             // this lane's best: register bm
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if (!(taken & (1u << m)) && (bm < 0 || v[m] > bv)) { bv = v[m]; bm = m; }
    const double best = wave_max(bm >= 0 ? bv : -__builtin_huge_val());
    int bi = -1;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const unsigned long long at = __ballot(bm == m && bv == best);
      if (bi < 0 && at != 0) bi = 64 * m + __ffsll(at) - 1;
    }
    if (bi < 0) {                            // (only NaN is left: the lowest expert not taken)
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const unsigned long long at = __ballot(!(taken & (1u << m)));
        if (bi < 0 && at != 0) bi = 64 * m + __ffsll(at) - 1;
      }
    }
    if ((bi & 63) == lane) taken |= 1u << (bi >> 6);
    if (j == 0) vmax = best;
    if (lane == j) { my_v = best; my_idx = bi; }
  }
  if (idx_l != nullptr) {                  // (a second place for the experts, and no weights wanted without the first)
    if (lane < top_k) idx_l[lane] = my_idx;
    if (idx_t == nullptr) return;
  }
  double part = 0.0;
#pragma unroll
  for (int m = 0; m < 4; ++m)
    if (lane + 64 * m < E) part += exp(v[m] - vmax);
  const double den = wave_sum(part), score = exp(my_v - vmax) / den;
  double sel_sum = 0.0;
  if (renorm)
    for (int j = 0; j < top_k; ++j) sel_sum += __shfl(score, j);
  if (lane < top_k) {
    idx_t[lane] = my_idx;
    w_t[lane] = (float)(renorm ? score / sel_sum : score);
  }
}


// The whole routing of a token or two (at most kFusedRoutePairs (token, expert) pairs) by one
// 1024-thread block: every (token, expert) gate dot product by one wavefront, with the lanes walking
// the 16-byte chunks of the rows and adding the exact bf16 x bf16 products in fp64 in the order the
// per-token routing kernel uses (the logits are bit-identical to that kernel's); then one wavefront
// per token takes the Top-k and the softmax weights and the token's pre-scale exponent.
// `logit` is LDS, T * E doubles; the selected experts and the exponents are left in LDS (idx_l, exp_l) for the
// __syncthreads() the caller follows this with, and written out by the one block that is asked to (`out`).
__device__ inline void route_small_body(double* logit, int32_t* idx_l, int32_t* exp_l, const uint16_t* __restrict__ x, const RouteArgs& ra,
                                        int T, int H, int E, int top_k, bool out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, chunks = H / 8;
  for (int p = wave; p < T * E; p += 16) {
    const int t = p / E, e = p - t * E;
    const uint4* xrow = reinterpret_cast<const uint4*>(x + size_t(t) * H);
    const uint4* wrow = reinterpret_cast<const uint4*>(ra.wg + size_t(e) * H);
    double acc = 0.0;
    constexpr int kAhead = 8;
    for (int c0 = lane; c0 < chunks; c0 += 64 * kAhead) {      // eight chunks of both rows in flight
      uint4 xv[kAhead], wv[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int c = c0 + 64 * u;
        xv[u] = c < chunks ? xrow[c] : make_uint4(0, 0, 0, 0);
        wv[u] = c < chunks ? wrow[c] : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {                   // (chunks in increasing order; a chunk of zeros adds nothing)
        const uint32_t xa[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w}, wa[4] = {wv[u].x, wv[u].y, wv[u].z, wv[u].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc = fma(bf16_to_double(xa[i] & 0xffffu), bf16_to_double(wa[i] & 0xffffu), acc);
          acc = fma(bf16_to_double(xa[i] >> 16), bf16_to_double(wa[i] >> 16), acc);
        }
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) logit[p] = acc + (ra.bias ? (double)ra.bias[e] : 0.0);
  }
  // the tokens' pre-scale exponents (ffn_common.h), by the last wavefronts, which have no product where there are fewer than 16
  if (15 - wave < T) {
    const int t = 15 - wave;
    const uint4* xrow = reinterpret_cast<const uint4*>(x + size_t(t) * H);
    uint32_t m = 0;
    for (int c0 = lane; c0 < chunks; c0 += 64 * 8) {
      uint4 xv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) xv[u] = xrow[min(c0 + 64 * u, chunks - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t xa[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) m = max(m, max(xa[i] & 0x7fffu, (xa[i] >> 16) & 0x7fffu));
      }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
    const int eb = int(m >> 7);
    const int se = eb == 0 ? 0 : min(60, max(-60, 127 - eb));
    if (lane == 0) exp_l[t] = se;
    if (lane == 0 && out) ra.tok_exp[t] = se;
  }
  __syncthreads();
  if (wave < T) {
    double v[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int e = lane + 64 * m;
      v[m] = e < E ? logit[wave * E + e] : 0.0;
    }
    select_topk(v, lane, E, top_k, ra.renorm, out ? ra.idx + size_t(wave) * top_k : nullptr, out ? ra.w + size_t(wave) * top_k : nullptr,
                idx_l + wave * top_k);
  }
}

}  // namespace lrc
