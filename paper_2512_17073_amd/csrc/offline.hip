// The offline half of the method on the device, in fp64: group-wise uniform quantization of a weight
// matrix (Section 2.3), its residual E = W - Qinv(Q(W)), the rank-r factors of the residual
// (Section 3.1 step 2: SVD_r(E) = U S V^T, stored as A = U sqrt(S), B = sqrt(S) V^T) and the kurtosis of
// a matrix (Section 3.1 step 1).  Not part of the hot path: these calls allocate their own buffers
// and synchronise.
//
// Factors: a randomized subspace iteration (Halko, Martinsson, Tropp) driven by a caller-supplied
// test matrix Omega, so that both sides of a comparison can use the same random numbers:
//   Y = E Omega;  repeat `power_iters` times:  Y <- E (E^T orth(Y));  Q = orth(Y);  Bm = Q^T E  (l x N)
//   SVD of the small matrix Bm by one-sided Jacobi rotations of its rows (Hestenes), which leaves
//   rows sigma_i w_i^T and accumulates the rotations G: Bm = G diag(sigma) W^T, so U = Q G.
// orth() is a Cholesky QR (Gram matrix, Cholesky factor, triangular solve), applied twice where
// the result is used as an orthonormal basis and once between the passes of the iteration, where only
// its span counts: the residual of a quantizer is close to white noise, its leading singular values
// are nearly flat, and the Gram matrix of l such directions is well conditioned.
// What the call cannot do without is six products with E (K x N times N x l, or transposed); they run
// on the fp64 matrix cores (dgemm_kernel).  Everything else is small: for l <= kSmallL it stays on the
// device without a host round trip, and the Jacobi rotations run on the l x l Cholesky factor of
// Bm Bm^T in the LDS of one block (Bm = L Q_b^T: rotating rows of Bm and of L is the same thing)
// instead of l - 1 launches per sweep over the l x N matrix (9.4 -> 0.26 ms at l = 40, N = 14336).  The
// whole call at 4096 x 14336, rank 32, l = 40, two passes: 24.2 -> 1.72 ms.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <type_traits>
#include <vector>

#include "gemm_cut.h"
#include "internal.h"
#include "offline_round.h"

namespace lrc {
namespace {

// ---------------------------------------------------------------------------------- quantizer
// One thread per (group, column): minimum and maximum of the group's `group` entries, then scale and
// zero rounded to fp16 before the codes are chosen (so the codes are optimal for the stored values),
// then the codes and, if wanted, the residual.  A constant group, or one whose scale rounds to zero
// or overflows in fp16, gets scale 1, zero = -min and codes 0.
__global__ __launch_bounds__(256) void quantize_kernel(const double* __restrict__ W, int K, int N, int bits, int group,
                                                       uint8_t* __restrict__ codes, uint16_t* __restrict__ scale,
                                                       uint16_t* __restrict__ zero, double* __restrict__ resid) {
#pragma clang fp contract(off)      // every product and sum rounded on its own, as written
  const int n = blockIdx.x * 256 + threadIdx.x, g = blockIdx.y;
  if (n >= N) return;
  const double* w = W + size_t(g) * group * N + n;
  double lo = w[0], hi = w[0];
  for (int i = 1; i < group; ++i) {
    const double v = w[size_t(i) * N];
    lo = v < lo ? v : lo;
    hi = v > hi ? v : hi;
  }
  const int levels = (1 << bits) - 1;
  uint16_t sb = f64_to_f16_bits((hi - lo) / double(levels));
  double s = f16_bits_to_f64(sb);
  const bool degenerate = !(s > 0.0) || (sb & 0x7fffu) >= 0x7c00u;
  uint16_t zb;
  if (degenerate) {
    sb = 0x3c00u; s = 1.0;
    zb = f64_to_f16_bits(-lo);
  } else {
    zb = f64_to_f16_bits(-lo / s);
  }
  const double z = f16_bits_to_f64(zb);
  scale[size_t(g) * N + n] = sb;
  zero[size_t(g) * N + n] = zb;
  for (int i = 0; i < group; ++i) {
    const size_t at = (size_t(g) * group + i) * N + n;
    const double v = w[size_t(i) * N];
    double q = degenerate ? 0.0 : __builtin_rint(v / s + z);      // round half to even
    q = q < 0.0 ? 0.0 : (q > double(levels) ? double(levels) : q);
    if (!(q == q)) q = 0.0;
    codes[at] = uint8_t(int(q));
    if (resid) resid[at] = v - (q - z) * s;
  }
}

// The same for the usual groups: 64 columns (CPL per lane) x one group per block, the group's rows shared
// by four wavefronts of R rows each, whose part stays in registers: the matrix is read once, 16 bytes
// per lane where N is even.  Minimum and maximum do not depend on the order they are taken in.
// Bound: HBM (read 8, write 9 bytes per entry): 1.0 GB at 4096 x 14336 in 163 us, 6.1 TB/s (a large streaming read
// reaches 5.9 here); reading the group twice, one column per thread, took 333.
template <int R, int CPL>
__global__ __launch_bounds__(256) void quantize_rows_kernel(const double* __restrict__ W, int K, int N, int bits,
                                                            uint8_t* __restrict__ codes, uint16_t* __restrict__ scale,
                                                            uint16_t* __restrict__ zero, double* __restrict__ resid) {
#pragma clang fp contract(off)      // every product and sum rounded on its own, as written
  typedef double vec_t __attribute__((ext_vector_type(CPL), aligned(8)));
  __shared__ double mm[2][4][64 * CPL];
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6, g = blockIdx.y;
  const int n = (blockIdx.x * 64 + lane) * CPL;
  const bool in = n < N;                                   // (CPL == 2: N is even)
  const size_t at = (size_t(g) * 4 + part) * R * N + (in ? n : N - CPL);
  vec_t w[R];
#pragma unroll
  for (int i = 0; i < R; ++i) w[i] = *reinterpret_cast<const vec_t*>(W + at + size_t(i) * N);
  const int levels = (1 << bits) - 1;
  double lo[CPL], hi[CPL], s[CPL], z[CPL];
  bool degenerate[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    // (the one-thread form starts from the group's first entry and skips NaNs that come later)
    lo[c] = part == 0 ? w[0][c] : HUGE_VAL;
    hi[c] = part == 0 ? w[0][c] : -HUGE_VAL;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      lo[c] = w[i][c] < lo[c] ? w[i][c] : lo[c];
      hi[c] = w[i][c] > hi[c] ? w[i][c] : hi[c];
    }
    mm[0][part][lane * CPL + c] = lo[c]; mm[1][part][lane * CPL + c] = hi[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    lo[c] = mm[0][0][lane * CPL + c]; hi[c] = mm[1][0][lane * CPL + c];
#pragma unroll
    for (int p = 1; p < 4; ++p) {
      const double a = mm[0][p][lane * CPL + c], b = mm[1][p][lane * CPL + c];
      lo[c] = a < lo[c] ? a : lo[c];
      hi[c] = b > hi[c] ? b : hi[c];
    }
    uint16_t sb = f64_to_f16_bits((hi[c] - lo[c]) / double(levels)), zb;
    s[c] = f16_bits_to_f64(sb);
    degenerate[c] = !(s[c] > 0.0) || (sb & 0x7fffu) >= 0x7c00u;
    if (degenerate[c]) {
      sb = 0x3c00u; s[c] = 1.0;
      zb = f64_to_f16_bits(-lo[c]);
    } else {
      zb = f64_to_f16_bits(-lo[c] / s[c]);
    }
    z[c] = f16_bits_to_f64(zb);
    if (in && part == 0) {
      scale[size_t(g) * N + n + c] = sb;
      zero[size_t(g) * N + n + c] = zb;
    }
  }
  if (!in) return;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    uint32_t q8 = 0;
    vec_t r;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const double v = w[i][c];
      double q = degenerate[c] ? 0.0 : __builtin_rint(v / s[c] + z[c]);      // round half to even
      q = q < 0.0 ? 0.0 : (q > double(levels) ? double(levels) : q);
      if (!(q == q)) q = 0.0;
      q8 |= uint32_t(uint8_t(int(q))) << (8 * c);
      r[c] = v - (q - z[c]) * s[c];
    }
    if constexpr (CPL == 2) *reinterpret_cast<uint16_t*>(codes + at + size_t(i) * N) = uint16_t(q8);
    else codes[at + size_t(i) * N] = uint8_t(q8);
    if (resid) *reinterpret_cast<vec_t*>(resid + at + size_t(i) * N) = r;
  }
}

// The same with the zero points refined by a half-quadratic solver ("HQQ-style weight optimization",
// Section 3.1 step 2; the published scheme: l_p error, p < 1, penalty beta growing by kappa per step).
// Per group, scale fixed, zero point z real-valued:
//   q = clamp(round(w / s + z));  e = shrink(w - (q - z) s);  z = mean(q - (w - e) / s);  beta *= kappa
// with shrink(x) = sign(x) max(|x| - |x|^(p-1) / beta, 0); then z is rounded to fp16 and the codes are
// chosen for the stored values.  Sums run in index order.
// shrink() is zero below tau = beta^(-1 / (2 - p)), where x = x^(p-1) / beta: an entry whose |x| is clearly
// below it (the usual case: |x| is at most half a step unless the code is clamped) needs no pow(), and
// (w - 0) / s is the quotient that chose the code, the same in every step.  G > 0: the group has G
// entries and their quotients stay in registers; a step in which some entry of the group is not far
// below the threshold is redone with the entries re-read.  G == 0: any group, re-read in every step (64 quotients in
// fp64 already take 346 of a lane's 512 registers: groups of 128 and 256 do not fit and stay here, 2.8 and 3.3 times as
// fast as before the threshold; 2048 x 1408: 674 and 1169 us).
// tau: beta^(-1 / (2 - p)), times tau_step = kappa^(-1 / (2 - p)) after every step.
// Bound: fp64 issue of one wavefront per SIMD (704 of them for 2048 x 1408), six operations per entry and step.
// 2048 x 1408, 3 bits, 20 steps: 975 us with pow() and two divisions per entry and step, 71 us with twelve
// operations and four selects in a dependent row, 35 us so (reading and writing the matrices is 8 of them).
template <int G>
__global__ __launch_bounds__(64) void quantize_refined_kernel(const double* __restrict__ W, int K, int N, int bits, int group_,
                                                               int iters, double p, double beta, double kappa, double tau, double tau_step,
                                                               uint8_t* __restrict__ codes, uint16_t* __restrict__ scale,
                                                               uint16_t* __restrict__ zero, double* __restrict__ resid) {
#pragma clang fp contract(off)
  const int n = blockIdx.x * 64 + threadIdx.x, g = blockIdx.y, group = G > 0 ? G : group_;
  if (n >= N) return;
  const double* w = W + size_t(g) * group * N + n;
  double ratio[G > 0 ? G : 1];                             // first the entries, then entry / scale
  double lo, hi;
  if constexpr (G > 0) {
#pragma unroll
    for (int i = 0; i < G; ++i) ratio[i] = w[size_t(i) * N];
    lo = hi = ratio[0];
#pragma unroll
    for (int i = 1; i < G; ++i) {
      lo = ratio[i] < lo ? ratio[i] : lo;
      hi = ratio[i] > hi ? ratio[i] : hi;
    }
  } else {
    lo = hi = w[0];
    for (int i = 1; i < group; ++i) {
      const double v = w[size_t(i) * N];
      lo = v < lo ? v : lo;
      hi = v > hi ? v : hi;
    }
  }
  const int levels = (1 << bits) - 1;
  uint16_t sb = f64_to_f16_bits((hi - lo) / double(levels));
  double s = f16_bits_to_f64(sb);
  const bool degenerate = !(s > 0.0) || (sb & 0x7fffu) >= 0x7c00u;
  double z;
  if (degenerate) { sb = 0x3c00u; s = 1.0; z = -lo; }
  else z = -lo / s;
  if constexpr (G > 0) {
#pragma unroll
    for (int i = 0; i < G; ++i) ratio[i] = ratio[i] / s;
  }
  auto clamped = [&](double r) {
    double q = __builtin_rint(r + z);
    return q < 0.0 ? 0.0 : (q > double(levels) ? double(levels) : q);
  };
  double r_lo = 0.0, r_hi = 0.0;                           // the group's smallest and largest quotient
  if constexpr (G > 0) {
    r_lo = lo / s; r_hi = hi / s;                          // (a quotient by one positive number keeps the order)
  }
  if (!degenerate) {
    double b = beta;
    for (int it = 0; it < iters; ++it) {
      double sum = 0.0;
      // |x| = |v - (q - z) s| is s |v / s - (q - z)| up to rounding (a few units in the last place of both terms)
      const double far = tau * (1.0 - 1e-6) / s;
      bool all_far = G > 0;
      if constexpr (G > 0) {
        // Six fp64 operations per entry.  |r - (q - z)| is at most one half where q is not clamped, and largest at
        // the group's ends where it is: the threshold is tested once for the group (with the magnitudes that
        // rounding is relative to), and a group it does not clear is redone entry by entry below, to the same sum.
        // The clamp is a maximum and a minimum: an entry that is not a number makes the sum, and so the zero
        // point, not a number whatever its q is, and the codes are chosen by clamped().  kWide entries at a time,
        // an operation for all of them before the next and an addition of the serial sum in between: a wavefront
        // has its SIMD to itself, and one entry after the other waits for every operation's result.
        const double top = double(levels), ends = fmax(r_hi + z - top, -(r_lo + z));
        all_far = fmax(ends, 0.5) + (fabs(r_lo) + fabs(r_hi) + fabs(z) + top) * 2e-14 < far;
        constexpr int kWide = 4;
        double q[kWide], add[kWide] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i <= G; i += kWide) {
#pragma unroll
          for (int op = 0; op < 4; ++op) {
            if (i < G) {
#pragma unroll
              for (int u = 0; u < kWide; ++u)
                q[u] = op == 0 ? ratio[i + u] + z : op == 1 ? __builtin_rint(q[u]) : op == 2 ? fmax(q[u], 0.0) : fmin(q[u], top);
            }
            sum += add[op];                                // (those of the entries before, in index order)
            __builtin_amdgcn_sched_barrier(0);
          }
          if (i < G) {
#pragma unroll
            for (int u = 0; u < kWide; ++u) add[u] = q[u] - ratio[i + u];
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      if (!all_far) {
        sum = 0.0;
#pragma unroll 1
        for (int i = 0; i < group; ++i) {
          const double v = w[size_t(i) * N], r = v / s, q = clamped(r);
          double add = q - r;
          if (!(fabs(r - (q - z)) + (fabs(r) + fabs(q - z)) * 1e-14 < far)) {
            const double x = v - (q - z) * s, ax = fabs(x);
            double e = 0.0;
            if (ax > 0.0) {
              const double t = ax - pow(ax, p - 1.0) / b;
              e = t > 0.0 ? (x < 0.0 ? -t : t) : 0.0;
            }
            add = q - (v - e) / s;
          }
          sum += add;
        }
      }
      z = sum / double(group);
      b *= kappa;
      tau *= tau_step;
    }
  }
  const uint16_t zb = f64_to_f16_bits(z);
  z = f16_bits_to_f64(zb);
  scale[size_t(g) * N + n] = sb;
  zero[size_t(g) * N + n] = zb;
  auto store = [&](int i, double v, double r) {
    const size_t at = (size_t(g) * group + i) * N + n;
    double q = degenerate ? 0.0 : clamped(r);
    if (!(q == q)) q = 0.0;
    codes[at] = uint8_t(int(q));
    if (resid) resid[at] = v - (q - z) * s;
  };
  if constexpr (G > 0) {
#pragma unroll
    for (int i0 = 0; i0 < G; i0 += 16) {                   // sixteen entries in flight
      double v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = resid ? w[size_t(i0 + i) * N] : 0.0;
#pragma unroll
      for (int i = 0; i < 16; ++i) store(i0 + i, v[i], ratio[i0 + i]);
    }
  } else {
    for (int i = 0; i < group; ++i) store(i, w[size_t(i) * N], w[size_t(i) * N] / s);
  }
}

// ---------------------------------------------------------------------------------- kurtosis
// Count, mean and sums of the second to fourth powers of the distance to the mean of a set of values; two
// sets are joined by Pebay's formulas, which lose nothing to cancellation, so one pass over the matrix
// is enough (115 us at 4096 x 14336, 80 at the streaming rate; the mean and then two centred sums took 390).
struct Moments { double n, mean, m2, m3, m4; };
__device__ inline Moments join(const Moments& a, const Moments& b) {
  if (a.n == 0.0) return b;
  if (b.n == 0.0) return a;
  const double n = a.n + b.n, d = b.mean - a.mean, dn = d / n, ab = a.n * b.n;
  Moments r;
  r.n = n;
  r.mean = a.mean + dn * b.n;
  const double t = d * dn * ab;            // (counts are multiplied in first: no term is smaller on the way than at the end)
  r.m2 = a.m2 + b.m2 + t;
  r.m3 = a.m3 + b.m3 + t * (a.n - b.n) * dn + 3.0 * dn * (a.n * b.m2 - b.n * a.m2);
  r.m4 = a.m4 + b.m4 + t * (a.n * a.n - ab + b.n * b.n) * dn * dn + 6.0 * (a.n * a.n * b.m2 + b.n * b.n * a.m2) * dn * dn +
         4.0 * dn * (a.n * b.m3 - b.n * a.m3);
  return r;
}
constexpr int kMomentTile = 16;          // values a thread holds at once
__device__ inline void join_block(Moments (&red)[256], const Moments& mine) {      // result in red[0]
  red[threadIdx.x] = mine;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = join(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
}
// Block b takes the tiles of 256 x kMomentTile values b, b + gridDim.x, ...; one result per block, joined by
// one block afterwards (a fixed order: deterministic), so that 40 bytes go to the host.
__global__ __launch_bounds__(256) void moment_kernel(const double* __restrict__ w, size_t n, Moments* __restrict__ out) {
  __shared__ Moments red[256];
  constexpr size_t kTile = 256 * kMomentTile;
  Moments acc{0.0, 0.0, 0.0, 0.0, 0.0};
  for (size_t t0 = size_t(blockIdx.x) * kTile; t0 < n; t0 += size_t(gridDim.x) * kTile) {
    double v[kMomentTile];
    Moments m{0.0, 0.0, 0.0, 0.0, 0.0};
    if (t0 + kTile <= n) {
#pragma unroll
      for (int u = 0; u < kMomentTile; ++u) v[u] = w[t0 + size_t(u) * 256 + threadIdx.x];
      double sum = v[0];
#pragma unroll
      for (int u = 1; u < kMomentTile; ++u) sum += v[u];
      m.n = kMomentTile;
      m.mean = sum * (1.0 / kMomentTile);
#pragma unroll
      for (int u = 0; u < kMomentTile; ++u) {
        const double d = v[u] - m.mean, d2 = d * d;
        m.m2 += d2; m.m3 = fma(d2, d, m.m3); m.m4 = fma(d2, d2, m.m4);
      }
      // (the mean of the tile is rounded: what is left of the first moment moves the others by less than
      // their own rounding)
    } else {
      for (int u = 0; u < kMomentTile; ++u) {
        const size_t i = t0 + size_t(u) * 256 + threadIdx.x;
        if (i < n) m = join(m, Moments{1.0, w[i], 0.0, 0.0, 0.0});
      }
    }
    acc = join(acc, m);
  }
  join_block(red, acc);
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}
__global__ __launch_bounds__(256) void moment_join_kernel(Moments* part, int parts) {
  __shared__ Moments red[256];
  Moments acc{0.0, 0.0, 0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < parts; i += 256) acc = join(acc, part[i]);
  join_block(red, acc);
  if (threadIdx.x == 0) part[0] = red[0];
}

// ---------------------------------------------------------------------------------- dense fp64 products
// C[M][Nc] = op(A) B with op(A)[i][k] = TRANS ? A[k * lda + i] : A[i * lda + k] and B[k * ldb + j], on
// v_mfma_f64_16x16x4.  The products here are tall and skinny: A is the K x N matrix, read once, and B
// is a few megabytes, so a block of four wavefronts takes 128 rows of C and all its columns up to
// 16 CT, a wavefront 32 rows (two tiles that share every B operand read from LDS).  The reduction dimension, in chunks of 32, is split
// over the blocks (gemm_cut.h), each writing its own partial C (dsum_kernel adds them in order).  The chunks of A
// come through a ring of registers, two chunks ahead, those of B through another and then the other half of LDS; all are requested
// before the current chunk is multiplied.  Inside
// a chunk, MFMA step (h, s) covers k = 16 h + 4 kq + s for lane group kq, so that a lane reads 32
// contiguous bytes of a row of A.  TRANS: a lane reads two adjacent entries of a row of A, which are
// rows 2 i and 2 i + 1 of the wavefront's 32: tile rt holds the rows of parity rt.
// Bound: HBM (470 MB per product at 4096 x 14336: 80 us at the streaming rate) and the fp64 matrix rate
// (5.6 GFLOP with 40 columns padded to 48: 80 us) about equally.  Measured, plain / transposed: 133 / 130 us with three
// blocks per CU that asked for one chunk ahead and had up to 14 % unequal work, 126 / 123 us so (512 equal blocks); without the products
// the loads took 101 / 97 us, without A's loads the products 99 / 112.  4096 x 14336 with 56 columns: a call of 2470 -> 2256 us, 14336 x
// 4096 with 72 (two column groups) 4140 -> 3595.
typedef double double4_t __attribute__((ext_vector_type(4)));
typedef double double2_t __attribute__((ext_vector_type(2), aligned(8)));
constexpr int kRing = 3;

// The loop over whole chunks has no branch around a load in it (a guarded load is a branch, and the compiler then
// waits for every load in flight before the next): the last chunks' prefetches repeat the last chunk, rows
// of a wavefront that would end past M start earlier (PAIR; for M < 32 the entries are read one by one,
// clamped), what lies past the edges of B becomes zero on its way into LDS, and a last partial chunk is
// read with clamped indices after the loop.
template <bool TRANS, int CT, bool PAIR = true>
__global__ __launch_bounds__(256, 2) void dgemm_kernel(GemmCut cut, int M, int Nc, int Kd, const double* __restrict__ A, int lda,
                                                    const double* __restrict__ B, int ldb, double* __restrict__ C, int ldc,
                                                    double* __restrict__ part, size_t part_stride) {
  constexpr int kPitch = 16 * CT + 4;                  // (lane groups 4 rows apart then sit in different halves of the banks)
  constexpr int kLoadsB = kGemmK * 16 * CT / 256;
  __shared__ double Bs[2][kGemmK * kPitch];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), i = lane & 15, kq = lane >> 4;
  const int j0 = blockIdx.x * (16 * CT), block = blockIdx.y;
  // this block's chunks, counted over all row blocks
  const long long hi = cut.end(block);
  for (long long at = cut.begin(block); at < hi;) {    // the row blocks among them
    const int y = int(at / cut.chunks), first = int(at - (long long)y * cut.chunks), last = int(min((long long)cut.chunks, first + (hi - at)));
    const int z = cut.part_of(block, y);
    at += last - first;
    const int m_first = y * kGemmRows + wave * 32;
    const int m0 = TRANS && PAIR ? max(0, min(m_first, M - 32)) : m_first;
    const int k_lo = first * kGemmK, k_hi = min(Kd, last * kGemmK);
    double4_t acc[2][CT];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = double4_t{0.0, 0.0, 0.0, 0.0};
    // a[rt][4 h + s]: this lane's A operand of step (h, s)
    const double* a_row[2] = {A + size_t(min(m0 + i, M - 1)) * lda + 4 * kq, A + size_t(min(m0 + 16 + i, M - 1)) * lda + 4 * kq};   // !TRANS
    const double* a_col = A + size_t(4 * kq) * lda + (PAIR ? m0 + 2 * i : 0);                                                  // TRANS
    const int c0 = min(m0 + 2 * i, M - 1), c1 = min(m0 + 2 * i + 1, M - 1);
    auto load_a = [&](int k0, double (&a)[2][8]) {           // a whole chunk
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if constexpr (TRANS) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const double* row = a_col + size_t(k0 + 16 * h + u) * lda;
            if constexpr (PAIR) {
              const double2_t v = *reinterpret_cast<const double2_t*>(row);
              a[0][4 * h + u] = v[0]; a[1][4 * h + u] = v[1];
            } else {
              a[0][4 * h + u] = row[c0]; a[1][4 * h + u] = row[c1];
            }
          }
        } else {
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) {
            const double* p = a_row[rt] + k0 + 16 * h;
            const double2_t v = *reinterpret_cast<const double2_t*>(p), w = *reinterpret_cast<const double2_t*>(p + 2);
            a[rt][4 * h] = v[0]; a[rt][4 * h + 1] = v[1]; a[rt][4 * h + 2] = w[0]; a[rt][4 * h + 3] = w[1];
          }
        }
    };
    auto load_a_edge = [&](int k0, double (&a)[2][8]) {      // past k_hi: any finite value, B is zero there
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = min(k0 + 16 * (u >> 2) + 4 * kq + (u & 3), k_hi - 1);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          a[rt][u] = TRANS ? A[size_t(k) * lda + (rt ? c1 : c0)] : A[size_t(min(m0 + 16 * rt + i, M - 1)) * lda + k];
      }
    };
    auto load_b = [&](int k0, double (&b)[kLoadsB]) {
#pragma unroll
      for (int u = 0; u < kLoadsB; ++u) {
        const int x = t + 256 * u, kk = x / (16 * CT), j = j0 + x % (16 * CT);
        b[u] = B[size_t(min(k0 + kk, k_hi - 1)) * ldb + min(j, Nc - 1)];
      }
    };
    auto store_b = [&](double* bs, int k0, const double (&b)[kLoadsB]) {
#pragma unroll
      for (int u = 0; u < kLoadsB; ++u) {
        const int x = t + 256 * u, kk = x / (16 * CT), j = j0 + x % (16 * CT);
        bs[kk * kPitch + x % (16 * CT)] = (k0 + kk < k_hi && j < Nc) ? b[u] : 0.0;
      }
    };
    auto multiply = [&](const double (&a)[2][8], const double* buf) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double* bs = buf + (16 * (u >> 2) + 4 * kq + (u & 3)) * kPitch + i;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const double b = bs[16 * ct];
          acc[0][ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][u], b, acc[0][ct], 0, 0, 0);
          acc[1][ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][u], b, acc[1][ct], 0, 0, 0);
        }
      }
    };
    const int whole = (k_hi - k_lo) / kGemmK;
    double a[kRing][2][8], b[kRing][kLoadsB];
    __syncthreads();                                       // (the row block before this one has been multiplied)
    if (whole > 0) {
      const int k_last = k_lo + (whole - 1) * kGemmK;
#pragma unroll
      for (int u = 0; u < kRing - 1; ++u) {
        load_b(min(k_lo + u * kGemmK, k_last), b[u]);
        __builtin_amdgcn_sched_barrier(0);                 // (loads return in order: B's, wanted first, are in front)
        load_a(min(k_lo + u * kGemmK, k_last), a[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
      store_b(Bs[0], k_lo, b[0]);
      __syncthreads();
      // chunk ch, in slot u of the rings
      auto step = [&](int ch, auto U) {
        constexpr int u = decltype(U)::value, slot = (u + kRing - 1) % kRing;
        const int ahead = min(k_lo + (ch + kRing - 1) * kGemmK, k_last);
        load_b(ahead, b[slot]);
        __builtin_amdgcn_sched_barrier(0);
        load_a(ahead, a[slot]);
        __builtin_amdgcn_sched_barrier(0);                 // (the requests stay in front of the products)
        multiply(a[u], Bs[ch & 1]);
        __builtin_amdgcn_sched_barrier(0);
        store_b(Bs[(ch + 1) & 1], min(k_lo + (ch + 1) * kGemmK, k_last), b[(u + 1) % kRing]);
        __syncthreads();
      };
      int ch = 0;
      for (; ch + kRing <= whole; ch += kRing) {           // (no way out of its middle: the waits at its head would be for that, too)
        step(ch, std::integral_constant<int, 0>{});
        step(ch + 1, std::integral_constant<int, 1>{});
        step(ch + 2, std::integral_constant<int, 2>{});
      }
      if (ch < whole) step(ch, std::integral_constant<int, 0>{});
      if (ch + 1 < whole) step(ch + 1, std::integral_constant<int, 1>{});
    }
    const int k_tail = k_lo + whole * kGemmK;
    if (k_tail < k_hi) {
      load_a_edge(k_tail, a[0]);
      load_b(k_tail, b[0]);
      store_b(Bs[whole & 1], k_tail, b[0]);
      __syncthreads();
      multiply(a[0], Bs[whole & 1]);
    }
    // register r of lane (i, kq): row kq + 4 r, column i of the tile
    double* Cz = z == 0 ? C : part + (z - 1) * part_stride;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rho = kq + 4 * r, m = TRANS ? m0 + 2 * rho + rt : m0 + 16 * rt + rho;
        if (m >= m_first && m < M)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const int j = j0 + 16 * ct + i;
            if (j < Nc) Cz[size_t(m) * ldc + j] = acc[rt][ct][r];
          }
      }
  }
}

// C[x] += the sum over z >= 1 (in order) of part[z - 1][x], of the parts that row x / Nc has: C holds part 0
// Bound: with few rows and many parts the chain of reads, so eight are requested together: 100 x 6116, rank 32, 31 -> 13.5 us for both sums of a
// call, the call 667-690 -> 635-651 us; 185 x 3366, rank 56, 39 -> 22 us and 1248-1259 -> 1202-1233; 4096 x 14336 41 -> 36 us of 1540.
__global__ __launch_bounds__(256) void dsum_kernel(GemmCut cut, const double* __restrict__ part, int Nc, size_t n, double* __restrict__ C) {
  const size_t x = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (x >= n) return;
  const int parts = cut.parts_of(int(x / Nc) / kGemmRows);
  double v = C[x];
  constexpr int kAhead = 8;
  for (int z = 1; z < parts; z += kAhead) {
    double p[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) p[u] = part[size_t(min(z + u, parts - 1) - 1) * n + x];
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (z + u < parts) v += p[u];
  }
  C[x] = v;
}

// part: room for gemm_part_doubles doubles.  keep_parts: leaves the partial sums there (returns their
// number); else C (ldc == Nc when the reduction is split) holds the product.
template <bool TRANS>
int dgemm(int M, int Nc, int Kd, const double* A, int lda, const double* B, int ldb, double* C, double* part, bool keep_parts = false) {
  const GemmCut g = gemm_cut(M, Nc, Kd, keep_parts ? kGramParts : 0);
  const dim3 grid(g.gx, g.blocks());
  const size_t cs = size_t(M) * Nc;
  double* out = keep_parts ? part : C;
  double* more = keep_parts ? part + cs : part;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, nullptr, g, M, Nc, Kd, A, lda, B, ldb, out, Nc, more, cs); };
  auto pick = [&](auto CT_) {
    constexpr int CT = decltype(CT_)::value;
    if constexpr (TRANS) {
      if (M < 32) return go(dgemm_kernel<true, CT, false>);
    }
    go(dgemm_kernel<TRANS, CT, true>);
  };
  switch (g.ct) {
    case 1: pick(std::integral_constant<int, 1>{}); break;
    case 2: pick(std::integral_constant<int, 2>{}); break;
    case 3: pick(std::integral_constant<int, 3>{}); break;
    default: pick(std::integral_constant<int, 4>{}); break;
  }
  if (g.parts > 1 && !keep_parts)
    hipLaunchKernelGGL(dsum_kernel, dim3((unsigned)((cs + 255) / 256)), dim3(256), 0, nullptr, g, part, Nc, cs, C);
  return g.parts;
}

// ---------------------------------------------------------------------------------- small l: everything in one block's LDS
constexpr int kSmallL = 96;              // two l x (l + 1) fp64 matrices fit the LDS of a CU

// 1 / sqrt(v) for a positive normal v, from the hardware's estimate and two Newton steps
__device__ inline double rsqrt_newton(double v) {
  double y = __builtin_amdgcn_rsq(v);
  y = fma(y * 0.5, fma(-v * y, y, 1.0), y);
  return fma(y * 0.5, fma(-v * y, y, 1.0), y);
}

// Lower Cholesky factor L of the l x l matrix G = sum of `parts` partial matrices, and L^-1 (the same
// elimination applied to the identity); *bad is set if a pivot is not positive.  One block, one barrier
// per column: column j and row j of the inverse are read by everyone and written by nobody in step j.
constexpr int kCholThreads = 1024;
__global__ __launch_bounds__(kCholThreads) void cholesky_small_kernel(const double* __restrict__ part, int parts, int l,
                                                             double* __restrict__ L, double* __restrict__ Linv, int* __restrict__ bad) {
  extern __shared__ double sm[];
  const int pitch = l + 1, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  double* G = sm;
  double* X = sm + l * pitch;
  for (int e = threadIdx.x; e < l * l; e += kCholThreads) {
    double pv[kGramParts];
#pragma unroll
    for (int z = 0; z < kGramParts; ++z) pv[z] = part[size_t(min(z, parts - 1)) * l * l + e];
    double v = pv[0];
#pragma unroll
    for (int z = 1; z < kGramParts; ++z) v += z < parts ? pv[z] : 0.0;
    const int r = e / l, c = e - r * l;
    G[r * pitch + c] = v;
    X[r * pitch + c] = r == c ? 1.0 : 0.0;
    L[e] = 0.0; Linv[e] = 0.0;
  }
  for (int j = 0; j < l; ++j) {
    __syncthreads();
    const double p = G[j * pitch + j];
    if (!(p > 0.0) && threadIdx.x == 0) *bad = 1;
    const double inv = rsqrt_newton(p > 0.0 ? p : 1.0);
    for (int x = threadIdx.x; x < l; x += kCholThreads) {
      if (x >= j) L[size_t(x) * l + j] = G[x * pitch + j] * inv;
      if (x <= j) Linv[size_t(j) * l + x] = X[j * pitch + x] * inv;
    }
    for (int r = j + 1 + ty; r < l; r += kCholThreads / 32) {
      const double f = G[r * pitch + j] * inv;
#pragma unroll
      for (int u = 0; u < kSmallL / 32; ++u) {
        const int c = tx + 32 * u;
        if (c > r) break;
        double* at = c <= j ? X + r * pitch + c : G + r * pitch + c;
        const double v = c <= j ? X[j * pitch + c] : G[c * pitch + j];
        *at = fma(-f, v * inv, *at);
      }
    }
  }
}

// out = in S for in [rows][l], S [l][cols] (ST: S is given transposed, [cols][l]); cols, l <= kSmallL.
// A wavefront holds its 16 rows in registers before it writes: out may be in.
template <bool ST>
__global__ __launch_bounds__(256) void rmul_kernel(const double* in, int rows, int l, const double* __restrict__ S, int cols, double* out,
                                                   const int* __restrict__ status) {
  extern __shared__ double sm[];
  if (status != nullptr && (status[0] | status[1] | status[2])) return;
  const int ct_n = (cols + 15) / 16, ks_n = (l + 3) / 4, pitch = 16 * ct_n + 4;
  for (int e = threadIdx.x; e < 4 * ks_n * 16 * ct_n; e += 256) {
    const int k = e / (16 * ct_n), c = e - k * (16 * ct_n);
    sm[k * pitch + c] = (k < l && c < cols) ? (ST ? S[size_t(c) * l + k] : S[size_t(k) * cols + c]) : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int r0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
  if (r0 >= rows) return;
  double a[kSmallL / 4];
  const double* row = in + size_t(min(r0 + i, rows - 1)) * l;
#pragma unroll
  for (int s = 0; s < kSmallL / 4; ++s) a[s] = s < ks_n ? row[min(4 * s + kq, l - 1)] : 0.0;   // (past l: times a zero row of S)
  for (int ct = 0; ct < ct_n; ++ct) {
    double4_t acc = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < kSmallL / 4; ++s)
      if (s < ks_n) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], sm[(4 * s + kq) * pitch + 16 * ct + i], acc, 0, 0, 0);
    const int c = 16 * ct + i;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rr = r0 + kq + 4 * r;
      if (rr < rows && c < cols) out[size_t(rr) * cols + c] = acc[r];
    }
  }
}

// B[r][n] = sum_j S[r][j] Z[n][j] for S [rank][l], Z [N][l]: the transposed product, stored in rows of n.
__global__ __launch_bounds__(256) void bt_kernel(const double* __restrict__ Z, int N, int l, const double* __restrict__ S, int rank,
                                                 double* __restrict__ B, const int* __restrict__ status) {
  extern __shared__ double sm[];
  if (status[0] | status[1] | status[2]) return;
  const int rt_n = (rank + 15) / 16, ks_n = (l + 3) / 4, pitch = 4 * ks_n + 1;
  for (int e = threadIdx.x; e < 16 * rt_n * 4 * ks_n; e += 256) {
    const int r = e / (4 * ks_n), k = e - r * (4 * ks_n);
    sm[r * pitch + k] = (r < rank && k < l) ? S[size_t(r) * l + k] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int n0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
  if (n0 >= N) return;
  double z[kSmallL / 4];
  const double* row = Z + size_t(min(n0 + i, N - 1)) * l;
#pragma unroll
  for (int s = 0; s < kSmallL / 4; ++s) z[s] = s < ks_n ? row[min(4 * s + kq, l - 1)] : 0.0;
  for (int rt = 0; rt < rt_n; ++rt) {
    double4_t acc = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < kSmallL / 4; ++s)
      if (s < ks_n) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sm[(16 * rt + i) * pitch + 4 * s + kq], z[s], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rr = 16 * rt + kq + 4 * r, n = n0 + i;
      if (rr < rank && n < N) B[size_t(rr) * N + n] = acc[r];
    }
  }
}

// Sum over the 16 lanes of a DPP row, in every lane (four exchanges inside the vector registers).
template <int CTRL> __device__ inline double dpp_add(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, int(uint32_t(u)), CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, int(uint32_t(u >> 32)), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}
__device__ inline double row16_sum(double v) {
  v = dpp_add<0xb1>(v);       // quad_perm 1, 0, 3, 2
  v = dpp_add<0x4e>(v);       // quad_perm 2, 3, 0, 1
  v = dpp_add<0x141>(v);      // row_half_mirror
  return dpp_add<0x140>(v);   // row_mirror
}
// One-sided Jacobi on the rows of W = L1 L2 (l x l, LDS), rotations accumulated in Gt: a round-robin
// tournament, 16 lanes per pair (all pairs of a step at once), one barrier per step, sweeps until the
// largest |<p, q>| / (|p| |q|) of a sweep is below 1e-14.  Then the rows in descending order of their
// norms sigma_i: sigma [rank], M [l][rank] = G sqrt(sigma) and Mi [rank][l] = G^T / sqrt(sigma).
// *unconverged is set after 30 sweeps.
// Bound: the serial chain of a step (LDS reads, sums over 16 lanes, the rotation's angle, LDS writes,
// barrier), l - 1 steps a sweep.  The tangent of the angle needs no more than the convergence does and
// is taken from reciprocal estimates with a Newton step; cosine and sine keep c^2 + s^2 = 1 to rounding.
// kU: ceil(l / 16), so that a pair's entries are read from LDS together.
template <int kU>
__global__ __launch_bounds__(1024) void jacobi_small_kernel(const double* __restrict__ L1, const double* __restrict__ L2, int l, int rank,
                                                            double* __restrict__ sigma, double* __restrict__ M, double* __restrict__ Mi,
                                                            const int* __restrict__ bad, int* __restrict__ unconverged) {
  extern __shared__ double sm[];
  __shared__ double norm2[kSmallL];
  __shared__ unsigned off[2];
  if (bad[0] | bad[1]) return;
  const int pitch = l + 1, lp = l + (l & 1), threads = blockDim.x;
  double* W = sm;
  double* Gt = sm + l * pitch;
  for (int e = threadIdx.x; e < l * l; e += threads) {
    const int r = e / l, c = e - r * l;
    double v = 0.0;
    for (int k = c; k <= r; ++k) v = fma(L1[size_t(r) * l + k], L2[size_t(k) * l + c], v);
    W[r * pitch + c] = v;
    Gt[r * pitch + c] = r == c ? 1.0 : 0.0;
  }
  if (threadIdx.x < 2) off[threadIdx.x] = 0;
  __syncthreads();
  const int k = threadIdx.x >> 4, e0 = threadIdx.x & 15;     // pair k of every step
  bool done = false;
  for (int sweep = 0; sweep < 30 && !done; ++sweep) {
    float worst = 0.f;
    // pair k of step st: rows (st + k) and (st - k) mod (lp - 1); pair 0: the last row and row st
    int p = k == 0 ? lp - 1 : k, q = k == 0 ? 0 : lp - 1 - k;
    for (int st = 0; st < lp - 1; ++st) {
      if (k < lp / 2 && p < l && q < l) {                    // (an odd l gets a bye)
        double* wp = W + p * pitch;
        double* wq = W + q * pitch;
        double x[kU], y[kU], gx[kU], gy[kU], al = 0.0, be = 0.0, ga = 0.0;
        double* gp = Gt + p * pitch;
        double* gq = Gt + q * pitch;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int e = e0 + 16 * u;
          const int ec = u < kU - 1 ? e : min(e, l - 1);
          x[u] = wp[ec]; y[u] = wq[ec]; gx[u] = gp[ec]; gy[u] = gq[ec];
        }
        x[kU - 1] = e0 + 16 * (kU - 1) < l ? x[kU - 1] : 0.0;
        y[kU - 1] = e0 + 16 * (kU - 1) < l ? y[kU - 1] : 0.0;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          al = fma(x[u], x[u], al); be = fma(y[u], y[u], be); ga = fma(x[u], y[u], ga);
        }
        al = row16_sum(al); be = row16_sum(be); ga = row16_sum(ga);
        if (al > 0.0 && be > 0.0) {
          const double rel = fabs(ga) * __builtin_amdgcn_rsq(al) * __builtin_amdgcn_rsq(be);   // (an estimate will do)
          worst = fmaxf(worst, float(rel));
          if (rel > 1e-16) {
            // t = 2 ga sign(be - al) / (|be - al| + sqrt((be - al)^2 + 4 ga^2)), scaled by the larger norm
            const double sc = __builtin_amdgcn_rcp(fmax(al, be)), d = (be - al) * sc, g2 = 2.0 * ga * sc;
            const double h2 = fma(d, d, g2 * g2), den = fabs(d) + h2 * __builtin_amdgcn_rsq(h2);
            double rc = __builtin_amdgcn_rcp(den);
            rc = fma(rc, fma(-den, rc, 1.0), rc);
            const double tt = (d >= 0.0 ? g2 : -g2) * rc;
            const double c = rsqrt_newton(fma(tt, tt, 1.0)), s = c * tt;
#pragma unroll
            for (int u = 0; u < kU; ++u) {
              const int e = e0 + 16 * u;
              if (u < kU - 1 || e < l) {
                wp[e] = c * x[u] - s * y[u];
                wq[e] = s * x[u] + c * y[u];
                gp[e] = c * gx[u] - s * gy[u];
                gq[e] = s * gx[u] + c * gy[u];
              }
            }
          }
        }
      }
      if (k != 0) p = p + 1 == lp - 1 ? 0 : p + 1;
      q = q + 1 == lp - 1 ? 0 : q + 1;
      __syncthreads();
    }
    // (two cells in turn: one is read while the other is cleared)
    atomicMax(&off[sweep & 1], __float_as_uint(worst));
    __syncthreads();
    done = __uint_as_float(off[sweep & 1]) < 1e-14f;
    if (threadIdx.x == 0) off[(sweep + 1) & 1] = 0;
    __syncthreads();
  }
  if (!done) {
    if (threadIdx.x == 0) *unconverged = 1;
    return;
  }
  for (int r = threadIdx.x; r < l; r += threads) {
    double v = 0.0;
    for (int c = 0; c < l; ++c) v = fma(W[r * pitch + c], W[r * pitch + c], v);
    norm2[r] = v;
  }
  __syncthreads();
  for (int r = threadIdx.x >> 4; r < l; r += threads / 16) {   // 16 lanes per row
    int at = 0;
    for (int c = 0; c < l; ++c) at += (norm2[c] > norm2[r] || (norm2[c] == norm2[r] && c < r)) ? 1 : 0;
    if (at >= rank) continue;
    const double sg = sqrt(norm2[r]), root = sqrt(sg), inv = sg > 0.0 ? 1.0 / root : 0.0;
    if (e0 == 0) sigma[at] = sg;
    for (int c = e0; c < l; c += 16) {                       // G[c][r] = Gt[r][c]
      M[size_t(c) * rank + at] = Gt[r * pitch + c] * root;
      Mi[size_t(at) * l + c] = Gt[r * pitch + c] * inv;
    }
  }
}

// [N][l] -> [l][N]
__global__ __launch_bounds__(256) void transpose_kernel(const double* __restrict__ Z, int N, int l, double* __restrict__ Bm) {
  __shared__ double tile[32][33];
  const int n0 = blockIdx.x * 32, c0 = blockIdx.y * 32, x = threadIdx.x & 31;
  for (int y = threadIdx.x >> 5; y < 32; y += 8)
    if (n0 + y < N && c0 + x < l) tile[y][x] = Z[size_t(n0 + y) * l + c0 + x];
  __syncthreads();
  for (int y = threadIdx.x >> 5; y < 32; y += 8)
    if (c0 + y < l && n0 + x < N) Bm[size_t(c0 + y) * N + n0 + x] = tile[x][y];
}

// ---------------------------------------------------------------------------------- Cholesky QR, larger l
// In-place lower Cholesky factor of the l x l matrix G (one block; right-looking): *bad is set if a
// pivot is not positive.
__global__ __launch_bounds__(1024) void cholesky_kernel(double* __restrict__ G, int l, int* __restrict__ bad) {
  __shared__ double d_sh;
  for (int j = 0; j < l; ++j) {
    if (threadIdx.x == 0) {
      const double p = G[size_t(j) * l + j];
      if (!(p > 0.0)) *bad = 1;
      d_sh = sqrt(p > 0.0 ? p : 1.0);
      G[size_t(j) * l + j] = d_sh;
    }
    __syncthreads();
    const double d = d_sh;
    for (int i = j + 1 + threadIdx.x; i < l; i += 1024) G[size_t(i) * l + j] /= d;
    __syncthreads();
    const int n = l - j - 1;
    for (long long idx = threadIdx.x; idx < (long long)n * n; idx += 1024) {
      const int i = j + 1 + int(idx / n), k = j + 1 + int(idx % n);
      if (k <= i) G[size_t(i) * l + k] -= G[size_t(i) * l + j] * G[size_t(k) * l + j];
    }
    __syncthreads();
  }
}

// Y <- Y L^-T for the lower-triangular L (l x l): one thread per row of Y (K rows), forward substitution.
__global__ __launch_bounds__(256) void trsm_kernel(double* __restrict__ Y, int K, int l, const double* __restrict__ L) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= K) return;
  double* y = Y + size_t(r) * l;
  for (int j = 0; j < l; ++j) {
    double s = y[j];
    for (int k = 0; k < j; ++k) s -= y[k] * L[size_t(j) * l + k];
    y[j] = s / L[size_t(j) * l + j];
  }
}

// ---------------------------------------------------------------------------------- one-sided Jacobi
// One step of a sweep: block b rotates rows (p, q) = pairs[2b], pairs[2b + 1] of Bm (l x N) so that
// they become orthogonal, and applies the same rotation to rows p, q of Gt (l x l).  *off receives
// the largest |<p, q>| / (|p| |q|) seen (as the bits of a non-negative float, by atomicMax).
__global__ __launch_bounds__(256) void jacobi_kernel(double* __restrict__ Bm, int N, double* __restrict__ Gt, int l,
                                                     const int* __restrict__ pairs, unsigned* __restrict__ off) {
  __shared__ double red[3][256];
  __shared__ double cs[2];
  const int p = pairs[2 * blockIdx.x], q = pairs[2 * blockIdx.x + 1];
  if (p < 0 || q < 0) return;
  double* bp = Bm + size_t(p) * N;
  double* bq = Bm + size_t(q) * N;
  double a = 0.0, b = 0.0, g = 0.0;
  for (int i = threadIdx.x; i < N; i += 256) {
    const double x = bp[i], y = bq[i];
    a = fma(x, x, a); b = fma(y, y, b); g = fma(x, y, g);
  }
  red[0][threadIdx.x] = a; red[1][threadIdx.x] = b; red[2][threadIdx.x] = g;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int m = 0; m < 3; ++m) red[m][threadIdx.x] += red[m][threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double alpha = red[0][0], beta = red[1][0], gamma = red[2][0];
    const double denom = sqrt(alpha * beta);
    const double rel = denom > 0.0 ? fabs(gamma) / denom : 0.0;
    atomicMax(off, __float_as_uint(float(rel)));
    double c = 1.0, s = 0.0;
    if (rel > 1e-16) {
      const double zeta = (beta - alpha) / (2.0 * gamma);
      const double t = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
      c = 1.0 / sqrt(1.0 + t * t);
      s = c * t;
    }
    cs[0] = c; cs[1] = s;
  }
  __syncthreads();
  const double c = cs[0], s = cs[1];
  if (s == 0.0) return;
  for (int i = threadIdx.x; i < N; i += 256) {
    const double x = bp[i], y = bq[i];
    bp[i] = c * x - s * y;
    bq[i] = s * x + c * y;
  }
  double* gp = Gt + size_t(p) * l;
  double* gq = Gt + size_t(q) * l;
  for (int i = threadIdx.x; i < l; i += 256) {
    const double x = gp[i], y = gq[i];
    gp[i] = c * x - s * y;
    gq[i] = s * x + c * y;
  }
}

__global__ __launch_bounds__(256) void row_norm2_kernel(const double* __restrict__ Bm, int N, double* __restrict__ out) {
  __shared__ double red[256];
  const double* b = Bm + size_t(blockIdx.x) * N;
  double a = 0.0;
  for (int i = threadIdx.x; i < N; i += 256) a = fma(b[i], b[i], a);
  red[threadIdx.x] = a;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// B[i][n] = Bm[sel[i]][n] * mul[i]
__global__ __launch_bounds__(256) void pick_rows_kernel(const double* __restrict__ Bm, int N, const int* __restrict__ sel,
                                                        const double* __restrict__ mul, double* __restrict__ B) {
  const int i = blockIdx.y, n = blockIdx.x * 256 + threadIdx.x;
  if (n < N) B[size_t(i) * N + n] = Bm[size_t(sel[i]) * N + n] * mul[i];
}

__global__ __launch_bounds__(256) void to_bf16_kernel(const double* __restrict__ in, size_t n, uint16_t* __restrict__ out) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  // (through fp32, as the stored factors are defined: exact for the magnitudes of a residual's factors)
  uint32_t u = __float_as_uint(float(in[i]));
  u += 0x7fffu + ((u >> 16) & 1u);
  out[i] = uint16_t(u >> 16);
}

}  // namespace
}  // namespace lrc

using namespace lrc;

#define OFF_HIP(expr)                                                                                \
  do {                                                                                               \
    hipError_t e_ = (expr);                                                                          \
    if (e_ != hipSuccess) {                                                                          \
      rc = set_error(e_ == hipErrorOutOfMemory ? MOE_LRC_ENOMEM : MOE_LRC_EHIP,                      \
                     std::string("offline: ") + #expr + ": " + hipGetErrorString(e_));               \
      goto done;                                                                                     \
    }                                                                                                \
  } while (0)

extern "C" {

int moe_lrc_offline_quantize(const double* W_dev, int K, int N, int bits, int group, uint8_t* codes_dev,
                             uint16_t* scale_dev, uint16_t* zero_dev, double* residual_dev, void* stream) {
  if (!W_dev || !codes_dev || !scale_dev || !zero_dev) return set_error(MOE_LRC_EINVAL, "offline_quantize: null argument");
  if (bits < 2 || bits > 4) return set_error(MOE_LRC_EINVAL, "offline_quantize: bits must be 2, 3 or 4");
  if (K <= 0 || N <= 0 || group <= 0 || K % group) return set_error(MOE_LRC_ESHAPE, "offline_quantize: K must be a positive multiple of group");
  // groups of 32, 64, 128 and 256 rows keep a quarter of the group in a thread's registers; pairs of
  // columns where N and the codes' address are even (the paths differ in speed only)
  const bool pairs = N % 2 == 0 && ((uintptr_t)codes_dev & 1) == 0;
  auto rows = [&](auto kernel, int cpl) {
    hipLaunchKernelGGL(kernel, dim3((N + 64 * cpl - 1) / (64 * cpl), K / group), dim3(256), 0, (hipStream_t)stream, W_dev, K, N, bits,
                       codes_dev, scale_dev, zero_dev, residual_dev);
  };
  if (group == 32) pairs ? rows(quantize_rows_kernel<8, 2>, 2) : rows(quantize_rows_kernel<8, 1>, 1);
  else if (group == 64) pairs ? rows(quantize_rows_kernel<16, 2>, 2) : rows(quantize_rows_kernel<16, 1>, 1);
  else if (group == 128) pairs ? rows(quantize_rows_kernel<32, 2>, 2) : rows(quantize_rows_kernel<32, 1>, 1);
  else if (group == 256) rows(quantize_rows_kernel<64, 1>, 1);
  else
    hipLaunchKernelGGL(quantize_kernel, dim3((N + 255) / 256, K / group), dim3(256), 0, (hipStream_t)stream, W_dev, K, N, bits, group,
                       codes_dev, scale_dev, zero_dev, residual_dev);
  LRC_HIP(hipGetLastError());
  return MOE_LRC_OK;
}

int moe_lrc_offline_quantize_refined(const double* W_dev, int K, int N, int bits, int group, int iters, double p, double beta,
                                     double kappa, uint8_t* codes_dev, uint16_t* scale_dev, uint16_t* zero_dev,
                                     double* residual_dev, void* stream) {
  if (!W_dev || !codes_dev || !scale_dev || !zero_dev) return set_error(MOE_LRC_EINVAL, "offline_quantize_refined: null argument");
  if (bits < 2 || bits > 4) return set_error(MOE_LRC_EINVAL, "offline_quantize_refined: bits must be 2, 3 or 4");
  if (iters < 0 || iters > 1000 || !(p > 0.0 && p <= 1.0) || !(beta > 0.0) || !(kappa >= 1.0))
    return set_error(MOE_LRC_EINVAL, "offline_quantize_refined: need 0 <= iters <= 1000, 0 < p <= 1, beta > 0, kappa >= 1");
  if (K <= 0 || N <= 0 || group <= 0 || K % group) return set_error(MOE_LRC_ESHAPE, "offline_quantize_refined: K must be a positive multiple of group");
  double tau = std::pow(beta, -1.0 / (2.0 - p));
  const double tau_step = std::pow(kappa, -1.0 / (2.0 - p));
  if (!(tau < HUGE_VAL)) tau = 0.0;        // (no finite start for the kernel's running threshold: every entry takes the pow())
  auto kernel = group == 32 ? quantize_refined_kernel<32> : group == 64 ? quantize_refined_kernel<64> : quantize_refined_kernel<0>;
  hipLaunchKernelGGL(kernel, dim3((N + 63) / 64, K / group), dim3(64), 0, (hipStream_t)stream, W_dev, K, N, bits, group,
                     iters, p, beta, kappa, tau, tau_step, codes_dev, scale_dev, zero_dev, residual_dev);
  LRC_HIP(hipGetLastError());
  return MOE_LRC_OK;
}

int moe_lrc_offline_kurtosis(const double* W_dev, size_t n, double* kappa) {
  if (!W_dev || !kappa || n == 0) return set_error(MOE_LRC_EINVAL, "offline_kurtosis: null argument or empty matrix");
  int rc = MOE_LRC_OK;
  const int blocks = int(std::min<size_t>(1024, (n + 256 * kMomentTile - 1) / (256 * kMomentTile)));
  Moments* d_part = nullptr;
  Moments m{0.0, 0.0, 0.0, 0.0, 0.0};
  OFF_HIP(hipMalloc((void**)&d_part, blocks * sizeof(Moments)));
  hipLaunchKernelGGL(moment_kernel, dim3(blocks), dim3(256), 0, nullptr, W_dev, n, d_part);
  hipLaunchKernelGGL(moment_join_kernel, dim3(1), dim3(256), 0, nullptr, d_part, blocks);
  OFF_HIP(hipMemcpy(&m, d_part, sizeof(Moments), hipMemcpyDeviceToHost));
  m.m2 /= m.n;                             // (the ratio of the means: m2 * m2 of the sums overflows n^2 times earlier)
  *kappa = m.m4 / m.n / (m.m2 * m.m2);
  if (*kappa < 1.0) *kappa = 1.0;          // (the least it can be: what a constant matrix leaves is rounding alone)
done:
  if (d_part) (void)hipFree(d_part);
  return rc;
}

int moe_lrc_offline_factors(const double* E_dev, int K, int N, int rank, const double* omega_dev, int l, int power_iters,
                            double* A_dev, double* B_dev, double* sigma_host, uint16_t* A_bf16_dev, uint16_t* B_bf16_dev) {
  if (!E_dev || !omega_dev || !A_dev || !B_dev) return set_error(MOE_LRC_EINVAL, "offline_factors: null argument");
  if (K <= 0 || N <= 0 || rank <= 0 || l < rank || l > K || l > N || l > 1088)
    return set_error(MOE_LRC_ESHAPE, "offline_factors: need 0 < rank <= l <= min(K, N, 1088)");
  if (power_iters < 0 || power_iters > 8) return set_error(MOE_LRC_EINVAL, "offline_factors: power_iters outside 0..8");
  int rc = MOE_LRC_OK;
  const bool small = l <= kSmallL;
  const int lp = l + (l & 1);                       // rows of the tournament (an odd l gets a bye)
  // one allocation for everything (a dozen of them, and their release, cost as much as a product)
  size_t bytes = 0;
  auto take = [&](size_t n) { const size_t at = bytes; bytes += (n + 255) & ~size_t(255); return at; };
  const size_t oY = take(size_t(K) * l * 8), oZ = take(size_t(N) * l * 8);
  const size_t oZ2 = take(factors_room(K, N, rank, l, small) * 8);
  const size_t oL1 = take(size_t(l) * l * 8), oL2 = take(size_t(l) * l * 8), oLi = take(size_t(l) * l * 8);
  const size_t oM = take(size_t(l) * rank * 8), oMi = take(size_t(l) * rank * 8);
  const size_t oGt = take(size_t(l) * l * 8), oNorm = take(size_t(l) * 8), oMul = take(size_t(rank) * 8), oSig = take(size_t(rank) * 8);
  const size_t oPairs = take(size_t(lp - 1) * lp * sizeof(int)), oSel = take(size_t(rank) * sizeof(int)), oStatus = take(4 * sizeof(int));
  uint8_t* base = nullptr;
  std::vector<int> h_pairs, order(l), h_sel(rank);
  std::vector<double> h_norm2(l), h_Gt, h_M, h_mul(rank), h_sig(rank);
  int h_status[4] = {0, 0, 0, 0};                   // sketch lost rank; Gram matrix of Bm not positive; rotations unconverged; scratch
  double *Y, *Z, *Z2, *part, *gram, *L1, *L2, *Li, *M, *Mi, *Gt, *norm2, *mul, *sig;
  int *pairs, *sel, *status;
  unsigned* off;
  size_t small_lds = 0, rmul_lds = 0;
  void (*jacobi)(const double*, const double*, int, int, double*, double*, double*, const int*, int*) = nullptr;
  // one Cholesky QR of X [rows][l] (in place, or into `to`); factor and its inverse in L, Li
  auto qr_once = [&](double* X, int rows, double* to, double* L, int* bad) {
    const int parts = dgemm<true>(l, l, rows, X, l, X, l, nullptr, gram, true);
    hipLaunchKernelGGL(cholesky_small_kernel, dim3(1), dim3(kCholThreads), small_lds, nullptr, gram, parts, l, L, Li, bad);
    if (to) hipLaunchKernelGGL(rmul_kernel<true>, dim3((rows + 63) / 64), dim3(256), rmul_lds, nullptr, X, rows, l, Li, l, to, (const int*)nullptr);
  };
  auto orth = [&](int reps) {
    for (int rep = 0; rep < reps; ++rep) {
      if (small) {
        qr_once(Y, K, Y, L1, status);
      } else {
        dgemm<true>(l, l, K, Y, l, Y, l, L1, part);
        hipLaunchKernelGGL(cholesky_kernel, dim3(1), dim3(1024), 0, nullptr, L1, l, status);
        hipLaunchKernelGGL(trsm_kernel, dim3((K + 255) / 256), dim3(256), 0, nullptr, Y, K, l, L1);
      }
    }
  };
  OFF_HIP(hipMalloc((void**)&base, bytes));
  Y = (double*)(base + oY); Z = (double*)(base + oZ); Z2 = part = (double*)(base + oZ2); gram = Z2 + size_t(N) * l;
  L1 = (double*)(base + oL1); L2 = (double*)(base + oL2); Li = (double*)(base + oLi); M = (double*)(base + oM); Mi = (double*)(base + oMi);
  Gt = (double*)(base + oGt); norm2 = (double*)(base + oNorm); mul = (double*)(base + oMul); sig = (double*)(base + oSig);
  pairs = (int*)(base + oPairs); sel = (int*)(base + oSel); status = (int*)(base + oStatus);
  off = (unsigned*)(status + 3);
  OFF_HIP(hipMemset(status, 0, 4 * sizeof(int)));
  if (small) {
    small_lds = size_t(2) * l * (l + 1) * 8;
    rmul_lds = size_t((l + 3) / 4 * 4) * ((l + 15) / 16 * 16 + 4) * 8;
    // (above 64 KB a kernel has to be allowed its LDS)
    OFF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&cholesky_small_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kSmallL * (kSmallL + 1) * 8));
    jacobi = l <= 16 ? jacobi_small_kernel<1> : l <= 32 ? jacobi_small_kernel<2> : l <= 48 ? jacobi_small_kernel<3>
             : l <= 64 ? jacobi_small_kernel<4> : l <= 80 ? jacobi_small_kernel<5> : jacobi_small_kernel<6>;
    OFF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(jacobi), hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kSmallL * (kSmallL + 1) * 8));
    for (const void* f : {reinterpret_cast<const void*>(&rmul_kernel<true>), reinterpret_cast<const void*>(&rmul_kernel<false>), reinterpret_cast<const void*>(&bt_kernel)})
      OFF_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kSmallL * (kSmallL + 4) * 8));
  }

  // ---- range finder
  dgemm<false>(K, l, N, E_dev, N, omega_dev, l, Y, part);               // Y = E Omega
  for (int it = 0; it < power_iters; ++it) {
    orth(1);
    dgemm<true>(N, l, K, E_dev, N, Y, l, Z, part);                      // Z = E^T Q
    dgemm<false>(K, l, N, E_dev, N, Z, l, Y, part);                     // Y = E Z
  }
  orth(2);
  dgemm<true>(N, l, K, E_dev, N, Y, l, Z, part);                        // Z = E^T Q = Bm^T

  if (small) {
    // ---- SVD of Bm = L1 L2 Q_b^T (Cholesky QR of Z, twice) by rotations of the rows of L1 L2
    qr_once(Z, N, Z2, L1, status + 1);
    qr_once(Z2, N, nullptr, L2, status + 1);
    hipLaunchKernelGGL(jacobi, dim3(1), dim3((lp / 2 * 16 + 63) / 64 * 64), small_lds, nullptr, L1, L2, l, rank, sig, M, Mi, status, status + 2);
    // A = Q G sqrt(sigma), B = rows of G^T Bm / sqrt(sigma) (neither is written if a step failed)
    hipLaunchKernelGGL(rmul_kernel<false>, dim3((K + 63) / 64), dim3(256), rmul_lds, nullptr, Y, K, l, M, rank, A_dev, status);
    hipLaunchKernelGGL(bt_kernel, dim3((N + 63) / 64), dim3(256), rmul_lds, nullptr, Z, N, l, Mi, rank, B_dev, status);
    OFF_HIP(hipGetLastError());
  }
  OFF_HIP(hipMemcpy(h_status, status, 3 * sizeof(int), hipMemcpyDeviceToHost));
  if (h_status[0]) { rc = set_error(MOE_LRC_ESHAPE, "offline_factors: the sketch lost rank (Gram matrix not positive definite)"); goto done; }
  if (h_status[2]) { rc = set_error(MOE_LRC_ESHAPE, "offline_factors: Jacobi sweeps did not converge"); goto done; }
  if (small && !h_status[1]) {
    OFF_HIP(hipMemcpy(h_sig.data(), sig, size_t(rank) * 8, hipMemcpyDeviceToHost));
    if (sigma_host) std::copy(h_sig.begin(), h_sig.end(), sigma_host);
  } else {
    // ---- larger l (or a Bm whose Gram matrix is not positive in fp64): SVD of Bm itself, sweeps of a
    //      round-robin tournament over its row pairs
    double* Bm = Z2;
    hipLaunchKernelGGL(transpose_kernel, dim3((N + 31) / 32, (l + 31) / 32), dim3(256), 0, nullptr, Z, N, l, Bm);
    h_pairs.assign(size_t(lp - 1) * lp, -1);
    for (int s = 0; s < lp - 1; ++s) {
      int* row = h_pairs.data() + size_t(s) * lp;
      for (int k = 0; k < lp / 2; ++k) {
        int a = k == 0 ? lp - 1 : (s + k) % (lp - 1), b = (s - k + (lp - 1)) % (lp - 1);
        if (a >= l || b >= l) { a = -1; b = -1; }
        row[2 * k] = a; row[2 * k + 1] = b;
      }
    }
    OFF_HIP(hipMemcpy(pairs, h_pairs.data(), h_pairs.size() * sizeof(int), hipMemcpyHostToDevice));
    h_Gt.assign(size_t(l) * l, 0.0);
    for (int i = 0; i < l; ++i) h_Gt[size_t(i) * l + i] = 1.0;
    OFF_HIP(hipMemcpy(Gt, h_Gt.data(), h_Gt.size() * 8, hipMemcpyHostToDevice));
    for (int sweep = 0; sweep < 30; ++sweep) {
      unsigned h_off = 0;
      OFF_HIP(hipMemset(off, 0, sizeof(unsigned)));
      for (int s = 0; s < lp - 1; ++s)
        hipLaunchKernelGGL(jacobi_kernel, dim3(lp / 2), dim3(256), 0, nullptr, Bm, N, Gt, l, pairs + size_t(s) * lp, off);
      OFF_HIP(hipMemcpy(&h_off, off, sizeof(unsigned), hipMemcpyDeviceToHost));
      float rel;
      std::memcpy(&rel, &h_off, 4);
      if (rel < 1e-14f) break;
      if (sweep == 29) { rc = set_error(MOE_LRC_ESHAPE, "offline_factors: Jacobi sweeps did not converge"); goto done; }
    }
    hipLaunchKernelGGL(row_norm2_kernel, dim3(l), dim3(256), 0, nullptr, Bm, N, norm2);
    OFF_HIP(hipMemcpy(h_norm2.data(), norm2, size_t(l) * 8, hipMemcpyDeviceToHost));
    OFF_HIP(hipMemcpy(h_Gt.data(), Gt, h_Gt.size() * 8, hipMemcpyDeviceToHost));
    // the `rank` largest singular values, in descending order; A = Q G_sel sqrt(sigma), B = rows / sqrt(sigma)
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return h_norm2[a] > h_norm2[b]; });
    h_M.assign(size_t(l) * rank, 0.0);
    for (int i = 0; i < rank; ++i) {
      const int src = order[i];
      const double sigma = std::sqrt(h_norm2[src]), root = std::sqrt(sigma);
      if (sigma_host) sigma_host[i] = sigma;
      h_sel[i] = src;
      h_mul[i] = sigma > 0.0 ? 1.0 / root : 0.0;
      for (int j = 0; j < l; ++j) h_M[size_t(j) * rank + i] = h_Gt[size_t(src) * l + j] * root;   // G[j][src] = Gt[src][j]
    }
    OFF_HIP(hipMemcpy(M, h_M.data(), h_M.size() * 8, hipMemcpyHostToDevice));
    OFF_HIP(hipMemcpy(mul, h_mul.data(), size_t(rank) * 8, hipMemcpyHostToDevice));
    OFF_HIP(hipMemcpy(sel, h_sel.data(), size_t(rank) * sizeof(int), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(pick_rows_kernel, dim3((N + 255) / 256, rank), dim3(256), 0, nullptr, Bm, N, sel, mul, B_dev);
    dgemm<false>(K, rank, l, Y, l, M, rank, A_dev, part);               // (Bm is done with)
  }
  if (A_bf16_dev) hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((size_t(K) * rank + 255) / 256)), dim3(256), 0, nullptr, A_dev, size_t(K) * rank, A_bf16_dev);
  if (B_bf16_dev) hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((size_t(rank) * N + 255) / 256)), dim3(256), 0, nullptr, B_dev, size_t(rank) * N, B_bf16_dev);
  OFF_HIP(hipGetLastError());
  OFF_HIP(hipDeviceSynchronize());
done:
  if (base) (void)hipFree(base);
  return rc;
}

int moe_lrc_offline_allocate_ranks(const double* kappa_host, int n, int r_avg, const int32_t* buckets_host, int n_buckets,
                                   int32_t* ranks_host) {
  if (!kappa_host || !buckets_host || !ranks_host) return set_error(MOE_LRC_EINVAL, "offline_allocate_ranks: null argument");
  if (n <= 0 || n_buckets <= 0 || r_avg < 0) return set_error(MOE_LRC_EINVAL, "offline_allocate_ranks: n, n_buckets must be positive, r_avg not negative");
  for (int i = 0; i < n_buckets; ++i)
    if (buckets_host[i] < 0) return set_error(MOE_LRC_EINVAL, "offline_allocate_ranks: negative bucket value");
  // in descending kurtosis order (equal values: lower index first), every matrix takes the largest
  // bucket value that keeps the running total within n * r_avg
  std::vector<int> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return kappa_host[a] > kappa_host[b]; });
  const long long budget = (long long)n * r_avg;
  long long used = 0;
  for (int i : order) {
    int best = 0;
    bool any = false;
    for (int j = 0; j < n_buckets; ++j)
      if (used + buckets_host[j] <= budget && (!any || buckets_host[j] > best)) { best = buckets_host[j]; any = true; }
    ranks_host[i] = any ? best : 0;
    used += ranks_host[i];
  }
  return MOE_LRC_OK;
}

int moe_lrc_selftest_half_rounding(const double* in_host, size_t n, uint16_t* out_host) {
  if (!in_host || !out_host) return set_error(MOE_LRC_EINVAL, "selftest_half_rounding: null argument");
  for (size_t i = 0; i < n; ++i) out_host[i] = f64_to_f16_bits(in_host[i]);
  return MOE_LRC_OK;
}

}  // extern "C"
