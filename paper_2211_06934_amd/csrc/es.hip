// Zero-order (evolution-strategies) gradient estimation on gfx950 (TorchOpt,
// Sec. 2.2 "Zero-order Differentiation"): the gradient of the Gaussian
// smoothing E_z[f(theta + s z)] is (1/s) E_z[f(theta + s z) z], estimated by
// Monte-Carlo over N noise vectors.  The noise is an input ([N][n], row-major,
// drawn by the caller), so both kernels are plain streams over it:
//   perturb:   row i = theta + s z_i (antithetic: row N + i = theta - s z_i)
//   estimate:  grad_j = scale * sum_i w_i z_ij   (weights from the caller's f)
// The estimate is a weighted reduction of N rows: a [1 x N] x [N x n] product
// with about 0.5 flop per byte, HBM-bound, so it is a stream (each lane owns one
// or several 16-byte slices of grad and walks the N rows), not a matrix-core
// contraction.
#include <cmath>

#include "adam_math.hpp"

namespace diffopt {
namespace {

constexpr int kEB = 256;   // threads per workgroup
constexpr int kRows = 8;   // noise rows per workgroup in perturb
// Perturb calls that read little take plain loads and kKeepRows rows per
// workgroup (twice the workgroups): theta is read again by every group of
// rows, and the noise often comes from the cache that its generator wrote.
// Measured on MI355X, microseconds with streaming loads and 8 rows / plain and
// 4, one set of buffers, then three in turn; antithetic, one row a sample below:
//   n = 300,001, N = 8       8.3 / 6.3, 8.9 / 7.3      6.6 / 5.1, 7.1 / 5.6
//   n = 112,261, N = 64      18.2 / 15.1, 19.4 / 16.1  12.0 / 9.2, 12.8 / 10.9
//   n = 600,001, N = 32      48.8 / 39.8, 50.1 / 40.0  31.1 / 27.8, 32.3 / 27.6
//   n = 8,300,000, N = 2     38.9 / 34.1, 39.8 / 37.7  26.2 / 24.7, 27.3 / 26.9
// The line lies at kPerturbKeepBytes for rows that stay on 16 bytes (above it
// one row a sample loses where the sets alternate: n = 8,300,000, N = 3 37.9 /
// 40.5, N = 5 60.7 / 66.1) and at kPerturbKeepOddBytes for others, whose
// neighbouring vectors share 32-byte sectors (n = 4,200,001, N = 16 186.7 /
// 170.3 and 112.7 / 103.1), unless theta alone takes much of the cache (n =
// 11,689,511, N = 2 58.9 / 60.4 and 38.2 / 40.7).  Such rows also store plainly
// up to kPerturbStoreBytes, so that the parts of a line meet in the cache (n =
// 1,200,001, N = 4 12.1 -> 11.0 us where the sets alternate, n = 600,001, N = 8
// 12.0 -> 11.3; above, N = 24 30.7 -> 37.4).
constexpr int kKeepRows = 4;
constexpr int64_t kPerturbKeepBytes = int64_t(96) << 20;
constexpr int64_t kPerturbKeepOddBytes = int64_t(320) << 20;
constexpr int64_t kPerturbKeepOddTheta = int64_t(8) << 20;  // parameters
constexpr int64_t kPerturbStoreBytes = int64_t(48) << 20;
constexpr int kUnroll = 8; // rows in flight per lane in estimate
constexpr int kMaxClasses = 8;  // phase classes of the noise rows
// Rows of the [N][n] noise start at 16-byte phases p_i = (base/16 + i nv) mod 8
// within the 128-byte lines; a wave's 64 vectors of a row then span 9 lines
// instead of 8 unless the lanes are shifted by p_i.  Rows i and i + P, with
// P = 8 / gcd(nv mod 8, 8), share a phase, so the rows are split into P
// phase classes and every workgroup takes kRows rows of one class, its lanes
// shifted by that class's phase: each wave touches whole lines of every row it
// reads.  At n = 11,689,512 (rows 32 bytes out of phase in turn) the
// unshifted layout fetched 15% more lines than it used; shifted, the kernel
// went from 1.84 to 1.64-1.71 ms.  The row stride inside a group (P, or a
// larger power of two) measured the same.
struct PerturbPlan {
  int64_t gstart[kMaxClasses + 1];  // first grid-y index of each class (gstart[P] = total)
  int32_t shift[kMaxClasses];       // lane shift of each class (vectors)
  int32_t P;                        // classes: rows i and i + P share a phase
};

// Grid: x over 4-element vectors of theta (shifted per class), y over groups
// of ROWS same-phase samples.  The dispatcher walks x fastest, so the chip
// works through one group of rows at a time (few DRAM pages open at once);
// theta is re-read per group, mostly from the Infinity Cache.  A lane issues
// all of its group's row loads first.  Rows are n elements apart, so with
// n % 4 != 0 (or pointers off 16 bytes) their vectors are only 4-byte aligned
// and the plan has one unshifted class; vector nv then holds the n % 4 last
// elements of each row, moved one by one.
template <int ROWS, bool KEEP, bool KEEP_OUT>
__global__ __launch_bounds__(kEB) void es_perturb_vec(const float* theta, const float* noise, int64_t N, int64_t n,
                                                       float sigma, int antithetic, float* out, PerturbPlan plan) {
  int r = 0;  // phase class of this group
  while (r + 1 < plan.P && (int64_t)blockIdx.y >= plan.gstart[r + 1]) ++r;
  const int64_t v = (int64_t)blockIdx.x * kEB + threadIdx.x - plan.shift[r];
  const int64_t nv = n >> 2;
  if (v < 0 || 4 * v >= n) return;
  const int64_t P = plan.P;
  const int64_t i0 = r + P * ((int64_t)ROWS * ((int64_t)blockIdx.y - plan.gstart[r]));  // first row; rows step by P
  const float* z = noise + 4 * v;
  float* o = out + 4 * v;
  if (v == nv) {
    for (int64_t i = i0; i < N && i < i0 + P * ROWS; i += P)
      for (int e = 0; e < (int)(n & 3); ++e) {
        const float x = z[i * n + e], t = theta[4 * v + e];
        o[i * n + e] = fmaf(sigma, x, t);
        if (antithetic) o[(N + i) * n + e] = fmaf(-sigma, x, t);
      }
    return;
  }
  const f32x4 t = ld4<KEEP>(theta + 4 * v);
  const auto in = [&](int64_t i) { return z + i * n; };
  const auto to = [&](int64_t i) { return o + i * n; };
  if (i0 + P * (ROWS - 1) < N) {
    f32x4 rw[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) rw[u] = ld4<KEEP>(in(i0 + P * u));
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int64_t i = i0 + P * u;
      f32x4 a, b;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[e] = fmaf(sigma, rw[u][e], t[e]);
        b[e] = fmaf(-sigma, rw[u][e], t[e]);
      }
      st4<KEEP_OUT>(to(i), a);
      if (antithetic) st4<KEEP_OUT>(to(N + i), b);
    }
  } else {
    for (int64_t i = i0; i < N; i += P) {
      const f32x4 rw = ld4<KEEP>(in(i));
      f32x4 a, b;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[e] = fmaf(sigma, rw[e], t[e]);
        b[e] = fmaf(-sigma, rw[e], t[e]);
      }
      st4<KEEP_OUT>(to(i), a);
      if (antithetic) st4<KEEP_OUT>(to(N + i), b);
    }
  }
}

// Each lane owns U 4-element slices of grad, kEB vectors apart, and
// accumulates the N rows in sample order, kUnroll rows in flight.  A
// workgroup thus covers kEB * U contiguous vectors of every row; rows
// start at varying phases of the 128-byte lines, so the lines at the ends of a
// workgroup's range are also fetched by its neighbours, and a wider range
// makes that a smaller share.  Vectors need only 4-byte alignment; the lane of
// vector nv takes the n % 4 last elements one by one.
template <int U>
__global__ __launch_bounds__(kEB) void es_estimate_vec(const float* noise, const float* __restrict__ w, int64_t N,
                                                        int64_t n, float scale, float* grad) {
  const int64_t v0 = (int64_t)blockIdx.x * (kEB * U) + threadIdx.x;
  const int64_t nv = n >> 2;
  f32x4 acc[U];
  bool on[U];
#pragma unroll
  for (int q = 0; q < U; ++q) {
    acc[q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    on[q] = v0 + (int64_t)q * kEB < nv;
    if (v0 + (int64_t)q * kEB == nv) {
      for (int64_t e = 4 * nv; e < n; ++e) {
        float t = 0.0f;
        for (int64_t i = 0; i < N; ++i) t = fmaf(w[i], noise[i * n + e], t);
        grad[e] = scale * t;
      }
    }
  }
  if (!on[0]) return;
  const auto row = [&](int64_t i, int q) {
    return noise + i * n + 4 * (v0 + (int64_t)q * kEB);
  };
  int64_t i = 0;
  for (; i + kUnroll <= N; i += kUnroll) {
    f32x4 r[kUnroll][U];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
#pragma unroll
      for (int q = 0; q < U; ++q)
        if (on[q]) r[u][q] = ld4(row(i + u, q));
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const float wi = w[i + u];
#pragma unroll
      for (int q = 0; q < U; ++q)
        if (on[q])
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[q][e] = fmaf(wi, r[u][q][e], acc[q][e]);
    }
  }
  for (; i < N; ++i) {
    const float wi = w[i];
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (on[q]) {
        const f32x4 r = ld4(row(i, q));
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[q][e] = fmaf(wi, r[e], acc[q][e]);
      }
  }
#pragma unroll
  for (int q = 0; q < U; ++q)
    if (on[q]) {
      f32x4 out;
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] = scale * acc[q][e];
      st4(grad + 4 * (v0 + (int64_t)q * kEB), out);
    }
}

// ---- estimates of few parameters: the samples split over a workgroup ---------
//
// With few parameters the one-lane-per-slice estimates leave most of the chip
// idle while each lane walks all N samples: they are bound by one serial
// chain.  Here a workgroup of kSB threads owns kSB / G slots (a slot: the E
// parameters one lane accumulates) and cuts the samples into G contiguous
// groups; each lane sums its group in sample order, and the G partial sums of
// a parameter are added through LDS in group order: first eight (or four)
// neighbouring groups, then those sums.  The order depends only on n, N and
// the entry point, so results are reproducible, and a sum of short ordered
// sums rounds no worse than one long chain.
constexpr int kSB = 1024;

// Samples [lo, hi) of group g of G.
__device__ __forceinline__ void group_range(int64_t N, int G, int g, int64_t& lo, int64_t& hi) {
  lo = N * g / G;
  hi = N * (g + 1) / G;
}

// Adds the G partial sums of each of the workgroup's SLOTS * E parameters:
// acc[e] is this lane's partial sum for parameter slot * E + e of the
// workgroup, slot = threadIdx.x % SLOTS, group = threadIdx.x / SLOTS.  Returns
// the total of parameter threadIdx.x for threads below SLOTS * E.  Every
// thread of the workgroup calls it.
template <int SLOTS, int E>
__device__ __forceinline__ float group_sum(const float (&acc)[E]) {
  constexpr int O = SLOTS * E;            // parameters of the workgroup
  constexpr int G = kSB / SLOTS;          // groups
  constexpr int PARTS = kSB / O;          // threads per parameter in the first pass
  constexpr int RUN = G / PARTS;          // groups per such thread (= E)
  static_assert(PARTS * O == kSB && RUN * PARTS == G, "whole passes");
  __shared__ float part[G * O];
  __shared__ float part2[kSB];
  const int t = threadIdx.x, slot = t % SLOTS, g = t / SLOTS;
#pragma unroll
  for (int e = 0; e < E; ++e) part[g * O + slot * E + e] = acc[e];
  __syncthreads();
  const int o = t % O, p = t / O;
  float x = part[p * RUN * O + o];
#pragma unroll
  for (int q = 1; q < RUN; ++q) x += part[(p * RUN + q) * O + o];
  if (PARTS == 1) return x;
  part2[t] = x;
  __syncthreads();
  float y = 0.0f;
  if (t < O) {
    y = part2[t];
#pragma unroll
    for (int q = 1; q < PARTS; ++q) y += part2[q * O + t];
  }
  return y;
}

// Explicit noise: a slot is a 4-element vector of the row (4-byte aligned;
// the last one may be short), SLOTS vectors per workgroup.
template <int SLOTS>
__global__ __launch_bounds__(kSB) void es_estimate_split(const float* noise, const float* __restrict__ w, int64_t N,
                                                          int64_t n, float scale, float* grad) {
  constexpr int kInFlight = 8;  // rows loaded before the first is added
  const int slot = threadIdx.x % SLOTS, g = threadIdx.x / SLOTS;
  const int64_t j = 4 * ((int64_t)blockIdx.x * SLOTS + slot);  // first parameter of the slot
  int64_t lo, hi;
  group_range(N, kSB / SLOTS, g, lo, hi);
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (j + 4 <= n) {
    const float* z = noise + j;
    int64_t i = lo;
    for (; i + kInFlight <= hi; i += kInFlight) {
      f32x4 r[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) r[u] = ld4(z + (i + u) * n);
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const float wi = w[i + u];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(wi, r[u][e], acc[e]);
      }
    }
    for (; i < hi; ++i) {
      const float wi = w[i];
      const f32x4 r = ld4(z + i * n);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(wi, r[e], acc[e]);
    }
  } else if (j < n) {
    const int left = (int)(n - j);
    for (int64_t i = lo; i < hi; ++i) {
      const float wi = w[i];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < left) acc[e] = fmaf(wi, noise[i * n + j + e], acc[e]);
    }
  }
  const float sum = group_sum<SLOTS, 4>(acc);
  const int64_t out = 4 * (int64_t)blockIdx.x * SLOTS + threadIdx.x;
  if (threadIdx.x < 4 * SLOTS && out < n) grad[out] = scale * sum;
}

// ---- Gaussian noise generated in registers -----------------------------------
//
// z_ij (sample i, parameter j) is a pure function of (seed, i, j), so the
// perturb and estimate kernels each regenerate the noise instead of reading
// an N x n array: the pass moves 4n + 8Nn bytes (antithetic) instead of
// about 4n + 20Nn.  The normals come from Philox-4x64-10 (Salmon et al.,
// SC 2011) blocks at counter (block, i, 0, 0) under key (seed, 0), through
// the Box-Muller transform.  Block 64 s + l (segment s of 512 parameters,
// slot l < 64) covers parameters 512 s + 4 l + e (words 0 and 1) and
// 512 s + 256 + 4 l + e (words 2 and 3), e < 4; even e takes its word's cosine
// normal, odd e the sine one.  A lane owns one block, so the 64 lanes of a
// wave own one segment and each of the wave's two 128-bit store
// instructions writes one contiguous 1 KiB run.

constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull;
constexpr uint64_t kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kPhiloxW1 = 0xBB67AE8584CAA73Bull;

// Full 128-bit product of a 64-bit constant and a 64-bit value from four
// 32 x 32 -> 64-bit multiply-adds, each carry folded into a multiply-add's
// addend (none of the sums can overflow 64 bits).  Forming the low and high
// halves separately (a 64-bit multiply and __umul64hi) repeats three of the
// four partial products.
template <uint64_t M>
__device__ __forceinline__ void mul128(uint64_t c, uint64_t& lo, uint64_t& hi) {
  constexpr uint64_t ml = M & 0xffffffffull, mh = M >> 32;
  const uint64_t cl = c & 0xffffffffull, ch = c >> 32;
  const uint64_t t0 = cl * ml;
  const uint64_t t1 = cl * mh + (t0 >> 32);
  const uint64_t t2 = ch * ml + (t1 & 0xffffffffull);
  hi = ch * mh + (t1 >> 32) + (t2 >> 32);
  lo = (t2 << 32) | (t0 & 0xffffffffull);
}

// Both products of a round, M0 c0 and M1 c2.  The third multiply-add takes the
// whole second one as its addend and its carry-out, as a lane mask in scalar
// registers, becomes the high word of the fourth one's addend: three moves and
// selects a product instead of five and a half moves and adds (205 instead of
// 240 VALU instructions per block and sample; the pass at n = 11,689,512, N =
// 64, perturb then estimate, 1.655 -> 1.598 ms: its generator keeps the chip at
// its power limit).  The two third
// multiply-adds and the selects share one asm statement because an SGPR
// written by a vector instruction may be read by another only two wait states
// later, which the compiler does not see to across asm statements: each mask
// is read two instructions after it is written (s_nop 0 is one wait state).
__device__ __forceinline__ void mul128_round(uint64_t c0, uint64_t c2, uint64_t& lo0, uint64_t& hi0, uint64_t& lo1,
                                             uint64_t& hi1) {
  constexpr uint32_t l0 = (uint32_t)kPhiloxM0, h0 = (uint32_t)(kPhiloxM0 >> 32);
  constexpr uint32_t l1 = (uint32_t)kPhiloxM1, h1 = (uint32_t)(kPhiloxM1 >> 32);
  const uint32_t c0l = (uint32_t)c0, c0h = (uint32_t)(c0 >> 32), c2l = (uint32_t)c2, c2h = (uint32_t)(c2 >> 32);
  const uint64_t a0 = (uint64_t)c0l * l0, a1 = (uint64_t)c2l * l1;
  const uint64_t b0 = (uint64_t)c0l * h0 + (a0 >> 32), b1 = (uint64_t)c2l * h1 + (a1 >> 32);
  uint64_t t0, t1, m0, m1;  // third sums and their carry masks
  uint32_t top0, top1;
  asm("v_mad_u64_u32 %0, %2, %6, %7, %8\n\t"
      "v_mad_u64_u32 %1, %3, %9, %10, %11\n\t"
      "s_nop 0\n\t"
      "v_cndmask_b32 %4, 0, 1, %2\n\t"
      "v_cndmask_b32 %5, 0, 1, %3"
      : "=&v"(t0), "=&v"(t1), "=&s"(m0), "=&s"(m1), "=&v"(top0), "=&v"(top1)
      : "v"(c0h), "s"(l0), "v"(b0), "v"(c2h), "s"(l1), "v"(b1));
  hi0 = (uint64_t)c0h * h0 + (((uint64_t)top0 << 32) | (t0 >> 32));
  hi1 = (uint64_t)c2h * h1 + (((uint64_t)top1 << 32) | (t1 >> 32));
  lo0 = (t0 << 32) | (a0 & 0xffffffffull);
  lo1 = (t1 << 32) | (a1 & 0xffffffffull);
}

// a ^ b ^ c on 64-bit words through the three-input bitwise instruction
// (truth table 0x96), one per 32-bit half instead of two two-input xors.
__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
  const uint32_t lo = __builtin_amdgcn_bitop3_b32((uint32_t)a, (uint32_t)b, (uint32_t)c, 0x96);
  const uint32_t hi = __builtin_amdgcn_bitop3_b32((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), 0x96);
  return ((uint64_t)hi << 32) | lo;
}

// Ten rounds of Philox-4x64: per round the two 64 x 64 -> 128-bit products
// M0 c0 and M1 c2, then c <- (hi1 ^ c1 ^ k0, lo1, hi0 ^ c3 ^ k1, lo0); the
// key advances by the Weyl increments between rounds.  The counter here is
// (block, sample, 0, 0) and the key (seed, 0).
__device__ __forceinline__ void philox_block(uint64_t block, uint64_t sample, uint64_t seed, uint64_t out[4]) {
  uint64_t c0 = block, c1 = sample, c2 = 0, c3 = 0;
  uint64_t k0 = seed, k1 = 0;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += kPhiloxW0;
      k1 += kPhiloxW1;
    }
    uint64_t lo0, hi0, lo1, hi1;
    // The first three rounds' products depend in part on the block alone or
    // on the sample and seed alone: ordinary code, which the compiler moves out
    // of the sample loop or to scalar registers.
    if (r < 3) {
      mul128<kPhiloxM0>(c0, lo0, hi0);
      mul128<kPhiloxM1>(c2, lo1, hi1);
    } else {
      mul128_round(c0, c2, lo0, hi0, lo1, hi1);
    }
    // The first two rounds are left to the compiler, which keeps their
    // sample- and seed-only terms in scalar registers.
    const uint64_t n0 = r < 2 ? hi1 ^ c1 ^ k0 : xor3(hi1, c1, k0);
    const uint64_t n2 = r < 2 ? hi0 ^ c3 ^ k1 : xor3(hi0, c3, k1);
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// Box-Muller on one 64-bit word: 24-bit uniforms u1 = (lo/2^8 + 1) 2^-24 in
// (0, 1] and u2 = (hi/2^8) 2^-24 in [0, 1), exact in fp32; r = sqrt(-2 ln u1),
// za = r cos(2 pi u2), zb = r sin(2 pi u2).  The transcendentals are the
// hardware instructions: v_log_f32 (log2, so ln u1 = ln 2 log2 u1),
// v_sqrt_f32, and v_sin_f32 / v_cos_f32, whose argument is in revolutions,
// so they take u2 itself.  Over all 2^24 values of each uniform, measured
// against fp64 on MI355X: sin and cos within 1.3e-7 absolute, r within
// 1.4e-7 relative, so each normal is within about 3.5e-7 r of its exact
// value.  The library's logf / sincospif are about three times as accurate
// and cost several times the instructions in a kernel whose time is set by
// this arithmetic.
__device__ __forceinline__ void box_muller(uint64_t w, float& za, float& zb) {
  const uint32_t lo = static_cast<uint32_t>(w), hi = static_cast<uint32_t>(w >> 32);
  const float u1 = static_cast<float>((lo >> 8) + 1u) * 0x1p-24f;
  const float u2 = static_cast<float>(hi >> 8) * 0x1p-24f;
  constexpr float kMinus2Ln2 = -1.38629436111989061f;
  const float r = __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(u1));
  za = r * __builtin_amdgcn_cosf(u2);
  zb = r * __builtin_amdgcn_sinf(u2);
}

// The eight normals of block `block` of sample `sample`: z[0..3] belong to
// the block's first four parameters, z[4..7] to its second four.
__device__ __forceinline__ void noise8(uint64_t block, uint64_t sample, uint64_t seed, float z[8]) {
  uint64_t w[4];
  philox_block(block, sample, seed, w);
#pragma unroll
  for (int q = 0; q < 4; ++q) box_muller(w[q], z[2 * q], z[2 * q + 1]);
}

// First parameter of the two runs of four that block b covers.
__device__ __forceinline__ int64_t run_start(int64_t b, int h) { return 512 * (b >> 6) + 256 * h + 4 * (b & 63); }

// Weight of sample i from the caller's evaluations f (method 0 plain: f_i;
// 1 baseline: f_i - f0; 2 antithetic: f_i - f_{N+i}).
__device__ __forceinline__ float es_weight(const float* __restrict__ f, const float* __restrict__ f0, int64_t N,
                                           int method, int64_t i) {
  if (method == 0) return f[i];
  if (method == 1) return f[i] - *f0;
  return f[i] - f[N + i];
}

// Perturb with line-aligned stores.  A workgroup's waves own as many
// consecutive segments (8 waves: 4096 parameters, 16 KiB of each output row);
// a row starts at a 16-byte phase d within its 128-byte lines
// (d = (address / 16) mod 8, n mod 32 = 8 at the ResNet-18 size).  Stored
// lane by lane, every wave's 1 KiB run would then begin and end inside a
// line, and each partially written line goes to memory in two parts from
// two waves: on MI355X the perturbation took 1.43 ms at n = 11,689,512
// against 1.09 ms at n = 11,689,984 (a multiple of 32).  Here the workgroup
// stages each sample's plus and minus rows in LDS, then stores every row
// in 64-chunk spans that start on a line, chunk c = 64 q + lane - d: only the
// two lines at the workgroup's ends are shared with a neighbour (1.18 ms).
// Measured on MI355X (n = 11,689,512, N = 64 antithetic, two rounds): 8 waves
// per workgroup 1.18 ms, 4 waves 1.20, 2 waves 1.24 (with the sample groups
// outermost in the grid; the order is now chunk-major, below).
#ifndef DIFFOPT_ES_LINE_WAVES
#define DIFFOPT_ES_LINE_WAVES 8
#endif
constexpr int kLW = DIFFOPT_ES_LINE_WAVES;  // waves (segments) per workgroup
// Samples per workgroup.  The grid is one-dimensional with the sample groups
// of one parameter chunk consecutive, so the dispatcher runs them side by side
// and they share the chunk's theta through the cache.  Measured (n =
// 11,689,512, N = 64 antithetic): 1, 2, 4, 8 samples per workgroup 1.100,
// 1.143, 1.143, 1.138 ms alone, equal when the estimate follows (the chip then
// runs at its power limit, and one sample per workgroup redoes the
// sample-independent part of the generator); the sample groups outermost 1.176.
// One row a sample (not antithetic): 0.839, 0.762, 0.718 ms for 1, 2, 4.
// Smaller calls take fewer by perturb_samples.
#ifndef DIFFOPT_ES_LINE_ROWS
#define DIFFOPT_ES_LINE_ROWS 4
#endif
constexpr int kLRows = DIFFOPT_ES_LINE_ROWS;
constexpr int kLB = 64 * kLW;
constexpr int kRowElems = kLW * 512;  // elements of one row per workgroup

// VEC: n % 4 == 0 and 16-byte aligned theta and out, so every row's phase d is
// a whole number of 16-byte chunks and LDS is read in aligned chunks.
// Otherwise rows start at any element of a line: the 16-byte chunks stored are
// still aligned in memory, each gathered from LDS at the row's element phase,
// and the chunks that reach past the workgroup's range (its two ends) are
// stored element by element.
template <bool VEC>
__global__ __launch_bounds__(kLB) void es_perturb_gauss_lines(const float* theta, int64_t N, int64_t n,
                                                               uint64_t seed, float sigma, int antithetic,
                                                               uint32_t groups, int rows_per_group, float* out) {
  __shared__ __attribute__((aligned(16))) float rows[2][kRowElems];  // the plus and minus rows of one sample
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t chunk = blockIdx.x / groups, group = blockIdx.x - chunk * groups;
  const int64_t b = (int64_t)chunk * kLB + threadIdx.x;
  const int64_t first = (int64_t)chunk * kRowElems;  // the workgroup's first parameter
  const int64_t left = n - first;
  const int elems = left < kRowElems ? (int)left : kRowElems;
  bool on[2];
  float t[8];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t j = run_start(b, h);
    on[h] = j < n;
    if (VEC || j + 4 <= n) {
      const f32x4 a = on[h] ? *reinterpret_cast<const f32x4u*>(theta + j) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int e = 0; e < 4; ++e) t[4 * h + e] = a[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) t[4 * h + e] = j + e < n ? theta[j + e] : 0.0f;
    }
  }
  const int64_t i0 = (int64_t)group * rows_per_group;
  const int64_t i1 = i0 + rows_per_group < N ? i0 + rows_per_group : N;
  const int nrows = antithetic ? 2 : 1;
  for (int64_t i = i0; i < i1; ++i) {
    if (on[0]) {  // a lane past the end computes nothing but still meets both barriers
      float z[8];
      noise8(b, i, seed, z);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 pa, pm;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          pa[e] = fmaf(sigma, z[4 * h + e], t[4 * h + e]);
          pm[e] = fmaf(-sigma, z[4 * h + e], t[4 * h + e]);
        }
        const int at = 512 * wave + 256 * h + 4 * lane;  // element run_start(b, h) of the row
        *reinterpret_cast<f32x4*>(&rows[0][at]) = pa;
        if (antithetic) *reinterpret_cast<f32x4*>(&rows[1][at]) = pm;
      }
    }
    __syncthreads();
    for (int r = 0; r < nrows; ++r) {
      float* row = out + (r ? N + i : i) * n + first;
      const int d = (int)((reinterpret_cast<uintptr_t>(row) >> 2) & 31u);  // row's phase in its line, in elements
      for (int q = wave; q <= 2 * kLW; q += kLW) {
        const int x = 4 * (64 * q + lane) - d;  // first element of this lane's chunk
        if (x >= 0 && x + 4 <= elems) {
          if (VEC) {
            st(reinterpret_cast<f32x4*>(row + x), *reinterpret_cast<const f32x4*>(&rows[r][x]));
          } else {
            const f32x4 y = {rows[r][x], rows[r][x + 1], rows[r][x + 2], rows[r][x + 3]};
            st(reinterpret_cast<f32x4*>(row + x), y);
          }
        } else if (!VEC) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (x + e >= 0 && x + e < elems) row[x + e] = rows[r][x + e];
        }
      }
    }
    __syncthreads();
  }
}

// Each lane owns the eight gradient entries of one Philox block and walks
// the N samples in order, regenerating the block's noise and accumulating
// w_i z_ij in fp32; the result is scaled once at the end.
template <bool VEC>
__global__ __launch_bounds__(kEB) void es_estimate_gauss(const float* __restrict__ f, const float* __restrict__ f0,
                                                          int64_t N, int method, int64_t n, uint64_t seed, float scale,
                                                          float* grad) {
  const int64_t b = (int64_t)blockIdx.x * kEB + threadIdx.x;
  const int64_t j[2] = {run_start(b, 0), run_start(b, 1)};
  if (j[0] >= n) return;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
  for (int64_t i = 0; i < N; ++i) {
    const float wi = es_weight(f, f0, N, method, i);
    float z[8];
    noise8(b, i, seed, z);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = fmaf(wi, z[e], acc[e]);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t left = n - j[h];
    if (left <= 0) continue;
    float* g = grad + j[h];
    if (VEC) {
      st(reinterpret_cast<f32x4*>(g),
         f32x4{scale * acc[4 * h], scale * acc[4 * h + 1], scale * acc[4 * h + 2], scale * acc[4 * h + 3]});
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < left) g[e] = scale * acc[4 * h + e];
    }
  }
}

// Few parameters: a slot is a Philox block, SLOTS blocks per workgroup, the
// samples split over the workgroup (see group_sum).  With 64 slots a wave
// holds one group, so its sample index stays in scalar registers.
template <int SLOTS>
__global__ __launch_bounds__(kSB) void es_estimate_gauss_split(const float* __restrict__ f,
                                                                const float* __restrict__ f0, int64_t N, int method,
                                                                int64_t n, uint64_t seed, float scale, float* grad) {
  const int slot = threadIdx.x % SLOTS;
  const int g = SLOTS == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / SLOTS) : threadIdx.x / SLOTS;
  const int64_t b = (int64_t)blockIdx.x * SLOTS + slot;
  int64_t lo, hi;
  group_range(N, kSB / SLOTS, g, lo, hi);
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
  if (run_start(b, 0) < n) {
    for (int64_t i = lo; i < hi; ++i) {
      const float wi = es_weight(f, f0, N, method, i);
      float z[8];
      noise8(b, i, seed, z);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = fmaf(wi, z[e], acc[e]);
    }
  }
  const float sum = group_sum<SLOTS, 8>(acc);
  const int o = threadIdx.x;
  const int64_t out = run_start((int64_t)blockIdx.x * SLOTS + o / 8, (o & 7) >> 2) + (o & 3);
  if (o < 8 * SLOTS && out < n) grad[out] = scale * sum;
}

// weights_i = scale * (method difference of the evaluations), for the
// explicit-noise estimate.
__global__ __launch_bounds__(kEB) void es_weights_kernel(const float* __restrict__ f, const float* __restrict__ f0,
                                                          int64_t N, int method, float scale, float* w) {
  const int64_t i = (int64_t)blockIdx.x * kEB + threadIdx.x;
  if (i < N) w[i] = scale * es_weight(f, f0, N, method, i);
}

// Slots per workgroup of a split estimate over `work` slots and N samples, or 0
// for the kernel that walks all samples in one lane: split while its lanes
// cannot fill the chip, and only where every group gets a sample.
// Measured on MI355X, microseconds a call back to back, plain (four slices a
// lane for explicit noise) / 64 slots / 16 slots; the smallest are bound by the
// calls (n = 1,761, N = 256: 3.5 in the kernel):
//   explicit noise (slots of 4)  n = 1,761, N = 256: 90 / 8.0 / 4.6;
//     n = 112,261, N = 64: 19.4 / 5.8 / 9.4; n = 400,001, N = 16: 6.3 / 7.5 / 22,
//     N = 64: 28.8 / 19.4 / 28, N = 256: 109 / 73 / 88; n = 1,000,003, N = 64:
//     38.8 / 44.1 / 67
//   generated noise (slots of 8)  n = 1,761, N = 64: 39 / 8.2 / 4.4;
//     n = 112,261, N = 64: 40 / 9.1 / 10.0; n = 400,001, N = 16: 12.4 / 10.3 / 25;
//     n = 2,000,003, N = 16: 29 / 34 / 111, N = 64: 110 / 101 / 120, N = 128:
//     206 / 188; n = 11,689,512, N = 32: 261 / 284, N = 64: 510 / 505
// Generated noise costs arithmetic only, so with four samples a group the
// split's finer workgroups win until they number tens of thousands.
int noise_split_slots(int64_t work, int64_t N) {
  if (N < 16 || work >= (N < 32 ? int64_t(1) << 16 : int64_t(1) << 17)) return 0;
  return work >= (int64_t(1) << 13) || N < 64 ? 64 : 16;
}

int gauss_split_slots(int64_t work, int64_t N) {
  if (N < 16 || work >= (N < 64 ? int64_t(1) << 16 : int64_t(1) << 20)) return 0;
  return work >= (int64_t(1) << 13) || N < 64 ? 64 : 16;
}

// Slices per lane of the estimate that walks all samples in one lane.  Four
// keep most of a line's users in one workgroup, which pays once every CU has
// work and the rows go out eight at a time; fewer samples leave a lane waiting
// for each row in turn, and fewer workgroups leave CUs idle.  Measured on
// MI355X, microseconds with 1 / 2 / 4 slices, three sets of buffers in turn:
//   n = 300,001    N = 5 3.6 / 6.0 / 9.3     N = 16 6.5 / 5.7 / 7.7
//   n = 600,001    N = 5 5.2 / 6.8 / 10.0    N = 16 9.4 / 10.6 / 8.8    N = 64 35.4 / 38.9 / 28.9
//   n = 1,200,001  N = 2 3.5 / 4.5 / 6.0     N = 12 12.9 / 15.4 / 19.6
//   n = 2,400,001  N = 2 6.4 / 6.0 / 7.7     N = 12 23.1 / 22.0 / 25.1
//   n = 4,200,001  N = 2 11.7 / 10.1 / 13.1  N = 5 21.2 / 18.6 / 26.1   N = 16 51.9 / 46.7 / 47.0
//   n = 8,300,000  N = 5 33.5 / 34.5 / 41.5  N = 8 48.5 / 48.8 / 48.3
//   n = 11,689,512, N = 64 540 / 510 / 500
int estimate_slices(int64_t nvec, int64_t N) {
  const int64_t wg4 = (nvec + kEB * 4 - 1) / (kEB * 4);  // workgroups with four slices
  if (N >= 16) return wg4 < 128 ? 1 : 4;
  if (wg4 < 400) return 1;
  return N < 8 || wg4 < 1500 ? 2 : 4;
}

constexpr int kMaxPerturbRows = 65535 * 8;
// Samples per workgroup of the generated-noise perturbation over `chunks`
// parameter chunks.  One while the chip holds all samples' workgroups in about
// two rounds (four of them fit a CU); beyond that a workgroup that reads theta
// once for several samples wins, the more so the fewer samples share a chunk's
// theta in the cache.  Antithetic calls of many samples write enough per sample
// that one per workgroup stays ahead until the grid is large.  Measured on
// MI355X, microseconds with 1 / 2 / 4 samples per workgroup; antithetic, one row
// a sample:
//   n = 524,000    N = 8 7.5 / 8.2 / 9.2       5.9 / 6.1 / 7.1
//                  N = 32 23.7 / 26.0 / 27.0   18.3 / 17.1 / 16.6
//   n = 600,001    N = 16 18.4 / 18.8 / 19.1   11.7 / 11.9 / 14.3
//   n = 1,000,000  N = 8 15.2 / 13.4 / 13.3    9.7 / 9.3 / 9.5
//                  N = 32 44.7 / 52.8 / 52.9   34.3 / 32.0 / 30.5
//   n = 2,000,000  N = 3 12.0 / 11.6 / 10.0    8.5 / 9.1 / 7.6 (three sets of buffers in turn)
//   n = 2,400,001  N = 3 13.7 / 14.3 / 14.9    9.5 / 11.4 / 11.3 (rows off 16 bytes: each
//                  sample's storing costs more and hides theta's second read)
//   n = 2,000,000  N = 8 28.5 / 26.2 / 26.5    19.3 / 16.9 / 15.9
//                  N = 12 37.6 / 38.6 / 40.4   26.7 / 24.9 / 23.4
//   n = 8,300,000  N = 3 43.5 / 40.1 / 37.8    28.9 / 29.2 / 24.5
//                  N = 8 109.6 / 93.8 / 103.1  74.0 / 66.0 / 61.1
int perturb_samples(int64_t chunks, int64_t N, bool antithetic, bool vec) {
  const int64_t single = chunks * N;  // workgroups of one sample each
  if (N <= 3) return single < (vec ? 1400 : 1900) ? 1 : kLRows;
  if (single < 1900) return 1;
  if (!antithetic) return single < 3600 ? 2 : kLRows;
  if (N < 12) return 2;
  return chunks * ((N + kLRows - 1) / kLRows) < 2048 ? 1 : kLRows;
}

bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool al4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

}  // namespace
}  // namespace diffopt

using namespace diffopt;

extern "C" int diffopt_es_perturb(const float* params, const float* noise, int64_t num_samples, int64_t n,
                                  double sigma, int32_t antithetic, float* out, void* stream) {
  clear_error();
  static const char* who = "diffopt_es_perturb";
  if (n < 0 || num_samples < 0) return fail(DIFFOPT_EINVAL, "%s: n and num_samples must be >= 0", who);
  if (!std::isfinite(sigma)) return fail(DIFFOPT_EINVAL, "%s: sigma must be finite", who);
  if (n == 0 || num_samples == 0) return DIFFOPT_OK;
  if (!params || !noise || !out) return fail(DIFFOPT_EINVAL, "%s: null required pointer", who);
  if (!al4(params) || !al4(noise) || !al4(out)) return fail(DIFFOPT_EINVAL, "%s: pointers must be 4-byte aligned", who);
  hipStream_t st = as_stream(stream);
  PerturbPlan plan{};
  plan.P = 1;
  const bool vec = n % 4 == 0 && al16(params) && al16(noise) && al16(out);
  if (vec) {  // whole 16-byte vectors: align the lanes to the lines
    const int64_t q = (n / 4) % 8;
    int64_t g = 8;  // gcd(q, 8)
    if (q != 0) {
      g = q;
      for (int64_t b = 8; b != 0;) {
        const int64_t t = g % b;
        g = b;
        b = t;
      }
    }
    const int64_t P = 8 / g;  // rows i and i + P share a phase
    plan.P = (int32_t)(P < num_samples ? P : num_samples);
    const int64_t base = (int64_t)((reinterpret_cast<uintptr_t>(noise) >> 4) & 7u);
    for (int r = 0; r < plan.P; ++r) plan.shift[r] = (int32_t)((base + (int64_t)r * q) & 7);  // row r's phase, in vectors
  }
  const auto groups = [&](int per) {  // rows split into groups of `per`, class by class
    int64_t gy = 0;
    for (int r = 0; r < plan.P; ++r) {
      plan.gstart[r] = gy;
      const int64_t rows = (num_samples - r + plan.P - 1) / plan.P;
      gy += (rows + per - 1) / per;
    }
    plan.gstart[plan.P] = gy;
    return gy;
  };
  bool keep = num_samples < (vec || n > kPerturbKeepOddTheta ? kPerturbKeepBytes : kPerturbKeepOddBytes) / 4 / n;
  int64_t gy = groups(keep ? kKeepRows : kRows);
  if (keep && gy > 65535) {  // more groups than the grid takes: the larger ones
    keep = false;
    gy = groups(kRows);
  }
  if (gy > 65535) return fail(DIFFOPT_EINVAL, "%s: num_samples too large (max about %d)", who, 65535 * kRows);
  const int64_t bx = ((n + 3) / 4 + 7 + kEB - 1) / kEB;  // lanes shifted by up to 7 vectors
  if (bx > 0x7fffffff) return fail(DIFFOPT_EINVAL, "%s: n too large", who);
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)bx, (unsigned)gy), dim3(kEB), 0, st, params, noise, num_samples, n,
                       (float)sigma, antithetic ? 1 : 0, out, plan);
  };
  if (!keep) go(es_perturb_vec<kRows, false, false>);
  else if (!vec && num_samples <= kPerturbStoreBytes / (antithetic ? 8 : 4) / n) go(es_perturb_vec<kKeepRows, true, true>);
  else go(es_perturb_vec<kKeepRows, true, false>);
  return launch_status(who);
}

extern "C" int diffopt_es_estimate(const float* noise, const float* weights, int64_t num_samples, int64_t n,
                                   double scale, float* grad, void* stream) {
  clear_error();
  static const char* who = "diffopt_es_estimate";
  if (n < 0 || num_samples < 0) return fail(DIFFOPT_EINVAL, "%s: n and num_samples must be >= 0", who);
  if (!std::isfinite(scale)) return fail(DIFFOPT_EINVAL, "%s: scale must be finite", who);
  if (n == 0) return DIFFOPT_OK;
  if (!grad || (num_samples > 0 && (!noise || !weights)))
    return fail(DIFFOPT_EINVAL, "%s: null required pointer", who);
  if (!al4(noise) || !al4(weights) || !al4(grad)) return fail(DIFFOPT_EINVAL, "%s: pointers must be 4-byte aligned", who);
  hipStream_t st = as_stream(stream);
  const int64_t nvec = (n + 3) / 4;
  const int slots = noise_split_slots(nvec, num_samples);
  const int slices = estimate_slices(nvec, num_samples);
  const int64_t per = slots ? slots : kEB * slices;  // vectors per workgroup
  const int64_t bx = (nvec + per - 1) / per;
  if (bx > 0x7fffffff) return fail(DIFFOPT_EINVAL, "%s: n too large", who);
  const dim3 grid((unsigned)bx);
  if (slots == 64)
    hipLaunchKernelGGL(es_estimate_split<64>, grid, dim3(kSB), 0, st, noise, weights, num_samples, n, (float)scale,
                       grad);
  else if (slots == 16)
    hipLaunchKernelGGL(es_estimate_split<16>, grid, dim3(kSB), 0, st, noise, weights, num_samples, n, (float)scale,
                       grad);
  else {
    const auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(kEB), 0, st, noise, weights, num_samples, n, (float)scale, grad);
    };
    slices == 1 ? go(es_estimate_vec<1>) : slices == 2 ? go(es_estimate_vec<2>) : go(es_estimate_vec<4>);
  }
  return launch_status(who);
}

namespace {

bool es_method_ok(int32_t method) { return method >= 0 && method <= 2; }

// 1 / (N s), or 1 / (2 N s) for antithetic sampling, formed in fp64 and
// rounded once.
float es_scale(int32_t method, int64_t num_samples, double sigma) {
  return static_cast<float>(1.0 / ((method == 2 ? 2.0 : 1.0) * static_cast<double>(num_samples) * sigma));
}

}  // namespace

extern "C" int diffopt_es_perturb_gaussian(const float* params, int64_t n, int64_t num_samples, uint64_t seed,
                                           double sigma, int32_t antithetic, float* out, void* stream) {
  clear_error();
  static const char* who = "diffopt_es_perturb_gaussian";
  if (n < 0 || num_samples < 0) return fail(DIFFOPT_EINVAL, "%s: n and num_samples must be >= 0", who);
  if (!std::isfinite(sigma)) return fail(DIFFOPT_EINVAL, "%s: sigma must be finite", who);
  if (n == 0 || num_samples == 0) return DIFFOPT_OK;
  if (!params || !out) return fail(DIFFOPT_EINVAL, "%s: null required pointer", who);
  if (!al4(params) || !al4(out)) return fail(DIFFOPT_EINVAL, "%s: pointers must be 4-byte aligned", who);
  if (num_samples > kMaxPerturbRows)
    return fail(DIFFOPT_EINVAL, "%s: num_samples too large (max %d)", who, kMaxPerturbRows);
  const int64_t blocks = 64 * ((n + 511) / 512);  // Philox blocks: 64 per 512 parameters
  if ((blocks + kEB - 1) / kEB > 0x7fffffff) return fail(DIFFOPT_EINVAL, "%s: n too large", who);
  const int64_t chunks = (blocks + kLB - 1) / kLB;
  const bool vec = n % 4 == 0 && al16(params) && al16(out);
  const int rows = perturb_samples(chunks, num_samples, antithetic != 0, vec);
  const int64_t groups = (num_samples + rows - 1) / rows;
  if (chunks * groups > 0x7fffffff) return fail(DIFFOPT_EINVAL, "%s: n x num_samples too large", who);
  hipStream_t st = as_stream(stream);
  const dim3 grid((unsigned)(chunks * groups));
  if (vec)
    hipLaunchKernelGGL(es_perturb_gauss_lines<true>, grid, dim3(kLB), 0, st, params, num_samples, n, seed,
                       (float)sigma, antithetic ? 1 : 0, (uint32_t)groups, rows, out);
  else
    hipLaunchKernelGGL(es_perturb_gauss_lines<false>, grid, dim3(kLB), 0, st, params, num_samples, n, seed,
                       (float)sigma, antithetic ? 1 : 0, (uint32_t)groups, rows, out);
  return launch_status(who);
}

extern "C" int diffopt_es_estimate_gaussian(const float* fvals, const float* f0, int64_t num_samples, int32_t method,
                                            int64_t n, uint64_t seed, double sigma, float* grad, void* stream) {
  clear_error();
  static const char* who = "diffopt_es_estimate_gaussian";
  if (n < 0 || num_samples < 0) return fail(DIFFOPT_EINVAL, "%s: n and num_samples must be >= 0", who);
  if (!es_method_ok(method)) return fail(DIFFOPT_EINVAL, "%s: method must be 0 (plain), 1 (baseline) or 2 "
                                         "(antithetic)", who);
  if (!std::isfinite(sigma) || sigma == 0.0) return fail(DIFFOPT_EINVAL, "%s: sigma must be finite and nonzero", who);
  if (n == 0) return DIFFOPT_OK;
  if (!grad || (num_samples > 0 && (!fvals || (method == 1 && !f0))))
    return fail(DIFFOPT_EINVAL, "%s: null required pointer (f0 is required by the baseline method)", who);
  if (!al4(grad) || (num_samples > 0 && !al4(fvals))) return fail(DIFFOPT_EINVAL, "%s: pointers must be 4-byte "
                                                                  "aligned", who);
  const int64_t blocks = 64 * ((n + 511) / 512);  // Philox blocks: 64 per 512 parameters
  const int64_t bx = (blocks + kEB - 1) / kEB;
  if (bx > 0x7fffffff) return fail(DIFFOPT_EINVAL, "%s: n too large", who);
  const float scale = num_samples > 0 ? es_scale(method, num_samples, sigma) : 0.0f;
  hipStream_t st = as_stream(stream);
  const int slots = gauss_split_slots(blocks, num_samples);
  if (slots) {
    const dim3 grid((unsigned)((blocks + slots - 1) / slots));
    if (slots == 64)
      hipLaunchKernelGGL(es_estimate_gauss_split<64>, grid, dim3(kSB), 0, st, fvals, f0, num_samples, (int)method, n,
                         seed, scale, grad);
    else
      hipLaunchKernelGGL(es_estimate_gauss_split<16>, grid, dim3(kSB), 0, st, fvals, f0, num_samples, (int)method, n,
                         seed, scale, grad);
    return launch_status(who);
  }
  if (n % 4 == 0 && al16(grad))
    hipLaunchKernelGGL(es_estimate_gauss<true>, dim3((unsigned)bx), dim3(kEB), 0, st, fvals, f0, num_samples,
                       (int)method, n, seed, scale, grad);
  else
    hipLaunchKernelGGL(es_estimate_gauss<false>, dim3((unsigned)bx), dim3(kEB), 0, st, fvals, f0, num_samples,
                       (int)method, n, seed, scale, grad);
  return launch_status(who);
}

extern "C" int diffopt_es_weights(const float* fvals, const float* f0, int64_t num_samples, int32_t method,
                                  double sigma, float* weights, void* stream) {
  clear_error();
  static const char* who = "diffopt_es_weights";
  if (num_samples < 0) return fail(DIFFOPT_EINVAL, "%s: num_samples must be >= 0", who);
  if (!es_method_ok(method)) return fail(DIFFOPT_EINVAL, "%s: method must be 0 (plain), 1 (baseline) or 2 "
                                         "(antithetic)", who);
  if (!std::isfinite(sigma) || sigma == 0.0) return fail(DIFFOPT_EINVAL, "%s: sigma must be finite and nonzero", who);
  if (num_samples == 0) return DIFFOPT_OK;
  if (!fvals || !weights || (method == 1 && !f0))
    return fail(DIFFOPT_EINVAL, "%s: null required pointer (f0 is required by the baseline method)", who);
  if (!al4(fvals) || !al4(weights)) return fail(DIFFOPT_EINVAL, "%s: pointers must be 4-byte aligned", who);
  const int64_t bx = (num_samples + kEB - 1) / kEB;
  if (bx > 0x7fffffff) return fail(DIFFOPT_EINVAL, "%s: num_samples too large", who);
  hipLaunchKernelGGL(es_weights_kernel, dim3((unsigned)bx), dim3(kEB), 0, as_stream(stream), fvals, f0, num_samples,
                     (int)method, es_scale(method, num_samples, sigma), weights);
  return launch_status(who);
}
