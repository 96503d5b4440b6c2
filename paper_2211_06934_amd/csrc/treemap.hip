// Leaf-direct ("tree map") differentiable Adam on gfx950: the fused step and
// its VJP applied to every leaf of parameter trees, reading and writing the
// leaves in place of flatten -> flat step -> unflatten (TorchOpt, Appendix D,
// Table 2 "Tree Map"; Sec. 2.3 for the step).  It saves the 8 bytes per element
// that each flatten or unflatten of an operand tree would move.
//
// Work decomposition: the segment table of tree.hip.  As there, the groups of a
// leaf are counted from the 128-byte line that holds the first byte of the
// leaf in one operand, the first output: group k covers the leaf's elements
// [4k - d, 4k - d + 4), d the leaf's element phase in that line, so waves store
// whole lines whatever the leaf's alignment; the table gives each leaf
// ceil(numel / 4) + 8 groups rounded up to a multiple of 8, which covers any
// phase, and the rest are empty.  Leaves start on 8-group boundaries, so no
// line of that operand is shared by two tiles (which run on different XCDs).  A
// workgroup stages its window of the table in LDS together with the leaf
// addresses of every operand tree, each lane binary-searches the window for
// its groups, issues every operand load of all of its groups, then computes
// and stores: 128-bit accesses (dword-aligned where an operand's phase differs)
// but for the elements at the ends of a leaf (see Whole).
// Trees that are views of one flat buffer (576 leaves, 3.6e6 elements, odd
// offsets) took an element path of serial 4-byte loads before: RMSProp with
// momentum, forward and VJP, 74.4 us against 38.2 now.
#include <type_traits>

#include "adam_math.hpp"
#include "optim_ops.hpp"
#include "segtable.hpp"

// Each workgroup covers one table tile (512 groups).  Measured on MI355X
// (20,000 leaves): the forward is fastest as 512 threads x 1 group (5.8 TB/s
// against 5.3 for 256 x 2), the VJP as 256 threads x 2 groups (5.7 against
// 5.55 for 512 x 1); 128 x 4 is slower for both.
#ifndef DIFFOPT_TM_FWD_BLOCK
#define DIFFOPT_TM_FWD_BLOCK 512
#endif
#ifndef DIFFOPT_TM_BWD_BLOCK
#define DIFFOPT_TM_BWD_BLOCK 256
#endif

namespace diffopt {
namespace {

constexpr int kFB = DIFFOPT_TM_FWD_BLOCK;
constexpr int kBB = DIFFOPT_TM_BWD_BLOCK;
static_assert(kTileGroups == kFB && kTileGroups % kBB == 0, "a workgroup must cover one table tile exactly");

// Device arrays of leaf addresses, one per operand tree (table order).
template <int NA>
struct LeafArrays {
  const uint64_t* a[NA];
};

// Stage the window of tile b: group offsets, element counts and one leaf
// address per operand.  Operands with a null array are skipped.  Returns the
// window length W.
template <int NA, int NT>
__device__ __forceinline__ int stage_window(const SegEntry* __restrict__ seg, const int64_t* __restrict__ tile_first,
                                            const LeafArrays<NA>& arr, int dense_orig, int64_t b, int64_t* s_goff,
                                            int64_t* s_numel, uint64_t (*s_ptr)[kWindowMax]) {
  const int64_t j0 = tile_first[b];
  const int W = (int)(tile_first[b + 1] - j0 + 1);
  for (int t = threadIdx.x; t <= W; t += NT) {
    const SegEntry e = seg[j0 + t];
    s_goff[t] = e.goff;
    if (t < W) {
      const int64_t leaf = dense_orig ? j0 + t : e.orig;
      // Every operand's address is loaded unconditionally (a null operand
      // reads the table instead and keeps 0): a load under the null test was
      // followed by its own wait.
      uint64_t v[NA];
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        const uint64_t* src = arr.a[q] ? arr.a[q] + leaf : reinterpret_cast<const uint64_t*>(seg);
        v[q] = *src;
      }
#pragma unroll
      for (int q = 0; q < NA; ++q) s_ptr[q][t] = arr.a[q] ? v[q] : 0;
      s_numel[t] = e.numel;
    }
  }
  return W;
}

__device__ __forceinline__ int find_leaf(const int64_t* s_goff, int W, int64_t gidx) {
  int lo = 0, hi = W - 1;  // s_goff[0] <= gidx by construction
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_goff[mid] <= gidx) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <typename T>
__device__ __forceinline__ gptr<T> at(uint64_t base, int64_t i) {
  return gaddr<T>(base) + i;
}

// Elements between the start of a leaf's 128-byte line and the leaf.
__device__ __forceinline__ int64_t line_phase(uint64_t leaf) { return (int64_t)((leaf >> 2) & 31u); }

// How a group's elements [e0, e0 + 4) within [0, nel) are moved.  A group whose
// four elements exist takes 128-bit accesses.  For the groups at the ends of a
// leaf there are two ways:
// - windows: four consecutive elements of the leaf there too, at the ends
//   inside the leaf, so that they hold elements of the neighbouring group as
//   well (whose lane may be overwriting them, where an output leaf is its
//   input leaf); those are computed and not stored.  A wave then makes one
//   pass whatever its lanes hold.  Leaves of fewer than four elements move
//   theirs together too, one by one (Few).
// - on their own, in a pass beside the vectors': element by element, or all
//   together (Few).
// The K-step kernels, whose passes are long, and the single steps served by
// the Infinity Cache (KEEP) take windows (K = 8, 5,000 leaves of up to 20,000
// elements: 292 us against 308 element by element; K = 10 on 576 packed leaves
// 144 against 165; one Adam step, 20,000 leaves of up to 50: 19.7 against 21.9).
// Single steps that stream from memory give the ends a pass of their own: there
// a wave whose lanes are not 16 bytes apart costs more than the extra pass
// (20,000 leaves of up to 65,536: forward 586 us with windows, 555 without).
struct Whole {
  int64_t e0;
  __device__ __forceinline__ f32x4 load(uint64_t leaf) const {
    return ld4(at<const float>(leaf, e0));
  }
  template <int N>
  __device__ __forceinline__ void store(const uint64_t (&leaf)[N], const f32x4 (&x)[N]) const {
#pragma unroll
    for (int q = 0; q < N; ++q) st4(at<float>(leaf[q], e0), x[q]);
  }
};

// One element, in every slot.
struct One {
  int64_t i;
  __device__ __forceinline__ f32x4 load(uint64_t leaf) const {
    const float x = *at<const float>(leaf, i);
    return f32x4{x, x, x, x};
  }
  template <int N>
  __device__ __forceinline__ void store(const uint64_t (&leaf)[N], const f32x4 (&x)[N]) const {
#pragma unroll
    for (int q = 0; q < N; ++q) *at<float>(leaf[q], i) = x[q][0];
  }
};

template <bool KEEP>
struct WindowOf {
  int64_t w;  // first element of the window
  int own;    // bit e: element w + e belongs to this group
  __device__ __forceinline__ WindowOf(int64_t e0, int64_t nel) {
    w = e0 < 0 ? 0 : (e0 + 4 <= nel ? e0 : nel - 4);
    const int d = (int)(e0 - w);  // -3..3
    own = d < 0 ? 15 >> -d : (15 << d) & 15;
  }
  __device__ __forceinline__ f32x4 load(uint64_t leaf) const {
    return ld4<KEEP>(at<const float>(leaf, w));
  }
  template <int N>
  __device__ __forceinline__ void store(const uint64_t (&leaf)[N], const f32x4 (&x)[N]) const {
    if (own == 15) {
#pragma unroll
      for (int q = 0; q < N; ++q) st4(at<float>(leaf[q], w), x[q]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (own >> e & 1)
#pragma unroll
          for (int q = 0; q < N; ++q) *at<float>(leaf[q], w + e) = x[q][e];
    }
  }
};

using Window = WindowOf<true>;

// A group's one to three elements; a slot without an element takes the group's
// last one, and computes and stores its value once more.
struct Few {
  int64_t first;
  int last;  // counted from the first
  __device__ __forceinline__ Few(int64_t e0, int64_t nel) {
    first = e0 < 0 ? 0 : e0;
    last = (int)((e0 + 4 < nel ? e0 + 4 : nel) - first) - 1;
  }
  __device__ __forceinline__ f32x4 load(uint64_t leaf) const {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 3; ++e) x[e] = *at<const float>(leaf, first + (e < last ? e : last));
    x[3] = x[2];
    return x;
  }
  template <int N>
  __device__ __forceinline__ void store(const uint64_t (&leaf)[N], const f32x4 (&x)[N]) const {
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
      for (int e = 0; e < 3; ++e) *at<float>(leaf[q], first + (e < last ? e : last)) = x[q][e];
  }
};

template <class V>
__device__ __forceinline__ V vector_at(int64_t e0, int64_t nel) {
  if constexpr (std::is_same_v<V, Window>) return Window(e0, nel);
  else return Whole{e0};
}

// The elements of a group that is not moved as a vector.
template <bool FEW, class Body>
__device__ __forceinline__ void other_elements(int64_t e0, int64_t nel, const Body& body) {
  if constexpr (FEW) {
    body(Few(e0, nel));
  } else {
    const int64_t end = e0 + 4 < nel ? e0 + 4 : nel;
    for (int64_t i = e0 < 0 ? 0 : e0; i < end; ++i) body(One{i});
  }
}

// Run a kernel's per-group code on the group's elements, if it has any.  With
// windows, leaves of fewer than four elements take a pass of their own beside
// the windows': all their elements together where the pass waits for memory
// (FEW), one after another where its arithmetic bounds it (recomputed VJP, K =
// 10, 50,000 leaves of up to 39 elements: 87 us against 93; the forward there
// 61 against 47).
template <bool KEEP, bool WINDOWS = KEEP, bool FEW = WINDOWS, class Body>
__device__ __forceinline__ void on_group(int64_t e0, int64_t nel, const Body& body) {
  if (e0 + 4 <= 0 || e0 >= nel) return;
  if constexpr (WINDOWS) {
    if (nel >= 4) body(WindowOf<KEEP>(e0, nel));
    else other_elements<FEW>(e0, nel, body);
  } else {
    if (e0 >= 0 && e0 + 4 <= nel) body(Whole{e0});
    else other_elements<false>(e0, nel, body);
  }
}

// One step on four elements.
__device__ __forceinline__ void fwd_group(f32x4& p, const f32x4& g, f32x4& m, f32x4& v, const AdamCoef& c) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const FwdOut o = fwd_elem(p[e], g[e], m[e], v[e], c);
    p[e] = o.p;
    m[e] = o.m;
    v[e] = o.v;
  }
}

template <bool HAS_MV>
__device__ __forceinline__ f32x4 bwd_group(const f32x4& dP, f32x4& dM, f32x4& dV, const f32x4& g, const f32x4& m,
                                           const f32x4& v, const AdamCoef& c) {
  f32x4 rg;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const BwdOut o = bwd_elem<HAS_MV>(dP[e], HAS_MV ? dM[e] : 0.0f, HAS_MV ? dV[e] : 0.0f, g[e], m[e], v[e], c);
    rg[e] = o.g;
    dM[e] = o.m;
    dV[e] = o.v;
  }
  return rg;
}

// Operands: 0 p, 1 g, 2 m, 3 v (inputs); 4 p', 5 m', 6 v' (outputs).
template <bool KEEP>
__global__ __launch_bounds__(kFB) void adam_fwd_tree_kernel(const SegEntry* __restrict__ seg,
                                                            const int64_t* __restrict__ tile_first, int64_t ngroups,
                                                            LeafArrays<7> arr, int dense_orig, AdamCoef c) {
  __shared__ int64_t s_goff[kWindowMax + 1];
  __shared__ int64_t s_numel[kWindowMax];
  __shared__ uint64_t s_ptr[7][kWindowMax];
  const int64_t b = blockIdx.x;
  const int W = stage_window<7, kFB>(seg, tile_first, arr, dense_orig, b, s_goff, s_numel, s_ptr);
  __syncthreads();
  const int64_t gidx = b * kTileGroups + threadIdx.x;
  if (gidx >= ngroups) return;
  const int t = find_leaf(s_goff, W, gidx);
  const int64_t e0 = 4 * (gidx - s_goff[t]) - line_phase(s_ptr[4][t]), nel = s_numel[t];
  const auto load = [&](const auto& a, f32x4(&x)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = a.load(s_ptr[q][t]);
  };
  const auto finish = [&](const auto& a, f32x4(&x)[4]) {
    const uint64_t out[3] = {s_ptr[4][t], s_ptr[5][t], s_ptr[6][t]};
    fwd_group(x[0], x[1], x[2], x[3], c);
    a.store(out, {x[0], x[2], x[3]});
  };
  const auto step = [&](const auto& a) {
    f32x4 x[4];
    load(a, x);
    finish(a, x);
  };
  if constexpr (KEEP) {
    on_group<KEEP>(e0, nel, step);
  } else {
    // The whole groups' loads are in flight while the lanes at the ends of
    // leaves move theirs, all of a group's at once: 600,000 leaves of up to 100
    // elements 286 -> 266 us against the ends after the vectors, one by one.
    const bool whole = e0 >= 0 && e0 + 4 <= nel;
    f32x4 x[4];
    if (whole) load(Whole{e0}, x);
    if (!whole && e0 + 4 > 0 && e0 < nel) step(Few(e0, nel));
    if (whole) finish(Whole{e0}, x);
  }
}

// Operands: 0 dP, 1 dM, 2 dV (null unless HAS_MV), 3 g, 4 m, 5 v (inputs);
// 6 dg, 7 dm, 8 dv (outputs).
template <bool HAS_MV, bool KEEP>
__global__ __launch_bounds__(kBB) void adam_bwd_tree_kernel(const SegEntry* __restrict__ seg,
                                                            const int64_t* __restrict__ tile_first, int64_t ngroups,
                                                            LeafArrays<9> arr, int dense_orig, AdamCoef c) {
  __shared__ int64_t s_goff[kWindowMax + 1];
  __shared__ int64_t s_numel[kWindowMax];
  __shared__ uint64_t s_ptr[9][kWindowMax];
  const int64_t b = blockIdx.x;
  const int W = stage_window<9, kBB>(seg, tile_first, arr, dense_orig, b, s_goff, s_numel, s_ptr);
  __syncthreads();

  constexpr int kBU = (int)(kTileGroups / kBB);  // groups per lane
  f32x4 P[kBU], Mb[kBU], Vb[kBU], G[kBU], M[kBU], V[kBU];
  using Vector = std::conditional_t<KEEP, Window, Whole>;
  int leaf[kBU], kind[kBU];  // kind 0: no element, 1: a vector, loaded here, 2: other elements, below
  int64_t e0[kBU];
#pragma unroll
  for (int u = 0; u < kBU; ++u) {
    const int64_t gidx = b * kTileGroups + (int64_t)u * kBB + threadIdx.x;
    kind[u] = 0;
    leaf[u] = 0;
    e0[u] = 0;
    if (gidx < ngroups) {
      const int t = find_leaf(s_goff, W, gidx);
      leaf[u] = t;
      e0[u] = 4 * (gidx - s_goff[t]) - line_phase(s_ptr[6][t]);
      const int64_t nel = s_numel[t];
      const bool any = e0[u] + 4 > 0 && e0[u] < nel;
      if (any && (KEEP ? nel >= 4 : e0[u] >= 0 && e0[u] + 4 <= nel)) {
        kind[u] = 1;
        const Vector a = vector_at<Vector>(e0[u], nel);
        P[u] = a.load(s_ptr[0][t]);
        if (HAS_MV) {
          Mb[u] = a.load(s_ptr[1][t]);
          Vb[u] = a.load(s_ptr[2][t]);
        }
        G[u] = a.load(s_ptr[3][t]);
        M[u] = a.load(s_ptr[4][t]);
        V[u] = a.load(s_ptr[5][t]);
      } else if (any) {
        kind[u] = 2;
      }
    }
  }
  // Ends of leaves first, while the vectors' loads are in flight (600,000 leaves
  // of up to 100 elements, streaming, 444 -> 395 us).
#pragma unroll
  for (int u = 0; u < kBU; ++u) {
    const int t = leaf[u];
    if (kind[u] == 2) {
      other_elements<KEEP>(e0[u], s_numel[t], [&](const auto& a) {
        const f32x4 p = a.load(s_ptr[0][t]);
        f32x4 dm = {0.0f, 0.0f, 0.0f, 0.0f}, dv = dm;
        if (HAS_MV) {
          dm = a.load(s_ptr[1][t]);
          dv = a.load(s_ptr[2][t]);
        }
        const f32x4 g = a.load(s_ptr[3][t]), m = a.load(s_ptr[4][t]), v = a.load(s_ptr[5][t]);
        const uint64_t out[3] = {s_ptr[6][t], s_ptr[7][t], s_ptr[8][t]};
        const f32x4 rg = bwd_group<HAS_MV>(p, dm, dv, g, m, v, c);
        a.store(out, {rg, dm, dv});
      });
    }
  }
#pragma unroll
  for (int u = 0; u < kBU; ++u) {
    const int t = leaf[u];
    if (kind[u] == 1) {
      const Vector a = vector_at<Vector>(e0[u], s_numel[t]);
      const uint64_t out[3] = {s_ptr[6][t], s_ptr[7][t], s_ptr[8][t]};
      const f32x4 rg = bwd_group<HAS_MV>(P[u], Mb[u], Vb[u], G[u], M[u], V[u], c);
      a.store(out, {rg, Mb[u], Vb[u]});
    }
  }
}

// ---- fused K-step leaf-direct kernels ----------------------------------------------
// The K-step driver, several steps a launch (kTK, kTLongK), as the flat driver
// does it: each lane finds its group once, then walks the steps with the running params
// (forward) or dM, dV (backward) in registers, loading the next step's inputs
// before the current step's arithmetic.  The window stages the leaf address
// of every operand tree of every step in dynamic LDS (NA x kWindowMax x 8
// bytes: 18.5 KiB for the backward at 8 steps, 27.5 for the forward at 16).  One
// group per lane, one
// table tile (512 groups) per workgroup.
constexpr int kTK = 8;  // steps per fused launch, VJP and small trees
// Steps per launch of the tiled forward: a boundary between launches sends
// the running params and moments through memory, 24 bytes per element (32 if
// the state there is not stored): 62 leaves, 1.2e7 elements, K = 10 (state 5
// stored) 96 -> 72 bytes per element, its forward 192 -> 143 us.
constexpr int kTLongK = 16;
constexpr int kUTB = (int)kTileGroups;
constexpr int kTBwdNA = 3 + 4 * kTK;  // 0 dP, 1 dmu, 2 dnu; per step s: 3+4s g, 4+4s mu, 5+4s nu, 6+4s dg

// Operands 0 p, 1 mu0, 2 nu0, 3 pK; per step s: 4+3s g, 5+3s mu_s+1, 6+3s nu_s+1.
template <int CAP>
struct TFwdArgsOf {
  const uint64_t* a[4 + 3 * CAP];
  AdamCoef c[CAP];
  int32_t K;
};
using TFwdArgs = TFwdArgsOf<kTK>;

// Execution order is reverse step order, as in the flat fused backward.
struct TBwdArgs {
  const uint64_t* a[kTBwdNA];
  AdamCoef c[kTK];
  int32_t K;
  int32_t init_mv;  // 0: dM = dV = 0 before the first step
};

// Stage the window of tile b for `na` operand trees: (operand, leaf) pairs
// are spread over the workgroup.  A NULL operand (a trajectory state the
// caller does not store) stages address 0 and is never dereferenced.  Ends
// with the workgroup synchronised.
template <int NT = kUTB>
__device__ __forceinline__ int stage_window_n(const SegEntry* __restrict__ seg, const int64_t* __restrict__ tile_first,
                                              const uint64_t* const* arrs, int na, int dense_orig, int64_t b,
                                              int64_t* s_goff, int64_t* s_numel, uint64_t* s_ptr) {
  const int64_t j0 = tile_first[b];
  const int W = (int)(tile_first[b + 1] - j0 + 1);
  for (int t = threadIdx.x; t <= W; t += NT) {
    const SegEntry e = seg[j0 + t];
    s_goff[t] = e.goff;
    if (t < W) s_numel[t] = e.numel;
  }
  for (int x = threadIdx.x; x < W * na; x += NT) {
    const int q = x / W, t = x - q * W;
    const int64_t leaf = dense_orig ? j0 + t : seg[j0 + t].orig;
    s_ptr[q * kWindowMax + t] = arrs[q] ? arrs[q][leaf] : 0;  // NULL operand: an unstored state
  }
  __syncthreads();
  return W;
}

template <bool KEEP, int CAP>
__global__ __launch_bounds__(kUTB) void adam_unrolled_fwd_tree_kernel(const SegEntry* __restrict__ seg,
                                                                     const int64_t* __restrict__ tile_first,
                                                                     int64_t ngroups, int dense_orig,
                                                                     TFwdArgsOf<CAP> a) {
  __shared__ int64_t s_goff[kWindowMax + 1];
  __shared__ int64_t s_numel[kWindowMax];
  extern __shared__ uint64_t s_ptr[];  // [na][kWindowMax]
  const int na = 4 + 3 * a.K;
  const int64_t b = blockIdx.x;
  const int W = stage_window_n(seg, tile_first, a.a, na, dense_orig, b, s_goff, s_numel, s_ptr);
  const int64_t gidx = b * kTileGroups + threadIdx.x;
  if (gidx >= ngroups) return;
  const int t = find_leaf(s_goff, W, gidx);
  const uint64_t* P = s_ptr + t;  // P[q * kWindowMax]: leaf address in operand q
#define OP(q) P[(q) * kWindowMax]
  on_group<KEEP, true>(4 * (gidx - s_goff[t]) - line_phase(OP(3)), s_numel[t], [&](const auto& x) {
    f32x4 p = x.load(OP(0)), m = x.load(OP(1)), v = x.load(OP(2));
    f32x4 g = x.load(OP(4));
    for (int s = 0; s < a.K; ++s) {
      f32x4 gn = g;
      if (s + 1 < a.K) gn = x.load(OP(4 + 3 * (s + 1)));
      fwd_group(p, g, m, v, a.c[s]);
      if (a.a[5 + 3 * s]) {  // uniform: a stored state
        x.template store<2>({OP(5 + 3 * s), OP(6 + 3 * s)}, {m, v});
      }
      g = gn;
    }
    x.template store<1>({OP(3)}, {p});
  });
#undef OP
}

template <bool KEEP>
__global__ __launch_bounds__(kUTB) void adam_unrolled_bwd_tree_kernel(const SegEntry* __restrict__ seg,
                                                                     const int64_t* __restrict__ tile_first,
                                                                     int64_t ngroups, int dense_orig, TBwdArgs a) {
  __shared__ int64_t s_goff[kWindowMax + 1];
  __shared__ int64_t s_numel[kWindowMax];
  extern __shared__ uint64_t s_ptr[];  // [na][kWindowMax]
  const int na = 3 + 4 * a.K;
  const int64_t b = blockIdx.x;
  const int W = stage_window_n(seg, tile_first, a.a, na, dense_orig, b, s_goff, s_numel, s_ptr);
  const int64_t gidx = b * kTileGroups + threadIdx.x;
  if (gidx >= ngroups) return;
  const int t = find_leaf(s_goff, W, gidx);
  const uint64_t* P = s_ptr + t;
#define OP(q) P[(q) * kWindowMax]
  on_group<KEEP, true>(4 * (gidx - s_goff[t]) - line_phase(OP(1)), s_numel[t], [&](const auto& x) {
    const f32x4 dP = x.load(OP(0));
    f32x4 dM = {0.0f, 0.0f, 0.0f, 0.0f}, dV = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 g = x.load(OP(3)), m = x.load(OP(4)), v = x.load(OP(5));
    if (a.init_mv) {
      dM = x.load(OP(1));
      dV = x.load(OP(2));
    }
    for (int s = 0; s < a.K; ++s) {
      f32x4 gn = g, mn = m, vn = v;
      if (s + 1 < a.K) {
        gn = x.load(OP(3 + 4 * (s + 1)));
        mn = x.load(OP(4 + 4 * (s + 1)));
        vn = x.load(OP(5 + 4 * (s + 1)));
      }
      const f32x4 rg = s == 0 && !a.init_mv ? bwd_group<false>(dP, dM, dV, g, m, v, a.c[s])
                                            : bwd_group<true>(dP, dM, dV, g, m, v, a.c[s]);
      x.template store<1>({OP(6 + 4 * s)}, {rg});
      g = gn;
      m = mn;
      v = vn;
    }
    x.template store<2>({OP(1), OP(2)}, {dM, dV});
  });
#undef OP
}

// ---- fused VJP over a run of steps whose moments were not stored ----------------
// Leaf-direct form of the flat driver's recomputing VJP: for a run of C steps
// j+1..j+C with only (mu_j, nu_j) stored, each lane reads that state and the
// C gradients of its group once, recomputes the run's moments in registers
// with the forward's recurrences, then walks the C VJP steps last first.
constexpr int kTRS = kRematSpan;
constexpr int kTRBwdNA = 5 + 2 * kTRS;  // 0 dP, 1 dmu, 2 dnu, 3 mu_j, 4 nu_j; per step s: 5+2s g, 6+2s dg

// Step s of a run is unrolled step j+1+s (ascending).
struct TRBwdArgs {
  const uint64_t* a[kTRBwdNA];
  AdamCoef c[kTRS];
  int32_t init_mv;  // 0: the run holds the last unrolled step (zero dM, dV before it)
};

// Workgroups per table tile: each stages the tile's whole window and takes
// its share of the tile's groups, one per lane.  With its register count
// (78 VGPRs at C = 3) a CU holds two 512-thread workgroups but five of 256
// threads; measured on MI355X (K = 3, 20,000 leaves) the split of 2 runs at
// 5.46 TB/s against 5.27 unsplit (4: 5.50, within noise).
#ifndef DIFFOPT_TRBWD_SPLIT
#define DIFFOPT_TRBWD_SPLIT 2
#endif
constexpr int kTRSplit = DIFFOPT_TRBWD_SPLIT;
constexpr int kTRB = kUTB / kTRSplit;
static_assert(kUTB % kTRSplit == 0, "the split must divide the tile");

template <int C, bool KEEP>
__global__ __launch_bounds__(kTRB) void adam_unrolled_bwd_tree_remat_kernel(const SegEntry* __restrict__ seg,
                                                                           const int64_t* __restrict__ tile_first,
                                                                           int64_t ngroups, int dense_orig,
                                                                           TRBwdArgs a) {
  __shared__ int64_t s_goff[kWindowMax + 1];
  __shared__ int64_t s_numel[kWindowMax];
  extern __shared__ uint64_t s_ptr[];  // [na][kWindowMax]
  constexpr int na = 5 + 2 * C;
  const int64_t b = blockIdx.x / kTRSplit;  // table tile
  const int W = stage_window_n<kTRB>(seg, tile_first, a.a, na, dense_orig, b, s_goff, s_numel, s_ptr);
  const int64_t gidx = b * kTileGroups + (int64_t)(blockIdx.x % kTRSplit) * kTRB + threadIdx.x;
  if (gidx >= ngroups) return;
  const int t = find_leaf(s_goff, W, gidx);
  const uint64_t* P = s_ptr + t;
#define OP(q) P[(q) * kWindowMax]
  on_group<KEEP, true, false>(4 * (gidx - s_goff[t]) - line_phase(OP(1)), s_numel[t], [&](const auto& x) {
    const f32x4 dP = x.load(OP(0));
    f32x4 M[C], V[C], G[C];  // M[s], V[s]: the moments step s consumed
    M[0] = x.load(OP(3));
    V[0] = x.load(OP(4));
#pragma unroll
    for (int s = 0; s < C; ++s) G[s] = x.load(OP(5 + 2 * s));
    f32x4 dM = {0.0f, 0.0f, 0.0f, 0.0f}, dV = {0.0f, 0.0f, 0.0f, 0.0f};
    if (a.init_mv) {
      dM = x.load(OP(1));
      dV = x.load(OP(2));
    }
#pragma unroll
    for (int s = 0; s + 1 < C; ++s) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        M[s + 1][e] = moment1(G[s][e], M[s][e], a.c[s]);
        V[s + 1][e] = moment2(G[s][e], V[s][e], a.c[s]);
      }
    }
#pragma unroll
    for (int s = C - 1; s >= 0; --s) {
      const f32x4 rg = s == C - 1 && !a.init_mv ? bwd_group<false>(dP, dM, dV, G[s], M[s], V[s], a.c[s])
                                                : bwd_group<true>(dP, dM, dV, G[s], M[s], V[s], a.c[s]);
      x.template store<1>({OP(6 + 2 * s)}, {rg});
    }
    x.template store<2>({OP(1), OP(2)}, {dM, dV});
  });
#undef OP
}

// Two such runs in one launch, the later steps first: the running dM, dV stay
// in registers between them, which saves their round trip and a second read
// of dP (20 bytes per element; 62 leaves, 1.2e7 elements, K = 10 in two runs of
// five: 128 -> 108 bytes, its
// VJP 263 -> 231 us).  C is the longer run's length; run r has
// len[r] <= C steps, and its operands start at 3 + r (2 + 2C): 0 mu_j, 1 nu_j;
// per step s: 2+2s g, 3+2s dg.
template <int C>
struct TRBwd2Args {
  const uint64_t* a[3 + 2 * (2 + 2 * C)];  // 0 dP, 1 dmu, 2 dnu
  AdamCoef c[2][C];
  int32_t len[2];
  int32_t init_mv;
};

template <int C>
__global__ __launch_bounds__(kTRB) void adam_unrolled_bwd_tree_remat2_kernel(const SegEntry* __restrict__ seg,
                                                                            const int64_t* __restrict__ tile_first,
                                                                            int64_t ngroups, int dense_orig,
                                                                            TRBwd2Args<C> a) {
  __shared__ int64_t s_goff[kWindowMax + 1];
  __shared__ int64_t s_numel[kWindowMax];
  extern __shared__ uint64_t s_ptr[];  // [na][kWindowMax]
  constexpr int na = 3 + 2 * (2 + 2 * C);
  const int64_t b = blockIdx.x / kTRSplit;  // table tile
  const int W = stage_window_n<kTRB>(seg, tile_first, a.a, na, dense_orig, b, s_goff, s_numel, s_ptr);
  const int64_t gidx = b * kTileGroups + (int64_t)(blockIdx.x % kTRSplit) * kTRB + threadIdx.x;
  if (gidx >= ngroups) return;
  const int t = find_leaf(s_goff, W, gidx);
  const uint64_t* P = s_ptr + t;
#define OP(q) P[(q) * kWindowMax]
  on_group<false, true, false>(4 * (gidx - s_goff[t]) - line_phase(OP(1)), s_numel[t], [&](const auto& x) {
    const f32x4 dP = x.load(OP(0));
    f32x4 dM = {0.0f, 0.0f, 0.0f, 0.0f}, dV = {0.0f, 0.0f, 0.0f, 0.0f};
    if (a.init_mv) {
      dM = x.load(OP(1));
      dV = x.load(OP(2));
    }
#pragma unroll 1
    for (int r = 0; r < 2; ++r) {
      const int len = a.len[r], o = 3 + r * (2 + 2 * C);
      f32x4 M[C], V[C], G[C];  // M[s], V[s]: the moments step s consumed
      M[0] = x.load(OP(o));
      V[0] = x.load(OP(o + 1));
#pragma unroll
      for (int s = 0; s < C; ++s)
        if (s < len) G[s] = x.load(OP(o + 2 + 2 * s));
#pragma unroll
      for (int s = 0; s + 1 < C; ++s) {
        if (s + 1 < len) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            M[s + 1][e] = moment1(G[s][e], M[s][e], a.c[r][s]);
            V[s + 1][e] = moment2(G[s][e], V[s][e], a.c[r][s]);
          }
        }
      }
#pragma unroll
      for (int s = C - 1; s >= 0; --s) {
        if (s < len) {
          const bool last = r == 0 && s == len - 1 && !a.init_mv;  // the last unrolled step
          const f32x4 rg = last ? bwd_group<false>(dP, dM, dV, G[s], M[s], V[s], a.c[r][s])
                                : bwd_group<true>(dP, dM, dV, G[s], M[s], V[s], a.c[r][s]);
          x.template store<1>({OP(o + 3 + 2 * s)}, {rg});
        }
      }
    }
    x.template store<2>({OP(1), OP(2)}, {dM, dV});
  });
#undef OP
}

// Fills and launches the two-run VJP: run r covers unrolled steps
// start[r] + 1 .. start[r] + len[r], start[0] = start[1] + len[1].
struct TwoRuns {
  const char* who;
  const diffopt_segtable* t;
  hipStream_t st;
  const uint64_t *dpK, *dmu0, *dnu0;
  const uint64_t* const* grads;
  const uint64_t* const* mu_traj;
  const uint64_t* const* nu_traj;
  const uint64_t* const* dgrads;
  int64_t count0;
  double lr, b1, b2, eps, eps_root;
  int64_t start[2];
  int len[2];
  int32_t init_mv;

  template <int C>
  void launch() const {
    TRBwd2Args<C> a{};
    a.a[0] = dpK;
    a.a[1] = dmu0;
    a.a[2] = dnu0;
    a.init_mv = init_mv;
    for (int r = 0; r < 2; ++r) {
      const uint64_t** op = a.a + 3 + r * (2 + 2 * C);
      a.len[r] = len[r];
      op[0] = mu_traj[start[r]];
      op[1] = nu_traj[start[r]];
      for (int s = 0; s < len[r]; ++s) {
        op[2 + 2 * s] = grads[start[r] + s];
        op[3 + 2 * s] = dgrads[start[r] + s];
        make_coef(who, count0 + start[r] + s, lr, b1, b2, eps, eps_root, &a.c[r][s]);
      }
    }
    const size_t lds = sizeof(uint64_t) * kWindowMax * (3 + 2 * (2 + 2 * C));
    hipLaunchKernelGGL(adam_unrolled_bwd_tree_remat2_kernel<C>, dim3((unsigned)(t->ntiles * kTRSplit)), dim3(kTRB),
                       lds, st, t->d_seg, t->d_tile_first, t->ngroups, t->dense_orig, a);
  }

  void run() const {  // a recomputed run has at least 2 steps
    switch (len[0] > len[1] ? len[0] : len[1]) {
      case 2: launch<2>(); break;
      case 3: launch<3>(); break;
      case 4: launch<4>(); break;
      case 5: launch<5>(); break;
      default: launch<6>(); break;
    }
  }
};
// Longer runs keep a launch of their own: with 7 or 8 steps the compiler puts
// the two-run kernel's arguments into scratch memory.  So do runs whose launches
// fit the Infinity Cache, where the round trip costs little and the second
// run's loads wait for the first (20,000 leaves of up to 50, K = 10: 83.8 us
// with two launches, 87.7 with one).
constexpr int64_t kTwoRunSteps = 6;

template <int C>
void launch_trbwd(const diffopt_segtable* t, const TRBwdArgs& a, hipStream_t st) {
  const size_t lds = sizeof(uint64_t) * kWindowMax * (5 + 2 * C);
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(t->ntiles * kTRSplit)), dim3(kTRB), lds, st, t->d_seg, t->d_tile_first,
                       t->ngroups, t->dense_orig, a);
  };
  if (keep_run_in_cache((20 + 8 * C + (a.init_mv ? 8 : 0)) * t->elems)) go(adam_unrolled_bwd_tree_remat_kernel<C, true>);
  else go(adam_unrolled_bwd_tree_remat_kernel<C, false>);
}

// Run length C is a template argument so the trajectory stays in registers.
int launch_trbwd_c(const char* who, int C, const diffopt_segtable* t, const TRBwdArgs& a, hipStream_t st) {
  switch (C) {
    case 1: launch_trbwd<1>(t, a, st); break;
    case 2: launch_trbwd<2>(t, a, st); break;
    case 3: launch_trbwd<3>(t, a, st); break;
    case 4: launch_trbwd<4>(t, a, st); break;
    case 5: launch_trbwd<5>(t, a, st); break;
    case 6: launch_trbwd<6>(t, a, st); break;
    case 7: launch_trbwd<7>(t, a, st); break;
    case 8: launch_trbwd<8>(t, a, st); break;
    default: return fail(DIFFOPT_EINVAL, "%s: recompute run of %d steps (at most %d)", who, C, kTRS);
  }
  return DIFFOPT_OK;
}
static_assert(kTRS == 8, "launch_trbwd_c instantiates run lengths 1..8");

// ---- small trees ------------------------------------------------------------------
// When the leaves fit a TinyTable the fused steps run one element per lane
// with the table in kernel arguments (no staged window, no barrier): a lane
// finds its leaf by a scan over the table, loads its leaf's address in every
// operand, then every input of every step, and only then computes.  The
// arithmetic per element is that of the kernels above, so the results are
// the same bit for bit.  Measured on MI355X for the 1,761-parameter tree at
// K = 5: about 7.4 and 8.2 us per fused forward and VJP launch through the
// staged window (each step a serial load and a four-element arithmetic chain
// per lane), which this form shortens to the latency of two dependent loads
// and one element's chain.
constexpr int kTinyB = 256;

// Leaf addresses as global-space pointers (see gptr): every load below is then
// a global_* instruction, counted by the vector-memory counter alone.
__device__ __forceinline__ gptr<const float> leaf_in(const uint64_t* arr, int orig) {
  return gaddr<const float>(arr[orig]);
}
__device__ __forceinline__ gptr<float> leaf_out(const uint64_t* arr, int orig) {
  return gaddr<float>(arr[orig]);
}

// The fused forward over K <= kTK steps (operands as in TFwdArgs, a.K == K).
// Every address and every input is loaded before the first step; an unstored
// step state takes the address of pK for its (unused) load slot, so no load
// waits behind a branch.
template <int K>
__global__ __launch_bounds__(kTinyB) void adam_unrolled_fwd_tree_tiny(TinyTable tt, TFwdArgs a) {
  warm_args(fold_lines(tt) ^ fold_lines(a));
  int leaf;
  int64_t i;
  if (!tiny_slot(tt, (int64_t)blockIdx.x * kTinyB + threadIdx.x, leaf, i)) return;
  const auto P0 = leaf_in(a.a[0], leaf);
  const auto M0 = leaf_in(a.a[1], leaf);
  const auto V0 = leaf_in(a.a[2], leaf);
  const auto PK = leaf_out(a.a[3], leaf);
  gptr<const float> Gp[K];
  gptr<float> Mo[K], Vo[K];
#pragma unroll
  for (int s = 0; s < K; ++s) {
    Gp[s] = leaf_in(a.a[4 + 3 * s], leaf);
    const bool kept = a.a[5 + 3 * s] != nullptr;  // uniform: a stored state
    Mo[s] = leaf_out(kept ? a.a[5 + 3 * s] : a.a[3], leaf);
    Vo[s] = leaf_out(kept ? a.a[6 + 3 * s] : a.a[3], leaf);
  }
  float p = P0[i], m = M0[i], v = V0[i];
  float G[K];
#pragma unroll
  for (int s = 0; s < K; ++s) G[s] = Gp[s][i];
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const FwdOut o = fwd_elem(p, G[s], m, v, a.c[s]);
    p = o.p;
    m = o.m;
    v = o.v;
    if (a.a[5 + 3 * s]) {
      Mo[s][i] = m;
      Vo[s][i] = v;
    }
  }
  PK[i] = p;
}

// The VJP over a run of C steps from one stored state (mu_j, nu_j), last step
// first, as adam_unrolled_bwd_tree_remat_kernel; the incoming and outgoing
// moment cotangents have their own operands so that the single-step VJP (C =
// 1, separate input and output trees) takes the same kernel.
constexpr int kTinyBwdNA = 7 + 2 * kTRS;  // 0 dP, 1 dM in, 2 dV in, 3 dM out, 4 dV out, 5 mu_j, 6 nu_j;
                                          // per step s: 7+2s g, 8+2s dg
struct TinyBwdArgs {
  const uint64_t* a[kTinyBwdNA];
  AdamCoef c[kTRS];
  int32_t init_mv;  // 0: zero dM, dV before the run's last step (operands 1, 2 unused)
};

template <int C>
__global__ __launch_bounds__(kTinyB) void adam_unrolled_bwd_tree_tiny(TinyTable tt, TinyBwdArgs a) {
  warm_args(fold_lines(tt) ^ fold_lines(a));
  int leaf;
  int64_t i;
  if (!tiny_slot(tt, (int64_t)blockIdx.x * kTinyB + threadIdx.x, leaf, i)) return;
  // without incoming moment cotangents their load slots read dP (unused)
  const auto DP = leaf_in(a.a[0], leaf);
  const auto DMi = leaf_in(a.init_mv ? a.a[1] : a.a[0], leaf);
  const auto DVi = leaf_in(a.init_mv ? a.a[2] : a.a[0], leaf);
  const auto DMo = leaf_out(a.a[3], leaf);
  const auto DVo = leaf_out(a.a[4], leaf);
  const auto Mj = leaf_in(a.a[5], leaf);
  const auto Vj = leaf_in(a.a[6], leaf);
  gptr<const float> Gp[C];
  gptr<float> DG[C];
#pragma unroll
  for (int s = 0; s < C; ++s) {
    Gp[s] = leaf_in(a.a[7 + 2 * s], leaf);
    DG[s] = leaf_out(a.a[8 + 2 * s], leaf);
  }
  const float dP = DP[i];
  const float dMi = DMi[i], dVi = DVi[i];
  float G[C], M[C], V[C];
  M[0] = Mj[i];
  V[0] = Vj[i];
#pragma unroll
  for (int s = 0; s < C; ++s) G[s] = Gp[s][i];
  float dM = a.init_mv ? dMi : 0.0f, dV = a.init_mv ? dVi : 0.0f;
#pragma unroll
  for (int s = 0; s + 1 < C; ++s) {
    M[s + 1] = moment1(G[s], M[s], a.c[s]);
    V[s + 1] = moment2(G[s], V[s], a.c[s]);
  }
#pragma unroll
  for (int s = C - 1; s >= 0; --s) {
    const BwdOut o = (s == C - 1 && !a.init_mv) ? bwd_elem<false>(dP, 0.0f, 0.0f, G[s], M[s], V[s], a.c[s])
                                                : bwd_elem<true>(dP, dM, dV, G[s], M[s], V[s], a.c[s]);
    DG[s][i] = o.g;
    dM = o.m;
    dV = o.v;
  }
  DMo[i] = dM;
  DVo[i] = dV;
}

unsigned tiny_blocks(const diffopt_segtable* t) { return (unsigned)((t->small.total + kTinyB - 1) / kTinyB); }

template <int K>
void launch_tiny_fwd(const diffopt_segtable* t, const TFwdArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((adam_unrolled_fwd_tree_tiny<K>), dim3(tiny_blocks(t)), dim3(kTinyB), 0, st, t->small, a);
}

void launch_tiny_fwd_k(const diffopt_segtable* t, const TFwdArgs& a, hipStream_t st) {
  switch (a.K) {  // 1 <= a.K <= kTK
    case 1: launch_tiny_fwd<1>(t, a, st); break;
    case 2: launch_tiny_fwd<2>(t, a, st); break;
    case 3: launch_tiny_fwd<3>(t, a, st); break;
    case 4: launch_tiny_fwd<4>(t, a, st); break;
    case 5: launch_tiny_fwd<5>(t, a, st); break;
    case 6: launch_tiny_fwd<6>(t, a, st); break;
    case 7: launch_tiny_fwd<7>(t, a, st); break;
    default: launch_tiny_fwd<8>(t, a, st); break;
  }
}
static_assert(kTK == 8, "launch_tiny_fwd_k instantiates 1..8 steps");

template <int C>
void launch_tiny_bwd(const diffopt_segtable* t, const TinyBwdArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((adam_unrolled_bwd_tree_tiny<C>), dim3(tiny_blocks(t)), dim3(kTinyB), 0, st, t->small, a);
}

int launch_tiny_bwd_c(const char* who, int C, const diffopt_segtable* t, const TinyBwdArgs& a, hipStream_t st) {
  switch (C) {
    case 1: launch_tiny_bwd<1>(t, a, st); break;
    case 2: launch_tiny_bwd<2>(t, a, st); break;
    case 3: launch_tiny_bwd<3>(t, a, st); break;
    case 4: launch_tiny_bwd<4>(t, a, st); break;
    case 5: launch_tiny_bwd<5>(t, a, st); break;
    case 6: launch_tiny_bwd<6>(t, a, st); break;
    case 7: launch_tiny_bwd<7>(t, a, st); break;
    case 8: launch_tiny_bwd<8>(t, a, st); break;
    default: return fail(DIFFOPT_EINVAL, "%s: recompute run of %d steps (at most %d)", who, C, kTRS);
  }
  return DIFFOPT_OK;
}

// ---- leaf-direct SGD-momentum and RMSProp ------------------------------------------
// The ops of optim_ops.hpp applied leaf by leaf, in the layout of the fused
// Adam kernels: one table tile per workgroup, one group per lane, the leaf
// address of every operand staged in the window.  Operands: the op's inputs,
// then its outputs.
template <class Op, bool KEEP>
__global__ __launch_bounds__(kUTB) void ew_tree_kernel(const SegEntry* __restrict__ seg,
                                                      const int64_t* __restrict__ tile_first, int64_t ngroups,
                                                      int dense_orig, LeafArrays<Op::NIN + Op::NOUT> arr, Op op) {
  constexpr int NA = Op::NIN + Op::NOUT;
  __shared__ int64_t s_goff[kWindowMax + 1];
  __shared__ int64_t s_numel[kWindowMax];
  __shared__ uint64_t s_ptr[NA * kWindowMax];
  const int64_t b = blockIdx.x;
  const int W = stage_window_n(seg, tile_first, arr.a, NA, dense_orig, b, s_goff, s_numel, s_ptr);
  const int64_t gidx = b * kTileGroups + threadIdx.x;
  if (gidx >= ngroups) return;
  const int t = find_leaf(s_goff, W, gidx);
  const uint64_t* P = s_ptr + t;
  on_group<KEEP>(4 * (gidx - s_goff[t]) - line_phase(P[Op::NIN * kWindowMax]), s_numel[t], [&](const auto& acc) {
    f32x4 x[Op::NIN], y[Op::NOUT];
#pragma unroll
    for (int a = 0; a < Op::NIN; ++a) x[a] = acc.load(P[a * kWindowMax]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float xi[Op::NIN], yo[Op::NOUT];
#pragma unroll
      for (int a = 0; a < Op::NIN; ++a) xi[a] = x[a][e];
      op.apply(xi, yo);
#pragma unroll
      for (int q = 0; q < Op::NOUT; ++q) y[q][e] = yo[q];
    }
    uint64_t out[Op::NOUT];
#pragma unroll
    for (int q = 0; q < Op::NOUT; ++q) out[q] = P[(Op::NIN + q) * kWindowMax];
    acc.store(out, y);
  });
}

// Small trees (a TinyTable): one element per lane, the table in the kernel
// arguments, every leaf address then every input loaded before the op, as in
// the small-tree Adam kernels; the same op.apply per element.
template <class Op>
__global__ __launch_bounds__(kTinyB) void ew_tree_tiny(TinyTable tt, LeafArrays<Op::NIN + Op::NOUT> arr, Op op) {
  warm_args(fold_lines(tt) ^ fold_lines(arr) ^ fold_lines(op));
  int leaf;
  int64_t i;
  if (!tiny_slot(tt, (int64_t)blockIdx.x * kTinyB + threadIdx.x, leaf, i)) return;
  gptr<const float> in[Op::NIN];
  gptr<float> out[Op::NOUT];
#pragma unroll
  for (int a = 0; a < Op::NIN; ++a) in[a] = leaf_in(arr.a[a], leaf);
#pragma unroll
  for (int q = 0; q < Op::NOUT; ++q) out[q] = leaf_out(arr.a[Op::NIN + q], leaf);
  float xi[Op::NIN], yo[Op::NOUT];
#pragma unroll
  for (int a = 0; a < Op::NIN; ++a) xi[a] = in[a][i];
  op.apply(xi, yo);
#pragma unroll
  for (int q = 0; q < Op::NOUT; ++q) out[q][i] = yo[q];
}

// Runner of the leaf-direct kernel for the *_variant selectors: every
// operand is a device array of leaf addresses.
struct TreeRun {
  const char* who;
  const diffopt_segtable* t;
  hipStream_t st;
  template <class Op>
  int go(const Op& op, const void* const* in, const void* const* out) {
    LeafArrays<Op::NIN + Op::NOUT> arr{};
    for (int a = 0; a < Op::NIN; ++a) arr.a[a] = static_cast<const uint64_t*>(in[a]);
    for (int q = 0; q < Op::NOUT; ++q) arr.a[Op::NIN + q] = static_cast<const uint64_t*>(out[q]);
    if (t->tiny)
      hipLaunchKernelGGL((ew_tree_tiny<Op>), dim3(tiny_blocks(t)), dim3(kTinyB), 0, st, t->small, arr, op);
    else if (keep_in_cache(4 * (int64_t)(Op::NIN + Op::NOUT) * t->elems))
      hipLaunchKernelGGL((ew_tree_kernel<Op, true>), dim3((unsigned)t->ntiles), dim3(kUTB), 0, st, t->d_seg,
                         t->d_tile_first, t->ngroups, t->dense_orig, arr, op);
    else
      hipLaunchKernelGGL((ew_tree_kernel<Op, false>), dim3((unsigned)t->ntiles), dim3(kUTB), 0, st, t->d_seg,
                         t->d_tile_first, t->ngroups, t->dense_orig, arr, op);
    return launch_status(who);
  }
};

int check_table(const char* who, const diffopt_segtable* t) {
  if (!t) return fail(DIFFOPT_EINVAL, "%s: table is NULL", who);
  if (t->elem_bytes != 4) return fail(DIFFOPT_EINVAL, "%s: the table must describe fp32 leaves (elem_bytes 4)", who);
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != t->device)
    return fail(DIFFOPT_EINVAL, "%s: the table lives on device %d, the current device is %d", who, t->device, dev);
  return DIFFOPT_OK;
}

int launch_fwd_tree(const diffopt_segtable* t, const LeafArrays<7>& arr, const AdamCoef& c, hipStream_t st) {
  if (t->ntiles == 0) return DIFFOPT_OK;
  if (keep_in_cache(28 * t->elems))
    hipLaunchKernelGGL(adam_fwd_tree_kernel<true>, dim3((unsigned)t->ntiles), dim3(kFB), 0, st, t->d_seg,
                       t->d_tile_first, t->ngroups, arr, t->dense_orig, c);
  else
    hipLaunchKernelGGL(adam_fwd_tree_kernel<false>, dim3((unsigned)t->ntiles), dim3(kFB), 0, st, t->d_seg,
                       t->d_tile_first, t->ngroups, arr, t->dense_orig, c);
  return launch_status("diffopt_adam_fwd_tree");
}

// Workgroups of the leaf-direct VJP resident per CU.  Its registers allow
// six (eight without incoming moment cotangents); with six reads and three writes per element that many oversubscribe
// the memory system, and five ran the 20,000-leaf tree's VJP 4% faster than the
// seven an earlier form allowed (four: the same; six: 1.5% slower).  The launch reserves otherwise unused dynamic
// LDS so that no more than kBwdTreeResident workgroups fit in a CU's 160 KiB.
constexpr int kBwdTreeResident = 5;
constexpr size_t kLdsPerCU = 160 * 1024;
constexpr size_t kBwdTreeStaticLds = (kWindowMax + 1) * 8 + kWindowMax * (8 + 9 * 8);
constexpr size_t kBwdTreeLdsPad = kLdsPerCU / kBwdTreeResident - kBwdTreeStaticLds - 256;
static_assert(kLdsPerCU / (kBwdTreeStaticLds + kBwdTreeLdsPad) == kBwdTreeResident,
              "the reserved LDS must leave room for exactly kBwdTreeResident workgroups");

template <int CAP>
void launch_unrolled_fwd_tree(const diffopt_segtable* t, const TFwdArgsOf<CAP>& a, hipStream_t st) {
  const size_t lds = sizeof(uint64_t) * kWindowMax * (4 + 3 * a.K);
  int64_t values = 4 + a.K;  // moved per element
  for (int s = 0; s < a.K; ++s) values += a.a[5 + 3 * s] ? 2 : 0;
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)t->ntiles), dim3(kUTB), lds, st, t->d_seg, t->d_tile_first, t->ngroups,
                       t->dense_orig, a);
  };
  if (keep_run_in_cache(4 * values * t->elems)) go(adam_unrolled_fwd_tree_kernel<true, CAP>);
  else go(adam_unrolled_fwd_tree_kernel<false, CAP>);
}

int launch_bwd_tree(const diffopt_segtable* t, const LeafArrays<9>& arr, const AdamCoef& c, hipStream_t st) {
  if (t->ntiles == 0) return DIFFOPT_OK;
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)t->ntiles), dim3(kBB), kBwdTreeLdsPad, st, t->d_seg, t->d_tile_first,
                       t->ngroups, arr, t->dense_orig, c);
  };
  if (arr.a[1])
    keep_in_cache(36 * t->elems) ? go(adam_bwd_tree_kernel<true, true>) : go(adam_bwd_tree_kernel<true, false>);
  else
    keep_in_cache(28 * t->elems) ? go(adam_bwd_tree_kernel<false, true>) : go(adam_bwd_tree_kernel<false, false>);
  return launch_status("diffopt_adam_bwd_tree");
}

}  // namespace
}  // namespace diffopt

using namespace diffopt;

extern "C" int diffopt_adam_fwd_tree(const diffopt_segtable* table, const uint64_t* params, const uint64_t* grad,
                                     const uint64_t* mu, const uint64_t* nu, int64_t count, double lr, double b1,
                                     double b2, double eps, double eps_root, const uint64_t* params_out,
                                     const uint64_t* mu_out, const uint64_t* nu_out, void* stream) {
  clear_error();
  static const char* who = "diffopt_adam_fwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  AdamCoef c;
  rc = make_coef(who, count, lr, b1, b2, eps, eps_root, &c);
  if (rc) return rc;
  if (table->ntiles == 0) return DIFFOPT_OK;
  if (!params || !grad || !mu || !nu || !params_out || !mu_out || !nu_out)
    return fail(DIFFOPT_EINVAL, "%s: null leaf-address array", who);
  if (table->tiny) {  // the fused forward at K = 1, its step state stored in the outputs
    TFwdArgs a{};
    a.K = 1;
    a.a[0] = params;
    a.a[1] = mu;
    a.a[2] = nu;
    a.a[3] = params_out;
    a.a[4] = grad;
    a.a[5] = mu_out;
    a.a[6] = nu_out;
    a.c[0] = c;
    launch_tiny_fwd<1>(table, a, as_stream(stream));
    return launch_status(who);
  }
  const LeafArrays<7> arr{{params, grad, mu, nu, params_out, mu_out, nu_out}};
  return launch_fwd_tree(table, arr, c, as_stream(stream));
}

extern "C" int diffopt_adam_bwd_tree(const diffopt_segtable* table, const uint64_t* dupdate, const uint64_t* dmu,
                                     const uint64_t* dnu, const uint64_t* grad, const uint64_t* mu,
                                     const uint64_t* nu, int64_t count, double lr, double b1, double b2, double eps,
                                     double eps_root, const uint64_t* dgrad, const uint64_t* dmu_in,
                                     const uint64_t* dnu_in, void* stream) {
  clear_error();
  static const char* who = "diffopt_adam_bwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  AdamCoef c;
  rc = make_coef(who, count, lr, b1, b2, eps, eps_root, &c);
  if (rc) return rc;
  if ((dmu == nullptr) != (dnu == nullptr))
    return fail(DIFFOPT_EINVAL, "%s: dmu and dnu must both be given or both be NULL", who);
  if (table->ntiles == 0) return DIFFOPT_OK;
  if (!dupdate || !grad || !mu || !nu || !dgrad || !dmu_in || !dnu_in)
    return fail(DIFFOPT_EINVAL, "%s: null leaf-address array", who);
  if (table->tiny) {  // the recomputing VJP over one step from the stored (mu, nu)
    TinyBwdArgs a{};
    a.init_mv = dmu != nullptr;
    a.a[0] = dupdate;
    a.a[1] = dmu;
    a.a[2] = dnu;
    a.a[3] = dmu_in;
    a.a[4] = dnu_in;
    a.a[5] = mu;
    a.a[6] = nu;
    a.a[7] = grad;
    a.a[8] = dgrad;
    a.c[0] = c;
    launch_tiny_bwd<1>(table, a, as_stream(stream));
    return launch_status(who);
  }
  const LeafArrays<9> arr{{dupdate, dmu, dnu, grad, mu, nu, dgrad, dmu_in, dnu_in}};
  return launch_bwd_tree(table, arr, c, as_stream(stream));
}

extern "C" int diffopt_adam_unrolled_fwd_tree(const diffopt_segtable* table, int64_t K, const uint64_t* p0,
                                              const uint64_t* const* grads, const uint64_t* const* mu_traj,
                                              const uint64_t* const* nu_traj, const uint64_t* pK, int64_t count0,
                                              double lr, double b1, double b2, double eps, double eps_root,
                                              void* stream) {
  clear_error();
  static const char* who = "diffopt_adam_unrolled_fwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  if (K < 1) return fail(DIFFOPT_EINVAL, "%s: K must be >= 1 (got %lld)", who, (long long)K);
  if (!grads || !mu_traj || !nu_traj) return fail(DIFFOPT_EINVAL, "%s: null pointer array", who);
  AdamCoef c;
  for (int64_t k = 1; k <= K; ++k) {
    rc = make_coef(who, count0 + k - 1, lr, b1, b2, eps, eps_root, &c);
    if (rc) return rc;
  }
  if (table->ntiles == 0) return DIFFOPT_OK;
  if (!p0 || !pK) return fail(DIFFOPT_EINVAL, "%s: null p0 or pK", who);
  for (int64_t k = 0; k < K; ++k)
    if (!grads[k]) return fail(DIFFOPT_EINVAL, "%s: null grads entry %lld", who, (long long)k);
  rc = check_trajectory(who, K, mu_traj, nu_traj, true, false);
  if (rc) return rc;
  hipStream_t st = as_stream(stream);
  // Steps k0+1..k0+steps in one launch.  Between launches the running moments
  // pass through the state stored at the boundary, or through the final-state
  // trees when it is not stored.
  const auto fill = [&](auto& a, int64_t k0, int64_t steps) {
    a.K = (int32_t)steps;
    a.a[0] = (k0 == 0) ? p0 : pK;
    a.a[1] = mu_traj[k0] ? mu_traj[k0] : mu_traj[K];
    a.a[2] = nu_traj[k0] ? nu_traj[k0] : nu_traj[K];
    a.a[3] = pK;
    for (int s = 0; s < a.K; ++s) {
      a.a[4 + 3 * s] = grads[k0 + s];
      a.a[5 + 3 * s] = mu_traj[k0 + s + 1];
      a.a[6 + 3 * s] = nu_traj[k0 + s + 1];
      make_coef(who, count0 + k0 + s, lr, b1, b2, eps, eps_root, &a.c[s]);
    }
    if (!a.a[5 + 3 * (a.K - 1)]) {
      a.a[5 + 3 * (a.K - 1)] = mu_traj[K];
      a.a[6 + 3 * (a.K - 1)] = nu_traj[K];
    }
  };
  const int64_t chunk = table->tiny ? kTK : kTLongK;
  for (int64_t k0 = 0; k0 < K; k0 += chunk) {
    const int64_t steps = K - k0 < chunk ? K - k0 : chunk;
    if (table->tiny) {
      TFwdArgs a{};
      fill(a, k0, steps);
      launch_tiny_fwd_k(table, a, st);
    } else if (steps <= kTK) {
      TFwdArgs a{};
      fill(a, k0, steps);
      launch_unrolled_fwd_tree(table, a, st);
    } else {
      TFwdArgsOf<kTLongK> a{};
      fill(a, k0, steps);
      launch_unrolled_fwd_tree(table, a, st);
    }
    rc = launch_status(who);
    if (rc) return rc;
  }
  return DIFFOPT_OK;
}

extern "C" int diffopt_adam_unrolled_bwd_tree(const diffopt_segtable* table, int64_t K, const uint64_t* dpK,
                                              const uint64_t* const* grads, const uint64_t* const* mu_traj,
                                              const uint64_t* const* nu_traj, const uint64_t* const* dgrads,
                                              const uint64_t* dmu0, const uint64_t* dnu0, int64_t count0, double lr,
                                              double b1, double b2, double eps, double eps_root, void* stream) {
  clear_error();
  static const char* who = "diffopt_adam_unrolled_bwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  if (K < 1) return fail(DIFFOPT_EINVAL, "%s: K must be >= 1 (got %lld)", who, (long long)K);
  if (!grads || !mu_traj || !nu_traj || !dgrads) return fail(DIFFOPT_EINVAL, "%s: null pointer array", who);
  AdamCoef c;
  for (int64_t k = 1; k <= K; ++k) {
    rc = make_coef(who, count0 + k - 1, lr, b1, b2, eps, eps_root, &c);
    if (rc) return rc;
  }
  if (table->ntiles == 0) return DIFFOPT_OK;
  if (!dpK || !dmu0 || !dnu0) return fail(DIFFOPT_EINVAL, "%s: null dpK, dmu0 or dnu0", who);
  if (dmu0 == dnu0) return fail(DIFFOPT_EINVAL, "%s: dmu0 and dnu0 must be distinct", who);
  for (int64_t k = 0; k < K; ++k)
    if (!grads[k] || !dgrads[k])
      return fail(DIFFOPT_EINVAL, "%s: null entry %lld in grads or dgrads", who, (long long)k);
  rc = check_trajectory(who, K, mu_traj, nu_traj, false, true);
  if (rc) return rc;
  hipStream_t st = as_stream(stream);
  // Last steps first: runs of steps whose input states are stored take one
  // launch per kTK steps; a run j+1..khi after one stored state j takes one
  // launch that recomputes the states it needs, two neighbouring ones together
  // where they stream from memory (TwoRuns).
  for (int64_t khi = K; khi >= 1;) {
    const int32_t init_mv = khi != K;  // the first launch starts from zero cotangents of mu_K, nu_K
    if (mu_traj[khi - 1]) {
      int32_t run = 0;
      while (run < kTK && khi - run >= 1 && mu_traj[khi - run - 1]) ++run;
      if (table->tiny && run == 1) {  // one step from its stored state: the small form at C = 1
        TinyBwdArgs a{};
        a.init_mv = init_mv;
        a.a[0] = dpK;
        a.a[1] = dmu0;
        a.a[2] = dnu0;
        a.a[3] = dmu0;
        a.a[4] = dnu0;
        a.a[5] = mu_traj[khi - 1];
        a.a[6] = nu_traj[khi - 1];
        a.a[7] = grads[khi - 1];
        a.a[8] = dgrads[khi - 1];
        make_coef(who, count0 + khi - 1, lr, b1, b2, eps, eps_root, &a.c[0]);
        launch_tiny_bwd<1>(table, a, st);
        khi -= 1;
        rc = launch_status(who);
        if (rc) return rc;
        continue;
      }
      TBwdArgs a{};
      a.K = run;
      a.init_mv = init_mv;
      a.a[0] = dpK;
      a.a[1] = dmu0;
      a.a[2] = dnu0;
      for (int s = 0; s < a.K; ++s) {
        const int64_t k = khi - s;  // unrolled step (1-based) run as the launch's step s
        a.a[3 + 4 * s] = grads[k - 1];
        a.a[4 + 4 * s] = mu_traj[k - 1];
        a.a[5 + 4 * s] = nu_traj[k - 1];
        a.a[6 + 4 * s] = dgrads[k - 1];
        make_coef(who, count0 + k - 1, lr, b1, b2, eps, eps_root, &a.c[s]);
      }
      const size_t lds = sizeof(uint64_t) * kWindowMax * (3 + 4 * a.K);
      const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)table->ntiles), dim3(kUTB), lds, st, table->d_seg,
                           table->d_tile_first, table->ngroups, table->dense_orig, a);
      };
      if (keep_run_in_cache((12 + 16 * a.K + (init_mv ? 8 : 0)) * table->elems)) go(adam_unrolled_bwd_tree_kernel<true>);
      else go(adam_unrolled_bwd_tree_kernel<false>);
      khi -= run;
    } else {
      int64_t j = khi - 1;
      while (!mu_traj[j]) --j;  // mu_traj[0] is stored; check_trajectory bounds khi - j by kTRS
      const int C = (int)(khi - j);
      if (table->tiny) {
        TinyBwdArgs a{};
        a.init_mv = init_mv;
        a.a[0] = dpK;
        a.a[1] = dmu0;
        a.a[2] = dnu0;
        a.a[3] = dmu0;
        a.a[4] = dnu0;
        a.a[5] = mu_traj[j];
        a.a[6] = nu_traj[j];
        for (int s = 0; s < C; ++s) {
          a.a[7 + 2 * s] = grads[j + s];
          a.a[8 + 2 * s] = dgrads[j + s];
          make_coef(who, count0 + j + s, lr, b1, b2, eps, eps_root, &a.c[s]);
        }
        rc = launch_tiny_bwd_c(who, C, table, a, st);
        if (rc) return rc;
        khi = j;
        rc = launch_status(who);
        if (rc) return rc;
        continue;
      }
      int64_t i = j;  // start of the run before it, if that is recomputed too: both in one launch
      if (j >= 1 && !mu_traj[j - 1])
        while (i == j || !mu_traj[i]) --i;
      if (i < j && C <= kTwoRunSteps && j - i <= kTwoRunSteps &&
          !keep_run_in_cache((20 + 8 * C + (init_mv ? 8 : 0)) * table->elems)) {
        TwoRuns{who, table, st, dpK, dmu0, dnu0, grads, mu_traj, nu_traj, dgrads, count0, lr, b1, b2, eps, eps_root,
                {j, i}, {C, (int)(j - i)}, init_mv}.run();
        khi = i;
        rc = launch_status(who);
        if (rc) return rc;
        continue;
      }
      TRBwdArgs a{};
      a.init_mv = init_mv;
      a.a[0] = dpK;
      a.a[1] = dmu0;
      a.a[2] = dnu0;
      a.a[3] = mu_traj[j];
      a.a[4] = nu_traj[j];
      for (int s = 0; s < C; ++s) {
        a.a[5 + 2 * s] = grads[j + s];
        a.a[6 + 2 * s] = dgrads[j + s];
        make_coef(who, count0 + j + s, lr, b1, b2, eps, eps_root, &a.c[s]);
      }
      rc = launch_trbwd_c(who, C, table, a, st);
      if (rc) return rc;
      khi = j;
    }
    rc = launch_status(who);
    if (rc) return rc;
  }
  return DIFFOPT_OK;
}

// ---- leaf-direct SGD-momentum and RMSProp entry points ---------------------------------

static int check_sgd_hyper(const char* who, double lr, double momentum) {
  if (!std::isfinite(lr)) return fail(DIFFOPT_EINVAL, "%s: lr must be finite", who);
  if (!(momentum >= 0.0 && std::isfinite(momentum)))
    return fail(DIFFOPT_EINVAL, "%s: momentum must be finite and >= 0", who);
  return DIFFOPT_OK;
}

extern "C" int diffopt_sgd_fwd_tree(const diffopt_segtable* table, const uint64_t* params, const uint64_t* grad,
                                    const uint64_t* trace, double lr, double momentum, int32_t nesterov,
                                    const uint64_t* params_out, const uint64_t* trace_out, void* stream) {
  clear_error();
  static const char* who = "diffopt_sgd_fwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  rc = check_sgd_hyper(who, lr, momentum);
  if (rc) return rc;
  if (table->ntiles == 0) return DIFFOPT_OK;
  const bool mom = momentum > 0.0;
  if (!params || !grad || !params_out || (mom && !trace_out))
    return fail(DIFFOPT_EINVAL, "%s: null leaf-address array", who);
  TreeRun run{who, table, as_stream(stream)};
  return sgd_fwd_variant(run, params, grad, mom ? trace : nullptr, params_out, mom ? trace_out : nullptr, lr,
                         momentum, nesterov != 0);
}

extern "C" int diffopt_sgd_bwd_tree(const diffopt_segtable* table, const uint64_t* dparams_out,
                                    const uint64_t* dtrace_out, double lr, double momentum, int32_t nesterov,
                                    const uint64_t* dgrad, const uint64_t* dtrace_in, void* stream) {
  clear_error();
  static const char* who = "diffopt_sgd_bwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  rc = check_sgd_hyper(who, lr, momentum);
  if (rc) return rc;
  if (table->ntiles == 0) return DIFFOPT_OK;
  const bool mom = momentum > 0.0;
  if (!dparams_out || !dgrad || (mom && !dtrace_in)) return fail(DIFFOPT_EINVAL, "%s: null leaf-address array", who);
  TreeRun run{who, table, as_stream(stream)};
  return sgd_bwd_variant(run, dparams_out, mom ? dtrace_out : nullptr, dgrad, mom ? dtrace_in : nullptr, lr,
                         momentum, nesterov != 0);
}

extern "C" int diffopt_rmsprop_fwd_tree(const diffopt_segtable* table, const uint64_t* params, const uint64_t* grad,
                                        const uint64_t* nu, const uint64_t* mom, double lr, double alpha, double eps,
                                        double eps_root, double momentum, const uint64_t* params_out,
                                        const uint64_t* nu_out, const uint64_t* mom_out, void* stream) {
  clear_error();
  static const char* who = "diffopt_rmsprop_fwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  RmsCoef c;
  rc = rms_coef(who, lr, alpha, eps, eps_root, momentum, &c);
  if (rc) return rc;
  if (table->ntiles == 0) return DIFFOPT_OK;
  const bool m = momentum > 0.0;
  if (!params || !grad || !nu || !params_out || !nu_out || (m && !mom_out))
    return fail(DIFFOPT_EINVAL, "%s: null leaf-address array", who);
  TreeRun run{who, table, as_stream(stream)};
  return rms_fwd_variant(run, params, grad, nu, m ? mom : nullptr, params_out, nu_out, m ? mom_out : nullptr, c, m);
}

extern "C" int diffopt_rmsprop_bwd_tree(const diffopt_segtable* table, const uint64_t* dparams_out,
                                        const uint64_t* dnu_out, const uint64_t* dmom_out, const uint64_t* grad,
                                        const uint64_t* nu, double lr, double alpha, double eps, double eps_root,
                                        double momentum, const uint64_t* dgrad, const uint64_t* dnu_in,
                                        const uint64_t* dmom_in, void* stream) {
  clear_error();
  static const char* who = "diffopt_rmsprop_bwd_tree";
  int rc = check_table(who, table);
  if (rc) return rc;
  RmsCoef c;
  rc = rms_coef(who, lr, alpha, eps, eps_root, momentum, &c);
  if (rc) return rc;
  if (table->ntiles == 0) return DIFFOPT_OK;
  const bool m = momentum > 0.0;
  if (!dparams_out || !grad || !nu || !dgrad || !dnu_in || (m && !dmom_in))
    return fail(DIFFOPT_EINVAL, "%s: null leaf-address array", who);
  TreeRun run{who, table, as_stream(stream)};
  return rms_bwd_variant(run, dparams_out, dnu_out, m ? dmom_out : nullptr, grad, nu, dgrad, dnu_in,
                         m ? dmom_in : nullptr, c, m);
}
