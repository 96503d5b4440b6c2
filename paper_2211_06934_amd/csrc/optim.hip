// The paper's other fused differentiable optimizers on gfx950, over flat
// buffers: SGD with momentum (optionally Nesterov) and RMSProp (optionally
// with momentum), each a fused forward and a fused VJP (TorchOpt, Sec. 1
// contribution (2)(i) and Sec. 2.3 "CPU/GPU-accelerated optimizers"); the
// arithmetic is in optim_ops.hpp.
// Like Adam they are HBM-bound elementwise streams; they share one generic
// kernel skeleton with the measured Adam launch shape (1024-thread workgroups,
// 512 for calls that fit the Infinity Cache, one 4-element vector per lane per
// array, vectors counted from a line boundary of the first output).
#include <cmath>
#include <initializer_list>

#include "optim_ops.hpp"

namespace diffopt {
namespace {

// Threads per workgroup of the calls that stream from memory and of those small
// enough for the Infinity Cache (measured with Adam's, see adam.hip).
constexpr int kStreamB = 1024;
constexpr int kKeepB = 512;

template <int NIN, int NOUT>
struct Streams {
  const float* in[NIN > 0 ? NIN : 1];
  float* out[NOUT];
};

template <class Op, int B, bool KEEP>
__global__ __launch_bounds__(B) void ew_vec(Streams<Op::NIN, Op::NOUT> s, int64_t n, int64_t head, Op op) {
  const int64_t nv = n >> 2;
  const int64_t ntiles = (nv + B - 1) / B;
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t i = t * B + threadIdx.x;
    if (i >= nv) continue;
    f32x4 x[Op::NIN];
#pragma unroll
    for (int a = 0; a < Op::NIN; ++a) x[a] = ld4<KEEP>(s.in[a] + 4 * i);
    f32x4 y[Op::NOUT];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float xi[Op::NIN], yo[Op::NOUT];
#pragma unroll
      for (int a = 0; a < Op::NIN; ++a) xi[a] = x[a][e];
      op.apply(xi, yo);
#pragma unroll
      for (int b = 0; b < Op::NOUT; ++b) y[b][e] = yo[b];
    }
#pragma unroll
    for (int b = 0; b < Op::NOUT; ++b) st4(s.out[b] + 4 * i, y[b]);
  }
  if (blockIdx.x == gridDim.x - 1) {
    int64_t e;
    if (edge_element<B>(n, head, e)) {
      float xi[Op::NIN], yo[Op::NOUT];
#pragma unroll
      for (int a = 0; a < Op::NIN; ++a) xi[a] = s.in[a][e];
      op.apply(xi, yo);
#pragma unroll
      for (int b = 0; b < Op::NOUT; ++b) s.out[b][e] = yo[b];
    }
  }
}

template <class Op>
int launch(const char* who, Streams<Op::NIN, Op::NOUT> s, int64_t n, const Op& op, hipStream_t st) {
  if (n == 0) return DIFFOPT_OK;
  const int64_t h = line_head(s.out[0], n);
  for (int a = 0; a < Op::NIN; ++a) s.in[a] += h;
  for (int b = 0; b < Op::NOUT; ++b) s.out[b] += h;
  n -= h;
  const bool keep = keep_in_cache(4 * (int64_t)(Op::NIN + Op::NOUT) * n);
  const int block = keep ? kKeepB : kStreamB;
  int64_t tiles = ((n >> 2) + block - 1) / block;
  if (tiles < 1) tiles = 1;
  if (tiles > 0x7fffffff) tiles = 0x7fffffff;
  if (keep)
    hipLaunchKernelGGL((ew_vec<Op, kKeepB, true>), dim3((unsigned)tiles), dim3(block), 0, st, s, n, h, op);
  else
    hipLaunchKernelGGL((ew_vec<Op, kStreamB, false>), dim3((unsigned)tiles), dim3(block), 0, st, s, n, h, op);
  return launch_status(who);
}

bool aligned4(const void* p) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

int check_ptrs(const char* who, std::initializer_list<const void*> ps) {
  for (const void* q : ps)
    if (!aligned4(q)) return fail(DIFFOPT_EINVAL, "%s: pointer %p is not 4-byte aligned", who, q);
  return DIFFOPT_OK;
}

// Runner of the flat-buffer kernels for the *_variant selectors.
struct FlatRun {
  const char* who;
  int64_t n;
  hipStream_t st;
  template <class Op>
  int go(const Op& op, const void* const* in, const void* const* out) {
    Streams<Op::NIN, Op::NOUT> s{};
    for (int a = 0; a < Op::NIN; ++a) s.in[a] = static_cast<const float*>(in[a]);
    for (int b = 0; b < Op::NOUT; ++b) s.out[b] = static_cast<float*>(const_cast<void*>(out[b]));
    return launch(who, s, n, op, st);
  }
};

}  // namespace
}  // namespace diffopt

using namespace diffopt;

extern "C" int diffopt_sgd_fwd(const float* params, const float* grad, const float* trace, int64_t n, double lr,
                               double momentum, int32_t nesterov, float* params_out, float* trace_out, void* stream) {
  clear_error();
  static const char* who = "diffopt_sgd_fwd";
  if (n < 0) return fail(DIFFOPT_EINVAL, "%s: n must be >= 0", who);
  if (!std::isfinite(lr)) return fail(DIFFOPT_EINVAL, "%s: lr must be finite", who);
  if (!(momentum >= 0.0 && std::isfinite(momentum)))
    return fail(DIFFOPT_EINVAL, "%s: momentum must be finite and >= 0", who);
  if (n == 0) return DIFFOPT_OK;
  const bool mom = momentum > 0.0;
  if (!params || !grad || !params_out || (mom && !trace_out))
    return fail(DIFFOPT_EINVAL, "%s: null required pointer", who);
  int rc = check_ptrs(who, {params, grad, trace, params_out, trace_out});
  if (rc) return rc;
  FlatRun run{who, n, as_stream(stream)};
  return sgd_fwd_variant(run, params, grad, trace, params_out, trace_out, lr, momentum, nesterov != 0);
}

extern "C" int diffopt_sgd_bwd(const float* dparams_out, const float* dtrace_out, int64_t n, double lr,
                               double momentum, int32_t nesterov, float* dgrad, float* dtrace_in, void* stream) {
  clear_error();
  static const char* who = "diffopt_sgd_bwd";
  if (n < 0) return fail(DIFFOPT_EINVAL, "%s: n must be >= 0", who);
  if (!std::isfinite(lr)) return fail(DIFFOPT_EINVAL, "%s: lr must be finite", who);
  if (!(momentum >= 0.0 && std::isfinite(momentum)))
    return fail(DIFFOPT_EINVAL, "%s: momentum must be finite and >= 0", who);
  if (n == 0) return DIFFOPT_OK;
  const bool mom = momentum > 0.0;
  if (!dparams_out || !dgrad || (mom && !dtrace_in)) return fail(DIFFOPT_EINVAL, "%s: null required pointer", who);
  int rc = check_ptrs(who, {dparams_out, dtrace_out, dgrad, dtrace_in});
  if (rc) return rc;
  FlatRun run{who, n, as_stream(stream)};
  return sgd_bwd_variant(run, dparams_out, dtrace_out, dgrad, dtrace_in, lr, momentum, nesterov != 0);
}

extern "C" int diffopt_rmsprop_fwd(const float* params, const float* grad, const float* nu, const float* mom,
                                   int64_t n, double lr, double alpha, double eps, double eps_root, double momentum,
                                   float* params_out, float* nu_out, float* mom_out, void* stream) {
  clear_error();
  static const char* who = "diffopt_rmsprop_fwd";
  if (n < 0) return fail(DIFFOPT_EINVAL, "%s: n must be >= 0", who);
  RmsCoef c;
  int rc = rms_coef(who, lr, alpha, eps, eps_root, momentum, &c);
  if (rc) return rc;
  if (n == 0) return DIFFOPT_OK;
  const bool m = momentum > 0.0;
  if (!params || !grad || !nu || !params_out || !nu_out || (m && !mom_out))
    return fail(DIFFOPT_EINVAL, "%s: null required pointer", who);
  rc = check_ptrs(who, {params, grad, nu, mom, params_out, nu_out, mom_out});
  if (rc) return rc;
  FlatRun run{who, n, as_stream(stream)};
  return rms_fwd_variant(run, params, grad, nu, mom, params_out, nu_out, mom_out, c, m);
}

extern "C" int diffopt_rmsprop_bwd(const float* dparams_out, const float* dnu_out, const float* dmom_out,
                                   const float* grad, const float* nu, int64_t n, double lr, double alpha, double eps,
                                   double eps_root, double momentum, float* dgrad, float* dnu_in, float* dmom_in,
                                   void* stream) {
  clear_error();
  static const char* who = "diffopt_rmsprop_bwd";
  if (n < 0) return fail(DIFFOPT_EINVAL, "%s: n must be >= 0", who);
  RmsCoef c;
  int rc = rms_coef(who, lr, alpha, eps, eps_root, momentum, &c);
  if (rc) return rc;
  if (n == 0) return DIFFOPT_OK;
  const bool m = momentum > 0.0;
  if (!dparams_out || !grad || !nu || !dgrad || !dnu_in || (m && !dmom_in))
    return fail(DIFFOPT_EINVAL, "%s: null required pointer", who);
  rc = check_ptrs(who, {dparams_out, dnu_out, dmom_out, grad, nu, dgrad, dnu_in, dmom_in});
  if (rc) return rc;
  FlatRun run{who, n, as_stream(stream)};
  return rms_bwd_variant(run, dparams_out, dnu_out, m ? dmom_out : nullptr, grad, nu, dgrad, dnu_in, dmom_in, c, m);
}
