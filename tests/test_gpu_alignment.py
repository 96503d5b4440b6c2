"""The kernels on buffers at any element offset: slices of larger buffers, in
one phase of the 128-byte lines or each in its own, give the aligned run's
results bit for bit and touch nothing around them.  Sizes sit at the edges of
the head and tail handling (heads of up to 31 elements, n % 4 tails, buffers
shorter than a line) and on both sides of the cached-call limit of each step."""
import os
import re

import pytest
import torch

pytestmark = pytest.mark.gpu

HYPER = (7, 1e-3, 0.9, 0.999, 1e-8, 1e-9)
PHASES = [[1] * 12, [4] * 12, [31] * 12, [1, 2, 3, 0, 5, 6, 7, 30, 9, 10, 31, 12], [0] * 6 + [3] * 6, [3] * 6 + [0] * 6]
GUARD = 40


def _values(count, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.empty(n, device="cuda").normal_(0.0, 0.1, generator=gen) for _ in range(count)]


class _Slices:
    """Copies of inputs, and outputs, at given element offsets of guarded buffers."""

    def __init__(self, phases):
        self.phases = list(phases)
        self.bufs = []

    def _buf(self, n):
        off = 32 + self.phases[len(self.bufs) % len(self.phases)]
        buf = torch.full((off + n + GUARD,), 7.0, device="cuda")
        self.bufs.append((buf, off, n))
        return buf[off:off + n]

    def take(self, x):
        y = self._buf(x.numel())
        y.copy_(x)
        return y

    def out(self, n):
        return self._buf(n)

    def check_guards(self):
        for buf, off, n in self.bufs:
            assert torch.all(buf[:off] == 7.0) and torch.all(buf[off + n:] == 7.0)


def _adam(P, x, S, n):
    p, g, m, v, dp, dm, dv = [S.take(t) for t in x]
    outs = [S.out(n) for _ in range(7)]
    P.adam_fwd(p, g, m, v, *HYPER, outs[0], outs[1], outs[2], update_out=outs[3])
    P.adam_bwd(dp, dm, dv, g, m, v, *HYPER, None, outs[4], outs[5], outs[6])
    zero = [S.out(n) for _ in range(4)]
    P.adam_bwd(dp, None, None, g, m, v, *HYPER, zero[3], zero[0], zero[1], zero[2])
    return outs + zero


def _sgd(P, x, S, n):
    p, g, t, dp, dt = [S.take(t) for t in x[:5]]
    outs = [S.out(n) for _ in range(4)]
    P.sgd_fwd(p, g, t, 0.1, 0.9, True, outs[0], outs[1])
    P.sgd_bwd(dp, dt, 0.1, 0.9, True, outs[2], outs[3])
    return outs


def _rmsprop(P, x, S, n):
    p, g, v, b, dp, dv, db = [S.take(t) for t in x]
    outs = [S.out(n) for _ in range(6)]
    h = (0.01, 0.99, 1e-8, 1e-9, 0.9)
    P.rmsprop_fwd(p, g, v, b, *h, outs[0], outs[1], outs[2])
    P.rmsprop_bwd(dp, dv, db, g, v, *h, outs[3], outs[4], outs[5])
    return outs


STEPS = {"adam": _adam, "sgd": _sgd, "rmsprop": _rmsprop}


@pytest.mark.parametrize("step", sorted(STEPS))
@pytest.mark.parametrize("n", [1, 3, 30, 31, 33, 64, 2047, 2053, 300_001, 6_000_000, 10_000_003])
def test_flat_steps_at_any_phase(step, n):
    import paper_2211_06934_amd as P
    x = _values(7, n, n % 1000)
    x[2].abs_()
    x[3].abs_()
    ref = STEPS[step](P, x, _Slices([0]), n)
    for phases in PHASES if n < 1_000_000 else PHASES[:1] + PHASES[3:4]:
        S = _Slices(phases)
        got = STEPS[step](P, x, S, n)
        torch.cuda.synchronize()
        for k, (a, b) in enumerate(zip(got, ref)):
            assert torch.equal(a, b), (step, n, phases, k)
        S.check_guards()


@pytest.mark.parametrize("n", [65_536, 65_537, 65_566, 300_003])
@pytest.mark.parametrize("K,kept", [(3, {3}), (3, {1, 2, 3}), (10, {5, 10}), (18, {8, 9, 16, 18})])
def test_unrolled_driver_at_any_phase(n, K, kept):
    # n at the small-buffer limit: a head must not push a call to the small
    # kernels, which take no head
    import paper_2211_06934_amd as P
    x = _values(K + 4, n, 5)
    x[2].abs_()

    def run(S):
        p, m, v, cot = [S.take(t) for t in x[:4]]
        g = [S.take(t) for t in x[4:]]
        mu = [m] + [S.out(n) if k in kept else None for k in range(1, K + 1)]
        nu = [v] + [S.out(n) if k in kept else None for k in range(1, K + 1)]
        pK, dg, dm, dv = S.out(n), [S.out(n) for _ in range(K)], S.out(n), S.out(n)
        P.adam_unrolled_fwd(p, g, mu, nu, pK, *HYPER)
        P.adam_unrolled_bwd(cot, g, mu, nu, dg, dm, dv, *HYPER)
        torch.cuda.synchronize()
        S.check_guards()
        return [pK, dm, dv, *dg, *(mu[k] for k in sorted(kept)), *(nu[k] for k in sorted(kept))]

    ref = run(_Slices([0]))
    for phases in PHASES:
        for k, (a, b) in enumerate(zip(run(_Slices(phases)), ref)):
            assert torch.equal(a, b), (n, K, phases, k)


def _trees(P, sizes, phases, values):
    """One tree per row of values: its leaves one after another in a guarded buffer, each tree at its own element phase."""
    table = P.segtable_create(sizes)
    S = _Slices(phases)
    flats = [S.take(x) if x is not None else S.out(sum(sizes)) for x in values]
    starts = [0]
    for k in sizes[:-1]:
        starts.append(starts[-1] + k)
    ptrs = [torch.tensor([f.data_ptr() + 4 * o for o in starts], dtype=torch.int64).cuda() for f in flats]
    return table, S, flats, ptrs


# tiled kernels (over 32 leaves): empty, tiny and line-sized leaves around tile
# edges, each tree's leaves at its own phases
TREE_SIZES = [0, 1, 2, 3, 4, 5, 31, 32, 33, 64, 100, 127, 2048, 2049, 7, 1, 0, 12345] + [1, 3, 513, 6] * 6
# above the cached-call limit of every step (the smallest moves 16 bytes per
# element) and of the K-step driver: the streaming forms
LARGE_TREE_SIZES = TREE_SIZES[:14] + [10_600_001] + TREE_SIZES[14:]


def limit_bytes(name):
    """A size limit of the dispatch rules, from the source that states it."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    text = open(os.path.join(root, "paper_2211_06934_amd", "csrc", "adam_math.hpp")).read()
    return int(re.search(r"constexpr int64_t %s = int64_t\((\d+)\) << 20;" % name, text).group(1)) << 20


@pytest.mark.parametrize("sizes,phases", [(TREE_SIZES, p) for p in PHASES] +
                         [(LARGE_TREE_SIZES, p) for p in (PHASES[0], PHASES[3])])
def test_leaf_direct_steps_at_any_phase(sizes, phases):
    import paper_2211_06934_amd as P
    n, K = sum(sizes), 10
    if sizes is LARGE_TREE_SIZES:
        assert 16 * n > limit_bytes("kKeepBytes") and 60 * n > limit_bytes("kKeepRunBytes")
    x = _values(8 + K, n, 11)
    x[2].abs_()
    x[3].abs_()
    p, g, m, v, dp, dm, dv = x[:7]

    flat = {}
    S = _Slices([0])
    flat["adam"] = _adam(P, x[:7], S, n)
    flat["sgd"] = _sgd(P, x[:7], S, n)
    flat["rmsprop"] = _rmsprop(P, x[:7], S, n)

    t, S, f, a = _trees(P, sizes, phases, [p, g, m, v, dp, dm, dv] + [None] * 9)
    P.adam_fwd_tree(t, a[0], a[1], a[2], a[3], *HYPER, a[7], a[8], a[9])
    P.adam_bwd_tree(t, a[4], a[5], a[6], a[1], a[2], a[3], *HYPER, a[10], a[11], a[12])
    P.adam_bwd_tree(t, a[4], None, None, a[1], a[2], a[3], *HYPER, a[13], a[14], a[15])
    torch.cuda.synchronize()
    for k, i in enumerate([0, 1, 2, 4, 5, 6, 7, 8, 9]):
        assert torch.equal(f[7 + k], flat["adam"][i]), ("adam", k)
    S.check_guards()

    t, S, f, a = _trees(P, sizes, phases, [p, g, m, v, dp] + [None] * 4)
    P.sgd_fwd_tree(t, a[0], a[1], a[2], 0.1, 0.9, True, a[5], a[6])
    P.sgd_bwd_tree(t, a[3], a[4], 0.1, 0.9, True, a[7], a[8])
    torch.cuda.synchronize()
    for k in range(4):
        assert torch.equal(f[5 + k], flat["sgd"][k]), ("sgd", k)
    S.check_guards()

    h = (0.01, 0.99, 1e-8, 1e-9, 0.9)
    t, S, f, a = _trees(P, sizes, phases, [p, g, m, v, dp, dm, dv] + [None] * 6)
    P.rmsprop_fwd_tree(t, a[0], a[1], a[2], a[3], *h, a[7], a[8], a[9])
    P.rmsprop_bwd_tree(t, a[4], a[5], a[6], a[1], a[2], *h, a[10], a[11], a[12])
    torch.cuda.synchronize()
    for k in range(6):
        assert torch.equal(f[7 + k], flat["rmsprop"][k]), ("rmsprop", k)
    S.check_guards()

    for kept in ({5, 10}, set(range(1, K + 1))):
        S = _Slices([0])
        mu = [m] + [S.out(n) if k in kept else None for k in range(1, K + 1)]
        nu = [v] + [S.out(n) if k in kept else None for k in range(1, K + 1)]
        pK, dg, d0, d1 = S.out(n), [S.out(n) for _ in range(K)], S.out(n), S.out(n)
        P.adam_unrolled_fwd(p, x[8:], mu, nu, pK, *HYPER)
        P.adam_unrolled_bwd(dp, x[8:], mu, nu, dg, d0, d1, *HYPER)
        order = sorted(kept)
        t, S, f, a = _trees(P, sizes, phases, [p, m, v, dp, *x[8:]] + [None] * (3 + K + 2 * len(kept)))
        at = 4 + K + 3 + K
        tmu = [a[1]] + [a[at + order.index(k)] if k in kept else None for k in range(1, K + 1)]
        tnu = [a[2]] + [a[at + len(kept) + order.index(k)] if k in kept else None for k in range(1, K + 1)]
        tg, out, tdg = a[4:4 + K], 4 + K, a[4 + K + 3:at]
        P.adam_unrolled_fwd_tree(t, a[0], tg, tmu, tnu, a[out], *HYPER)
        P.adam_unrolled_bwd_tree(t, a[3], tg, tmu, tnu, tdg, a[out + 1], a[out + 2], *HYPER)
        torch.cuda.synchronize()
        for k, (got, want) in enumerate(zip(f[out:], [pK, d0, d1, *dg, *(mu[k] for k in order), *(nu[k] for k in order)])):
            assert torch.equal(got, want), ("unrolled", sorted(kept), k)
        S.check_guards()
