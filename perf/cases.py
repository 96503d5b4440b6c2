"""The work a user of this framework has it do, as cases that can be timed and checked.

Every case goes through public entry points of ``paper_2211_06934_amd`` on
device memory that the caller owns, the way a program that uses them calls
them: its buffers, leaf-address arrays and segment tables are made once, its
values change from call to call.  Seven kinds of work, which between them
cover the framework's operators in both directions:

  step_flat    one differentiable optimizer step and its VJP on a flat buffer
  step_tree    the same on a parameter tree, leaf by leaf (no flattening)
  unroll_pack  pack p and K gradient trees, K fused Adam steps, their VJP, unpack
  unroll_tree  K fused Adam steps and their VJP on the leaves themselves
  meta         Listing 1's inner loop on a module (MetaAdam and its siblings)
  es           the zero-order estimator: perturbed points, then the estimate
  copy         tree.flatten and tree.unflatten of a parameter tree

A tree's leaves lie in one arena per operand: ``separate`` leaves start on
512-byte boundaries, as torch's allocator places a module's parameters;
``packed`` leaves follow one another without a gap, as parameters that are
views of one flat buffer do.  Outputs that are trees come back as their arena
(zeros in the gaps).
"""
import math

import numpy as np
import torch

import paper_2211_06934_amd as P

HYPER = dict(lr=1e-3, b1=0.9, b2=0.999, eps=1e-8)
REMAT_SPAN = 8  # longest run of unrolled steps whose moments the VJP recomputes
PAPER_SEED = 20221112


# ---- trees ------------------------------------------------------------------


def _convnet():
    sizes, c = [], 1
    for _ in range(4):
        sizes += [64 * c * 9, 64, 64, 64]
        c = 64
    return sizes + [5 * 64, 5]


def _resnet18():
    sizes, cin = [64 * 3 * 49, 64, 64], 64
    for cout, stride in ((64, 1), (128, 2), (256, 2), (512, 2)):
        for block in range(2):
            sizes += [cout * cin * 9, cout, cout, cout * cout * 9, cout, cout]
            if block == 0 and (stride != 1 or cin != cout):
                sizes += [cout * cin, cout, cout]
            cin = cout
    return sizes + [1000 * 512, 1000]


def _sizes(case):
    """Elements of each leaf: a network of this repository's workloads, or
    leaves of log-uniform size."""
    tree = case["tree"]
    if tree == "mlp":
        return [40, 40, 1600, 40, 40, 1]
    if tree == "convnet":
        return _convnet()
    if tree == "convnet32":
        return _convnet() * 32
    if tree == "resnet18":
        return _resnet18()
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([PAPER_SEED, 4, int(case["tree_seed"])])))
    x = np.exp(rng.uniform(0.0, math.log(case["max_leaf"]), size=case["leaves"]))
    return [int(v) for v in np.clip(np.rint(x), 1, case["max_leaf"]).astype(np.int64)]


class _Layout:
    """Where a tree's leaves lie in an arena of 4-byte elements."""

    def __init__(self, sizes, layout, elem=4):
        numel = np.asarray(sizes, dtype=np.int64)
        step = 512 // elem if layout == "separate" else 1
        room = (numel + step - 1) // step * step
        self.numel = [int(v) for v in numel]
        self.start = np.concatenate([[0], np.cumsum(room)[:-1]])
        self.total = int(room.sum())
        self.n = int(numel.sum())
        self.offsets = torch.from_numpy(self.start * elem).to("cuda")

    def ptrs(self, arena):
        """Device array of the leaves' addresses in this arena."""
        return self.offsets + arena.data_ptr()

    def inside(self):
        """Mask of the arena's elements that belong to a leaf."""
        edge = torch.zeros(self.total + 1, dtype=torch.int32, device="cuda")
        at = torch.from_numpy(self.start).to("cuda")
        end = torch.from_numpy(self.start + np.asarray(self.numel)).to("cuda")
        one = torch.ones(len(self.numel), dtype=torch.int32, device="cuda")
        edge.index_add_(0, at, one)
        edge.index_add_(0, end, -one)
        return edge[:-1].cumsum(0) > 0


# ---- inputs -----------------------------------------------------------------


class _Draw:
    """Seeded normal draws on the device."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed) * 7919 + 17)

    def __call__(self, n, std, offset=0):
        x = torch.empty(n + offset, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=self.gen)
        return x[offset:]


def _new(n, offset=0):
    return torch.zeros(n + offset, dtype=torch.float32, device="cuda")[offset:]


def _stored(K):
    """Moment states the caller keeps: the last one and as few evenly spaced
    others as the VJP needs."""
    runs = -(-K // REMAT_SPAN)
    return {(K * r) // runs for r in range(1, runs)} | {K}


# ---- the cases --------------------------------------------------------------


def listed():
    return [
        # A few-shot regression learner's inner loop replayed on recorded gradients: the smallest tree, where
        # launches and latency are all there is.
        {"name": "unroll_tree_mlp_k5", "kind": "unroll_tree", "tree": "mlp", "layout": "separate", "K": 5, "warm": False},
        # The same on an image network, a long inner loop (two recompute runs in the VJP).
        {"name": "unroll_tree_resnet18_k10", "kind": "unroll_tree", "tree": "resnet18", "layout": "separate", "K": 10, "warm": False},
        # A very wide tree (many small modules) run through the flat form: batched pack, fused steps, batched unpack.
        {"name": "unroll_pack_20000_k3", "kind": "unroll_pack", "tree": "loguniform", "leaves": 20000, "max_leaf": 65536, "tree_seed": 0,
         "layout": "separate", "K": 3, "warm": False},
        # An interior Adam step of a live loop on that tree, leaf by leaf, forward and VJP.
        {"name": "step_tree_adam_20000", "kind": "step_tree", "opt": "adam", "tree": "loguniform", "leaves": 20000, "max_leaf": 65536, "tree_seed": 0,
         "layout": "separate"},
        # RMSProp with momentum on 32 task copies of a conv-net whose parameters are views of one flat buffer (odd offsets).
        {"name": "step_tree_rmsprop_packed", "kind": "step_tree", "opt": "rmsprop", "tree": "convnet32", "layout": "packed"},
        # The largest flat buffer: one interior Adam step with every cotangent, forward and VJP.
        {"name": "step_flat_adam_1e9", "kind": "step_flat", "opt": "adam", "n": 1_000_000_000, "offset": 0},
        # SGD with momentum on the second of two parameter groups of one flat buffer: a slice at an odd element.
        {"name": "step_flat_sgd_group", "kind": "step_flat", "opt": "sgd", "n": 11_689_511, "offset": 1},
        # Listing 1 on a module: K differentiable MetaAdam steps on few-shot regression, then the meta-gradient.
        {"name": "meta_adam_mlp_k5", "kind": "meta", "opt": "adam", "width": 40, "K": 5, "shots": 10},
        # Zero-order gradient of a small policy network, the noise drawn by the caller, f(theta) as the baseline.
        {"name": "es_noise_mlp", "kind": "es", "n": 1761, "samples": 256, "method": "baseline", "noise": "caller"},
        # Zero-order gradient of a conv-net, antithetic, the noise generated in the kernels; an odd row length.
        {"name": "es_convnet", "kind": "es", "n": 112_261, "samples": 64, "method": "antithetic", "noise": "kernel"},
        # The same at image-network size.
        {"name": "es_resnet18", "kind": "es", "n": 11_689_512, "samples": 64, "method": "antithetic", "noise": "kernel"},
        # Flatten and unflatten of a bf16 parameter tree (a checkpoint or a broadcast buffer).
        {"name": "copy_resnet18_bf16", "kind": "copy", "tree": "resnet18", "layout": "separate", "dtype": "bfloat16"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_tree(rng, most):
    """A random tree of at most `most` elements in all (expected size kept well below)."""
    pick = rng.random()
    if pick < 0.25:
        return {"tree": rng.choice(["mlp", "convnet", "convnet32", "resnet18"])}
    leaves = _log(rng, 2, 20000)
    top = max(4.0, min(65536.0, 4.0 * most / leaves))
    return {"tree": "loguniform", "leaves": leaves, "max_leaf": _log(rng, 4, top), "tree_seed": rng.randrange(1 << 20)}


def draw(rng):
    kind = rng.choice(["step_flat", "step_tree", "unroll_pack", "unroll_tree", "meta", "es", "es", "copy"])
    case = {"kind": kind}
    if kind == "step_flat":
        case.update(opt=rng.choice(["adam", "sgd", "rmsprop"]), n=_log(rng, 1000, 5e8), offset=rng.choice([0, 0, 0, 1, 2, 3]))
    elif kind == "step_tree":
        case.update(opt=rng.choice(["adam", "sgd", "rmsprop"]), layout=rng.choice(["separate", "separate", "packed"]), **_draw_tree(rng, 1.2e8))
    elif kind in ("unroll_pack", "unroll_tree"):
        K = rng.randint(1, 12)
        case.update(K=K, warm=rng.random() < 0.3, layout=rng.choice(["separate", "separate", "packed"]), **_draw_tree(rng, 1.2e8 * 3 / max(K, 3)))
    elif kind == "meta":
        case.update(opt=rng.choice(["adam", "sgd", "rmsprop"]), width=_log(rng, 8, 512), K=rng.randint(1, 6), shots=_log(rng, 5, 100))
    elif kind == "es":
        n = _log(rng, 1000, 1.2e7)
        case.update(n=n, samples=_log(rng, 8, max(9.0, min(512.0, 7e8 / n))), method=rng.choice(["plain", "baseline", "antithetic", "antithetic"]),
                    noise=rng.choice(["kernel", "kernel", "caller"]))
    else:
        case.update(layout=rng.choice(["separate", "packed"]), dtype=rng.choice(["float32", "bfloat16", "uint8"]))
        tree = _draw_tree(rng, 3e7)
        if "leaves" in tree:
            tree["leaves"] = min(tree["leaves"], 4096)
        case.update(tree)
    return case


# ---- optimizer steps --------------------------------------------------------

_RMS = dict(lr=1e-2, alpha=0.99, eps=1e-8, eps_root=1e-8, momentum=0.9)
_SGD = dict(lr=0.1, momentum=0.9, nesterov=True)
_COUNT = 100  # an interior step: warm moments

_STEP_IN = {"adam": ["p", "g", "m", "v", "dp", "dm", "dv"], "sgd": ["p", "g", "m", "dp", "dm"], "rmsprop": ["p", "g", "v", "m", "dp", "dv", "dm"]}
_STEP_OUT = {"adam": ["p1", "m1", "v1", "dg", "dm0", "dv0"], "sgd": ["p1", "m1", "dg", "dm0"], "rmsprop": ["p1", "v1", "m1", "dg", "dv0", "dm0"]}


def _step_values(opt, n, seed, offset=0):
    """Buffers of one interior step: parameters, gradients, warm state (m: first moment, trace or
    momentum buffer; v: second moment), cotangents of the step's outputs."""
    r = _Draw(seed)
    S = {"p": r(n, 0.05, offset), "g": r(n, 1e-3, offset)}
    S["m"] = r(n, 1e-4, offset).abs_()
    if opt != "sgd":
        S["v"] = r(n, 1e-4, offset).abs_()
    for k in _STEP_IN[opt]:
        if k not in S:
            S[k] = r(n, 1.0, offset)
    return S


def _run_step_flat(S):
    opt = S["opt"]
    if opt == "adam":
        h = (_COUNT, HYPER["lr"], HYPER["b1"], HYPER["b2"], HYPER["eps"], 0.0)
        P.adam_fwd(S["p"], S["g"], S["m"], S["v"], *h, S["p1"], S["m1"], S["v1"])
        P.adam_bwd(S["dp"], S["dm"], S["dv"], S["g"], S["m"], S["v"], *h, None, S["dg"], S["dm0"], S["dv0"])
    elif opt == "sgd":
        h = (_SGD["lr"], _SGD["momentum"], _SGD["nesterov"])
        P.sgd_fwd(S["p"], S["g"], S["m"], *h, S["p1"], S["m1"])
        P.sgd_bwd(S["dp"], S["dm"], *h, S["dg"], S["dm0"])
    else:
        h = (_RMS["lr"], _RMS["alpha"], _RMS["eps"], _RMS["eps_root"], _RMS["momentum"])
        P.rmsprop_fwd(S["p"], S["g"], S["v"], S["m"], *h, S["p1"], S["v1"], S["m1"])
        P.rmsprop_bwd(S["dp"], S["dv"], S["dm"], S["g"], S["v"], *h, S["dg"], S["dv0"], S["dm0"])
    return [S[k] for k in _STEP_OUT[opt]]


def _run_step_tree(S):
    opt, t, a = S["opt"], S["table"], S["ptr"]
    if opt == "adam":
        h = (_COUNT, HYPER["lr"], HYPER["b1"], HYPER["b2"], HYPER["eps"], 0.0)
        P.adam_fwd_tree(t, a["p"], a["g"], a["m"], a["v"], *h, a["p1"], a["m1"], a["v1"])
        P.adam_bwd_tree(t, a["dp"], a["dm"], a["dv"], a["g"], a["m"], a["v"], *h, a["dg"], a["dm0"], a["dv0"])
    elif opt == "sgd":
        h = (_SGD["lr"], _SGD["momentum"], _SGD["nesterov"])
        P.sgd_fwd_tree(t, a["p"], a["g"], a["m"], *h, a["p1"], a["m1"])
        P.sgd_bwd_tree(t, a["dp"], a["dm"], *h, a["dg"], a["dm0"])
    else:
        h = (_RMS["lr"], _RMS["alpha"], _RMS["eps"], _RMS["eps_root"], _RMS["momentum"])
        P.rmsprop_fwd_tree(t, a["p"], a["g"], a["v"], a["m"], *h, a["p1"], a["v1"], a["m1"])
        P.rmsprop_bwd_tree(t, a["dp"], a["dv"], a["dm"], a["g"], a["v"], *h, a["dg"], a["dv0"], a["dm0"])
    return [S[k] for k in _STEP_OUT[opt]]


def _adam64(p, g, m, v, count, h, eps_root):
    """One Adam step in 64 bits: (p', m', v')."""
    c1, c2 = -math.expm1((count + 1) * math.log(h["b1"])), -math.expm1((count + 1) * math.log(h["b2"]))
    m1 = h["b1"] * m + (1 - h["b1"]) * g
    v1 = h["b2"] * v + (1 - h["b2"]) * g * g
    d = (v1 / c2 + eps_root).sqrt_().add_(h["eps"])
    return p - (h["lr"] / c1) * m1 / d, m1, v1


def _adam64_vjp(dp, dm, dv, g, m, v, count, h, eps_root):
    """Chain rule through _adam64 in 64 bits: cotangents of (g, m, v)."""
    c1, c2 = -math.expm1((count + 1) * math.log(h["b1"])), -math.expm1((count + 1) * math.log(h["b2"]))
    m1 = h["b1"] * m + (1 - h["b1"]) * g
    s = ((h["b2"] * v + (1 - h["b2"]) * g * g) / c2 + eps_root).sqrt_()
    d = s + h["eps"]
    still = s == 0  # 0/0: the mean of the two one-sided derivatives in g, 0 in v
    dm1 = dm - dp * (h["lr"] / c1) / d
    dv1 = dv + torch.where(still, torch.zeros_like(s), dp * (h["lr"] / c1) * m1 / (d * d) / (2 * c2 * s))
    return (1 - h["b1"]) * dm1 + 2 * (1 - h["b2"]) * g * dv1, h["b1"] * dm1, h["b2"] * dv1


def _step64(opt, x):
    """One step and its VJP in 64 bits; x maps input names to 64-bit tensors, the answer output names."""
    if opt == "adam":
        p1, m1, v1 = _adam64(x["p"], x["g"], x["m"], x["v"], _COUNT, HYPER, 0.0)
        dg, dm0, dv0 = _adam64_vjp(x["dp"], x["dm"], x["dv"], x["g"], x["m"], x["v"], _COUNT, HYPER, 0.0)
        return {"p1": p1, "m1": m1, "v1": v1, "dg": dg, "dm0": dm0, "dv0": dv0}
    if opt == "sgd":
        lr, mu = _SGD["lr"], _SGD["momentum"]
        t1 = mu * x["m"] + x["g"]
        dt = x["dm"] - lr * mu * x["dp"]
        return {"p1": x["p"] - lr * (x["g"] + mu * t1), "m1": t1, "dg": dt - lr * x["dp"], "dm0": mu * dt}
    h = _RMS
    v1 = h["alpha"] * x["v"] + (1 - h["alpha"]) * x["g"] * x["g"]
    s = (v1 + h["eps_root"]).sqrt_()
    d = s + h["eps"]
    b1 = h["momentum"] * x["m"] + x["g"] / d
    db = x["dm"] - h["lr"] * x["dp"]
    dv1 = x["dv"] - db * x["g"] / (2 * s * d * d)
    return {"p1": x["p"] - h["lr"] * b1, "v1": v1, "m1": b1, "dg": db / d + 2 * (1 - h["alpha"]) * x["g"] * dv1, "dv0": h["alpha"] * dv1,
            "dm0": h["momentum"] * db}


def _exact_step(opt, n, values, inside=None):
    out = {k: torch.empty(n, dtype=torch.float64, device="cuda") for k in _STEP_OUT[opt]}
    chunk = 1 << 26
    for a in range(0, n, chunk):
        part = {k: values[k][a:a + chunk].double() for k in _STEP_IN[opt]}
        for k, v in _step64(opt, part).items():
            out[k][a:a + chunk] = v
    if inside is not None:
        for v in out.values():
            v[~inside] = 0.0
    return [out[k] for k in _STEP_OUT[opt]]


# ---- K unrolled steps -------------------------------------------------------


def _unroll_hyper(case):
    return (100 if case["warm"] else 0, HYPER["lr"], HYPER["b1"], HYPER["b2"], HYPER["eps"], 1e-8)


def _unroll_inputs(case, L, seed):
    r, K = _Draw(seed), case["K"]
    p = r(L.total, 0.05)
    g = [r(L.total, 1e-2) for _ in range(K)]
    flat = L.n if case["kind"] == "unroll_pack" else L.total
    state = [r(flat, 1e-4).abs_() for _ in range(2)] if case["warm"] else [_new(flat), _new(flat)]
    return p, g, state, r(flat, 1.0)


def _prepare_unroll(case, seed):
    K, L = case["K"], _Layout(_sizes(case), case["layout"])
    p, g, state, cot = _unroll_inputs(case, L, seed)
    table, keep = P.segtable_create(L.numel), _stored(K)
    S = dict(kind=case["kind"], K=K, table=table, hyper=_unroll_hyper(case))
    if case["kind"] == "unroll_tree":
        traj = [[state[i]] + [_new(L.total) if k in keep else None for k in range(1, K + 1)] for i in range(2)]
        pK, dg, dm, dv = _new(L.total), [_new(L.total) for _ in range(K)], _new(L.total), _new(L.total)
        S.update(p=L.ptrs(p), g=[L.ptrs(x) for x in g], mu=[None if x is None else L.ptrs(x) for x in traj[0]],
                 nu=[None if x is None else L.ptrs(x) for x in traj[1]], pK=L.ptrs(pK), cot=L.ptrs(cot), dg=[L.ptrs(x) for x in dg], dm=L.ptrs(dm), dv=L.ptrs(dv),
                 out=[pK, traj[0][K], traj[1][K], dm, dv, *dg], own=(p, g, state, cot, traj))
    else:
        traj = [[state[i]] + [_new(L.n) if k in keep else None for k in range(1, K + 1)] for i in range(2)]
        pK, dg = _new(L.total), [_new(L.total) for _ in range(K)]
        S.update(p=L.ptrs(p), g=[L.ptrs(x) for x in g], pK=L.ptrs(pK), dg=[L.ptrs(x) for x in dg], flat_p=_new(L.n), flat_g=[_new(L.n) for _ in range(K)],
                 mu=traj[0], nu=traj[1], flat_pK=_new(L.n), cot=cot, flat_dg=[_new(L.n) for _ in range(K)], dm=_new(L.n), dv=_new(L.n), own=(p, g))
        S["out"] = [pK, S["mu"][K], S["nu"][K], S["dm"], S["dv"], *dg]
    return S


def _run_unroll(S):
    h = S["hyper"]
    if S["kind"] == "unroll_tree":
        P.adam_unrolled_fwd_tree(S["table"], S["p"], S["g"], S["mu"], S["nu"], S["pK"], *h)
        P.adam_unrolled_bwd_tree(S["table"], S["cot"], S["g"], S["mu"], S["nu"], S["dg"], S["dm"], S["dv"], *h)
    else:
        P.tree_flatten_batch(S["table"], [S["p"]] + S["g"], [S["flat_p"]] + S["flat_g"])
        P.adam_unrolled_fwd(S["flat_p"], S["flat_g"], S["mu"], S["nu"], S["flat_pK"], *h)
        P.adam_unrolled_bwd(S["cot"], S["flat_g"], S["mu"], S["nu"], S["flat_dg"], S["dm"], S["dv"], *h)
        P.tree_unflatten_batch(S["table"], [S["flat_pK"]] + S["flat_dg"], [S["pK"]] + S["dg"])
    return S["out"]


def _exact_unroll(case, seed):
    K, L = case["K"], _Layout(_sizes(case), case["layout"])
    p, g, state, cot = _unroll_inputs(case, L, seed)
    inside = L.inside()
    flat = case["kind"] == "unroll_pack"
    if flat:
        p, g = p[inside], [x[inside] for x in g]
    h, count = HYPER, 100 if case["warm"] else 0
    x, m, v = p.double(), state[0].double(), state[1].double()
    kept = []
    for k in range(K):
        kept.append((m, v))
        x, m, v = _adam64(x, g[k].double(), m, v, count + k, h, 1e-8)
    dm, dv, dg, dp = torch.zeros_like(m), torch.zeros_like(v), [None] * K, cot.double()
    for k in range(K - 1, -1, -1):
        dg[k], dm, dv = _adam64_vjp(dp, dm, dv, g[k].double(), *kept[k], count + k, h, 1e-8)
        kept[k] = None
    trees, states = [x, *dg], [m, v, dm, dv]
    if flat:
        spread = []
        for t in trees:
            out = torch.zeros(L.total, dtype=torch.float64, device="cuda")
            out[inside] = t
            spread.append(out)
        trees = spread
    else:
        for t in trees + states:
            t[~inside] = 0.0
    return [trees[0], *states, *trees[1:]]


# ---- Listing 1 on a module --------------------------------------------------


class _Net(torch.nn.Module):
    def __init__(self, params):
        super().__init__()
        for name, p in params.items():
            self.register_parameter(name, torch.nn.Parameter(p))

    def forward(self, x):
        return _net(self._parameters, x)


def _net(w, x):
    x = torch.tanh(torch.nn.functional.linear(x, w["w1"], w["b1"]))
    x = torch.tanh(torch.nn.functional.linear(x, w["w2"], w["b2"]))
    return torch.nn.functional.linear(x, w["w3"], w["b3"])


def _loss(y, t):
    return ((y - t) ** 2).mean()


_META = {"adam": dict(lr=1e-3, b1=0.9, b2=0.999, eps=1e-8, eps_root=1e-8), "sgd": dict(lr=1e-2, momentum=0.9, nesterov=True),
         "rmsprop": dict(lr=1e-3, alpha=0.99, eps=1e-8, eps_root=1e-8, momentum=0.9)}


def _meta_inputs(case, seed):
    r, w = _Draw(seed), case["width"]
    params = {"w1": r(w, 1.0).view(w, 1), "b1": r(w, 0.1), "w2": r(w * w, w ** -0.5).view(w, w), "b2": r(w, 0.1), "w3": r(w, w ** -0.5).view(1, w), "b3": r(1, 0.1)}
    x = [r(case["shots"], 2.0).view(-1, 1) for _ in range(2)]  # support and query inputs of one task
    amp, phase = r(1, 1.0) + 2.0, r(1, 1.0)
    return params, x, [amp * torch.sin(t + phase) for t in x]


def _run_meta(S):
    net, meta = S["net"], S["meta"]
    for name, p in meta.items():  # the task starts from the meta parameters
        net._parameters[name] = p
    opt = {"adam": P.MetaAdam, "sgd": P.MetaSGD, "rmsprop": P.MetaRMSProp}[S["opt"]](net, **_META[S["opt"]])
    for _ in range(S["K"]):
        opt.step(_loss(net(S["x"][0]), S["y"][0]))
    outer = _loss(net(S["x"][1]), S["y"][1])
    grads = torch.autograd.grad(outer, list(meta.values()))
    return [outer.detach(), *grads, *(p.detach() for p in net._parameters.values())]


def _exact_meta(case, seed):
    params, x, y = _meta_inputs(case, seed)
    x, y = [t.double() for t in x], [t.double() for t in y]
    meta = {k: v.double().requires_grad_() for k, v in params.items()}
    w, h, opt = dict(meta), _META[case["opt"]], case["opt"]
    m, v = ({k: torch.zeros_like(t, requires_grad=False) for k, t in meta.items()} for _ in range(2))
    for step in range(case["K"]):
        grads = dict(zip(w, torch.autograd.grad(_loss(_net(w, x[0]), y[0]), list(w.values()), create_graph=True)))
        for k, g in grads.items():
            if opt == "adam":
                c1, c2 = 1 - h["b1"] ** (step + 1), 1 - h["b2"] ** (step + 1)
                m[k] = h["b1"] * m[k] + (1 - h["b1"]) * g
                v[k] = h["b2"] * v[k] + (1 - h["b2"]) * g * g
                w[k] = w[k] - h["lr"] * (m[k] / c1) / ((v[k] / c2 + h["eps_root"]).sqrt() + h["eps"])
            elif opt == "sgd":
                m[k] = h["momentum"] * m[k] + g
                w[k] = w[k] - h["lr"] * (g + h["momentum"] * m[k])
            else:
                v[k] = h["alpha"] * v[k] + (1 - h["alpha"]) * g * g
                m[k] = h["momentum"] * m[k] + g / ((v[k] + h["eps_root"]).sqrt() + h["eps"])
                w[k] = w[k] - h["lr"] * m[k]
    outer = _loss(_net(w, x[1]), y[1])
    grads = torch.autograd.grad(outer, list(meta.values()))
    return [outer.detach(), *grads, *(t.detach() for t in w.values())]


# ---- zero-order estimation --------------------------------------------------

_SIGMA = 0.02


def _es_rows(case):
    return (2 if case["method"] == "antithetic" else 1) * case["samples"]


def _es_inputs(case, seed):
    r = _Draw(seed)
    theta = r(case["n"], 0.05)
    f0 = r(1, 0.1) + 1.0
    fvals = r(_es_rows(case), 0.1) + f0  # the caller's evaluations at the perturbed points
    noise = r(case["samples"] * case["n"], 1.0).view(case["samples"], case["n"]) if case["noise"] == "caller" else None
    return theta, f0, fvals, noise


def _prepare_es(case, seed):
    theta, f0, fvals, noise = _es_inputs(case, seed)
    return dict(case, seed=seed + 1, theta=theta, f0=f0, fvals=fvals, noise_rows=noise, points=_new(_es_rows(case) * case["n"]).view(_es_rows(case), -1),
                weights=_new(case["samples"]), grad=_new(case["n"]))


def _run_es(S):
    N, method = S["samples"], S["method"]
    f0 = S["f0"] if method == "baseline" else None
    if S["noise"] == "kernel":
        P.es_perturb_gaussian(S["theta"], N, S["seed"], _SIGMA, method == "antithetic", S["points"])
        P.es_estimate_gaussian(S["fvals"], method, N, S["seed"], _SIGMA, S["grad"], f0=f0)
    else:
        P.es_perturb(S["theta"], S["noise_rows"], _SIGMA, method == "antithetic", S["points"])
        P.es_weights(S["fvals"], method, N, _SIGMA, S["weights"], f0=f0)
        P.es_estimate(S["noise_rows"], S["weights"], 1.0, S["grad"])
    return [S["points"], S["grad"]]


_LOW = 0xFFFFFFFF


def _signed(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _mul128(c, const):
    """(low, high) 64-bit halves of c times a 64-bit constant, c a tensor of 64-bit patterns."""
    cl, ch, ml, mh = c & _LOW, (c >> 32) & _LOW, const & _LOW, const >> 32
    t0 = cl * ml
    t1 = ch * ml + ((t0 >> 32) & _LOW)
    t2 = cl * mh + (t1 & _LOW)
    return (t2 << 32) | (t0 & _LOW), ch * mh + ((t1 >> 32) & _LOW) + ((t2 >> 32) & _LOW)


def _philox_normals(sample, n, seed):
    """The n standard normals of one sample in 64 bits: Philox-4x64-10 blocks (block, sample, 0, 0) under the key
    (seed, 0), Box-Muller on each 64-bit word; parameter j = 512 s + 256 h + 4 l + e takes block 64 s + l, word
    2 h + e // 2, the cosine normal for even e."""
    segs = -(-n // 512)
    block = torch.arange(64 * segs, dtype=torch.int64, device="cuda")
    c = [block, torch.full_like(block, sample), torch.zeros_like(block), torch.zeros_like(block)]
    k0, k1, mask = seed & (2 ** 64 - 1), 0, 2 ** 64 - 1
    for _ in range(10):
        lo0, hi0 = _mul128(c[0], 0xD2E7470EE14C6C93)
        lo1, hi1 = _mul128(c[2], 0xCA5A826395121157)
        c = [hi1 ^ c[1] ^ _signed(k0), lo1, hi0 ^ c[3] ^ _signed(k1), lo0]
        k0, k1 = (k0 + 0x9E3779B97F4A7C15) & mask, (k1 + 0xBB67AE8584CAA73B) & mask
    z = torch.empty(segs, 2, 64, 4, dtype=torch.float64, device="cuda")
    for w in range(4):
        u1 = (((c[w] & _LOW) >> 8) + 1).double() * 2.0 ** -24
        u2 = (((c[w] >> 32) & _LOW) >> 8).double() * 2.0 ** -24
        r = (-2.0 * u1.log()).sqrt()
        z[:, w // 2, :, 2 * (w % 2)] = (r * torch.cos(2 * math.pi * u2)).view(segs, 64)
        z[:, w // 2, :, 2 * (w % 2) + 1] = (r * torch.sin(2 * math.pi * u2)).view(segs, 64)
    return z.view(-1)[:n]


def _exact_es(case, seed):
    theta, f0, fvals, noise = _es_inputs(case, seed)
    N, n, anti = case["samples"], case["n"], case["method"] == "antithetic"
    theta, f = theta.double(), fvals.double()
    w = f[:N] - f[N:] if anti else (f - f0.double() if case["method"] == "baseline" else f)
    w = w / ((2 if anti else 1) * N * _SIGMA)
    points = torch.empty(_es_rows(case), n, dtype=torch.float64, device="cuda")
    grad = torch.zeros(n, dtype=torch.float64, device="cuda")
    for i in range(N):
        z = _philox_normals(i, n, seed + 1) if noise is None else noise[i].double()
        points[i] = theta + _SIGMA * z
        if anti:
            points[N + i] = theta - _SIGMA * z
        grad += w[i] * z
    return [points, grad]


# ---- tree copies ------------------------------------------------------------


def _prepare_copy(case, seed):
    dtype = getattr(torch, case["dtype"])
    L = _Layout(_sizes(case), case["layout"], torch.empty((), dtype=dtype).element_size())
    arena = _Draw(seed)(L.total, 1.0)
    arena = (arena * 40 + 128).clamp_(0, 255).to(dtype) if dtype == torch.uint8 else arena.to(dtype)
    back = torch.zeros_like(arena)
    cut = [(int(a), int(a) + k) for a, k in zip(L.start, L.numel)]
    return dict(tree={"leaf%05d" % i: arena[a:b] for i, (a, b) in enumerate(cut)}, leaves=[back[a:b] for a, b in cut], back=back)


def _run_copy(S):
    flat, spec = P.tree.flatten(S["tree"])
    P.tree.unflatten(flat, spec, out_leaves=S["leaves"])
    return [flat, S["back"]]


# ---- the interface ----------------------------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step_flat":
        S = _step_values(case["opt"], case["n"], seed, case["offset"])
        for k in _STEP_OUT[case["opt"]]:
            S[k] = _new(case["n"], case["offset"])
        return dict(S, kind=kind, opt=case["opt"])
    if kind == "step_tree":
        L = _Layout(_sizes(case), case["layout"])
        S = _step_values(case["opt"], L.total, seed)
        for k in _STEP_OUT[case["opt"]]:
            S[k] = _new(L.total)
        return dict(S, kind=kind, opt=case["opt"], table=P.segtable_create(L.numel), ptr={k: L.ptrs(x) for k, x in S.items()})
    if kind in ("unroll_pack", "unroll_tree"):
        return _prepare_unroll(case, seed)
    if kind == "meta":
        params, x, y = _meta_inputs(case, seed)
        net = _Net(params)
        return dict(kind=kind, opt=case["opt"], K=case["K"], net=net, meta=dict(net._parameters), x=x, y=y)
    if kind == "es":
        return _prepare_es(case, seed)
    return dict(_prepare_copy(case, seed), kind=kind)


def run(state):
    kind = state["kind"]
    if kind == "step_flat":
        return _run_step_flat(state)
    if kind == "step_tree":
        return _run_step_tree(state)
    if kind in ("unroll_pack", "unroll_tree"):
        return _run_unroll(state)
    if kind == "meta":
        return _run_meta(state)
    if kind == "es":
        return _run_es(state)
    return _run_copy(state)


def work(case):
    """Bytes and operations of the calls of one pass: every operand of a call read once, every result written once."""
    kind = case["kind"]
    if kind in ("step_flat", "step_tree"):
        n = case["n"] if kind == "step_flat" else sum(_sizes(case))
        values, flops = {"adam": (16, 45), "sgd": (9, 8), "rmsprop": (15, 40)}[case["opt"]]
        return {"bytes": 4 * values * n, "flops": flops * n}
    if kind in ("unroll_pack", "unroll_tree"):
        n, K = sum(_sizes(case)), case["K"]
        kept = len(_stored(K))
        fwd = 3 + K + 2 * kept + 1  # p, m, v and the gradients; the kept states, p_K
        bwd = 1 + 2 * kept + K + K + 2  # the cotangent, the kept states before the last and the first, gradients; their cotangents, dm, dv
        copies = 4 * (K + 1) if kind == "unroll_pack" else 0
        return {"bytes": 4 * n * (fwd + bwd + copies), "flops": 45 * n * K}
    if kind == "meta":
        w, K = case["width"], case["K"]
        n = w * w + 4 * w + 1
        return {"bytes": 4 * n * (16 * K + 2), "flops": K * (45 * n + 2 * 12 * n * case["shots"])}
    if kind == "es":
        n, N = case["n"], case["samples"]
        noise = 0 if case["noise"] == "kernel" else 2 * N * n
        return {"bytes": 4 * (2 * n + _es_rows(case) * n + noise), "flops": n * N * (4 if case["noise"] == "caller" else 100)}
    elem = {"float32": 4, "bfloat16": 2, "uint8": 1}[case["dtype"]]
    return {"bytes": 4 * elem * sum(_sizes(case)), "flops": 0}


def tolerance(case):
    """About four times what the paths show against exact() over draws of every kind: 2e-7 to 3e-7 (largest single value
    7e-6) for the steps and the estimator, 1.3e-5 (1.5e-4) for the meta-gradient, whose update divides by |g| and so
    amplifies the rounding of the model's own gradients."""
    if case["kind"] == "copy":
        return "exact"
    if case["kind"] == "meta":
        return {"rel": 6e-5, "max": 1e-3}
    return {"rel": 1.5e-6, "max": 5e-5}


def exact(case, seed):
    kind = case["kind"]
    if kind == "step_flat":
        return _exact_step(case["opt"], case["n"], _step_values(case["opt"], case["n"], seed, case["offset"]))
    if kind == "step_tree":
        L = _Layout(_sizes(case), case["layout"])
        return _exact_step(case["opt"], L.total, _step_values(case["opt"], L.total, seed), L.inside())
    if kind in ("unroll_pack", "unroll_tree"):
        return _exact_unroll(case, seed)
    if kind == "meta":
        return _exact_meta(case, seed)
    if kind == "es":
        return _exact_es(case, seed)
    return None
