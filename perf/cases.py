"""What a user of the library has it do, as cases to be timed.

A case is a dict of plain values.  `listed()` holds the named ones, `draw(rng)` gives others of
the same ranges, `prepare` makes what a program has in hand before the call (inputs, buffers, a
plan or a context it keeps), `run` is one pass through the public entry points, `work` the bytes
and operations a pass cannot do without, and `exact` the same outputs in 64 bits from plain torch.

Kinds of case:
  run       points on the GPU -> similarity, preference, sweeps, labels, net similarity
  batch     many small problems through one persistent launch
  features  the warm start's per-point features of a context
  train     minibatch Adam steps of the warm start's perceptron
  forward   the perceptron's predictions for every point
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1403_7394_amd import hap

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "f64": torch.float64}
BUILDS = {"direct": hap.BUILD_DIRECT, "direct_l2": hap.BUILD_DIRECT_L2, "gemm": hap.BUILD_GEMM,
          "bf16": hap.BUILD_BF16, "bf16x3": hap.BUILD_BF16X3}
SCHEDULES = {"sequential": hap.SCHEDULE_SEQUENTIAL, "mrhap": hap.SCHEDULE_MRHAP}


def _run(name, n, d, levels, dtype, damping, iters, stable, blobs, points=False, build="direct", pref="median",
         schedule="sequential", kappa=0.0, noise=0.0):
    c = dict(kind="run", n=n, d=d, levels=levels, dtype=dtype, damping=damping, iters=iters, stable=stable, blobs=blobs,
             points=points, build=build, pref=pref, schedule=schedule, kappa=kappa, noise=noise)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the parity workload: a small FP64 problem, every kernel of it a few microseconds
        _run("small_f64_300", 300, 2, 3, "f64", 0.5, 200, 0, 3, noise=1e-12),
        # a 2-D shape set of the paper's size, one level, run until its labels settle
        _run("shapes_788", 788, 2, 1, "f32", 0.9, 500, 50, 7),
        # an ordinary problem under the paper's MapReduce schedule, a size that is no power of two
        _run("mrhap_3000", 3000, 2, 3, "f32", 0.9, 100, 0, 24, schedule="mrhap"),
        # an ordinary FP64 problem with tie-break noise
        _run("f64_2500", 2500, 8, 2, "f64", 0.5, 60, 0, 16, noise=1e-12),
        # an image of 103 x 103 pixels with random preferences (Section 4 of the paper)
        _run("image_10609", 10609, 3, 3, "f32", 0.5, 30, 0, 16, build="direct_l2", pref="random"),
        # the headline workload: 8192 2-D points, three levels, 500 iterations or 50 stable
        _run("plain_8192", 8192, 2, 3, "f32", 0.9, 500, 50, 64, points=True),
        # 64-dimensional points, similarity on the matrix cores, four levels
        _run("precision_32768", 32768, 64, 4, "f32", 0.9, 30, 0, 256, build="bf16x3"),
        # the largest problem one GPU takes, one level
        _run("eval_65536", 65536, 32, 1, "f32", 0.9, 30, 0, 1024),
        # 512 independent problems of 64 to 2048 points in 16-D, one launch
        dict(name="batch_512", kind="batch", count=512, n_lo=64, n_hi=2048, d=16, levels=3, damping=0.8, iters=50,
             stable=0),
        # the warm start: features of a training problem, the training loop, the predictions
        dict(name="features_8192", kind="features", n=8192, d=2, dtype="f32", blobs=16),
        dict(name="train_4096", kind="train", rows=65536, batch=4096, n_in=32, hidden=128, n_out=3, steps=20,
             precision="bf16"),
        dict(name="forward_65536", kind="forward", rows=65536, n_in=32, hidden=128, n_out=3, precision="bf16"),
    ]


def _spread(rng, lo, hi):
    """A size between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "small", "mid", "mid", "f64", "large", "batch", "features", "train", "forward"])
    if kind == "small":
        n = _spread(rng, 48, 1100)
        dtype = rng.choice(["f32", "f64"])
        stable = rng.choice([0, 0, 20, 50])
        return _run(None, n, rng.choice([2, 3, 5, 16]), rng.randint(1, 4), dtype, rng.choice([0.5, 0.7, 0.9]),
                    rng.randint(30, 250), stable, rng.randint(2, 12), pref=rng.choice(["median", "random"]),
                    schedule=rng.choice(["sequential", "sequential", "mrhap"]), noise=1e-12 if dtype == "f64" else 0.0)
    if kind == "mid":
        n = _spread(rng, 1000, 8000)
        d = rng.choice([2, 3, 7, 16])
        levels = rng.randint(1, 4)
        schedule = rng.choice(["sequential", "sequential", "mrhap"])
        kappa = rng.choice([0.0, 0.0, 0.25, 0.5]) if schedule == "sequential" else 0.0
        points = d in (2, 3) and kappa == 0.0 and rng.random() < 0.5
        return _run(None, n, d, levels, "f32", rng.choice([0.5, 0.8, 0.9]), rng.randint(20, 120),
                    rng.choice([0, 0, 25]), rng.randint(4, 64), points=points,
                    build="direct" if points else rng.choice(["direct", "direct", "gemm"]),
                    pref=rng.choice(["median", "median", "random"]), schedule=schedule, kappa=kappa)
    if kind == "f64":
        return _run(None, _spread(rng, 600, 5000), rng.choice([2, 5, 8, 16]), rng.randint(1, 3), "f64",
                    rng.choice([0.5, 0.9]), rng.randint(10, 60), 0, rng.randint(4, 32),
                    build=rng.choice(["direct", "direct", "gemm"]), noise=1e-12)
    if kind == "large":
        n = _spread(rng, 8192, 30000)
        d = rng.choice([2, 3, 16, 64])
        points = n <= 16384 and d in (2, 3) and rng.random() < 0.5
        return _run(None, n, d, rng.randint(1, 4), "f32", rng.choice([0.5, 0.9]), rng.randint(8, 30), 0,
                    rng.randint(16, 256), points=points,
                    build="direct" if points else rng.choice(["direct", "gemm", "bf16", "bf16x3"]),
                    pref=rng.choice(["median", "median", "random"]))
    if kind == "batch":
        n_hi = rng.choice([200, 500, 1000, 2048])
        return dict(kind="batch", count=_spread(rng, 24, 320), n_lo=32, n_hi=n_hi, d=rng.choice([2, 5, 16, 32]),
                    levels=rng.randint(1, 3), damping=rng.choice([0.5, 0.8]), iters=rng.randint(10, 60),
                    stable=rng.choice([0, 0, 20]))
    if kind == "features":
        return dict(kind="features", n=_spread(rng, 500, 12000), d=rng.choice([2, 8, 32]),
                    dtype=rng.choice(["f32", "f32", "f64"]), blobs=rng.randint(3, 64))
    dims = dict(n_in=32, hidden=rng.choice([64, 96, 128, 256]), n_out=rng.randint(1, 4),
                precision=rng.choice(["bf16", "bf16", "f32"]))
    if kind == "train":
        return dict(kind="train", rows=_spread(rng, 4000, 100000), batch=_spread(rng, 250, 8192),
                    steps=rng.randint(5, 30), **dims)
    return dict(kind="forward", rows=_spread(rng, 500, 100000), **dims)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _points(case, seed):
    """Gaussian blobs; RGB pixels where the similarity is the distance between colours."""
    g = np.random.default_rng([seed, 11])
    n, d, k = case["n"], case["d"], case["blobs"]
    spread = 100.0 if d == 2 else 10.0 if d < 32 else 2.0
    if case.get("build") == "direct_l2":
        x = g.uniform(0.0, 255.0, (k, d))[g.integers(0, k, n)] + g.standard_normal((n, d)) * 12.0
        return np.clip(np.rint(x), 0.0, 255.0)
    centres = g.standard_normal((k, d)) * spread if d >= 32 else g.uniform(-spread, spread, (k, d))
    blob = g.integers(0, k, n)
    return centres[blob] + g.standard_normal((n, d)) * g.uniform(0.5, 2.0, k)[blob][:, None]


def _preferences(case, seed):
    """None (the median) or one random preference per point, in the range of the similarities."""
    if case.get("pref", "median") == "median":
        return None
    g = np.random.default_rng([seed, 13])
    lo = -1e6 if case["build"] == "direct_l2" else -100.0 * case["d"]
    return g.uniform(lo, 0.0, case["n"])


def _lead(n, dtype):
    w = 4 if dtype == "f32" else 2
    return (n + w - 1) // w * w


def _mlp_inputs(case, seed):
    g = np.random.default_rng([seed, 17])
    rows, a, h, o = case["rows"], case["n_in"], case["hidden"], case["n_out"]
    X = g.standard_normal((rows, a)).astype(np.float32) * g.uniform(0.1, 1.5, a).astype(np.float32)
    parts = []
    for fi, fo in ((a, h), (h, h), (h, o)):
        parts += [g.standard_normal(fi * fo) * math.sqrt(2.0 / fi), g.uniform(-0.05, 0.05, fo)]
    P = np.concatenate(parts).astype(np.float32)
    T = idx = None
    if case["kind"] == "train":
        T = np.tanh(X[:, :o] * 1.5 + 0.3 * g.standard_normal((rows, o))).astype(np.float32)
        idx = g.integers(0, rows, case["batch"] * case["steps"]).astype(np.int32)
    return X, T, idx, P


def _batch_inputs(case, seed):
    g = np.random.default_rng([seed, 19])
    # the sizes are the case's own (the plan is kept across inputs); the points are the seed's
    sizes = _batch_sizes(case)
    out = []
    for n in sizes:
        k = int(g.integers(4, 33))
        c = g.uniform(-10.0, 10.0, (k, case["d"]))
        out.append((c[g.integers(0, k, n)] + g.standard_normal((n, case["d"]))).astype(np.float32))
    return sizes, out


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("run", "features"):
        n, dt = case["n"], DTYPES[case["dtype"]]
        X = torch.from_numpy(_points(case, seed)).to(dt).to(DEV)
        S = torch.empty((n, _lead(n, case["dtype"])), dtype=dt, device=DEV)
        code = hap.HAP_F32 if case["dtype"] == "f32" else hap.HAP_F64
        levels = case.get("levels", 1)
        ws = torch.empty(hap.workspace_size(n, levels, code), dtype=torch.uint8, device=DEV)
        st = dict(case=case, X=X, S=S[:, :n], ws=ws)
        if kind == "run":
            p = _preferences(case, seed)
            st["pref"] = None if p is None else torch.from_numpy(p).to(dt).to(DEV)
        else:
            hap.build_similarity(X, st["S"])
            st["hap"] = hap.Hap(st["S"], 1, 0.9, workspace=ws)
        return st
    if kind == "batch":
        sizes, xs = _batch_inputs(case, seed)
        X = torch.from_numpy(np.concatenate(xs)).to(DEV)
        plan = hap.HapBatch(sizes, case["d"], case["levels"])
        return dict(case=case, X=X, plan=plan, out=plan.outputs(X.device))
    X, T, idx, P = _mlp_inputs(case, seed)
    prec = hap.HAP_BF16 if case["precision"] == "bf16" else hap.HAP_F32
    m = hap.Mlp(torch.from_numpy(P).to(DEV), case["n_in"], case["hidden"], case["n_out"], precision=prec)
    st = dict(case=case, X=torch.from_numpy(X).to(DEV), mlp=m)
    if kind == "train":
        st.update(T=torch.from_numpy(T).to(DEV), idx=torch.from_numpy(idx).to(DEV))
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "run":
        X, S = state["X"], state["S"]
        hap.build_similarity(X, S, mode=BUILDS[case["build"]], noise_rel=case["noise"], seed=1)
        with hap.Hap(S, case["levels"], case["damping"], pref=state["pref"], workspace=state["ws"],
                     schedule=SCHEDULES[case["schedule"]], kappa=case["kappa"]) as h:
            if case["points"]:
                h.set_points(X)
            res = h.iterate(case["iters"], case["stable"])
            labels, counts = [], []
            for level in range(case["levels"]):
                e, k = h.exemplars(level)
                labels.append(e)
                counts.append(k)
            return dict(labels=labels, counts=counts, iterations=res.iters, converged=res.converged,
                        preference=np.array(h.preference()), net_similarity=np.array([h.net_similarity(-1)]))
    if kind == "batch":
        labels, ns, iters = state["plan"].run(state["X"], case["damping"], case["iters"], case["stable"],
                                              out=state["out"])
        return dict(labels=labels, net_similarity=ns, iterations=iters)
    if kind == "features":
        return state["hap"].warm_features()
    if kind == "train":
        m = state["mlp"]
        loss = m.train(state["X"], state["T"], state["idx"], case["batch"], case["steps"], 1e-3)
        return dict(loss=loss, params=m.params)
    return state["mlp"].forward(state["X"])


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

ON_CHIP = 256 << 20       # messages of a problem below this need not leave the chip between sweeps


def _sweep_work(n, w, levels, iters, points):
    """Bytes and operations of the sweeps: rho and alpha of every level read and written once per
    iteration and S read once per iteration (not at all from points), unless they fit on the chip;
    about 20 operations per element, level and iteration."""
    cells = float(n) * n
    state = cells * w * (2 * levels + (0 if points else 1))
    bytes_ = 0.0 if state <= ON_CHIP else iters * (levels * 4.0 + (0.0 if points else 1.0)) * cells * w
    return bytes_, 20.0 * cells * levels * iters


def work(case):
    kind = case["kind"]
    if kind == "run":
        n, d, w = case["n"], case["d"], 4 if case["dtype"] == "f32" else 8
        # with a stop rule the run may end early: at least its stable iterations are done
        iters = case["stable"] + 1 if case["stable"] and case["levels"] == 1 else case["iters"]
        b, f = _sweep_work(n, w, case["levels"], iters, case["points"])
        return dict(bytes=b + float(n) * n * w + n * d * w + 4.0 * n * case["levels"], flops=f + 3.0 * n * n * d)
    if kind == "batch":
        sizes = _batch_sizes(case)
        b = f = 0.0
        total = sum(_state_bytes(n, case["levels"]) for n in sizes)
        iters = min(case["iters"], case["stable"] + 1) if case["stable"] else case["iters"]
        for n in sizes:
            sb, sf = _sweep_work(n, 4, case["levels"], iters, False)
            if total > ON_CHIP:
                sb = iters * (case["levels"] * 4.0 + 1.0) * n * n * 4
            b += sb + 4.0 * n * (case["d"] + case["levels"])
            f += sf + 3.0 * n * n * case["d"]
        return dict(bytes=b, flops=f)
    if kind == "features":
        n, w = case["n"], 4 if case["dtype"] == "f32" else 8
        return dict(bytes=float(n) * n * w + 4.0 * n * hap.WARM_FEATURES, flops=15.0 * n * n)
    a, h, o = case["n_in"], case["hidden"], case["n_out"]
    weights = a * h + h * h + h * o
    if kind == "train":
        return dict(bytes=case["steps"] * (4.0 * case["batch"] * (a + o + 1) + 28.0 * weights),
                    flops=case["steps"] * 6.0 * case["batch"] * weights)
    return dict(bytes=4.0 * case["rows"] * (a + o) + 4.0 * weights, flops=2.0 * case["rows"] * weights)


def _batch_sizes(case):
    gs = np.random.default_rng([23, case["count"], case["n_hi"]])
    return [int(v) for v in gs.integers(case["n_lo"], case["n_hi"] + 1, case["count"])]


def _state_bytes(n, levels):
    return 4.0 * n * n * (2 * levels + 1)


# ---------------------------------------------------------------------------
# The same outputs in 64 bits
# ---------------------------------------------------------------------------

BLOCK = 2048              # rows handled at a time


def _similarity64(X, root, dev):
    n = X.shape[0]
    X = torch.from_numpy(np.ascontiguousarray(X)).to(dev)
    S = torch.empty((n, n), dtype=torch.float64, device=dev)
    for r in range(0, n, BLOCK):
        b = torch.zeros((min(BLOCK, n - r), n), dtype=torch.float64, device=dev)
        for k in range(X.shape[1]):
            b += (X[r:r + BLOCK, k:k + 1] - X[:, k][None, :]).square_()
        S[r:r + BLOCK] = -(b.sqrt_() if root else b)
    return S


def _median64(S):
    """Mean of the two middle off-diagonal values, by bisection on counts (no sort of N^2 values)."""
    n = S.shape[0]
    k = n * (n - 1) // 2
    lo, hi = float(S.min()), 0.0

    def below(v):                       # off-diagonal values <= v
        return int((S <= v).sum()) - (n if v >= 0.0 else 0)

    for _ in range(80):
        mid = 0.5 * (lo + hi)
        if mid <= lo or mid >= hi:
            break
        if below(mid) >= k:
            hi = mid
        else:
            lo = mid
    vals = [float(torch.where(S[r:r + BLOCK] <= hi, S[r:r + BLOCK], -math.inf).max()) for r in range(0, n, BLOCK)]
    first = max(vals)
    if below(first) > k:
        return first
    nxt = math.inf
    for r in range(0, n, BLOCK):
        b = S[r:r + BLOCK]
        b = torch.where(b > first, b, math.inf)
        i = torch.arange(b.shape[0], device=S.device)
        b[i, r + i] = math.inf
        nxt = min(nxt, float(b.min()))
    return 0.5 * (first + nxt)


def _hap64(S, pref, levels, lam, iters, stable, mrhap=False, kappa=0.0):
    """Hierarchical affinity propagation in FP64 on torch tensors; returns the labels per level."""
    n, dev = S.shape[0], S.device
    S.fill_diagonal_(0.0)
    zeros = lambda: torch.zeros(n, dtype=torch.float64, device=dev)  # noqa: E731
    R = [torch.zeros_like(S) for _ in range(levels)]
    A = [torch.zeros_like(S) for _ in range(levels)]
    c = [zeros() for _ in range(levels)]
    phi = [zeros() for _ in range(levels)]
    Q = [zeros() for _ in range(levels)]
    delta = [zeros() for _ in range(levels)]
    tau = [None] * levels

    def blocks():
        for r in range(0, n, BLOCK):
            yield r, min(n, r + BLOCK)

    def sim(r0, r1, level):
        b = S[r0:r1] + delta[level][r0:r1, None] if kappa else S[r0:r1].clone()
        i = torch.arange(r0, r1, device=dev)
        b[i - r0, i] = pref[r0:r1]
        return b

    def responsibility(level):
        q = zeros()
        for r0, r1 in blocks():
            s = sim(r0, r1, level)
            y = A[level][r0:r1] + s
            m, k = y.max(dim=1)
            i = torch.arange(r0, r1, device=dev)
            y[i - r0, k] = -math.inf
            m2 = y.max(dim=1).values
            del y
            top = (-m) if tau[level] is None else torch.minimum(tau[level][r0:r1], -m)
            oth = (-m2) if tau[level] is None else torch.minimum(tau[level][r0:r1], -m2)
            new = s + top[:, None]
            new[i - r0, k] = s[i - r0, k] + oth
            rr = R[level][r0:r1]
            rr.mul_(lam).add_(new, alpha=1.0 - lam)
            pos = rr.clamp(min=0.0)
            pos[i - r0, i] = rr[i - r0, i]
            q += pos.sum(dim=0)
        Q[level] = q

    def availability(level):
        base = Q[level] if level == levels - 1 else c[level] + phi[level] + Q[level]
        for r0, r1 in blocks():
            rr = R[level][r0:r1]
            i = torch.arange(r0, r1, device=dev)
            new = (base[None, :] - rr.clamp(min=0.0)).clamp_(max=0.0)
            new[i - r0, i] = base[r0:r1] - rr[i - r0, i]
            A[level][r0:r1].mul_(lam).add_(new, alpha=1.0 - lam)

    def row_max(level, with_s):
        out = zeros()
        for r0, r1 in blocks():
            out[r0:r1] = (A[level][r0:r1] + (sim(r0, r1, level) if with_s else R[level][r0:r1])).max(dim=1).values
        return out

    def off_diagonal_max(level):
        out = zeros()
        for r0, r1 in blocks():
            b = A[level][r0:r1] + R[level][r0:r1]
            i = torch.arange(r0, r1, device=dev)
            b[i - r0, i] = -math.inf
            out[r0:r1] = b.max(dim=1).values
        return out

    def labels():
        return torch.stack([torch.cat([(A[l][r0:r1] + R[l][r0:r1]).argmax(dim=1) for r0, r1 in blocks()])
                            for l in range(levels)])

    old, same = None, 0
    for t in range(1, iters + 1):
        if mrhap:
            if t > 1:
                cn = [row_max(l, False) for l in range(levels)]
                for l in range(1, levels):
                    tau[l] = cn[l - 1] + Q[l - 1]
                c = cn
            for l in range(levels):
                responsibility(l)
            phi = [row_max(l + 1, True) for l in range(levels - 1)] + [zeros()]
            for l in range(levels):
                availability(l)
        else:
            for l in range(levels):
                responsibility(l)
                availability(l)
                if l + 1 < levels:
                    tau[l + 1] = c[l] + Q[l]
                if l > 0:
                    phi[l - 1] = row_max(l, True)
                c[l] = row_max(l, False)
                if kappa and l + 1 < levels:
                    delta[l + 1] = delta[l] + kappa * off_diagonal_max(l)
        if stable:
            new = labels()
            same = same + 1 if old is not None and bool((new == old).all()) else 0
            old = new
            if same >= stable:
                break
    return labels()


def _exact_run(case, seed):
    # about 25 passes over a matrix per level and iteration, at a few TB/s
    if 25.0 * 8 * case["n"] ** 2 * case["levels"] * case["iters"] / 3e12 > 12.0 or case["n"] > 50000:
        return None
    dev = DEV if torch.cuda.is_available() else "cpu"
    dt = np.float32 if case["dtype"] == "f32" else np.float64
    X = _points(case, seed).astype(dt).astype(np.float64)
    S = _similarity64(X, case["build"] == "direct_l2", dev)
    n = case["n"]
    # the tie-break noise (1e-12 of the value) is left out: it is below the outputs' own resolution
    p = _preferences(case, seed)
    if p is None:
        pv = torch.full((n,), _median64(S), dtype=torch.float64, device=dev)
    else:
        pv = torch.from_numpy(p.astype(dt).astype(np.float64)).to(dev)
    lab = _hap64(S, pv, case["levels"], case["damping"], case["iters"], case["stable"],
                 mrhap=case["schedule"] == "mrhap", kappa=case["kappa"])
    i = torch.arange(n, device=dev)
    ns = sum(float(torch.where(e == i, pv, S[i, e]).sum()) for e in lab)
    first = float(pv[0])
    return dict(labels=[None] * case["levels"], counts=[None] * case["levels"], iterations=None, converged=None,
                preference=np.array([first] * case["levels"]), net_similarity=np.array([ns]))


def _exact_batch(case, seed):
    sizes, xs = _batch_inputs(case, seed)
    if case["iters"] * case["levels"] * case["count"] > 12000 or case["stable"]:
        return None
    dev = DEV if torch.cuda.is_available() else "cpu"
    out = np.zeros((case["count"], case["levels"] + 1))
    for b, x in enumerate(xs):
        S = _similarity64(x.astype(np.float64), False, dev)
        n = S.shape[0]
        p = _median64(S)
        pv = torch.full((n,), p, dtype=torch.float64, device=dev)
        lab = _hap64(S, pv, case["levels"], case["damping"], case["iters"], 0)
        i = torch.arange(n, device=dev)
        for l, e in enumerate(lab):
            out[b, l] = float(torch.where(e == i, pv, S[i, e]).sum())
        out[b, -1] = out[b, :-1].sum()
    return dict(labels=None, net_similarity=torch.from_numpy(out), iterations=None)


def _exact_features(case, seed):
    dev = DEV if torch.cuda.is_available() else "cpu"
    dt = np.float32 if case["dtype"] == "f32" else np.float64
    S = _similarity64(_points(case, seed).astype(dt).astype(np.float64), False, dev)
    n = S.shape[0]
    p = _median64(S)
    a = abs(p)
    F = torch.empty((n, hap.WARM_FEATURES), dtype=torch.float64, device=dev)
    D = torch.empty((n, 6), dtype=torch.float64, device=dev)
    near = torch.empty((n, 16), dtype=torch.int64, device=dev)
    for r in range(0, n, BLOCK):
        b = S[r:r + BLOCK]
        i = torch.arange(b.shape[0], device=dev)
        off = b.clone()
        off[i, r + i] = -math.inf
        v, near[r:r + BLOCK] = off.topk(16, dim=1)
        F[r:r + BLOCK, :16] = v / a
        cnt = (off > p).sum(dim=1).double()
        F[r:r + BLOCK, 17] = cnt / (n - 1)
        F[r:r + BLOCK, 18] = b.sum(dim=1) / (n - 1) / a
        F[r:r + BLOCK, 19] = torch.log1p(cnt) / 10
        for m in range(6):
            D[r:r + BLOCK, m] = (off - p * 2.0 ** -m).clamp_(min=0.0).sum(dim=1) / a
    F[:, 16] = p / a
    F[:, 20:26] = torch.log1p(D) / 10
    top = D[near].amax(dim=1)
    big = torch.maximum(D, top)
    F[:, 26:32] = torch.where(big > 0, (D - top) / big, torch.zeros_like(big))
    return F


def _unpack(P, a, h, o):
    at, out = 0, []
    for shape in ((a, h), (h,), (h, h), (h,), (h, o), (o,)):
        k = math.prod(shape)
        out.append(P[at:at + k].reshape(shape))
        at += k
    return out


def _mlp64(P, X, case):
    W1, b1, W2, b2, W3, b3 = _unpack(P, case["n_in"], case["hidden"], case["n_out"])
    return torch.relu(torch.relu(X @ W1 + b1) @ W2 + b2) @ W3 + b3


def _exact_train(case, seed):
    X, T, idx, P = _mlp_inputs(case, seed)
    X, T = torch.from_numpy(X).double(), torch.from_numpy(T).double()
    P = torch.from_numpy(P).double().requires_grad_(True)
    m, v = torch.zeros_like(P), torch.zeros_like(P)
    losses = []
    for s in range(case["steps"]):
        rows = torch.from_numpy(idx[s * case["batch"]:(s + 1) * case["batch"]].astype(np.int64))
        loss = (_mlp64(P, X[rows], case) - T[rows]).square().mean()
        g, = torch.autograd.grad(loss, P)
        losses.append(float(loss.detach()))
        with torch.no_grad():
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            P -= 1e-3 * (m / (1 - 0.9 ** (s + 1))) / ((v / (1 - 0.999 ** (s + 1))).sqrt() + 1e-8)
    return dict(loss=torch.tensor(losses, dtype=torch.float64), params=P.detach())


def exact(case, seed):
    kind = case["kind"]
    if kind == "run":
        return _exact_run(case, seed)
    if kind == "batch":
        return _exact_batch(case, seed)
    if kind == "features":
        return _exact_features(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    X, _, _, P = _mlp_inputs(case, seed)
    with torch.no_grad():
        return _mlp64(torch.from_numpy(P).double(), torch.from_numpy(X).double(), case)
