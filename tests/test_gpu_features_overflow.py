"""The warm start's features of rows whose nearest values all but fill a few groups of columns, or are equal by
the hundred: more values reach the feature kernel's first bound than its list of 512 holds, once or several
times over.  Points that repeat in runs of 16 columns (rows in registers and rows read twice), few places,
and rows with fewer than 16 allowed pairs.  Tolerances as in test_gpu_features.py."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(hap, n, dtype, kind):
    dt = torch.float32 if dtype == "f32" else torch.float64
    rng = np.random.default_rng(n)
    if kind == "cyclic":      # the neighbours of a point lie in one run of 16 columns in 1024
        x = 50.0 * ((np.arange(n) // 16) % 64)[:, None] + rng.standard_normal((n, 2))
    elif kind == "drift":     # the same, nearer from run to run
        k = np.arange(n)
        x = np.stack([np.where(k % 1024 < 240, -k / n, 1e3 + rng.uniform(0, 1e3, n)), np.zeros(n)], axis=1)
    elif kind == "equal":
        x = rng.integers(0, 2, (n, 2)).astype(np.float64)
    else:
        x = rng.standard_normal((n, 2)) + 12 * rng.integers(0, 4, (n, 1))
    X = torch.from_numpy(x).to(dt).to(DEV)
    w = 4 if dtype == "f32" else 2
    S = torch.empty((n, (n + w - 1) // w * w), dtype=dt, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    if kind == "forbidden":
        S[torch.rand((n, n), device=DEV, generator=torch.Generator(DEV).manual_seed(1)) < 0.995] = -float("inf")
    return S


def reference(S, p):
    n = S.shape[0]
    a = abs(float(p))
    F = torch.empty((n, 32), dtype=torch.float64, device=DEV)
    D = torch.empty((n, 6), dtype=torch.float64, device=DEV)
    near = torch.empty((n, 16), dtype=torch.int64, device=DEV)
    for r in range(0, n, 2048):
        i = torch.arange(r, min(n, r + 2048), device=DEV)[:, None]
        k = torch.arange(n - 1, device=DEV)[None, :]
        cols = k + (k >= i)
        off = S[r:r + 2048].gather(1, cols).double()
        top, at = torch.sort(off, dim=1, descending=True, stable=True)   # equal values keep their column order
        near[r:r + 2048] = cols.gather(1, at[:, :16])
        F[r:r + 2048, :16] = top[:, :16] / a
        cnt = (off > float(p)).sum(dim=1).double()
        F[r:r + 2048, 17] = cnt / (n - 1)
        F[r:r + 2048, 18] = off.sum(dim=1) / (n - 1) / a
        F[r:r + 2048, 19] = torch.log1p(cnt) / 10
        D[r:r + 2048] = torch.stack([(off - float(p) * 2.0 ** -m).clamp(min=0.0).sum(dim=1) for m in range(6)], dim=1) / a
    F[:, 16] = float(p) / a
    F[:, 20:26] = torch.log1p(D) / 10
    M = D[near].amax(dim=1)
    big = torch.maximum(D, M)
    F[:, 26:32] = torch.where(big > 0, (D - M) / big, torch.zeros_like(big))
    return F


@pytest.mark.parametrize("n,dtype,kind", [(8192, "f32", "cyclic"), (8001, "f64", "cyclic"), (9001, "f64", "cyclic"),
                                          (17001, "f32", "cyclic"), (17001, "f32", "drift"), (8192, "f32", "drift"),
                                          (3000, "f32", "equal"), (3001, "f64", "equal"), (17000, "f32", "equal"),
                                          (600, "f32", "forbidden"), (2001, "f64", "forbidden")])
def test_features_of_overfull_lists(hap_gpu, n, dtype, kind):
    S = problem(hap_gpu, n, dtype, kind)
    p = -1.0 if kind == "equal" else -9.0
    h = hap_gpu.Hap(S, 1, 0.5, pref=p)
    F = h.warm_features().double()
    h.close()
    ref = reference(S, p)
    exact = [*range(16), 16, 17]
    assert torch.equal(F[:, exact], ref[:, exact].float().double())
    rest = [c for c in range(32) if c not in exact]
    a, b = F[:, rest], ref[:, rest]
    fin = torch.isfinite(b)
    assert torch.equal(fin, torch.isfinite(a))
    assert ((a - b).abs()[fin] <= 1e-6 * b.abs()[fin].clamp(min=1.0)).all()


def test_the_order_of_the_points_does_not_decide_the_time(hap_gpu):
    """Points in cyclic order take no more than three times as long as points in random order (sixteen more
    reads of every row took ten times as long)."""
    times = {}
    for kind in ("blobs", "cyclic"):
        h = hap_gpu.Hap(problem(hap_gpu, 8192, "f32", kind), 1, 0.5, pref=-9.0)
        h.warm_features()
        best = float("inf")
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            h.warm_features()
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        times[kind] = best
        h.close()
    assert times["cyclic"] < 3.0 * times["blobs"], times
