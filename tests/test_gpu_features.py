"""The warm start's features at the edges of the feature kernel's forms: rows of one to sixteen vectors per
thread, rows read twice, fewer points than features, more equal values than the list of candidates holds,
forbidden pairs.  The nearest values are exact (FP32 of the FP64 quotient); counts are exact; sums and soft
counts are FP64 sums rounded once to FP32, whose order differs (1e-6)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def reference(S, p):
    n = S.shape[0]
    a = abs(float(p))
    off = S.double().clone()
    i = torch.arange(n, device=DEV)
    off[i, i] = -float("inf")
    k = min(16, n - 1)
    # stable: equal values keep their column order
    top, near = torch.sort(off, dim=1, descending=True, stable=True)
    top, near = top[:, :k], near[:, :k]
    F = torch.empty((n, 32), dtype=torch.float64, device=DEV)
    F[:, :k] = top / a
    F[:, k:16] = top[:, k - 1:k] / a
    F[:, 16] = float(p) / a
    cnt = (off > p).sum(dim=1).double()
    F[:, 17] = cnt / (n - 1)
    z = S.double().clone()
    z[i, i] = 0.0
    F[:, 18] = z.sum(dim=1) / (n - 1) / a
    F[:, 19] = torch.log1p(cnt) / 10
    D = torch.stack([(off - float(p) * 2.0 ** -m).clamp(min=0.0).sum(dim=1) for m in range(6)], dim=1) / a
    F[:, 20:26] = torch.log1p(D) / 10
    M = D[near].amax(dim=1).clamp(min=0.0)
    big = torch.maximum(D, M)
    F[:, 26:32] = torch.where(big > 0, (D - M) / big, torch.zeros_like(big))
    return F


@pytest.mark.parametrize("n,dtype,kind", [(2, "f32", "blobs"), (16, "f64", "blobs"), (18, "f32", "blobs"),
                                          (1024, "f32", "blobs"), (1025, "f64", "blobs"), (4097, "f32", "blobs"),
                                          (8193, "f32", "blobs"), (16385, "f32", "blobs"), (1500, "f32", "equal"),
                                          (1300, "f64", "equal"), (700, "f32", "forbidden")])
def test_features(hap_gpu, n, dtype, kind):
    dt = torch.float32 if dtype == "f32" else torch.float64
    rng = np.random.default_rng(n)
    if kind == "equal":       # a few places, so that rows hold hundreds of equal values
        x = rng.integers(0, 2, (n, 2)).astype(np.float64)
    else:
        x = rng.standard_normal((n, 2)) + 12 * rng.integers(0, 4, (n, 1))
    X = torch.from_numpy(x).to(dt).to(DEV)
    w = 4 if dtype == "f32" else 2
    S = torch.empty((n, (n + w - 1) // w * w), dtype=dt, device=DEV)[:, :n]
    hap_gpu.build_similarity(X, S)
    if kind == "forbidden":
        S[torch.rand((n, n), device=DEV, generator=torch.Generator(DEV).manual_seed(1)) < 0.3] = -float("inf")
    p = -1.0 if kind == "equal" else -9.0
    F = hap_gpu.Hap(S, 1, 0.5, pref=p).warm_features().double()
    ref = reference(S, p)
    exact = [*range(16), 16, 17]
    assert torch.equal(F[:, exact], ref[:, exact].float().double())
    rest = [c for c in range(32) if c not in exact]
    a, b = F[:, rest], ref[:, rest]
    fin = torch.isfinite(b)
    assert torch.equal(fin, torch.isfinite(a))
    assert ((a - b).abs()[fin] <= 1e-6 * b.abs()[fin].clamp(min=1.0)).all()
