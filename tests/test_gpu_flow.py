"""The row pass with several rows of a workgroup in flight (FP32, four chunks per thread, two to 64 rows
per workgroup) against the streaming pass with the same rows per workgroup, bit for bit: messages of every
level at the edges of its rows (one to eight waves per row, one and several rows per group, the last
vector and the last chunk ragged, a single point more or less than they hold)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# n, threads per row, rows per workgroup
SHAPES = [(3, 64, 2), (257, 64, 4), (258, 64, 5), (1023, 64, 64), (1024, 64, 3), (1025, 128, 8), (2047, 128, 9),
          (2049, 256, 7), (4095, 256, 64), (4097, 512, 33)]


def run(hap, S, X, shape, iters, lam, pref, **kw):
    h = hap.Hap(S, 3 if S.shape[0] < 2000 else 2, lam, pref=pref, **{k: v for k, v in kw.items() if k != "blocks"})
    h.set_launch(*shape[:3], streaming=shape[3], blocks=kw.get("blocks", False), unfused=True)
    if X is not None:
        h.set_points(X)
    h.iterate(iters)
    got = [h.messages(level) for level in range(h.levels)] + [dict(labels=h.labels())]
    h.close()
    return got


@pytest.mark.parametrize("n,threads,rb", SHAPES)
@pytest.mark.parametrize("form", ["plain", "blocks", "lam0", "mrhap", "kappa", "points2", "points3", "forbidden"])
def test_equals_the_streaming_pass(hap_gpu, n, threads, rb, form):
    hap = hap_gpu
    d = 3 if form == "points3" else 2
    rng = np.random.default_rng([n, rb])
    X = torch.from_numpy((rng.standard_normal((n, d)) * 3 + 20 * rng.integers(0, 4, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    pref = None
    if form == "forbidden":
        # similarities of minus infinity, as for pairs that may not join
        S[torch.rand((n, n), device=DEV, generator=torch.Generator(DEV).manual_seed(n)) < 0.3] = -float("inf")
        pref = -50.0
    kw = dict(blocks=form == "blocks")
    if form == "mrhap":
        kw["schedule"] = hap.SCHEDULE_MRHAP
    if form == "kappa":
        kw["kappa"] = 0.5
    lam = 0.0 if form == "lam0" else 0.6
    pts = X if form.startswith("points") else None
    a = run(hap, S, pts, (threads, 4, rb, False), 5, lam, pref, **kw)
    b = run(hap, S, None, (1024, (n + 4095) // 4096, rb, True), 5, lam, pref, **kw)
    for x, y in zip(a, b):
        for k in x:
            assert torch.equal(torch.nan_to_num(x[k], nan=7e30), torch.nan_to_num(y[k], nan=7e30)), (form, k)


@pytest.mark.parametrize("n,threads,rb", [s for s in SHAPES if s[1] < 512] + [(2, 64, 1), (255, 64, 1), (300, 64, 1), (513, 128, 1), (1100, 256, 1)])
@pytest.mark.parametrize("levels", [2, 4])
def test_fused_levels_equal_the_per_level_passes(hap_gpu, n, threads, rb, levels):
    """The MapReduce schedule's all-level pass with several rows in flight."""
    hap = hap_gpu
    rng = np.random.default_rng([n, rb, levels])
    X = torch.from_numpy((rng.standard_normal((n, 2)) * 3 + 20 * rng.integers(0, 4, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    got = []
    for unfused in (False, True):
        h = hap.Hap(S, levels, 0.6, schedule=hap.SCHEDULE_MRHAP)
        h.set_launch(*((threads, 4, rb) if not unfused else (1024, (n + 4095) // 4096, rb)), streaming=unfused,
                     unfused=unfused)
        assert bool(h.launch_flags() & hap.LAUNCH_FUSED) == (not unfused)
        h.iterate(5)
        got.append([h.messages(level) for level in range(levels)] + [dict(labels=h.labels())])
        h.close()
    for x, y in zip(*got):
        for k in x:
            assert torch.equal(x[k], y[k]), k


@pytest.mark.parametrize("n", [8193, 12288, 12289, 16384])
def test_held_rows_of_six_and_eight_chunks(hap_gpu, n):
    """The default pass of FP32 rows of 8192 < n <= 16384 against the streaming shape it reports."""
    hap = hap_gpu
    rng = np.random.default_rng(n)
    X = torch.from_numpy(rng.standard_normal((n, 2)).astype(np.float32) * 10).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    got = []
    for explicit in (False, True):
        h = hap.Hap(S, 2, 0.7)
        shape = h.get_launch()
        assert shape == (1024, (n + 4095) // 4096, (n + 255) // 256, True)
        if explicit:
            h.set_launch(*shape[:3], streaming=True)
        h.iterate(3)
        got.append([h.messages(level) for level in range(2)] + [dict(labels=h.labels())])
        h.close()
    for x, y in zip(*got):
        for k in x:
            assert torch.equal(x[k], y[k]), k
