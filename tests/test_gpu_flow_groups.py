"""The row pass with several rows in flight where a workgroup has two to four rows of 128 threads: as many groups as
rows, against the streaming pass with the same rows per workgroup, bit for bit; and the time of two rows against three."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_flow import run

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def similarity(hap, n, d=2):
    rng = np.random.default_rng(n)
    X = torch.from_numpy((rng.standard_normal((n, d)) * 3 + 20 * rng.integers(0, 4, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    return X, S


@pytest.mark.parametrize("n", [1025, 2047, 2048])
@pytest.mark.parametrize("rb", [2, 3, 4])
@pytest.mark.parametrize("form", ["plain", "blocks", "mrhap", "kappa", "points2", "points3"])
def test_equals_the_streaming_pass(hap_gpu, n, rb, form):
    hap = hap_gpu
    X, S = similarity(hap, n, 3 if form == "points3" else 2)
    kw = dict(blocks=form == "blocks")
    if form == "mrhap":
        kw["schedule"] = hap.SCHEDULE_MRHAP
    if form == "kappa":
        kw["kappa"] = 0.5
    a = run(hap, S, X if form.startswith("points") else None, (128, 4, rb, False), 5, 0.6, None, **kw)
    b = run(hap, S, None, (1024, 1, rb, True), 5, 0.6, None, **kw)
    for x, y in zip(a, b):
        for k in x:
            assert torch.equal(x[k], y[k]), (form, k)


@pytest.mark.parametrize("n,rb", [(1025, 2), (2047, 3), (2048, 2), (2045, 4)])
@pytest.mark.parametrize("levels", [2, 4])
def test_fused_levels_equal_the_per_level_passes(hap_gpu, n, rb, levels):
    hap = hap_gpu
    _, S = similarity(hap, n)
    got = []
    for unfused in (False, True):
        h = hap.Hap(S, levels, 0.6, schedule=hap.SCHEDULE_MRHAP)
        h.set_launch(*((128, 4, rb) if not unfused else (1024, 1, rb)), streaming=unfused, unfused=unfused)
        assert bool(h.launch_flags() & hap.LAUNCH_FUSED) == (not unfused)
        h.iterate(5)
        got.append([h.messages(level) for level in range(levels)] + [dict(labels=h.labels())])
        h.close()
    for x, y in zip(*got):
        for k in x:
            assert torch.equal(x[k], y[k]), k


@pytest.mark.parametrize("form", ["plain", "points", "mrhap"])
def test_two_rows_are_no_slower_than_three(hap_gpu, form):
    """Idle groups made the row pass of two-row workgroups slower than that of three-row ones by 13 to 20 %; with
    as many groups as rows it is 0.92 to 0.99 of it."""
    hap = hap_gpu
    n = 2000
    X, S = similarity(hap, n)
    row = {}
    for rb in (2, 3):
        with hap.Hap(S, 2, 0.9, pref=-50.0, schedule=hap.SCHEDULE_MRHAP if form == "mrhap" else 0) as h:
            if form == "points":
                h.set_points(X)
            h.set_launch(128, 4, rb)
            best = float("inf")
            for _ in range(12):
                h.profile(True)
                h.iterate(16)
                ms, k, _, _ = h.profile_read()
                best = min(best, ms / k)
            row[rb] = best
    assert row[2] < 1.06 * row[3], row
