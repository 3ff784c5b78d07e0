"""Per-launch timing under the MapReduce schedule's all-level pass times the launches that a run without it makes:
the same messages and stop, the column sums counted once per level, and the time of one launch for all of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def similarity(hap, n):
    rng = np.random.default_rng(n)
    X = torch.from_numpy((rng.standard_normal((n, 2)) + 12 * rng.integers(0, 4, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    return S


@pytest.mark.parametrize("n", [300, 1500])
@pytest.mark.parametrize("levels", [2, 4])
def test_timed_and_untimed_runs_agree(hap_gpu, n, levels):
    hap = hap_gpu
    S = similarity(hap, n)
    got = []
    for timed in (False, True):
        with hap.Hap(S, levels, 0.5, pref=-20.0, schedule=hap.SCHEDULE_MRHAP) as h:
            assert h.launch_flags() & hap.LAUNCH_FUSED
            h.profile(timed, every=3)
            res = h.iterate(200, 10)
            got.append((res.iters, res.converged, [h.messages(l) for l in range(levels)], h.labels()))
    (i0, c0, m0, e0), (i1, c1, m1, e1) = got
    assert (i0, c0) == (i1, c1) and torch.equal(e0, e1)
    for x, y in zip(m0, m1):
        for k in x:
            assert torch.equal(x[k], y[k]), k


def test_the_column_sums_are_timed_as_they_run(hap_gpu):
    hap = hap_gpu
    S = similarity(hap, 2000)
    per_sweep = []
    for unfused in (False, True):
        with hap.Hap(S, 4, 0.5, pref=-20.0, schedule=hap.SCHEDULE_MRHAP) as h:
            h.set_launch(unfused=unfused)
            h.iterate(5)
            h.profile(True)
            h.iterate(30)
            row_ms, row_n, col_ms, col_n = h.profile_read()
            assert (row_n, col_n) == (30 * (4 if unfused else 1), 30 * 4)
            per_sweep.append(col_ms / 30)
    # one launch against four
    assert per_sweep[0] < 0.6 * per_sweep[1], per_sweep
