"""hap_exemplars: the copied labels and the count of distinct ones at the edges of the count kernel's words of
32 points and strides of 1024, for the whole problem and for a row block; the preferences of every level."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [2, 31, 32, 33, 1023, 1024, 1025, 5000])
def test_labels_count_and_preferences(hap_gpu, n):
    rng = np.random.default_rng(n)
    X = torch.from_numpy((rng.standard_normal((n, 2)) + 9 * rng.integers(0, 6, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap_gpu.build_similarity(X, S)
    pref = torch.from_numpy(rng.uniform(-30.0, -1.0, (3, n)).astype(np.float32)).to(DEV)
    h = hap_gpu.Hap(S, 3, 0.5, pref=pref)
    assert h.preference() == [float(v) for v in pref[:, 0]]
    h.iterate(0)
    h.iterate(4)
    for rows in (n, max(1, n // 2)):
        h.set_row_count(rows)
        for level in range(3):
            out = torch.full((n + 1,), -7, dtype=torch.int32, device=DEV)
            e, k = h.exemplars(level, out=out)
            assert int(out[n]) == -7
            assert k == len(torch.unique(e[:rows]))
            assert (e[:n] >= 0).all() and (e[:n] < n).all()
