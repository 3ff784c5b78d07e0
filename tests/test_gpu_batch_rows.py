"""The batched form's row groups at the edges of a wave's and a group's columns: every problem against the
single-problem path with one row per workgroup (the same row-ordered column sums), labels equal."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SIZES = [2, 3, 63, 64, 65, 255, 256, 257, 700, 1023, 1024, 1025, 1500, 2047, 2048]


@pytest.mark.parametrize("shape", [(512, 64, 4), (1024, 64, 4), (512, 64, 2), (256, 64, 1)])
@pytest.mark.parametrize("split", [0, 512])
def test_rows_match_the_single_problem_path(hap_gpu, shape, split):
    hap = hap_gpu
    d, levels, lam, iters = 3, 2, 0.6, 7
    rng = np.random.default_rng(3)
    xs = [(rng.standard_normal((n, d)) * 2 + 12 * rng.integers(0, 5, (n, 1))).astype(np.float32) for n in SIZES]
    X = torch.from_numpy(np.concatenate(xs)).to(DEV)
    bt = hap.HapBatch(SIZES, d, levels)
    bt.set_launch(*shape)
    bt.set_split(split, 4)
    labels, ns, its = bt.run(X, lam, iters)
    torch.cuda.synchronize()
    assert (its.cpu() == iters).all()
    members, rows = bt.members()
    for b, x in enumerate(xs):
        n = len(x)
        S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
        hap.build_similarity(torch.from_numpy(x).to(DEV), S)
        h = hap.Hap(S, levels, lam)
        h.set_launch(rows_per_block=1 if members[b] == 1 else rows[b], blocks=True)
        h.iterate(iters)
        assert torch.equal(h.labels(), bt.labels_of(labels, b)), n
        total = h.net_similarity(-1)
        assert abs(float(ns[b, levels]) - total) <= 1e-12 * abs(total)
        h.close()
