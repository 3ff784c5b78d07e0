"""FP64 rows of 2048 < n < 4096: states on either side of the size up to which the row pass keeps them in
the Infinity Cache (256 MB), against the streaming pass with the same rows per workgroup, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("schedule", ["sequential", "mrhap"])
@pytest.mark.parametrize("n,levels", [(2049, 1), (3328, 1), (3329, 1), (2560, 2), (2561, 2), (4095, 1)])
def test_equals_the_streaming_pass(hap_gpu, n, levels, schedule):
    hap = hap_gpu
    rng = np.random.default_rng(n)
    X = torch.from_numpy(rng.standard_normal((n, 2)) * 3 + 20 * rng.integers(0, 4, (n, 1))).to(DEV)
    S = torch.empty((n, (n + 1) // 2 * 2), dtype=torch.float64, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    got = []
    for shape in ((512, 4, False), (1024, (n + 2047) // 2048, True)):
        h = hap.Hap(S, levels, 0.6, schedule=hap.SCHEDULE_MRHAP if schedule == "mrhap" else hap.SCHEDULE_SEQUENTIAL)
        h.set_launch(shape[0], shape[1], (n + 255) // 256, streaming=shape[2])
        h.iterate(5)
        got.append([h.messages(level) for level in range(levels)] + [dict(labels=h.labels())])
        h.close()
    for x, y in zip(*got):
        for k in x:
            assert torch.equal(torch.nan_to_num(x[k], nan=7e30), torch.nan_to_num(y[k], nan=7e30)), k
