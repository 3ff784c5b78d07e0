"""Column sums in row order (one row per workgroup) at the edges of the kernel's tiles of 256 partial rows
and 16 columns, against the oracle, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import hap_ref
from oracle import similarity as sim

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [2, 15, 17, 255, 256, 257, 511, 512, 513, 1025])
def test_row_ordered_sums_match_the_oracle(hap_gpu, n, dtype):
    rng = np.random.default_rng(n)
    X = (rng.standard_normal((n, 2)) * 2 + 15 * rng.integers(0, 3, (n, 1))).astype(dtype)
    w = 2 if dtype == np.float64 else 4
    S = torch.zeros((n, (n + w - 1) // w * w), dtype=torch.from_numpy(X).dtype, device=DEV)[:, :n]
    hap_gpu.build_similarity(torch.from_numpy(X).to(DEV), S)
    Sh = S.cpu().numpy()
    p = dtype(-20.0)
    h = hap_gpu.Hap(S, 2, 0.6, pref=float(p))
    assert h.get_launch()[2] == (1 if n <= 512 or dtype == np.float64 else (n + 255) // 256)
    h.set_launch(rows_per_block=1)
    h.iterate(5)
    ref = hap_ref.hap(Sh, np.full(n, p, dtype=dtype), 2, 0.6, 5, dtype=dtype)
    for level in range(2):
        got = h.messages(level)
        assert np.array_equal(got["rho"].cpu().numpy(), ref.state.rho[level])
        assert np.array_equal(got["alpha"].cpu().numpy(), ref.state.alpha[level])
        assert np.array_equal(got["tau"].cpu().numpy(), ref.state.tau[level])
