"""Rows of 256 threads on both sides of the rules that choose their pass: cached and non-temporal accesses (a state
within the Infinity Cache or past it, few and many rows per workgroup), and two rows per workgroup in flight or one
at a time; against the streaming pass with the same rows per workgroup, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def compare(hap, n, levels, rb, form, unfused):
    rng = np.random.default_rng([n, rb])
    X = torch.from_numpy((rng.standard_normal((n, 2)) * 3 + 20 * rng.integers(0, 4, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    kw = dict(schedule=hap.SCHEDULE_MRHAP) if form == "mrhap" else dict(kappa=0.5) if form == "kappa" else {}
    with hap.Hap(S, levels, 0.6, **kw) as a, hap.Hap(S, levels, 0.6, **kw) as b:
        a.set_launch(256, 4, rb, unfused=unfused)
        if form == "points":
            a.set_points(X)
        assert bool(a.launch_flags() & hap.LAUNCH_FUSED) == (form == "mrhap" and not unfused)
        b.set_launch(1024, 1, rb, streaming=True, unfused=True)
        for h in (a, b):
            h.iterate(5)
        for level in range(levels):
            x, y = a.messages(level), b.messages(level)
            for k in x:
                assert torch.equal(x[k], y[k]), (level, k)
        assert torch.equal(a.labels(), b.labels())


@pytest.mark.parametrize("form", ["plain", "mrhap", "kappa", "points"])
@pytest.mark.parametrize("n,levels,rb", [(2600, 4, 4), (2752, 4, 4), (2752, 4, 5), (4096, 1, 3), (4095, 2, 3), (2750, 2, 2),
                                         (2751, 2, 2)])
def test_per_level_pass(hap_gpu, n, levels, rb, form):
    compare(hap_gpu, n, levels, rb, form, True)


@pytest.mark.parametrize("n,levels,rb", [(4096, 2, 16), (4095, 3, 16), (3050, 4, 4), (3062, 4, 4), (3250, 2, 2), (3251, 2, 2)])
def test_all_level_pass(hap_gpu, n, levels, rb):
    compare(hap_gpu, n, levels, rb, "mrhap", False)
