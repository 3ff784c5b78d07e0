"""The second maximum of alpha + s beside columns that compare with nothing: padding that holds NaN or infinity, damping 0
(which makes NaN of the padding's alpha), and NaN similarities; the ragged end in the first and in later chunks of a
thread.  Messages against the FP32 oracle bit for bit (one row per workgroup), every form with rows in flight
against the streaming pass, and the batched form's labels against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import hap_ref
from oracle import similarity as sim

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FILLS = [0.0, float("nan"), float("inf")]


def problem(hap, n, fill):
    rng = np.random.default_rng(n)
    X = torch.from_numpy((rng.standard_normal((n, 2)) * 3 + 15 * rng.integers(0, 6, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.full((n, (n + 3) // 4 * 4), fill, dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    return X, S


@pytest.mark.parametrize("fill", FILLS)
@pytest.mark.parametrize("lam", [0.0, 0.5])
@pytest.mark.parametrize("n", [5, 49, 50, 51, 65, 201, 257])
def test_one_row_per_workgroup_equals_the_oracle(hap_gpu, n, lam, fill):
    _, S = problem(hap_gpu, n, fill)
    Sn = S.cpu().numpy().copy()
    for T in (2, 5):
        r = hap_ref.hap(Sn, -30.0, 2, lam, T, dtype=np.float32)
        with hap_gpu.Hap(S, 2, lam, pref=-30.0) as h:
            h.set_launch(rows_per_block=1)
            h.iterate(T)
            for level in range(2):
                m = h.messages(level)
                assert np.array_equal(m["rho"].cpu().numpy(), r.state.rho[level]), (T, level)
                assert np.array_equal(m["alpha"].cpu().numpy(), r.state.alpha[level]), (T, level)
            assert np.array_equal(h.labels().cpu().numpy(), r.labels)


@pytest.mark.parametrize("form", ["plain", "points", "kappa", "mrhap", "fused"])
@pytest.mark.parametrize("fill,lam", [(0.0, 0.0), (float("nan"), 0.7), (float("inf"), 0.7)])
@pytest.mark.parametrize("n,threads,rb", [(33, 64, 2), (253, 64, 9), (261, 64, 3), (489, 128, 2), (509, 128, 8), (510, 128, 17),
                                          (1021, 256, 5), (1033, 256, 5), (2045, 512, 8), (241, 64, 1), (501, 128, 1),
                                          (1001, 256, 1)])
def test_rows_in_flight_equal_the_streaming_pass(hap_gpu, n, threads, rb, fill, lam, form):
    hap = hap_gpu
    X, S = problem(hap, n, fill)
    kw = dict(schedule=hap.SCHEDULE_MRHAP) if form in ("mrhap", "fused") else dict(kappa=0.5) if form == "kappa" else {}
    with hap.Hap(S, 2, lam, pref=-30.0, **kw) as a, hap.Hap(S, 2, lam, pref=-30.0, **kw) as b:
        a.set_launch(threads, 4, rb, unfused=form != "fused")
        if form == "points":
            a.set_points(X)
        assert bool(a.launch_flags() & hap.LAUNCH_FUSED) == (form == "fused")
        b.set_launch(1024, 1, rb, streaming=True, unfused=True)
        for h in (a, b):
            h.iterate(6)
        for level in range(2):
            x, y = a.messages(level), b.messages(level)
            for k in x:
                assert torch.equal(x[k], y[k]), (level, k)
        assert torch.equal(a.labels(), b.labels())


@pytest.mark.parametrize("col", range(9))
def test_a_similarity_that_is_not_a_number(hap_gpu, col):
    """One NaN similarity in a column of every row: no comparison takes it."""
    hap = hap_gpu
    n = 300
    _, S = problem(hap, n, 0.0)
    S[:, col] = float("nan")
    out = []
    for shape in ((64, 4, 2, False), (128, 4, 1, False), (1024, 1, 2, True), (1024, 1, 1, True)):
        with hap.Hap(S, 1, 0.5, pref=-30.0) as h:
            h.set_launch(*shape[:3], streaming=shape[3])
            h.iterate(4)
            out.append(h.messages(0)["rho"].nan_to_num(nan=7e30))
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])


@pytest.mark.parametrize("threads,groups", [(256, 1), (512, 2), (512, 4), (1024, 4)])
def test_batched_problems_without_damping(hap_gpu, threads, groups):
    sizes = [5, 6, 41, 201, 253, 257, 509, 1021, 1029]
    rng = np.random.default_rng(4)
    xs = [(rng.standard_normal((n, 2)) * 2 + 12 * rng.integers(0, 5, (n, 1))).astype(np.float32) for n in sizes]
    plan = hap_gpu.HapBatch(sizes, 2, 2)
    plan.set_launch(threads, 0, groups)
    labels, _, _ = plan.run(torch.from_numpy(np.concatenate(xs)).to(DEV), 0.0, 3, 0)
    for b, x in enumerate(xs):
        S = sim.similarity(x.astype(np.float64)).astype(np.float32)
        r = hap_ref.hap(S, sim.median_offdiag(S, np.float32), 2, 0.0, 3, dtype=np.float32)
        assert np.array_equal(plan.labels_of(labels, b).cpu().numpy(), r.labels), sizes[b]
    plan.close()
