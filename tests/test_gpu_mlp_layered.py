"""The perceptron's fused kernels against the layer-by-layer path in every instance, bit for bit: the same network with
33 inputs, the added ones zero, is too wide for the fused kernels, and products with zeros leave every sum as it
was.  Batches of less than a tile of 32 rows to more tiles than the device holds workgroups (256 to 1536, by instance),
and more than the 24 tiles whose operands a weight gradient loads at once."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_warm import DEV, mlp_problem

pytestmark = pytest.mark.gpu
WIDE = 33


def wider(flat, n_in, hidden):
    """Parameters with WIDE inputs, zero weights for the added ones."""
    pad = np.zeros((WIDE - n_in) * hidden, dtype=np.float32)
    return np.concatenate([flat[:n_in * hidden], pad, flat[n_in * hidden:]])


def narrower(flat, n_in, hidden):
    return torch.cat([flat[:n_in * hidden], flat[WIDE * hidden:]])


def both(hap, seed, rows, n_in, hidden, n_out, prec):
    code = hap.HAP_F32 if prec == "f32" else hap.HAP_BF16
    flat, X, T = mlp_problem(seed, rows, n_in, hidden, n_out)
    Xw = np.zeros((rows, WIDE), dtype=np.float32)
    Xw[:, :n_in] = X
    d = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    fused = hap.Mlp(d(flat), n_in, hidden, n_out, precision=code)
    layered = hap.Mlp(d(wider(flat, n_in, hidden)), WIDE, hidden, n_out, precision=code)
    return fused, layered, d(X), d(Xw), d(T)


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("n_in,hidden,n_out,rows", [(32, 64, 4, 33), (7, 33, 2, 97), (32, 96, 1, 24 * 32),
                                                    (16, 100, 16, 1000), (32, 128, 3, 4096), (32, 128, 3, 16500),
                                                    (32, 256, 3, 65), (30, 200, 5, 1500), (32, 256, 2, 8500),
                                                    (32, 64, 1, 33000)])
def test_training(hap_gpu, n_in, hidden, n_out, rows, prec):
    a, b, X, Xw, T = both(hap_gpu, 51, rows, n_in, hidden, n_out, prec)
    tol = 2.0 * rows * n_out * 2.0 ** -53    # the loss adds the same FP64 squares in another order
    (la, ga), (lb, gb) = a.loss_grad(X, T), b.loss_grad(Xw, T)
    assert torch.equal(ga, narrower(gb, n_in, hidden))
    assert abs(la - lb) <= tol * abs(lb)
    steps = 3
    idx = torch.from_numpy(np.random.default_rng(5).integers(0, rows, rows * steps).astype(np.int32)).to(DEV)
    ha, hb = a.train(X, T, idx, rows, steps, 1e-3), b.train(Xw, T, idx, rows, steps, 1e-3)
    assert torch.equal(a.params, narrower(b.params, n_in, hidden))
    cnt = b.count
    for k in range(2):
        assert torch.equal(a.opt_state[k * a.count:(k + 1) * a.count], narrower(b.opt_state[k * cnt:(k + 1) * cnt], n_in, hidden))
    assert ((ha - hb).abs() <= tol * hb.abs()).all()


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("n_in,hidden,n_out,rows", [(5, 40, 2, 1), (32, 64, 2, 50001), (32, 128, 3, 40000),
                                                    (31, 256, 16, 9000)])
def test_forward(hap_gpu, n_in, hidden, n_out, rows, prec):
    a, b, X, Xw, _ = both(hap_gpu, 52, rows, n_in, hidden, n_out, prec)
    assert torch.equal(a.forward(X), b.forward(Xw))
