"""The perceptron's fused kernels (n_in <= 32, hidden <= 256, n_out <= 16) at the edges of their tiles
of 32 rows, 16 and 32 hidden units, 16 outputs: the forward pass against the FP64 oracle, the
gradient and the Adam steps against the layer-by-layer path, bit for bit."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import warm
from test_gpu_warm import DEV, U32, UBF16, forward_bound, mlp_problem

pytestmark = pytest.mark.gpu

SHAPES = [(32, 128, 3, 1), (32, 64, 4, 33), (7, 33, 2, 97), (16, 100, 16, 289), (32, 256, 3, 65), (1, 1, 1, 31)]


def layered_bytes(n_in, hidden, n_out, rows):
    """Workspace of the layer-by-layer path: its activations, their gradients, the parameter
    gradient and the loss, each rounded up to 256 bytes."""
    count = n_in * hidden + hidden + hidden * hidden + hidden + hidden * n_out + n_out
    parts = [rows * n_in, rows * n_out, rows * hidden, rows * hidden, rows * n_out, rows * n_out, rows * hidden,
             rows * hidden, count, 16]
    return sum((4 * p + 255) // 256 * 256 for p in parts)


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("n_in,hidden,n_out,rows", SHAPES)
def test_forward_within_derived_bound(hap_gpu, n_in, hidden, n_out, rows, prec):
    flat, X, _ = mlp_problem(31, rows, n_in, hidden, n_out)
    m = hap_gpu.Mlp(torch.from_numpy(flat).to(DEV), n_in, hidden, n_out,
                    precision=hap_gpu.HAP_F32 if prec == "f32" else hap_gpu.HAP_BF16)
    out = torch.full((rows + 1, n_out + 1), 7.0, device=DEV)
    Y = m.forward(torch.from_numpy(X).to(DEV), out=out[:rows, :n_out])
    P = warm.unpack(flat.astype(np.float64), n_in, hidden, n_out)
    ref, _ = warm.forward(P, X.astype(np.float64))
    bound = forward_bound(P, X, U32 if prec == "f32" else UBF16, max(hidden, n_in))
    assert np.all(np.abs(Y.cpu().numpy() - ref) <= bound + 1e-30)
    assert (out[rows] == 7.0).all() and (out[:, n_out] == 7.0).all()


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("n_in,hidden,n_out,rows", SHAPES)
def test_training_equals_the_layered_path(hap_gpu, n_in, hidden, n_out, rows, prec):
    lib = hap_gpu.load()
    code = hap_gpu.HAP_F32 if prec == "f32" else hap_gpu.HAP_BF16
    flat, X, T = mlp_problem(32, rows, n_in, hidden, n_out)
    X, T = torch.from_numpy(X).to(DEV), torch.from_numpy(T).to(DEV)
    small = layered_bytes(n_in, hidden, n_out, rows)
    full = ctypes.c_size_t()
    assert lib.hap_mlp_workspace_size(n_in, hidden, n_out, rows, ctypes.byref(full)) == 0
    assert small < full.value       # so that the smaller workspace selects the layered path
    steps = 3
    idx = torch.from_numpy(np.random.default_rng(5).integers(0, rows, rows * steps).astype(np.int32)).to(DEV)
    ws = torch.empty(full.value, dtype=torch.uint8, device=DEV)
    P = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    got = []
    for nbytes in (small, full.value):
        p = torch.from_numpy(flat).to(DEV)
        grad, loss = torch.empty_like(p), torch.empty((), dtype=torch.float64, device=DEV)
        st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert lib.hap_mlp_loss_grad(P(p), n_in, hidden, n_out, code, P(X), n_in, P(T), n_out, rows, P(grad), P(loss),
                                     P(ws), nbytes, st) == 0
        opt = torch.zeros(2 * p.numel(), device=DEV)
        hist = torch.empty(steps, dtype=torch.float64, device=DEV)
        assert lib.hap_mlp_train(P(p), P(opt), n_in, hidden, n_out, code, 0, P(X), n_in, P(T), n_out, rows, P(idx),
                                 rows, steps, 1e-3, P(hist), P(ws), nbytes, st) == 0
        # without a loss history
        assert lib.hap_mlp_train(P(p), P(opt), n_in, hidden, n_out, code, steps, P(X), n_in, P(T), n_out, rows, P(idx),
                                 rows, 1, 1e-3, None, P(ws), nbytes, st) == 0
        torch.cuda.synchronize()
        got.append((grad, opt, p, loss, hist))
    (g0, o0, p0, l0, h0), (g1, o1, p1, l1, h1) = got
    assert torch.equal(g0, g1) and torch.equal(o0, o1) and torch.equal(p0, p1)
    # the loss adds the same FP64 squares in another order: at most rows * n_out roundings apart
    tol = 2.0 * rows * n_out * 2.0 ** -53
    assert abs(l0 - l1) <= tol * abs(l0) and ((h0 - h1).abs() <= tol * h0.abs()).all()
