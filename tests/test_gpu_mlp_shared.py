"""The perceptron's forward pass with outputs in the memory of its inputs: the values of a pass into memory of its
own, whatever the two row strides."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_warm import DEV, mlp_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("place", ["packed", "columns", "shifted", "beside"])
def test_outputs_over_inputs(hap_gpu, place, prec):
    rows, n_in, hidden, n_out = 40000, 32, 128, 3
    flat, X, _ = mlp_problem(41, rows, n_in, hidden, n_out)
    m = hap_gpu.Mlp(torch.from_numpy(flat).to(DEV), n_in, hidden, n_out,
                    precision=hap_gpu.HAP_F32 if prec == "f32" else hap_gpu.HAP_BF16)
    X = torch.from_numpy(X).to(DEV)
    expect = m.forward(X)
    buf = X.clone()
    if place == "packed":      # rows of three values over the first rows of 32
        out = buf.view(-1)[:rows * n_out].view(rows, n_out)
    elif place == "columns":   # a row's outputs over its own inputs
        out = buf[:, 5:5 + n_out]
    elif place == "beside":    # columns next to the inputs
        buf = torch.cat([buf, torch.zeros((rows, 8), device=DEV)], dim=1)
        buf, out = buf[:, :n_in], buf[:, n_in + 2:n_in + 2 + n_out]
    else:                      # a row's outputs over another row's inputs
        out = torch.cat([buf, torch.zeros((33, n_in), device=DEV)])
        buf = out[:rows]
        out = out[33:, :n_out]
    assert torch.equal(m.forward(buf, out=out), expect)
