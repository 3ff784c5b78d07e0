"""hap_exemplars writes the labels into whatever memory it was given by the same route with and without the count:
ordinary and pinned host memory, and an offset into device memory."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", ["pageable", "pinned", "device"])
def test_labels_with_and_without_the_count(hap_gpu, kind):
    n = 600
    rng = np.random.default_rng(3)
    X = torch.from_numpy((rng.standard_normal((n, 2)) + 9 * rng.integers(0, 6, (n, 1))).astype(np.float32)).to(DEV)
    S = torch.empty((n, n), dtype=torch.float32, device=DEV)
    hap_gpu.build_similarity(X, S)
    with hap_gpu.Hap(S, 1, 0.5) as h:
        h.iterate(10)
        expect, k = h.exemplars(0)
        expect = expect.cpu().numpy()
        got = []
        for counted in (False, True):
            if kind == "pageable":
                buf = np.full(n + 2, -7, dtype=np.int32)
                at = buf.ctypes.data + 4
            else:
                buf = torch.full((n + 2,), -7, dtype=torch.int32, device=DEV) if kind == "device" else \
                    torch.full((n + 2,), -7, dtype=torch.int32).pin_memory()
                at = buf.data_ptr() + 4
            count = ctypes.c_int32(-1)
            status = h._lib.hap_exemplars(h._ctx, 0, ctypes.c_void_p(at), ctypes.byref(count) if counted else None)
            torch.cuda.synchronize()
            out = buf if kind == "pageable" else buf.cpu().numpy()
            assert out[0] == -7 and out[-1] == -7
            if status == hap_gpu.HAP_OK:
                assert np.array_equal(out[1:-1], expect)
                assert count.value == (k if counted else -1)
            got.append(status)
        assert got[0] == got[1]
        assert kind == "pageable" or got[0] == hap_gpu.HAP_OK
