"""Which pass runs FP32 rows of 8192 < n <= 16384: the held-row pass, whatever part of the default launch is set
again, read back and set, or chosen by the tuner."""
import json

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1403_7394_amd import autotune

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def similarity(hap, n):
    rng = np.random.default_rng(n)
    X = torch.from_numpy(rng.standard_normal((n, 2)).astype(np.float32) * 10).to(DEV)
    S = torch.empty((n, (n + 3) // 4 * 4), dtype=torch.float32, device=DEV)[:, :n]
    hap.build_similarity(X, S)
    return S


def held(hap, h):
    return bool(h.launch_flags() & hap.LAUNCH_HELD)


@pytest.mark.parametrize("n", [8192, 8193, 12289, 16384, 16385])
def test_settings_that_keep_the_shape_keep_the_pass(hap_gpu, n):
    hap = hap_gpu
    with hap.Hap(similarity(hap, n), 1, 0.5, pref=-5.0) as h:
        shape = h.get_launch()
        assert held(hap, h) == (n > 8192)
        for change in (dict(eager=True), dict(blocks=True), dict(rows_per_block=3), dict(eager=False, blocks=False)):
            h.set_launch(**change)
            assert held(hap, h) == (n > 8192), change
        h.set_launch(*shape[:3], streaming=shape[3])
        assert h.get_launch() == shape and held(hap, h) == (n > 8192)
        if n > 8192:
            h.set_launch(1024, -(-n // 4096) + 1, streaming=True)   # more chunks than the rows need
            assert not held(hap, h)


def test_the_tuner_offers_the_held_pass(hap_gpu, tmp_path, monkeypatch):
    hap = hap_gpu
    n = 9000
    cache = tmp_path / "tuning.json"
    monkeypatch.setenv("HAP_TUNING_CACHE", str(cache))
    S = similarity(hap, n)
    with hap.Hap(S, 1, 0.5, pref=-5.0) as h:
        best = autotune.tune_sweep(h)
        assert held(hap, h) and h.get_launch() == best
    # a shape stored for a longer row of the same bucket is not taken over
    stored = json.loads(cache.read_text())
    key, = stored
    stored[key] = [1024, 4, 63, True, 1.0]
    cache.write_text(json.dumps(stored))
    with hap.Hap(S, 1, 0.5, pref=-5.0) as h:
        autotune.tune_sweep(h)
        assert held(hap, h)
