"""The held-row pass at the lengths it runs by default (six and eight chunks, sixteen with a ragged end) against
the streaming pass, bit for bit, under both schedules, with contiguous row blocks and with the Eq. 2.7 offsets."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_held_launch import held, similarity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels", [(8193, 3), (12290, 2), (16384, 2)])
@pytest.mark.parametrize("form", ["plain", "blocks", "mrhap", "kappa"])
def test_equals_the_streaming_pass(hap_gpu, n, levels, form):
    hap = hap_gpu
    S = similarity(hap, n)
    kw = dict(schedule=hap.SCHEDULE_MRHAP) if form == "mrhap" else dict(kappa=0.5) if form == "kappa" else {}
    with hap.Hap(S, levels, 0.6, pref=-20.0, **kw) as a, hap.Hap(S, levels, 0.6, pref=-20.0, **kw) as b:
        a.set_launch(blocks=form == "blocks")
        b.set_launch(1024, -(-n // 4096) + 1, streaming=True, blocks=form == "blocks")
        assert held(hap, a) and not held(hap, b) and a.get_launch()[2] == b.get_launch()[2]
        for h in (a, b):
            h.iterate(4)
        for level in range(levels):
            x, y = a.messages(level), b.messages(level)
            for k in x:
                assert torch.equal(x[k], y[k]), (level, k)
            del x, y
        assert torch.equal(a.labels(), b.labels())


@pytest.mark.parametrize("n,form", [(16385, "plain"), (20001, "kappa"), (20002, "mrhap"), (20000, "blocks")])
def test_sixteen_ragged_chunks_equal_the_streaming_pass(hap_gpu, n, form):
    """The default pass of 16384 < n < 32768: 512 threads x 16 chunks with a ragged end."""
    hap = hap_gpu
    S = similarity(hap, n)
    kw = dict(schedule=hap.SCHEDULE_MRHAP) if form == "mrhap" else dict(kappa=0.5) if form == "kappa" else {}
    with hap.Hap(S, 2, 0.6, pref=-20.0, **kw) as a, hap.Hap(S, 2, 0.6, pref=-20.0, **kw) as b:
        a.set_launch(blocks=form == "blocks")
        rb = (n + 255) // 256
        assert a.get_launch() == (512, 16, rb, True) and held(hap, a)
        b.set_launch(1024, -(-n // 4096), rb, streaming=True, blocks=form == "blocks")
        assert not held(hap, b)
        for h in (a, b):
            h.iterate(4)
        for level in range(2):
            x, y = a.messages(level), b.messages(level)
            for k in x:
                assert torch.equal(x[k], y[k]), (level, k)
            del x, y
        assert torch.equal(a.labels(), b.labels())
