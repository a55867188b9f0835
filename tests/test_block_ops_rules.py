"""Which calls the block kernels take: the rules that do not ask for a GPU."""
import pytest

torch = pytest.importorskip("torch")
ops = pytest.importorskip("paper_2410_15352_amd._block_ops")
blk = pytest.importorskip("paper_2410_15352_amd.block")


@pytest.mark.parametrize("width,gains,takes", [(64, 64, True), (64, 128, False), (128, 64, False), (64, 1, False),
                                               (12, 12, False), (4096, 4096, True), (4104, 4104, False)])
def test_norm_takes_one_gain_per_element(monkeypatch, width, gains, takes):
    """The kernel reads `width` gains: any other number must not reach it."""
    monkeypatch.setattr(ops, "usable", lambda *t: True)
    x, g = torch.empty(3, width, dtype=torch.bfloat16), torch.ones(gains, dtype=torch.bfloat16)
    assert ops.norm_usable(x, g) == takes
    assert not ops.norm_usable(x, g.expand(2, gains))


def test_norm_of_another_width_is_refused():
    with pytest.raises(RuntimeError):
        blk.RMSNorm(64)(torch.randn(3, 128).to(torch.bfloat16))
