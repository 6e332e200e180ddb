"""The K split of the gate's logits, read from its workspace (host only): T * E fp32 partials per slice."""
import pytest

moe = pytest.importorskip("paper_2606_10493_amd")


def _slices(t, h, e):
    n = moe.moe_router_workspace(t, h, e)
    assert n % (4 * t * e) == 0
    return n // (4 * t * e)


@pytest.mark.parametrize("h,e", [(7168, 256), (2048, 128), (4096, 16)])
def test_large_calls_keep_two_accumulators(h, e):
    """From 32768 to 65280 tokens two slices: one accumulator over all of H has 1.4 times their error."""
    assert [_slices(t, h, e) for t in (16384, 32640, 32768, 40000, 65280, 65281)] == [2, 2, 2, 2, 2, 1]


def test_slices_fill_the_chip_and_divide_h():
    for t in (256, 300, 512, 1000, 4096, 8192):
        for h in (256, 5120, 7168):
            for e in (8, 256, 300, 1024):
                ks = _slices(t, h, e)
                assert (h // 32) % ks == 0
                tiles = -(-t // 128) * -(-e // 256)
                assert ks == 1 or (ks - 1) * tiles < 256
