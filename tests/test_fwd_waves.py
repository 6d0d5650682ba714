"""How many waves a dense forward's workgroups have: the sizes measured with
both forms take the faster one (CPU; the figures are beside the rule)."""
import pytest

from paper_2609_13612_amd import _lib

COPIED, NEOX, INTER = 0, 1, 2
NONE, CAUSAL, WINDOW = 0, 1, 2


def _waves(B, H, Hkv, S, D, rope, mask, window=0, bias=0):
    return _lib.load().af_fwd_waves(B, H, Hkv, S, D, rope, mask, window, bias)


@pytest.mark.parametrize("case,waves", [
    # keys rotated in the loop: four waves while they fit one round of 256 workgroups
    ((1, 32, 8, 256, 128, NEOX, CAUSAL), 4), ((2, 32, 8, 512, 128, NEOX, NONE), 4), ((4, 12, 12, 512, 64, INTER, NONE), 4),
    ((10, 8, 8, 270, 128, INTER, NONE), 8), ((10, 8, 8, 270, 128, NEOX, NONE), 4),
    # more than a round without a mask: lost 10 to 28 %
    ((6, 16, 2, 400, 128, NEOX, NONE), 8), ((10, 8, 8, 512, 128, INTER, NONE), 8), ((3, 12, 12, 1000, 64, NEOX, NONE), 8),
    ((6, 40, 8, 176, 128, NEOX, NONE), 8), ((3, 12, 12, 919, 64, INTER, NONE), 8),
    # and with one: won at D = 64, and under most windows
    ((3, 12, 12, 1000, 64, NEOX, CAUSAL), 4), ((6, 32, 8, 270, 128, INTER, CAUSAL), 8), ((3, 12, 12, 1000, 64, NEOX, WINDOW, 100), 4),
    ((10, 8, 2, 1000, 64, NEOX, WINDOW, 100), 4), ((3, 32, 8, 512, 128, NEOX, WINDOW, 100), 8),   # 20.7 / 23.6, 23.0 / 20.1
    # 17.0 / 22.5, 18.3 / 20.3, 15.4 / 24.5, 25.7 / 39.3, 9.1 / 10.4
    ((4, 12, 12, 790, 64, NEOX, WINDOW, 337), 4), ((4, 12, 12, 1024, 64, NEOX, WINDOW, 256), 4), ((6, 16, 16, 604, 64, NEOX, WINDOW, 66), 4),
    ((6, 24, 8, 423, 128, NEOX, WINDOW, 23), 4), ((8, 8, 2, 534, 64, NEOX, WINDOW, 29), 4),
    # all four-wave workgroups resident, eight waves in two rounds, or the same number of either: 23.1 / 35.7, 9.2 / 15.0
    ((6, 16, 16, 616, 64, NEOX, NONE), 4), ((8, 40, 8, 35, 128, INTER, WINDOW, 32), 4),
    # the interleaved four-wave kernel spills at D = 128
    ((1, 32, 8, 512, 128, INTER, CAUSAL), 8), ((1, 32, 8, 512, 128, INTER, WINDOW, 100), 4),
    ((1, 32, 8, 600, 128, NEOX, CAUSAL), 8), ((1, 12, 12, 1100, 64, NEOX, CAUSAL), 8),
    # tiles copied to LDS
    ((1, 32, 8, 2048, 128, COPIED, CAUSAL), 4), ((1, 32, 8, 8192, 128, COPIED, CAUSAL), 8), ((4, 12, 12, 2048, 64, COPIED, NONE), 4),
    ((1, 12, 12, 4096, 64, COPIED, NONE), 8), ((1, 12, 12, 4096, 64, COPIED, NONE, 0, 1), 8),
    ((1, 12, 12, 4096, 64, COPIED, NONE, 0, 2), 4), ((1, 12, 12, 4096, 64, COPIED, CAUSAL), 4),
    ((1, 16, 4, 3000, 128, COPIED, NONE, 0, 1), 8), ((2, 16, 4, 3000, 128, COPIED, NONE, 0, 1), 4),
    ((1, 16, 4, 3000, 128, COPIED, NONE, 0, 2), 4), ((1, 32, 8, 4096, 128, COPIED, CAUSAL, 0, 1), 8), ((3, 24, 8, 4102, 128, COPIED, CAUSAL, 0, 1), 4),
    ((1, 32, 8, 4096, 128, COPIED, CAUSAL, 0, 0), 4)])
def test_measured_sizes(case, waves):
    assert _waves(*case) == waves


def test_other_sizes_are_four_or_eight():
    for B in (1, 3, 100):
        for H, Hkv in ((1, 1), (6, 2), (64, 1)):
            for S in (1, 63, 256, 1025, 1 << 20):
                for D in (64, 128):
                    for rope in (0, 1, 2):
                        for mask, window in ((0, 0), (1, 0), (2, 1), (2, S)):
                            for bias in (0, 1, 2):
                                assert _waves(B, H, Hkv, S, D, rope, mask, window, bias) in (4, 8)
