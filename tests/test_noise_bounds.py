"""The bounds on the Gumbel noise that the sampling kernel uses to skip tokens.

The kernel bounds a token's noise from the bits of its tail probability as a float
instead of evaluating the two logarithms: from above by an offset less a multiple of
those bits, and, where that bound is large enough, from below by it minus a fixed gap.
A wrong bound would make the kernel skip a token that can win, so both are checked here
against the oracle's noise for every one of the 2^23 values the uniform variate takes,
with the constants read from the kernel's header, as is the overall range.
"""
import pathlib
import re

import numpy as np
import pytest

import oracle

HEADER = pathlib.Path(__file__).resolve().parents[1] / "paper_2609_03844_amd" / "csrc" / "sbw_device.hpp"


def header_constants():
    text = HEADER.read_text()
    out = {}
    for name, value in re.findall(r"constexpr float (k\w+) = ([-+0-9.eE]+)f;", text):
        out[name] = np.float32(float(value))
    return out


@pytest.fixture(scope="module")
def every_draw():
    x = np.arange(1 << 23, dtype=np.uint32) << np.uint32(9)   # the low 9 bits do not enter u
    return x, oracle.gumbel_of_draws(x).astype(np.float64)


def test_overall_range(every_draw):
    _, g = every_draw
    k = header_constants()
    assert k["kGumbelLo"] < g.min() and g.max() < k["kGumbelHi"]


def test_bounds_from_the_bits_of_the_tail_probability(every_draw):
    """With any low bits of the draw: they do not enter the variate, nor the bound."""
    x, g = every_draw
    k = header_constants()
    for low in (0, 0x1A5, 0x1FF):
        y = (~(x | np.uint32(low)) & np.uint32(0xFFFFFE00)) | np.uint32(0x100)
        bits = y.astype(np.float32).view(np.uint32).astype(np.float32).astype(np.float64)
        upper = np.float64(k["kNoiseBitsOffset"]) - np.float64(k["kNoiseBitsScale"]) * bits
        assert (upper - g).min() > 0.0005                    # room for the fp32 logarithm and fma
        tail = upper > np.float64(k["kNoiseUpperRange"])
        assert np.all(y[tail] < 1 << 30)                     # q < 1/4 wherever the bound is that large
        assert (upper - g)[tail].max() < np.float64(k["kNoiseGap"]) - 0.003
