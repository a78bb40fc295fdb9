"""conv_small (the smallest forward passes in one launch) at the edges of its tiles, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1504_04343_amd import synth
from gpu_util import gpu_forward, layer, odims

pytestmark = pytest.mark.gpu

#          name       N   C    H   W    O  K  s  p  g
LAYERS = [layer("one",      1,   1,  1,  1,   1, 3, 1, 2),      # one channel, a padded 1 x 1 plane
          layer("listed",   4,   3, 32, 32,  16, 5, 1, 2),
          layer("odd",      3,   7, 11, 13,   9, 3, 1, 1),      # rows and positions to spare
          layer("groups",   2,  12,  9,  8,  10, 3, 1, 0, 2),
          layer("stride",   2,   5, 23, 21,   6, 4, 3, 2),
          layer("k11",      2,   4, 15, 14,   5, 11, 4, 5),     # 484 products, most taps outside
          layer("kd512",    1, 128,  7,  7,  33, 2, 1, 0),      # the most products
          layer("kd8",      5,   2,  9,  9,  13, 2, 1, 0),      # one product per wave
          layer("kd9",      2,   1,  9,  9,   3, 3, 1, 0)]      # waves without products


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_1504_04343_amd import binding
    return binding


def run(B, L, x, w, b):
    B.cct_profile_enable(True)
    got = gpu_forward(B, L, x, w, b, B.LOWER_AUTO)
    B.cct_profile_enable(False)
    return got, [e["name"] for e in B.cct_profile_read()]


@pytest.mark.parametrize("bias", [True, False], ids=["bias", "no_bias"])
@pytest.mark.parametrize("L", LAYERS, ids=lambda L: L.name)
def test_forward(B, L, bias):
    """Sums in 64 bits: a result is off by its own rounding, 2^-24 of it, and 2^-45 of what was added up."""
    x, w, b = synth.make_x(L, 2), synth.make_w(L, 2), synth.make_bias(L, 2) if bias else None
    got, names = run(B, L, x, w, b)
    assert names == ["conv_small"]
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    size = oracle.conv_forward(odims(oracle, L), np.abs(x), np.abs(w), None if b is None else np.abs(b))
    assert (np.abs(got - want) <= 2.0 ** -24 * np.abs(want) + 2.0 ** -45 * size + 2.0 ** -149).all()


def test_not_finite(B):
    """Infinities and NaN reach exactly the results they reach in fp32: not those of taps outside the tensor."""
    L = layer("nf", 3, 6, 13, 13, 10, 3, 1, 1)
    x, w, b = synth.make_x(L, 5), synth.make_w(L, 5), synth.make_bias(L, 5)
    x[0, 0, 0, 0], x[1, 1, 5, 6], x[1, 2, 12, 12] = np.inf, -np.inf, np.nan
    w[3, 1, 1, 2], w[7, 0, 0, 0], w[9, 0, 2, 2], w[5] = np.inf, np.nan, -np.inf, 0.0
    got, names = run(B, L, x, w, b)
    assert names == ["conv_small"]
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    assert (np.isnan(got) == np.isnan(want)).all() and (np.isinf(got) == np.isinf(want)).all()
    inf, ok = np.isinf(want), np.isfinite(want)
    assert (np.sign(got[inf]) == np.sign(want[inf])).all()
    assert np.abs(got[ok] - want[ok]).max() <= 1e-6 * np.abs(want[ok]).max()


@pytest.mark.parametrize("L", [layer("wide", 16, 16, 14, 14, 64, 3, 1, 1), layer("long", 1, 129, 7, 7, 8, 2, 1, 0),
                               layer("1x1", 2, 33, 7, 9, 34, 1)],
                         ids=lambda L: L.name)
def test_larger_layers_and_forced_types_run_elsewhere(B, L):
    x, w, b = synth.make_x(L, 2), synth.make_w(L, 2), synth.make_bias(L, 2)
    got, names = run(B, L, x, w, b)
    assert "conv_small" not in names
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()
    B.cct_profile_enable(True)
    gpu_forward(B, LAYERS[1], synth.make_x(LAYERS[1], 2), synth.make_w(LAYERS[1], 2), None, B.LOWER_TYPE1)
    B.cct_profile_enable(False)
    assert "conv_small" not in [e["name"] for e in B.cct_profile_read()]
