"""conv_bwdw_few (backward-weights of layers with few channels, x and dy in place): the sizes where it can go wrong,
against the oracle.  Three bf16 terms hold a product of two fp32 values to 2^-25: the fp32 path's tolerance."""
import numpy as np
import pytest

import oracle
from paper_1504_04343_amd import synth
from gpu_util import TOL_F32, gpu_backward_weights, layer, odims, rel_err

pytestmark = pytest.mark.gpu

# name, N, C, H, W, O, K, stride, pad, groups; the kernels of a tile and blocks of 128 lowered rows that should run
SHAPES = [
    (layer("conv1",      19,  3, 99, 67,  96, 11, 4, 0), 96, 3),     # 3 images in the last group, 15 columns in two strips
    (layer("conv1_pad",  65,  3, 61, 83, 193, 11, 4, 5), 96, 3),     # rows above and below the image; 3 row tiles, 1 kernel in the last
    (layer("seven",      40,  3, 56, 49,  64,  7, 2, 3), 64, 2),
    (layer("seven_s1",   33,  4, 30, 41,  65,  7, 1, 3), 96, 2),
    (layer("five",       64,  4, 32, 57,  32,  5, 1, 2), 32, 1),
    (layer("three",     128,  8, 40, 43,  40,  3, 1, 1), 64, 1),
    (layer("past_96",   100, 10, 41, 37, 101,  3, 1, 1), 64, 1),     # 37 kernels in the second tile
    (layer("past_96_7",  64,  3, 61, 59, 128,  7, 2, 3), 64, 2),
    (layer("three_g2",  100, 16, 33, 35,  60,  3, 2, 1, 2), 32, 1),
]


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_1504_04343_amd import binding
    return binding


def run(B, L, x, dy, chunk=None):
    B.cct_profile_enable(True)
    got = gpu_backward_weights(B, L, x, dy, chunk=chunk)
    B.cct_profile_enable(False)
    return got, [e["name"] for e in B.cct_profile_read()]


@pytest.mark.parametrize("L,rows,blocks", SHAPES, ids=[s[0].name for s in SHAPES])
def test_against_the_oracle(B, L, rows, blocks):
    x, dy = synth.make_x(L, 3), synth.make_dy(L, 3)
    (dw, db), names = run(B, L, x, dy)
    assert "conv_bwdw_few<%d, %d>" % (rows, blocks) in names, names
    want = oracle.conv_backward_weights(odims(oracle, L), x, dy)
    assert rel_err(dw, want[0]) <= TOL_F32 and rel_err(db, want[1]) <= TOL_F32


def test_in_chunks(B):
    """Chunks of 32 images, a last one of one: added to what the chunks before left."""
    L = SHAPES[1][0]
    x, dy = synth.make_x(L, 4), synth.make_dy(L, 4)
    (dw, db), names = run(B, L, x, dy, chunk=32)
    assert any(n.startswith("conv_bwdw_few") for n in names), names
    want = oracle.conv_backward_weights(odims(oracle, L), x, dy)
    assert rel_err(dw, want[0]) <= TOL_F32 and rel_err(db, want[1]) <= TOL_F32


@pytest.mark.parametrize("L", [SHAPES[0][0], SHAPES[2][0]], ids=["conv1", "seven"])
def test_not_finite_inputs(B, L):
    """Infinities, NaN and values beyond bf16's range reach exactly the weights they reach in fp32."""
    x, dy = synth.make_x(L, 5), synth.make_dy(L, 5)
    # 1e37 times a gradient below 10 stays in fp32's range, where a product that left it would be another infinity, whose
    # sum with a real one is NaN in fp32 and not in the oracle's 64 bits
    x[0, 0, 3, 0], x[1, 1, 0, 5], x[2, 2, 7, 7], x[-1, 1, 2, 2] = np.inf, -np.inf, np.nan, 1e37
    dy[0, 1, 2, 0], dy[1, 7, 0, 3], dy[3, 9, 1, 1] = np.inf, np.nan, 1e37
    (dw, db), names = run(B, L, x, dy)
    assert any(n.startswith("conv_bwdw_few") for n in names), names
    want = oracle.conv_backward_weights(odims(oracle, L), x, dy)
    for got, ref in ((dw, want[0]), (db, want[1])):
        assert (np.isnan(got) == np.isnan(ref)).all()
        over = np.abs(ref) > np.finfo(np.float32).max
        assert (np.isinf(got) == (over & ~np.isnan(ref))).all()
        ok = np.isfinite(got)
        big = ok & (np.abs(ref) > 1e30)
        assert (np.abs(got[big] - ref[big]) <= 1e-5 * np.abs(ref[big])).all()
        assert rel_err(got[ok & ~big], ref[ok & ~big]) <= TOL_F32


def test_bias_gradient_of_long_columns(B):
    """A row that leaves the rows below it under half a unit of the last place: added one by one in fp32 all 39 are lost,
    2^-24 of the result each.  A tree of 16 values, a sum over the rows in 64 bits, 512 partial sums as
    two sums of four in each of 64 strips and their tree: at most 4 + 1 + (2 + 2) + 6 roundings."""
    L = layer("long", 1024, 1, 42, 34, 32, 3, 1, 0)
    x, dy = synth.make_x(L, 6), np.zeros((L.N, L.O, L.Hout, L.Wout), np.float32)
    dy[::8] = 1.0
    dy[::8, :, 0] = 2.0**24
    (dw, db), names = run(B, L, x, dy)
    assert any(n.startswith("conv_bwdw_few") for n in names), names
    want = dy[:, 0].astype(np.float64).sum()
    assert np.abs(db / want - 1.0).max() <= 16 * 2.0**-24


def test_partial_sums_of_several_launches(B):
    """More than 256 MiB of partial sums: two launches, the second one's added to what the first left."""
    L = layer("two_launches", 233, 23, 6, 59, 960, 4)  # of 216 and 17 images
    assert 30 * ((L.Wout + 7) // 8) * 4 * L.O * L.C * L.K**2 > 2**28
    x, dy = synth.make_x(L, 7), synth.make_dy(L, 7)
    (dw, db), names = run(B, L, x, dy)
    assert any(n.startswith("conv_bwdw_few") for n in names), names
    idx = np.random.default_rng(7).choice(dw.size, 2000, replace=False)
    assert rel_err(dw.ravel()[idx], oracle.conv_backward_weights_at(odims(oracle, L), x, dy, idx)) <= TOL_F32
    assert rel_err(db, dy.sum((0, 2, 3), dtype=np.float64)) <= TOL_F32
