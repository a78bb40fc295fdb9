"""conv_bwdw_img (backward-weights on granules of 8 images) at the sizes where it can go wrong, against
the oracle.  fp32 tolerance: three bf16 terms hold a product of two fp32 values to 2^-25; bf16: the
operands' rounding."""
import numpy as np
import pytest

import oracle
from paper_1504_04343_amd import synth
from gpu_util import TOL_BF16, TOL_F32, desc_of, dev, gpu_backward_weights, layer, odims, rel_err

pytestmark = pytest.mark.gpu

KERNEL = "conv_bwdw_img"

#          name         N    C   H   W    O  K  s  p  g
LAYERS = [
    layer("m128",     64, 192, 13, 13, 128, 3, 1, 1),
    layer("m64",      90, 384, 13, 13,  64, 3, 1, 1),           # 64-row tile; last granule holds 2 images
    layer("m192",     33, 192, 13, 13, 192, 3, 1, 1),           # one image in the last granule
    layer("m130",     40, 240, 14, 13, 260, 3, 1, 0, 2),        # rows beyond a tile; channels 3*32 + 24
    layer("c48",      25,  96, 20, 17, 256, 5, 1, 2, 2),        # a short last channel block
    layer("c70",      41, 170, 21, 17, 100, 2, 1, 1),           # even kernel; 100 of 128 rows
    layer("s2",       48, 192, 25, 23, 128, 3, 2, 1),
    layer("k1",       64, 512, 20, 14, 192, 1, 1, 0),           # a single tap
]


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_1504_04343_amd import binding
    return binding


def ran(B, call):
    B.cct_profile_enable(True)
    got = call()
    B.cct_profile_enable(False)
    return got, [e["name"] for e in B.cct_profile_read()]


def check(got, L, x, dy, tol):
    dw, db = oracle.conv_backward_weights(odims(oracle, L), x, dy)
    assert rel_err(got[0], dw) <= tol
    if got[1] is not None:
        assert rel_err(got[1], db) <= TOL_F32


@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("L", LAYERS, ids=[L.name for L in LAYERS])
def test_backward_weights(B, L, bf16):
    x, dy = synth.make_x(L, 3), synth.make_dy(L, 3)
    got, names = ran(B, lambda: gpu_backward_weights(B, L, x, dy, 0, int(bf16), want_dbias=L.N != 33))
    assert any(n.startswith(KERNEL) for n in names), names
    check(got, L, x, dy, TOL_BF16 if bf16 else TOL_F32)


@pytest.mark.parametrize("chunk", [40, 56, 8])
def test_chunks(B, chunk):
    """A workspace for fewer images takes the batch in chunks that add up (the last one shorter); one for
    too few runs the kernel that needs no copy of the tensors."""
    L = layer("chunks", 100, 192, 13, 13, 128, 3, 1, 1)
    x, dy = synth.make_x(L, 4), synth.make_dy(L, 4)
    got, names = ran(B, lambda: gpu_backward_weights(B, L, x, dy, chunk=chunk))
    assert any(n.startswith(KERNEL) for n in names) == (chunk >= 32), names
    check(got, L, x, dy, TOL_F32)


def test_precision(B):
    """No further from 64 bits than the fp32 matrix instructions' sums (measured 8e-7 in the 2-norm)."""
    L = layer("prec", 64, 192, 13, 13, 128, 3, 1, 1, x_dist="relu_normal")
    x, dy = synth.make_x(L, 1), synth.make_dy(L, 1)
    got = gpu_backward_weights(B, L, x, dy)[0].astype(np.float64)
    want = oracle.conv_backward_weights(odims(oracle, L), x, dy)[0]
    assert np.linalg.norm(got - want) / np.linalg.norm(want) <= 8e-7


# Random signs: a level of a pairwise sum adds about half a unit in the last place, 2^-25, of the result (2-norm).
@pytest.mark.parametrize("L,kernel,levels", [
    (layer("conv", 50, 384, 13, 13, 256, 3, 1, 1, 2), KERNEL, 14),      # 8 images, 32 pixels, 64 strips
    (layer("fc", 256, 16, 2, 2, 4096, 2), "dbias_columns", 8)], ids=["conv", "fc"])
def test_bias_gradient_is_summed_pairwise(B, L, kernel, levels):
    rng = np.random.default_rng(3)
    x = rng.standard_normal((L.N, L.C, L.H, L.W), dtype=np.float32)
    dy = rng.standard_normal((L.N, L.O, L.Hout, L.Wout), dtype=np.float32)
    (_, db), names = ran(B, lambda: gpu_backward_weights(B, L, x, dy))
    assert any(n.startswith(kernel) for n in names), names
    want = dy.astype(np.float64).sum((0, 2, 3))
    assert np.linalg.norm(db - want) / np.linalg.norm(want) <= 2.0 ** -25 * levels ** 0.5


@pytest.mark.parametrize("e,f", [(-118, 88), (-70, 40), (70, -50), (103, -83), (110, -90)], ids=lambda e: "2^%d" % e)
def test_range_of_fp32(B, e, f):
    """An operand of any magnitude that fp32 holds keeps its 24 bits (error as in test_precision)."""
    L = layer("range", 48, 192, 13, 13, 128, 3, 1, 1)
    x, dy = np.ldexp(synth.make_x(L, 4), e).astype(np.float32), np.ldexp(synth.make_dy(L, 4), f).astype(np.float32)
    (dw, _), names = ran(B, lambda: gpu_backward_weights(B, L, x, dy))
    assert any(n.startswith(KERNEL) for n in names), names
    want = oracle.conv_backward_weights(odims(oracle, L), x, dy)[0]
    assert np.linalg.norm(dw.astype(np.float64) - want) <= 8e-7 * np.linalg.norm(want)


def test_not_finite_inputs(B):
    """Infinities, NaN and values beyond bf16's range reach exactly the weights they reach in fp32."""
    L = layer("nf", 48, 192, 13, 13, 128, 3, 1, 1)
    x, dy = synth.make_x(L, 5), synth.make_dy(L, 5)
    x[0, 0, 0, 0], x[1, 1, 5, 6], x[1, 2, 12, 12], x[-1, 3, 4, 4] = np.inf, -np.inf, np.nan, 3.4e38
    dy[3, 7, 0, 0], dy[47, 9, 12, 12] = np.inf, 3.4e38
    dy[:, 11] = 0.0
    (got, _), names = ran(B, lambda: gpu_backward_weights(B, L, x, dy))
    assert any(n.startswith(KERNEL) for n in names), names
    want, _ = oracle.conv_backward_weights(odims(oracle, L), x, dy)
    assert (np.isnan(got) == np.isnan(want)).all()
    over = np.abs(want) > np.finfo(np.float32).max
    assert (np.isinf(got) == (over & ~np.isnan(want))).all()
    inf = np.isinf(got)
    assert (np.sign(got[inf]) == np.sign(want[inf])).all()
    ok = np.isfinite(got)
    big = ok & (np.abs(want) > 1e30)
    assert (np.abs(got[big] - want[big]) <= 1e-5 * np.abs(want[big])).all()
    assert rel_err(got[ok & ~big], want[ok & ~big]) <= TOL_F32


def test_more_weights_than_31_bits_count(B):
    """2.4e9 weights in one group: an index that passes through 32 bits turns negative from row 14564 on.
    Rows on both sides of it against 64-bit sums, and the floats in front of dw stay as they were."""
    import torch
    N, C, H, O, K = 32, 16384, 5, 16384, 3
    assert O * C * K * K > 2 ** 31
    rng = np.random.default_rng(9)
    x = rng.standard_normal((N, C, H, H), dtype=np.float32)
    dy = rng.standard_normal((N, O, H - K + 1, H - K + 1), dtype=np.float32)
    d = B.make_desc(N, C, H, H, O, K)
    ws = B.alloc_workspace(d, B.PASS_BACKWARD_WEIGHTS, N)
    front = 1 << 16
    buf = torch.full((front + O * C * K * K,), 7.0, device="cuda")
    dw = buf[front:].view(O, C, K, K)
    _, names = ran(B, lambda: (B.cct_conv_backward_weights(d, dev(x), dev(dy), dw, None, ws), torch.cuda.synchronize()))
    assert any(n.startswith(KERNEL) for n in names), names
    assert bool((buf[:front] == 7.0).all())
    rows = [0, 1, 14563, 14564, O - 1]
    win = np.lib.stride_tricks.sliding_window_view(x, (K, K), (2, 3)).astype(np.float64)   # [N][C][r][c][K][K]
    want = np.tensordot(dy[:, rows].astype(np.float64), win, ((0, 2, 3), (0, 2, 3)))       # [rows][C][K][K]
    assert rel_err(dw[rows].cpu().numpy(), want) <= TOL_F32


@pytest.mark.parametrize("L", [layer("r90", 42, 100, 14, 12, 90, 3, 1, 1), layer("r161", 35, 130, 11, 13, 322, 3, 1, 1, 2),
                               layer("r192", 32, 33, 9, 17, 192, 5, 1, 2)], ids=["r90", "r161", "r192"])
def test_tiles_of_96_rows(B, L):
    """Rows that end inside a tile, columns that end inside a stage of four; a tile's 96 rows are loaded as 128."""
    x, dy = synth.make_x(L, 5), synth.make_dy(L, 5)
    got, names = ran(B, lambda: gpu_backward_weights(B, L, x, dy))
    assert any(n.startswith(KERNEL + "<96") for n in names), names
    check(got, L, x, dy, TOL_F32)
    # every partial product in its place: a third term lost or misplaced is 2e-6, the sums (measured 1.2e-7) at most
    # what test_precision allows
    want = oracle.conv_backward_weights(odims(oracle, L), x, dy)[0]
    assert np.linalg.norm(got[0].astype(np.float64) - want) / np.linalg.norm(want) <= 8e-7


@pytest.mark.parametrize("L", [layer("few64", 27, 33, 11, 11, 9, 7, 4, 3), layer("few64_g", 119, 64, 14, 14, 16, 5, 1, 2),
                               layer("short86", 11, 17, 15, 15, 86, 7, 1, 3), layer("short112", 52, 64, 7, 7, 112, 7, 2, 3)],
                         ids=lambda L: L.name)
def test_tiles_of_64_rows(B, L):
    """Few kernels, and launches too short for larger tiles (14 against 50 us on a lowered matrix, 41 against 84; 25
    against 30 in a tile of 96 rows, 26 against 31 in one of 128)."""
    x, dy = synth.make_x(L, 6), synth.make_dy(L, 6)
    got, names = ran(B, lambda: gpu_backward_weights(B, L, x, dy))
    assert any(n.startswith(KERNEL + "<64") for n in names), names
    check(got, L, x, dy, TOL_F32)
