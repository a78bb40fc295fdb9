"""conv_fused_split (fp32 operands as sums of three bf16 terms): the forms of the kernel at the sizes
where they can go wrong, against the oracle.  The tolerance is the fp32 path's: six bf16 products hold
a product of two fp32 values to 2^-25, less than the rounding of one fp32 accumulation."""
import numpy as np
import pytest

import oracle
from paper_1504_04343_amd import synth
from gpu_util import TOL_F32, desc_of, dev, gpu_backward_data, gpu_forward, layer, odims, rel_err

pytestmark = pytest.mark.gpu

KERNEL = "conv_fused_split"

#       name        N   C    H   W    O  K  s  p  g
FORWARD = [
    layer("m32",    2,  16,  9, 11,  36, 3, 1, 1),           # 32-row tiles, rows to spare
    layer("m16",    3,  80, 12, 14,  16, 3, 1, 1),           # half of a 32-row tile
    layer("m64",    7,  32, 13, 13,  64, 3, 1, 1),           # 64-row tile, tiles across images
    layer("m128",  33,  40, 13, 13, 128, 3, 1, 1, 2),        # channels past a group's last one
    layer("m192",  26,  16, 28, 28, 192, 3, 1, 0),           # rows no multiple of 128, one channel group
    layer("c9",     3,   9, 12, 17,  61, 3, 1, 2),           # channels that fill half of a group
    layer("k2",     5,  48, 10, 10,  40, 2, 1, 1),           # four taps
    layer("k4",     2,  24, 15, 12,  70, 4, 1, 2),
    layer("k5",     4,  48, 27, 27, 130, 5, 1, 2),           # tiles cut per image
    layer("k7",     2,  16, 37, 40,  36, 7, 1, 3),           # odd tap count: zero tile; three cells per thread
    layer("k6",     3,  20, 14, 14,  44, 6, 1, 0),
    layer("wide",   2,  16, 14, 56,  64, 3, 1, 1),           # one workgroup per CU
    layer("s2cells", 3, 32, 15, 17,  48, 3, 2, 1),           # strided windows over the tensor's own cells
    layer("s2d2",   5,  16, 57, 57,  40, 5, 2, 0),           # space to depth by 2 (three taps), odd plane
    layer("s2d2p",  5,  12, 57, 56,  64, 3, 2, 1),           # two taps, padded
    layer("s2d2k7", 4,   6, 64, 61,  37, 7, 2, 3),           # four taps
    layer("s2d4",   5,   3, 63, 65,  96, 11, 4, 0),
    layer("s2d4p",  4,   2, 64, 63,  40, 8, 4, 3),
    layer("s2d4one", 1,  3, 67, 67,  36, 11, 4, 2),          # the tensor's only image
]
BACKWARD = [
    layer("b20",    3,  20,  9, 11,  64, 3, 1, 1),           # part of a 32-row tile
    layer("b32",    2,  36,  9, 11,  16, 3, 1, 1),
    layer("b128",  33, 128, 13, 13,  40, 3, 1, 1),
    layer("b_k5",   4,  48, 27, 27,  64, 5, 1, 2),
    layer("b_p0",   3,  33, 12, 10,  25, 4, 1, 0),
    layer("b_s4",   3,   3, 63, 65,  32, 11, 4, 0),          # depth to space, 16-byte stores
    layer("b_s2",   4,  20, 21, 23,  48, 3, 2, 1),
    layer("b_s3",   4,  10, 21, 23,  48, 5, 3, 2),
]


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_1504_04343_amd import binding
    return binding


def ran(B, call):
    """The call's result and the names of the kernels it launched."""
    B.cct_profile_enable(True)
    got = call()
    B.cct_profile_enable(False)
    return got, [e["name"] for e in B.cct_profile_read()]


def ids(layers):
    return [L.name for L in layers]


@pytest.mark.parametrize("L", FORWARD, ids=ids(FORWARD))
def test_forward(B, L):
    x, w, b = synth.make_x(L, 3), synth.make_w(L, 3), synth.make_bias(L, 3)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, b, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL) for n in names), names
    assert rel_err(got, oracle.conv_forward(odims(oracle, L), x, w, b)) <= TOL_F32


@pytest.mark.parametrize("L", BACKWARD, ids=ids(BACKWARD))
def test_backward_data(B, L):
    w, dy = synth.make_w(L, 3), synth.make_dy(L, 3)
    got, names = ran(B, lambda: gpu_backward_data(B, L, w, dy, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL) for n in names), names
    assert rel_err(got, oracle.conv_backward_data(odims(oracle, L), w, dy)) <= TOL_F32


def test_precision(B):
    """Closer to 64 bits than an fp32 accumulation of 2304 products can be expected to come: an MFMA's sums of 16
    products measure 2.3e-7 (2-norm) as one chain and less in parts, sums of 2 products 6e-7."""
    L = layer("prec", 8, 256, 13, 13, 128, 3, 1, 1, x_dist="relu_normal")
    x, w = synth.make_x(L, 1), synth.make_w(L, 1)
    got = gpu_forward(B, L, x, w, None, B.LOWER_FUSED).astype(np.float64)
    want = oracle.conv_forward(odims(oracle, L), x, w, None)
    assert np.linalg.norm(got - want) / np.linalg.norm(want) <= 4e-7


@pytest.mark.parametrize("L", [layer("p32", 11, 96, 27, 27, 256, 5, 1, 2, 2), layer("p64", 49, 384, 13, 13, 256, 3, 1, 1, 2),
                               layer("p_k7", 6, 80, 28, 28, 352, 7, 2, 3)], ids=lambda L: L.name)
def test_precision_of_small_layers(B, L):
    """32- and 64-row tiles sum the contraction in parts of 8 pairs of tiles (K = 7) or 9 to 25 tiles.  The error of a
    part is a random walk, at most 2^-24 / sqrt(3) * sqrt(25 / 2) = 1.2e-7 of the part's sum, and falls with the root of
    the number of parts, whose own sum adds as much again at most; as one chain of 200 to 350 roundings these come out
    at 2e-7 to 4e-7."""
    rng = np.random.default_rng(7)
    w = rng.standard_normal((L.O, L.C // L.groups, L.K, L.K), dtype=np.float32)
    dy = rng.standard_normal((L.N, L.O, L.Hout, L.Wout), dtype=np.float32)
    got, names = ran(B, lambda: gpu_backward_data(B, L, w, dy, B.LOWER_FUSED))
    assert any(n.startswith((KERNEL + "<1, 2", KERNEL + "<2, 2")) for n in names), names
    want = oracle.conv_backward_data(odims(oracle, L), w, dy)
    assert np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want) <= 1.5e-7


def test_images_larger_than_their_regrouped_form(B):
    """Stride 4, 8 x 8 kernels, 11 x 11 pixels: only 8 x 8 of them are read, but the 128 images of a workgroup lie
    19.4 MB apart.  Whole numbers with sums below 2^24: exact in any order."""
    import torch
    L = layer("apart", 129, 40000, 11, 11, 16, 8, 4, 0)
    gen = torch.Generator(device="cuda").manual_seed(5)
    ints = lambda lo, hi, *shape: torch.randint(lo, hi, shape, generator=gen, device="cuda", dtype=torch.float32)
    x, w, b = ints(-1, 2, L.N, L.C, L.H, L.W), ints(-2, 3, L.O, L.C, L.K, L.K), ints(-9, 10, L.O)
    y = torch.full((L.N, L.O, 1, 1), float("nan"), device="cuda")
    d = desc_of(B, L, B.LOWER_FUSED)
    B.cct_conv_forward(d, x, w, b, y, B.alloc_workspace(d, B.PASS_FORWARD, None))
    want = b.double().expand(L.N, L.O).clone()
    for c in range(0, L.C, 4000):
        want += x[:, c:c + 4000, :8, :8].reshape(L.N, -1).double() @ w[:, c:c + 4000].reshape(L.O, -1).double().T
    assert torch.equal(y.double().view(L.N, L.O), want)


@pytest.mark.parametrize("e,f", [(-118, 88), (-70, 40), (70, -50), (103, -83), (110, -90)], ids=lambda e: "2^%d" % e)
@pytest.mark.parametrize("L", [layer("r_k3", 2, 40, 13, 13, 70, 3, 1, 1), layer("r_s2d", 2, 3, 31, 31, 40, 11, 4, 0)],
                         ids=lambda L: L.name)
def test_range_of_fp32(B, L, e, f):
    """An operand of any magnitude that fp32 holds keeps its 24 bits (2^-118: the terms' last bits would lie below
    bf16's smallest number; 2^103 and 2^110: values that do not scale), the other one brings the results to 2^-30 or 2^20.
    The bound is that of an fp32 chain of 400 products, 2^-24 / sqrt(3) * sqrt(400 / 2)."""
    x, w = synth.make_x(L, 4), synth.make_w(L, 4)
    x, w = np.ldexp(x, e).astype(np.float32), np.ldexp(w, f).astype(np.float32)
    dy = np.ldexp(synth.make_dy(L, 4), e).astype(np.float32)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, None, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL) for n in names), names
    want = oracle.conv_forward(odims(oracle, L), x, w, None)
    assert np.linalg.norm(got.astype(np.float64) - want) <= 5e-7 * np.linalg.norm(want)
    got, names = ran(B, lambda: gpu_backward_data(B, L, w, dy, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL) for n in names), names
    want = oracle.conv_backward_data(odims(oracle, L), w, dy)
    assert np.linalg.norm(got.astype(np.float64) - want) <= 5e-7 * np.linalg.norm(want)


SPECIAL = [("plain", layer("nf", 3, 16, 13, 13, 40, 3, 1, 1)),
           ("s2d", layer("nf2", 3, 3, 31, 31, 40, 7, 4, 0)),
           ("zero_tile", layer("nf7", 2, 16, 13, 13, 40, 7, 1, 3))]


@pytest.mark.parametrize("L", [L for _, L in SPECIAL], ids=[n for n, _ in SPECIAL])
def test_not_finite_inputs(B, L):
    """Infinities, NaN and values beyond bf16's range reach exactly the outputs they reach in fp32."""
    x, w, b = synth.make_x(L, 5), synth.make_w(L, 5), synth.make_bias(L, 5)
    x[0, 0, 0, 0], x[1, 1, 5, 6], x[1, 2, 12, 12], x[-1, 1, 4, 4] = np.inf, -np.inf, np.nan, 3.4e38
    x[0, 2, 9, 9] = np.float32(1e38)
    w[3, 1, 1, 2], w[7, 0, 0, 0], w[9, 0, 2, 2] = np.inf, np.nan, 3.4e38
    w[11] = 0.0
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, b, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL) for n in names), names
    od = odims(oracle, L)
    want = oracle.conv_forward(od, x, w, b)
    assert (np.isnan(got) == np.isnan(want)).all()
    over = np.abs(want) > np.finfo(np.float32).max     # infinite, or beyond fp32
    assert (np.isinf(got) == (over & ~np.isnan(want))).all()
    inf = np.isinf(got)
    assert (np.sign(got[inf]) == np.sign(want[inf])).all()
    ok = np.isfinite(got)
    big = ok & (np.abs(want) > 1e30)
    assert (np.abs(got[big] - want[big]) <= 1e-5 * np.abs(want[big])).all()
    assert rel_err(got[ok & ~big], want[ok & ~big]) <= TOL_F32


def check_not_finite(got, want):
    """got: fp32, want: 64 bits."""
    assert (np.isnan(got) == np.isnan(want)).all()
    over = np.abs(want) > np.finfo(np.float32).max
    assert (np.isinf(got) == (over & ~np.isnan(want))).all()
    inf = np.isinf(got)
    assert (np.sign(got[inf]) == np.sign(want[inf])).all()
    ok = np.isfinite(got)
    big = ok & (np.abs(want) > 1e30)
    assert (np.abs(got[big] - want[big]) <= 1e-5 * np.abs(want[big])).all()
    assert rel_err(got[ok & ~big], want[ok & ~big]) <= TOL_F32


@pytest.mark.parametrize("L", [layer("nf_s1", 3, 40, 13, 13, 16, 3, 1, 1), layer("nf_k4", 3, 33, 12, 10, 25, 4, 1, 0),
                               layer("nf_s2", 3, 20, 21, 23, 48, 3, 2, 1), layer("nf_s4", 3, 3, 31, 33, 32, 11, 4, 0)],
                         ids=lambda L: L.name)
def test_not_finite_backward_data(B, L):
    w, dy = synth.make_w(L, 5), synth.make_dy(L, 5)
    dy[0, 0, 0, 0], dy[1, 1, 2, 3], dy[1, 2, -1, -1], dy[-1, 1, 1, 1] = np.inf, -np.inf, np.nan, 3.4e38
    w[3, 1, 1, 2], w[7, 0, 0, 0], w[9, 2, 2, 2] = np.inf, np.nan, 3.4e38
    got, names = ran(B, lambda: gpu_backward_data(B, L, w, dy, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL) for n in names), names
    check_not_finite(got, oracle.conv_backward_data(odims(oracle, L), w, dy))


@pytest.mark.parametrize("value", [np.inf, np.nan], ids=["inf", "nan"])
@pytest.mark.parametrize("L", [layer("d_s1", 3, 40, 13, 13, 40, 3, 1, 1), layer("d_s2", 3, 20, 21, 23, 48, 3, 2, 1)],
                         ids=lambda L: L.name)
def test_many_not_finite_values(B, L, value):
    """Some values everywhere and all of one image: blocks in which many or all results are not finite."""
    x, w, dy = synth.make_x(L, 5), synth.make_w(L, 5), synth.make_dy(L, 5)
    for t in (x, dy):
        t.reshape(-1)[::701] = value
        t[1] = value
        t[2] = np.abs(t[2])                    # infinities of one sign there
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, None, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL) for n in names), names
    check_not_finite(got, oracle.conv_forward(odims(oracle, L), x, w, None))
    check_not_finite(gpu_backward_data(B, L, np.abs(w), dy, B.LOWER_FUSED),
                     oracle.conv_backward_data(odims(oracle, L), np.abs(w), dy))


def test_workspace_for_the_fp32_kernel_matrix_is_still_enough(B):
    """A workspace that holds the fp32 kernel matrix but not its three terms runs the fp32 kernel."""
    import torch
    L = layer("ws", 4, 64, 13, 13, 128, 3, 1, 1)
    x, w, b = synth.make_x(L, 3), synth.make_w(L, 3), synth.make_bias(L, 3)
    d = desc_of(B, L, B.LOWER_FUSED)
    full = B.cct_conv_workspace_bytes(d, B.PASS_FORWARD)
    ws = torch.empty(full * 2 // 3, dtype=torch.uint8, device="cuda")
    y = torch.full((L.N, L.O, L.Hout, L.Wout), float("nan"), device="cuda")
    _, names = ran(B, lambda: (B.cct_conv_forward(d, dev(x), dev(w), dev(b), y, ws), torch.cuda.synchronize()))
    assert not any(n.startswith(KERNEL) for n in names), names
    assert rel_err(y.cpu().numpy(), oracle.conv_forward(odims(oracle, L), x, w, b)) <= TOL_F32


# The 2-norm error of up to 1600 products with every partial product in its place: the six bf16 products hold 2^-25 of
# each, the chain of at most 75 roundings 2^-24 / sqrt(3) * sqrt(75 / 2) = 2.1e-7.  A third term lost or read from the
# wrong place is 2^-18 / sqrt(3) of a product and more, 2e-6; m * m left out 1e-6.
ALL_TERMS = 3e-7


def norm_err(got, want):
    return np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want)


# tiles of 128 and 96 rows (256 column tiles), rows to spare, one channel group and an odd number of them
FORMS = [layer("t96", 200, 24, 13, 13, 96, 3, 1, 1), layer("t80_k5", 200, 16, 13, 13, 80, 5, 1, 2),
         layer("t96_k4", 200, 40, 13, 13, 90, 4, 1, 2), layer("t96_s2d", 150, 3, 67, 67, 96, 11, 4, 0),
         layer("t128_k5", 200, 48, 13, 13, 128, 5, 1, 2), layer("t128_k2", 240, 16, 13, 13, 128, 2, 1, 0),
         layer("t64_k5", 200, 48, 13, 13, 60, 5, 1, 2), layer("t32_k3", 9, 80, 13, 13, 30, 3, 1, 1)]


@pytest.mark.parametrize("L", FORMS, ids=ids(FORMS))
def test_row_tiles(B, L):
    x, w, b = synth.make_x(L, 6), synth.make_w(L, 6), synth.make_bias(L, 6)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, b, B.LOWER_FUSED))
    form = {"t96": "<2, 3", "t80": "<2, 3", "t12": "<4, 2", "t64": "<2, 2", "t32": "<1, 2"}[L.name[:3]]
    assert any(n.startswith(KERNEL + form) for n in names), names
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    assert rel_err(got, want) <= TOL_F32
    assert norm_err(got, want) <= ALL_TERMS
    # values that are not finite, met by whole tiles and by the rows and positions of another wave
    x[0, 0, 0, 0], x[1, 1, 5, 6], x[-1, 2, 12, 12], w[3, 1, 1, 1], w[-1, 0, 0, 0] = np.inf, -np.inf, np.nan, 3.4e38, np.inf
    check_not_finite(gpu_forward(B, L, x, w, b, B.LOWER_FUSED), oracle.conv_forward(odims(oracle, L), x, w, b))


# The form of the kernel by what a launch holds: unrolled taps in blocks of 32 x 32 on 32 rows and for workgroups that have
# their CU alone (few of them, or cells that fill more than half of the LDS), pairs of taps in blocks of 16 x 16 for others.
BLOCKS = [(layer("lone32_k3", 4, 64, 28, 28, 128, 3, 1, 1), "<1, 2, 3, 1, 32>"),
          (layer("lone32_k5", 2, 48, 27, 27, 128, 5, 1, 2), "<1, 2, 5, 1, 32>"),
          (layer("lone32_s2d", 2, 32, 27, 27, 40, 5, 2, 2), "<1, 2, 3, 2, 32>"),
          (layer("lone32_s4", 1, 3, 67, 67, 36, 11, 4, 0), "<1, 2, 3, 4, 32>"),
          (layer("lone64_k3", 50, 40, 27, 27, 60, 3, 1, 1), "<2, 2, 3, 1, 32>"),
          (layer("lone64_k5", 50, 32, 27, 27, 60, 5, 1, 2), "<2, 2, 5, 1, 32>"),
          (layer("wide64", 20, 16, 40, 88, 60, 3, 1, 1), "<2, 2, 3, 1, 32>"),
          (layer("wide128", 8, 16, 64, 88, 128, 3, 1, 1), "<4, 2, 3, 1, 32>"),
          (layer("pairs64_k3", 68, 40, 27, 27, 60, 3, 1, 1), "<2, 2, 3, 1, 16>"),
          (layer("pairs128_k3", 200, 16, 13, 13, 128, 3, 1, 1), "<4, 2, 3, 1, 16>"),
          (layer("long64_k5", 180, 64, 27, 27, 40, 5, 1, 2), "<2, 2, 5, 1, 16>"),
          (layer("long128_k5", 200, 48, 13, 13, 128, 5, 1, 2), "<4, 2, 5, 1, 16>")]


@pytest.mark.parametrize("L,form", BLOCKS, ids=[L.name for L, _ in BLOCKS])
def test_form_follows_the_launch(B, L, form):
    x, w, b = synth.make_x(L, 7), synth.make_w(L, 7), synth.make_bias(L, 7)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, b, B.LOWER_FUSED))
    assert any(n == KERNEL + form for n in names), names
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    assert rel_err(got, want) <= TOL_F32
    assert norm_err(got, want) <= ALL_TERMS


@pytest.mark.parametrize("L,form", [(layer("rows450", 200, 16, 13, 13, 450, 3, 1, 1), "<2, 3, 3, 1, 16>"),
                                    (layer("rows449", 240, 32, 13, 13, 449, 3, 1, 1), "<4, 2, 3, 1, 16>"),
                                    (layer("rows464_few", 24, 16, 17, 17, 464, 3, 1, 1), "<2, 2, 3, 1, 16>"),
                                    (layer("rows470_k2", 200, 16, 13, 13, 470, 2, 1, 0), "<4, 2, 0, 1, 16>")],
                         ids=lambda v: v.name if hasattr(v, "name") else v)
def test_rows_that_96_and_128_fill(B, L, form):
    """Five tiles of 96 rows or four of 128: the one with the lower estimate, smaller tiles where four leave CUs empty."""
    x, w = synth.make_x(L, 8), synth.make_w(L, 8)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, None, B.LOWER_FUSED))
    assert any(n == KERNEL + form for n in names), names
    want = oracle.conv_forward(odims(oracle, L), x, w, None)
    assert rel_err(got, want) <= TOL_F32
    assert norm_err(got, want) <= ALL_TERMS


# Backward-data on tiles of 96 rows: stride 1, two groups, and the strided form, whose rows are channels x residues and
# whose results are stored depth to space (stride 2: rows 48 .. 95 belong to the waves whose last 16 rows are a half-filled
# block of the repair; stride 3: rows that end inside a quad)
BACKWARD_96 = [layer("b96", 200, 96, 13, 13, 40, 3, 1, 1), layer("b90_g", 130, 180, 13, 13, 64, 5, 1, 2, 2),
               layer("b96_k4", 200, 70, 13, 13, 24, 4, 1, 2), layer("b96_s2", 200, 24, 26, 26, 48, 3, 2, 1),
               layer("b90_s3", 200, 10, 39, 39, 40, 5, 3, 1), layer("b80_s4", 150, 5, 60, 60, 32, 8, 4, 2)]


@pytest.mark.parametrize("L", BACKWARD_96, ids=ids(BACKWARD_96))
def test_backward_data_on_96_rows(B, L):
    w, dy = synth.make_w(L, 6), synth.make_dy(L, 6)
    got, names = ran(B, lambda: gpu_backward_data(B, L, w, dy, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL + "<2, 3") for n in names), names
    want = oracle.conv_backward_data(odims(oracle, L), w, dy)
    assert rel_err(got, want) <= TOL_F32
    assert norm_err(got, want) <= ALL_TERMS
    # values that are not finite, in every block of a wave's rows
    dy[0, 0, 0, 0], dy[1, 1, 5, 6], dy[-1, 2, -1, -1] = np.inf, -np.inf, np.nan
    w[3, 1, 1, 1], w[5, -1, 0, 0], w[7, L.C // L.groups // 2, 1, 0] = 3.4e38, np.inf, np.nan
    check_not_finite(gpu_backward_data(B, L, w, dy, B.LOWER_FUSED), oracle.conv_backward_data(odims(oracle, L), w, dy))


def test_forward_on_96_rows_in_groups(B):
    L = layer("g96", 130, 40, 13, 13, 190, 3, 1, 1, 2)
    x, w, b = synth.make_x(L, 6), synth.make_w(L, 6), synth.make_bias(L, 6)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, b, B.LOWER_FUSED))
    assert any(n.startswith(KERNEL + "<2, 3") for n in names), names
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    assert rel_err(got, want) <= TOL_F32
    assert norm_err(got, want) <= ALL_TERMS


# tiles of 48 x 192: rows to spare, positions cut per image and across images, one channel group and an odd number, three
# row tiles, three images in a tile
ROWS_48 = [
    layer("k5_48", 80, 24, 27, 27, 90, 5, 1, 2, 2),
    layer("k3_48", 150, 33, 25, 23, 48, 3, 1, 1),
    layer("k3_144", 200, 20, 19, 24, 143, 3, 1, 0),
    layer("small_48", 870, 48, 12, 9, 41, 3, 1, 1),
]


def on_48(names):
    return any(n.startswith("conv_fused_split<1, 3, ") for n in names)


@pytest.mark.parametrize("L", ROWS_48, ids=ids(ROWS_48))
def test_forward_on_48_rows(B, L):
    x, w, b = synth.make_x(L, 6), synth.make_w(L, 6), synth.make_bias(L, 6)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, b, B.LOWER_FUSED))
    assert on_48(names), names
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    assert rel_err(got, want) <= TOL_F32 and norm_err(got, want) <= ALL_TERMS


BACKWARD_48 = [layer("b_k5_48", 60, 96, 27, 27, 40, 5, 1, 2, 2), layer("b_s4_48", 150, 3, 83, 95, 40, 11, 4, 0)]


@pytest.mark.parametrize("L", BACKWARD_48, ids=ids(BACKWARD_48))
def test_backward_data_on_48_rows(B, L):
    w, dy = synth.make_w(L, 6), synth.make_dy(L, 6)
    got, names = ran(B, lambda: gpu_backward_data(B, L, w, dy, B.LOWER_FUSED))
    assert on_48(names), names
    want = oracle.conv_backward_data(odims(oracle, L), w, dy)
    assert rel_err(got, want) <= TOL_F32 and norm_err(got, want) <= ALL_TERMS


@pytest.mark.parametrize("L", [ROWS_48[0], ROWS_48[1]], ids=["k5_48", "k3_48"])
def test_not_finite_inputs_on_48_rows(B, L):
    """A wave's 48 positions are a block of 32 and half a block whose other half is another wave's."""
    x, w = synth.make_x(L, 5), synth.make_w(L, 5)
    x[0, 1, 1, 9], x[3, 0, 2, 20], x[7, 2, 11, 11], x[-1, 1, -1, -1] = np.inf, -np.inf, np.nan, np.inf
    w[33, 1, 1, 1], w[2, 0, 0, 2] = np.inf, np.nan
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, None, B.LOWER_FUSED))
    assert on_48(names), names
    check_not_finite(got, oracle.conv_forward(odims(oracle, L), x, w, None))


# tiles of 64 x 160: positions across images and cut per image, rows to spare, channels past a group's last one
WIDE_64 = [layer("wide_k3", 95, 140, 26, 27, 59, 3, 1, 1), layer("wide_k5", 44, 260, 27, 27, 100, 5, 1, 2, 2)]


@pytest.mark.parametrize("L", WIDE_64, ids=ids(WIDE_64))
def test_forward_on_160_positions(B, L):
    x, w, b = synth.make_x(L, 6), synth.make_w(L, 6), synth.make_bias(L, 6)
    got, names = ran(B, lambda: gpu_forward(B, L, x, w, b, B.LOWER_FUSED))
    assert any("wide" in n for n in names), names
    want = oracle.conv_forward(odims(oracle, L), x, w, b)
    assert rel_err(got, want) <= TOL_F32 and norm_err(got, want) <= ALL_TERMS
    x[0, 1, 1, 9], x[3, 0, 2, 20], x[7, 2, 11, 11], w[33, 1, 1, 1], w[2, 0, 0, 2] = np.inf, -np.inf, np.nan, np.inf, np.nan
    check_not_finite(gpu_forward(B, L, x, w, None, B.LOWER_FUSED), oracle.conv_forward(odims(oracle, L), x, w, None))
