"""conv_granules (bf16 forward / backward-data on granules of 8 channels) at the sizes where it can go wrong,
against the oracle: the bf16 path's tolerance, and against the same operands rounded on the host, where
only fp32 accumulation is left."""
import numpy as np
import pytest

import oracle
from paper_1504_04343_amd import synth
from gpu_util import TOL_BF16, dev, gpu_backward_data, gpu_forward, layer, odims, rel_err

pytestmark = pytest.mark.gpu

KERNEL = "conv_granules"

#          name       N    C   H   W    O  K  s  p  g
FORWARD = [
    layer("m128",    64, 128, 13, 13, 128, 3, 1, 1),
    layer("m64",     70,  64, 17, 13, 192, 3, 1, 1),          # 64-row tiles, tiles across images
    layer("odd",     33, 106, 21, 19, 130, 5, 1, 2, 2),       # 53 channels a group: a granule of 5; 65 rows
    layer("stride",  40,  96, 25, 23, 100, 3, 2, 1),
    layer("k1",      64, 200, 20, 14,  70, 1, 1, 0),          # a single tap
    layer("k1s2",    64, 176, 28, 28,  32, 1, 2, 0),
    layer("k11",     14,   3, 99, 95,  96, 11, 4, 0),         # three channels, 121 taps
]
BACKWARD = [
    layer("b_m128",  64, 128, 13, 13, 128, 3, 1, 1),
    layer("b_odd",   33, 106, 21, 19, 130, 5, 1, 2, 2),
    layer("b_p0",    50,  70, 17, 18, 120, 3, 1, 0),
    layer("b_k1",    64,  70, 20, 14, 200, 1, 1, 0),
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


def rounded(a):
    """The values as bf16, round to nearest even."""
    u = a.view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) >> 16 << 16).astype(np.uint32).view(np.float32).reshape(a.shape)


# A sum of up to 1600 exact products of bf16 values in fp32, one rounding per 16: far below 1e-5 of the largest.
TOL_ROUNDED = 1e-5


@pytest.mark.parametrize("chunk", [None, 33, 8], ids=["whole", "chunks", "small"])
@pytest.mark.parametrize("L", FORWARD, ids=[L.name for L in FORWARD])
def test_forward(B, L, chunk):
    if chunk and chunk > L.N:
        chunk = L.N
    x, w, b = synth.make_x(L, 3), synth.make_w(L, 3), synth.make_bias(L, 3)
    for bias in (b, None):
        got, names = ran(B, lambda: gpu_forward(B, L, x, w, bias, 0, 1, chunk=chunk))
        if chunk is None:
            assert any(n.startswith(KERNEL) for n in names), names
        assert rel_err(got, oracle.conv_forward(odims(oracle, L), x, w, bias)) <= TOL_BF16
        assert rel_err(got, oracle.conv_forward(odims(oracle, L), rounded(x), rounded(w), bias)) <= TOL_ROUNDED


@pytest.mark.parametrize("L", BACKWARD, ids=[L.name for L in BACKWARD])
def test_backward_data(B, L):
    w, dy = synth.make_w(L, 3), synth.make_dy(L, 3)
    got, names = ran(B, lambda: gpu_backward_data(B, L, w, dy, 0, 1))
    assert any(n.startswith(KERNEL) for n in names), names
    assert rel_err(got, oracle.conv_backward_data(odims(oracle, L), w, dy)) <= TOL_BF16
    assert rel_err(got, oracle.conv_backward_data(odims(oracle, L), rounded(w), rounded(dy))) <= TOL_ROUNDED


def pass_bytes(L, backward, images):
    """Workspace of the granules of so many images and of the kernels."""
    C, M, P = (L.O, L.C, L.Hout + 2 * (L.K - 1 - L.pad)) if backward else (L.C, L.O, L.H + 2 * L.pad)
    Q = L.Wout + 2 * (L.K - 1 - L.pad) if backward else L.W + 2 * L.pad
    n8, up = -(-C // L.groups // 8), lambda v: -(-v // 256) * 256
    return up(images * L.groups * n8 * P * Q * 16) + up(n8 * L.K ** 2 * M * 16)


@pytest.mark.parametrize("backward,L", [(False, FORWARD[3]), (False, FORWARD[4]),
                                        (True, layer("b_odd", 73, 106, 21, 19, 130, 5, 1, 2, 2))],
                         ids=lambda v: getattr(v, "name", None))
def test_in_chunks(B, backward, L):
    """A workspace for 37 images (33 of the 40): granules, with a last chunk shorter than the first.  One for less
    than 32: the other kernels."""
    import torch
    x, w, b, dy = (m(L, 3) for m in (synth.make_x, synth.make_w, synth.make_bias, synth.make_dy))
    d = B.make_desc(L.N, L.C, L.H, L.W, L.O, L.K, L.stride, L.pad, L.groups, 0, 1)
    p = B.PASS_BACKWARD_DATA if backward else B.PASS_FORWARD
    assert pass_bytes(L, backward, L.N) == B.cct_conv_workspace_bytes(d, p)
    for images in (min(37, L.N - 7), 31):
        ws = torch.empty(pass_bytes(L, backward, images), dtype=torch.uint8, device="cuda")
        out = torch.full((x if backward else dy).shape, float("nan"), device="cuda")
        B.cct_profile_enable(True)
        if backward:
            B.cct_conv_backward_data(d, dev(w), dev(dy), out, ws)
        else:
            B.cct_conv_forward(d, dev(x), dev(w), dev(b), out, ws)
        torch.cuda.synchronize()
        B.cct_profile_enable(False)
        launches = sum(e["launches"] for e in B.cct_profile_read() if e["name"].startswith(KERNEL))
        assert launches == (2 if images > 31 else 0)
        for f, tol in ((lambda a: a, TOL_BF16), (rounded, TOL_ROUNDED)):
            want = (oracle.conv_backward_data(odims(oracle, L), f(w), f(dy)) if backward else
                    oracle.conv_forward(odims(oracle, L), f(x), f(w), b))
            assert rel_err(out.cpu().numpy(), want) <= tol
