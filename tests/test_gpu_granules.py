"""conv_granules (bf16 forward / backward-data on granules of 8 channels) at the sizes where it can go wrong,
against the oracle: the bf16 path's tolerance, and against the same operands rounded on the host, where
only fp32 accumulation is left."""
import numpy as np
import pytest

import oracle
from paper_1504_04343_amd import synth
from gpu_util import TOL_BF16, gpu_backward_data, gpu_forward, layer, odims, rel_err

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
