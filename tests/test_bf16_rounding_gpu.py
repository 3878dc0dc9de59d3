"""Stores to bfloat16 round to nearest, ties to even, bit for bit as the integer
formula does, over ties, subnormals, the overflow edge, infinities and NaN."""
import numpy as np
import pytest

from tests.gpu_util import torch

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def rounded(f):
    """Nearest-even bfloat16 bits of float32 values; a NaN keeps its sign and top
    bits and becomes quiet."""
    u = f.view(np.uint32).astype(np.uint64)
    up = ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    return np.where(np.isnan(f), ((u >> 16) | 0x40).astype(np.uint16), up)


def bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def stencil(values, coe, dt, dst):
    """A 1 x 1 window of weight 1, with the point function: float arithmetic, one
    rounding into the storage type."""
    n = values.numel()
    out = torch.zeros(n, dtype=dst, device="cuda")
    p = b.mxs_create_2d(n, 1, n, b.MXS_X, b.MXS_P, dt, 0, 0, 0, 0, [1.0], coe, values, out)
    b.mxs_compute(p)
    torch.cuda.synchronize()
    b.mxs_destroy(p)
    return out


def every_bf16():
    return torch.from_numpy(np.arange(1 << 16, dtype=np.uint16).view(np.int16).copy()).cuda().view(torch.bfloat16)


def test_identity_returns_every_value():
    x = every_bf16()
    got, want = bits(stencil(x, None, b.MXS_BF16, torch.bfloat16)), bits(x)
    nan = np.isnan(x.float().cpu().numpy())
    assert np.array_equal(got[~nan] & 0x7fff, want[~nan] & 0x7fff)         # -0 + 0 is +0
    assert np.array_equal(got[~nan][want[~nan] != 0x8000], want[~nan][want[~nan] != 0x8000])
    assert np.isnan(stencil(x, None, b.MXS_BF16, torch.bfloat16).float().cpu().numpy())[nan].all()


# f(c) = c0 + c1 c with exact constants: scalings onto ties and odd remainders
# (257 / 256 and 129 / 128 of 8-bit mantissas), into the subnormals, up to and
# past the largest value
@pytest.mark.parametrize("c0,c1", [(0.0, 257.0 / 256), (0.0, 129.0 / 128), (0.0, 0.99609375), (0.0, 1.0 + 2.0 ** -16),
                                   (0.0, 2.0 ** -120), (0.0, 3.0 * 2.0 ** -110), (0.0, 2.0 ** 120),
                                   (0.0, 1.99609375), (0.0, 1.998046875), (2.0 ** -130, 257.0 / 256),
                                   (1.0, 2.0 ** -9), (-1.0, 2.0 ** -9), (float("inf"), 1.0)])
def test_rounding_of_computed_values(c0, c1):
    x = every_bf16()
    got = bits(stencil(x, [c0, c1], b.MXS_BF16, torch.bfloat16))
    with np.errstate(all="ignore"):
        # c1 c + c0 rounded once to float: c1 c is exact in double here, and where
        # c0 is not zero it is exact in float too, so a fused and an unfused
        # evaluation agree
        f = (np.float64(c1) * x.double().cpu().numpy() + np.float64(c0)).astype(np.float32)
    want = rounded(f)
    nan = np.isnan(f)
    assert np.array_equal(got[nan] & 0x7f80, np.full(nan.sum(), 0x7f80)) and ((got[nan] & 0x7f) != 0).all()
    same = got[~nan] == want[~nan]
    zero = (want[~nan] & 0x7fff) == 0
    assert (same | (zero & ((got[~nan] & 0x7fff) == 0))).all()


def test_neighbours_in_a_vector_do_not_matter():
    """Values are converted two at a time."""
    rng = np.random.default_rng(89)
    x = every_bf16()[torch.from_numpy(rng.permutation(1 << 16)).cuda()]
    coe = [0.0, 257.0 / 256]
    a = bits(stencil(x, coe, b.MXS_BF16, torch.bfloat16))
    c = bits(stencil(x.roll(1), coe, b.MXS_BF16, torch.bfloat16))
    nan = np.isnan(x.float().cpu().numpy())
    assert np.array_equal(a[~nan], np.roll(c, -1)[~nan])
