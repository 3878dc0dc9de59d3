"""Batched 1D stencils keep signals apart: non-finite values of one signal reach
no output of another, and within a signal only the outputs whose window holds
them."""
import numpy as np
import pytest

import oracle
from paper_1902_09931_amd import workloads as wl
from tests.gpu_util import TORCH, code, torch

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

# one to four taps, and the fewest and most of wider windows
TAPS = [(0, 0), (1, 0), (0, 1), (2, 1), (1, 3), (3, 3), (0, 6), (4, 5), (8, 8), (16, 0)]
# few signals (one vector per thread) and many (several), ends at every place in a vector
BATCHES = {"few": [40, 24, 33, 64, 29, 17, 41, 18, 512, 19], "many": [61, 64, 67, 18, 130, 33] * 8000}


def apply(v, offs, periodic, L, R, w, coe, dt):
    out = torch.zeros_like(v)
    p = b.mxs_create_1d_batch(offs, b.MXS_P if periodic else b.MXS_NP, code(dt), L, R, w, coe, v, out)
    b.mxs_compute(p)
    torch.cuda.synchronize()
    b.mxs_destroy(p)
    return out


@pytest.mark.parametrize("batch", list(BATCHES))
@pytest.mark.parametrize("L,R", TAPS)
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_neighbouring_signals_do_not_matter(dt, L, R, batch):
    offs = np.concatenate([[0], np.cumsum(BATCHES[batch])]).astype(np.int64)
    rng = np.random.default_rng(43)
    odd = torch.from_numpy(np.repeat(np.arange(len(offs) - 1) % 2 == 1, np.diff(offs))).cuda()
    v = torch.from_numpy(rng.uniform(-1, 1, offs[-1])).to(TORCH[dt]).cuda()
    w = rng.uniform(-1, 1, L + R + 1)
    for periodic in (True, False):
        for coe in (None, wl.CUBIC_MINUS_LINEAR):
            plain = apply(v, offs, periodic, L, R, w, coe, dt)
            for bad in (float("nan"), float("inf")):
                for side in (odd, ~odd):
                    got = apply(torch.where(side, torch.full_like(v, bad), v), offs, periodic, L, R, w, coe, dt)
                    assert torch.equal(got[~side], plain[~side])


@pytest.mark.parametrize("L,R", TAPS)
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_a_nan_reaches_the_windows_that_hold_it(dt, L, R):
    offs = np.concatenate([[0], np.cumsum(BATCHES["few"])]).astype(np.int64)
    rng = np.random.default_rng(47)
    w = rng.uniform(0.5, 1, L + R + 1)
    for at in (0, 1, 39, 40, 63, 64, 97, 161, 247, 265, 300, 301, int(offs[-1]) - 1):
        vals = rng.uniform(-1, 1, offs[-1])
        vals[at] = np.nan
        for periodic in (True, False):
            got = apply(torch.from_numpy(vals).to(TORCH[dt]).cuda(), offs, periodic, L, R, w, None, dt)
            ref = np.zeros_like(vals)
            oracle.stencil1d_batch(vals, offs, L, R, w, periodic, out=ref)
            assert np.array_equal(np.isnan(got.double().cpu().numpy()), np.isnan(ref)), at
