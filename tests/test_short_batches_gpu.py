"""Ragged batches on both sides of the rules that choose their launches: the
one-launch kernels bounded by class 4 (lines of at most 1024 elements) and by
class 16, and one launch per class for large batches."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import code, round_to, to_device, torch
from tests.test_solve_gpu import PENTA, TRI, check

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def solve(coef, lengths, dt, seed):
    rng = np.random.default_rng(seed)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    rhs = rng.uniform(-1, 1, offs[-1])
    dev = to_device(rhs, dt)
    out = torch.empty_like(dev)
    p = b.mxs_create_cyclic_solve(len(coef) - 1, coef, b.MXS_LINES_RAGGED, 0, 0, 0, offs, code(dt), dev, out)
    info = b.mxs_plan_info(p)
    b.mxs_compute(p)
    torch.cuda.synchronize()
    b.mxs_destroy(p)
    ref = oracle.cyclic_solve_batch(oracle.circulant_bands(coef), offs, round_to(rhs, dt))
    check(out.double().cpu().numpy(), ref, dt)
    return info


EDGES = [[5, 256, 257, 64, 512, 513, 1024, 1023],           # class 4 kernel
         [5, 1024, 1025, 300, 2048, 700],                   # class 8 present
         [4096, 6, 2049, 256, 4095],                        # class 16
         [700, 800], [256], [4096, 4095], [4097, 300, 40]]  # one class; long lines beside


@pytest.mark.parametrize("lengths", EDGES, ids=lambda v: "-".join(map(str, v)))
@pytest.mark.parametrize("coef", [TRI, PENTA], ids=["tri", "penta"])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_small_batches(dt, coef, lengths):
    solve(coef, lengths, dt, 3)


@pytest.mark.parametrize("coef,limit", [(TRI, 32768), (PENTA, 14000)], ids=["tri", "penta"])
def test_forms_on_both_sides_of_the_limit(coef, limit):
    lengths = np.random.default_rng(4).integers(5, 400, limit + 1)
    assert "form=units launches=1 " in solve(coef, lengths[:limit], "f64", 5)
    assert "form=classes launches=2 " in solve(coef, lengths, "f64", 5)
