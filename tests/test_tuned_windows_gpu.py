"""Layouts tuned for one window serve only windows that can run in them."""
import numpy as np
import pytest

from tests.gpu_util import code, to_device, torch
from tests.test_stencil_gpu import DIRS, check_against_oracle

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("direction,windows", [
    ("X", [(1, 1, 0, 0), (2, 0, 0, 0), (0, 1, 0, 0)]), ("X", [(2, 2, 0, 0), (3, 1, 0, 0), (0, 4, 0, 0)]),
    ("X", [(4, 4, 0, 0), (8, 0, 0, 0), (3, 3, 0, 0)]), ("XY", [(1, 1, 1, 1), (0, 2, 1, 1), (1, 0, 1, 1)]),
    ("XY", [(2, 2, 2, 2), (4, 0, 2, 2), (1, 2, 2, 2)])], ids=lambda v: v if isinstance(v, str) else str(len(v)))
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_uncentred_windows_after_a_centred_one_is_tuned(dt, direction, windows):
    """The same grid, type and window bucket, tuned one after the other: the
    centred one may be tuned to take x neighbours from lanes."""
    rng = np.random.default_rng(67)
    for nx, ny in ((2048, 600), (1030, 515)):
        u = rng.uniform(-1, 1, (ny, nx))
        din = to_device(u, dt)
        for ext in windows:
            L, R, T, B = ext
            w = rng.uniform(-1, 1, (T + B + 1) * (L + R + 1))
            dout = torch.zeros_like(din)
            p = b.mxs_create_2d(nx, ny, nx, DIRS[direction], b.MXS_P, code(dt), L, R, T, B, w, None, din, dout)
            try:
                b.mxs_autotune(p)
                info = b.mxs_plan_info(p)
                b.mxs_compute(p)
                torch.cuda.synchronize()
            finally:
                b.mxs_destroy(p)
            print(ext, info)
            check_against_oracle(u, dout.double().cpu().numpy(), direction, True, ext, w, None, dt)
