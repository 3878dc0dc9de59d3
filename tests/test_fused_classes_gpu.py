"""The kernels of the fused Cahn-Hilliard step by the widths of the grids: the
quad kernel for classes of rows of a multiple of 4 elements, the row kernel for
the others and wherever its shape is fixed."""
import math

import pytest

from paper_1902_09931_amd import workloads as wl
from tests.gpu_util import to_device, torch
from tests.test_ch_gpu import FUSED_SIZES
from tests.test_strips_gpu import test_fused_step_at_tile_edges as fused_step_against_the_oracle

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

# (ny, nx) over the five classes of rows, no width a multiple of 4; each class
# alone; widths that are beside ones that are not, in one class
ODD = [(40, 33), (17, 253), (37, 301), (23, 511), (40, 602), (24, 1001), (21, 1027), (13, 2047), (11, 3001), (9, 4095)]
ENSEMBLES = [ODD, [(70, 254)], [(71, 509)], [(67, 1023)], [(66, 2045)], [(65, 4094)], [(30, 300), (29, 301)]]


def info(sizes):
    c0s = [wl.ch_initial(ny, nx, seed=1) for ny, nx in sizes]
    bufs = [[to_device(c, "f64") for _ in range(3)] for c in c0s]
    h = [2 * math.pi / nx for _, nx in sizes]
    p = b.mxs_ch_ensemble_create([s[1] for s in sizes], [s[0] for s in sizes], h, h, [0.1 * v * v for v in h], 1.0,
                                 0.01, b.MXS_F64, [q[0] for q in bufs], [q[1] for q in bufs], [q[2] for q in bufs])
    try:
        b.mxs_ch_set_step_mode(p, b.MXS_CH_FUSED)
        return b.mxs_plan_info(p)
    finally:
        b.mxs_destroy(p)


def test_which_classes_take_the_quad_kernel(monkeypatch):
    assert " quad_classes=0/5 " in info(ODD) + " "
    assert " quad_classes=4/5 " in info(FUSED_SIZES) + " "   # 250 is no multiple of 4
    assert " quad_classes=5/5 " in info([s for s in FUSED_SIZES if s[1] % 4 == 0]) + " "
    for rows, cols in (("4", "1"), ("8", "1"), ("4", "2"), ("4", None), (None, "1")):
        for name, v in (("MXS_CH_FUSED_ROWS", rows), ("MXS_CH_FUSED_COLS", cols)):
            monkeypatch.delenv(name, raising=False)
            if v:
                monkeypatch.setenv(name, v)
        text = info(FUSED_SIZES) + " "
        assert f" fused_rows={rows or 4} fused_cols={cols or 1} quad_classes=0/5 " in text, text


@pytest.mark.parametrize("sizes", ENSEMBLES, ids=lambda s: f"{len(s)}-{s[-1][1]}")
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_widths_that_are_no_multiple_of_4(sizes, dt):
    fused_step_against_the_oracle(sizes, dt)


@pytest.mark.parametrize("rows,cols", [(4, 1), (8, 1), (4, 2)])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_fixed_shapes_of_the_row_kernel(monkeypatch, rows, cols, dt):
    monkeypatch.setenv("MXS_CH_FUSED_ROWS", str(rows))
    monkeypatch.setenv("MXS_CH_FUSED_COLS", str(cols))
    fused_step_against_the_oracle([(16, 64), (21, 512), (13, 1000), (9, 2048), (9, 4096), (10, 3002)], dt)
