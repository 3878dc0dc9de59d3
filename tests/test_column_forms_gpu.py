"""Column solves on both sides of the rule that chooses between strips and three
phases: many columns of few rows, and ensembles of flat grids."""
import math

import numpy as np
import pytest

import oracle
from paper_1902_09931_amd import workloads as wl
from tests.gpu_util import TORCH, code, round_to, to_device, torch
from tests.test_strips_gpu import PENTA, TRI, US

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

# (nx, ny, strips expected for (double, float, bfloat16)), tridiagonal then pentadiagonal
EDGES = [(10000, 20, (1, 1, 1), (0, 0, 0)), (10001, 20, (0, 0, 0), (0, 0, 0)), (5000, 40, (1, 1, 1), (1, 1, 1)),
         (5001, 40, (1, 1, 1), (1, 0, 1)), (7001, 149, (1, 1, 1), (0, 0, 1)), (12000, 199, (0, 1, 0), (0, 0, 0)),
         (12000, 200, (1, 1, 0), (0, 0, 0)), (14001, 400, (1, 1, 1), (1, 0, 0)), (20001, 400, (1, 1, 0), (1, 0, 0)), (40000, 512, (1, 1, 0), (1, 1, 0)),
         (5001, 1100, (1, 1, 1), (1, 1, 0)), (9001, 1025, (1, 1, 1), (1, 0, 0)), (100001, 5, (0, 0, 0), (0, 0, 0))]


@pytest.mark.parametrize("nx,ny,tri,penta", EDGES)
@pytest.mark.parametrize("k,dt", enumerate(["f64", "f32", "bf16"]), ids=["f64", "f32", "bf16"])
def test_solves_on_both_sides_of_the_rule(nx, ny, tri, penta, k, dt):
    """As test_column_strips_match_oracle, with the form the rule states."""
    rng = np.random.default_rng(nx + ny)
    r = round_to(rng.uniform(-1, 1, (ny, nx)), dt)
    rhs = to_device(r, dt)
    for coef, strips in ((TRI, tri[k]), (PENTA, penta[k])):
        x = torch.zeros_like(rhs)
        p = b.mxs_create_cyclic_solve(len(coef) - 1, coef, b.MXS_LINES_COLS, nx, ny, nx, None, code(dt), rhs, x)
        info = b.mxs_plan_info(p)
        b.mxs_compute(p)
        torch.cuda.synchronize()
        b.mxs_destroy(p)
        assert ("columns=strips" in info) == bool(strips), info
        ref = oracle.cyclic_solve_grid(oracle.circulant_bands(coef), 0, r)
        tol = 1e-12 * np.abs(ref).max() + US[dt] * np.abs(ref)
        assert np.all(np.abs(x.double().cpu().numpy() - ref) <= tol)


@pytest.mark.parametrize("count,ny,nx,strips", [(9, 66, 1000, (0, 0, 0)), (8, 66, 1000, (1, 1, 1)),
                                                (11, 256, 1000, (1, 0, 0)), (11, 400, 1000, (1, 1, 0)),
                                                (3, 2020, 100, (0, 0, 0)), (3, 2016, 100, (1, 1, 1)),
                                                (1, 8, 8, (1, 1, 1)), (2, 9, 60, (1, 1, 1)), (1, 31, 301, (1, 1, 1)),
                                                (1, 32, 2052, (1, 1, 1)), (4, 33, 1000, (1, 1, 1)),
                                                (1, 63, 500, (1, 1, 1)), (6, 64, 1000, (1, 0, 1)),
                                                (9, 64, 1000, (0, 0, 0))])
@pytest.mark.parametrize("k,dt", enumerate(["f64", "f32", "bf16"]), ids=["f64", "f32", "bf16"])
def test_ensembles_on_both_sides_of_the_rule(count, ny, nx, strips, k, dt):
    """A fused step of equal grids takes the form the rule states, gives every
    grid the same bits, and is within the bounds of test_fused_step_at_tile_edges
    of the oracle."""
    dx, dy = 2 * math.pi / nx, 2 * math.pi / ny
    step = 0.1 * min(dx, dy) ** 2
    c0 = round_to(wl.ch_initial(ny, nx, seed=79), dt)
    q = [[to_device(c0, dt), to_device(c0, dt), torch.zeros((ny, nx), dtype=TORCH[dt], device="cuda")]
         for _ in range(count)]
    p = b.mxs_ch_ensemble_create([nx] * count, [ny] * count, [dx] * count, [dy] * count, [step] * count, 1.0, 0.01,
                                 code(dt), [v[0] for v in q], [v[1] for v in q], [v[2] for v in q])
    try:
        b.mxs_ch_set_step_mode(p, b.MXS_CH_FUSED)
        assert ("columns=strips" in b.mxs_plan_info(p)) == bool(strips[k]), b.mxs_plan_info(p)
        b.mxs_ch_step(p, 1, False)
        torch.cuda.synchronize()
        got = torch.stack([next(t for t in v if t.data_ptr() == b.mxs_ch_state(p, g)[1]) for g, v in enumerate(q)])
    finally:
        b.mxs_destroy(p)
    assert torch.equal(got, got[:1].expand_as(got))
    _, oc = oracle.ch_run(c0, c0, 1, dx, dy, step, 1.0, 0.01)
    err = np.abs(got[0].double().cpu().numpy() - oc)
    if dt == "f64":
        _, on = oracle.ch_run_nudged(c0, c0, 1, dx, dy, step, 1, 1.0, 0.01)
        bound = max(1e-12 * np.abs(oc).max(), 2 * np.abs(on - oc).max())
    else:
        a = 2.0 / 3.0 * 0.01 * step
        hx, hy = dx ** -2, dy ** -2
        m = np.abs(c0).max()
        s_max = (a * (16 * hx * hx + 16 * hy * hy + 32 * hx * hy) * m
                 + 2.0 / 3.0 * step * 4 * (hx + hy) * (m ** 3 + m))
        bound = 2 * US[dt] * np.abs(oc) + 1.15 ** 2 * (32 + 2) * 2.0 ** -24 * s_max
    assert np.all(err <= bound)
