"""Stencils, WENO advection, user functions and diagnostics at the sizes where
their tiles end: widths just below and above a strip (the last strip is shifted
back over its neighbour), rows whose pitch is no multiple of a vector, signal
ends inside a vector, grids of a few tiles."""
import math

import numpy as np
import pytest

import oracle
from oracle.diagnostics import coarsening_k1, coarsening_s
from paper_1902_09931_amd import workloads as wl
from tests.gpu_util import U_STORE, code, rel_err, round_to, stencil_bound, to_device, torch
from tests.test_diag_gpu import make_plan
from tests.test_fn_gpu import run_fn
from tests.test_stencil_gpu import DIRS, check_against_oracle, run_1d
from tests.test_weno_gpu import fields, run

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

# windows of the row form (1, 4 and 8 rows of halo), of the block forms (3, 5
# and 9 rows; x neighbours from lanes, half-width 1, 2 and 4) and uncentred
WINDOWS = [("X", (1, 1, 0, 0)), ("X", (2, 2, 0, 0)), ("X", (4, 4, 0, 0)), ("X", (3, 1, 0, 0)), ("X", (8, 8, 0, 0)),
           ("Y", (0, 0, 1, 1)), ("Y", (0, 0, 4, 4)), ("Y", (0, 0, 3, 5)), ("XY", (1, 1, 1, 1)), ("XY", (2, 2, 2, 2)),
           ("XY", (0, 2, 1, 0))]
# strips are 64, 128 or 256 threads of 2 (FP64) or 4 elements
WIDTHS = [17, 127, 129, 256, 257, 258, 259, 511, 515, 1023, 1025, 1027]


@pytest.mark.parametrize("tuned", [False, True])
@pytest.mark.parametrize("direction,ext", WINDOWS, ids=lambda v: v if isinstance(v, str) else "".join(map(str, v)))
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_stencil2d_strip_ends(dt, direction, ext, tuned):
    L, R, T, B = ext
    rng = np.random.default_rng(23)
    w = rng.uniform(-1, 1, (T + B + 1) * (L + R + 1))
    for k, nx in enumerate(WIDTHS if not tuned else (129, 1027)):
        ny = (17, 18, 25, 40)[k % 4]
        ld = nx + (0, 1, 0, 3)[k % 4]
        coe = wl.CUBIC_MINUS_LINEAR if k % 3 == 2 else None
        u = rng.uniform(-1, 1, (ny, nx))
        din = to_device(u, dt, ld, fill=float("nan"))
        for periodic in (True, False):
            dout = torch.full((ny, ld), float("nan"), dtype=din.dtype, device="cuda")
            p = b.mxs_create_2d(nx, ny, ld, DIRS[direction], b.MXS_P if periodic else b.MXS_NP, code(dt),
                                L, R, T, B, w, coe, din, dout)
            try:
                if tuned:
                    b.mxs_autotune(p)
                b.mxs_compute(p)
                torch.cuda.synchronize()
            finally:
                b.mxs_destroy(p)
            got = dout.double().cpu().numpy()
            assert np.isnan(got[:, nx:]).all(), (nx, ld)
            check_against_oracle(u, got[:, :nx], direction, periodic, ext, w, coe, dt)


# every remainder of a signal's start and end in a vector, signals shorter than
# one vector, and batches of one to many vectors per thread
BATCHES = {"one": [17], "short": [5] * 40 + [6, 7, 5, 9, 5, 5, 8], "ends": list(range(40, 75)),
           "long": [3001, 17, 4099, 5, 2050], "many": [61, 64, 67, 5, 130] * 3000}


@pytest.mark.parametrize("batch", list(BATCHES))
@pytest.mark.parametrize("L,R", [(2, 2), (1, 0), (0, 4)])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_stencil1d_signal_ends(dt, L, R, batch):
    offs = np.concatenate([[0], np.cumsum(BATCHES[batch])]).astype(np.int64)
    rng = np.random.default_rng(29)
    vals = rng.uniform(-1, 1, offs[-1])
    w = rng.uniform(-1, 1, L + R + 1)
    vv = round_to(vals, dt)
    for periodic in (True, False):
        for coe in (None, wl.CUBIC_MINUS_LINEAR):
            got = run_1d(vals, offs, periodic, L, R, w, coe, dt)
            ref = np.full_like(vv, np.nan)
            oracle.stencil1d_batch(vv, offs, L, R, w, periodic, coe=coe, out=ref)
            written = ~np.isnan(ref)
            assert np.array_equal(~np.isnan(got), written)
            if dt == "f64":
                assert rel_err(got, ref, written) <= 1e-12
                continue
            s_abs = oracle.stencil1d_batch(np.abs(vv), offs, L, R, np.abs(w), periodic,
                                           coe=None if coe is None else np.abs(coe))
            bound = stencil_bound(dt, s_abs, ref, L + R + 1, 0 if coe is None else len(coe))
            assert np.all(np.abs(got - ref)[written] <= bound[written])


@pytest.mark.parametrize("layout", [None, "1,0,64,0", "1,1,128,1"])
@pytest.mark.parametrize("shape,ld_pad", [((7, 127), 0), ((8, 129), 0), ((33, 255), 1), ((9, 257), 2), ((40, 513), 3),
                                          ((12, 1025), 0), ((300, 515), 0)])
def test_weno_strip_ends(monkeypatch, shape, ld_pad, layout):
    if layout:
        monkeypatch.setenv("MXS_WENO_TILE", layout)
    phi, u, v = fields(*shape, seed=31)
    got, info = run(phi, u, v, 0.02, 0.01, ld_pad)
    if layout:
        assert "rows=1 " in info
    assert rel_err(got, oracle.weno_adv(phi, u, v, 0.02, 0.01)) <= 1e-12


@pytest.mark.parametrize("shape,ld_pad", [((4, 4), 0), ((5, 63), 1), ((33, 65), 0), ((17, 257), 5), ((64, 1030), 0)])
@pytest.mark.parametrize("periodic", [True, False])
def test_user_function_tile_ends(shape, ld_pad, periodic):
    for dt in ("f64", "f32", "bf16"):
        got, ref, mag, info = run_fn("corners", shape, dt, periodic, ld_pad, seed=37)
        written = ~np.isnan(ref)
        assert np.array_equal(~np.isnan(got), written), info
        err = np.abs(got - ref)[written]
        if dt == "f64":
            assert err.max() <= 1e-12 * np.abs(ref[written]).max(), info
        else:
            assert np.all(err <= (64 * 2.0 ** -24 * mag + U_STORE[dt] * np.abs(ref))[written]), info


@pytest.mark.parametrize("shape", [(8, 8), (8, 16), (16, 8), (32, 1024), (2048, 16), (4096, 8), (128, 2048)])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_coarsening_transform_sizes(dt, shape):
    ny, nx = shape
    c = round_to(wl.ch_initial(ny, nx, seed=41, amplitude=0.5), dt)
    p, _, dx, dy, _ = make_plan(c, dt, dx=2 * math.pi / nx, dy=3 * math.pi / ny)
    try:
        s, k1 = b.mxs_ch_coarsening(p)
    finally:
        b.mxs_destroy(p)
    assert s == pytest.approx(coarsening_s(c), rel=1e-12)
    assert k1 == pytest.approx(coarsening_k1(c, dx, dy), rel=1e-12)
