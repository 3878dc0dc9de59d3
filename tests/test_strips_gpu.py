"""Column solves held in registers (one launch per solve) and the quad kernel
of the fused Cahn-Hilliard step, at the sizes where their tiles end."""
import math

import numpy as np
import pytest

import oracle
from paper_1902_09931_amd import workloads as wl
from tests.gpu_util import TORCH, code, rel_err, round_to, to_device, torch

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

TRI = [2.5, -1.0]
PENTA = [1.0 + 6.0 * 20.0, -4.0 * 20.0, 20.0]
US = {"f64": 2.0 ** -53, "f32": 2.0 ** -24, "bf16": 2.0 ** -8}

# (nx, ny): one row per thread, last segments of one row and of a full one, a
# last wavefront that holds one segment, idle wavefronts, the largest columns
# of every shape (512, 1024 and 2048 rows), partial strips, and columns just
# past the longest shape (three phases)
GRIDS = [(5, 5), (3, 63), (9, 64), (4, 65), (7, 257), (30, 511), (33, 512), (12, 513), (21, 1024), (2049, 37),
         (2100, 1000), (2064, 1024), (17, 1025), (8, 2047), (50, 2048), (2801, 1100), (2816, 2048), (19, 2049)]


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("coef", [TRI, PENTA], ids=["tri", "penta"])
@pytest.mark.parametrize("nx,ny", GRIDS)
def test_column_strips_match_oracle(nx, ny, coef, dt):
    """x within 1e-12 of max |x| plus one storage rounding of the oracle, in
    place and not, with a padded pitch; the padding is not written."""
    rng = np.random.default_rng(nx + 7 * ny)
    ld = nx + 3
    r = round_to(rng.uniform(-1, 1, (ny, ld)), dt)
    ref = oracle.cyclic_solve_grid(oracle.circulant_bands(coef), 0, np.ascontiguousarray(r[:, :nx]))
    tol = 1e-12 * np.abs(ref).max() + US[dt] * np.abs(ref)
    for in_place in (False, True):
        rhs = to_device(r, dt)
        x = rhs if in_place else torch.full_like(rhs, 7.0)
        p = b.mxs_create_cyclic_solve(len(coef) - 1, coef, b.MXS_LINES_COLS, nx, ny, ld, None, code(dt), rhs, x)
        info = b.mxs_plan_info(p)
        b.mxs_compute(p)
        torch.cuda.synchronize()
        b.mxs_destroy(p)
        assert ("columns=strips" in info) == (ny <= 2048), info
        got = x.double().cpu().numpy()
        assert np.all(np.abs(got[:, :nx] - ref) <= tol)
        assert np.array_equal(got[:, nx:], r[:, nx:] if in_place else np.full((ny, 3), 7.0))


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("coef", [TRI, PENTA], ids=["tri", "penta"])
@pytest.mark.parametrize("nx,ny", [(33, 4096), (17, 4097), (5, 4128), (40, 7278), (16, 8191), (3, 8192), (18, 8193)])
def test_tall_columns_match_oracle(nx, ny, coef, dt):
    """Columns of 128, 129, 256 and 257 segments: phase B with 8 or 16
    segments per thread in registers, or neither; same bound as above."""
    rng = np.random.default_rng(ny)
    r = round_to(rng.uniform(-1, 1, (ny, nx)), dt)
    ref = oracle.cyclic_solve_grid(oracle.circulant_bands(coef), 0, r)
    rhs = to_device(r, dt)
    x = torch.empty_like(rhs)
    p = b.mxs_create_cyclic_solve(len(coef) - 1, coef, b.MXS_LINES_COLS, nx, ny, nx, None, code(dt), rhs, x)
    b.mxs_compute(p)
    torch.cuda.synchronize()
    b.mxs_destroy(p)
    assert np.all(np.abs(x.double().cpu().numpy() - ref) <= 1e-12 * np.abs(ref).max() + US[dt] * np.abs(ref))


# (ny, nx) of one ensemble per entry: strips of every shape, several
# instances of different heights in one launch, rows of every length class of
# the quad kernel with full and partial last quads, lanes and wavefronts, row
# counts that are no multiple of the 4 (or 2) rows of a workgroup, and widths
# that are no multiple of 4 beside ones that are
ENSEMBLES = [
    [(70, 8), (66, 12), (65, 64), (97, 68), (128, 256)],
    [(75, 260), (66, 500), (513, 512)],
    [(1024, 516), (67, 1000), (70, 1024)],
    [(69, 1028), (66, 2044), (81, 2048)],
    [(67, 2052), (66, 4092), (65, 4096)],
    [(300, 24), (520, 30), (71, 33)],
    [(1025, 16), (1100, 40)],
    [(90, 1500), (1030, 1600)],
]


@pytest.mark.parametrize("sizes", ENSEMBLES)
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_fused_step_at_tile_edges(sizes, dt):
    """Fused steps against the oracle.  FP64 after 6 steps: 1e-12 of max |C|
    or twice the oracle's own rounding spread (its run with every window
    weight and band value one ulp the other way), whichever is larger.
    FP32 and BF16, one step from C^{-1} = C^0 (where the exact state is
    stored): against the oracle's step, |dC| <= 2 u_s |C| + 1.15^2 (32 + 2)
    u_32 max S, S the per-point sum of the magnitudes of R's terms and 1.15
    the largest infinity norm of the inverse line operators."""
    D, GAMMA = 1.0, 0.01
    c0s = [round_to(wl.ch_initial(ny, nx, seed=60 + k), dt) for k, (ny, nx) in enumerate(sizes)]
    bufs = [[to_device(c, dt), to_device(c, dt), torch.zeros(c.shape, dtype=TORCH[dt], device="cuda")] for c in c0s]
    nx, ny = [s[1] for s in sizes], [s[0] for s in sizes]
    dxs, dys = [2 * math.pi / v for v in nx], [2 * math.pi / v for v in ny]
    dts = [0.1 * min(a, c) ** 2 for a, c in zip(dxs, dys)]
    steps = 6 if dt == "f64" else 1
    plan = b.mxs_ch_ensemble_create(nx, ny, dxs, dys, dts, D, GAMMA, code(dt), [q[0] for q in bufs],
                                    [q[1] for q in bufs], [q[2] for q in bufs])
    try:
        b.mxs_ch_set_step_mode(plan, b.MXS_CH_FUSED)
        b.mxs_ch_step(plan, steps, True)
        torch.cuda.synchronize()
        got = []
        for k, q in enumerate(bufs):
            cur = b.mxs_ch_state(plan, k)[1]
            got.append(next(t for t in q if t.data_ptr() == cur).double().cpu().numpy())
    finally:
        b.mxs_destroy(plan)
    for k, c0 in enumerate(c0s):
        _, oc = oracle.ch_run(c0, c0, steps, dxs[k], dys[k], dts[k], D, GAMMA)
        err = np.abs(got[k] - oc)
        if dt == "f64":
            _, on = oracle.ch_run_nudged(c0, c0, steps, dxs[k], dys[k], dts[k], 1, D, GAMMA)
            bound = max(1e-12 * np.abs(oc).max(), 2 * np.abs(on - oc).max())
        else:
            a = 2.0 / 3.0 * D * GAMMA * dts[k]
            hx, hy = dxs[k] ** -2, dys[k] ** -2
            m = np.abs(c0).max()
            s_max = (a * (16 * hx * hx + 16 * hy * hy + 32 * hx * hy) * m
                     + 2.0 / 3.0 * D * dts[k] * 4 * (hx + hy) * (m ** 3 + m))
            bound = 2 * US[dt] * np.abs(oc) + 1.15 ** 2 * (32 + 2) * 2.0 ** -24 * s_max
        print(f"{dt} {sizes[k]}: max |GPU - oracle| {err.max():.3e}, max ratio {(err / bound).max():.3f}")
        assert np.all(err <= bound), sizes[k]


def test_fused_replays_with_strips_equal_eager_steps():
    """Graph replays of a fused step with strip columns, with eager work
    between them, give the eager states bit for bit."""
    c0 = wl.ch_initial(200, 148, seed=5)
    runs = []
    for graph in (False, True):
        h = 2 * math.pi / 148
        q = [to_device(c0, "f64"), to_device(c0, "f64"), torch.zeros(c0.shape, dtype=torch.float64, device="cuda")]
        p = b.mxs_ch_create(148, 200, h, 2 * math.pi / 200, 0.1 * h * h, 1.0, 0.01, b.MXS_F64, *q)
        b.mxs_ch_set_step_mode(p, b.MXS_CH_FUSED)
        assert "columns=strips" in b.mxs_plan_info(p)
        states = []
        for _ in range(7):
            b.mxs_ch_step(p, 1, graph)
            torch.cuda.synchronize()
            _ = torch.ones(1000, device="cuda").sum().item()
            states.append(torch.stack(q).clone())
        b.mxs_destroy(p)
        runs.append(states)
    assert all(torch.equal(x, y) for x, y in zip(*runs))
    assert rel_err(runs[0][-1].cpu().numpy(), runs[1][-1].cpu().numpy()) == 0.0


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("ny", [4096, 4097, 6000, 8193])
def test_tall_separate_and_persistent_steps_are_equal(ny, dt):
    """Phase B keeps 8, 16 or no segments per thread in registers in the
    separate form and none in the persistent one: the states are the same bit
    for bit."""
    nx = 40
    c0 = wl.ch_initial(ny, nx, seed=6)
    h = 2 * math.pi / nx
    runs = []
    for mode in (b.MXS_CH_SEPARATE, b.MXS_CH_PERSISTENT):
        q = [to_device(c0, dt), to_device(c0, dt), torch.zeros((ny, nx), dtype=TORCH[dt], device="cuda")]
        p = b.mxs_ch_create(nx, ny, h, h, 0.1 * h * h, 1.0, 0.01, code(dt), *q)
        b.mxs_ch_set_step_mode(p, mode)
        b.mxs_ch_step(p, 4, False)
        b.mxs_ch_mass(p)
        b.mxs_destroy(p)
        runs.append(torch.stack(q))
    assert torch.equal(*runs)


def test_default_stream_is_torchs_current_stream():
    """Calls without a stream run on torch's current one, inside and outside
    a stream context."""
    assert b._stream(None) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert b._stream(None) == s.cuda_stream
    assert b._stream(None) == torch.cuda.current_stream().cuda_stream
