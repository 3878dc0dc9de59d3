"""Calls of so many lines, columns or tiles that one launch cannot hold a
workgroup for each: a launch holds fewer than 2^32 threads and is cut off without
an error beyond that."""
import numpy as np
import pytest

from tests.gpu_util import torch

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

TRI = [2.5, -1.0]
# inverse of circ(-1, 2.5, -1) of three elements
INV3 = np.linalg.inv(np.array([[2.5, -1, -1], [-1, 2.5, -1], [-1, -1, 2.5]]))


def fill(shape, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=gen)


def check(x, r, dim):
    """x against INV3 r along dim (three elements) in double, in pieces: 1e-12 of
    max |x| and one rounding to float."""
    inv = torch.from_numpy(INV3).cuda()
    n = r.shape[1 - dim]
    for k in range(0, n, 1 << 24):
        xs, rs = (v.narrow(1 - dim, k, min(1 << 24, n - k)).double() for v in (x, r))
        ref = rs @ inv if dim == 1 else inv @ rs
        assert bool((xs - ref).abs().le(1e-12 * 2 + 2.0 ** -24 * ref.abs()).all()), k


@pytest.mark.parametrize("form", ["classes", "units", "rows"])
def test_lines_beyond_one_launch(monkeypatch, form):
    n = (1 << 26) + 3
    r = fill((n, 3), 71)
    x = torch.zeros_like(r)
    if form == "rows":
        p = b.mxs_create_cyclic_solve(1, TRI, b.MXS_LINES_ROWS, 3, n, 3, None, b.MXS_F32, r, x)
    else:
        monkeypatch.setenv("MXS_RAGGED_FORM", form)
        p = b.mxs_create_cyclic_solve(1, TRI, b.MXS_LINES_RAGGED, 0, 0, 0, np.arange(n + 1, dtype=np.int64) * 3,
                                      b.MXS_F32, r, x)
    try:
        b.mxs_compute(p)
        torch.cuda.synchronize()
    finally:
        b.mxs_destroy(p)
    check(x, r, 1)


def test_columns_beyond_one_launch():
    nx = (1 << 27) + 5
    r = fill((3, nx), 73)
    x = torch.zeros_like(r)
    p = b.mxs_create_cyclic_solve(1, TRI, b.MXS_LINES_COLS, nx, 3, nx, None, b.MXS_F32, r, x)
    try:
        b.mxs_compute(p)
        torch.cuda.synchronize()
    finally:
        b.mxs_destroy(p)
    check(x, r, 0)


@pytest.mark.parametrize("half,ny", [(1, 403_000_000), (2, 269_000_000), (4, 537_000_000)])
def test_columns_of_more_rows_than_blocks_in_one_launch(half, ny):
    """One periodic column of ny rows: against shifted sums in double, in pieces,
    to the float bound of 2 half + 1 terms of at most 1 and one rounding."""
    u = fill((ny, 1), 83)
    out = torch.full_like(u, float("nan"))
    w = np.linspace(-1, 1, 2 * half + 1)
    p = b.mxs_create_2d(1, ny, 1, b.MXS_Y, b.MXS_P, b.MXS_F32, 0, 0, half, half, w, None, u, out)
    try:
        b.mxs_compute(p)
        torch.cuda.synchronize()
    finally:
        b.mxs_destroy(p)
    taps = 2 * half + 1
    for k in range(0, ny, 1 << 25):
        n = min(1 << 25, ny - k)
        rows = torch.arange(k - half, k + n + half, device="cuda") % ny
        v = u[rows, 0].double()
        ref = sum(float(w[q]) * v[q:q + n] for q in range(taps))
        err = (out[k:k + n, 0].double() - ref).abs()
        assert bool(err.le((taps + 2) * 2.0 ** -24 * taps).all()), k   # (a NaN fails)


def test_user_function_grids_beyond_one_launch_are_refused():
    """140 million rows of one column: 17.5 million chunks of 256 threads."""
    ny = 140_000_000
    u = torch.ones(ny, 1, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros_like(u)
    source = "__device__ mxs_real same(const mxs_real *const *w, const mxs_real *coe, int loc) { return w[0][loc]; }"
    p = b.mxs_create_2d_fn(1, ny, 1, b.MXS_Y, b.MXS_P, b.MXS_BF16, 0, 0, 1, 1, [u], out, None, source, "same")
    try:
        with pytest.raises(Exception, match="more workgroups than one launch holds"):
            b.mxs_compute(p)
    finally:
        b.mxs_destroy(p)
