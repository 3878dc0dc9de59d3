"""The WENO advection term over the scales of its inputs: the floor 1e-99 of the
weights acts on the differences divided by the spacing, whatever the spacing."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import rel_err, torch
from tests.test_weno_gpu import run

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("h", [1e-6, 0.02, 1.0, 1e6])
@pytest.mark.parametrize("slope", [1e-60, 1e-52, 1e-50, 1e-49, 1e-48, 1e-46, 1e-30, 1.0, 1e40])
def test_slopes_around_the_floor(slope, h):
    """Slopes whose squares lie below, at and above the floor, to the 1e-12 of
    the other WENO tests."""
    rng = np.random.default_rng(53)
    ny, nx = 24, 70
    phi = slope * h * rng.uniform(-1, 1, (ny, nx))
    u, v = rng.uniform(-1, 1, (ny, nx)), rng.uniform(-1, 1, (ny, nx))
    got, _ = run(phi, u, v, h, 2 * h)
    assert rel_err(got, oracle.weno_adv(phi, u, v, h, 2 * h)) <= 1e-12


@pytest.mark.parametrize("h", [1e-130, 1e-3, 1.0, 1e130])
def test_a_constant_field_has_no_advection(h):
    rng = np.random.default_rng(59)
    u, v = rng.uniform(-1, 1, (9, 40)), rng.uniform(-1, 1, (9, 40))
    got, _ = run(np.full((9, 40), 3.0), u, v, h, h)
    assert np.array_equal(got, np.zeros((9, 40)))


def test_velocities_and_spacings_of_any_size():
    """Products that stay in range when the derivative is formed first."""
    rng = np.random.default_rng(61)
    phi, v = 1e-200 * rng.uniform(-1, 1, (8, 32)), np.zeros((8, 32))
    u = 1e305 * rng.uniform(0.5, 1, (8, 32))
    got, _ = run(phi, u, v, 1e-10, 1.0)
    ref = oracle.weno_adv(phi, u, v, 1e-10, 1.0)
    assert np.isfinite(ref).all() and rel_err(got, ref) <= 1e-12
