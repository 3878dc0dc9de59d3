"""Replayed Cahn-Hilliard steps equal eager ones bit for bit: the plan's own
graphs of the persistent step, also after a tuning that changes its tables, and
steps that a caller captures into a graph."""
import math

import pytest

from paper_1902_09931_amd import workloads as wl
from tests.gpu_util import TORCH, code, to_device, torch

pytestmark = pytest.mark.gpu

b = pytest.importorskip("paper_1902_09931_amd.binding")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

MODES = {"separate": b.MXS_CH_SEPARATE, "persistent": b.MXS_CH_PERSISTENT, "fused": b.MXS_CH_FUSED}


class Run:
    def __init__(self, ny, nx, dt, mode):
        h = 2 * math.pi / nx
        c0 = wl.ch_initial(ny, nx, seed=97)
        self.q = [to_device(c0, dt), to_device(c0, dt), torch.zeros((ny, nx), dtype=TORCH[dt], device="cuda")]
        self.p = b.mxs_ch_create(nx, ny, h, 2 * math.pi / ny, 0.1 * h * h, 1.0, 0.01, code(dt), *self.q)
        b.mxs_ch_set_step_mode(self.p, MODES[mode])

    def states(self):
        prev, cur = b.mxs_ch_state(self.p)
        return torch.stack([next(t for t in self.q if t.data_ptr() == a) for a in (prev, cur)]).clone()

    def close(self):
        b.mxs_destroy(self.p)


def eager_work():
    torch.cuda.synchronize()
    return torch.ones(1000, device="cuda").sum().item()


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_persistent_replays_equal_eager_steps(dt):
    graph, eager = Run(200, 148, dt, "persistent"), Run(200, 148, dt, "persistent")
    try:
        for k in range(8):
            b.mxs_ch_step(graph.p, 1, True)
            eager_work()
            b.mxs_ch_step(eager.p, 1, False)
            assert torch.equal(graph.states(), eager.states()), k
        assert "step=persistent" in b.mxs_plan_info(graph.p) and "persist_graph=1" in b.mxs_plan_info(graph.p)
        b.mxs_ch_mass(graph.p)
    finally:
        graph.close()
        eager.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_graphs_captured_before_a_tuning_are_not_replayed_after_it(dt):
    """Every rotation captured, then tables rebuilt by the tuning and by the
    return to the persistent form."""
    graph, eager = Run(300, 260, dt, "persistent"), Run(300, 260, dt, "persistent")
    try:
        b.mxs_ch_step(graph.p, 4, True)
        b.mxs_ch_step(eager.p, 4, False)
        b.mxs_autotune(graph.p)
        b.mxs_ch_set_step_mode(graph.p, b.MXS_CH_SEPARATE)
        b.mxs_ch_step(graph.p, 2, True)
        b.mxs_ch_step(eager.p, 2, False)
        b.mxs_ch_set_step_mode(graph.p, b.MXS_CH_PERSISTENT)
        for k in range(6):
            b.mxs_ch_step(graph.p, 1, True)
            eager_work()
            b.mxs_ch_step(eager.p, 1, False)
            assert torch.equal(graph.states(), eager.states()), k
        assert "persist_graph=1" in b.mxs_plan_info(graph.p)
        b.mxs_ch_mass(graph.p)
    finally:
        graph.close()
        eager.close()


# strips, three column phases (2100 rows), and widths of the row and the quad kernel
@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("mode", ["separate", "fused"])
@pytest.mark.parametrize("ny,nx,dt", [(200, 148, "f64"), (2100, 40, "f64"), (64, 301, "f32"), (130, 1028, "bf16")])
def test_steps_captured_by_the_caller(ny, nx, dt, mode, use_graph):
    """Three steps, one turn of the plan's three buffers, in a graph of the
    caller's, replayed with eager work between the replays."""
    cap, eager = Run(ny, nx, dt, mode), Run(ny, nx, dt, mode)
    try:
        b.mxs_ch_step(cap.p, 3, use_graph)
        b.mxs_ch_step(eager.p, 3, False)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            b.mxs_ch_step(cap.p, 3, use_graph)
        for k in range(4):
            g.replay()
            eager_work()
            b.mxs_ch_step(eager.p, 3, False)
            assert torch.equal(cap.states(), eager.states()), k
        b.mxs_ch_step(cap.p, 2, use_graph)
        b.mxs_ch_step(eager.p, 2, False)
        assert torch.equal(cap.states(), eager.states())
        assert b.mxs_ch_steps_taken(cap.p) == 8     # what was enqueued, not what was replayed
    finally:
        cap.close()
        eager.close()
