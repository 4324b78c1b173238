"""A step captured into a graph stands by itself: what the context knew when
the step was captured (that the ghost zones were filled) need not hold when it
is replayed, and what was only captured has not run."""

import numpy as np
import pytest

from workloads import bondi, fm_torus, interior, linear_mode

pytestmark = pytest.mark.gpu


def _case(name):
    if name == "torus":
        g, P = fm_torus(24, 22, 7)[0:2]
        return g, P, 13 / 9, 1e-3
    if name == "torus_flat":
        g, P = fm_torus(17, 12, 1)[0:2]
        return g, P, 13 / 9, 1e-3
    if name == "bondi":   # frozen radial ghosts: a ghost fill per stage
        g, P = bondi(20, 18, 6)[0:2]
        return g, P, 4 / 3, 1e-3
    g, P = linear_mode("fast", 12, ndim=3, amp=0.05)[0:2]
    return g, P, 4 / 3, 0.02


@pytest.mark.parametrize("name", ["mode", "torus", "torus_flat", "bondi"])
def test_replayed_step_after_a_load(name):
    """Warm-up step, captured step, load of another state (its ghosts, except
    frozen ones, not filled), replays with eager work between them: every
    replay is the eager step of that state bit for bit, and so are eager steps
    and loads among the replays."""
    import torch
    from paper_2408_01361_amd import grmhd as gr
    grid, P, gam, dt = _case(name)
    Q = P.copy()
    Q[:2] *= 1.01
    if name != "bondi":
        ghosts = np.ones(P.shape[1:], bool)
        ghosts[3:-3, 3:-3, 3:-3] = False
        Q[:, ghosts] = 7.0
    P, Q = torch.from_numpy(P).cuda(), torch.from_numpy(Q).cuda()
    ref = gr.Grmhd(grid, gam, recon=1)
    ref.load(Q)
    want = []
    for _ in range(4):
        ref.step(dt)
        want.append(ref.prims().cpu().numpy())
    torch.cuda.synchronize()

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = gr.Grmhd(grid, gam, recon=1, stream=stream)
        s.load(P)
        s.step(dt)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            s.step(dt)
        s.load(Q)
        graph.replay()
        stream.synchronize()
        assert np.array_equal(s.prims().cpu().numpy(), want[0]), "first replay"
        (P * 2.0).sum().item()
        graph.replay()
        s.step(dt)
        assert np.array_equal(s.prims().cpu().numpy(), want[2]), "eager step after a replay"
        graph.replay()
        stream.synchronize()
        assert np.array_equal(interior(s.prims().cpu().numpy()), interior(want[3])), "third replay"
        # a captured step that is not replayed leaves the state as it was
        s.load(Q)
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=stream):
            s.step(dt)
        s.step(dt)
        assert np.array_equal(s.prims().cpu().numpy(), want[0]), "eager step after a capture"
        stream.synchronize()
