"""A step at the CFL dt of the device (step_cfl) against the same step at the
dt the host reads (dt, then step): one reduction, so the same dt and the same
state bit for bit, whatever launches read the dt and wherever its final pass
runs."""

import numpy as np
import pytest

from workloads import fm_torus

pytestmark = pytest.mark.gpu

GAM = 13.0 / 9.0


def _same(shape, nsteps, **kw):
    import torch
    from paper_2408_01361_amd import grmhd as gr
    grid, P, info = fm_torus(*shape)
    a, b = gr.Grmhd(grid, GAM, **kw), gr.Grmhd(grid, GAM, **kw)
    for s in (a, b):
        s.load(torch.from_numpy(P).cuda())
        if kw.get("ct"):
            s.load_faces(torch.from_numpy(info["faces"]).cuda())
    for n in range(nsteps):
        a.step_cfl()      # (the first one right after the load: no dt reduced before)
        dt = b.dt()
        b.step(dt)
        assert a.last_dt() == dt
        assert torch.equal(a.prims(), b.prims()), n
        if kw.get("ct"):
            assert torch.equal(a.faces(), b.faces()), n


@pytest.mark.parametrize("opts", [dict(), dict(precision=1), dict(floors=True), dict(floors=True, fofc=True), dict(inverter=2)],
                         ids=["plain", "mixed", "floors", "fofc", "implicit"])
@pytest.mark.parametrize("ct", [1, 2])
@pytest.mark.parametrize("shape", [(24, 22, 7), (64, 32, 72), (64, 64, 64)], ids=["small", "largest", "above"])
def test_face_ct_advances_its_faces_with_the_steps_dt(shape, ct, opts):
    """64x32x72 has 576 workgroups of partials, the most that an update
    reduces."""
    _same(shape, 3, recon=1, ct=ct, **opts)


@pytest.mark.parametrize("opts", [dict(recon=0), dict(recon=1), dict(recon=1, precision=1)], ids=["mc", "weno5", "mixed"])
@pytest.mark.parametrize("integrator", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", [(64, 32, 72), (61, 33, 73), (60, 61, 58), (64, 64, 64)],
                         ids=["largest", "above", "resident_and_late", "1024"])
def test_every_integrator_steps_with_one_dt(shape, integrator, opts):
    """576 workgroups of partials, the most that an update reduces; 640; and
    960 and 1024, more workgroups than are resident at a time: the last ones
    start when the first have left their results."""
    _same(shape, 4, integrator=integrator, **opts)


@pytest.mark.parametrize("precision", [0, 1])
def test_no_cfl_step_without_a_signal_speed(precision):
    """Cold gas at rest in flat space has no signal speed: there is no step
    size, and a device-dt step leaves the state as it is.  With internal
    energy in a single zone, that zone's rate is the grid's."""
    import torch
    from paper_2408_01361_amd import grmhd as gr
    from workloads import GridSpec
    grid = GridSpec(9, 8, 7)
    P = torch.zeros((8, 13, 14, 15), dtype=torch.float64, device="cuda")
    P[0] = 1.0
    s = gr.Grmhd(grid, GAM, precision=precision)
    s.load(P)
    with pytest.raises(gr.GrmhdError):
        s.dt()
    with pytest.raises(gr.GrmhdError):
        gr.cfl_dt_noalloc(grid, GAM, P)
    s.step_cfl()
    with pytest.raises(gr.GrmhdError):
        s.last_dt()
    assert torch.equal(s.prims(), P)
    P[1, 5, 6, 7] = 0.1
    s.load(P)
    u = 0.1
    cs = (GAM * (GAM - 1.0) * u / (1.0 + GAM * u)) ** 0.5
    assert s.dt() == pytest.approx(0.9 / (cs * (9 + 8 + 7)), rel=1e-14)
    assert gr.cfl_dt_noalloc(grid, GAM, P) == s.dt()


@pytest.mark.parametrize("flat", [True, False])
def test_infinite_density_is_cold(flat):
    """A zone of infinite density (and finite energy and field) has no sound or
    Alfven speed: the oracle's rate of it is its flow's, and the CFL step that
    of the other zones."""
    import torch
    import oracle
    from paper_2408_01361_amd import grmhd as gr
    from workloads import GridSpec
    if flat:
        grid, gam = GridSpec(9, 8, 7), GAM
        rng = np.random.default_rng(2)
        P = np.array([1, .5, .05, .02, .01, .5, .3, .2])[:, None, None, None] * (
            1 + 0.1 * rng.uniform(-1, 1, (8, 13, 14, 15)))
    else:
        (grid, P), gam = fm_torus(16, 12, 4)[0:2], 13 / 9
    P[0, 5, 8, 9] = np.inf
    want = oracle.estimate_dt(oracle.cfg(grid, gam=gam), P)
    assert np.isfinite(want) and want > 0.0
    s = gr.Grmhd(grid, gam)
    s.load(torch.from_numpy(P).cuda())
    assert s.dt() == pytest.approx(want, rel=1e-13)
    P[0, 5, 8, 9] = np.nan
    s.load(torch.from_numpy(P).cuda())
    with pytest.raises(gr.GrmhdError):
        s.dt()
