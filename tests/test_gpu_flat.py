"""Grids with one zone along a periodic x3: the step computes one plane for
all (they are equal), and differences along x3 vanish.  The same grid with
outflow x3 boundaries goes through the general kernels with three planes of
faces; one zone's outflow and periodic ghosts are the same zone, so both must
give the same interior zones bit for bit, and the flat path's x3 ghosts, filled
when the state is read, must be the zone itself.  (The flux correction treats
marked zones differently at the two kinds of boundary; its flat case is
held to the oracle in test_gpu_floors_fofc.py.)"""

import dataclasses

import numpy as np
import pytest

from workloads import fm_torus, interior, linear_mode, magnetised_blast, BC_OUTFLOW

pytestmark = pytest.mark.gpu


def _run(torch, gr, grid, P, gam, **kw):
    s = gr.Grmhd(grid, gam, **kw)
    s.load(torch.from_numpy(P).cuda())
    for _ in range(2):
        s.step_cfl()
    s.step(0.5 * s.last_dt())
    return s.prims().cpu().numpy(), s.counters()


@pytest.mark.parametrize("opts", [dict(recon=0), dict(recon=1), dict(recon=2), dict(recon=5), dict(recon=7), dict(recon=1, precision=1),
                                  dict(recon=0, integrator=1), dict(recon=1, integrator=2), dict(recon=1, integrator=3),
                                  dict(recon=1, inverter=1, floors=True), dict(recon=0, inverter=2)],
                         ids=lambda o: "-".join(f"{k}{int(v)}" for k, v in o.items()))
@pytest.mark.parametrize("case", ["torus33x29", "mode40x5", "blast48", "torus6x3"])
def test_flat_grid_equals_the_general_path(case, opts):
    import torch
    from paper_2408_01361_amd import grmhd as gr
    gam = 13 / 9
    if case.startswith("torus"):
        n1, n2 = (int(v) for v in case[5:].split("x"))
        grid, P = fm_torus(n1, n2, 1)[0:2]
    elif case == "mode40x5":
        grid, P = linear_mode("fast", 40, ndim=2)[0:2]
        grid, P, gam = dataclasses.replace(grid, n2=5), np.ascontiguousarray(P[:, :, :11]), 4 / 3
    else:
        grid, P = magnetised_blast(48, noise=0.05, seed=2)
        gam = 4 / 3
    open_ = dataclasses.replace(grid, bc=tuple(grid.bc[:4]) + (BC_OUTFLOW, BC_OUTFLOW))
    a, ca = _run(torch, gr, grid, P, gam, **opts)
    b, cb = _run(torch, gr, open_, P, gam, **opts)
    assert np.array_equal(interior(a), interior(b), equal_nan=True)
    assert ca == cb
    for k in range(7):
        assert np.array_equal(a[:, k], a[:, 3], equal_nan=True)
