"""GPU-vs-oracle parity of the floors and the first-order flux correction.

Workloads: the magnetised cylindrical blast (flat space, 48^2, MC and WENO5),
where the high-order step loses zones to failed inversions, and the coarse
magnetised torus (Kerr), whose atmosphere zones at the torus edge fail
without floors.  Both sides advance with the oracle's dt; the bar is the
step bar (relative L1 of every primitive at most 1e-12) and the same
counters: failed inversions, floor activations, marked zones, fluid-frame
fallbacks.  The marks are decided in FP64 on both sides from the same
operations (flat space: bit for bit)."""

import numpy as np
import pytest

import oracle
from parity_util import rel_l1, check, NOISY_MODE
from workloads import (magnetised_blast, fm_torus, linear_mode, interior, RECON_MC, RECON_WENO5)

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_01361_amd import grmhd as gr
    return torch, gr


def run_both(grid, P, gam, recon, nsteps, floors, fofc, inverter=0, precision=0, **fp):
    torch, gr = _setup()
    c = oracle.cfg(grid, gam=gam, recon=recon, floors=floors, fofc=fofc, inverter=inverter, **fp)
    alt, _, _ = oracle.run(c, P, -1, nsteps, fma=True)
    ref, fails, dts = oracle.run(c, P, -1, nsteps)
    st = oracle.last_stats()
    run_both.alt = alt
    s = gr.Grmhd(grid, gam, recon=recon, floors=floors, fofc=fofc, inverter=inverter,
                 precision=precision, **fp)
    s.load(torch.from_numpy(P).cuda())
    for dt in dts:
        s.step(float(dt))
    out = s.prims().cpu().numpy()
    return out, ref, s.counters(), st, s, dts


CASES = {
    "blast48_mc_fofc": (lambda: magnetised_blast(48), 4 / 3, RECON_MC, 4, False, True),
    "blast48_mc_floors_fofc": (lambda: magnetised_blast(48), 4 / 3, RECON_MC, 6, True, True),
    "blast48_weno_floors_fofc": (lambda: magnetised_blast(48), 4 / 3, RECON_WENO5, 6, True, True),
    "blast48_weno_floors": (lambda: magnetised_blast(48), 4 / 3, RECON_WENO5, 6, True, False),
    "torus24_weno_floors_fofc": (lambda: fm_torus(24, 24, 8)[0:2], 13 / 9, RECON_WENO5, 3, True, True),
    "torus20x28x6_mc_floors": (lambda: fm_torus(20, 28, 6)[0:2], 13 / 9, RECON_MC, 3, True, False),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_floors_fofc_parity(case):
    make, gam, recon, nsteps, floors, fofc = CASES[case]
    grid, P = make()
    out, ref, cnt, st, _, dts = run_both(grid, P, gam, recon, nsteps, floors, fofc)
    print(case, "gpu", cnt, "oracle", st, flush=True)
    assert cnt == st
    assert (st["fofc_zones"] > 0) == fofc or st["floor_hits"] > 0
    check(out, ref, label=case, alt=run_both.alt)


def test_kastaun_with_floors_and_fofc():
    grid, P = magnetised_blast(48)
    out, ref, cnt, st, _, _ = run_both(grid, P, 4 / 3, RECON_WENO5, 6, True, True, inverter=1)
    print("kastaun blast", cnt, st)
    assert cnt == st
    check(out, ref, label="kastaun blast", alt=run_both.alt)


def test_implicit_recovery_with_floors():
    grid, P = magnetised_blast(48)
    out, ref, cnt, st, _, _ = run_both(grid, P, 4 / 3, RECON_WENO5, 6, True, False, inverter=2)
    print("implicit blast floors", cnt, st)
    assert cnt == st
    check(out, ref, label="implicit blast floors", alt=run_both.alt)


def test_donor_cell_step_parity():
    """The first-order scheme alone (donor-cell states everywhere)."""
    for make, gam, noisy in ((lambda: linear_mode("fast", 32, ndim=2)[0:2], 4 / 3, NOISY_MODE),
                             (lambda: fm_torus(20, 28, 6)[0:2], 13 / 9, ())):
        grid, P = make()
        out, ref, cnt, st, _, dts = run_both(grid, P, gam, oracle.RECON_DONOR, 2, False, False)
        print("donor", cnt, st)
        assert cnt["fails"] == st["fails"]
        check(out, ref, noisy, label="donor", alt=run_both.alt)


def test_fofc_and_floors_are_a_no_op_on_smooth_flow():
    """Nothing marked, nothing floored: the step equals the plain one bit for
    bit on the GPU too."""
    torch, gr = _setup()
    grid, P, _, _ = linear_mode("fast", 24, ndim=2)
    outs = []
    for fl, fo in ((False, False), (True, True)):
        s = gr.Grmhd(grid, 4 / 3, recon=RECON_WENO5, floors=fl, fofc=fo)
        s.load(torch.from_numpy(P).cuda())
        for _ in range(3):
            s.step_cfl()
        outs.append(s.prims().cpu().numpy())
        c = s.counters()
        assert c["fofc_zones"] == 0 and c["floor_hits"] == 0
    assert np.array_equal(outs[0], outs[1])


def test_fofc_removes_failures_and_keeps_divb_and_cfl():
    """The blast with the correction: no failures where the plain step has
    some, corner div B at roundoff, and the device CFL step (its rate
    partials come from the final pass) equals the oracle's dt."""
    torch, gr = _setup()
    grid, P = magnetised_blast(48)
    plain = gr.Grmhd(grid, 4 / 3, recon=RECON_MC)
    plain.load(torch.from_numpy(P).cuda())
    s = gr.Grmhd(grid, 4 / 3, recon=RECON_MC, fofc=True)
    s.load(torch.from_numpy(P).cuda())
    for _ in range(4):
        plain.step_cfl()
        s.step_cfl()
    assert plain.status()[0] > 0
    cnt = s.counters()
    assert cnt["fails"] == 0 and cnt["fofc_zones"] > 0
    mx, _ = s.divb()
    assert mx < 1e-13 * 0.07 / grid.dx[0]
    out = s.prims().cpu().numpy()
    s.step_cfl()
    c = oracle.cfg(grid, gam=4 / 3, recon=RECON_MC, fofc=True)
    assert s.last_dt() == pytest.approx(oracle.estimate_dt(c, out), rel=1e-14)


def test_mixed_precision_with_fofc_runs_and_keeps_divb():
    """FP32 fluxes with the correction (no oracle: the reduced-precision path
    is measured against FP64): div B stays at FP64 roundoff, no failures,
    density within 1e-3 relative L1 of the FP64 run."""
    torch, gr = _setup()
    grid, P = magnetised_blast(48)
    res = []
    for prec in (gr.PREC_FP64, gr.PREC_MIXED):
        s = gr.Grmhd(grid, 4 / 3, recon=RECON_MC, fofc=True, floors=True, precision=prec)
        s.load(torch.from_numpy(P).cuda())
        dt = s.dt()
        for _ in range(4):
            s.step(dt)
        res.append((s.prims().cpu().numpy(), s.counters(), s.divb()[0]))
    (a, ca, _), (b, cb, db) = res
    print("fp64", ca, "mixed", cb)
    assert cb["fails"] == 0
    assert db < 1e-13 * 0.07 / grid.dx[0]
    A, B = interior(a)[0], interior(b)[0]
    assert np.abs(A - B).sum() / np.abs(A).sum() < 1e-3


def test_long_torus_run_with_kastaun_floors_and_correction():
    """Production settings on the 64^3 magnetised torus (WENO5, Kastaun
    recovery, floors and the first-order flux correction), 1000 device-side
    CFL steps (t ~ 70 M): every primitive finite, density at or above its
    geometric floor and internal energy at it to the drift-frame
    injection's re-inversion (1e-6), the field's corner divergence at
    roundoff, the torus body kept, and no failed inversion: where the
    updated energy of a cold atmosphere zone leaves no positive internal
    energy, the recovery's clamped specific energy stands and the energy
    floor supplies u (1D_W fails in those zones instead)."""
    torch, gr = _setup()
    grid, P, _ = fm_torus(64, 64, 64)
    s = gr.Grmhd(grid, 13 / 9, recon=RECON_WENO5, inverter=gr.INV_KASTAUN, floors=True, fofc=True)
    s.load(torch.from_numpy(P).cuda())
    t = 0.0
    for n in range(1000):
        s.step_cfl()
        t += s.last_dt()
        if n % 250 == 249:
            print("step", n + 1, "t", t, s.counters(), flush=True)
    out = interior(s.prims().cpu().numpy())
    assert np.isfinite(out).all()
    x1, _, _ = grid.centers()
    r = np.exp(x1[3:-3])[None, None, :]
    fl = gr.FLOOR_DEFAULTS
    assert (out[0] >= fl["rho_min_geom"] * r ** -1.5 * (1 - 1e-12)).all()
    assert (out[1] >= fl["u_min_geom"] * r ** -2.5 * (1 - 1e-6)).all()
    assert out[0].max() > 0.5 * interior(P)[0].max()
    cnt = s.counters()
    assert cnt["fails"] == 0, cnt
    mx, _ = s.divb()
    scale = np.abs(interior(P[5:8])).max() / min(grid.dx[:2])
    print("t", t, "counters", cnt, "divb max", mx, "scale", scale)
    assert mx < 1e-12 * scale


def _reach_case(shape, bc, floors, roll):
    import dataclasses
    from workloads import BC_OUTFLOW, BC_PERIODIC
    grid, P = magnetised_blast(48, noise=0.05 if floors else 0.0, seed=3)
    n1, n2, n3 = shape
    B = {"outflow": (BC_OUTFLOW,) * 6, "periodic": (BC_PERIODIC,) * 6,
         "mixed": (BC_PERIODIC, BC_PERIODIC, BC_OUTFLOW, BC_OUTFLOW, BC_PERIODIC, BC_PERIODIC)}[bc]
    at = lambda n, r: (np.arange(n) + r + max(0, (48 - n) // 2)) % 48
    I = np.repeat(interior(P)[:, :, at(n2, 0)][..., at(n1, roll)], n3, axis=1)
    Q = np.pad(I, ((0, 0), (3, 3), (3, 3), (3, 3)), mode="edge")
    return dataclasses.replace(grid, n1=n1, n2=n2, n3=n3, bc=B), Q


@pytest.mark.parametrize("shape,bc,floors,roll", [
    ((48, 48, 1), "periodic", False, 24), ((48, 48, 1), "outflow", True, 12), ((37, 5, 3), "periodic", True, 20),
    ((37, 6, 4), "mixed", True, 12), ((1, 40, 2), "periodic", True, 0), ((70, 9, 1), "mixed", True, 30)])
def test_final_pass_where_the_correction_reaches(shape, bc, floors, roll):
    """The final pass of the correction repeats the update only at zones that
    share a face or an edge with a marked one (across periodic boundaries
    too): prims, counters and the CFL step that follows are the oracle's, on
    grids narrower than a stencil, with rows that are not a multiple of a
    wavefront, and with open, periodic and mixed boundaries that the blast's
    edge lies across.  Bars: the step bar, as above; the CFL step 1e-12 (it
    follows the prims)."""
    grid, Q = _reach_case(shape, bc, floors, roll)
    out, ref, cnt, st, s, dts = run_both(grid, Q, 4 / 3, RECON_MC, 3, floors, True)
    print(shape, bc, "gpu", cnt, "oracle", st, flush=True)
    assert st["fofc_zones"] > 0
    assert cnt == st
    check(out, ref, label=f"{shape} {bc}", alt=run_both.alt)
    c = oracle.cfg(grid, gam=4 / 3, recon=RECON_MC, floors=floors, fofc=True)
    _, _, more = oracle.run(c, Q, -1, 4)
    assert abs(s.dt() - more[3]) <= 1e-12 * more[3]
