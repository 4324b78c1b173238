"""The recoveries' range: prims scaled by powers of ten (density and energy by
10^k, the field by 10^(k/2), which leaves the flow the same) recover like the
unscaled ones while the squares that each method forms are in the range of
FP64, and past it fail rather than return something else."""

import numpy as np
import pytest

from workloads import GridSpec

pytestmark = pytest.mark.gpu


def _recover(inverter, k):
    import torch
    from paper_2408_01361_amd import grmhd as gr
    grid = GridSpec(8, 8, 6)
    rng = np.random.default_rng(4)
    P = np.array([1.0, 1.0, 0.2, 0.1, 0.0, 1.0, 0.3, 0.2])[:, None, None, None] * (
        1.0 + 0.1 * rng.uniform(-1, 1, (8, 12, 14, 14)))
    P[:2] *= 10.0 ** k
    P[5:] *= 10.0 ** (k / 2)
    P = torch.from_numpy(P).cuda()
    s = gr.Grmhd(grid, 4.0 / 3.0, inverter=inverter)
    out, n, _ = s.cons_to_prims(s.prims_to_cons(P), 1.01 * P)
    I = (slice(None),) + (slice(3, -3),) * 3
    return n, ((out - P).abs() / P.abs().clamp_min(1e-300))[I][:2].max().item()


# Kastaun forms D^2 (exact to a part in 2^52 down to 1e-154, to one in 1e8 at
# 1e-158), the implicit solver the square of a Jacobian column of order 10^-k.
@pytest.mark.parametrize("inverter,k,bar", [(1, 0, 1e-12), (1, 150, 1e-12), (1, -150, 1e-12), (1, -155, 1e-12),
                                            (1, -158, 1e-6), (1, 153, 1e-12), (2, 0, 1e-10), (2, -150, 1e-10), (2, 150, 1e-10),
                                            (2, 155, 1e-10), (2, 160, 1e-10), (0, 50, 1e-12), (0, -50, 1e-12)])
def test_scaled_prims_recover(inverter, k, bar):
    n, err = _recover(inverter, k)
    assert n == 0 and err <= bar, (n, err)


@pytest.mark.parametrize("k", [-163, -170])
def test_kastaun_refuses_where_the_square_vanishes(k):
    assert _recover(1, k)[0] == 8 * 8 * 6


@pytest.mark.parametrize("rho", [1e200, 1e206, 1e250, 1e300])
def test_kastaun_recovers_a_dense_zone(rho):
    """Past the range of D^2 the squared momentum counts as zero, past that of
    D^3/2 the momentum along the field too: the zone still recovers, its density
    to the Lorentz factor that is lost (1.03 here), its field exactly."""
    import torch
    from paper_2408_01361_amd import grmhd as gr
    grid = GridSpec(8, 8, 6)
    rng = np.random.default_rng(4)
    P = np.array([1.0, 1.0, 0.2, 0.1, 0.05, 1.0, 0.3, 0.2])[:, None, None, None] * (
        1.0 + 0.1 * rng.uniform(-1, 1, (8, 12, 14, 14)))
    P[0, 6, 7, 8] = rho
    P = torch.from_numpy(P).cuda()
    s = gr.Grmhd(grid, 4.0 / 3.0, inverter=1)
    out, n, _ = s.cons_to_prims(s.prims_to_cons(P), 1.01 * P)
    got, want = out.cpu().numpy()[:, 6, 7, 8], P.cpu().numpy()[:, 6, 7, 8]
    gamma = np.sqrt(1.0 + (want[2:5] ** 2).sum())
    assert n == 0 and np.array_equal(got[5:], want[5:])
    assert abs(got[0] / (gamma * want[0]) - 1.0) <= 1e-13 and np.isfinite(got).all()
