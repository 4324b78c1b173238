"""The gradient in the adiabatic index on a torus whose WENO5 face states
undershoot at its edge (density and internal energy below zero there, and
inversions that fail), against central differences of the step itself."""

import pytest

from workloads import fm_torus

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(33, 47, 3), (64, 64, 1)])
def test_gamma_gradient_of_an_undershooting_torus(shape):
    """The bar: the difference of the quotients of two step sizes (their
    truncation), and the roundoff of the smaller one, 1e-13 of the misfit's
    terms over 2h."""
    import torch
    from paper_2408_01361_amd import grmhd as gr
    grid, P, _ = fm_torus(*shape)
    P = torch.from_numpy(P).cuda()
    gam = 13.0 / 9.0
    s = gr.Grmhd(grid, gam, recon=1)
    s.load(P)
    dt = 0.5 * s.dt()
    G = torch.rand(P.shape, generator=torch.Generator(device="cuda").manual_seed(3), dtype=torch.float64,
                   device="cuda")
    _, grad = s.step_vjp(P, dt, G)

    def terms(x):
        t = gr.Grmhd(grid, x, recon=1)
        t.load(P)
        t.step(dt)
        return (G * t.prims())[:, 3:-3, 3:-3, 3:-3]

    fd = {h: ((terms(gam + h) - terms(gam - h)).sum() / (2 * h)).item() for h in (1e-3, 1e-4)}
    bar = abs(fd[1e-3] - fd[1e-4]) + 1e-13 * terms(gam).abs().sum().item() / 2e-4
    print("gradient", grad, "differences", fd, "bar", bar)
    assert bar < 1e-4 * abs(grad)
    assert abs(grad - fd[1e-4]) <= bar
