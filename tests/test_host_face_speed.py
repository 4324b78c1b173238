"""The adjoint of a face state through the fast speed of larger magnitude,
compiled for the host (tests/host/face_speed_host.cpp), on the states that a
high-order reconstruction makes next to a steep edge: density, internal
energy or both undershot below zero.  There the quadratic of the signal speeds
may have a negative leading coefficient or no real root, and the root of
larger magnitude is not the one that the sign of its linear term names."""

import math
import os
import shutil
import struct
import subprocess

import numpy as np
import pytest

import oracle
from test_host_sanitized import FLAGS, HOST, _run
from test_oracle_pins import _random_prims
from workloads.torus import torus_grid


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("face_speed")
    exe = str(d / "face_speed")
    subprocess.run(["g++", *FLAGS, "-I", HOST, "-o", exe, os.path.join(HOST, "face_speed_host.cpp")], check=True,
                   capture_output=True, text=True)
    return exe, d


@pytest.mark.parametrize("direction", [1, 2, 3])
def test_adjoint_of_undershot_face_states(program, direction):
    """Reverse sweep against dual numbers, both of them with the larger root
    on a tie (states without motion along x2 and x3 have one).  States whose
    discriminant is within 1e-3 of zero (relative to its terms) are left out:
    there the speed has an unbounded derivative.  The bar, 1e-9 of the sum of
    the products' terms, is the roundoff of the dual form's A = u^t u^t -
    c^2 (g^tt + u^t u^t), which cancels to 1/u^t^2 >~ 1e-3, through a
    discriminant of 1e-3 of its terms, over some ten operations."""
    exe, d = program
    grid = torus_grid(8, 8, 1)
    c = oracle.cfg(grid, gam=13.0 / 9.0)
    rng = np.random.default_rng(20 + direction)
    n = 3000
    x1, x2 = rng.uniform(math.log(1.05), math.log(1000.0), n), rng.uniform(0.02, 0.98, n)
    P = _random_prims(rng, n, c, x1, x2)
    kind = np.arange(n) % 5
    P[kind == 1, 0] *= -1.0
    P[kind == 2, 1] *= -1.0
    P[kind == 3, :2] *= -1.0
    P[kind == 4, 1 + direction] = 0.0
    rows = np.column_stack([x1, x2, rng.uniform(1.1, 1.7, n), P, rng.normal(size=(n, 17))])
    hdr = struct.pack("<3i2d", n, 1, direction, grid.a, grid.hslope)
    out = np.frombuffer(_run(exe, d, hdr + rows.tobytes(), "d%d" % direction), dtype=np.float64).reshape(n, 29)
    rev, dual, scale, A, disc = out[:, :9], out[:, 9:18], out[:, 18:27], out[:, 27], out[:, 28]
    use = np.abs(disc) > 1e-3
    assert use.sum() > 0.8 * n
    assert (A[use] < 0).sum() > 100 and (disc[use] < 0).sum() > 100
    assert (np.abs(rev - dual) <= 1e-9 * scale)[use].all()
