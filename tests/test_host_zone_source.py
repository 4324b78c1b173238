"""The momentum source as the update kernels form it (structured metric,
paired derivative entries, refined reciprocals), compiled for the host
(tests/host/zone_source_host.cpp), against the oracle's connection form."""

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
from workloads import GridSpec
from workloads.torus import torus_grid


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("zone_source")
    exe = str(d / "zone_source")
    subprocess.run(["g++", *FLAGS, "-I", HOST, "-o", exe, os.path.join(HOST, "zone_source_host.cpp")], check=True,
                   capture_output=True, text=True)
    return exe, d


@pytest.mark.parametrize("metric", ["kerr", "flat"])
def test_zone_source_against_the_oracle(program, metric):
    """Fuzzed states from inside the horizon to r = 1000.  The forms differ in
    rounding only, which the terms of the connection form amplify where they
    cancel: within 1e-12 of |S1| + |S2|, the bar of the library's other form
    of the same source."""
    exe, d = program
    grid = torus_grid(8, 8, 1) if metric == "kerr" else GridSpec(4, 4, 4)
    gam = 13.0 / 9.0
    c = oracle.cfg(grid, gam=gam)
    rng = np.random.default_rng(14)
    n = 2000
    if metric == "kerr":
        x1, x2 = rng.uniform(math.log(1.05), math.log(1000.0), n), rng.uniform(0.02, 0.98, n)
    else:
        x1, x2 = rng.uniform(0.0, 1.0, n), rng.uniform(0.0, 1.0, n)
    P = _random_prims(rng, n, c, x1, x2)
    hdr = struct.pack("2i3d", n, int(metric == "kerr"), gam, grid.a, grid.hslope)
    got = np.frombuffer(_run(exe, d, hdr + np.column_stack([x1, x2, P]).tobytes(), metric),
                        dtype=np.float64).reshape(n, 2)
    ref = np.array([oracle.point_source(c, P[q], x1[q], x2[q]) for q in range(n)])
    if metric == "flat":
        assert not got.any() and not ref.any()
        return
    mag = np.abs(ref[:, 2:4]).sum(axis=1)
    assert (mag > 0).all()
    assert (np.abs(got - ref[:, 2:4]).max(axis=1) <= 1e-12 * mag).all()
