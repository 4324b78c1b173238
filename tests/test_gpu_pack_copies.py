"""Loading and reading packs whose blocks differ much in size: the copies take
one workgroup per 256 zones that there are, not per zone of the largest block."""

import pytest

from workloads import GridSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[256] + 240 * [8], 240 * [8] + [256], [1, 2, 30, 3, 29], [5]],
                         ids=["large_first", "large_last", "ragged", "one"])
def test_pack_round_trip(sizes):
    """One 256^3 block among 240 small ones: the largest block's workgroups
    for every block would be more threads than a launch may have (2^32)."""
    import torch
    from paper_2408_01361_amd import grmhd as gr
    n = max(sizes)
    pack = gr.Pack(GridSpec(n, n, n), sizes, [(0, 0, 0)] * len(sizes), 4.0 / 3.0, recon=0)
    P = torch.rand(pack.prim_doubles, generator=torch.Generator(device="cuda").manual_seed(1), dtype=torch.float64,
                   device="cuda")
    pack.load(P)
    assert torch.equal(pack.prims(), P)
    pack.close()
