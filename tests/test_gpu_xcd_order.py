"""Lattices that the caches hold give each of the 8 XCDs consecutive work-groups
in the one-point kernels, in place of every eighth one. The order changes no
value: one point per work-item equals four bit for bit, for numbers of
work-groups below, at and beside multiples of eight, on both kinds of grid, and
a step in place equals a step between two arrays."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_common import near_rest_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1309_1983_amd
    paper_1309_1983_amd.lib()


# 1, 3, 7, 8, 9, 27, 18 and 70 work-groups; the last two on two-dimensional grids
@pytest.mark.parametrize("shape", [(4, 3, 1), (12, 5, 3), (36, 5, 7), (20, 12, 8), (60, 4, 9), (100, 7, 9), (256, 2, 9),
                                   (128, 10, 14)])
def test_order_changes_no_value(shape):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    flags = W.random_flags(N, 5, 0.2, 0.05)
    fl = torch.from_numpy(flags == 0).cuda()
    F = torch.from_numpy(W.random_force_field(N, 7, 1e-4).astype(np.float32))
    s0 = torch.from_numpy(near_rest_state(N, 11))
    got = []
    for kw in ({"cells_per_lane": 1}, {"cells_per_lane": 4}, {"pattern": "aa"}):
        lat = Lattice(*shape, 0.7, flags=flags, **kw)
        lat.set_wall_velocity(0.05, -0.02, 0.03)
        lat.set_force(F)
        lat.set_populations(s0)
        lat.step(4)
        rho, u = lat.macros()
        lat.check_finite()
        got.append((lat.populations()[:, fl], rho[fl], u[:, fl]))
        lat.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b), shape
