"""Steps that a reverse sweep recomputes are launched in another group order and
residency than the rollout's: the gradients do not depend on how many there are."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1309_1983_amd
    paper_1309_1983_amd.lib()


# either side of 2^19 points in the cache, on the one- and the two-dimensional
# grid; beyond the cache with and without porous geometry
@pytest.mark.parametrize("shape,solid", [((96, 78, 70), 0.1), ((96, 78, 72), 0.1), ((64, 100, 84), 0.0),
                                         ((192, 110, 90), 0.15), ((194, 110, 90), 0.0)])
def test_gradients_do_not_depend_on_the_checkpoints(shape, solid):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    flags = W.random_flags(N, 8, solid, solid / 4) if solid else None
    gen = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda *s: torch.rand(*s, device="cuda", generator=gen) - 0.5  # noqa: E731
    rho, u, F, g = 1 + 0.02 * rnd(N), 0.04 * rnd(3, N), 2e-3 * rnd(3, N), rnd(3, N)
    lat = Lattice(*shape, 0.7, flags=flags)
    lat.set_wall_velocity(0.03, -0.01, 0.02)
    lat.set_force(F)
    lat.init_equilibrium(rho, u)
    s0 = lat.populations()
    out = []
    for K in (1, 9, 4, 2):   # nothing is recomputed with the first two
        lat.set_populations(s0)
        lat.forward_checkpointed(9, K)
        out.append(lat.adjoint(g))
        again = lat.adjoint(g)
        assert torch.equal(again[0], out[-1][0]) and again[1] == out[-1][1], K
    lat.close()
    for gF, gt in out[1:]:
        assert torch.equal(gF, out[0][0]) and gt == out[0][1]
