"""The number of points per work-item where only other options are given: the
options of the several-point step do not widen the step of a small lattice
without solid points, which takes one point per work-item."""
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


@pytest.mark.parametrize("kw", [{}, {"gather_mode": "early"}, {"gather_mode": "flags_first"}, {"groups_per_cu": -1},
                                {"groups_per_cu": 4}, {"block": (32, 8)}])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_small_solid_free_lattices_keep_one_point(kw, storage):
    from paper_1309_1983_amd import Lattice
    shape = (32, 32, 64)
    N = int(np.prod(shape))
    s0 = torch.from_numpy(near_rest_state(N, 5))
    F = torch.from_numpy(W.random_force_field(N, 6, 1e-4).astype(np.float32))
    out = []
    for options in (kw, {"cells_per_lane": 4}):
        lat = Lattice(*shape, 0.8, storage=storage, **options)
        lat.set_force(F)
        lat.set_populations(s0)
        name = lat.step_kernel_name()
        assert ("k_step_ab<" in name) == (options is kw), (options, name)
        lat.step(4)
        out.append(lat.populations())
        lat.close()
    assert torch.equal(*out)


# hardly a solid point, and 16-bit rows of 256 points: one point per work-item,
# except where pairs of steps go through boxes in LDS (the last case)
@pytest.mark.parametrize("shape,storage,solids,one", [((80, 40, 38), "f32", 3, True), ((80, 40, 38), "f16", 3, True),
                                                      ((48, 44, 40), "bf16", 1, True), ((264, 45, 17), "f16", 0, True),
                                                      ((256, 40, 17), "bf16", 900, True), ((72, 70, 68), "f32", 0, True),
                                                      ((72, 66, 64), "f32", 1, True), ((32, 32, 32), "f32", 1, False)])
def test_few_solid_points_and_long_rows(shape, storage, solids, one):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    flags = np.zeros(N, np.uint8)
    flags[np.random.RandomState(4).choice(N, solids, replace=False)] = 2
    fl = torch.from_numpy(flags == 0).cuda()
    s0 = torch.from_numpy(near_rest_state(N, 5))
    out = []
    for options in ({}, {"cells_per_lane": 4}):
        lat = Lattice(*shape, 0.8, flags=flags, storage=storage, **options)
        lat.set_wall_velocity(0.02, 0.01, -0.03)
        lat.set_populations(s0)
        name = lat.step_kernel_name()
        assert ("k_step_ab<" in name) == (one and not options), (options, name)
        for _ in range(3):
            lat.step(1)
        rho, u = lat.macros()
        out.append((lat.populations()[:, fl], rho, u))
        lat.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)


# two steps per launch beside on-site walls: the cost of a plane does not fall
# with the width of the tile (48 columns in the second and third)
@pytest.mark.parametrize("shape,pair", [((192, 128, 100), True), ((144, 120, 130), False), ((144, 144, 144), False),
                                        ((112, 112, 112), False)])
def test_pairs_beside_onsite_walls(shape, pair):
    from paper_1309_1983_amd import Lattice
    flags = W.onsite_cavity_flags(*shape)
    fl = torch.from_numpy((flags != 1) & (flags != 2)).cuda()
    out = []
    for options in ({}, {"cells_per_lane": 1}):
        lat = Lattice(*shape, 0.8, flags=flags, **options)
        lat.set_wall_velocity(0.02, 0.01, 0.0)
        assert ("k_step_pair<" in lat.step_kernel_name()) == (pair and not options)
        lat.step(5)
        out.append(lat.populations()[:, fl])
        lat.close()
    assert torch.equal(*out)
