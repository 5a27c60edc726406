"""Small two-array lattices (no more boxes of 16 x 4 x 2 points than compute
units) take two steps per launch through boxes in LDS. Both steps do the
one-step kernels' arithmetic on values rounded to the storage format in
between, so n steps in one call equal n calls of one step bit for bit on every
fluid point, and so do the trajectories that the adjoint reads."""
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


def _lattice(shape, flags, storage, force, **kw):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    lat = Lattice(*shape, 0.7, flags=flags, storage=storage, **kw)
    lat.set_wall_velocity(0.05, -0.02, 0.03)
    if force == "uniform":
        lat.set_force((1e-4, -2e-5, 3e-5))
    elif force == "field":
        lat.set_force(torch.from_numpy(W.random_force_field(N, 7, 1e-4).astype(np.float32)))
    lat.set_populations(torch.from_numpy(near_rest_state(N, 11)))
    return lat


# one box, its edges and remainders, single rows, columns and planes, the most boxes
SHAPES = [(1, 1, 1), (2, 1, 3), (16, 4, 2), (17, 5, 3), (15, 3, 1), (1, 64, 17), (63, 9, 13), (32, 32, 32), (250, 4, 31)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage,force", [("f32", None), ("f32", "field"), ("f16", "uniform"), ("bf16", "field")])
@pytest.mark.parametrize("solid", [0.0, 0.25])
def test_boxes_equal_single_steps(shape, storage, force, solid):
    N = int(np.prod(shape))
    flags = W.random_flags(N, 5, solid, solid / 3) if solid else np.zeros(N, np.uint8)
    fl = torch.from_numpy(flags == 0).cuda()
    one, two = (_lattice(shape, flags, storage, force) for _ in range(2))
    for n in (2, 5):   # a launch of two; two launches of two and a single step
        for _ in range(n):
            one.step(1)
        two.step(n)
        assert torch.equal(two.populations()[:, fl], one.populations()[:, fl]), (shape, storage, force, n)
    ref = one.step_macros(1) if one.step(3) is None else None
    got = two.step_macros(4)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    one.close()
    two.close()


def test_trajectories_and_checks():
    from paper_1309_1983_amd import LBMError
    shape = (30, 17, 21)
    N = int(np.prod(shape))
    flags = W.random_flags(N, 6, 0.2, 0.05)
    g = torch.from_numpy(W.random_velocity(N, 5, 1.0).astype(np.float32)).cuda()
    out = []
    for kw in ({}, {"cells_per_lane": 1}):   # the option keeps single steps
        lat = _lattice(shape, flags, "f32", "field", **kw)
        lat.forward_checkpointed(11, 4)
        out.append(lat.adjoint(g))
        lat.close()
    assert torch.equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
    # a check after every third step falls between the two steps of a launch
    lat = _lattice(shape, flags, "f32", None, check_interval=3)
    lat.step(2)
    f = lat.populations()
    f[3, int(np.flatnonzero(flags == 0)[1234])] = float("nan")
    lat.set_populations(f)
    with pytest.raises(LBMError, match="NONFINITE"):
        lat.step(2)
    lat.close()
