"""Rows that do not fill whole waves run on a one-dimensional grid over each
plane; an explicit work-group shape keeps the two-dimensional one. Both give
the same values: steps, state and fields on the fluid points, and the adjoint
against a lattice whose rows are cut into the same points differently."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_common import near_rest_state

pytestmark = pytest.mark.gpu

Q = 19


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1309_1983_amd
    paper_1309_1983_amd.lib()


# row lengths around a wave and its quarters, one point and four points per work-item
@pytest.mark.parametrize("nx", [1, 3, 63, 65, 127, 132, 12, 252])
@pytest.mark.parametrize("storage,pattern", [("f32", "ab"), ("f16", "aa"), ("bf16", "ab")])
def test_flat_rows_equal_two_dimensional_grid(nx, storage, pattern):
    from paper_1309_1983_amd import Lattice
    shape = (nx, 7, 5)
    N = int(np.prod(shape))
    flags = W.random_flags(N, 3, 0.15, 0.05)
    s0 = torch.from_numpy(near_rest_state(N, 4))
    F = torch.from_numpy(W.random_force_field(N, 5, 1e-4).astype(np.float32))
    fl = torch.from_numpy(flags == 0).cuda()
    got = []
    for kw in ({}, {"block": (64, 2), "cells_per_lane": 1}):
        lat = Lattice(*shape, 0.8, flags=flags, storage=storage, pattern=pattern, **kw)
        lat.set_wall_velocity(0.05, -0.02, 0.03)
        lat.set_force(F)
        lat.set_populations(s0)
        lat.step(3)
        rho, u = lat.macros()
        got.append((lat.populations()[:, fl], rho, u))
        lat.check_finite()
        lat.close()
    for a, b in zip(*got):
        assert torch.equal(a, b), (shape, storage, pattern)


@pytest.mark.parametrize("nx", [66, 126, 130])
def test_adjoint_on_flat_rows_equals_one_point_reverse_step(nx):
    """Two points per work-item on a one-dimensional grid against one point
    per work-item: dL/dF bit for bit, dL/dtau to FP64 summation order."""
    from paper_1309_1983_amd import Lattice
    shape = (nx, 6, 5)
    N = int(np.prod(shape))
    flags = W.random_flags(N, 8, 0.15, 0.05)
    F = torch.from_numpy(W.random_force_field(N, 9, 1e-3).astype(np.float32))
    g = torch.from_numpy(W.random_velocity(N, 10, 1.0).astype(np.float32)).cuda()
    out = []
    for kw in ({}, {"cells_per_lane": 1}):
        lat = Lattice(*shape, 0.7, flags=flags, **kw)
        lat.set_wall_velocity(0.03, -0.01, 0.02)
        lat.set_force(F)
        lat.set_populations(torch.from_numpy(near_rest_state(N, 11)))
        lat.forward_checkpointed(5, 2)
        out.append(lat.adjoint(g))
        lat.close()
    assert torch.equal(out[0][0], out[1][0])
    # the same FP32 terms, summed per work-group and then over groups in FP64
    assert abs(out[0][1] - out[1][1]) <= 1e-12 * N * max(1.0, abs(out[0][1]))
