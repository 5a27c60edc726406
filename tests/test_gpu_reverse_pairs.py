"""The reverse step with two points per work-item, which lattices of 2^20 points
and more with planes off the 64-byte lines take, against the one-point reverse
step: dL/dF bit for bit, dL/dtau to FP64 summation order."""
import ctypes

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


def _partials(shape, cells_per_lane):
    """Work-groups of the reverse step (a partial sum each): what the adjoint
    workspace holds besides its two states."""
    from paper_1309_1983_amd import _abi
    opt, sizes = _abi.lbm_options(), _abi.lbm_buffer_sizes()
    _abi.lib().lbm_options_default(ctypes.byref(opt))
    opt.cells_per_lane = cells_per_lane
    _abi.call("lbm_query_buffer_sizes", *shape, ctypes.byref(opt), ctypes.byref(sizes))
    return (sizes.adjoint_bytes - 2 * ((sizes.state_bytes + 255) // 256 * 256)) // 8


# 65 pairs a row (one-dimensional grid); 1, 2 and 4 pairs a row (two-dimensional)
@pytest.mark.parametrize("shape", [(130, 90, 92), (2, 725, 724), (4, 513, 513), (8, 363, 363)])
@pytest.mark.parametrize("force", [None, "uniform", "field"])
@pytest.mark.parametrize("solid", [0.0, 0.2])
def test_two_point_reverse_step_equals_one_point(shape, force, solid):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    # groups of two points in 64 work-items against one point in 256
    assert _partials(shape, 0) > 1.5 * _partials(shape, 1), shape
    flags = W.random_flags(N, 8, solid, solid / 4) if solid else None
    gen = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda *s: torch.rand(*s, device="cuda", generator=gen) - 0.5  # noqa: E731
    rho, u, F, g = 1 + 0.02 * rnd(N), 0.04 * rnd(3, N), 2e-3 * rnd(3, N), rnd(3, N)
    out = []
    for cells_per_lane in (0, 1):
        lat = Lattice(*shape, 0.7, flags=flags, cells_per_lane=cells_per_lane)
        lat.set_wall_velocity(0.03, -0.01, 0.02)
        if force == "uniform":
            lat.set_force((1e-4, -2e-4, 3e-5))
        elif force == "field":
            lat.set_force(F)
        lat.init_equilibrium(rho, u)
        lat.forward_checkpointed(5, 2)
        out.append(lat.adjoint(g))
        lat.close()
    assert torch.equal(out[0][0], out[1][0])
    # the same FP32 terms, summed per work-group and then over groups in FP64
    assert abs(out[0][1] - out[1][1]) <= 1e-12 * N * max(1.0, abs(out[0][1]))
