"""Forms that only large lattices choose, against small ones that do not: a
lattice whose flags, state, force and loss gradient repeat with a period in y
and z evolves as the periodic lattice of one period does, bit for bit (the
arithmetic of a point depends on its neighbours' values alone).

Covered: non-temporal stores of the one-point step (AB arrays of more than
256 MiB together, rows on 64-byte lines), the one-point reverse step with
them, and the reverse step with two points per work-item (2^20 points and
more, planes off the 64-byte lines)."""
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


def _tile(a, shape, ry, rz):
    nx, ny, nz = shape
    a = np.asarray(a)
    return np.tile(a.reshape(a.shape[:-1] + (nz, ny, nx)), (1,) * (a.ndim - 1) + (rz, ry, 1)).reshape(a.shape[:-1] + (-1,))


def _tile_t(t, shape, ry, rz):
    nx, ny, nz = shape
    lead = t.shape[:-1]
    return t.reshape(*lead, nz, ny, nx).repeat(*(1,) * len(lead), rz, ry, 1).reshape(*lead, -1)


@pytest.mark.parametrize("storage,shape", [("f32", (64, 84, 84)), ("f16", (128, 84, 84)), ("bf16", (96, 98, 98))])
@pytest.mark.parametrize("solid", [0.0, 0.3])
def test_streamed_steps_equal_one_period(storage, shape, solid):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    flags = W.random_flags(N, 3, solid, solid / 5) if solid else np.zeros(N, np.uint8)
    s0, F = near_rest_state(N, 4), W.random_force_field(N, 5, 1e-4).astype(np.float32)
    got = []
    for rep in (1, 2):
        sh = (shape[0], shape[1] * rep, shape[2] * rep)
        lat = Lattice(*sh, 0.8, flags=_tile(flags, shape, rep, rep), storage=storage)
        lat.set_wall_velocity(0.05, -0.02, 0.03)
        lat.set_force(torch.from_numpy(_tile(F, shape, rep, rep)))
        lat.set_populations(torch.from_numpy(_tile(s0, shape, rep, rep)))
        lat.step(3)
        rho, u = lat.macros()
        lat.check_finite()
        fl = torch.from_numpy(_tile(flags, shape, rep, rep) == 0).cuda()
        got.append((lat.populations() * fl, rho * fl, u * fl))
        lat.close()
    for a, b in zip(*got):
        assert torch.equal(_tile_t(a, shape, 2, 2), b), (storage, shape, solid)


# the first repeats to more than 256 MiB on aligned rows; the second to 2^20 points off the lines
@pytest.mark.parametrize("shape", [(128, 60, 60), (130, 45, 46)])
@pytest.mark.parametrize("solid", [0.0, 0.2])
def test_large_reverse_steps_equal_one_period(shape, solid):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    flags = W.random_flags(N, 7, solid, solid / 4) if solid else np.zeros(N, np.uint8)
    s0, F = near_rest_state(N, 8), W.random_force_field(N, 9, 1e-3).astype(np.float32)
    g = W.random_velocity(N, 10, 1.0).astype(np.float32)
    got = []
    for rep in (1, 2):
        sh = (shape[0], shape[1] * rep, shape[2] * rep)
        lat = Lattice(*sh, 0.7, flags=_tile(flags, shape, rep, rep))
        lat.set_wall_velocity(0.03, -0.01, 0.02)
        lat.set_force(torch.from_numpy(_tile(F, shape, rep, rep)))
        lat.set_populations(torch.from_numpy(_tile(s0, shape, rep, rep)))
        lat.forward_checkpointed(5, 2)
        gF, gt = lat.adjoint(torch.from_numpy(_tile(g, shape, rep, rep)).cuda())
        got.append((gF.clone(), gt))
        lat.close()
    assert torch.equal(_tile_t(got[0][0], shape, 2, 2), got[1][0])
    # four times the same FP32 terms, summed in FP64 in another order
    assert abs(got[1][1] - 4 * got[0][1]) <= 1e-12 * 4 * N * max(1.0, abs(got[0][1]))
