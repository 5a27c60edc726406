"""Sizes at the limits of the launch grids. With the default work-group a row of
nx points takes a group of bx x by points, and ny/by may be at most 65535; rows
that run on a one-dimensional grid keep that limit. The first test runs without a
GPU; the second steps such a lattice."""
import ctypes

import numpy as np
import pytest

import workloads as W


# (nx, by): rows below a wave, of one to four part-filled waves, of whole waves, of 256 and 512 points
@pytest.mark.parametrize("nx,by", [(1, 256), (2, 128), (3, 4), (12, 4), (63, 4), (64, 4), (65, 2), (100, 2), (128, 2),
                                   (130, 1), (200, 1), (260, 1), (512, 1)])
@pytest.mark.parametrize("storage,pattern", [(0, 0), (1, 0), (2, 1)])
def test_limit_of_ny(nx, by, storage, pattern):
    from paper_1309_1983_amd import _abi
    L = _abi.lib()
    out = _abi.lbm_buffer_sizes()
    opt = _abi.lbm_options()
    L.lbm_options_default(ctypes.byref(opt))
    opt.storage, opt.pattern = storage, pattern
    opt.cells_per_lane = 1   # several points per work-item have a limit of their own
    for ny, want in ((65535 * by, _abi.LBM_OK), (65535 * by + 1, _abi.LBM_ERR_INVALID)):
        if nx * ny >= 1 << 30:
            continue
        assert L.lbm_query_buffer_sizes(nx, ny, 1, ctypes.byref(opt), ctypes.byref(out)) == want, (nx, ny)


@pytest.mark.gpu
@pytest.mark.parametrize("nx", [3, 12])
@pytest.mark.parametrize("pattern", ["ab", "aa"])
def test_many_short_rows(nx, pattern):
    import torch
    from paper_1309_1983_amd import Lattice
    from tests.gpu_common import near_rest_state
    shape = (nx, 70000, 2)
    N = int(np.prod(shape))
    flags = W.random_flags(N, 3, 0.1, 0.02)
    fl = torch.from_numpy(flags == 0).cuda()
    s0 = torch.from_numpy(near_rest_state(N, 4))
    got = []
    for kw in ({}, {"block": (4, 64), "cells_per_lane": 1}):   # the second on a two-dimensional grid
        lat = Lattice(*shape, 0.8, flags=flags, pattern=pattern, **kw)
        lat.set_wall_velocity(0.03, -0.01, 0.02)
        lat.set_populations(s0)
        lat.step(5)
        got.append(lat.populations()[:, fl])
        lat.close()
    assert torch.equal(*got)
