"""lbm_step takes steps two per launch on large two-array lattices (the
two-step kernel). Both of its steps do the one-step kernels' arithmetic on
values rounded to the storage format in between, so n steps in one call equal
n calls of one step bit for bit on every fluid point."""
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


def _state(N, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rho = 1 + 0.02 * (torch.rand(N, device="cuda", generator=g) - 0.5)
    u = 0.04 * (torch.rand(3, N, device="cuda", generator=g) - 0.5)
    return rho, u


def _flags(kind, shape):
    N = int(np.prod(shape))
    if kind == "random":   # every neighbour pattern, moving walls among them
        return W.random_flags(N, 5, 0.15, 0.05)
    if kind == "random_resting":
        return W.random_flags(N, 6, 0.1, 0.0)
    return {"cavity": W.cavity_flags, "duct": W.duct_flags, "onsite": W.onsite_cavity_flags}[kind](*shape) if kind else None


CASES = [
    # (shape, geometry, storage, force): tiles of 64-66 columns and up to 13 rows
    ((131, 97, 83), "random", "f32", "field"),            # odd rows, ragged last tiles
    ((128, 104, 80), "cavity", "f32", None),              # whole tiles, moving lid
    ((160, 130, 90), "random_resting", "f32", "uniform"),  # last tile half wide
    ((98, 110, 100), "duct", "f32", "field"),
    ((133, 90, 88), None, "f32", None),                   # periodic: row ends wrap
    ((64, 150, 110), None, "f32", "field"),               # one tile per row, wrapping onto itself
    ((131, 130, 228), None, "f16", "field"),
    ((128, 130, 228), None, "bf16", "field"),
    ((66, 260, 228), None, "f16", None),
    ((132, 131, 131), "onsite", "f32", None),             # on-site nodes on faces, edges and corners
    ((223, 120, 100), "onsite", "f32", None),
    ((140, 110, 98), "cavity", "f32", None),              # 47 columns taken as 48
    ((184, 130, 150), None, "f16", None),                  # 62 as 64
]


def _lattice(shape, flags, storage, force, **kw):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    lat = Lattice(*shape, 0.7, flags=flags, storage=storage, **kw)
    lat.set_wall_velocity(0.05, -0.02, 0.03)
    if force == "uniform":
        lat.set_force((1e-5, -2e-5, 3e-6))
    elif force == "field":
        lat.set_force(torch.from_numpy(W.random_force_field(N, 7, 1e-4).astype(np.float32)))
    lat.init_equilibrium(*_state(N, 11))
    return lat


@pytest.mark.parametrize("case", range(len(CASES)))
def test_two_steps_per_launch_equal_single_steps(case):
    shape, kind, storage, force = CASES[case]
    flags = _flags(kind, shape)
    fl = slice(None) if flags is None else torch.from_numpy((flags != 1) & (flags != 2)).cuda()
    one, two = (_lattice(shape, flags, storage, force) for _ in range(2))
    assert "k_step_pair" in two.step_kernel_name(), (shape, two.step_kernel_name())
    done = 0
    for n in (2, 5):   # a pair; two pairs and a single step
        for _ in range(n):
            one.step(1)
        two.step(n)
        done += n
        assert torch.equal(two.populations()[:, fl], one.populations()[:, fl]), (CASES[case], done)
    one.close()
    two.close()


def test_pairs_leave_output_steps_checks_and_options_as_they_are():
    from paper_1309_1983_amd import LBMError
    shape, kind, storage, force = CASES[0]
    flags = _flags(kind, shape)
    fl = torch.from_numpy(flags == 0).cuda()
    one, two = (_lattice(shape, flags, storage, force) for _ in range(2))
    for _ in range(3):
        one.step(1)
    ref = one.step_macros(1)
    got = two.step_macros(4)      # a pair, a single step, the storing step
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    assert torch.equal(two.populations()[:, fl], one.populations()[:, fl])
    one.close()
    two.close()
    # a check after every third step falls between the two steps of a pair
    lat = _lattice(shape, flags, storage, force, check_interval=3)
    lat.step(2)
    f = lat.populations()
    f[3, int(torch.nonzero(fl)[1234])] = float("nan")
    lat.set_populations(f)
    with pytest.raises(LBMError, match="NONFINITE"):
        lat.step(2)
    lat.close()
    # on-site nodes under a force, or beside moving walls, keep single steps
    flags = _flags("onsite", (223, 120, 100))
    lat = _lattice((223, 120, 100), flags, "f32", "uniform")
    assert "k_step_pair" not in lat.step_kernel_name()
    lat.close()
    flags[(flags == 1) & (np.arange(flags.size) < 223 * 120)] = 2
    lat = _lattice((223, 120, 100), flags, "f32", None)
    assert "k_step_pair" not in lat.step_kernel_name()
    lat.close()
    # the event log and the one-step kernel's options keep single steps
    for kw in ({"timing": 8}, {"cells_per_lane": 1}, {"block": (64, 1)}, {"gather_mode": "early", "cells_per_lane": 0},
               {"groups_per_cu": -1}):
        lat = _lattice((128, 104, 80), _flags("cavity", (128, 104, 80)), "f32", None, **kw)
        assert "k_step_pair" not in lat.step_kernel_name(), kw
        lat.step(3)
        if "timing" in kw:
            assert len(lat.step_times()) == 3
        lat.close()
