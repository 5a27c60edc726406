"""16-bit two-array lattices beyond the cache whose rows do not fill waves and
whose planes begin off the lines: a row per work-group, against other groups."""
import numpy as np
import pytest
import torch

from tests.gpu_common import near_rest_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_1309_1983_amd
    paper_1309_1983_amd.lib()


# the first and last row lengths of the range (193, 1023), one point more than
# whole waves, and one less
@pytest.mark.parametrize("shape,storage", [((193, 151, 155), "f16"), ((257, 133, 132), "bf16"), ((511, 93, 94), "f16"),
                                           ((513, 93, 95), "bf16"), ((1023, 63, 70), "f16")])
def test_a_row_per_group_equals_other_groups(shape, storage):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    flags = np.zeros(N, np.uint8)
    flags[np.random.RandomState(8).choice(N, N // 50, replace=False)] = 2
    s0 = torch.from_numpy(near_rest_state(N, 5))
    out = []
    for options in ({}, {"block": (64, 2)}):
        lat = Lattice(*shape, 0.8, flags=flags, storage=storage, **options)
        lat.set_wall_velocity(0.02, 0.01, -0.03)
        lat.set_populations(s0)
        lat.step(3)
        rho, u = lat.step_macros(1)
        out.append((lat.populations(), rho.clone(), u.clone()))
        lat.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
