"""Steps captured into a HIP graph: the two arrays are swapped after every
step, so a graph of an even number of steps finds the state where it left it
and advances the flow by that number at every replay, with the program's own
steps between the replays; two graphs of an odd number each, captured one
after the other, advance it in turn."""
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


# two steps per launch through boxes and through tiles, one step per launch
# between two arrays, and in place
@pytest.mark.parametrize("shape,pattern", [((32, 20, 18), "ab"), ((128, 128, 64), "ab"), ((64, 64, 64), "ab"),
                                           ((32, 20, 18), "aa")])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 6, 7])
@pytest.mark.parametrize("own", [False, True])
def test_replayed_steps_advance_the_flow(shape, pattern, n, own):
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    s0 = torch.from_numpy(near_rest_state(N, 5))
    flags = W.cavity_flags(*shape)
    fl = torch.from_numpy(flags == 0).cuda()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())

    def lattice(**kw):
        lat = Lattice(*shape, 0.7, flags=flags, pattern=pattern, stream=stream, **kw)
        lat.set_wall_velocity(0.05, 0.0, 0.02)
        lat.set_populations(s0)
        return lat

    with torch.cuda.stream(stream):
        ref = lattice(cells_per_lane=1)   # one step per launch
        lat = lattice(torch_buffers=own)
        assert ("k_step_pair<" in lat.step_kernel_name()) == (shape == (128, 128, 64))
        lat.step(7)   # also loads the kernels, which a capture must not do
        lat.set_populations(s0)
        stream.synchronize()
        graphs = [torch.cuda.CUDAGraph() for _ in range(1 + n % 2)]
        for g in graphs:
            with torch.cuda.graph(g, stream=stream):
                lat.step(n)
        stream.synchronize()
        for k in range(3):
            for g in graphs:
                g.replay()
            ref.step(n * len(graphs))
            assert torch.equal(lat.populations()[:, fl], ref.populations()[:, fl]), ("replay", k)
            lat.step(2)
            ref.step(2)
            assert torch.equal(lat.populations()[:, fl], ref.populations()[:, fl]), ("steps after replay", k)
            stream.synchronize()
    lat.close()
    ref.close()


@pytest.mark.parametrize("shape", [(32, 20, 18), (128, 64, 64)])
@pytest.mark.parametrize("n", [2, 4, 5])
def test_fields_captured_once_follow_the_steps(shape, n):
    """rho and u read by a graph captured before the steps: an even number of
    steps ends in the array that the graph reads."""
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        lat = Lattice(*shape, 0.7, stream=stream)
        lat.set_populations(torch.from_numpy(near_rest_state(N, 6)))
        lat.step(4)
        lat.macros()
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            rho, u = lat.macros()
        for k in range(3):
            lat.step(n)
            if n % 2:
                lat.step(n)
            g.replay()
            r, v = lat.macros()
            assert torch.equal(rho, r) and torch.equal(u, v), k
            stream.synchronize()
        lat.close()


@pytest.mark.parametrize("shape", [(32, 20, 18), (128, 128, 64)])
@pytest.mark.parametrize("T,K", [(1, 1), (2, 1), (2, 5), (5, 5), (6, 3), (12, 6), (13, 6), (14, 6)])
def test_rollouts_end_in_the_array_that_single_steps_end_in(shape, T, K):
    """The fields after a rollout, read by a graph captured before it: after
    one of an even number of steps, or after two of an odd number."""
    from paper_1309_1983_amd import Lattice
    N = int(np.prod(shape))
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        one = Lattice(*shape, 0.7, stream=stream, cells_per_lane=1)   # one step per launch
        lat = Lattice(*shape, 0.7, stream=stream)
        assert ("k_step_pair<" in lat.step_kernel_name()) == (shape == (128, 128, 64))
        s0 = torch.from_numpy(near_rest_state(N, 6))
        for x in (one, lat):
            x.set_populations(s0)
        lat.macros()
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            rho, u = lat.macros()
        for _ in range(3):
            for _ in range(1 + T % 2):
                lat.forward_checkpointed(T, K)
                one.step(T)
            g.replay()
            r, v = one.macros()
            assert torch.equal(rho, r) and torch.equal(u, v)
            r, v = lat.macros()
            assert torch.equal(rho, r) and torch.equal(u, v)
            stream.synchronize()
        lat.close()
        one.close()
