"""A copy of more work-items than one launch may have (2^32 of four floats each):
the copy probe, and with it the checkpoint of a state of 9.04e8 points and more."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_copy_beyond_one_launch():
    from paper_1309_1983_amd import copy_f32
    n = (1 << 34) + 1003
    if torch.cuda.mem_get_info()[0] < 2 * 4 * n + (8 << 30):
        pytest.skip("needs 145 GB of device memory")
    a, b = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    part = 1 << 28
    for k in range(0, n, part):
        m = min(part, n - k)
        torch.arange(m, device="cuda", dtype=torch.float32, out=a[k:k + m]).add_(float(k // part))
    b.fill_(-1.0)
    copy_f32(a, b)
    for k in range(0, n, part):
        assert torch.equal(a[k:k + part], b[k:k + part]), k
    del a, b
    torch.cuda.empty_cache()
