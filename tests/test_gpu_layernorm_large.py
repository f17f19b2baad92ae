"""ss_embbag_forward_ln on a batch whose workgroups, one vector per lane group, pass 2^32 threads
(64 GiB of y): the last vectors are written as the first ones are.  fp32 vectors of 64 values of
size 1: 1e-5 of them is the bound of the repository's other normalization tests.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_more_than_two_to_the_32_threads():
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    n, D, L, R = (1 << 28) + 1, 64, 2, 1000
    if torch.cuda.mem_get_info(dev)[0] < 90 << 30:
        pytest.skip("needs 90 GiB of free device memory")
    w = torch.randn(R, D, device=dev)
    idx = torch.randint(0, R, (1, n, L), device=dev, dtype=torch.int32)
    y = torch.zeros(1, n, D, device=dev)
    mean, rstd = torch.zeros(1, n, device=dev), torch.zeros(1, n, device=dev)
    B.ss_embbag_forward_ln(B.Tables([w]), idx, None, None, None, 1e-5, y, mean, rstd)
    for part in (slice(0, 1000), slice(n // 2, n // 2 + 1000), slice(n - 1000, n)):
        x = w[idx[0, part].long()].sum(1)
        want = torch.nn.functional.layer_norm(x.double(), (D,), eps=1e-5)
        assert torch.allclose(y[0, part].double(), want, rtol=1e-5, atol=1e-5)
    del y, idx, mean, rstd
    torch.cuda.empty_cache()
