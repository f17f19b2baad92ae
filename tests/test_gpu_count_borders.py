"""ss_count_accesses at the borders of its workgroups (2048 and 8192 lookups) and of the rule that
picks them (524288 lookups in all), with remainders, n_valid inside a workgroup's lookups, one row
that takes them all and popular rows next to each other.  Held to exact equality with numpy.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,Bc,L,nv", [
    (1, 1, 1, None), (1, 2047, 1, None), (3, 2049, 1, 2048), (2, 683, 3, 600), (7, 8191, 1, 0),
    (1, 524_287, 1, None), (1, 524_288, 1, 524_287), (64, 8192, 1, 8191), (5, 34_953, 3, 30_001),
])
def test_counts_match_numpy(T, Bc, L, nv):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(T + Bc + L)
    R, n = 5000, Bc if nv is None else nv
    idx = np.minimum(rng.zipf(1.3, (T, Bc, L)), R) - 1
    idx[0] = 17                                      # one table: one row
    c = B.AccessCounters(T, R, dev)
    n_valid = None if nv is None else torch.tensor([nv], dtype=torch.int32, device=dev)
    for _ in range(2):                               # counters accumulate
        B.ss_count_accesses(c, torch.from_numpy(idx.astype(np.int32)).to(dev), n_valid)
    for t in range(T):
        want = 2 * np.bincount(idx[t, :n].reshape(-1), minlength=R)
        assert np.array_equal(c.counts[t].cpu().numpy(), want), t
