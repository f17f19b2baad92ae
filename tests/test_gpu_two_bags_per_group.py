"""Lookup of bags of 2 to 7 at the border where a lane group takes two of them (2048 workgroups
with one each): one below it, at it and beyond, an odd number of bags per group, n_valid inside
a tile, rows that fill their lanes and rows that do not, rows of more than 64 f4.  Rows are added
in bag order in fp32, so numpy's fp32 sum in that order is bit for bit the same.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,groups", [(4, 256), (36, 16), (64, 16), (260, 4)])
@pytest.mark.parametrize("L", [2, 3, 4, 7])
@pytest.mark.parametrize("T,tiles,rest,nv", [(1, 2047, 0, None), (1, 2048, 0, None),
                                             (8, 256, -1, 3), (3, 683, 1, 2)])
def test_two_bags_per_group(D, groups, L, T, tiles, rest, nv):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(D + L + tiles)
    Bc = tiles * groups + rest
    n = Bc if nv is None else Bc - groups - nv
    W = rng.uniform(-1, 1, (T, 50, D)).astype(np.float32)
    idx = rng.integers(0, 50, (T, Bc, L)).astype(np.int32)
    idx[:, n:] = -1                      # bags past n_valid hold no usable index
    out = torch.full((T, Bc, D), 7.0, device=dev)
    n_valid = None if nv is None else torch.tensor([n], dtype=torch.int32, device=dev)
    tb = B.Tables([torch.from_numpy(w).to(dev) for w in W])
    B.ss_embbag_forward(tb, torch.from_numpy(idx).to(dev), n_valid, out)
    got = out.cpu().numpy()
    for t in range(T):
        want = W[t][idx[t, :n, 0]]
        for l in range(1, L):
            want = want + W[t][idx[t, :n, l]]
        assert np.array_equal(got[t, :n], want), t
    assert np.all(got[:, n:] == 7.0)
