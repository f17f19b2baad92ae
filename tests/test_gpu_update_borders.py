"""The update of batches at the border of one and two workgroups per table (64, 16, 8 and 4 strips
of 8, 4, 8 and 8 lookups at rows of 16, 64, 128 and 256 floats), with one row that takes all
lookups or all but one, and with none that repeats.  Against numpy in fp64: a sum of n gradients
of size 1 in fp32 is off by at most n * 2^-24 * n, in practice far less: 1e-6 * n asserted.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,full", [(16, 512), (64, 64), (128, 64), (256, 32), (36, 64), (8, 1024)])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_batches_around_one_workgroup(D, full, more):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(D + more)
    T, R, Bc = 3, 5000, full + more
    W = rng.uniform(-1, 1, (T, R, D)).astype(np.float32)
    grad = rng.uniform(-1, 1, (T, Bc, D)).astype(np.float32)
    idx = np.full((T, Bc, 1), 7, np.int32)
    idx[1, Bc // 2] = 3
    idx[2, :, 0] = rng.permutation(R)[:Bc]
    want = W.astype(np.float64)
    for t in range(T):
        np.add.at(want[t], idx[t, :, 0], -0.5 * grad[t].astype(np.float64))
    tb = B.Tables([torch.from_numpy(w.copy()).to(dev) for w in W])
    ws = torch.empty(B.ss_backward_workspace_bytes(T, Bc, 1, D), dtype=torch.uint8, device=dev)
    B.ss_embbag_backward_update(tb, torch.from_numpy(idx).to(dev), None,
                                torch.from_numpy(grad).to(dev), 0.5, ws)
    for t in range(T):
        np.testing.assert_allclose(tb.weights[t].cpu().numpy(), want[t], rtol=1e-6, atol=1e-6 * Bc)
