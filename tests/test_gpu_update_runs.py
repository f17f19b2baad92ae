"""The update with runs of every length from 1 to a few strips and beyond, so that runs begin and
end in every strip of a workgroup (64, 32, 16 and 8 strips of 8, 8, 4 and 8 lookups at rows of 16,
32, 64 and 128 floats).  Against numpy in fp64: a sum of n gradients of size 1 in fp32 is off by at
most n * 2^-24 * n, in practice far less: 1e-6 * n asserted.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [8, 16, 28, 32, 64, 128])
@pytest.mark.parametrize("lengths", [range(1, 60), range(60, 90), [7, 8, 9, 64, 65, 72, 73, 100, 4],
                                     [2] * 700])
def test_runs_of_every_length(D, lengths):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(D + sum(lengths))
    T, R = 2, 1000
    W = rng.uniform(-1, 1, (T, R, D)).astype(np.float32)
    rows = [np.repeat(rng.permutation(R)[:len(lengths)], list(lengths)) for _ in range(T)]
    idx = np.stack([rng.permutation(r) for r in rows]).astype(np.int32)[:, :, None]
    n = idx.shape[1]
    grad = rng.uniform(-1, 1, (T, n, D)).astype(np.float32)
    want = W.astype(np.float64)
    for t in range(T):
        np.add.at(want[t], idx[t, :, 0], -0.5 * grad[t].astype(np.float64))
    tb = B.Tables([torch.from_numpy(w.copy()).to(dev) for w in W])
    ws = torch.empty(B.ss_backward_workspace_bytes(T, n, 1, D), dtype=torch.uint8, device=dev)
    B.ss_embbag_backward_update(tb, torch.from_numpy(idx).to(dev), None,
                                torch.from_numpy(grad).to(dev), 0.5, ws)
    for t in range(T):
        np.testing.assert_allclose(tb.weights[t].cpu().numpy(), want[t], rtol=1e-6,
                                   atol=1e-6 * max(lengths))
