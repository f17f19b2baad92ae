"""Lookup of short bags at the edges of how its kernels cut their work: bags below 4, below 8,
below 16, and from there on, in launches of one bag per lane group; rows that fill their lanes
and rows that do not, rows of more than 64 f4; n_valid inside a tile.  And
ss_sample_drop for inputs of at most four lookups, which one lane each takes.

The lookup adds rows in bag order in fp32, so numpy's fp32 sum in that order is bit for bit the
same; the counts are integers.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [4, 36, 64, 128, 260])
@pytest.mark.parametrize("L", [2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33])
def test_bags_are_added_in_order(D, L):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(1000 * D + L)
    for T, Bc, nv in ((2, 131, 130), (9, 67, None), (1, 1, None)):
        W = rng.uniform(-1, 1, (T, 300, D)).astype(np.float32)
        idx = rng.integers(0, 300, (T, Bc, L)).astype(np.int32)
        if nv is not None:
            idx[:, nv:] = -1             # bags past n_valid hold no usable index
        n = Bc if nv is None else nv
        out = torch.full((T, Bc, D), 7.0, device=dev)
        n_valid = None if nv is None else torch.tensor([nv], dtype=torch.int32, device=dev)
        tb = B.Tables([torch.from_numpy(w).to(dev) for w in W])
        B.ss_embbag_forward(tb, torch.from_numpy(idx).to(dev), n_valid, out)
        got = out.cpu().numpy()
        for t in range(T):
            want = W[t][idx[t, :n, 0]]
            for l in range(1, L):
                want = want + W[t][idx[t, :n, l]]
            assert np.array_equal(got[t, :n], want), (T, Bc, t)
        assert np.all(got[:, n:] == 7.0)


@pytest.mark.parametrize("T,L,H,S", [(1, 1, 1, 1), (1, 2, 3, 255), (3, 1, 4, 257), (1, 4, 5, 999),
                                     (4, 1, 700, 140_000)])      # several rounds per lane
def test_few_lookups_per_input(T, L, H, S):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(T + L + H + S)
    R = 4 * H + 10
    hot = [np.sort(rng.choice(np.arange(2, R - 2), H, replace=False)).astype(np.int32)
           for _ in range(T)]
    drift = rng.choice([0.0, 1e-4, 2e-4, 1e-3, np.nan], (T, H)).astype(np.float32).astype(float)
    sidx = rng.integers(0, R, (T, S, L)).astype(np.int32)
    for t in range(T):
        at = rng.random((S, L)) < 0.8
        sidx[t][at] = rng.choice(hot[t], at.sum())
    tb = B.Tables([torch.zeros(R, 4, device=dev) for _ in range(T)])
    hs = B.HotState(tb, [torch.from_numpy(h).to(dev) for h in hot])
    row_drift = np.full((T, R), np.nan)
    for t in range(T):
        hs.drift[t].copy_(torch.from_numpy(drift[t]))
        row_drift[t, hot[t]] = drift[t]
    d = np.stack([row_drift[t][sidx[t]] for t in range(T)])
    thr = [5e-4, 0.0, 1e-4, float("inf"), 5e-4, 3e-4]
    counts = torch.full((len(thr) + 1,), -1, dtype=torch.int32, device=dev)
    sidx_d = torch.from_numpy(sidx).to(dev)
    for alpha in range(T * L + 2):
        B.ss_sample_drop(hs, sidx_d, alpha, thr, counts)
        got = counts.cpu().numpy()
        for k, v in enumerate(thr):
            stale = (d <= np.float64(np.float32(v))).sum(axis=(0, 2)) if v > 0 else np.zeros(S, int)
            assert got[k] == (stale >= alpha).sum(), (alpha, k)
        assert got[-1] == -1
