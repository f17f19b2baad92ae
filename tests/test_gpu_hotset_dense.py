"""Selections that take many rows (wavefronts that write a row per lane), few, and both in one
table: equal counts cut in the middle of a bitmap word, at its ends and at the ends of a
wavefront's 8192 rows, caps inside a dense stretch, tables that end inside a word.  Held to
exact equality with numpy.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def counts_of(kind, R, rng):
    if kind == "const":
        return np.full(R, 5, np.int64)
    if kind == "flat":
        return rng.poisson(3.0, R)
    if kind == "blocks":                 # dense and empty stretches of odd lengths
        return np.where((np.arange(R) // 611) % 3 == 0, 9, 0) + (rng.random(R) < 0.01)
    return rng.integers(0, 1 << 31, R)


@pytest.mark.parametrize("kind", ["const", "flat", "blocks", "wide"])
@pytest.mark.parametrize("R", [31, 1000, 8192, 8193, 40_000, 65_537])
def test_dense_selections(kind, R):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(R + len(kind))
    T = 2
    cnt = np.stack([counts_of(kind, R, rng) for _ in range(T)])
    c = B.AccessCounters(T, R, dev)
    for t in range(T):
        c.counts[t].copy_(torch.from_numpy(cnt[t].astype(np.int32)))
    ws = torch.empty(B.ss_select_hot_workspace_bytes(T, R), dtype=torch.uint8, device=dev)
    words = (R + 31) // 32

    def outputs(n):
        return ([torch.full((n + 3,), -7, dtype=torch.int32, device=dev) for _ in range(T)],
                [torch.full((words + 1,), -7, dtype=torch.int32, device=dev) for _ in range(T)])

    def check(ids, bits, t, want, cap):
        got = ids[t].cpu().numpy()
        n = min(cap, len(want))
        assert np.array_equal(got[:n], want[:n]) and np.all(got[n:] == -7)
        flags = np.zeros(words * 32, bool)
        flags[want] = True
        b = bits[t].cpu().numpy().astype(np.uint32)
        assert np.array_equal(b[:-1], np.packbits(flags, bitorder="little").view(np.uint32))
        assert b[-1] == np.uint32(-7 & 0xFFFFFFFF)

    for H in sorted({1, 7, 32, 33, R // 3, R // 2, 8192, R - 1, R} & set(range(1, R + 1))):
        ids, bits = outputs(H)
        B.ss_select_hot_top(c, H, ids, bits, ws)
        for t in range(T):
            order = np.argsort(-cnt[t], kind="stable")[:H]
            check(ids, bits, t, np.sort(order), H)
    for lam, cap in ((0.0, R), (0.0, R // 2 + 1), (4 / 1000, R), (4 / 1000, R // 5 + 1)):
        ids, bits = outputs(cap)
        ids = [x[:cap] for x in ids]
        n_hot = torch.zeros(T, dtype=torch.int32, device=dev)
        B.ss_select_hot_ratio(c, lam, 1000, ids, bits, n_hot, ws)
        for t in range(T):
            want = np.flatnonzero(cnt[t] / 1000 >= lam)
            check(ids, bits, t, want, cap)
            assert int(n_hot[t]) == len(want)
