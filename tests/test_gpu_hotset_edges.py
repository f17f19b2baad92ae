"""Hot-set identification at the edges of how its kernels cut their work: the three sizes of a
counting workgroup, one and several histogram workgroups per table, the H-th largest count in
an exact bin, in a bin that one or several further passes split, and in the last one; tables
whose counters are only 4-byte aligned; more blocks of rows than the last step sums up by
itself.  Integer work, held to exact equality with numpy.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def select(counts, H):
    """Rows by count (larger first), equal counts by id; the first H, ascending."""
    order = np.lexsort((np.arange(counts.size), -counts.astype(np.int64)))
    return np.sort(order[:H]).astype(np.int32)


@pytest.mark.parametrize("T,Bn,L", [
    (1, 511, 1), (1, 513, 1),            # 256 threads x 2: one workgroup, one and a lookup
    (8, 32_769, 1),                      # 1024 x 2
    (4, 10_241, 21),                     # 1024 x 8, remainder
])
def test_counts(T, Bn, L):
    from paper_2404_04270_amd import binding as B
    rng = np.random.default_rng(T + Bn + L)
    R = 40_000
    idx = ((rng.zipf(1.2, (T, Bn, L)) - 1) % R).astype(np.int32)
    ac = B.AccessCounters(T, R, torch.device("cuda:0"))
    B.ss_count_accesses(ac, torch.from_numpy(idx).cuda())
    for t in range(T):
        assert np.array_equal(ac.counts[t].cpu().numpy(), np.bincount(idx[t].ravel(), minlength=R))


@pytest.mark.parametrize("T,R,top", [
    (1, 8192, 1023), (1, 8193, 1024),    # one histogram workgroup; the last exact bin, the first range
    (3, 30_001, 2047), (3, 30_001, 70_000),       # several; rows of odd tables start unaligned
    (2, 20_003, 0xFFFFFFFF),             # all further passes
    (1, 9_000_000, 3),                   # more than 2048 blocks of 4096 rows
])
def test_top_rows(T, R, top):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(R + top % 1000)
    lo = max(0, top - 5000)              # counts of a narrow range: neighbours differ by one
    counts = rng.integers(lo, top + 1, (T, R), dtype=np.uint64).astype(np.uint32)
    flat = torch.from_numpy(counts.view(np.int32)).to(dev)
    ac = B.AccessCounters(T, R, dev, list(flat.unbind(0)))
    ws = torch.empty(B.ss_select_hot_workspace_bytes(T, R), dtype=torch.uint8, device=dev)
    ws.fill_(0xCD)
    for H in (1, R // 7, R - 1):
        ids = [torch.full((H,), -7, dtype=torch.int32, device=dev) for _ in range(T)]
        bits = [torch.full(((R + 31) // 32,), -1, dtype=torch.int32, device=dev) for _ in range(T)]
        B.ss_select_hot_top(ac, H, ids, bits, ws)
        for t in range(T):
            want = select(counts[t], H)
            assert np.array_equal(ids[t].cpu().numpy(), want), (H, t)
            mask = np.zeros(bits[t].numel() * 32, bool)
            mask[want] = True
            assert np.array_equal(bits[t].cpu().numpy().view(np.uint32),
                                  np.packbits(mask, bitorder="little").view(np.uint32)), (H, t)
