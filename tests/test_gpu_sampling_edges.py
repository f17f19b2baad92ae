"""ss_sample_drop at the edges of how its kernel cuts its work: 64 inputs per workgroup and
round, more inputs than the workgroups that run at once take in one round, hot sets of 1 to 5
rows (the last search step fetches four), lookups in front of, between and behind the hot ids,
thresholds that equal drifts, repeated thresholds, NaN drifts, one wavefront and eight.
Integer counts, held to exact equality with numpy.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,S,L", [
    (1, 1, 63, 1), (1, 2, 64, 2), (2, 3, 65, 1), (2, 4, 129, 3), (3, 5, 1000, 2),
    (9, 1000, 70_001, 1),                # several rounds per workgroup
    (5, 33, 500, 9),                     # more lookups than eight wavefronts take at once
])
def test_counts_match_numpy(T, H, S, L):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(T + H + S + L)
    R = 4 * H + 10
    hot = [np.sort(rng.choice(np.arange(2, R - 2), H, replace=False)).astype(np.int32)
           for _ in range(T)]
    levels = np.float32([0.0, 1e-4, 2e-4, 5e-4, 1e-3, np.nan]).astype(np.float64)
    drift = rng.choice(levels, (T, H))
    sidx = rng.integers(0, R, (T, S, L)).astype(np.int32)
    for t in range(T):                   # most lookups hit hot rows
        at = rng.random((S, L)) < 0.8
        sidx[t][at] = rng.choice(hot[t], at.sum())
    tb = B.Tables([torch.zeros(R, 4, device=dev) for _ in range(T)])
    hs = B.HotState(tb, [torch.from_numpy(h).to(dev) for h in hot])
    for t in range(T):
        hs.drift[t].copy_(torch.from_numpy(drift[t]))
    thr = [5e-4, 0.0, 1e-4, float("inf"), 5e-4, 3e-4, 1e-9]
    row_drift = np.full((T, R), np.nan)
    for t in range(T):
        row_drift[t, hot[t]] = drift[t]
    d = np.stack([row_drift[t][sidx[t]] for t in range(T)])              # [T, S, L]
    counts = torch.full((len(thr) + 1,), -1, dtype=torch.int32, device=dev)
    sidx_d = torch.from_numpy(sidx).to(dev)
    for alpha in sorted({0, 1, T * L // 2, T * L, T * L + 1}):
        B.ss_sample_drop(hs, sidx_d, alpha, thr, counts)
        got = counts.cpu().numpy()
        for k, v in enumerate(thr):
            v32 = np.float64(np.float32(v))
            stale = (d <= v32).sum(axis=(0, 2)) if v > 0 else np.zeros(S, int)
            assert got[k] == (stale >= alpha).sum(), (alpha, k)
        assert got[-1] == -1
