"""ss_sample_drop where an input is split over several lanes of a wavefront: 64, 16 and 4 inputs
per workgroup (samples of up to 12288, 4096 and 16384 inputs, inputs of more than 32, 128 and 1024
lookups), at and beside those borders, with remainders of every size.  Integer counts, held to
exact equality with numpy.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def check(T, L, S, H=40):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(T * L + S)
    R = 4 * H + 10
    hot = [np.sort(rng.choice(np.arange(2, R - 2), H, replace=False)).astype(np.int32)
           for _ in range(T)]
    drift = rng.choice([0.0, 1e-4, 2e-4, 1e-3, np.nan], (T, H), p=[.3, .3, .2, .15, .05])
    drift = drift.astype(np.float32).astype(float)
    sidx = rng.integers(0, R, (T, S, L)).astype(np.int32)
    for t in range(T):                   # most lookups hit hot rows
        at = rng.random((S, L)) < 0.8
        sidx[t][at] = rng.choice(hot[t], at.sum())
    tb = B.Tables([torch.zeros(R, 4, device=dev) for _ in range(T)])
    hs = B.HotState(tb, [torch.from_numpy(h).to(dev) for h in hot])
    row_drift = np.full((T, R), np.nan)
    for t in range(T):
        hs.drift[t].copy_(torch.from_numpy(drift[t]))
        row_drift[t, hot[t]] = drift[t]
    thr = [5e-4, 0.0, 1e-4, float("inf"), 2e-4]
    stale = np.zeros((len(thr), S), int)
    for t in range(T):
        d = row_drift[t][sidx[t]]
        for k, v in enumerate(thr):
            if v > 0:
                stale[k] += (d <= np.float64(np.float32(v))).sum(axis=1)
    counts = torch.full((len(thr) + 1,), -1, dtype=torch.int32, device=dev)
    sidx_d = torch.from_numpy(sidx).to(dev)
    middle = [int(np.median(stale[k])) for k in (0, 2, 3)]
    for alpha in sorted({0, 1, T * L, T * L + 1, *middle}):
        B.ss_sample_drop(hs, sidx_d, alpha, thr, counts)
        got = counts.cpu().numpy()
        assert list(got[:-1]) == [(s >= alpha).sum() for s in stale], (T, L, S, alpha)
        assert got[-1] == -1


@pytest.mark.parametrize("T,L", [(4, 8), (3, 11), (16, 8), (3, 43), (26, 20)])   # 32 33 128 129 520
@pytest.mark.parametrize("S", [1, 3, 5, 17, 67, 1001])
def test_few_inputs(T, L, S):
    check(T, L, S)


@pytest.mark.parametrize("T,L,S", [(3, 43, 4095), (3, 43, 4096), (3, 11, 4095), (3, 11, 8191),
                                   (3, 11, 8192), (4, 8, 8191), (3, 43, 4097), (3, 11, 12_288),
                                   (3, 11, 12_289), (33, 32, 4097), (41, 25, 16_384),
                                   (41, 25, 16_385), (32, 32, 4097)])
def test_borders_of_the_sample_size(T, L, S):
    check(T, L, S)


@pytest.mark.parametrize("T,L", [(5, 1), (3, 2), (7, 1), (2, 4), (9, 1)])
@pytest.mark.parametrize("S", [32_768, 32_769])
def test_five_to_eight_lookups_in_registers(T, L, S):
    check(T, L, S)
