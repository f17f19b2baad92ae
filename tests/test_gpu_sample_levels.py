"""ss_sample_levels + ss_level_counts against ss_sample_drop with alpha = T * L: the same whole numbers
for every form of input; and the threshold search that takes them against the one over
ss_sample_drop."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _hot(T, R, H, gen, odd):
    from paper_2404_04270_amd import binding as B
    tables = B.Tables([torch.zeros(R, 4, device="cuda") for _ in range(T)])
    ids = [torch.randperm(R, device="cuda", generator=gen)[:H].sort().values.int()
           for _ in range(T)]
    hot = B.HotState(tables, ids, diagnostics=True)
    for d in hot.drift:
        d.copy_(10.0 ** (torch.rand(H, device="cuda", dtype=torch.float64, generator=gen) * 4 - 5))
        if odd and H > 2:
            d[0], d[1], d[2] = float("nan"), float("inf"), 0.0
    return tables, hot, ids


@pytest.mark.parametrize("T,R,H,S,L,cold", [
    (1, 50, 1, 1, 1, 0.0), (1, 50, 3, 300, 1, 0.1), (2, 60, 4, 1000, 2, 0.0), (3, 70, 5, 64, 3, 0.02),
    (26, 4000, 500, 4097, 1, 0.001), (26, 4000, 300, 65, 5, 0.0), (8, 900, 100, 5000, 16, 0.001),
    (4, 900, 100, 300, 300, 0.0), (1, 400, 40, 131072, 1, 0.2), (1, 400, 40, 131073, 1, 0.2),
    (2, 400, 40, 300000, 2, 0.1), (1, 400, 40, 65536, 2, 0.2), (2, 400, 40, 65537, 1, 0.2),
    (1, 400, 40, 3, 2, 0.0),
])
@pytest.mark.parametrize("odd", [False, True])
def test_levels_count_what_sample_drop_counts(T, R, H, S, L, cold, odd):
    from paper_2404_04270_amd import binding as B
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T * 7919 + S)
    _, hot, ids = _hot(T, R, H, gen, odd)
    sidx = torch.stack([i[torch.randint(0, H, (S, L), device="cuda", generator=gen)] for i in ids])
    other = torch.rand(T, S, L, device="cuda", generator=gen) < cold
    sidx[other] = torch.randint(-1, R + 2, (int(other.sum()),), device="cuda", generator=gen,
                                dtype=torch.int32)
    levels = torch.full((S,), -7.0, device="cuda")
    B.ss_sample_levels(hot, sidx, levels)
    some = float(np.float32(hot.drift[0][-1].item()))
    thr = [1e-2, 0.0, some, 1e-5, math.inf, 3e-4, -1.0, 1e30, 1e-4, 1e-3] + \
        [10.0 ** (-5 + 4 * k / 53) for k in range(54)]
    assert len(thr) == B.MAX_LEVEL_THRESHOLDS
    got = torch.full((len(thr),), 77, dtype=torch.int32, device="cuda")
    want = torch.empty(len(thr), dtype=torch.int32, device="cuda")
    for n in (1, len(thr)):
        B.ss_level_counts(levels, thr[:n], got)
        for k in range(0, n, B.MAX_THRESHOLDS):
            part = thr[:n][k:k + B.MAX_THRESHOLDS]
            B.ss_sample_drop(hot, sidx, T * L, part, want[k:])
        assert torch.equal(got[:n], want[:n])
    assert torch.equal(got, want)


def test_levels_of_another_length_are_refused():
    # ss_level_counts counts all of its levels: a tail that no sample filled would be counted too
    from paper_2404_04270_amd import binding as B
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    _, hot, ids = _hot(2, 100, 10, gen, False)
    sidx = torch.stack([i[torch.randint(0, 10, (50, 1), device="cuda", generator=gen)] for i in ids])
    for n in (49, 51, 64):
        levels = torch.zeros(n, device="cuda")
        with pytest.raises(B.SlipstreamError):
            B.ss_sample_levels(hot, sidx, levels)
        assert not bool(levels.any())
    buffer = torch.zeros(64, device="cuda")
    B.ss_sample_levels(hot, sidx, buffer[:50])
    assert bool((buffer[:50] > 0).all()) and not bool(buffer[50:].any())


def test_no_hot_rows():
    from paper_2404_04270_amd import binding as B
    empty = torch.zeros(1, 1, dtype=torch.int64, device="cuda")
    levels = torch.zeros(5, device="cuda")
    sidx = torch.zeros(1, 5, 2, dtype=torch.int32, device="cuda")
    B._check(B._lib.ss_sample_levels(1, empty.data_ptr(), 0, empty.data_ptr(), sidx.data_ptr(), 5, 2,
                                     levels.data_ptr(), B._stream_ptr(None)))
    assert bool(levels.isnan().all())


@pytest.mark.parametrize("budget,passes", [(0.2, 2), (0.2, 0), (0.2, 1), (0.7, 3), (0.0, 2), (1.5, 2),
                                           (-1.0, 2)])
def test_search_is_the_same(budget, passes):
    from paper_2404_04270_amd import binding as B
    from paper_2404_04270_amd.sampling import SamplingBlock, ladder_search
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    tables, hot, ids = _hot(4, 3000, 200, gen, False)
    sidx = torch.stack([i[torch.randint(0, 200, (3000, 1), device="cuda", generator=gen)]
                        for i in ids])
    block = SamplingBlock(tables, hot, sidx, alpha=4, population=100000)
    got = block.find_threshold(budget, 1e-6, 1e-1, passes)
    want = ladder_search(lambda ts: [e["hi"] for e in block.estimate(ts)], 1e-6, 1e-1, budget,
                         passes, B.MAX_THRESHOLDS)
    assert got == want


def test_searches_of_one_block_from_two_threads():
    import threading
    from paper_2404_04270_amd.sampling import SamplingBlock
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    tables, hot, ids = _hot(4, 3000, 200, gen, False)
    sidx = torch.stack([i[torch.randint(0, 200, (3000, 1), device="cuda", generator=gen)]
                        for i in ids])
    block = SamplingBlock(tables, hot, sidx, alpha=4, population=100000)
    ranges = [(0.2, 1e-6, 1e-1), (0.5, 1e-5, 1e-2)]
    want = [block.find_threshold(*r) for r in ranges]
    torch.cuda.synchronize()
    wrong, errors = [0, 0], []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(40):
                    wrong[k] += block.find_threshold(*ranges[k]) != want[k]
        except Exception as e:         # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors and wrong == [0, 0], (errors, wrong)
