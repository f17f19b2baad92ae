"""The one-launch grouping of a table's lookups, at the borders of its plan: no lookup may be lost,
doubled or filed under another row.  Weights, gradients and the learning rate are small whole
numbers, so every sum is exact in fp32 whatever its order and the result has to be equal."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _rows(kind, shape, R, gen):
    dev = "cuda"
    if kind == "one":                      # a single class holds all lookups
        return torch.full(shape, R - 1, device=dev)
    if kind == "few":                      # rows a power of two apart, below the votes of a heavy row
        n = max(1, min(25, R // 64))
        return torch.randint(0, n, shape, device=dev, generator=gen) * (R // n)
    if kind == "uniform":
        return torch.randint(0, R, shape, device=dev, generator=gen)
    u = torch.rand(shape, device=dev, dtype=torch.float64, generator=gen)       # skewed
    return ((R + 1.0) ** (u ** 3) - 1.0).long().clamp_(0, R - 1)


@pytest.mark.parametrize("T,R,B,L,kind,stale", [
    (1, 1, 1, 1, "one", 0.0), (2, 2, 300, 1, "uniform", 0.0),
    (3, 64, 255, 1, "skewed", 0.3), (3, 64, 256, 1, "one", 0.0), (3, 4096, 257, 1, "few", 0.0),
    (5, 1000, 128, 4, "skewed", 0.5), (5, 1000, 171, 3, "uniform", 1.0),
    (40, 5000, 1000, 1, "skewed", 0.1), (7, 65536, 2048, 1, "few", 0.2),
    (9, 65537, 2049, 1, "skewed", 0.0), (100, 500, 4096, 1, "uniform", 0.0),
    (2, 1 << 20, 4097, 1, "few", 0.0), (26, 100000, 8192, 1, "skewed", 0.2),
    (30, 300, 8191, 1, "uniform", 0.0), (1, 1 << 20, 16384, 1, "one", 0.0),
    (1, 1 << 20, 16383, 1, "few", 0.0), (70, 3000, 16384, 1, "skewed", 0.1),
    (1, 200_000_000, 8192, 1, "skewed", 0.0),          # row and position need 64 bits
    (2, 20_000_000, 700, 20, "uniform", 0.3),
])
def test_grouping_loses_nothing(T, R, B, L, kind, stale):
    from paper_2404_04270_amd import binding as Bd
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T * 1000003 + B * 31 + L)
    D = 4
    weights = [torch.zeros(R, D, device="cuda") for _ in range(T)]
    tables = Bd.Tables(weights)
    bits = tables.new_bits()
    idx = _rows(kind, (T, B, L), R, gen)
    flagged = torch.zeros(T, R, dtype=torch.bool, device="cuda") if stale else None
    if stale:
        for t in range(T):
            rows = idx[t].unique()
            rows = rows[torch.rand(rows.numel(), device="cuda", generator=gen) < stale]
            flagged[t, rows] = True
            word = torch.zeros(bits[t].numel(), dtype=torch.int64, device="cuda")
            word.index_add_(0, rows >> 5, torch.ones_like(rows) << (rows & 31))
            bits[t].copy_(torch.where(word >= 1 << 31, word - (1 << 32), word))
    n = B - B // 3
    n_valid = torch.tensor([n], dtype=torch.int32, device="cuda")
    grad = torch.randint(-8, 9, (T, B, D), device="cuda", generator=gen).float()
    ws = torch.empty(Bd.ss_backward_workspace_bytes(T, B, L, D), dtype=torch.uint8, device="cuda")
    for valid, count in ((None, B), (n_valid, n)):
        before = [w.clone() for w in weights] if R <= 1 << 20 else None
        ws.fill_(0xA5)                     # nothing may depend on what the workspace held
        Bd.ss_embbag_backward_update(tables, idx.int(), valid, grad, 1.0, ws)
        for t in range(T):
            rows, sums = idx[t, :count].unique(return_inverse=True)
            want = torch.zeros(rows.numel(), D, dtype=torch.float64, device="cuda")
            want.index_add_(0, sums.reshape(-1),
                            grad[t, :count].double().repeat_interleave(L, 0))
            if stale:
                want[flagged[t, rows]] = 0
            start = before[t][rows].double() if before else 0.0
            assert torch.equal(weights[t][rows].double(), start - want), (t, count)
            if before:                     # and no other row was touched
                after = weights[t].clone()
                after[rows] = before[t][rows]
                assert torch.equal(after, before[t]), (t, count)
            else:
                assert int((weights[t] != 0).any(1).sum()) <= rows.numel()
                weights[t].zero_()


@pytest.mark.parametrize("T,B", [
    (100, 4096), (65, 2049), (129, 2048), (200, 1500), (300, 1025), (3, 1500), (2, 2047), (2, 8193),
    (1, 16384), (5, 16383),
])
def test_fused_grouping_leaves_the_bits_of_the_separate_calls(T, B):
    # the lists of both have to be in the same order: it decides which runs of equal rows cross the
    # borders of strips and workgroups, and so how their sums round
    from paper_2404_04270_amd import binding as Bd
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T * 31 + B)
    R, D = 500, 8
    idx = _rows("skewed", (T, B, 1), R, gen).int()
    grad = torch.randn(T, B, D, device="cuda", generator=gen)
    start = torch.randn(T, R, D, device="cuda", generator=gen)
    n_valid = torch.tensor([B - 7], dtype=torch.int32, device="cuda")
    ws = torch.empty(Bd.ss_backward_workspace_bytes(T, B, 1, D), dtype=torch.uint8, device="cuda")
    left = []
    for fused in (False, True):
        w = start.clone()
        tables = Bd.Tables(list(w.unbind(0)))
        out = torch.zeros(T, B, D, device="cuda")
        ws.fill_(0xA5)
        if fused:
            Bd.ss_embbag_forward_grouped(tables, idx, n_valid, out, ws)
        else:
            Bd.ss_embbag_forward(tables, idx, n_valid, out)
            Bd.ss_embbag_backward_prepare(tables, idx, n_valid, ws)
        Bd.ss_embbag_backward_apply(tables, B, 1, grad, 0.01, ws)
        left.append((out, w))
    assert torch.equal(left[0][0], left[1][0])
    assert torch.equal(left[0][1], left[1][1])


def _best_us(call):
    call()
    best = float("inf")
    for _ in range(5):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(10):
            call()
        end.record()
        end.synchronize()
        best = min(best, begin.elapsed_time(end) * 100.0)
    return best


@pytest.mark.parametrize("L", [2, 3, 4, 8])
def test_periodic_bags_take_no_longer_than_the_same_lookups_in_any_order(L):
    # L constant ids in every bag: each of them has its share of a class's lookups, at places that
    # repeat with the bags.  Ids that are not recognized as heavy cost a comparison per pair of
    # their lookups (64 tables, of which some have ids of one class: 40 times as long and more),
    # recognized ones the same in any order of the lookups.
    from paper_2404_04270_amd import binding as Bd
    T, R, B = 64, 1 << 20, 16384 // L
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L)
    tables = Bd.Tables([torch.empty(1, 4, device="cuda") for _ in range(T)])
    tables.rows = R                        # (the grouping reads no weights)
    tables._refresh_struct()
    ids = torch.randint(0, R, (T, 1, L), device="cuda", generator=gen, dtype=torch.int32)
    bags = ids.expand(T, B, L).contiguous()
    mixed = torch.stack([b.reshape(-1)[torch.randperm(B * L, device="cuda", generator=gen)]
                         for b in bags]).view_as(bags)
    ws = torch.empty(Bd.ss_backward_workspace_bytes(T, B, L, 4), dtype=torch.uint8, device="cuda")
    us = [_best_us(lambda: Bd.ss_embbag_backward_prepare(tables, i, None, ws))
          for i in (bags, mixed)]
    assert us[0] < 2.0 * us[1], us


def test_heavy_rows_whose_hashes_agree_take_no_longer_than_others():
    # Two rows of one class that have all of its lookups between them.  The votes compare ten bits of a
    # hash of the row: where these agree, the rows still have to be told apart, as a row that is not
    # recognized costs a comparison per pair of its lookups.  64 tables x 16384 lookups of 2^20 rows:
    # eight classes, by the highest three bits of the mixed row id.
    from paper_2404_04270_amd import binding as Bd
    T, key_bits, class_bits, B = 64, 20, 3, 8192
    R, mix = 1 << key_bits, 0x9E3779B1
    rem = key_bits - class_bits
    mixed = (torch.arange(R) * mix) & (R - 1)
    cls, above = mixed >> rem, mixed & ((1 << rem) - 1)
    hashed = ((above * mix) & 0xFFFFFFFF) >> 22
    first = 12345
    same_class = cls == cls[first]
    agree = (same_class & (hashed == hashed[first])).nonzero().flatten()
    other = (same_class & (hashed != hashed[first])).nonzero().flatten()
    agree = agree[agree != first]
    assert agree.numel() > T
    tables = Bd.Tables([torch.empty(1, 4, device="cuda") for _ in range(T)])
    tables.rows = R                        # (the grouping reads no weights)
    tables._refresh_struct()
    ws = torch.empty(Bd.ss_backward_workspace_bytes(T, B, 2, 4), dtype=torch.uint8, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    which = torch.randint(0, 2, (T, 2 * B), device="cuda", generator=gen)
    us = []
    for second in (agree, other):
        ids = torch.stack([torch.full((T,), first), second[:T]], dim=1).int().cuda()
        idx = ids.gather(1, which).view(T, B, 2)
        us.append(_best_us(lambda: Bd.ss_embbag_backward_prepare(tables, idx, None, ws)))
    assert us[0] < 2.0 * us[1], us
