"""A workspace sized for the largest batch serves every smaller one (a program sizes it once and
ends an epoch with a short batch): ss_layernorm_backward_workspace_bytes falls in none of its
arguments, across the borders where the backward pass takes fewer vectors per workgroup.  On the
GPU: two short batches that get more workgroups than the largest, in a workspace of the largest
batch's size, with what lies behind the workspace left alone.
"""
import numpy as np
import pytest
import torch

from paper_2404_04270_amd import binding as B


@pytest.mark.parametrize("T,D", [(26, 64), (8, 128), (4, 256), (1, 4), (3, 36), (40, 512), (600, 16),
                                 (65535, 4)])
def test_workspace_never_falls_with_the_batch(T, D):
    sizes = np.array([B.ss_layernorm_backward_workspace_bytes(T, D, n) for n in range(1, 20_000)])
    assert np.all(np.diff(sizes) >= 0)


@pytest.mark.parametrize("Bcap", [1, 129, 2048, 2520, 2521, 4096, 65536])
def test_workspace_never_falls_with_tables_or_row_length(Bcap):
    by_tables = [B.ss_layernorm_backward_workspace_bytes(T, 64, Bcap) for T in range(1, 1200)]
    assert np.all(np.diff(by_tables) >= 0)
    by_dim = [B.ss_layernorm_backward_workspace_bytes(26, D, Bcap) for D in range(4, 1025, 4)]
    assert np.all(np.diff(by_dim) >= 0)


def test_every_split_fits():
    """2 * T rows of dim floats for every workgroup of each split into 8, 4 or 2 vectors per lane
    group, as the split is chosen: halved while that leaves under 512 workgroups."""
    for T, D in ((26, 64), (8, 128), (1, 1024), (7, 20)):
        ng = 256 // min(64, 1 << (D // 4 - 1).bit_length())
        for n in list(range(1, 3000, 7)) + [2520, 4096, 20_161, 65_536]:
            tiles = 8
            while tiles > 2 and T * n < 512 * ng * tiles:
                tiles //= 2
            need = 2 * T * -(-n // (ng * tiles)) * D * 4
            assert B.ss_layernorm_backward_workspace_bytes(T, D, n) >= need, (T, D, n)


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,largest,short", [(26, 64, 4096, 2520), (8, 128, 4096, 2047)])
def test_short_batch_in_the_largest_batchs_workspace(T, D, largest, short):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(T + D)
    need = B.ss_layernorm_backward_workspace_bytes(T, D, largest)
    flat = torch.full((need + 4096,), 77, dtype=torch.uint8, device=dev)
    x = torch.randn(T, short, D, device=dev, generator=gen)
    dy = torch.randn(T, short, D, device=dev, generator=gen)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    mean, rstd = torch.empty(T, short, device=dev), torch.empty(T, short, device=dev)
    dg, db = torch.empty(T, D, device=dev), torch.empty(T, D, device=dev)
    B.ss_layernorm_forward(x, None, None, None, 1e-5, y, mean, rstd)
    B.ss_layernorm_backward(dy, x, None, None, mean, rstd, dx, dg, db, flat[:need])
    assert torch.all(flat[need:] == 77)
    # sums of `short` products of two normal values in fp32: error in practice sqrt(short) * eps
    # * their size, asserted at 1e-6 * sqrt(short) * the largest
    x64, dy64 = x.double(), dy.double()
    xh = (x64 - x64.mean(-1, keepdim=True)) / (x64.var(-1, unbiased=False, keepdim=True) + 1e-5).sqrt()
    for got, terms in ((dg, dy64 * xh), (db, dy64)):
        np.testing.assert_allclose(got.cpu().numpy(), terms.sum(1).cpu().numpy(), rtol=1e-5,
                                   atol=1e-6 * short ** 0.5 * float(terms.abs().max()))
