"""Feature normalization at the edges of how the kernels cut their work: vectors per lane
group (4 forward, 2 backward, with remainders), 2 / 4 / 8 vectors per group and workgroup in
the backward pass (T * Bcap against 512 workgroups), rows that fill their lanes and rows that
do not, bags of one lookup, of several and of more than 32.  Against plain PyTorch in fp64.

Tolerances: y and dx are short sums of D <= 260 products, rtol 1e-5 of the largest value;
dgamma / dbeta add n terms of size about s in fp32: error below eps * n * s, in practice
eps * sqrt(n) * s, asserted at 1e-6 * sqrt(n) * s.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
EPS = 1e-5

SHAPES = [
    # T, Bcap, D, L, n_valid
    (1, 1, 4, 1, None),              # one vector in the whole launch
    (3, 67, 64, 1, 66),              # remainders of 4 and of 2
    (2, 1000, 256, 1, None),         # 2 vectors per group and workgroup
    (4, 2100, 256, 1, 2099),         # 4
    (4, 4100, 256, 1, None),         # 8
    (2, 333, 64, 33, 300),           # bags of more than 32, row fills its lanes
    (2, 129, 36, 7, None),           # row leaves lanes idle
    (1, 50, 260, 2, 49),             # two f4 per lane
]


@pytest.mark.parametrize("T,Bc,D,L,nv", SHAPES)
def test_fused_normalization_matches_fp64(T, Bc, D, L, nv):
    from paper_2404_04270_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000 * T + Bc + D + L)
    R, n = 500, Bc if nv is None else nv
    W = torch.empty(T, R, D, device=dev).uniform_(-0.05, 0.05, generator=gen)
    idx = torch.randint(0, R, (T, Bc, L), device=dev, generator=gen, dtype=torch.int32)
    dy = torch.randn(T, Bc, D, device=dev, generator=gen) * 0.01
    gamma = torch.rand(T, D, device=dev, generator=gen) + 0.5
    beta = torch.randn(T, D, device=dev, generator=gen) * 0.1
    tb = B.Tables(list(W.unbind(0)))
    n_valid = None if nv is None else torch.tensor([nv], dtype=torch.int32, device=dev)
    y = torch.full((T, Bc, D), 7.0, device=dev)
    dx = torch.full((T, Bc, D), 7.0, device=dev)
    mean, rstd = torch.zeros(T, Bc, device=dev), torch.zeros(T, Bc, device=dev)
    dg, db = torch.zeros(T, D, device=dev), torch.zeros(T, D, device=dev)
    ws = torch.empty(max(256, B.ss_layernorm_backward_workspace_bytes(T, D, Bc)),
                     dtype=torch.uint8, device=dev)
    B.ss_embbag_forward_ln(tb, idx, n_valid, gamma, beta, EPS, y, mean, rstd)
    B.ss_embbag_ln_backward(tb, idx, n_valid, dy, gamma, mean, rstd, dx, dg, db, ws)
    torch.cuda.synchronize()

    W64, dy64 = W.double().cpu(), dy.double().cpu()[:, :n]
    ix = idx.long().cpu()[:, :n]
    g64, b64 = gamma.double().cpu()[:, None], beta.double().cpu()[:, None]
    x = torch.stack([W64[t][ix[t]].sum(1) for t in range(T)])
    rs = 1.0 / (x.var(-1, unbiased=False, keepdim=True) + EPS).sqrt()
    xh = (x - x.mean(-1, keepdim=True)) * rs
    g = g64 * dy64
    want_dx = rs * (g - g.mean(-1, keepdim=True) - xh * (g * xh).mean(-1, keepdim=True))
    for got, want in ((y, xh * g64 + b64), (dx, want_dx)):
        assert torch.all(got[:, n:] == 7.0)
        np.testing.assert_allclose(got.cpu()[:, :n].numpy(), want.numpy(), rtol=1e-5,
                                   atol=1e-5 * float(want.abs().max()))
    for got, terms in ((dg, dy64 * xh), (db, dy64)):
        np.testing.assert_allclose(got.cpu().numpy(), terms.sum(1).numpy(), rtol=1e-5,
                                   atol=1e-6 * n ** 0.5 * float(terms.abs().max()))
