"""The stencil's forms against the oracle and each other: interface layout,
16 or 32 sites per workgroup, blocked and natural walks, odd extents."""
import numpy as np
import pytest

import synth
from oracle import wilson

pytestmark = pytest.mark.gpu

M_W = -1.6
EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg

    return sg, torch


# 16 and 288 sites fill their last workgroup, the others leave 1, 2, 5, 10 and 15 sites over
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (3, 5, 2, 7), (17, 3, 5, 7), (5, 2, 11, 3), (5, 7, 3, 3), (2, 3, 9, 29),
                                  (4, 6, 3, 4), (3, 3, 7, 17)])
def test_matvec_odd_lattices(env, dims):
    sg, torch = env
    print("matvec", dims, flush=True)
    mu = 0.4
    links = synth.random_links(dims, 3)
    x = synth.gaussian_source(dims, 4)
    ref = wilson.hw_matrix(links, dims, mu, M_W) @ x
    ctx = sg.sgn_create(links, dims, mu, M_W)
    try:
        n = x.size
        buf = torch.zeros(n + 5, dtype=torch.complex128, device="cuda")
        buf[:n] = torch.from_numpy(x).cuda()
        xd = buf[:n].clone()
        y = torch.full_like(xd, float("nan"))
        sg.sgn_matvec(ctx, xd, y)
        # an entry is one term plus 8 hops of 6 products (two spins, three
        # colours) of a unit link entry with x: 49 terms, a few roundings each
        kappa = 1.0 / (8.0 + 2.0 * M_W)
        bound = 4 * 49 * EPS * (1.0 + 8 * 6 * kappa * np.exp(mu)) * np.abs(x).max()
        assert np.abs(y.cpu().numpy() - ref).max() <= bound
        y2 = torch.full_like(xd, float("nan"))
        sg.sgn_matvec_noalloc(ctx, xd, y2)
        assert torch.equal(y, y2)
        # x and y sharing memory
        for fn in (sg.sgn_matvec, sg.sgn_matvec_noalloc):
            buf[:n] = xd
            fn(ctx, buf[:n], buf[5:n + 5])
            assert torch.equal(buf[5:n + 5], y)
    finally:
        sg.sgn_destroy(ctx)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_site_splits_bitwise_equal(env, prec):
    # 13 sources of a 6^4 lattice take 32 sites per workgroup, one takes 16
    sg, torch = env
    print("site splits", prec, flush=True)
    dims, k, nrhs = (6, 6, 6, 6), 12, 13
    ctx = sg.sgn_create(synth.random_links(dims, 5), dims, 0.3, M_W)
    try:
        if prec == "mixed":
            sg.sgn_set_precision(ctx, sg.SGN_PREC_MIXED)
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 50 + r) for r in range(nrhs)])).cuda()
        Y, y = torch.empty_like(X), torch.empty_like(X[0])
        sg.sgn_apply_batched_fixed(ctx, X, Y, k)
        for r in (0, nrhs - 1):
            sg.sgn_apply_fixed(ctx, X[r], y, k)
            assert torch.equal(y, Y[r]), r
    finally:
        sg.sgn_destroy(ctx)
