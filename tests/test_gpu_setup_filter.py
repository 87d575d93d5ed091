"""The deflation setup's Chebyshev recurrence runs inside the stencil (two
launches a step): the lowest degrees, where terms are missing, and both site
splits of the stencil with a partly filled last workgroup."""
import numpy as np
import pytest

import synth
from oracle import deflation, wilson

pytestmark = pytest.mark.gpu
M_W = -1.6


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg

    return sg, torch


@pytest.mark.parametrize("degree", [1, 2, 3])
def test_low_degrees_match_dense_oracle(env, degree):
    # tolerances of the default degree's comparison with the dense oracle
    sg, torch = env
    print("filter degree", degree, flush=True)
    dims, m = (3, 3, 3, 4), 6
    links = synth.random_links(dims, 32)
    S0, T0, lam0, _ = deflation.critical_from_dense(wilson.hw_matrix(links, dims, 0.3, M_W).toarray(), m)
    ctx = sg.sgn_create(links, dims, 0.3, M_W)
    try:
        sg.sgn_set_deflation_filter(ctx, degree)
        sg.sgn_deflate(ctx, m)
        stats = sg.sgn_deflate_stats(ctx)
        assert stats["filter_degree"] == degree  # the filtered run converged
        S = sg.sgn_deflate_export(ctx)[0].cpu().numpy()
        assert np.abs(S @ S.conj().T - S0 @ S0.conj().T).max() < 1e-9
    finally:
        sg.sgn_destroy(ctx)


@pytest.mark.parametrize("dims", [(3, 3, 3, 5), (13, 11, 11, 11)])  # 16 and 32 sites a workgroup
def test_schur_pair_residual(env, dims):
    sg, torch = env
    print("filter", dims, flush=True)
    m = 2
    ctx = sg.sgn_create(synth.random_links(dims, 5), dims, 0.2, M_W)
    try:
        sg.sgn_deflate(ctx, m)
        assert sg.sgn_deflate_stats(ctx)["filter_degree"] == 16
        S, T, ev = sg.sgn_deflate_export(ctx)
        AS = torch.empty(m, S.shape[0], dtype=torch.complex128, device="cuda")
        for j in range(m):
            sg.sgn_matvec(ctx, S[:, j].contiguous(), AS[j])
        res = AS.T - S @ torch.from_numpy(T).cuda()
        # the setup's own bound on the residual relative to the operator, whose norm is below 10
        assert float(res.norm()) <= 1e-9
    finally:
        sg.sgn_destroy(ctx)
