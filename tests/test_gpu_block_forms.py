"""The block process picks its column groups and update kernel by the rows,
sources and columns of a launch: every form adds the same numbers in the same
order, so a source alone and the same source in a large batch agree bitwise,
and both agree with the one-vector process up to rounding (1e-10 relative, the
bound of the other fixed-k comparisons)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

M_W = -1.6


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg

    return sg, torch


# update by whole rows for the batch (1.2 times the least entries) and by
# quarters alone; a last block of 8 columns after blocks of 16 (packed); 9
# columns (the least that is not packed); fewer rows than a chunk; row
# remainders of the update's 16- and 32-row workgroups (N = 12 mod 32) with a
# deflated part; the largest launch that makes two stencil applications at once
# (256 workgroups of four sites) against the next larger one
@pytest.mark.parametrize("dims,m,block,k,nrhs", [
    ((6, 6, 6, 6), 0, 16, 112, 14), ((6, 6, 6, 6), 0, 16, 104, 15), ((3, 3, 3, 5), 0, 9, 40, 9),
    ((2, 2, 2, 2), 0, 16, 37, 3), ((3, 5, 5, 5), 4, 13, 57, 24), ((4, 4, 4, 5), 3, 8, 44, 40),
    ((4, 4, 8, 8), 0, 16, 35, 2), ((2, 3, 2, 5), 0, 5, 18, 40),
    # more than 65536 rows, where the chunks grow: whole rows in the batch
    ((7, 11, 7, 11), 0, 16, 88, 4), ((11, 7, 7, 12), 2, 16, 80, 4)])
def test_forms_bitwise_equal(env, dims, m, block, k, nrhs):
    sg, torch = env
    print("block forms", dims, m, block, k, nrhs, flush=True)
    ctx = sg.sgn_create(synth.random_links(dims, 7), dims, 0.3, M_W)
    try:
        if m:
            sg.sgn_deflate(ctx, m)
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 90 + r) for r in range(nrhs)])).cuda()
        Y, y, ref = torch.empty_like(X), torch.empty_like(X[0]), torch.empty_like(X[0])
        sg.sgn_apply_fixed(ctx, X[0], ref, k)
        sg.sgn_set_block_steps(ctx, block)
        sg.sgn_apply_batched_fixed(ctx, X, Y, k)
        for r in (0, nrhs - 1):
            sg.sgn_apply_fixed(ctx, X[r], y, k)
            assert torch.equal(y, Y[r]), r
        assert float((Y[0] - ref).norm() / ref.norm()) <= 1e-10
    finally:
        sg.sgn_destroy(ctx)
