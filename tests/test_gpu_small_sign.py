"""The small sign of a batch: launches of a multiple of eight matrices give
every XCD whole matrices, other launches deal the tiles out, and the update
product makes the stopping test.  A matrix's sums are the same either way, so
a source alone and in the batch agree bitwise."""
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


# n = m + k of the matrices: 1, one tile, one row past a tile, 17 tiles of a
# row (one 16 x 16 block a workgroup, then 2 x 2)
@pytest.mark.parametrize("m,k", [(0, 1), (3, 13), (0, 17), (0, 257)])
@pytest.mark.parametrize("nrhs", [7, 8, 16])
def test_small_sign_batches(env, m, k, nrhs):
    sg, torch = env
    print("small sign", m, k, nrhs, flush=True)
    dims = (3, 3, 4, 4)
    ctx = sg.sgn_create(synth.random_links(dims, 3), dims, 0.2, M_W)
    try:
        if m:
            sg.sgn_deflate(ctx, m)
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 70 + r) for r in range(nrhs)])).cuda()
        Y, y = torch.empty_like(X), torch.empty_like(X[0])
        sg.sgn_apply_batched_fixed(ctx, X, Y, k)
        for r in (0, 5, nrhs - 1):
            sg.sgn_apply_fixed(ctx, X[r], y, k)
            assert torch.equal(y, Y[r]), r
    finally:
        sg.sgn_destroy(ctx)
