"""The block process's update pass takes its rows in chunks of its own: every
row of every vector is updated on lattices whose rows are no multiple of a
chunk, packed (s <= 8) and by halves of 16, alone and in batches."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

M_W = -1.6


@pytest.mark.parametrize("dims,m,block,k,nrhs", [
    ((4, 4, 4, 4), 4, 2, 30, 16), ((4, 5, 7, 9), 0, 8, 41, 5), ((3, 5, 7, 11), 2, 6, 37, 9),
    # more than 65536 rows: chunks of the dot pass that are no multiple of the update's rows
    ((7, 11, 7, 11), 0, 7, 44, 3), ((11, 7, 7, 12), 2, 16, 50, 5), ((12, 12, 12, 12), 0, 8, 33, 3),
    ((12, 12, 12, 12), 0, 16, 49, 2), ((10, 10, 10, 11), 0, 16, 60, 6),
    # 150000 rows over the sources: whole rows also for short bases (one source: quarters)
    ((6, 6, 6, 6), 3, 16, 37, 10), ((5, 5, 6, 9), 0, 11, 30, 10), ((3, 3, 7, 11), 0, 13, 29, 18),
    ((3, 3, 7, 11), 0, 13, 29, 19)])
def test_every_row_is_updated(dims, m, block, k, nrhs):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg

    print("block rows", dims, m, block, k, nrhs, flush=True)
    ctx = sg.sgn_create(synth.random_links(dims, 17), dims, 0.3, M_W)
    try:
        if m:
            sg.sgn_deflate(ctx, m)
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 190 + r) for r in range(nrhs)])).cuda()
        Y, y, ref = torch.empty_like(X), torch.empty_like(X[0]), torch.empty_like(X[0])
        sg.sgn_apply_fixed(ctx, X[0], ref, k)  # the one-vector process
        sg.sgn_set_block_steps(ctx, block)
        sg.sgn_apply_batched_fixed(ctx, X, Y, k)
        for r in (0, nrhs - 1):
            sg.sgn_apply_fixed(ctx, X[r], y, k)
            assert torch.equal(y, Y[r]), r
        # a row that no workgroup took would differ by the size of its entries
        assert float((Y[0] - ref).norm() / ref.norm()) <= 1e-10
        assert float((Y[0] - ref).abs().max() / ref.abs().max()) <= 1e-9
    finally:
        sg.sgn_destroy(ctx)
