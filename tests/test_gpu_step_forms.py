"""The one-vector step's dot and update passes choose their form by the number
of row tiles (512 rows) and sources: every form adds the same numbers in the
same order, so a source alone and the same source in a large batch (the
general form) agree bitwise."""
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


# row tiles: 1, 8 (the last lattice of whole columns), 9 (the first of parts),
# 24 (three tiles a part), 64 (the last of parts), 65
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("dims,m,k,nrhs", [
    ((2, 2, 2, 4), 0, 30, 64), ((4, 4, 4, 5), 6, 70, 12), ((2, 2, 2, 43), 0, 45, 16), ((4, 4, 8, 8), 5, 40, 6),
    ((2, 5, 13, 21), 3, 20, 3), ((2, 8, 9, 19), 0, 20, 2),
    # one source: 4, 8 and 16 columns a workgroup, with remainders
    ((5, 5, 6, 6), 6, 151, 5), ((2, 5, 13, 21), 3, 100, 5), ((2, 5, 13, 21), 0, 205, 5)])
def test_forms_bitwise_equal(env, dims, m, k, nrhs, prec):
    sg, torch = env
    print("forms", dims, m, k, nrhs, prec, flush=True)
    ctx = sg.sgn_create(synth.random_links(dims, 7), dims, 0.3, M_W)
    try:
        if prec == "mixed":
            sg.sgn_set_precision(ctx, sg.SGN_PREC_MIXED)
        if m:
            sg.sgn_deflate(ctx, m)
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 90 + r) for r in range(nrhs)])).cuda()
        Y, y = torch.empty_like(X), torch.empty_like(X[0])
        sg.sgn_apply_batched_fixed(ctx, X, Y, k)
        for r in {0, nrhs - 1}:
            sg.sgn_apply_fixed(ctx, X[r], y, k)
            assert torch.equal(y, Y[r]), r
    finally:
        sg.sgn_destroy(ctx)


def test_long_basis_spans(env):
    # more columns than the update pass by parts keeps coefficients of at once
    sg, torch = env
    print("long basis", flush=True)
    dims, k, nrhs = (2, 2, 2, 43), 1045, 15
    ctx = sg.sgn_create(synth.random_links(dims, 8), dims, 0.3, M_W)
    try:
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 30 + r) for r in range(nrhs)])).cuda()
        Y, y = torch.empty_like(X), torch.empty_like(X[0])
        sg.sgn_apply_batched_fixed(ctx, X, Y, k)
        sg.sgn_apply_fixed(ctx, X[0], y, k)
        assert torch.equal(y, Y[0])
    finally:
        sg.sgn_destroy(ctx)


@pytest.mark.parametrize("prec,k,nrhs", [("fp64", 40, 4), ("mixed", 60, 5)])
def test_streamed_tiles(env, prec, k, nrhs):
    # 12^4: the columns of the batch exceed the caches, so most of their tiles
    # are streamed; those of one source do not
    sg, torch = env
    print("streamed", prec, k, nrhs, flush=True)
    dims = (12, 12, 12, 12)
    ctx = sg.sgn_create(synth.random_links(dims, 9), dims, 0.3, M_W)
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


def _reductions(sg, torch, dims, nrhs, k, prec):
    """(steps, reduction launches) of an apply with k columns, and its result"""
    ctx = sg.sgn_create(synth.random_links(dims, 11), dims, 0.3, M_W)
    try:
        sg.sgn_set_precision(ctx, prec)
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 70 + r) for r in range(nrhs)])).cuda()
        Y = torch.empty_like(X)
        sg.sgn_set_profiling(ctx, True)
        sg.sgn_profile_reset(ctx)
        if nrhs == 1:
            sg.sgn_apply_fixed(ctx, X[0], Y[0], k)
        else:
            sg.sgn_apply_batched_fixed(ctx, X, Y, k)
        n = {name: st["launches"] for name, st in sg.sgn_profile_read(ctx).items()}
        return n["krylov_dot"], n.get("krylov_reduce", 0), Y
    finally:
        sg.sgn_destroy(ctx)


# short bases go without the reduction launch (one is left, at the end), long
# ones with it: from 5000 tiles x slots x columns on in batches (one source: 18000,
# FP32 10000), on lattices of 8 tiles or fewer from 20000 (FP32 5000)
@pytest.mark.parametrize("dims,nrhs,k,prec,first", [
    ((5, 6, 7, 8), 2, 120, 0, 63), ((5, 6, 7, 8), 3, 120, 1, 42), ((5, 6, 6, 7), 4, 100, 1, 42),
    ((6, 7, 7, 8), 1, 350, 0, 322), ((5, 6, 6, 7), 1, 360, 1, 334), ((4, 4, 4, 4), 8, 150, 1, 105),
    ((4, 4, 4, 5), 8, 330, 0, 313), ((5, 6, 6, 7), 1, 300, 0, 601)])
def test_long_bases_take_the_reduction(env, dims, nrhs, k, prec, first):
    sg, torch = env
    print("long bases", dims, nrhs, k, prec, flush=True)
    steps, reds, Y = _reductions(sg, torch, dims, nrhs, k, prec)
    tiles = (12 * int(np.prod(dims)) + 511) // 512
    # steps with 0 .. k - 1 columns, then one dot pass with k for the last column
    want = max(0, k - first) + (1 if tiles > 8 or first <= k else 0)
    assert steps == k + 1 and reds == want, (steps, reds, want)
    # the same bits as one source alone (nrhs > 1) or as in a batch of 16
    other = 1 if nrhs > 1 else 16
    ctx = sg.sgn_create(synth.random_links(dims, 11), dims, 0.3, M_W)
    try:
        sg.sgn_set_precision(ctx, prec)
        x = torch.from_numpy(synth.gaussian_source(dims, 70)).cuda()
        y = torch.empty_like(x)
        if other == 1:
            sg.sgn_apply_fixed(ctx, x, y, k)
        else:
            X = x.repeat(other, 1)
            Y2 = torch.empty_like(X)
            sg.sgn_apply_batched_fixed(ctx, X, Y2, k)
            y = Y2[other - 1]
        assert torch.equal(y, Y[0])
    finally:
        sg.sgn_destroy(ctx)
