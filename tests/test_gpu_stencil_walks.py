"""The component-major stencil with 32 sites a workgroup, in the walk of 4D
blocks (every apply on large lattices): bitwise what the interface-layout form
of sgn_matvec and the natural order give, in all the forms that applies and
the deflation setup launch."""
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


# 16^4 and 16.8.12.44 walk in blocks by themselves, the others where set
@pytest.mark.parametrize("dims,blocks", [((16, 16, 16, 16), (0, 0, 0)), ((16, 8, 12, 44), (0, 0, 0)),
                                         ((8, 8, 16, 16), (4, 8, 4)), ((8, 8, 16, 16), (8, 4, 16)),
                                         ((7, 13, 11, 17), (0, 0, 0))])
def test_layouts_agree(env, dims, blocks):
    sg, torch = env
    print("layouts", dims, blocks, flush=True)
    ctx = sg.sgn_create(synth.random_links(dims, 21), dims, 0.3, M_W)
    try:
        sg.sgn_set_stencil_blocks(ctx, *blocks)
        x = torch.from_numpy(synth.gaussian_source(dims, 2100)).cuda()
        y = torch.empty_like(x)
        sg.sgn_matvec(ctx, x, y)
        # buffers that share memory go through the component-major form
        buf = torch.empty(x.numel() + 4, dtype=x.dtype, device="cuda")
        for rep in range(2):
            buf[: x.numel()].copy_(x)
            torch.cuda.synchronize()
            sg.sgn_matvec(ctx, buf[: x.numel()], buf[4:])
            assert torch.equal(buf[4:], y), rep
    finally:
        sg.sgn_destroy(ctx)


# 16384 sites: 512 workgroups of 32 sites for one source
@pytest.mark.parametrize("form", ["fp64", "mixed", "block", "batch", "mixed batch", "block batch"])
def test_applies_in_every_walk(env, form):
    sg, torch = env
    print("walks", form, flush=True)
    dims, k, nrhs = (8, 8, 16, 16), 19, 3 if "batch" in form else 1
    ctx = sg.sgn_create(synth.random_links(dims, 22), dims, 0.3, M_W)
    try:
        if "mixed" in form:
            sg.sgn_set_precision(ctx, sg.SGN_PREC_MIXED)
        if "block" in form:
            sg.sgn_set_block_steps(ctx, 8)
        X = torch.from_numpy(np.stack([synth.gaussian_source(dims, 2200 + r) for r in range(nrhs)])).cuda()
        ref = None
        for blocks in ((-1, 0, 0), (4, 8, 4), (8, 16, 2), (4, 4, 16), (0, 0, 0)):
            sg.sgn_set_stencil_blocks(ctx, *blocks)
            Y = torch.empty_like(X)
            if nrhs == 1:
                sg.sgn_apply_fixed(ctx, X[0], Y[0], k)
            else:
                sg.sgn_apply_batched_fixed(ctx, X, Y, k)
            if ref is None:
                ref = Y
            assert torch.equal(Y, ref), blocks
    finally:
        sg.sgn_destroy(ctx)


def test_apply_with_the_default_walk(env):
    # 16^4: the blocked walk without being set
    sg, torch = env
    print("default walk", flush=True)
    dims = (16, 16, 16, 16)
    ctx = sg.sgn_create(synth.random_links(dims, 23), dims, 0.3, M_W)
    try:
        x = torch.from_numpy(synth.gaussian_source(dims, 2300)).cuda()
        for prec in (sg.SGN_PREC_FP64, sg.SGN_PREC_MIXED):
            sg.sgn_set_precision(ctx, prec)
            y, z = torch.empty_like(x), torch.empty_like(x)
            sg.sgn_set_stencil_blocks(ctx, 0, 0, 0)
            sg.sgn_apply_fixed(ctx, x, y, 6)
            sg.sgn_set_stencil_blocks(ctx, -1)
            sg.sgn_apply_fixed(ctx, x, z, 6)
            assert torch.equal(y, z), prec
    finally:
        sg.sgn_destroy(ctx)


def test_setup_filter_in_every_walk(env):
    # the filter's recurrence (two further terms in the second application)
    sg, torch = env
    print("filter walks", flush=True)
    dims = (8, 8, 16, 16)
    ref = None
    for blocks in ((-1, 0, 0), (4, 8, 4)):
        ctx = sg.sgn_create(synth.random_links(dims, 24), dims, 0.3, M_W)
        try:
            sg.sgn_set_stencil_blocks(ctx, *blocks)
            sg.sgn_deflate(ctx, 4)
            S, T, _ = sg.sgn_deflate_export(ctx)
            if ref is None:
                ref = (S.clone(), np.array(T))
            assert torch.equal(S, ref[0]) and np.array_equal(T, ref[1])
        finally:
            sg.sgn_destroy(ctx)
