"""Launch shapes and captured steps in every form of the one-vector step's dot
and update passes: whole columns (6 row tiles), parts (30 tiles, one and three
sources, with a basis that outgrows them) and tiles (65)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

M_W = -1.6

WHOLE, PARTS, TILES = (4, 4, 4, 4), (5, 6, 6, 7), (7, 7, 7, 8)


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg

    return sg, torch


class _Field:
    def __init__(self, env, dims, prec, nrhs, m=5):
        self.sg, self.torch = env
        self.ctx = self.sg.sgn_create(synth.random_links(dims, 31), dims, 0.3, M_W)
        self.sg.sgn_set_precision(self.ctx, prec)
        if m:
            self.sg.sgn_deflate(self.ctx, m)
        self.X = self.torch.from_numpy(np.stack([synth.gaussian_source(dims, 3100 + r) for r in range(nrhs)])).cuda()

    def apply(self, k, nrhs=None):
        X = self.X if nrhs is None else self.X[:nrhs]
        Y = self.torch.empty_like(X)
        if X.shape[0] == 1:
            self.sg.sgn_apply_fixed(self.ctx, X[0], Y[0], k)
        else:
            self.sg.sgn_apply_batched_fixed(self.ctx, X, Y, k)
        return Y

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        self.sg.sgn_destroy(self.ctx)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims,nrhs,k", [(WHOLE, 1, 60), (PARTS, 1, 60), (PARTS, 3, 70), (TILES, 1, 40),
                                         (TILES, 3, 40)])
def test_launch_shapes_are_neutral(env, dims, nrhs, k, prec):
    sg, torch = env
    print("shapes", dims, nrhs, prec, flush=True)
    with _Field(env, dims, prec, nrhs) as f:
        for uw in (8, 16):
            ref = None
            for ub in (4, 8, 16):
                for cpw in (1, 2, 4):
                    sg.sgn_set_tuning(f.ctx, ub, cpw, uw)
                    Y = f.apply(k)
                    ref = Y if ref is None else ref
                    assert torch.equal(Y, ref), (ub, cpw, uw)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims,nrhs,k", [(WHOLE, 9, 60), (PARTS, 2, 80), (PARTS, 7, 60), (TILES, 3, 40),
                                         ((4, 4, 4, 6), 3, 1060)])
def test_sixteen_update_wavefronts(env, dims, nrhs, k, prec):
    sg, torch = env
    print("16 wavefronts", dims, nrhs, k, prec, flush=True)
    with _Field(env, dims, prec, nrhs, m=0) as f:
        Y8 = f.apply(k)
        sg.sgn_set_tuning(f.ctx, 8, 4, 16)
        Y = f.apply(k)
        # a source alone and in the batch, bit for bit
        for r in {0, nrhs - 1}:
            y = torch.empty_like(f.X[r])
            sg.sgn_apply_fixed(f.ctx, f.X[r], y, k)
            assert torch.equal(y, Y[r]), r
        # other sums of the same numbers: rounding of the basis, carried through the Krylov process
        rel = float(torch.linalg.vector_norm(Y - Y8) / torch.linalg.vector_norm(Y8))
        print("  relative difference", rel, flush=True)
        assert rel < (1e-10 if prec == 0 else 1e-4)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims,nrhs,ks", [(PARTS, 1, (96, 350)), (PARTS, 3, (64, 100)), (TILES, 1, (50, 64)),
                                          (TILES, 3, (40, 66)), ((3, 5, 5, 6), 4, (90, 130))])
def test_captured_steps_in_every_form(env, dims, nrhs, ks, prec):
    sg, torch = env
    print("captured", dims, nrhs, ks, prec, flush=True)
    with _Field(env, dims, prec, nrhs) as f:
        direct = [f.apply(k) for k in ks]
        for steps in (2, 16):
            sg.sgn_set_step_graphs(f.ctx, steps)
            for rep in range(3):  # captures, then replays, with eager work between them
                for k, ref in zip(ks, direct):
                    Y = f.apply(k)
                    _ = (Y * 2.0).abs().sum().item()
                    assert torch.equal(Y, ref), (steps, rep, k)
            if nrhs > 1:  # another set of running sources
                Y = f.apply(ks[0], nrhs - 1) if nrhs > 2 else None
                assert Y is None or torch.equal(Y, direct[0][: nrhs - 1])
