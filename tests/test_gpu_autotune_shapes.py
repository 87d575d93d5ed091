"""autotune times shapes that are kernels of their own and keeps the default
shape unless another is clearly faster."""
import types

import pytest

import synth

pytestmark = pytest.mark.gpu

M_W = -1.6


@pytest.fixture()
def ctx():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg

    dims = (4, 4, 4, 4)
    c = sg.sgn_create(synth.random_links(dims, 84), dims, 0.3, M_W)
    yield c
    sg.sgn_destroy(c)


def _fake(monkeypatch, at, cost):
    """timed applies that take cost(update_batch, dot_cols); returns the shapes set"""
    shapes, clock = [], [0.0]

    def set_tuning(ctx, ub, cpw, uw):
        shapes.append((ub, cpw))

    def apply(*args):
        clock[0] += cost(*shapes[-1])

    monkeypatch.setattr(at, "sgn_set_tuning", set_tuning)
    monkeypatch.setattr(at, "sgn_apply_fixed", apply)
    monkeypatch.setattr(at, "time", types.SimpleNamespace(perf_counter=lambda: clock[0]))
    return shapes


def test_distinct_shapes_and_margin(ctx, monkeypatch):
    from paper_0704_3486_amd import autotune as at

    print("shapes", flush=True)
    shapes = _fake(monkeypatch, at, lambda ub, cpw: 1.0 if (ub, min(cpw, 2)) == (8, 2) else 0.995)
    r = at.autotune(ctx, k=20, reps=1)
    timed = shapes[:-1]
    assert len({(ub, min(cpw, 2)) for ub, cpw in timed}) == len(timed) == 6
    assert (r["update_batch"], min(r["dot_cols"], 2)) == (8, 2)  # half a per cent is noise
    shapes = _fake(monkeypatch, at, lambda ub, cpw: 0.9 if (ub, cpw) == (16, 1) else 1.0)
    r = at.autotune(ctx, k=20, reps=1)
    assert (r["update_batch"], r["dot_cols"]) == (16, 1) == shapes[-1]
