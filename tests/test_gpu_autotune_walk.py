"""autotune_stencil chooses the walk by what the applies run: the stencil of
the component-major layout, inside applies, in the context's precision."""
import pytest

import synth

pytestmark = pytest.mark.gpu

M_W = -1.6


@pytest.mark.parametrize("prec", [0, 1])
def test_walk_is_timed_on_applies(prec):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg
    from paper_0704_3486_amd.autotune import STENCIL_BLOCKS, autotune_stencil

    dims = (8, 8, 8, 16)
    print("walk", prec, flush=True)
    ctx = sg.sgn_create(synth.random_links(dims, 83), dims, 0.3, M_W)
    try:
        sg.sgn_set_precision(ctx, prec)
        sg.sgn_set_profiling(ctx, True)
        sg.sgn_profile_reset(ctx)
        r = autotune_stencil(ctx, reps=2)
        n = {name: st["launches"] for name, st in sg.sgn_profile_read(ctx).items()}
        assert r["blocks"] in STENCIL_BLOCKS and r["us"] > 0
        # several walks, each with a warm-up and two timed applies of several steps
        assert n.get("krylov_update", 0) >= 3 * 3 * 2, n
        x = torch.from_numpy(synth.gaussian_source(dims, 8300)).cuda()
        y1, y2 = torch.empty_like(x), torch.empty_like(x)
        sg.sgn_apply_fixed(ctx, x, y1, 20)
        sg.sgn_set_stencil_blocks(ctx, -1)
        sg.sgn_apply_fixed(ctx, x, y2, 20)
        assert torch.equal(y1, y2)
    finally:
        sg.sgn_destroy(ctx)
