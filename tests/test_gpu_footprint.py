"""sgn_footprint_bytes covers what a batched apply keeps per source, the dot
pass's partial sums of small lattices (eight parts) among them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

M_W = -1.6


@pytest.mark.parametrize("dims,m", [((2, 2, 2, 4), 0), ((4, 4, 4, 4), 6), ((4, 4, 5, 6), 0), ((6, 6, 6, 6), 4)])
@pytest.mark.parametrize("prec", [0, 1])
def test_footprint_counts_the_parts(dims, m, prec):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0704_3486_amd as sg

    print("footprint", dims, m, prec, flush=True)
    ctx = sg.sgn_create(synth.random_links(dims, 3), dims, 0.3, M_W)
    try:
        sg.sgn_set_precision(ctx, prec)
        if m:
            sg.sgn_deflate(ctx, m)
        N = 12 * int(np.prod(dims))
        ldq, vt = (N + 63) // 64 * 64, 8 if prec else 16
        for kmax, nrhs in ((100, 64), (300, 64), (N - m, 2)):
            ncap, n = m + kmax + 1, m + kmax
            tiles = max(8, (N + 511) // 512)
            slot = ldq * (kmax + 1) * vt  # Krylov columns
            slot += ldq * (2 * 16 + vt + 2 * 16) + (2 * ldq * vt if prec else 0)  # candidates, stencil result, x, y
            slot += 16 * (ncap * ncap + n * n + max(m, 1) + 2 * ncap)  # H, its sign, coefficients
            slot += 16 * 2 * ncap * (1 + tiles)  # a, b and their partial sums
            slot += 16 * 3 * n * n  # the sign iteration
            assert sg.sgn_footprint_bytes(ctx, kmax, nrhs) >= nrhs * slot, (kmax, nrhs)
        if N <= 448:  # one source: the same partial sums
            ncap = m + 101
            assert sg.sgn_footprint_bytes(ctx, 100, 1) >= 16 * (ldq * (ncap + 3) + ncap * ncap + 4 * 100 * 100 +
                                                                4 * ncap + 2 * 8 * ncap)
    finally:
        sg.sgn_destroy(ctx)
