"""Launch-shape autotuner for the Arnoldi step's dot and update passes.

The update pass's column-load batch (4, 8, 16) and the columns whose loads a
wavefront of the dot pass issues together (1, 2; 4 acts as 2) form every sum
in the same order, so any of them gives bitwise the same result; which is
fastest depends on the lattice size, the precision and the number of sources in
flight.  `autotune` times the six shapes that are kernels of their own on the
context itself (sgn_apply_fixed, or sgn_apply_batched_fixed for several
sources, at a given Krylov dimension) and keeps the fastest.  On small lattices
some of the six are the same kernel (the header says which), so the default
shape stays unless another is faster by more than MARGIN.  The choice is
recorded in a JSON cache keyed by lattice, precision, deflation size, sources,
Krylov dimension and device, so a later process with the same key sets it
without timing (also one that a former version of the library wrote: the
results are the same, and deleting the file has the shapes timed anew).

This module only schedules and times calls of the library; all arithmetic
runs in its kernels.
"""
from __future__ import annotations

import itertools
import json
import os
import statistics
import time

from . import (sgn_apply_batched_fixed, sgn_apply_fixed, sgn_deflation_size, sgn_get_dims, sgn_get_precision,
               sgn_get_tuning, sgn_matvec, sgn_set_stencil_blocks, sgn_set_tuning)

UPDATE_BATCH = (4, 8, 16)
DOT_COLS = (1, 2)
DEFAULT = (8, 2)  # the library's default shape
MARGIN = 0.01
# stencil walk blocks (By, Bz, Bt) tried by autotune_stencil: the default
# rule, the natural order and blocks around the default
STENCIL_BLOCKS = ((0, 0, 0), (-1, 0, 0), (4, 16, 2), (4, 16, 8), (4, 8, 8), (8, 8, 2), (8, 8, 4), (2, 8, 4),
                  (8, 4, 4))
STENCIL_STEPS = 4
STENCIL_MARGIN = 0.015  # of a short apply, about a quarter of which is stencils; below it the default walk stays


def _key(ctx, nrhs, k, device):
    dims, n = sgn_get_dims(ctx)
    return "|".join(str(v) for v in ("x".join(map(str, dims)), n, sgn_get_precision(ctx), sgn_deflation_size(ctx),
                                        nrhs, k, device))


def _load(path):
    if path and os.path.exists(path):
        with open(path) as f:
            return json.load(f)
    return {}


def autotune(ctx, k=256, nrhs=1, cache=None, reps=3):
    """Pick the fastest bitwise-neutral launch shape for this context and set
    it.  k: Krylov dimension of the timed applies (about the k the workload
    reaches); nrhs: sources per batched apply (1: sgn_apply).  cache: JSON
    file path or None.  Returns {"update_batch", "dot_cols", "ms", "cached"}
    (ms: per apply of the chosen shape, None when taken from the cache)."""
    import torch

    device = torch.cuda.get_device_name()
    key = _key(ctx, nrhs, k, device)
    table = _load(cache)
    _, _, uw = sgn_get_tuning(ctx)
    if key in table:
        ub, cpw = table[key]["update_batch"], table[key]["dot_cols"]
        sgn_set_tuning(ctx, ub, cpw, uw)
        return {"update_batch": ub, "dot_cols": cpw, "ms": None, "cached": True}

    _, n = sgn_get_dims(ctx)
    gen = torch.Generator(device="cuda").manual_seed(12345)
    X = torch.randn(nrhs, n, dtype=torch.complex128, device="cuda", generator=gen)
    Y = torch.empty_like(X)
    torch.cuda.synchronize()  # the library reads X on the context's stream

    def run():
        if nrhs == 1:
            sgn_apply_fixed(ctx, X[0], Y[0], k)
        else:
            sgn_apply_batched_fixed(ctx, X, Y, k)

    times = {}
    for ub, cpw in itertools.product(UPDATE_BATCH, DOT_COLS):
        sgn_set_tuning(ctx, ub, cpw, uw)
        run()  # warm-up (first launches of these kernel instances)
        best = float("inf")
        for _ in range(reps):
            t0 = time.perf_counter()
            run()
            best = min(best, time.perf_counter() - t0)
        times[(ub, cpw)] = best
    (ub, cpw), t = min(times.items(), key=lambda kv: kv[1])
    if t > (1.0 - MARGIN) * times[DEFAULT]:
        (ub, cpw), t = DEFAULT, times[DEFAULT]
    sgn_set_tuning(ctx, ub, cpw, uw)
    if cache:
        table = _load(cache)  # merge with what other processes wrote meanwhile
        table[key] = {"update_batch": ub, "dot_cols": cpw, "ms": round(1e3 * t, 4)}
        os.makedirs(os.path.dirname(os.path.abspath(cache)), exist_ok=True)
        tmp = cache + ".tmp"
        with open(tmp, "w") as f:
            json.dump(table, f, indent=1, sort_keys=True)
        os.replace(tmp, cache)
    return {"update_batch": ub, "dot_cols": cpw, "ms": round(1e3 * t, 4), "cached": False}


def autotune_stencil(ctx, reps=10):
    """Pick the fastest stencil walk (sgn_set_stencil_blocks; results are
    bitwise the same for every walk) for this context's applies by timing
    short ones (sgn_apply_fixed with STENCIL_STEPS Krylov steps, in the
    context's precision and block mode, mostly stencils): the applies work in
    the component-major layout, sgn_matvec by itself in the interface layout.
    Shapes that do not fit the lattice are skipped, and the default walk stays
    unless another is faster by more than STENCIL_MARGIN.  Returns
    {"blocks": (By, Bz, Bt), "us": per matvec}."""
    import torch

    from . import SgnError

    _, n = sgn_get_dims(ctx)
    gen = torch.Generator(device="cuda").manual_seed(4321)
    x = torch.randn(n, dtype=torch.complex128, device="cuda", generator=gen)
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    walks = []
    for blocks in STENCIL_BLOCKS:
        try:
            sgn_set_stencil_blocks(ctx, *blocks)
        except SgnError:
            continue
        sgn_apply_fixed(ctx, x, y, STENCIL_STEPS)  # warm-up
        walks.append(blocks)
    ratios = {blocks: [] for blocks in walks}
    for _ in range(2 * reps):  # the walks in turn, each against the default one of its round
        t = {}
        for blocks in walks:
            sgn_set_stencil_blocks(ctx, *blocks)
            t0 = time.perf_counter()
            sgn_apply_fixed(ctx, x, y, STENCIL_STEPS)
            t[blocks] = time.perf_counter() - t0
        for blocks in walks:
            ratios[blocks].append(t[blocks] / t[walks[0]])
    middle = {blocks: statistics.median(r) for blocks, r in ratios.items()}
    best = min(walks, key=middle.get)
    if middle[best] > 1.0 - STENCIL_MARGIN:
        best = walks[0]
    sgn_set_stencil_blocks(ctx, *best)
    sgn_matvec(ctx, x, y)  # warm-up
    t0 = time.perf_counter()
    for _ in range(reps):
        sgn_matvec(ctx, x, y)
    us = 1e6 * (time.perf_counter() - t0) / reps
    return {"blocks": best, "us": round(us, 2)}
