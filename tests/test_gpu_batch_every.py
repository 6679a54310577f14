"""Stacks of a batch whose every pair is evaluated share one launch of each kernel, and
each gets bit for bit what its own call gives: few references, few or no shifts, pruning
off, pieces that end inside a row tile, one particle, and a workspace that takes
the batch in several pieces."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
GROUPS = ("polar", "bound", "tighten", "fine", "corr", "merge")
# references, search range, particles, rescore_rows (16 bits), pruning
STACKS = [(8, 2, 300, 4, -1), (5, 3, 170, 1, 0), (8, 1, 1001, 4, -1), (70, 0, 1999, 4, -1), (3, 2, 1, 4, -1), (41, 2, 37, 8, 0)]


# rings: one count per lane group, so that FP32 takes one instance; edges of the buckets
@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("r_max,variant", [(3, -1), (28, -1), (28, 1), (36, -1), (40, 1), (48, -1), (64, -1)])
@pytest.mark.parametrize("cap", [32 << 30, 96 << 20])
def test_one_launch_of_each_kernel(precision, r_max, variant, cap):
    from paper_2011_05755_amd import mra, synth
    print(f"[gpu-batch-every] {precision} rings {r_max} variant {variant} cap {cap >> 20} MiB", flush=True)
    stacks, want = [], []
    with mra.Context(0, workspace_cap=cap) as ctx:
        for i, (K, T, N, rows, prune) in enumerate(STACKS):
            L = 2 * r_max + 8 + 2 * i
            N = N if r_max < 40 else (N + 3) // 4
            blobs = synth.make_blobs(K, L, seed=(i, r_max), rho_max=r_max + 2.0, sigma=(0.4, 2.0))
            parts, _ = synth.make_particles(blobs, N, T, 0.1, seed=(i, 1), device=DEV)
            ctx.load_refs(i, synth.render_refs(blobs).to(DEV), r_min=1, r_max=r_max, shift_max=T, precision=precision,
                          rescore_rows=rows if precision != "fp32" else 0)
            ctx.set_tuning(i, corr_variant=variant, prune=prune)
            want.append(ctx.align(i, parts).to_numpy())
            stacks.append((i, parts, -1, mra.AlignResult.empty(N, DEV)))
        for _ in range(2):    # the second time in a workspace that holds the first one's keys
            ctx.profile(True)
            ctx.align_batch(stacks)
            torch.cuda.synchronize()
            ran = {g: ctx.profile_read(g)[1] for g in GROUPS}
            ctx.profile(False)
            if cap > 1 << 30:
                assert ran == dict(polar=1, bound=0, tighten=0, fine=0, corr=1, merge=1), ran
            for (i, _, _, out), w in zip(stacks, want):
                got = out.to_numpy()
                for f in got:
                    x, y = (v.view(np.int32) if v.dtype.kind == "f" else v for v in (got[f], w[f]))
                    assert np.array_equal(x, y), (i, f, np.flatnonzero(x != y)[:5])
                out.cc.zero_(), out.flat_index.zero_()


# stacks of few pairs in all take every pair in one launch; a few of them beside stacks
# that don't join those stacks' wave
@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("sizes,every", [([(50, 8), (41, 8), (50, 5), (33, 1)], True), ([(8, 300), (200, 500)], False)])
def test_way_of_a_batch(precision, sizes, every):
    from paper_2011_05755_amd import mra, synth
    print(f"[gpu-batch-every] {precision} {sizes}", flush=True)
    stacks, want = [], []
    with mra.Context(0) as ctx:
        for i, (K, N) in enumerate(sizes):
            blobs = synth.make_blobs(K, 64, seed=(i, K), rho_max=28.0)
            parts, _ = synth.make_particles(blobs, N, 2, 0.1, seed=(i, 1), device=DEV)
            ctx.load_refs(i, synth.render_refs(blobs).to(DEV), r_min=1, r_max=28, shift_max=2, precision=precision)
            want.append(ctx.align(i, parts).to_numpy())
            stacks.append((i, parts, -1, mra.AlignResult.empty(N, DEV)))
        ctx.profile(True)
        ctx.align_batch(stacks)
        torch.cuda.synchronize()
        ran = {g: ctx.profile_read(g)[1] for g in ("polar", "bound", "corr")}
        ctx.profile(False)
    assert ran == dict(polar=1, bound=int(not every), corr=int(every)), ran
    for (i, _, _, out), w in zip(stacks, want):
        got = out.to_numpy()
        for f in got:
            x, y = (v.view(np.int32) if v.dtype.kind == "f" else v for v in (got[f], w[f]))
            assert np.array_equal(x, y), (i, f, np.flatnonzero(x != y)[:5])
