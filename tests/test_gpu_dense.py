"""Particles of which nearly every pair is live (references that are particles
themselves, blank images) among ordinary ones: alone and in batches, at every ring
bucket and search range, bit for bit the result of evaluating every pair, and in
about its time (before, evaluating their pairs a few at a time took 3 to 20 times
it)."""

import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
PRECISIONS = ["fp32", "bf16", "fp16"]


def stack(L, K, T, N, r_max, seed=11):
    """(references, particles): every third particle noise of its own, every seventh blank;
    half of the references particles, the others clean."""
    from paper_2011_05755_amd import synth
    blobs = synth.make_blobs(K, L, seed=(seed, L), rho_max=r_max + 1.0)
    refs = synth.render_refs(blobs).to(DEV)
    refs[::2] = synth.make_particles(blobs, K, T, 0.05, seed=(seed, 1), device=DEV)[0][::2]
    parts, _ = synth.make_particles(blobs, N, T, 0.2, seed=(seed, 2), device=DEV)
    parts[1::3] = torch.randn(parts[1::3].shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)
    parts[4::7] = 0.0
    return refs.contiguous(), parts


def same(a, b, what):
    for f in a:
        x, y = (v.view(np.int32) if v.dtype.kind == "f" else v for v in (a[f], b[f]))
        assert np.array_equal(x, y), (what, f, np.flatnonzero(x != y)[:5])


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("L,r_max,T,K,N", [(24, 9, 0, 200, 900), (64, 32, 1, 41, 2800), (64, 28, 2, 41, 2300),
                                           (76, 35, 3, 33, 300), (90, 40, 2, 48, 400), (110, 48, 2, 43, 400),
                                           (140, 64, 4, 17, 220), (160, 64, 8, 17, 60)])
def test_dense_particles(precision, L, r_max, T, K, N):
    from paper_2011_05755_amd import mra
    print(f"[gpu-dense] {precision} L={L} T={T} K={K} N={N}", flush=True)
    refs, parts = stack(L, K, T, N, r_max)
    got = []
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs, r_min=1, r_max=r_max, shift_max=T, precision=precision)
        for prune in (1, 0):
            ctx.set_tuning(0, prune=prune)
            got.append((ctx.align(0, parts, with_cc2=True).to_numpy(), ctx.align(0, parts).to_numpy()))
    same(got[0][0], got[1][0], "cc2")
    same(got[0][1], got[1][1], "plain")


@pytest.mark.parametrize("precision", PRECISIONS)
def test_dense_particles_in_a_batch(precision):
    from paper_2011_05755_amd import mra
    print(f"[gpu-dense] {precision} batch", flush=True)
    with mra.Context(0) as ctx:
        stacks, want = [], []
        for i, (L, r_max, T, K, N) in enumerate([(64, 28, 2, 100, 300), (76, 32, 1, 150, 300), (64, 25, 3, 100, 150),
                                                 (90, 33, 2, 100, 150), (96, 36, 2, 100, 150)]):
            refs, parts = stack(L, K, T, N, r_max, seed=20 + i)
            ctx.load_refs(i, refs, r_min=1, r_max=r_max, shift_max=T, precision=precision)
            ctx.set_tuning(i, prune=0)
            want.append(ctx.align(i, parts).to_numpy())
            ctx.set_tuning(i)
            stacks.append((i, parts, -1, mra.AlignResult.empty(N, DEV)))
        for _ in range(2):
            ctx.align_batch(stacks)
            for (i, _, _, o), w in zip(stacks, want):
                same(o.to_numpy(), w, f"stack {i}")


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("kind", ["particles", "blank"])
def test_dense_particles_take_the_time_of_every_pair(precision, kind):
    from paper_2011_05755_amd import mra, synth
    L, K, T, N = 76, 100, 3, 1000
    print(f"[gpu-dense] {precision} {kind} time", flush=True)
    blobs = synth.make_blobs(K, L, seed=(3, 0), rho_max=28.0)
    parts, _ = synth.make_particles(blobs, N, T, 0.05, seed=(3, 1), device=DEV)
    refs = parts[:K].clone() if kind == "particles" else synth.render_refs(blobs).to(DEV)
    if kind == "blank":
        parts.zero_()
    ms = []
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs, r_min=1, r_max=35, shift_max=T, precision=precision)
        for prune in (1, 0):
            ctx.set_tuning(0, prune=prune)
            out = ctx.align(0, parts)
            t = []
            for _ in range(5):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                ctx.align(0, parts, out=out)
                torch.cuda.synchronize()
                t.append(time.perf_counter() - t0)
            ms.append(min(t) * 1e3)
    # (the bounds, and in FP32 the rows' operand once more, come on top of every pair)
    assert ms[0] < 2 * ms[1], ms
