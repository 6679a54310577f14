"""Bounds first, at sizes that take that way (checked by the kernels that are launched):
special pixels and references, every option, particles left to the whole chip, and
batches, bit for bit the result of evaluating every pair."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
PRECISIONS = ["fp32", "bf16", "fp16"]


def stack(L, K, T, N, r_max, snr=0.05, seed=41):
    from paper_2011_05755_amd import synth
    blobs = synth.make_blobs(K, L, seed=(seed, 0), rho_max=r_max + 1.0)
    parts, _ = synth.make_particles(blobs, N, T, snr, seed=(seed, 1), device=DEV)
    return synth.render_refs(blobs).to(DEV), parts


def launched(ctx, call):
    """(results, numbers of bound and correlation launches)"""
    ctx.profile(True)
    out = call()
    torch.cuda.synchronize()
    ran = [ctx.profile_read(g)[1] for g in ("bound", "corr")]
    ctx.profile(False)
    return out, ran


def same(a, b, what=""):
    for f in a:
        x, y = a[f], b[f]
        if x.dtype.kind == "f":     # every NaN counts as equal
            x, y = (np.where(np.isnan(v), np.float32(0), v).view(np.int32) + np.isnan(v) * 3 for v in (x, y))
        assert np.array_equal(x, y), (what, f, np.flatnonzero(x != y)[:5])


def both(precision, refs, parts, r_max, T, **kw):
    from paper_2011_05755_amd import mra
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs.contiguous(), r_max=r_max, shift_max=T, precision=precision, **{"r_min": 1, **kw})
        for cc2 in (True, False):
            ctx.set_tuning(0)
            got, ran = launched(ctx, lambda: ctx.align(0, parts, with_cc2=cc2))
            assert ran == [1, 0], ran
            ctx.set_tuning(0, prune=0)
            same(got.to_numpy(), ctx.align(0, parts, with_cc2=cc2).to_numpy(), f"cc2 {cc2}")


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("kw", [dict(), dict(mirror=False), dict(normalize=False), dict(rescore_rows=0), dict(rescore_rows=8),
                                dict(r_min=3)])
def test_special_pixels_and_options(precision, kw):
    print(f"[gpu-bounds-first] {precision} {kw}", flush=True)
    refs, parts = stack(76, 100, 3, 170, 35)
    parts[3] = 0.0
    parts[17, 36, 39] = float("nan")
    parts[18, 2, 2] = float("nan")      # outside every ring
    parts[29, 37, 37] = float("inf")
    parts[30, 71, 38] = -float("inf")   # reached by some shifts only
    for i, scale in enumerate((1e-42, 1e-38, 1e-30, 1e-20, 1e-10, 1e10, 1e20, 1e30, 3e34, 1e36)):
        parts[40 + 7 * i] *= scale
    parts[150] = 1.0
    parts[151, :, :38] = 0.0
    both(precision, refs, parts, 35, 3, **kw)


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("kind", ["scales", "noise", "same"])
def test_special_references(precision, kind):
    print(f"[gpu-bounds-first] {precision} references {kind}", flush=True)
    refs, parts = stack(76, 100, 3, 150, 35)
    if kind == "scales":    # raw CC, references of sizes up to 10^8 apart
        refs = refs * torch.logspace(-4, 4, 100, device=DEV)[:, None, None]
    elif kind == "noise":   # references that are particles
        refs = parts[:100].clone()
    else:                   # references in identical pairs: ties between them
        refs[1::2] = refs[0::2]
    both(precision, refs, parts, 35, 3, normalize=kind != "scales")


# every pair of every particle live; the step limit of each launch size
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("K,N", [(210, 260), (41, 2400), (20, 8400)])
def test_left_over(precision, K, N):
    print(f"[gpu-bounds-first] {precision} left over K={K} N={N}", flush=True)
    refs, _ = stack(64, K, 2, K, 31, 0.02, seed=8)
    refs = stack(64, K, 2, K, 31, 0.02, seed=9)[1]
    both(precision, refs, stack(64, K, 2, N, 31, 0.02, seed=9)[1], 31, 2)


# a ring bucket each of 16-bit forms (FP32: the resident and the streamed operand)
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("shapes", [((64, 28, 2, 100, 300), (76, 32, 1, 150, 300), (64, 25, 3, 100, 150)),
                                    ((90, 33, 2, 100, 151), (96, 36, 2, 100, 150), (90, 39, 1, 200, 150)),
                                    ((110, 44, 2, 100, 151), (128, 62, 2, 70, 220), (110, 48, 3, 60, 120), (128, 52, 3, 41, 150))])
def test_batches(precision, shapes):
    from paper_2011_05755_amd import mra
    print(f"[gpu-bounds-first] {precision} batch {shapes}", flush=True)
    stacks, want = [], []
    with mra.Context(0) as ctx:
        for i, (L, r_max, T, K, N) in enumerate(shapes):
            refs, parts = stack(L, K, T, N, r_max, seed=60 + i)
            refs[::3] = parts[:refs[::3].shape[0]]   # particles: some of the stack are dense
            parts[5] = 0.0
            parts[7, L // 2, L // 2] = float("nan")
            ctx.load_refs(i, refs, r_min=1, r_max=r_max, shift_max=T, precision=precision)
            ctx.set_tuning(i, prune=0)
            want.append(ctx.align(i, parts).to_numpy())
            ctx.set_tuning(i)
            stacks.append((i, parts, -1, mra.AlignResult.empty(N, DEV)))
        _, ran = launched(ctx, lambda: ctx.align_batch(stacks))
        assert ran[0] == (2 if len(shapes) == 4 else 1) and ran[1] == 0, ran
        for (i, _, _, out), w in zip(stacks, want):
            same(out.to_numpy(), w, shapes[i])
