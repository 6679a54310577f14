"""Which way an alignment takes, read from the kernel groups that it launched: every
pair evaluated (few pairs, pruning off), or bounds first.  Whatever the way, the
results are bit for bit the same: at every ring bucket, noise-free and noisy,
without mirrors or normalisation, with reference sets replaced in between, and in
a batch of one stack."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
PRECISIONS = ["fp32", "bf16", "fp16"]
GROUPS = ("polar", "bound", "tighten", "fine", "fine2", "corr", "corr2", "merge")


@pytest.fixture(scope="module")
def ctx():
    from paper_2011_05755_amd import mra
    c = mra.Context(0)
    yield c
    c.close()


def stack(L, K, T, N, r_max, snr=0.05, seed=31, mirror=True):
    from paper_2011_05755_amd import synth
    blobs = synth.make_blobs(K, L, seed=(seed, L), rho_max=r_max + 1.0)
    parts, _ = synth.make_particles(blobs, N, T, snr, seed=(seed, 1), device=DEV, mirror=mirror)
    return synth.render_refs(blobs).to(DEV), parts


def run(ctx, call):
    """(results, groups that were launched)"""
    ctx.profile(True)
    out = call()
    torch.cuda.synchronize()
    ran = {g for g in GROUPS if ctx.profile_read(g)[1]}
    ctx.profile(False)
    return out.to_numpy(), ran


def same(a, b):
    for f in a:
        x, y = (v.view(np.int32) if v.dtype.kind == "f" else v for v in (a[f], b[f]))
        assert np.array_equal(x, y), (f, np.flatnonzero(x != y)[:5])


def bounds_first(precision, cc2=True):
    ran = {"polar", "bound", "fine"} | ({"fine2"} if cc2 else set())
    return ran | ({"tighten"} if precision == "fp32" else set())


def every_pair(cc2=True):
    return {"polar", "corr", "merge"} | ({"corr2"} if cc2 else set())


def both(ctx, precision, parts, expect):
    """The default way is `expect`; pruning off gives the same by evaluating every pair."""
    ctx.set_tuning(0)
    got, ran = run(ctx, lambda: ctx.align(0, parts, with_cc2=True))
    assert ran == expect, ran
    ctx.set_tuning(0, prune=0)
    want, ran = run(ctx, lambda: ctx.align(0, parts, with_cc2=True))
    assert ran == every_pair(), ran
    same(got, want)
    return want


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("snr", [None, 0.05])
@pytest.mark.parametrize("L,r_max,T,K,N", [(24, 9, 2, 400, 400), (64, 32, 3, 60, 171), (76, 35, 3, 100, 60),
                                           (90, 40, 2, 80, 170), (110, 48, 2, 81, 170), (140, 64, 4, 17, 200)])
def test_bounds_first(ctx, precision, snr, L, r_max, T, K, N):
    print(f"[gpu-routes] {precision} L={L} K={K} N={N} snr={snr}", flush=True)
    refs, parts = stack(L, K, T, N, r_max, snr)
    ctx.load_refs(0, refs, r_min=1, r_max=r_max, shift_max=T, precision=precision)
    both(ctx, precision, parts, bounds_first(precision))


# few particles, few pairs per particle (one reference tile, no shifts), and row tiles
# whose references are split in one, several and as many parts as there are
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("L,r_max,T,K,N", [(64, 28, 2, 21, 1), (64, 28, 2, 50, 29), (64, 28, 2, 41, 90), (64, 28, 0, 60, 1000),
                                           (48, 20, 2, 8, 1300), (96, 46, 2, 30, 14)])
def test_every_pair(ctx, precision, L, r_max, T, K, N):
    print(f"[gpu-routes] {precision} L={L} K={K} N={N}", flush=True)
    refs, parts = stack(L, K, T, N, r_max)
    ctx.load_refs(0, refs, r_min=1, r_max=r_max, shift_max=T, precision=precision)
    want = both(ctx, precision, parts, every_pair())
    # a batch of one stack is that stack's call
    from paper_2011_05755_amd import mra
    out = mra.AlignResult.empty(N, DEV)

    def batch():
        ctx.align_batch([(0, parts, -1, out)])
        return out
    for prune in (-1, 0):
        ctx.set_tuning(0, prune=prune)
        got, ran = run(ctx, batch)
        assert ran == every_pair(cc2=False), ran
        same(got, {f: want[f] for f in got})


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("kw", [dict(mirror=False), dict(normalize=False, r_min=3)])
def test_options(ctx, precision, kw):
    print(f"[gpu-routes] {precision} {kw}", flush=True)
    refs, parts = stack(76, 100, 3, 70, 35, 0.2, mirror=kw.get("mirror", True))
    ctx.load_refs(0, refs, r_max=35, shift_max=3, precision=precision, **{"r_min": 1, **kw})
    both(ctx, precision, parts, bounds_first(precision))


@pytest.mark.parametrize("precision", PRECISIONS)
def test_replaced_references(precision):
    from paper_2011_05755_amd import mra
    print(f"[gpu-routes] {precision} replaced references", flush=True)
    kw = dict(r_min=1, r_max=35, shift_max=3, precision=precision)
    sets = [stack(76, 100, 3, 60, 35, seed=s) for s in (1, 2, 3)]
    want = []
    for refs, parts in sets:
        with mra.Context(0) as c:
            c.load_refs(0, refs, **kw)
            c.set_tuning(0, prune=0)
            want.append(c.align(0, parts, with_cc2=True).to_numpy())
    with mra.Context(0) as c:
        for i in (0, 1, 2, 0, 2, 1):    # from the third load on in a replaced set's buffers
            c.load_refs(0, sets[i][0], **kw)
            got, ran = run(c, lambda: c.align(0, sets[i][1], with_cc2=True))
            assert ran == bounds_first(precision), ran
            same(got, want[i])


def test_small_reference_sets_scale_into_the_bounds():
    """FP32 references below 2^-113 (raw CC): the bounds' FP16 operand takes the largest finite scale."""
    from paper_2011_05755_amd import mra
    refs, parts = stack(76, 100, 3, 60, 35)
    got = []
    with mra.Context(0) as c:
        for s in (1.0, 2.0 ** -118):
            c.load_refs(0, (refs * s).contiguous(), r_min=1, r_max=35, shift_max=3, normalize=False)
            r, ran = run(c, lambda: c.align(0, parts, with_cc2=True))
            assert ran == bounds_first("fp32"), ran
            c.set_tuning(0, prune=0)
            same(r, c.align(0, parts, with_cc2=True).to_numpy())
            got.append(r)
    np.testing.assert_array_equal(got[0]["flat_index"], got[1]["flat_index"])
    np.testing.assert_array_equal(np.ldexp(got[0]["cc"], -118), got[1]["cc"])


# sizes beyond the rule on pairs, in every row here
@pytest.mark.parametrize("precision,K,r_max,N,cc2,every", [
    ("bf16", 8, 28, 1600, False, True), ("bf16", 16, 28, 1300, False, True), ("fp16", 16, 46, 700, False, True),
    ("bf16", 17, 28, 2600, False, False), ("fp32", 16, 28, 1100, False, False), ("bf16", 16, 28, 700, True, False),
    ("fp16", 16, 12, 800, False, False)])
def test_few_references(ctx, precision, K, r_max, N, cc2, every):
    from paper_2011_05755_amd import mra
    print(f"[gpu-routes] {precision} K={K} r_max={r_max} N={N} cc2={cc2}", flush=True)
    refs, parts = stack(2 * r_max + 8, K, 3, N, r_max)
    ctx.load_refs(0, refs, r_min=1, r_max=r_max, shift_max=3, precision=precision)
    expect = every_pair(cc2) if every else bounds_first(precision, cc2)
    got, ran = run(ctx, lambda: ctx.align(0, parts, with_cc2=cc2))
    assert ran == expect, ran
    # the other way: with the runner-up bounds come first, without pruning they don't
    ctx.set_tuning(0, prune=-1 if every else 0)
    want, ran = run(ctx, lambda: ctx.align(0, parts, with_cc2=True))
    assert ran == (bounds_first(precision) if every else every_pair()), ran
    same(got, {f: want[f] for f in got})
    if cc2:
        return
    ctx.set_tuning(0)
    out = [mra.AlignResult.empty(N, DEV) for _ in range(2)]
    ctx.profile(True)
    ctx.align_batch([(0, parts, -1, o) for o in out])
    torch.cuda.synchronize()
    assert {g for g in GROUPS if ctx.profile_read(g)[1]} == expect
    ctx.profile(False)
    for o in out:
        same(o.to_numpy(), {f: want[f] for f in got})


# few rings keep many pairs live: more pairs than a box full of rings may have evaluate
# all of them (R4 6 and 9; tile pairs per CU: 41)
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("L,r_max,every", [(65, 21, True), (76, 36, False)])
def test_few_rings(ctx, precision, L, r_max, every):
    print(f"[gpu-routes] {precision} L={L} rings {r_max}", flush=True)
    refs, parts = stack(L, 263, 2, 103, r_max)
    ctx.load_refs(0, refs, r_min=1, r_max=r_max, shift_max=2, precision=precision)
    got, ran = run(ctx, lambda: ctx.align(0, parts))
    assert ran == (every_pair(False) if every else bounds_first(precision, False)), ran
    ctx.set_tuning(0, prune=0)
    want, _ = run(ctx, lambda: ctx.align(0, parts))
    same(got, want)
