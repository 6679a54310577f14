"""The bounds of the pruned alignment: whatever the input, evaluating only the
pairs whose bound can win gives bit for bit the result of evaluating every
pair.  Launches large enough for the pruned kernels (more than 12 row-tile x
reference-tile products per CU of a 256-CU GPU), at every ring bucket, search
range and option, and with the inputs on which a bound could go wrong:
all-zero images (every candidate ties), NaN and infinite pixels, pixels near
the ends of the float range, references of very different size, and
references that are themselves noise (bounds that prune nothing)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FIELDS = ("ref", "shift_x", "shift_y", "psi", "mirror", "flat_index", "cc", "cc2")


def log(msg):
    print(f"[gpu-bound] {msg}", flush=True)


@pytest.fixture(scope="module")
def ctx():
    from paper_2011_05755_amd import mra
    c = mra.Context(0)
    yield c
    c.close()


def both(ctx, parts, refs, r_max, T, **kw):
    """(pruned, unpruned) results as NumPy arrays."""
    ctx.load_refs(0, refs, r_min=kw.pop("r_min", 1), r_max=r_max, shift_max=T, **kw)
    got = []
    for prune in (1, 0):
        ctx.set_tuning(0, prune=prune)
        r = ctx.align(0, parts, with_cc2=True)
        torch.cuda.synchronize()
        got.append(r.to_numpy())
    return got


def assert_same(got):
    for f in FIELDS:
        a, b = got[0][f], got[1][f]
        if a.dtype.kind == "f":  # every NaN counts as equal
            a, b = (np.where(np.isnan(v), np.float32(0), v).view(np.int32) + np.isnan(v) * 3 for v in (a, b))
        assert np.array_equal(a, b), (f, np.flatnonzero(a != b)[:5])


def stack(L, K, T, N, r_max, snr=0.05, seed=41):
    from paper_2011_05755_amd import synth
    dev = torch.device("cuda", 0)
    blobs = synth.make_blobs(K, L, seed=(seed, 0), rho_max=r_max + 1.0)
    refs = synth.render_refs(blobs).to(dev)
    parts, _ = synth.make_particles(blobs, N, T, snr, seed=(seed, 1), device=dev)
    return refs, parts


# one case per ring bucket (R4 <= 8, 9..10, 11..12, 13..16) and at their edges
@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("L,r_max,T,K,N", [(24, 9, 2, 41, 170), (64, 32, 3, 24, 171), (76, 33, 2, 41, 170),
                                           (90, 40, 2, 48, 170), (96, 41, 1, 72, 310), (110, 48, 2, 43, 170),
                                           (120, 49, 2, 41, 170), (140, 64, 4, 17, 105)])
def test_every_ring_bucket(ctx, precision, L, r_max, T, K, N):
    log(f"{precision} L={L} rings 1..{r_max} T={T} K={K} N={N}")
    refs, parts = stack(L, K, T, N, r_max)
    assert_same(both(ctx, parts, refs, r_max, T, precision=precision))


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("kw", [dict(mirror=False), dict(normalize=False), dict(rescore_rows=0), dict(rescore_rows=8),
                                dict(r_min=7)])
def test_options(ctx, precision, kw):
    log(f"{precision} {kw}")
    refs, parts = stack(64, 56, 2, 145, 28)
    assert_same(both(ctx, parts, refs, 28, 2, precision=precision, **kw))


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
def test_special_pixels(ctx, precision):
    log(f"{precision}: zero, NaN, infinite, tiny and huge particles among ordinary ones")
    refs, parts = stack(64, 41, 2, 200, 28)
    parts[3] = 0.0
    parts[17, 30, 33] = float("nan")
    parts[18, 2, 2] = float("nan")      # outside every ring
    parts[29, 31, 31] = float("inf")
    parts[30, 61, 32] = -float("inf")   # reached by some shifts only
    for i, scale in enumerate((1e-42, 1e-38, 1e-30, 1e-20, 1e-10, 1e10, 1e20, 1e30, 3e34, 1e36)):
        parts[40 + 7 * i] *= scale
    parts[150] = 1.0
    parts[151, :, :32] = 0.0
    assert_same(both(ctx, parts, refs, 28, 2, precision=precision))


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("kind", ["scales", "noise", "same"])
def test_special_references(ctx, precision, kind):
    log(f"{precision}: references {kind}")
    refs, parts = stack(64, 42, 2, 171, 28)
    kw = {}
    if kind == "scales":    # raw CC, references of sizes up to 10^8 apart
        refs = refs * torch.logspace(-4, 4, 42, device=refs.device)[:, None, None]
        kw["normalize"] = False
    elif kind == "noise":   # references that are particles
        refs = parts[:42].clone()
    else:                   # references in identical pairs: ties between them
        refs[1::2] = refs[0::2]
    assert_same(both(ctx, parts, refs.contiguous(), 28, 2, precision=precision, **kw))
