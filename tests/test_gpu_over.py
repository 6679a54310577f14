"""Particles left to the whole chip: with references that are themselves noise
every pair of every particle is live, so each particle passes the step limit,
the list of those left over fills up and the rest go on where they are.  At each
step limit, bit for bit the result of evaluating every pair."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("K,N", [(41, 180), (210, 60), (41, 1500), (12, 8400)])
def test_left_over(precision, K, N):
    from paper_2011_05755_amd import mra, synth
    print(f"[gpu-over] {precision} K={K} N={N}", flush=True)
    dev = torch.device("cuda", 0)
    L, T, r_max = 24, 2, 9
    blobs = synth.make_blobs(K, L, seed=(7, K), rho_max=10.0)
    parts, _ = synth.make_particles(blobs, N, T, 0.02, seed=(7, N), device=dev)
    refs = synth.make_particles(blobs, K, T, 0.02, seed=(8, N), device=dev)[0].contiguous()
    got = []
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs, r_min=1, r_max=r_max, shift_max=T, precision=precision)
        for prune in (1, 0, 1):
            ctx.set_tuning(0, prune=prune)
            r = ctx.align(0, parts, with_cc2=True)
            torch.cuda.synchronize()
            got.append(r.to_numpy())
    for f in ("ref", "shift_x", "shift_y", "psi", "mirror", "flat_index", "cc", "cc2"):
        for other in (got[0], got[2]):
            a, b = (v.view(np.int32) if v.dtype.kind == "f" else v for v in (other[f], got[1][f]))
            assert np.array_equal(a, b), (f, np.flatnonzero(a != b)[:5])
