"""The FP16 form at the ends of the float range.  A particle's operand is scaled
by a power of two of its own, so a particle times 2^k has the same winner and
CC and runner-up times 2^k exactly, as long as no pixel times 512 and no CC leaves
the range; a particle that does not scale into FP16 (a pixel that is not finite,
or times 512 is not) has no winner.  On both ways, few particles (every pair
evaluated) and many (only the pairs that can win)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

INT = ("ref", "shift_x", "shift_y", "psi", "mirror", "flat_index")


def run(refs, parts, rows):
    from paper_2011_05755_amd import mra
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs, r_min=1, r_max=28, shift_max=2, precision="fp16", rescore_rows=rows)
        r = ctx.align(0, parts, with_cc2=True)
        torch.cuda.synchronize()
        return r.to_numpy()


def stack(N):
    from paper_2011_05755_amd import synth
    dev = torch.device("cuda", 0)
    blobs = synth.make_blobs(41, 64, seed=(5, 0), rho_max=28.0)
    parts, _ = synth.make_particles(blobs, N, 2, 0.1, seed=(5, N), device=dev)
    return synth.render_refs(blobs).to(dev), parts


@pytest.mark.parametrize("rows", [0, 4])
@pytest.mark.parametrize("N", [24, 400])
@pytest.mark.parametrize("top", [126, -20])
def test_powers_of_two(N, rows, top):
    print(f"[gpu-fp16-range] N={N} rows={rows} 2^{top}", flush=True)
    refs, parts = stack(N)
    k = top - int(np.ceil(np.log2(512.0 * float(parts.abs().max()))))
    want, got = run(refs, parts, rows), run(refs, (parts.double() * 2.0 ** k).float(), rows)
    for f in INT:
        np.testing.assert_array_equal(got[f], want[f], err_msg=f)
    for f in ("cc", "cc2"):
        w = np.ldexp(want[f].astype(np.float64), k).astype(np.float32)
        assert np.isfinite(w).all() and (w != 0).all()
        np.testing.assert_array_equal(got[f], w, err_msg=f)


@pytest.mark.parametrize("rows", [0, 4])
@pytest.mark.parametrize("N", [24, 400])
def test_out_of_range(N, rows):
    print(f"[gpu-fp16-range] N={N} rows={rows} out of range", flush=True)
    refs, parts = stack(N)
    want = run(refs, parts, rows)
    bad = {2: float("inf"), 5: -float("inf"), 11: 2.0 ** 120, 20: 3e38}
    for n, v in bad.items():
        parts[n, 61, 32] = v          # reached by some shifts only
    got = run(refs, parts, rows)
    ok = np.array([n not in bad for n in range(N)])
    for f in INT + ("cc", "cc2"):
        np.testing.assert_array_equal(got[f][ok], want[f][ok], err_msg=f)
    for f, v in (("ref", -1), ("flat_index", -1), ("shift_x", 0), ("shift_y", 0), ("psi", 0), ("mirror", 0)):
        assert (got[f][~ok] == v).all(), f
    assert np.isnan(got["cc"][~ok]).all() and np.isnan(got["cc2"][~ok]).all()
