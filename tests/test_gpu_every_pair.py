"""Every pair evaluated, FP32: the forms with the ring count compiled in (1 to 9 rings
per lane group, at the edges of each) give bit for bit the results of the streamed
form, which takes any ring count."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r_max", [1, 4, 5, 8, 9, 12, 13, 16, 17, 20, 21, 24, 25, 28, 29, 32, 33, 36])
def test_ring_counts(r_max):
    from paper_2011_05755_amd import mra, synth
    dev = torch.device("cuda", 0)
    L, K, T, N = 2 * r_max + 10, 11, 1, 13
    print(f"[gpu-every-pair] rings 1..{r_max}", flush=True)
    refs = synth.render_refs(synth.make_blobs(K, L, seed=(r_max, 0), rho_max=r_max + 1.0, sigma=(0.4, 2.0))).to(dev)
    parts = torch.randn((N, L, L), generator=torch.Generator(device=dev).manual_seed(r_max), device=dev)
    parts += refs[torch.arange(N, device=dev) % K]
    got = {}
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs, r_min=1, r_max=r_max, shift_max=T)
        for v in (0, 1, 2):
            ctx.set_tuning(0, corr_variant=v, prune=0)
            got[v] = ctx.align(0, parts, with_cc2=True).to_numpy()
    for v in (0, 1):
        for f in got[2]:
            np.testing.assert_array_equal(got[v][f].view(np.int32), got[2][f].view(np.int32), err_msg=f"variant {v} {f}")
