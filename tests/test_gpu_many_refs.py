"""More references than one packing launch holds, and than 2^32 elements of the
16-bit operand: a particle that is one of them finds itself, whichever it is, and
evaluating only the pairs that can win gives what evaluating every pair gives."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_the_last_of_many_references():
    from paper_2011_05755_amd import mra
    K, L = 530000, 8
    print(f"[gpu-many-refs] K={K}", flush=True)
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    refs = torch.randn((K, L, L), generator=g, device=dev)
    pick = [0, 7, 4096, 262144, 340001, 524287, 524288, 529992, K - 1]
    parts = refs[torch.as_tensor(pick, device=dev)].contiguous()
    got = []
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs, r_min=1, r_max=3, shift_max=0, mirror=False)
        for prune in (1, 0):
            ctx.set_tuning(0, prune=prune)
            got.append(ctx.align(0, parts).to_numpy())
    for f in got[0]:
        np.testing.assert_array_equal(got[0][f], got[1][f], err_msg=f)
    assert got[0]["ref"].tolist() == pick
    assert (got[0]["psi"] == 0).all()
