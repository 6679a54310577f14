"""More references than one packing launch holds, and than 2^32 elements of the
16-bit operand: a particle that is one of them finds itself, whichever it is, and
evaluating only the pairs that can win gives what evaluating every pair gives."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_the_last_of_many_references(precision):
    from paper_2011_05755_amd import mra
    K, L = 530000, 12
    print(f"[gpu-many-refs] {precision} K={K}", flush=True)
    dev = torch.device("cuda", 0)
    refs = torch.randn((K, L, L), generator=torch.Generator(device=dev).manual_seed(3), device=dev)
    pick = [0, 7, 4096, 262144, 340001, 524287, 524288, 529992, K - 1] + list(range(500000, 529000, 1450))
    parts = refs[torch.as_tensor(pick, device=dev)].contiguous()
    got = []
    with mra.Context(0) as ctx:
        ctx.load_refs(0, refs, r_min=1, r_max=4, shift_max=1, mirror=False, precision=precision)
        for prune in (1, 0):
            ctx.set_tuning(0, prune=prune)
            ctx.profile(True)
            got.append(ctx.align(0, parts).to_numpy())
            assert (ctx.profile_read("bound")[1] > 0) == (prune == 1)
    for f in got[0]:
        np.testing.assert_array_equal(got[0][f], got[1][f], err_msg=f)
    assert got[0]["ref"].tolist() == pick
    for f in ("shift_x", "shift_y", "psi"):
        assert (got[0][f] == 0).all()
