"""Reference sets replaced under one id: the buffers of a replaced set serve the
next set of its sizes, which must change no result, whatever came between."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("K", [1, 13])
def test_replaced_references(precision, K):
    from paper_2011_05755_amd import mra, synth
    dev = torch.device("cuda", 0)
    L, T, N, r_max = 64, 2, 40, 27
    sets = []
    for seed in (1, 2, 3):
        blobs = synth.make_blobs(K, L, seed=(seed, 0), rho_max=28.0)
        refs = synth.render_refs(blobs).to(dev)
        parts, _ = synth.make_particles(blobs, N, T, 0.1, seed=(seed, 1), device=dev)
        sets.append((refs, parts))
    kw = dict(r_min=1, r_max=r_max, shift_max=T, precision=precision)

    def fresh(i):
        with mra.Context(0) as c:
            c.load_refs(0, sets[i][0], **kw)
            r = c.align(0, sets[i][1], with_cc2=True).to_numpy()
            q, n = c.debug_refs(0)
            torch.cuda.synchronize()
            return r, q.cpu().numpy(), n.cpu().numpy()

    want = [fresh(i) for i in range(3)]
    with mra.Context(0) as ctx:
        def check(i):
            got = ctx.align(0, sets[i][1], with_cc2=True).to_numpy()
            q, n = ctx.debug_refs(0)
            for f in got:
                np.testing.assert_array_equal(got[f], want[i][0][f], err_msg=f)
            np.testing.assert_array_equal(q.cpu().numpy(), want[i][1])
            np.testing.assert_array_equal(n.cpu().numpy(), want[i][2])

        for i in (0, 1, 2, 0, 2):   # the third load on takes a replaced set's buffers
            ctx.load_refs(0, sets[i][0], **kw)
            check(i)
        # a set that is refused leaves the loaded one as it was, and the next loads sound
        bad = sets[1][0].clone()
        bad[K - 1] = 0.0
        with pytest.raises(mra.MRAError) as e:
            ctx.load_refs(0, bad, **kw)
        assert e.value.code == mra.MRA_E_DEGENERATE
        check(2)
        # other sizes between two loads of the same
        ctx.load_refs(0, torch.cat([sets[0][0]] * 2), **kw)
        ctx.load_refs(0, sets[1][0], **kw)
        check(1)
        # two ids: one's buffers are not the other's
        ctx.load_refs(5, sets[2][0], **kw)
        ctx.load_refs(0, sets[0][0], **kw)
        ctx.load_refs(0, sets[1][0], **kw)
        check(1)
        np.testing.assert_array_equal(ctx.align(5, sets[2][1]).cc.cpu().numpy(), want[2][0]["cc"])
        ctx.unload_refs(5)
        ctx.load_refs(0, sets[0][0], **kw)
        check(0)
