"""The 16-bit particle operand over the ways its samples are taken: every
pattern in which 8 rows wrap over the shift grid (1, 3, 5, 7 and more columns,
particles that start at each row of a tile), windows smaller than the image,
and images that leave a CU room for one workgroup of 8 to 16 waves.  A shift by
whole pixels moves the taps and changes no weight, so the CC table of a search
over shifts is, bit for bit, that of the shifted images searched at shift 0;
copies of one image, which start at different rows of a tile, have one table."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["bf16", "fp16"])
@pytest.mark.parametrize("L,r_max,T", [(40, 12, 1), (64, 27, 2), (76, 35, 3), (64, 20, 4), (64, 20, 5), (64, 15, 8),
                                       (90, 20, 3), (96, 46, 2), (128, 62, 4), (160, 64, 8)])
def test_table_of_shifts_is_that_of_shifted_images(precision, L, r_max, T):
    from paper_2011_05755_amd import mra, synth
    dev = torch.device("cuda", 0)
    K, copies, S1 = 2, 8 if T < 8 else 3, 2 * T + 1
    blobs = synth.make_blobs(K, L, seed=(L, T), rho_max=r_max + 1.0)
    refs = synth.render_refs(blobs).to(dev)
    parts, _ = synth.make_particles(blobs, 1, T, 0.1, seed=(L, 9), device=dev)
    img = torch.zeros_like(parts[0])
    img[T:L - T, T:L - T] = parts[0, T:L - T, T:L - T]   # a shift loses no pixel
    if L // 2 - r_max - 2 * T > 4:
        img[T, T] = 50.0 * img.abs().max()               # in no sample, but in the FP16 scale
    shifted = torch.stack([torch.roll(img, (-dy, -dx), (0, 1)) for dy in range(-T, T + 1) for dx in range(-T, T + 1)])
    with mra.Context(0) as ctx:
        kw = dict(r_min=1, r_max=r_max, precision=precision)
        ctx.load_refs(0, refs, shift_max=T, **kw)
        got = ctx.debug_cctable(0, img.expand(copies, L, L).contiguous())
        ctx.load_refs(0, refs, shift_max=0, **kw)
        want = ctx.debug_cctable(0, shifted)
        torch.cuda.synchronize()
    want = want.reshape(S1, S1, K, 2, 256).permute(2, 3, 0, 1, 4)
    got = got.reshape(copies, K, 2, S1, S1, 256)
    assert want.abs().max() > 0
    for c in range(copies):
        assert torch.equal(got[c], want), (c, int((got[c] != want).sum()))
