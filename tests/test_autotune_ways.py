"""The autotuner times only what can change the time of the sample's call: a
stand-in context that records its launches, on the CPU."""

import json

import pytest

from paper_2011_05755_amd import autotune, mra


class Refset:
    L, n_rings, K, shift_max, precision = 76, 35, 100, 3, "fp32"


class Ctx:
    """Accepts variants 0 .. 2, launches the correlation kernel for up to 40 particles,
    and takes longest with the default variant."""

    refsets = {0: Refset}

    def __init__(self):
        self.tuning, self.launched, self.recording, self.timed = (0, 0, 0), {}, False, []

    def set_tuning(self, rid, corr_variant=-1, chunk_particles=0, run_tiles=0):
        if corr_variant > 2:
            raise mra.MRAError(mra.MRA_E_INVAL, "variant cannot serve this geometry")
        self.tuning = (max(corr_variant, 0), chunk_particles, run_tiles)

    def get_tuning(self, rid):
        return self.tuning[:2]

    def profile(self, enable):
        self.launched, self.recording = {} if enable else self.launched, enable

    def profile_read(self, group):
        return 0.1, self.launched.get(group, 0)

    def align(self, rid, parts):
        assert self.recording
        self.launched = {"polar": 1, "corr" if parts.shape[0] <= 40 else "fine": 1}


class Parts:
    def __init__(self, n):
        self.shape = (n, 76, 76)


def timer(ctx, rid, parts, reps):
    ctx.timed.append(ctx.tuning)
    v, c, r = ctx.tuning
    return 5.0 - v - (0.5 if c == 128 else 0.0) - (0.1 if r else 0.0)


def test_a_sample_with_bounds_first_keeps_the_default_variant(tmp_path):
    ctx, cache = Ctx(), autotune.Cache(str(tmp_path / "t.json"))
    e = autotune.tune(ctx, 0, Parts(4096), cache=cache, timer=timer)
    assert {t[0] for t in ctx.timed} == {0} and {t[2] for t in ctx.timed} == {0}
    assert len(ctx.timed) == len(autotune.DEFAULT_CHUNKS)
    assert (e["corr_variant"], e["chunk_particles"], e["run_tiles"], e["variant_timed"]) == (0, 128, 0, False)
    assert ctx.tuning == (0, 128, 0) and not ctx.recording
    cache.save()
    other = Ctx()
    assert autotune.apply(other, 0, autotune.Cache(str(tmp_path / "t.json")))
    assert other.tuning == (0, 128, 0)


def test_a_sample_of_few_pairs_times_the_variants(tmp_path):
    ctx = Ctx()
    e = autotune.tune(ctx, 0, Parts(40), timer=timer)
    assert {t[0] for t in ctx.timed} == {0, 1, 2} and {t[2] for t in ctx.timed} == {0}
    assert (e["corr_variant"], e["variant_timed"]) == (2, True)
    cache = autotune.Cache(str(tmp_path / "t.json"))
    cache.put(autotune.refset_key(ctx, 0), e)
    other = Ctx()
    assert autotune.apply(other, 0, cache) and other.tuning[0] == 2


@pytest.mark.parametrize("timed", [None, False])
def test_a_variant_that_was_not_timed_is_not_applied(tmp_path, timed):
    path = tmp_path / "old.json"
    entry = dict(corr_variant=2, chunk_particles=128, run_tiles=4, ms=1.0)
    if timed is not None:
        entry["variant_timed"] = timed
    path.write_text(json.dumps({"L76-R35-K128-T3-fp32": entry}))
    ctx = Ctx()
    assert autotune.apply(ctx, 0, autotune.Cache(str(path)))
    assert ctx.tuning[:2] == (0, 128)
