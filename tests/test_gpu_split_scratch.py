"""The scratch of the split launches over a context's life: taken, given back
when the HBM budget runs out, taken again at another size.  Results never change
with it."""
import numpy as np
import pytest

from gpu_cases import say
from test_gpu_split import GEOMS, _spec

pytestmark = pytest.mark.gpu


def test_multi_call_after_its_scratch_was_given_back():
    """A multi-lens call shape is captured as a graph; between two calls of the
    shape its split scratch is given back, then re-allocated smaller."""
    from paper_2503_08586_amd import binding
    say("case: multi-lens plan, split scratch given back and taken again")
    sp = _spec(GEOMS[2], 60, 11, 0)
    with binding.LensContext(0, hbm_budget_bytes=24 << 20) as c:
        lids = [c.load(sp), c.load(sp)]
        props = [sp.proposals, sp.proposals[:33]]
        ref = np.concatenate(c.loglike_multi(lids, props))
        assert np.array_equal(np.concatenate(c.loglike_multi(lids, props)), ref)
        more, per = [], c.info(lids[0])["device_bytes"]
        try:
            while True:
                more.append(c.load(sp))
        except binding.LensError as e:
            assert e.status == binding.LENS_ENOMEM
        # the budget is full: no split scratch, then a little, then much of it
        for room in (0, 5 << 20, 12 << 20):
            while more and (24 << 20) - c.stats()["hbm_used_bytes"] < room + per:
                c.unload(more.pop())
            for _ in range(2):
                assert np.array_equal(np.concatenate(c.loglike_multi(lids, props)), ref)


@pytest.mark.parametrize("kind", [dict(amplitudes=1), dict(precision=0, mass_model=1)], ids=["solved", "power_law"])
def test_chunks_of_one_call(kind):
    """A call whose images do not fit a tight budget's scratch, in chunks that fill the
    chip, the last one short; and the same proposals as one chunk each."""
    from paper_2503_08586_amd import binding
    say("case: one call in several split chunks, %s" % kind)
    n = 5003
    sp = _spec((70, 65, 4, 13, "disc"), n, 21, 0)
    with binding.LensContext(0) as c, binding.LensContext(0, hbm_budget_bytes=400 << 20) as t:
        whole, tight = c.load(sp, **kind), t.load(sp, **kind)
        used = [x.stats()["hbm_used_bytes"] for x in (c, t)]
        ref, got = c.loglike(whole, sp.proposals), t.loglike(tight, sp.proposals)
        held = [x.stats()["hbm_used_bytes"] - u for x, u in zip((c, t), used)]
        assert held[0] > 120 << 20 and 60 << 20 < held[1] < 110 << 20   # several chunks there
        assert np.array_equal(got, ref)
        parts = [c.loglike(whole, sp.proposals[a:a + 700]) for a in range(0, n, 700)]
        assert np.array_equal(np.concatenate(parts), ref)


def test_split_launches_take_their_scratch():
    """The contexts that the bit comparisons hold apart do differ: one with room has
    split scratch after its first call, one without has none."""
    from paper_2503_08586_amd import binding
    say("case: who holds split scratch")
    sp = _spec(GEOMS[1], 41, 5, 0)
    grew = []
    for budget in (0, 4 << 20, 12 << 20):
        with binding.LensContext(0, hbm_budget_bytes=budget) as c:
            lid = c.load(sp)
            pd, u = sp.proposals, c.stats()["hbm_used_bytes"]
            c.loglike(lid, pd)
            grew.append(c.stats()["hbm_used_bytes"] - u)
    assert grew[0] >= 4 << 20 and grew[1] < 1 << 20 and grew[2] >= 2 << 20


def test_scratch_grows_with_the_calls():
    from paper_2503_08586_amd import binding
    say("case: split scratch grown between calls on one stream")
    sp = _spec(GEOMS[2], 4000, 9, 0)
    with binding.LensContext(0) as c:
        lid = c.load(sp, mass_model=1)
        ref = c.loglike(lid, sp.proposals)
    with binding.LensContext(0) as c:
        lid = c.load(sp, mass_model=1)
        for n in (1, 300, 4000, 7, 2500):
            assert np.array_equal(c.loglike(lid, sp.proposals[:n]), ref[:n])
