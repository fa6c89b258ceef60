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
