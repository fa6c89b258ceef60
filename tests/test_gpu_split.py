"""The split launches (lens_split.hip: one call cut over proposals, pixels and
strips) against the fused kernels (one workgroup per proposal): the same bits,
for every convolution, light model and mass, on images whose strips, pixel
waves and PSF windows have remainders.  A context whose HBM budget leaves no
room for the split launches' scratch runs the fused kernels; one with little
room runs the split launches in several chunks."""
import numpy as np
import pytest

from gpu_cases import say
from paper_2503_08586_amd import synth

pytestmark = pytest.mark.gpu

KINDS = [dict(precision=0), dict(precision=1), dict(precision=2), dict(precision=3), dict(precision=0, mass_model=1),
         dict(precision=1, mass_model=1), dict(amplitudes=1), dict(amplitudes=1, light_model=1),
         dict(amplitudes=1, light_model=2), dict(amplitudes=1, light_model=3),
         dict(amplitudes=1, light_model=3, mass_model=1)]
# ny, nx, s, k, mask
GEOMS = [(1, 1, 1, 1, "all"), (17, 33, 4, 11, "all"), (70, 65, 2, 13, "disc"), (45, 90, 3, 41, "ring"),
         (33, 20, 8, 63, "all"), (40, 40, 2, 5, "sparse"), (24, 31, 2, 9, "empty"),
         (53, 230, 1, 31, "all")]


@pytest.fixture(scope="module")
def ctxs():
    from paper_2503_08586_amd import binding
    # no split scratch below 4 MB of free budget; 2-3 MB of it at 12 MB
    cs = [binding.LensContext(0), binding.LensContext(0, hbm_budget_bytes=4 << 20),
          binding.LensContext(0, hbm_budget_bytes=12 << 20)]
    yield cs
    for c in cs:
        c.close()


def _spec(geom, n, seed, light):
    ny, nx, s, k, kind = geom
    rng = np.random.default_rng(seed)
    yy, xx = np.mgrid[0:ny, 0:nx]
    r = np.hypot(yy - 0.5 * (ny - 1), xx - 0.5 * (nx - 1))
    mask = {"all": r >= 0, "disc": r < 0.45 * min(ny, nx), "ring": (r > 8) & (r < 20),
            "sparse": rng.random((ny, nx)) < 0.03, "empty": r < 0}[kind].astype(np.uint8)
    psf = synth.moffat_psf(k, 0.15, 3.0, 0.07)
    psf = psf * rng.uniform(0.5, 1.5, psf.shape)
    p = synth.draw_params(rng, n)
    p[:, 19] = rng.uniform(1.5, 2.5, n)
    p[n // 2, [1, 10, 15]] = -0.3             # outside the domain of every light model
    p[n // 3, 1] = 0.2                        # the direct deflection
    if light == 3:
        p = synth.double_component_params(rng, p)
    sigma = rng.uniform(0.005, 0.02, (ny, nx))
    return synth.LensSpec(ny, nx, 0.07, s, psf, sigma, mask, p[0], p, sigma, 0.1 * rng.random((ny, nx)))


@pytest.mark.parametrize("geom", GEOMS, ids=lambda g: "%dx%d-s%d-k%d-%s" % g)
@pytest.mark.parametrize("kind", KINDS, ids=lambda k: "-".join("%s%d" % (a[:4], v) for a, v in k.items()))
def test_split_equals_fused(ctxs, kind, geom):
    import torch
    from paper_2503_08586_amd import binding
    say("case: split against fused, %s, %s" % (kind, geom))
    n = 41
    sp = _spec(geom, n, 7 + geom[0], kind.get("light_model", 0))
    lids = [c.load(sp, **kind) for c in ctxs]
    split, fused, chunks = (c.loglike_amps(lid, sp.proposals) for c, lid in zip(ctxs, lids))
    assert np.isneginf(fused[0][n // 2]) and np.isfinite(np.delete(fused[0], n // 2)).all()
    for a, b, c in zip(split, fused, chunks):
        assert np.array_equal(a, b, equal_nan=True)
        assert np.array_equal(c, b, equal_nan=True)
    # the smallest call, and the allocation-free one
    one = ctxs[0].loglike(lids[0], sp.proposals[3:4])
    assert one[0] == fused[0][3]
    pd = torch.from_numpy(sp.proposals).cuda()
    od = torch.zeros(n, dtype=torch.float64, device="cuda")
    binding.lens_loglike_batch_device_noalloc(ctxs[0].ctx, lids[0], pd, od)
    assert np.array_equal(od.cpu().numpy(), fused[0])
    for c, lid in zip(ctxs, lids):
        c.unload(lid)


def test_split_many_lenses(ctxs):
    """Several lenses of each kind in one multi-lens call, some with nothing to do."""
    say("case: split against persistent, many lenses")
    got = []
    for c in (ctxs[0], ctxs[1], ctxs[2]):
        lids, props = [], []
        for i, kind in enumerate(KINDS + KINDS[:4]):
            sp = _spec(GEOMS[1:][i % 6], 1 + 13 * (i % 4) if i != 5 else 60, 100 + i, kind.get("light_model", 0))
            lids.append(c.load(sp, **kind))
            props.append(sp.proposals if i != 7 else sp.proposals[:0])
        a = c.loglike_multi(lids, props)
        b = c.loglike_multi(lids, props)      # the captured graph again
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
        got.append(np.concatenate(a))
        for lid in lids:
            c.unload(lid)
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[2], got[1])


def test_scratch_given_back():
    """Split scratch never stands in the way of what the HBM budget used to admit."""
    from paper_2503_08586_amd import binding
    say("case: split scratch given back to the budget")
    sp = _spec(GEOMS[2], 8, 3, 0)
    with binding.LensContext(0, hbm_budget_bytes=16 << 20) as c:
        first = c.load(sp)
        ref = c.loglike(first, sp.proposals)
        used = c.stats()["hbm_used_bytes"]
        assert used > 2 << 20                 # the scratch is held
        per = c.info(first)["device_bytes"]
        lids = [c.load(sp) for _ in range(((16 << 20) - (1 << 20)) // per - 2)]
        assert c.stats()["hbm_used_bytes"] <= 16 << 20
        assert np.array_equal(c.loglike(lids[-1], sp.proposals), ref)


def test_captured_call_outlives_the_scratch():
    """A device-buffer call recorded into a caller's graph does not depend on split
    scratch, which the HBM budget may take back before the graph is replayed."""
    import torch
    from paper_2503_08586_amd import binding
    say("case: captured call, split scratch taken back")
    sp = _spec(GEOMS[2], 8, 3, 0)
    with binding.LensContext(0, hbm_budget_bytes=16 << 20) as c:
        first = c.load(sp)
        ref = c.loglike(first, sp.proposals)
        pd = torch.from_numpy(sp.proposals).cuda()
        od = torch.zeros(8, dtype=torch.float64, device="cuda")
        st = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            c.loglike_device(first, pd, od)           # this stream's scratch
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            c.loglike_device(first, pd, od)
        per = c.info(first)["device_bytes"]
        for _ in range(((16 << 20) - (3 << 20)) // per - 2):
            c.load(sp)
        for _ in range(3):
            od.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(od.cpu().numpy(), ref)
