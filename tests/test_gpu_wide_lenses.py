"""The widest masks that a workgroup's LDS holds, per convolution mode: the ring of
k binned rows may take 159,152 bytes.  Such lenses load, and their likelihood is
the oracle's."""
import numpy as np
import pytest

import oracle
from gpu_cases import TOL_BF16, TOL_FP32, oracle_loglike, rel_err, say
from paper_2503_08586_amd import synth

pytestmark = pytest.mark.gpu
RING = 159152

# precision or solved light model, PSF side
KINDS = [(dict(precision=0), 63), (dict(precision=1), 63), (dict(precision=1), 11), (dict(precision=2), 63),
         (dict(precision=3), 63), (dict(amplitudes=1), 63), (dict(amplitudes=1, light_model=1), 63),
         (dict(amplitudes=1, light_model=2), 63), (dict(amplitudes=1, light_model=3), 63)]


def widest(kind, k):
    """Columns of the widest mask at one output row per strip."""
    up = lambda v, n: -(-v // n) * n
    prec = kind.get("precision", 0)
    if prec == 0:
        elem, step, halo = 4 * {0: 2, 1: 1, 2: 1, 3: 4}[kind.get("light_model", 0)] if "amplitudes" in kind else 4, 4, 4 * ((k + 6) // 4)
    else:
        elem, step, halo = {1: 4, 2: 2, 3: 6}[prec], 16, up(k + 15, 32 if prec == 1 else 8)
    return min(4096, (RING // (k * elem) - halo) // step * step)


def _check(kind, k, mass):
    from paper_2503_08586_amd import binding
    nx = widest(kind, k)
    say("case: %d masked columns, PSF side %d, %s, mass %d" % (nx, k, kind, mass))
    ny, s, dpix, light = 3, 1, 8.0 / nx, kind.get("light_model", 0)
    rng = np.random.default_rng(nx)
    psf = synth.moffat_psf(k, 0.15, 3.0, 0.05)
    P = synth.draw_params(rng, 3)
    P[:, 19] = rng.uniform(1.6, 2.4, 3) if mass else 0.0
    if light == 3:
        P = synth.double_component_params(rng, P)
    orc = oracle.default()
    truth = P[0].copy()
    img = orc.model_image(ny, nx, dpix, s, psf, truth, stage=1) if light != 3 else 0.05 * rng.random((ny, nx))
    sigma = np.full((ny, nx), 0.01)
    sp = synth.LensSpec(ny, nx, dpix, s, psf, sigma, np.ones((ny, nx), np.uint8), truth, P, sigma,
                        img + 0.01 * rng.normal(size=(ny, nx)))
    with binding.LensContext(0) as c:
        lid = c.load(sp, psf_tail=-1.0, mass_model=mass, **kind)
        assert c.info(lid)["psf_used"] == k
        got = c.loglike(lid, P)
        if mass:   # the fused and the multi-lens kernels have as little room for the tables
            with binding.LensContext(0, hbm_budget_bytes=4 << 20) as f:
                fid = f.load(sp, psf_tail=-1.0, mass_model=mass, **kind)
                assert np.array_equal(f.loglike(fid, P), got)
                assert np.array_equal(np.concatenate(f.loglike_multi([fid, fid], [P, P])), np.tile(got, 2))
            assert np.array_equal(np.concatenate(c.loglike_multi([lid, lid], [P, P])), np.tile(got, 2))
    if "amplitudes" in kind:
        ref, chi2 = orc.loglike_light(sp.geom, sp.psf, sp.data, sp.sigma, sp.mask, P, light, (1.0,) * 4,
                                      return_chi2=True)[:2]
        C = orc.loglike_norm(sp.sigma, sp.mask)
    else:
        ref, chi2, C = oracle_loglike(sp, P)
    e = rel_err(got, ref, chi2, C)
    say("max err %.2e" % e.max())
    assert np.all(e <= (TOL_BF16 if kind.get("precision") == 2 else TOL_FP32))


@pytest.mark.parametrize("kind,k", KINDS, ids=lambda v: str(v))
def test_widest_isothermal(kind, k):
    _check(kind, k, 0)


@pytest.mark.parametrize("kind,k", KINDS, ids=lambda v: str(v))
def test_widest_power_law(kind, k):
    """No room for the deflection tables beside such a ring: the series instead."""
    _check(kind, k, 1)
