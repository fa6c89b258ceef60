"""Sources as flat as the domain admits (q in (0, 1]), aligned with the mass or nearly
so: their quadratic form keeps its accuracy in the frame of the mass ellipse."""
import numpy as np
import pytest

from gpu_cases import TOL_FP32, oracle_data, oracle_loglike, rel_err, say
from paper_2503_08586_amd import synth

pytestmark = pytest.mark.gpu
S = synth.SLOT


@pytest.mark.parametrize("mass", [0, 1])
@pytest.mark.parametrize("q", [1e-10, 1e-9, 1e-6, 1e-3, 0.05])
def test_flat_source_aligned_with_the_mass(q, mass):
    from paper_2503_08586_amd import binding
    say("case: source q %g, mass model %d" % (q, mass))
    spec = synth.config1(nprop=1)[0]
    oracle_data(spec)
    rng = np.random.default_rng(4)
    P = np.repeat(spec.truth[None], 24, axis=0)
    P[:, S["phi_m"]] = rng.uniform(0.1, 3.0, 24)
    P[:, S["phi_s"]] = P[:, S["phi_m"]] + np.where(np.arange(24) % 2, 0.0, q * rng.normal(size=24))
    P[:, S["q_s"]] = q
    P[:, 19] = rng.uniform(1.8, 2.2, 24) if mass else 0.0
    with binding.LensContext(0) as c:
        got = c.loglike(c.load(spec, mass_model=mass), P)
    ref, chi2, C = oracle_loglike(spec, P)
    e = rel_err(got, ref, chi2, C)
    say("max err %.2e" % e.max())
    assert np.all(np.isfinite(got)) and np.all(e <= TOL_FP32)
