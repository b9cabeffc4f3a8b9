"""Gamma shapes far below one, where y is small beyond the z at which the
generator's nodes change from the series of P to the continued fraction of Q.

Tolerance: both sides round the same fp64 value to fp32; their fp64 errors stay
below 1e-9 for these shapes and draws (the rounding of 1 - P, about 2^-52 ln(1/a)
/ a relative to the tail), so they differ by at most one fp32 step (2^-23
relative); two steps are allowed."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2602_18560_amd import gbsub as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha_g", [1e-4, 1e-3, 5e-3, 7e-3, 0.02, 0.3])
def test_small_gamma_shapes(alpha_g):
    n = 2000
    lam = dict(alpha_pl=-2.9, alpha_g=alpha_g, beta_g=1.0, mu_g=-21.0, mu=-22.0, sigma=0.2, rho=0.5)
    dc = G.generate(G.population(**lam), 5, n)
    got = [x.cpu().numpy().astype(np.float64) for x in (dc.A, dc.f, dc.fdot)]
    want = [x.astype(np.float64) for x in O.pop_draw(O.population(**lam), 5, n)[:3]]
    for g, w, what in zip(got, want, ("A", "f", "fdot")):
        rel = np.max(np.abs(g - w) / w)
        print(f"alpha_g {alpha_g} {what}: max rel {rel:.2e}", flush=True)
        assert rel <= 2.0 ** -22, (what, rel)
