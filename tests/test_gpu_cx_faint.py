"""The injection's moment path (k_cx_faint): catalogs of 2^16 sources and
more, whose faint sources are summed per centre bin before one transform.
The bar is the template model's own (identical candidates, resolved set and
bodies; rho^2, S, X and h within 1e-9), against the oracle, which adds one
term-by-term template per source."""
import math

import numpy as np
import pytest

from paper_2602_18560_amd.inputs import RunConfig, YEAR_S, template_phases
from test_gpu_cx import assert_cx_parity, cat_of

pytestmark = pytest.mark.gpu

N_MIN = 1 << 16          # the path's smallest catalog
T = YEAR_S


def _grid(n_bins, W, f_min=5e-4):
    k0 = math.floor(f_min * T + 0.5)
    return RunConfig(t_obs_s=T, f_min_hz=k0 / T, f_max_hz=(k0 + n_bins - 1) / T, window_bins=W), k0


def _centres(case, rng):
    """Centre bins (on the grid of 3000) of the case's faint sources."""
    if case == "one centre":            # shared by the block's waves, a coarser unit of the sums
        return np.full(N_MIN, 1500)
    if case == "few per centre":        # 1 .. 40 sources a centre: one template each, or moments
        c = np.repeat(np.arange(3000), 1 + np.arange(3000) % 40)
        return np.r_[c, rng.integers(0, 3000, N_MIN - c.size)] if c.size < N_MIN else c
    if case == "edges":                 # binning-tile and grid edges, and just outside the grid
        return rng.choice([-64, -63, -1, 0, 1, 1022, 1023, 1024, 2047, 2048, 2998, 2999, 3000, 3062, 3063], N_MIN)
    return rng.integers(0, 3000, N_MIN)


@pytest.mark.parametrize("case", ["one centre", "few per centre", "edges", "chirps and phases"])
def test_moment_path(case):
    run, k0 = _grid(3000, 101)
    rng = np.random.default_rng(41)
    c = _centres(case, rng)
    n = c.size
    d = rng.uniform(-1e-3, 1e-3, n)
    if case == "chirps and phases":     # both sides of the path's largest |fdot| T^2 (1/pi)
        d = rng.uniform(-0.45, 0.45, n)
    f = (k0 + c + rng.uniform(-0.49, 0.49, n) - d / 2) / T
    A = 10 ** rng.uniform(-26, -24, n)
    A[:40] = 10 ** rng.uniform(-22.5, -21, 40)          # a few that resolve
    cat = cat_of(A, f, d / T ** 2)
    pa, pe = template_phases(n, 41)
    if case == "chirps and phases":     # phases of many turns as well
        pa[::3] *= np.float32(1e5)
        pe[::5] -= np.float32(300.0)
    assert_cx_parity(cat, pa, pe, run, case)


def test_smallest_catalog_without_the_path():
    run, k0 = _grid(3000, 101)
    rng = np.random.default_rng(42)
    n = N_MIN - 1
    cat = cat_of(10 ** rng.uniform(-26, -23, n), (k0 + rng.uniform(0, 2999, n)) / T, np.zeros(n))
    pa, pe = template_phases(n, 42)
    assert_cx_parity(cat, pa, pe, run, "2^16 - 1 sources")


@pytest.mark.parametrize("n_bins,n", [(24000, N_MIN), (24000, 18 * 4096 + 1), (40000, 17 * 4096 + 1)],
                         ids=["short rows", "matrix larger than the spectra", "one source in the last row"])
def test_grouping_rows(n_bins, n):
    """The faint sources' grouping in rows of 4096 sources (its matrix lies in
    the spectra) or of 16384 (it does not fit there)."""
    run, k0 = _grid(n_bins, 101)
    rng = np.random.default_rng(43)
    A = 10 ** rng.uniform(-26, -24, n)
    A[::2000] = 10 ** rng.uniform(-22.5, -21, A[::2000].size)
    cat = cat_of(A, (k0 + rng.uniform(0, n_bins - 1, n)) / T, np.zeros(n))
    pa, pe = template_phases(n, 43)
    assert_cx_parity(cat, pa, pe, run, f"{n_bins} bins {n} sources")
