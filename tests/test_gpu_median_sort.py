"""The median's sort and selection at their edges: unions that end on and off
a 64-position word, one window word, windows over buckets of 32 and of 64
ranks, empty bins among occupied ones, and values that share sort keys in
long runs (an outlier stretches the key range), in tile mode and in split
mode.

Nothing is resolved (the threshold is out of reach), so S = C median + S_instr
of the catalog's own spectrum: bit for bit the definition on the run's X (the
selection does no arithmetic), and X within the fixed-point bound of the sum
of the powers (2^-62 of the largest, 1e-12 of a bin's, per source)."""
import numpy as np
import pytest

from paper_2602_18560_amd import gbsub as G
from paper_2602_18560_amd.inputs import YEAR_S, Catalog

pytestmark = pytest.mark.gpu

GRIDS = [
    # bins, window, split budget (1: never, 65535: every body)
    (5, 7, 0), (64, 1, 0), (64, 63, 65535), (2048, 65, 1), (2111, 1001, 1), (2112, 1025, 1), (3072, 1023, 65535),
    (5000, 513, 65535), (4097, 2801, 1), (9000, 1001, 1),
]


@pytest.mark.parametrize("values", ["outlier", "gaps", "plateaus"])
@pytest.mark.parametrize("B,W,split", GRIDS)
def test_median_selection(B, W, split, values):
    rng = np.random.default_rng(B + W)
    T, k0 = YEAR_S, 40_000
    bins = np.arange(B)
    A = 3e-22 * (1.0 + 0.01 * rng.random(B))         # powers within 2 %
    if values == "outlier":
        A[rng.integers(0, B)] *= 1e3                   # 2^20 in power: 5e-4 of a key apart
    elif values == "gaps":
        keep = rng.random(B) < 0.4
        keep[0] = True
        bins, A = bins[keep], A[keep]
    else:
        A = 3e-22 * rng.choice([1.0, 1.0 + 2e-6, 3.0, 1e3], B, p=[0.4, 0.4, 0.19, 0.01])
    n = len(A)
    cat = Catalog(A=A.astype(np.float32), f=((k0 + bins) / T).astype(np.float64).astype(np.float32),
                  fdot=np.zeros(n, np.float32), id=np.arange(n, dtype=np.uint32))
    kw = dict(t_obs_s=T, f_min_hz=k0 / T, f_max_hz=(k0 + B - 1) / T, window_bins=W, snr_threshold=1e9, kappa=0.0)
    ctx = G.Context(G.default_config(**kw, split_blocks=split))
    try:
        s = ctx.run(G.DeviceCatalog.from_host(cat))
        S, X, sx = (ctx.spectrum(k) for k in (G.SPEC_SN, G.SPEC_X_RESIDUAL, G.SPEC_S_INSTR))
    finally:
        ctx.close()
    assert s.n_resolved == 0
    # the definition, on the run's own X
    C = 729.0 / 512.0
    if B < W:
        want = np.full(B, np.sort(X)[(B + 1) // 2 - 1])
    else:
        h = (W - 1) // 2
        a = np.clip(np.arange(B) - h, 0, B - W)
        want = np.array([np.partition(X[i:i + W], h)[h] for i in a])
    np.testing.assert_array_equal(S, C * want + sx)
    # and that X is the catalog's
    P = np.zeros(B)
    kk = np.floor(cat.f.astype(np.float64) * T + 0.5).astype(int) - k0
    inside = (kk >= 0) & (kk < B)
    np.add.at(P, kk[inside], cat.A[inside].astype(np.float64) ** 2 * T / 2)
    np.testing.assert_allclose(X, P, rtol=1e-10, atol=0)
