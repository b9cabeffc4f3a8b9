"""Bodies of two and of three launches on catalogs whose dirty tiles fit the
split budget in one body and outgrow it in the next, with several parts a tile
and a short last tile.

Two tiles of 2048 bins (the second has 700), window 101, 4 parts a tile.  A
loud source A near the boundary masks B, which masks C; A's window reach ends
inside the first tile, B's crosses into the second.  A faint source D stays
(power model: over 2200 bins, so its rho^2 adds the part sums of 1/S).  Budget
4 (one tile): bodies 0 and 1 see 2 dirty tiles and 1, body 2 (two launches, by
the count of body 1) 2 tiles in 8 parts on 4 blocks, and body 3 takes three
launches again.  Budget 1: never two launches; 65535: always.

Tolerances: S of the running median does not depend on the form (exact); the
running mean is a sum of at most 2200 terms of one sign, so 2200 x 2^-52 =
5e-13 relative.  rho^2 of the power model is made of differences of prefix sums
over the parts its track touches: 600 terms and roundings of 2^-52 each,
relative to those parts' whole sum of 1/S, which is 4e4 times the track's
own under the loud source A; the test computes that bound from the oracle's S.
The template model's data are rounded to 2^-50 of the loudest source, whose
power is 1e9 times the noise: 1e-9 as in the model's other tests."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2602_18560_amd import gbsub as G
from paper_2602_18560_amd.inputs import YEAR_S, Catalog, RunConfig

pytestmark = pytest.mark.gpu

T, K0, B, CENTRE = YEAR_S, 100_000, 2748, 1928


def build(model, est):
    run = RunConfig(t_obs_s=T, f_min_hz=K0 / T, f_max_hz=(K0 + B - 1) / T, window_bins=101, estimator=est)
    s0 = O.sinstr_table(O.make_config(run))[CENTRE]
    if model == "cx":
        k = K0 + CENTRE + np.array([0.5, 40.5, 20.5, -899.9])
        P, f, fd = s0 * np.array([1e9, 4e3, 15.0, 0.5]), k / T, np.zeros(4)
    else:
        lo = CENTRE + np.array([-64, 20, 45, -1500])
        n = np.array([128, 60, 20, 2200])
        P, fd = n * s0 * np.array([1e4, 0.7, 0.75, 1e-3]), (n - 0.5) / T ** 2
        f = (K0 + lo + (n - 1) // 2) / T - fd * T / 2
    cat = Catalog(A=np.sqrt(2 * P / T).astype(np.float32), f=f.astype(np.float32), fdot=fd.astype(np.float32),
                  id=np.arange(4, dtype=np.uint32))
    return run, cat


@pytest.mark.parametrize("est", [0, 1])
@pytest.mark.parametrize("model", ["power", "cx"])
def test_form_follows_the_count_of_the_body_before(model, est):
    run, cat = build(model, est)
    ph = np.zeros(4, np.float32)
    cfg = O.make_config(run)
    if model == "cx":
        r = O.cx_run(cat, ph, ph, cfg)
        want_r2, tol_r2, S_ref, tol = r.rho2_last, 1e-9, r.S_final, 1e-9
    else:
        r = O.run(cat, cfg, trace=True, trace_fields=("S", "cand", "rho2"))
        want_r2, tol_r2, S_ref, tol = np.full(4, np.nan), np.full(4, np.nan), r.S_final, 5e-13
        for t in r.trace:
            for i, x in zip(t["cand"], t["rho2"]):
                if x < 0:
                    continue
                tr = O.track(cfg, float(cat.A[i]), float(cat.f[i]), float(cat.fdot[i]))
                lo, hi = tr["glo"], tr["ghi"] + 1
                parts = np.sum(1 / t["S"][lo // 512 * 512:(hi + 511) // 512 * 512])
                want_r2[i] = x
                tol_r2[i] = tol + 600 * 2.0 ** -52 * parts / np.sum(1 / t["S"][lo:hi])
    assert r.iter_of.tolist() == [0, 1, 2, -1] and r.n_iter == 4 and r.min_rel_margin > 1e-3
    runs = {}
    for budget, launches in ((1, None), (4, 3 if model == "cx" else 5), (65535, 0)):
        for prof in (False, True, False):
            ctx = G.Context(G.config_from_run(run, split_blocks=budget))
            print(f"[body form] {model} est {est} budget {budget} profiling {prof}", flush=True)
            try:
                ctx.set_profiling(prof)
                if model == "cx":
                    res = G.CxRun(ctx)
                    s = res.run(G.DeviceCxCatalog.from_host(cat, ph, ph))
                    S = np.stack([res.spectrum(ch, G.SPEC_SN) for ch in (0, 1)])
                else:
                    res = ctx
                    s = ctx.run(G.DeviceCatalog.from_host(cat))
                    S = ctx.spectrum(G.SPEC_SN)
                ids, it, r2 = res.candidates()
                if prof and launches is not None:
                    assert ctx.kernel_stats()["xupdate"]["launches"] == launches
            finally:
                ctx.close()
            assert s.n_iter == 4 and ids.tolist() == [0, 1, 2, 3] and it.tolist() == [0, 1, 2, -1]
            assert np.all(np.abs(r2 / want_r2 - 1) <= tol_r2)
            assert np.max(np.abs(S / S_ref - 1)) <= tol
            if budget in runs:                     # whatever the host's timing: the same bits
                np.testing.assert_array_equal(S, runs[budget][0])
                np.testing.assert_array_equal(r2, runs[budget][1])
            runs[budget] = S, r2
    if est == 0:
        for budget in (4, 65535):
            np.testing.assert_array_equal(runs[budget][0], runs[1][0])
