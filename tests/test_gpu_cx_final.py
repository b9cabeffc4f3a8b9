"""The template model's evaluations after the loop (catalogs of 2^14 sources or
more), counted and timed with the SNR family.  One loud source in every tile
resolves in body 0, so body 1 refilters every tile and settles: every
candidate is evaluated in body 0, and every one left once more, in body 1 or,
where the bound put it off, after the loop.  Whole numbers: exact.  rho^2
against the oracle: 1e-9 as in the model's other tests (the data's unit is
2^-50 of the loudest source, 1e6 times the noise)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2602_18560_amd import gbsub as G
from paper_2602_18560_amd.inputs import YEAR_S, Catalog, RunConfig, template_phases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 14) - 1, 1 << 14])
def test_every_evaluation_is_counted(n):
    T, k0, B = YEAR_S, 100_000, 19 * 2048
    run = RunConfig(t_obs_s=T, f_min_hz=k0 / T, f_max_hz=(k0 + B - 1) / T, window_bins=31, kappa=0.0)
    rng = np.random.default_rng(7)
    S0 = O.sinstr_table(O.make_config(run))
    loud = np.arange(1024, B - 500, 2048)
    k = np.concatenate([loud, rng.integers(100, B - 100, n - loud.size)])
    P = S0[k] * np.where(np.arange(n) < loud.size, 1e6, rng.uniform(0.01, 0.05, n))
    cat = Catalog(A=np.sqrt(2 * P / T).astype(np.float32), f=((k0 + k + 0.3) / T).astype(np.float32),
                  fdot=np.zeros(n, np.float32), id=np.arange(n, dtype=np.uint32))
    pa, pe = template_phases(n, 3)
    ctx = G.Context(G.config_from_run(run))
    print(f"[cx final] n {n}", flush=True)
    try:
        ctx.set_profiling(True)
        cx = G.CxRun(ctx)
        s = cx.run(G.DeviceCxCatalog.from_host(cat, pa, pe))
        st = ctx.kernel_stats()["snr"]
        ids, it, r2 = cx.candidates()
    finally:
        ctx.close()
    ref = O.cx_run(cat, pa, pe, O.make_config(run))
    assert ref.n_near == 0 and ref.n_iter == s.n_iter == 2
    assert np.array_equal(it, ref.iter_of) and s.n_candidates == n and s.n_resolved == loud.size
    assert st["units"] == n + (n - loud.size)
    assert st["launches"] == 2 + (n >= 1 << 14)
    assert np.max(np.abs(r2 / ref.rho2_last - 1)) <= 1e-9
