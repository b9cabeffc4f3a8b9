"""Contexts that use one workspace in turn: each finds grid tables of its own,
whatever ran there in between (a context of another tile size, a batch slot, the
template model).  Whole results equal those of a context with a workspace to
itself, bit for bit: the same kernels on the same inputs, exact sums."""
import numpy as np
import pytest

from paper_2602_18560_amd import gbsub as G
from paper_2602_18560_amd.inputs import YEAR_S, Population, RunConfig, draw_catalog, template_phases

pytestmark = pytest.mark.gpu


def outputs(ctx):
    ids, it, r2 = ctx.candidates()
    return ctx.spectrum(G.SPEC_SN), ctx.spectrum(G.SPEC_S_INSTR), ids, it, r2


def batch_run(ctx, dc, ws):
    b = G.Batch(1)
    try:
        k = b.admit(ctx, dc, ws=ws)
        while b.poll()[1]:
            b.step(4)
        assert b.retire(k)[0] == G.OK
    finally:
        b.close()


@pytest.mark.parametrize("between", ["run", "batch", "templates"])
def test_one_workspace_in_turn(between):
    import torch
    cat = draw_catalog(Population(n=20000, seed=1, f_lo=1e-3, f_hi=1.6e-3))
    # tracks of some hundred to some thousand bins: their candidate test reads the prefix tables
    cat.fdot[:] = (np.random.default_rng(4).uniform(100, 3000, cat.n) / YEAR_S ** 2).astype(np.float32)
    run = RunConfig(t_obs_s=YEAR_S, f_min_hz=1e-3, f_max_hz=1.6e-3, window_bins=101)
    pa, pe = template_phases(cat.n, 1)
    dc = G.DeviceCatalog.from_host(cat)
    own = G.Context(G.config_from_run(run))
    a = G.Context(G.config_from_run(run))
    b = G.Context(G.config_from_run(run, tile_bins=256))
    try:
        own.run(dc)
        want = outputs(own)
        assert 0 < want[2].size < cat.n
        cx = G.CxRun(a)
        ws = torch.zeros(max(a.workspace_size(cat.n), b.workspace_size(cat.n), cx.workspace_size(cat.n)) + 512,
                         dtype=torch.uint8, device="cuda")
        for turn in range(3):
            print(f"[shared workspace] {between} turn {turn}", flush=True)
            a.run(dc, ws=ws)
            got = outputs(a)
            for g, w in zip(got, want):
                np.testing.assert_array_equal(g, w)
            if between == "run":
                b.run(dc, ws=ws)
            elif between == "batch":
                batch_run(b, dc, ws)
            else:
                cx.run(G.DeviceCxCatalog.from_host(cat, pa, pe), ws=ws)
    finally:
        for c in (own, a, b):
            c.close()
