"""The two-launch bodies' block-to-part map where a body has more dirty parts
than the launch has blocks.  Running mean over 2801 bins (tiles of 256): a loud
source masks two fainter ones 1300 bins away, each of which masks a still
fainter one 1300 bins further out, so the bodies subtract 1, 2 and 2 sources
and dirty 12, 22 and 24 tiles; a split budget of 14 starts the two-launch bodies at
the first and is outgrown by the next.  The work of a part does not depend on
the launch: everything equals the run that never splits, bit for bit."""
import numpy as np
import pytest

from paper_2602_18560_amd import gbsub as G
from paper_2602_18560_amd.inputs import YEAR_S, Catalog

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["power", "cx"])
def test_more_entries_than_blocks(model):
    T, k0, B, mid = YEAR_S, 100_000, 20_000, 10_000
    off = np.array([0, -1300, 1300, -2600, 2600])
    P = 1e-33 * np.array([1.0, 3e-3, 3e-3, 9e-6, 9e-6])
    cat = Catalog(A=np.sqrt(2 * P / T).astype(np.float32), f=((k0 + mid + off) / T).astype(np.float32),
                  fdot=np.zeros(5, np.float32), id=np.arange(5, dtype=np.uint32))
    ph = np.zeros(5, np.float32)
    out = []
    for budget in (1, 14, 65535):
        ctx = G.Context(G.default_config(t_obs_s=T, f_min_hz=k0 / T, f_max_hz=(k0 + B - 1) / T, window_bins=2801,
                                         estimator=1, split_blocks=budget))
        print(f"[next entries] {model} budget {budget}", flush=True)
        try:
            if model == "cx":
                cx = G.CxRun(ctx)
                cx.run(G.DeviceCxCatalog.from_host(cat, ph, ph))
                S = np.stack([cx.spectrum(ch, G.SPEC_SN) for ch in (0, 1)])
                X = np.stack([cx.spectrum(ch, G.SPEC_X_RESIDUAL) for ch in (0, 1)])
                ids, it = cx.resolved()
            else:
                ctx.run(G.DeviceCatalog.from_host(cat))
                S, X = ctx.spectrum(G.SPEC_SN), ctx.spectrum(G.SPEC_X_RESIDUAL)
                ids, it = ctx.resolved()
        finally:
            ctx.close()
        assert ids.tolist() == [0, 1, 2, 3, 4] and it.tolist() == [0, 1, 1, 2, 2]
        assert not X.any()
        out.append(S)
    for S in out[1:]:
        np.testing.assert_array_equal(S, out[0])
