"""The work units of gbsub_kernel_stats: the bins that each family's own launches
worked on.  Catalog of test_gpu_body_form: bodies 1, 2 and 3 convert X on the
first tile (2048 of 2748 bins); they filter the first tile, both, and the first
(power model) or both (template model).  X update launches: one ahead of a
body of three launches that none has preceded and one at its end (power
model), one a body of three launches (template model).  Whole numbers: exact."""
import numpy as np
import pytest

from paper_2602_18560_amd import gbsub as G
from tests.test_gpu_body_form import B, build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,budget,launches,x,med", [
    ("power", 1, 5, B + 3 * 2048, B + 2048 + B + 2048),
    ("power", 4, 5, B + 3 * 2048, B + 2048 + B + 2048),
    ("power", 65535, 0, 0, B + 2048 + B + 2048),
    ("cx", 1, 4, B + 3 * 2048, 2 * (B + 2048 + 2 * B)),
    ("cx", 4, 3, B + 2 * 2048, 2 * (B + 2048 + 2 * B)),
    ("cx", 65535, 0, 0, 2 * (B + 2048 + 2 * B)),
])
def test_units_are_those_of_the_familys_launches(model, budget, launches, x, med):
    run, cat = build(model, 0)
    ph = np.zeros(cat.n, np.float32)
    ctx = G.Context(G.config_from_run(run, split_blocks=budget))
    print(f"[units] {model} budget {budget}", flush=True)
    try:
        ctx.set_profiling(True)
        if model == "cx":
            G.CxRun(ctx).run(G.DeviceCxCatalog.from_host(cat, ph, ph))
        else:
            ctx.run(G.DeviceCatalog.from_host(cat))
        st = ctx.kernel_stats()
    finally:
        ctx.close()
    assert (st["xupdate"]["launches"], st["xupdate"]["units"], st["median"]["units"]) == (launches, x, med)
