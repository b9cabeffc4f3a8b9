"""The resolved list at the sizes where its sort changes path: one sorting
block and its padding, several blocks and a ragged last one, and either side
of the largest list sorted by chunks.  Whole numbers: exact."""
import ctypes

import numpy as np
import pytest

from paper_2602_18560_amd import gbsub as G
from paper_2602_18560_amd.inputs import YEAR_S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 127, 129, 2048, 2049, 9001, 131072, 131073])
@pytest.mark.parametrize("model", ["power", "cx"])
def test_resolved_list_sizes(n, model):
    """Loud monochromatic sources 24 bins apart (at most two in a window of 31
    bins), every one resolved in the first body, with opaque 32-bit ids in
    random order; 16 faint ones stay."""
    import torch
    rng = np.random.default_rng(n)
    T = 4 * YEAR_S
    k = 20_000 + 24 * np.arange(n + 16)
    f = (k / T).astype(np.float32)
    B_hi = (k[-1] + 200) / T
    A = np.full(n + 16, 1e-19, dtype=np.float32)
    A[n:] = 1e-26
    ids = rng.choice(1 << 32, n + 16, replace=False).astype(np.uint32)
    o = rng.permutation(n + 16)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x[o])).cuda()  # noqa: E731
    cfg = G.default_config(t_obs_s=T, f_min_hz=19_000 / T, f_max_hz=B_hi, window_bins=31, kappa=0.0)
    z = np.zeros(n + 16, dtype=np.float32)
    ctx = G.Context(cfg)
    print(f"[resolved list] {model} n {n}", flush=True)
    try:
        if model == "cx":
            s = G.CxRun(ctx).run(G.DeviceCxCatalog(dev(A), dev(f), dev(z), dev(z), dev(z), dev(ids.view(np.int32))))
        else:
            s = ctx.run(G.DeviceCatalog(dev(A), dev(f), dev(z), dev(ids.view(np.int32))))
        name = "gbsub_cx_resolved" if model == "cx" else "gbsub_resolved"
        assert s.n_resolved == n
        want = np.sort(ids[:n])
        for rep in range(2):
            h_ids, h_it = np.empty(n, np.uint32), np.full(n, 7, np.int32)
            d_ids = torch.empty(n, dtype=torch.int32, device="cuda")
            d_it = torch.full((n,), 7, dtype=torch.int32, device="cuda")
            torch.cuda.synchronize()
            m = ctypes.c_uint64()
            fn = getattr(G.load(), name)
            assert fn(ctx.h, h_ids.ctypes.data_as(ctypes.c_void_p), h_it.ctypes.data_as(ctypes.c_void_p), n,
                      ctypes.byref(m), 0) == G.OK
            assert fn(ctx.h, ctypes.c_void_p(d_ids.data_ptr()), ctypes.c_void_p(d_it.data_ptr()) if rep == 0 else None,
                      n, ctypes.byref(m), 1) == G.OK
            assert m.value == n
            np.testing.assert_array_equal(h_ids, want)
            np.testing.assert_array_equal(d_ids.cpu().numpy().view(np.uint32), want)
            assert not h_it.any()
            if rep == 0:
                assert not d_it.any().item()
    finally:
        ctx.close()
