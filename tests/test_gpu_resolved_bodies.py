"""The resolved list's loop bodies, on lists of several sorting blocks and on one
sorted by radix passes: pairs of a loud source and one that it masks (running
mean over 31 bins), 48 bins apart, so half of the list resolves in body 0 and
half in body 1, with opaque 32-bit ids in random order.  Whole numbers: exact."""
import ctypes

import numpy as np
import pytest

from oracle import oracle as O
from paper_2602_18560_amd import gbsub as G
from paper_2602_18560_amd.inputs import YEAR_S, Catalog, RunConfig

pytestmark = pytest.mark.gpu


def pairs(groups):
    T, k0 = 4 * YEAR_S, 20_000
    B = 48 * groups + 200
    run = RunConfig(t_obs_s=T, f_min_hz=k0 / T, f_max_hz=(k0 + B - 1) / T, window_bins=31, estimator=1)
    S0 = O.sinstr_table(O.make_config(run))
    k = 100 + 48 * np.arange(groups)
    k = np.concatenate([k, k + 5])
    P = S0[k] * np.repeat([1e4, 1e2], groups)
    rng = np.random.default_rng(groups)
    o = rng.permutation(2 * groups)
    ids = rng.choice(1 << 32, 2 * groups, replace=False).astype(np.uint32)
    cat = Catalog(A=np.sqrt(2 * P / T).astype(np.float32)[o], f=((k0 + k) / T).astype(np.float32)[o],
                  fdot=np.zeros(2 * groups, np.float32), id=ids)
    return run, cat, (o >= groups).astype(np.int32)


@pytest.mark.parametrize("model,groups", [("power", 700), ("power", 2100), ("power", 66_000), ("cx", 2100)])
def test_ids_and_bodies(model, groups):
    import torch
    run, cat, body = pairs(groups)
    z = np.zeros(cat.n, np.float32)
    if model == "power":
        assert np.array_equal(O.run(cat, O.make_config(run), spectra=False).iter_of, body)
    o = np.argsort(cat.id)
    ctx = G.Context(G.config_from_run(run))
    print(f"[resolved bodies] {model} groups {groups}", flush=True)
    try:
        if model == "cx":
            s = G.CxRun(ctx).run(G.DeviceCxCatalog.from_host(cat, z, z))
            fn = G.load().gbsub_cx_resolved
        else:
            s = ctx.run(G.DeviceCatalog.from_host(cat))
            fn = G.load().gbsub_resolved
        assert s.n_resolved == cat.n and s.n_iter == 3
        ids = torch.empty(cat.n, dtype=torch.int32, device="cuda")
        it = torch.empty(cat.n, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        m = ctypes.c_uint64()
        assert fn(ctx.h, ctypes.c_void_p(ids.data_ptr()), ctypes.c_void_p(it.data_ptr()), cat.n, ctypes.byref(m), 1) == G.OK
        assert m.value == cat.n
        np.testing.assert_array_equal(ids.cpu().numpy().view(np.uint32), cat.id[o])
        np.testing.assert_array_equal(it.cpu().numpy(), body[o])
    finally:
        ctx.close()
