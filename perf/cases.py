"""The performance cases: what users of the framework have it do.

A pass is a whole call with what a user takes from it: the subtraction of a
catalog (power model or complex templates) with the estimated PSD on the
device, the resolved list and (power model) the coarse-grained spectrum, a
batch of catalogs run together, or a catalog drawn from the population
model.  Sizes, grids and windows follow inputs.py, bench.py and the tests:
T of 1, 2 and 4 years with windows of 251, 501 and 1001 bins (2001 for the
running mean), bands of [0.3, 10] and [0.1, 30] mHz, and 1e5 to 3e7 sources
per job.  All runs use the default FP64 arithmetic; the FP32 modes exist for
the precision comparison only (they are slower and less exact than FP64).

Catalogs follow inputs.py's recipe, drawn on the GPU: f ~ f^-3, a Gamma(1.5)
amplitude joined by a Gaussian copula (rho = 0.5) to the log-normal scatter
of fdot ~ f^(11/3).
"""
import ctypes
import math

import numpy as np
import torch

from paper_2602_18560_amd import gbsub as G

YEAR = 31557600.0
WINDOW = {1: 251, 2: 501, 4: 1001}      # window per observation time (years)
FULL = (1e-4, 3e-2)                     # the job stream's band (Hz)
SHORT = (3e-4, 1e-2)                    # the 1e4 catalog's band
PAPER_BAND = (1e-4, 1e-2)               # support of the population model
MODEL = dict(alpha_pl=-2.9, alpha_g=1.96, beta_g=1.8, mu_g=-21.0, mu=-22.0, sigma=0.18, rho=0.99)


def listed():
    power = dict(kind="power", estimator=0)
    return [
        # a smoke-sized call on a band of a few thousand bins: launches and latency
        dict(power, name="power 600, narrow band", n=600, years=1, f_lo=2e-3, f_hi=2.11e-3, window=101),
        # the 1e4 catalog: one year, the oracle-scale workload
        dict(power, name="power 1e4", n=10_000, years=1, f_lo=SHORT[0], f_hi=SHORT[1], window=251),
        # an ordinary job of the stream, small end
        dict(power, name="power 2.3e5, 2 yr", n=230_017, years=2, f_lo=FULL[0], f_hi=FULL[1], window=501),
        # the headline workload: 1e7 sources, four years
        dict(power, name="power 1e7", n=10_000_000, years=4, f_lo=FULL[0], f_hi=FULL[1], window=1001),
        # the largest job of the stream
        dict(power, name="power 3e7", n=30_000_000, years=4, f_lo=FULL[0], f_hi=FULL[1], window=1001),
        # the running mean over N = 2000 bins, the paper's production estimator
        dict(kind="power", name="power 1e7, mean", estimator=1, n=10_000_000, years=4, f_lo=FULL[0], f_hi=FULL[1],
             window=2001),
        # uneven catalogs sharing every launch (a service's ordinary load)
        dict(kind="batch", name="batch of 8", catalogs=8, n_lo=100_000, n_hi=1_500_000, years=1, f_lo=FULL[0],
             f_hi=FULL[1], window=251, estimator=0),
        # the complex-template data model: oracle scale, an odd middle size, the full catalog
        dict(kind="cx", name="templates 1e4", n=10_000, years=1, f_lo=SHORT[0], f_hi=SHORT[1], window=251, estimator=0),
        dict(kind="cx", name="templates 4.1e5, 2 yr, mean", n=411_111, years=2, f_lo=FULL[0], f_hi=FULL[1],
             window=2001, estimator=1),
        dict(kind="cx", name="templates 1e7", n=10_000_000, years=4, f_lo=FULL[0], f_hi=FULL[1], window=1001, estimator=0),
        # catalogs drawn on the GPU: the paper's figure, and a small one
        dict(kind="generate", name="draw 7.5e6", n=7_500_000, **MODEL),
        dict(kind="generate", name="draw 2e4", n=20_011, **MODEL),
    ]


def _log(rng, lo, hi):
    return int(round(10 ** rng.uniform(math.log10(lo), math.log10(hi))))


def draw(rng):
    kind = rng.choice(["power", "power", "power", "mean", "batch", "cx", "cx", "generate"])
    if kind == "generate":
        return dict(kind="generate", n=_log(rng, 1e4, 1e7), alpha_pl=rng.uniform(-4, -2), alpha_g=rng.uniform(1, 3),
                    beta_g=rng.uniform(1, 3), mu_g=rng.uniform(-22, -20), mu=rng.uniform(-23, -21),
                    sigma=rng.uniform(0.1, 0.3), rho=rng.uniform(0, 0.99))
    years = rng.choice([1, 2, 4])
    band = rng.choice([FULL, FULL, SHORT, None])
    if band is None:                    # part of the band
        lo = 10 ** rng.uniform(math.log10(2e-4), math.log10(5e-3))
        band = (lo, lo * rng.uniform(1.05, 3.0))
    case = dict(years=years, f_lo=band[0], f_hi=band[1], window=WINDOW[years], estimator=0)
    if kind == "batch":
        hi = _log(rng, 2e5, 1.5e6)
        return dict(case, kind="batch", catalogs=rng.randint(3, 8), n_lo=100_000, n_hi=hi, years=1, window=251)
    if kind == "mean":
        case.update(estimator=1, window=2 * rng.randint(100, 1000) + 1)
    elif rng.random() < 0.4:
        case["window"] = 2 * rng.randint(15, 1000) + 1
    # a band of a few thousand bins holds a small catalog
    bins = (case["f_hi"] - case["f_lo"]) * years * YEAR
    top = 1e7 if kind == "cx" else 3e7
    return dict(case, kind="cx" if kind == "cx" else "power", n=_log(rng, 300, min(top, max(1000.0, 30 * bins))))


# ------------------------------------------------------------------ inputs

_TABLE = {}


def _gamma_of_normal(z, k=1.5):
    """Quantile of Gamma(k) at Phi(z), interpolated in (z, log y)."""
    if k not in _TABLE:
        ly = torch.linspace(math.log(1e-9), math.log(80.0), 1 << 16, dtype=torch.float64)
        a = torch.full_like(ly, k)
        p, q = torch.special.gammainc(a, ly.exp()), torch.special.gammaincc(a, ly.exp())
        zz = torch.where(p < 0.5, torch.special.ndtri(p), -torch.special.ndtri(q))
        ok = torch.isfinite(zz)
        _TABLE[k] = (zz[ok].cuda(), ly[ok].cuda())
    zt, lt = _TABLE[k]
    j = torch.searchsorted(zt, z.clamp(float(zt[0]), float(zt[-1]))).clamp(1, zt.numel() - 1)
    w = (z - zt[j - 1]) / (zt[j] - zt[j - 1])
    return torch.exp(lt[j - 1] + w.clamp(0, 1) * (lt[j] - lt[j - 1]))


def _catalog(n, f_lo, f_hi, seed, phases=False):
    """A, f, fdot fp32 (and the two channel phases) of n sources, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kw = dict(generator=g, device="cuda", dtype=torch.float64)
    u = torch.rand(n, **kw)
    f = (f_lo ** -2 + u * (f_hi ** -2 - f_lo ** -2)) ** -0.5
    z1 = torch.randn(n, **kw)
    z2 = 0.5 * z1 + math.sqrt(0.75) * torch.randn(n, **kw)
    A = 1e-23 * (2.0 * _gamma_of_normal(z1))
    fd = 1e-16 * (f / 1e-3) ** (11.0 / 3.0) * torch.exp(0.5 * z2)
    out = [A.float(), f.float(), fd.float()]
    if phases:
        out += [(torch.rand(n, **kw) * (2 * math.pi)).float() for _ in range(2)]
    return out


def _config(case):
    return G.default_config(t_obs_s=case["years"] * YEAR, f_min_hz=case["f_lo"], f_max_hz=case["f_hi"],
                            window_bins=case["window"], estimator=case["estimator"])


def _grid(case):
    T = case["years"] * YEAR
    k0 = math.floor(case["f_lo"] * T + 0.5)
    return T, k0, math.floor(case["f_hi"] * T + 0.5) - k0 + 1


def _sizes(case):
    c = case["catalogs"]
    r = case["n_hi"] / case["n_lo"]
    return [int(case["n_lo"] * r ** (j / (c - 1))) + j for j in range(c)]


def _ids(n):
    return torch.arange(n, dtype=torch.int32, device="cuda")


def _list(n):
    """Device memory for the resolved list of a catalog of n sources (-1 past its end)."""
    return {k: torch.full((n,), -1, dtype=torch.int32, device="cuda") for k in ("ids", "bodies")}


def _power_state(case, n, seed):
    A, f, fd = _catalog(n, case["f_lo"], case["f_hi"], seed)
    ctx = G.Context(_config(case))
    ctx.ensure_workspace(n)
    S = torch.empty(_grid(case)[2], dtype=torch.float64, device="cuda")
    return dict(ctx=ctx, cat=G.DeviceCatalog(A, f, fd, _ids(n)), S=S, **_list(n))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "power":
        return dict(case=case, **_power_state(case, case["n"], seed))
    if kind == "batch":
        jobs = [_power_state(case, n, 1000 * seed + j) for j, n in enumerate(_sizes(case))]
        return dict(case=case, jobs=jobs, batch=G.Batch(len(jobs)), stream=torch.cuda.Stream())
    if kind == "cx":
        n = case["n"]
        A, f, fd, pa, pe = _catalog(n, case["f_lo"], case["f_hi"], seed, phases=True)
        ctx = G.Context(_config(case))
        cx = G.CxRun(ctx)
        cx.ensure_workspace(n)
        S = torch.empty((2, _grid(case)[2]), dtype=torch.float64, device="cuda")
        return dict(case=case, ctx=ctx, cx=cx, cat=G.DeviceCxCatalog(A, f, fd, pa, pe, _ids(n)), S=S, **_list(n))
    pop = G.population(**{k: case[k] for k in MODEL}, f_lo_hz=PAPER_BAND[0], f_hi_hz=PAPER_BAND[1])
    n = case["n"]
    mk = lambda dt: torch.empty(n, dtype=dt, device="cuda")  # noqa: E731
    out = G.DeviceCatalog(mk(torch.float32), mk(torch.float32), mk(torch.float32), mk(torch.int32))
    return dict(case=case, pop=pop, seed=seed, n=n, out=out)


def _call(name, *args):
    status = getattr(G.load(), name)(*args)
    if status != G.OK:
        raise G.GbsubError(status, name)


def _resolved(name, j):
    """The resolved list into the job's device memory, through the C ABI."""
    m = ctypes.c_uint64()
    _call(name, j["ctx"].h, ctypes.c_void_p(j["ids"].data_ptr()), ctypes.c_void_p(j["bodies"].data_ptr()),
          j["ids"].numel(), ctypes.byref(m), 1)
    return m.value


def _results(j, s):
    """What a user takes from a finished power-model run: the PSD on the
    device, the coarse-grained spectrum and the resolved list."""
    j["ctx"].spectrum(G.SPEC_SN, out=j["S"])
    f, sp, hc, cnt = j["ctx"].coarse()
    m = _resolved("gbsub_resolved", j)
    return dict(S=j["S"], coarse=[f, sp, hc], ids=j["ids"], bodies=j["bodies"],
                counts=np.array([s.n_iter, s.n_candidates, m, *cnt]))


def run(state):
    kind = state["case"]["kind"]
    if kind == "power":
        return _results(state, state["ctx"].run(state["cat"]))
    if kind == "batch":
        batch, stream = state["batch"], state["stream"]
        slots = [batch.admit(j["ctx"], j["cat"], stream=stream) for j in state["jobs"]]
        running = len(slots)
        while running:
            batch.step(4, stream)
            _, running = batch.poll(stream)
        out = []
        for j, k in zip(state["jobs"], slots):
            status, s = batch.retire(k, stream)
            if status != G.OK:
                raise G.GbsubError(status, "batched run")
            out.append(_results(j, s))
        return out
    if kind == "cx":
        S = state["S"]
        s = state["cx"].run(state["cat"])
        nb = ctypes.c_uint64()
        for ch in (0, 1):              # the PSD of each channel, into device memory
            _call("gbsub_cx_spectrum", state["ctx"].h, ch, G.SPEC_SN, ctypes.c_void_p(S[ch].data_ptr()), S.shape[1],
                  ctypes.byref(nb), 1)
        m = _resolved("gbsub_cx_resolved", state)
        return dict(S=S, ids=state["ids"], bodies=state["bodies"], counts=np.array([s.n_iter, s.n_candidates, m]))
    o = G.generate(state["pop"], state["seed"], state["n"], out=state["out"])
    return [o.A, o.f, o.fdot, o.id]


def work(case):
    """Inputs read once, results written once, and the arithmetic that no
    method avoids (a source's frequency track or phase constants, a draw's
    random numbers and inverse CDFs)."""
    if case["kind"] == "generate":
        return dict(bytes=16 * case["n"], flops=400 * case["n"])
    B = _grid(case)[2]
    if case["kind"] == "cx":
        return dict(bytes=20 * case["n"] + 16 * B, flops=200 * case["n"])
    n, m = (sum(_sizes(case)), case["catalogs"]) if case["kind"] == "batch" else (case["n"], 1)
    return dict(bytes=12 * n + 8 * B * m, flops=20 * n)


# ------------------------------------------------------------------ the same in plain 64-bit torch

C_LIGHT, ARM, C_MED = 299792458.0, 2.5e9, 729.0 / 512.0
RTH2 = 49.0
CUT2 = ((1.0 / 7.0) * 7.0) ** 2


def _s_instr(f):
    u = f / (C_LIGHT / (2 * math.pi * ARM))
    w = 2 * math.pi * f
    wc2 = (w / C_LIGHT) ** 2
    oms = (15e-12) ** 2 * (1 + (2e-3 / f) ** 4) * wc2
    tm = (3e-15) ** 2 * (1 + (4e-4 / f) ** 2) * (1 + (f / 8e-3) ** 4) / w ** 4 * wc2
    s2, co = torch.sin(u) ** 2, torch.cos(u)
    saa = 8 * s2 * (4 * (1 + co + co * co) * tm + (2 + co) * oms)
    return saa / (16 * s2 * u * u * (0.45 / (1 + 0.7 * u * u)))


def _window(X, Sx, case, dirty, S):
    """Updates S on the bins `dirty` from the windows of X (shifted inward
    at the grid edges; the whole grid when it is shorter than the window)."""
    B, W = X.numel(), case["window"]
    median = case["estimator"] == 0
    if B < W:
        S[:] = C_MED * torch.sort(X).values[(B + 1) // 2 - 1] + Sx if median else torch.mean(X + Sx)
        return
    view = (X if median else X + Sx).unfold(0, W, 1)
    for ks in torch.split(dirty, 1 << 15):
        rows = view[(ks - (W - 1) // 2).clamp(0, B - W)]
        S[ks] = C_MED * torch.kthvalue(rows, (W + 1) // 2, dim=1).values + Sx[ks] if median else rows.mean(1)


def _reach(lo, hi, B, W):
    """Bins whose window holds a bin of some track [lo, hi]."""
    if B < W:
        return torch.arange(B, device="cuda")
    h = (W - 1) // 2
    a = torch.where(lo <= W - 1, 0, lo - h)
    b = torch.where(hi >= B - W, B - 1, hi + h)
    d = torch.zeros(B + 1, dtype=torch.int64, device="cuda")
    d.index_add_(0, a, torch.ones_like(a))
    d.index_add_(0, b + 1, -torch.ones_like(b))
    return torch.nonzero(torch.cumsum(d, 0)[:B] > 0).squeeze(1)


def _track_sums(v, lo, hi):
    """sum of v over [lo, hi] for each track."""
    P, out = 512, torch.zeros(lo.numel(), dtype=torch.float64, device="cuda")
    pad = torch.nn.functional.pad(v, (0, -v.numel() % P)).view(-1, P)
    pre = torch.cumsum(pad, 1).reshape(-1)
    blk = torch.nn.functional.pad(torch.cumsum(pad.sum(1), 0), (1, 0))
    wide = hi - lo >= 64
    below = torch.where(lo % P == 0, 0.0, pre[(lo - 1).clamp(min=0)])
    out[:] = blk[hi // P] - blk[lo // P] - below + pre[hi]
    short = torch.nonzero(~wide).squeeze(1)
    for j in torch.split(short, 1 << 20):
        k = lo[j][:, None] + torch.arange(64, device="cuda")
        out[j] = torch.where(k <= hi[j][:, None], v[k.clamp(max=v.numel() - 1)], 0.0).sum(1)
    return out


def _exact_power(case, n, seed):
    A, f, fd = (x.double() for x in _catalog(n, case["f_lo"], case["f_hi"], seed))
    T, k0, B = _grid(case)
    Sx = _s_instr((k0 + torch.arange(B, device="cuda")).double() / T)
    nn = 1 + torch.floor(fd.abs() * T * T)
    c = torch.floor((f + fd * T * 0.5) * T + 0.5) - k0
    lo = c - torch.floor((nn - 1) * 0.5)
    hi = lo + nn - 1
    q = A * A * T * 0.5 / nn
    live = torch.nonzero((hi >= 0) & (lo <= B - 1)).squeeze(1)
    lo, hi, q = lo[live].clamp(min=0).long(), hi[live].clamp(max=B - 1).long(), q[live]
    cand = torch.nonzero(4 * q * _track_sums(1 / Sx, lo, hi) >= CUT2).squeeze(1)
    clo, chi, cq = lo[cand], hi[cand], q[cand]
    body = torch.full_like(cand, -1)
    here = torch.ones(live.numel(), dtype=torch.bool, device="cuda")
    S = torch.empty(B, dtype=torch.float64, device="cuda")
    dirty = torch.arange(B, device="cuda")
    t = 0
    while True:
        one = here & (lo == hi)
        X = torch.zeros(B, dtype=torch.float64, device="cuda").index_add_(0, lo[one], q[one])
        w = here & (lo < hi)
        D = torch.zeros(B + 1, dtype=torch.float64, device="cuda")
        D.index_add_(0, lo[w], q[w]).index_add_(0, hi[w] + 1, -q[w])
        X += torch.cumsum(D[:B], 0)
        X.clamp_(min=0)
        _window(X, Sx, case, dirty, S)
        new = (body < 0) & (4 * cq * _track_sums(1 / S, clo, chi) > RTH2)
        t += 1
        if not bool(new.any()):
            break
        body[new] = t - 1
        here[cand[new]] = False
        dirty = _reach(clo[new], chi[new], B, case["window"])
    coarse, cnt = _coarse(S, T, k0)
    return dict(S=S, coarse=coarse, ids=None, bodies=None,
                counts=np.array([t, cand.numel(), int((body >= 0).sum()), *cnt]))


def _coarse(S, T, k0):
    f = (k0 + torch.arange(S.numel(), device="cuda")).double() / T
    e = torch.tensor([1e-4 * 100.0 ** (j / 100) for j in range(100)] + [1e-2], dtype=torch.float64, device="cuda")
    k = torch.searchsorted(e, f, right=True) - 1
    k[f == 1e-2] = 99
    ok = (k >= 0) & (k < 100)
    cnt = torch.bincount(k[ok], minlength=100).double()
    fm, sm = (torch.zeros(100, dtype=torch.float64, device="cuda").index_add_(0, k[ok], v[ok]) / cnt.clamp(min=1)
              for v in (f, S))
    return [x.cpu().numpy() for x in (fm, sm, torch.sqrt(fm * sm))], cnt.long().cpu().numpy()


def _templates(A, f, fd, T):
    """(central index, U [m, 128] at offsets -64 .. 63) of each source."""
    q = torch.floor((f + fd * T * 0.5) * T + 0.5)
    x = torch.arange(128, device="cuda").double() / 128
    ph = (f * T - q)[:, None] * x + (0.5 * fd * T * T)[:, None] * x * x
    s = torch.polar((0.5 * A)[:, None].expand_as(ph).contiguous(), 2 * math.pi * (ph - torch.round(ph)))
    return q, torch.fft.fftshift(torch.fft.fft(s, dim=1) * (T / 128), dim=1)


def _exact_cx(case, seed):
    n = case["n"]
    A, f, fd, pa, pe = (x.double() for x in _catalog(n, case["f_lo"], case["f_hi"], seed, phases=True))
    T, k0, B = _grid(case)
    Sx = _s_instr((k0 + torch.arange(B, device="cuda")).double() / T)
    off = torch.arange(-64, 64, device="cuda")
    h = torch.zeros((4, B + 256), dtype=torch.float64, device="cuda")     # re, im of A and E, with margins
    ok = ((fd * T * T).abs() < 1 << 20) & (((f + fd * T * 0.5) * T + 0.5).abs() < 2.0 ** 52)
    c = torch.floor((f + fd * T * 0.5) * T + 0.5) - k0
    ok &= (c + 63 >= 0) & (c - 64 <= B - 1)
    src = torch.nonzero(ok).squeeze(1)

    def add(j, sign, cut=None):
        """Adds sign x the templates of sources j to h; with cut, the sources whose rho_0^2 reaches it."""
        found = []
        for jj in torch.split(j, 1 << 19):
            qq, U = _templates(A[jj], f[jj], fd[jj], T)
            k = (qq.long() - k0)[:, None] + off
            on = (k >= 0) & (k < B)
            flat = (k + 128).reshape(-1)
            for c_, ph in enumerate((pa[jj], pe[jj])):
                H = U * torch.polar(torch.full_like(ph, sign), ph)[:, None]
                h[2 * c_].index_add_(0, flat, H.real.reshape(-1))
                h[2 * c_ + 1].index_add_(0, flat, H.imag.reshape(-1))
            if cut is not None:
                p = U.real ** 2 + U.imag ** 2
                r0 = (8 / T) * torch.where(on, p / Sx[k.clamp(0, B - 1)], 0.0).sum(1)
                found.append(jj[r0 >= cut])
        return torch.cat(found) if found else j[:0]

    cand = add(src, 1.0, CUT2)
    body = torch.full_like(cand, -1)
    S = torch.empty((2, B), dtype=torch.float64, device="cuda")
    dirty, t = torch.arange(B, device="cuda"), 0
    while True:
        for ch in (0, 1):
            X = (2 / T) * (h[2 * ch] ** 2 + h[2 * ch + 1] ** 2)[128:128 + B].contiguous()
            _window(X, Sx, case, dirty, S[ch])
        left = torch.nonzero(body < 0).squeeze(1)
        new = []
        for jj in torch.split(left, 1 << 19):
            i = cand[jj]
            qq, U = _templates(A[i], f[i], fd[i], T)
            k = (qq.long() - k0)[:, None] + off
            kc = k.clamp(0, B - 1)
            p = torch.where((k >= 0) & (k < B), U.real ** 2 + U.imag ** 2, 0.0)
            r2 = (4 / T) * (p * (1 / S[0][kc] + 1 / S[1][kc])).sum(1)
            new.append(jj[r2 > RTH2])
        new = torch.cat(new) if new else left
        t += 1
        if new.numel() == 0:
            break
        body[new] = t - 1
        add(cand[new], -1.0)
        cb = c[cand[new]].long()
        dirty = _reach((cb - 64).clamp(min=0), (cb + 63).clamp(max=B - 1), B, case["window"])
    return dict(S=S, ids=None, bodies=None, counts=np.array([t, cand.numel(), int((body >= 0).sum())]))


def _philox(ctr, block, seed):
    """Four 32-bit words of Philox4x32-10 per counter, as int64."""
    m32 = 0xFFFFFFFF
    c = [ctr & m32, (ctr >> 32) & m32, torch.full_like(ctr, block), torch.zeros_like(ctr)]
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c


def _exact_generate(case, seed):
    out = [torch.empty(case["n"], dtype=torch.float64, device="cuda") for _ in range(3)]
    for s in range(0, case["n"], 1 << 21):
        i = torch.arange(s, min(s + (1 << 21), case["n"]), device="cuda")
        w = _philox(i, 0, seed) + _philox(i, 1, seed)
        u = [(((w[2 * j] << 21) | (w[2 * j + 1] >> 11)).double() + 0.5) * 2.0 ** -53 for j in range(4)]
        rad = torch.sqrt(-2 * torch.log(u[0]))
        z1, n2 = rad * torch.cos(2 * math.pi * u[1]), rad * torch.sin(2 * math.pi * u[1])
        n3 = torch.sqrt(-2 * torch.log(u[2])) * torch.cos(2 * math.pi * u[3])
        z2 = case["rho"] * z1 + math.sqrt(1 - case["rho"] ** 2) * n2
        e = case["alpha_pl"] + 1
        lo, hi = PAPER_BAND[0] ** e, PAPER_BAND[1] ** e
        f = (lo + 0.5 * torch.erfc(-z1 / math.sqrt(2)) * (hi - lo)) ** (1 / e)
        a = torch.full_like(z2, case["alpha_g"])
        p, q = 0.5 * torch.erfc(-z2 / math.sqrt(2)), 0.5 * torch.erfc(z2 / math.sqrt(2))
        # bisection on log y, from the smaller of the two tails
        yl, yh = torch.full_like(z2, -80.0), torch.full_like(z2, 6.0)
        for _ in range(62):
            ym = 0.5 * (yl + yh)
            y = ym.exp()
            low = torch.where(p <= 0.5, torch.special.gammainc(a, y) < p, torch.special.gammaincc(a, y) > q)
            yl, yh = torch.where(low, ym, yl), torch.where(low, yh, ym)
        x = torch.exp(0.5 * (yl + yh)) / case["beta_g"]
        sl = slice(s, s + i.numel())
        out[0][sl] = 10.0 ** (torch.exp(case["sigma"] * n3) + case["mu"]) * f ** (2.0 / 3.0)
        out[1][sl] = f
        out[2][sl] = 10.0 ** (x + case["mu_g"])
    return [*out, None]


def exact(case, seed):
    if case["kind"] == "power":
        return _exact_power(case, case["n"], seed)
    if case["kind"] == "batch":
        return [_exact_power(case, n, 1000 * seed + j) for j, n in enumerate(_sizes(case))]
    if case["kind"] == "cx":
        return _exact_cx(case, seed)
    return _exact_generate(case, seed)
