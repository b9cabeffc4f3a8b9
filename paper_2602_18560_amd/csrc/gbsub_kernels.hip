// gbsub_kernels.hip -- HIP kernels (gfx950) of the iterative galactic-binary
// subtraction.
//
// Data layout in HBM (all structure-of-arrays, see gbsub_internal.h):
//   catalog     A, f, fdot fp32 [n]            read by the two prep passes
//   S_instr     sx, 1/sx fp64 [B] + 1/S_instr prefix tables (per grid, cached)
//   binned power Xn (one-bin tracks) and D (difference array of wider
//               tracks): 128-bit fixed point [B], [B+1]; X = Xn + prefix(D)
//   X, S, in-part prefix of 1/S: fp64 [B]; tile- and part-level tables
//   candidates  SoA records (source, clipped track, q, q in fixed point, iter)
//
// Every per-bin power sum is exact integer arithmetic on multiples of 2^L
// (L from the largest amplitude), so the binned spectrum does not depend on
// the order in which atomics land and subtracting a source is exact.  The
// SNR and the median read fp64 values converted from it with one rounding.

#include "gbsub_internal.h"
#include "gbsub_device.h"
#include <hip/hip_ext.h>

#include <math.h>

namespace gbs {

#define DEVI __device__ __forceinline__

// ------------------------------------------------------------------ helpers

DEVI I128 i128_add(I128 a, I128 b)
{
    I128 r;
    r.lo = a.lo + b.lo;
    r.hi = a.hi + b.hi + (int64_t)(r.lo < a.lo);
    return r;
}

DEVI I128 i128_from(int64_t v)
{
    I128 r;
    r.lo = (uint64_t)v;
    r.hi = v < 0 ? -1 : 0;
    return r;
}

// Exact, order-independent: adds v into the 128-bit accumulator *p.
DEVI void atomic_add_i128(I128 *p, int64_t v)
{
    const uint64_t vlo = (uint64_t)v;
    const int64_t vhi = v < 0 ? -1 : 0;
    const uint64_t old = atomicAdd((unsigned long long *)&p->lo, (unsigned long long)vlo);
    const int64_t add_hi = vhi + (int64_t)((uint64_t)(old + vlo) < old);
    if (add_hi != 0) atomicAdd((unsigned long long *)&p->hi, (unsigned long long)add_hi);
}

// Correctly rounded conversion of a non-negative 128-bit integer to fp64.
DEVI double i128_to_double(I128 v)
{
    if (v.hi < 0) return 0.0;   // cannot happen for a sum of non-negative powers
    if (v.hi == 0) return (double)v.lo;
    const uint64_t hi = (uint64_t)v.hi;
    const int lz = __clzll(hi);
    uint64_t top = lz ? ((hi << lz) | (v.lo >> (64 - lz))) : hi;
    const uint64_t rest = v.lo << lz;
    top |= (uint64_t)(rest != 0);       // sticky bit keeps round-to-nearest exact
    return ldexp((double)top, 64 - lz);
}

DEVI void split_sum_add(SplitSum *p, int64_t v)
{
    atomicAdd((unsigned long long *)&p->h, (unsigned long long)(v >> 32));   // floor(v / 2^32)
    atomicAdd((unsigned long long *)&p->l, (unsigned long long)((uint64_t)v & 0xFFFFFFFFull));
}

DEVI I128 split_sum_value(SplitSum s)
{
    I128 x;
    x.lo = (uint64_t)s.h << 32;
    x.hi = s.h >> 32;
    I128 y;
    y.lo = s.l;
    y.hi = 0;
    return i128_add(x, y);
}

// ---- double-fp32 (compensated FP32 mode)
//
// TwoSum (Knuth): s + e == a + b exactly, s = fl(a + b).  An FF add keeps the
// rounding error of the high parts and adds the low parts (the "sloppy"
// double-float addition, error O(2^-44) relative); FastTwoSum normalises.
DEVI FF ff_two_sum(float a, float b)
{
    FF r;
    r.hi = a + b;
    const float bb = r.hi - a;
    r.lo = (a - (r.hi - bb)) + (b - bb);
    return r;
}

DEVI FF ff_norm(float s, float e)                 // |s| >= |e|
{
    FF r;
    r.hi = s + e;
    r.lo = e - (r.hi - s);
    return r;
}

DEVI FF ff_add(FF a, FF b)
{
    const FF s = ff_two_sum(a.hi, b.hi);
    return ff_norm(s.hi, s.lo + (a.lo + b.lo));
}

DEVI FF ff_neg(FF a)
{
    FF r;
    r.hi = -a.hi;
    r.lo = -a.lo;
    return r;
}

DEVI FF ff_of(float x)
{
    FF r;
    r.hi = x;
    r.lo = 0.0f;
    return r;
}

DEVI float ff_float(FF a) { return a.hi + a.lo; }

// Compensated accumulation by atomics: the atomic add on hi returns the
// value it added v to; TwoSum of that value and v gives the exact rounding
// error of the sum it stored, which goes to lo.  hi + lo is then the sum up
// to the roundings of lo (second order), whatever the order of the atomics.
DEVI void ff_atomic_add(FF *p, float v)
{
    const float old = atomicAdd(&p->hi, v);
    const float e = ff_two_sum(old, v).lo;
    if (e != 0.0f) atomicAdd(&p->lo, e);
}

// Fixed-point unit 2^L: every per-bin power q <= A_max^2 T / 2 maps to an
// integer below 2^62, so 2^65 sources fit in one 128-bit accumulator.
DEVI int fx_exp(uint32_t amax_bits, double T)
{
    const double a = (double)__uint_as_float(amax_bits);
    const double pmax = ((a * a) * T) * 0.5;
    if (!(pmax > 0.0)) return 0;
    return ilogb(pmax) - 61;
}

DEVI uint64_t to_fx(double q, int L) { return (uint64_t)rint(ldexp(q, -L)); }

// The FP32 modes hold powers and PSDs scaled by 2^sc (exact): the largest
// one-bin power becomes ~2^20, so S_instr (~1e-40 in SI units, below the
// fp32 normal range) and its reciprocal stay representable; rho^2 is
// unchanged by the scale.
DEVI int f32_scale(uint32_t amax_bits, double T)
{
    const double a = (double)__uint_as_float(amax_bits);
    const double pmax = ((a * a) * T) * 0.5;
    if (!(pmax > 0.0)) return 128;
    return 20 - ilogb(pmax);
}

DEVI int lane_id() { return __lane_id(); }


// Makes the compiler produce v here (an empty asm that reads it): loads
// issued together stay together instead of being sunk into the branches
// that use them, each with its own wait.
DEVI void pin(float v) { asm volatile("" ::"v"(v)); }
DEVI void pin(double v) { asm volatile("" ::"v"(v)); }
DEVI void pin(uint64_t v) { asm volatile("" ::"v"(v)); }

template <typename T>
DEVI T shfl_up_t(T x, int d) { return __shfl_up(x, d, 64); }

DEVI I128 shfl_up_t(I128 x, int d)
{
    I128 r;
    r.lo = (uint64_t)__shfl_up((unsigned long long)x.lo, d, 64);
    r.hi = (int64_t)__shfl_up((long long)x.hi, d, 64);
    return r;
}

DEVI FF shfl_up_t(FF x, int d)
{
    FF r;
    r.hi = __shfl_up(x.hi, d, 64);
    r.lo = __shfl_up(x.lo, d, 64);
    return r;
}

DEVI double add_t(double a, double b) { return a + b; }
DEVI FF add_t(FF a, FF b) { return ff_add(a, b); }
DEVI float add_t(float a, float b) { return a + b; }
DEVI I128 add_t(I128 a, I128 b) { return i128_add(a, b); }
DEVI uint32_t add_t(uint32_t a, uint32_t b) { return a + b; }

template <typename T> DEVI T zero_t();
template <> DEVI double zero_t<double>() { return 0.0; }
template <> DEVI float zero_t<float>() { return 0.0f; }
template <> DEVI uint32_t zero_t<uint32_t>() { return 0u; }
template <> DEVI I128 zero_t<I128>() { I128 z; z.lo = 0; z.hi = 0; return z; }
template <> DEVI FF zero_t<FF>() { return ff_of(0.0f); }

// Inclusive scan of a u32 across the 64 lanes of a wave (DPP row shifts and
// row broadcasts; every lane must be active).
DEVI uint32_t wave_scan_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return v;
}

// Smallest (largest) word of the wave, in lane 63.
DEVI uint32_t wave_min_u32(uint32_t v)
{
    auto low = [&](int x) { v = min(v, (uint32_t)x); };
    low(__builtin_amdgcn_update_dpp(-1, (int)v, 0x111, 0xF, 0xF, false));
    low(__builtin_amdgcn_update_dpp(-1, (int)v, 0x112, 0xF, 0xF, false));
    low(__builtin_amdgcn_update_dpp(-1, (int)v, 0x114, 0xF, 0xF, false));
    low(__builtin_amdgcn_update_dpp(-1, (int)v, 0x118, 0xF, 0xF, false));
    low(__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xA, 0xF, false));
    low(__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xC, 0xF, false));
    return v;
}
DEVI uint32_t wave_max_u32(uint32_t v) { return ~wave_min_u32(~v); }

// Inclusive scan across the 64 lanes of a wave.
template <typename T>
DEVI T wave_incl_scan(T x)
{
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        T y = shfl_up_t(x, d);
        if (lane >= d) x = add_t(x, y);
    }
    return x;
}

template <> DEVI uint32_t wave_incl_scan<uint32_t>(uint32_t x) { return wave_scan_u32(x); }

// Exclusive scan across the WG threads of a block; *total gets the block sum.
// `sh` must hold WG/64 elements.  Contains __syncthreads().
template <typename T, int NT = WG>
DEVI T block_excl_scan(T x, T *sh, T *total)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    T inc = wave_incl_scan(x);
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    T pre = zero_t<T>(), tot = zero_t<T>();
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        if (w < wave) pre = add_t(pre, sh[w]);
        tot = add_t(tot, sh[w]);
    }
    __syncthreads();
    T ex = shfl_up_t(inc, 1);
    if (lane == 0) ex = zero_t<T>();
    *total = tot;
    return add_t(pre, ex);
}

DEVI double wave_sum(double x)
{
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}


// sum_{k=lo..hi} 1/v[k] from the tile tables (inclusive in-tile prefix `pre`,
// exclusive tile prefix `tl`); short ranges are summed bin by bin in
// ascending order.
DEVI double range_inv_sum(const double *v, const double *pre, const double *tl, int lo, int hi,
                          int tile)
{
    if (hi - lo + 1 <= NARROW) {
        double s = 0.0;
        for (int k = lo; k <= hi; ++k) s += 1.0 / v[k];
        return s;
    }
    const int tlo = div_p2(lo, tile), thi = div_p2(hi, tile);
    const double below = mod_p2(lo, tile) == 0 ? 0.0 : pre[lo - 1];
    if (tlo == thi) return pre[hi] - below;
    return ((tl[thi] - tl[tlo]) - below) + pre[hi];
}

// ------------------------------------------------------------------ grid tables


__global__ __launch_bounds__(WG) void k_sinstr(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    const int k = blockIdx.x * WG + threadIdx.x;
    if (k >= g.B) return;
    const double f = (double)(g.k0 + k) / g.T;
    const double v = sinstr_dev(f, g.oms_pm, g.tm_fm, g.arm_m);
    d.sx[k] = v;
    d.isx[k] = 1.0 / v;
}

// In-tile inclusive prefix of 1/v and the tile sums (one block per tile).
__global__ __launch_bounds__(WG) void k_inv_prefix(const Slot *S)
{
    __shared__ double sh[WG / 64];
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    const double *v = d.sx;
    double *pre = d.isx_pre, *tsum = d.isx_tsum;
    const int tile = blockIdx.x, R = g.tile / WG;
    if (tile >= g.nt) return;
    const int base = tile * g.tile + threadIdx.x * R;
    double loc[8];
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int k = base + r;
        if (r < R) s += (k < g.B) ? 1.0 / v[k] : 0.0;
        loc[r] = s;
    }
    double tot;
    const double ex = block_excl_scan(s, sh, &tot);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int k = base + r;
        if (r < R && k < g.B) pre[k] = ex + loc[r];
    }
    if (threadIdx.x == 0) tsum[tile] = tot;
}

// Exclusive prefix over the tile sums (single block).  Each thread owns a
// contiguous run of ceil(n / WG) entries: its loads are all issued at once
// (no chain of per-chunk scans waiting on memory), one block scan combines
// the run totals, and a second pass over the (cached) run writes the prefix.
template <typename T, int NT = WG, typename A = T>
DEVI void block_scan_array(const T *in, T *out, int n)
{
    __shared__ A sh[NT / 64];
    constexpr int RUN = 8;                 // runs this short stay in registers
    const int per = (n + NT - 1) / NT;
    const int b = min((int)threadIdx.x * per, n), e = min(b + per, n);
    if (per <= RUN) {
        // every load of the run issued before the first use (clamped
        // indices, no branches around the loads)
        A v[RUN];
#pragma unroll
        for (int r = 0; r < RUN; ++r) v[r] = (A)in[min(b + r, n - 1 < 0 ? 0 : n - 1)];
        A s = zero_t<A>();
#pragma unroll
        for (int r = 0; r < RUN; ++r)
            if (b + r < e) s = add_t(s, v[r]);
        A tot;
        A run = block_excl_scan<A, NT>(s, sh, &tot);
#pragma unroll
        for (int r = 0; r < RUN; ++r) {
            if (b + r < e) {
                out[b + r] = (T)run;
                run = add_t(run, v[r]);
            }
        }
        if (threadIdx.x == 0) out[n] = (T)tot;
        return;
    }
    A s = zero_t<A>();
#pragma unroll 8
    for (int i = b; i < e; ++i) s = add_t(s, (A)in[i]);
    A tot;
    A run = block_excl_scan<A, NT>(s, sh, &tot);
#pragma unroll 8
    for (int i = b; i < e; ++i) {
        const A x = (A)in[i];
        out[i] = (T)run;
        run = add_t(run, x);
    }
    if (threadIdx.x == 0) out[n] = (T)tot;
}

__global__ __launch_bounds__(WG) void k_sx_scan(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    block_scan_array<double>(d.isx_tsum, d.isx_tile, g.nt);
}

// (min, max) of 1/S_instr over each segment of SEG_BINS bins (one wave per
// segment): bounds that decide most one-bin candidate tests without the
// table value of the source's bin.
__global__ __launch_bounds__(WG) void k_isx_seg(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    const int seg = blockIdx.x * (WG / 64) + (threadIdx.x >> 6);
    const int nseg = (g.B + SEG_BINS - 1) / SEG_BINS;
    if (seg >= nseg) return;
    double mn = INFINITY, mx = -INFINITY;
    for (int k = seg * SEG_BINS + lane_id(); k < min((seg + 1) * SEG_BINS, g.B); k += 64) {
        const double x = d.isx[k];
        mn = fmin(mn, x);
        mx = fmax(mx, x);
    }
    for (int o = 32; o >= 1; o >>= 1) {
        mn = fmin(mn, __shfl_xor(mn, o, 64));
        mx = fmax(mx, __shfl_xor(mx, o, 64));
    }
    if (lane_id() == 0) d.isx_seg[seg] = make_double2(mn, mx);
}

// ------------------------------------------------------------------ reset

// Clears the per-run state of a slot: control block, tile counters, dirty
// stamps (every tile is dirty for the first loop body, t = 0).
// It also writes the slot's descriptor to device memory (a copy from the host
// ahead of the run cost its own 2 us and the 8 to 10 us until the next kernel).
__global__ __launch_bounds__(WG) void k_reset(Slot sl, Slot *ds)
{
    const Grid &g = sl.g;
    const Dev &d = sl.d;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *ds = sl;
        Ctl *c = d.ctl;
        c->amax_bits = 0;
        c->bad = 0;
        c->n_cand = 0;
        c->done = 0;
        c->n_iter = 0;
        c->n_resolved = 0;
        c->n_chunks = 0;
        c->cand_cursor = 0;
        c->n_events = 0;
        c->iter = 0;
        c->n_near = 0;
        c->min_margin = 0x7FF0000000000000ull;   // +inf
        c->units_x = 0;
        c->units_med = (uint64_t)g.B;            // the first body filters every bin
        c->units_snr = 0;
        c->status = 0;
        c->med_split = (uint32_t)g.nt <= g.split_tiles;   // every tile is dirty
        c->n_sdl = (uint32_t)g.nt;
        c->xupd = 0;
        c->tail_due = 0;
        c->res_cursor = 0;
    }
    for (int i = blockIdx.x * WG + threadIdx.x; i < g.nt; i += gridDim.x * WG) {
        d.xstamp[i] = 0;          // body 0 converts and filters every tile
        d.sstamp[i] = 0;
        d.sdl[i] = (uint32_t)i;
        d.Dadj[i].h = 0;
        d.Dadj[i].l = 0;
    }
}

// ------------------------------------------------------------------ prep
//
// Per source (Sec. "Signal parametrization"; appendix "Subtraction
// algorithm", steps 2-3): power P = A^2 T / 2, mid-track frequency
// f + fdot T/2, centre bin floor(fbar T + 1/2) - k0, n = 1 + floor(|fdot| T^2)
// bins, per-bin power q = P/n, track clipped to the grid; rho_0^2 against
// S_instr; candidate iff rho_0^2 >= (kappa rho_th)^2.
//
// Binning without global atomics: a count pass tallies the binning events
// of each block of PREP_SRC sources per tile in LDS and writes that row of
// counts; a column pass gives every (block, tile) its first slot among the
// tile's events (the counts of the blocks before it) and the tile totals;
// after a scan of the totals, a scatter pass writes every event to its
// tile's contiguous segment; accumulation blocks then sum up to ACC_EV
// events of one tile in LDS (exact 128-bit integers) and write the tile's
// bins, hot tiles through partial sums reduced by a last pass.

struct Trk {
    bool ok, live;
    int glo, ghi;
    double q;
};

// Track and per-bin power of one source (no candidate test).
DEVI Trk track_geom(const Grid &g, float Af, float Ff, float FDf)
{
    Trk t;
    t.ok = false;
    t.live = false;
    t.glo = 0;
    t.ghi = -1;
    t.q = 0.0;
    const double a = (double)Af, f = (double)Ff, fd = (double)FDf;
    bool ok = isfinite(a) && a >= 0.0 && isfinite(f) && f > 0.0 && isfinite(fd);
    const double P = ((a * a) * g.T) * 0.5;
    const double fbar = f + (fd * g.T) * 0.5;
    const double x = fbar * g.T + 0.5;
    const double s = (fabs(fd) * g.T) * g.T;
    if (!ok) return t;
    t.ok = true;
    // 2^52 bins or more away, or long (beyond exact integers): at most 2^-52
    // of the power in any bin; no power on the grid
    if (!(fabs(x) < 4503599627370496.0 && s < 4503599627370496.0)) return t;
    // integer-valued fp64 throughout (|values| < 2^53: exact)
    const double c = floor(x) - (double)g.k0;
    const double nn = g.track_single ? 1.0 : 1.0 + floor(s);
    const double lo = c - floor((nn - 1.0) * 0.5);
    const double hi = lo + (nn - 1.0);
    t.q = nn == 1.0 ? P : P / nn;
    const double gl = fmax(lo, 0.0);
    const double gh = fmin(hi, (double)(g.B - 1));
    if (gl > gh) return t;
    t.live = true;
    t.glo = (int)gl;
    t.ghi = (int)gh;
    return t;
}

// rho_0^2 >= (kappa rho_th)^2 against S_instr.  Short tracks sum the stored
// reciprocals 1/S_instr bin by bin in ascending order (the same values and
// order as summing 1/S_instr directly), longer ones use the prefix tables.
// x0 = 1/S_instr of the track's first bin, loaded by the caller.
DEVI bool cand_test(const Grid &g, const Dev &d, const Trk &t, double x0)
{
    if (!t.live) return false;
    double sum;
    if (t.glo == t.ghi) {
        sum = x0;
    } else if (t.ghi - t.glo + 1 <= NARROW) {
        sum = x0;
        for (int k = t.glo + 1; k <= t.ghi; ++k) sum += d.isx[k];
    } else {
        sum = range_inv_sum(d.sx, d.isx_pre, d.isx_tile, t.glo, t.ghi, g.tile);
    }
    return (4.0 * t.q) * sum >= g.cut2;
}

DEVI int tile_of(int bin, int tile) { return div_p2(bin, tile); }

// Count pass: events per tile and candidates of this block.  The per-tile
// counts are 16-bit halves of LDS words (at most 2 PREP_SRC < 2^16 events
// of a block fall in one tile), which keeps the block's LDS at 16 KB; the
// packed words are the block's row of bhist.
DEVI void k_prep_count_body(const Grid &g, const Dev &d, const float *A, const float *F, const float *FD, uint64_t n,
                            uint32_t *hist)
{
    // sources per thread in flight: four, with six waves per SIMD (eight, with
    // three, took 93 us for 1e7 sources instead of 65)
    constexpr int CB = 4;
    static_assert(PREP_SRC % (CB * WG) == 0 && PREP_SRC_MIN % (CB * WG) == 0, "whole batches");
    __shared__ uint32_t scand, samax;
    auto hadd = [&](int b) { atomicAdd(&hist[b >> 1], 1u << (16 * (b & 1))); };
    for (int b = threadIdx.x; b < (g.nt + 1) / 2; b += WG) hist[b] = 0;
    if (threadIdx.x == 0) {
        scand = 0;
        samax = 0;
    }
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * d.prep_src;
    uint32_t cc = 0, bad = 0, amax = 0;
    // CB sources per thread in flight: loads first, then the tracks and
    // the S_instr gathers of the candidate tests
    for (int r0 = 0; r0 < (int)d.prep_src / WG; r0 += CB) {
        float a[CB], f[CB], fd[CB];
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            const uint64_t i = base + (uint64_t)(r0 + q) * WG + threadIdx.x;
            const bool in = i < n;
            const uint64_t ic = in ? i : n - 1;        // unconditional loads: all in flight at once
            const float av = A[ic], fv = F[ic], fdv = FD[ic];
            a[q] = in ? av : 0.0f;
            f[q] = in ? fv : 1.0f;
            fd[q] = in ? fdv : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            pin(a[q]);
            pin(f[q]);
            pin(fd[q]);
        }
        Trk t[CB];
#pragma unroll
        for (int q = 0; q < CB; ++q) t[q] = track_geom(g, a[q], f[q], fd[q]);
        // Bounds from the (min, max) of 1/S_instr over the segments under the
        // track decide most tests without the table values.  One bin:
        // rho_0^2 = (4q) (1/S_instr) lies between (4q) min and (4q) max (the
        // product is monotone).  2 .. NARROW bins (at most two segments): the
        // fp64 sum of the n values lies within n min (1 - n 2^-53) and
        // n max (1 + n 2^-53), so a margin of 1e-12 on n min and n max is
        // safe.  Otherwise, or if the cut falls between the bounds, the table
        // values decide (their gathers all in flight).
        double2 sb[CB], se[CB];
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            sb[q] = d.isx_seg[t[q].live ? t[q].glo / SEG_BINS : 0];
            se[q] = d.isx_seg[t[q].live ? t[q].ghi / SEG_BINS : 0];
        }
        bool cand[CB], exact[CB];
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            const double q4 = 4.0 * t[q].q;
            const int nb = t[q].ghi - t[q].glo + 1;
            const bool one = t[q].live && nb == 1;
            const bool few = t[q].live && nb > 1 && nb <= NARROW;
            const double mn = fmin(sb[q].x, se[q].x), mx = fmax(sb[q].y, se[q].y);
            const double lo = few ? q4 * ((double)nb * mn) * (1.0 - 1e-12) : q4 * mn;
            const double hi = few ? q4 * ((double)nb * mx) * (1.0 + 1e-12) : q4 * mx;
            const bool yes = (one || few) && lo >= g.cut2;
            const bool no = (one || few) && hi < g.cut2;
            cand[q] = yes;
            exact[q] = t[q].live && !yes && !no;
        }
        double x0[CB];
#pragma unroll
        for (int q = 0; q < CB; ++q) x0[q] = exact[q] ? d.isx[t[q].glo] : 0.0;
#pragma unroll
        for (int q = 0; q < CB; ++q)
            if (exact[q]) cand[q] = cand_test(g, d, t[q], x0[q]);
#pragma unroll
        for (int q = 0; q < CB; ++q) {
            const uint64_t i = base + (uint64_t)(r0 + q) * WG + threadIdx.x;
            const bool in = i < n;
            const bool c = in && t[q].ok && cand[q];
            const uint64_t m = (uint64_t)__ballot(c);
            const uint64_t w0 = i - (uint64_t)lane_id();       // first source of this wave
            if (lane_id() == 0 && w0 < n) d.cbits[w0 >> 6] = m;
            if (!in) continue;
            if (!t[q].ok) {
                bad = 1;
                continue;
            }
            amax = max(amax, __float_as_uint(a[q]));      // A >= 0: bit patterns in value order
            if (t[q].live) {
                hadd(tile_of(t[q].glo, g.tile));
                if (t[q].glo != t[q].ghi && t[q].ghi + 1 < g.B) hadd(tile_of(t[q].ghi + 1, g.tile));
            }
            cc += c;
        }
    }
    for (int s = 32; s >= 1; s >>= 1) {
        cc += (uint32_t)__shfl_xor((int)cc, s, 64);
        amax = max(amax, (uint32_t)__shfl_xor((int)amax, s, 64));
    }
    if (lane_id() == 0 && cc) atomicAdd(&scand, cc);
    if (lane_id() == 0 && amax) atomicMax(&samax, amax);
    __syncthreads();
    // per-block results (k_prep_plan combines them: no atomics on one address)
    if (threadIdx.x == 0) {
        d.blk_cand[blockIdx.x] = scand;
        d.blk_amax[blockIdx.x] = samax;
    }
    const int hw = (g.nt + 1) / 2;
    for (int b = threadIdx.x; b < hw; b += WG) d.bhist[(size_t)blockIdx.x * hw + b] = hist[b];
    if (bad) atomicOr(&d.ctl->bad, 1u);
}

__global__ __launch_bounds__(WG) void k_prep_count(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active || (uint64_t)blockIdx.x * sl.d.prep_src >= sl.n) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    __shared__ uint32_t hist[NBK_MAX / 2];
    k_prep_count_body(g, d, sl.A, sl.F, sl.FD, sl.n, hist);
}


// Column pass: for each tile, the exclusive prefix over the prep blocks of
// its event counts (where each block's events start inside the tile's
// segment) and the tile's total.  A block takes CS_COL tiles, its threads
// NV ranges of the prep blocks: each sums its range, a prefix over the ranges
// gives each its start, and each walks its range again writing the offsets.
// (1e7 sources, 1843 tiles: 22 us; 64 tiles per block, 30 us; 16, 23 us, and 39
// against 31 us at 3686 tiles, for the shorter rows.)
__global__ __launch_bounds__(CS_WG) void k_prep_colscan(const Slot *S)
{
    constexpr int NV = CS_WG / CS_COL;
    __shared__ uint32_t part[NV][CS_COL + 1];
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    const int q0 = threadIdx.x % CS_COL, w = threadIdx.x / CS_COL;
    const int tile = blockIdx.x * CS_COL + q0;
    const bool ok = tile < g.nt;
    const int col = ok ? tile : g.nt - 1;                      // a valid column; results dropped
    const int nb = (int)((sl.n + d.prep_src - 1) / d.prep_src);
    const int per = (nb + NV - 1) / NV;
    const int b0 = min(w * per, nb), b1 = min(b0 + per, nb);
    const size_t row = 2 * (size_t)((g.nt + 1) / 2);          // 16-bit counts per bhist row
    const uint16_t *h16 = reinterpret_cast<const uint16_t *>(d.bhist);
    constexpr int U = 16;
    uint32_t sum = 0;
    for (int bb = b0; bb < b1; bb += U) {
        uint32_t c[U];
#pragma unroll
        for (int q = 0; q < U; ++q) c[q] = h16[(size_t)min(bb + q, b1 - 1) * row + col];
#pragma unroll
        for (int q = 0; q < U; ++q) sum += bb + q < b1 ? c[q] : 0u;
    }
    part[w][q0] = sum;
    __syncthreads();
    // exclusive prefix over the ranges, one wave per column
    for (int c = threadIdx.x >> 6; c < CS_COL; c += CS_WG / 64) {
        const int l = lane_id();
        const uint32_t x = l < NV ? part[l][c] : 0u;
        const uint32_t inc = wave_scan_u32(x);
        if (l < NV) part[l][c] = inc - x;
        if (l == 63 && blockIdx.x * CS_COL + c < g.nt) d.btot[blockIdx.x * CS_COL + c] = inc;
    }
    __syncthreads();
    uint32_t run = part[w][q0];
    for (int bb = b0; bb < b1; bb += U) {
        uint32_t c[U];
#pragma unroll
        for (int q = 0; q < U; ++q) c[q] = h16[(size_t)min(bb + q, b1 - 1) * row + col];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (bb + q < b1) {
                if (ok) d.boff[(size_t)(bb + q) * g.nt + tile] = run;
                run += c[q];
            }
        }
    }
}

DEVI uint32_t acc_events(int k) { return k == 0 ? (uint32_t)ACC_EV_MIN : (uint32_t)ACC_EV / 4u * (uint32_t)(k + 1); }

// Plan (one block): tile bases, accumulation blocks and partial-sum slots;
// clears the tile sums of D.
__global__ __launch_bounds__(PLAN_T) void k_prep_plan(const Slot *S)
{
    __shared__ uint32_t sh[PLAN_T / 64];
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;

    // the candidates of the count blocks: their exclusive prefix is each
    // scatter block's first candidate slot
    const int nb = (int)((sl.n + d.prep_src - 1) / d.prep_src);
    uint32_t am = 0;                                   // the largest A
    for (int b = threadIdx.x; b < nb; b += PLAN_T) am = max(am, d.blk_amax[b]);
    block_scan_array<uint32_t, PLAN_T>(d.blk_cand, d.blk_cand, nb);   // in place: each thread rereads its own run

    // The events of an accumulation block (at most ACC_EV, acc_events' choices):
    // the fewest that leave at most ACC_GRID full blocks, so that a hot tile
    // spreads over the chip, and whose hot tiles' partial sums fit.  (2.3e5
    // sources, whose hot tile has more than 65536 events: k_accum 18 us, 25 with
    // blocks of 65536; 1e7 sources 53 us, as before; at most 1024 full blocks
    // instead of 256 doubled their reduction to 30 us.)
    constexpr int RUN = NBK_MAX / PLAN_T, NC = 4;
    constexpr int NV = PLAN_T / 64;
    __shared__ uint32_t s_need[NC + 2][NV];            // per wave: slots by choice, events, largest A
    const int b0 = (int)threadIdx.x * RUN;
    uint32_t cnt[RUN], need[NC + 1] = {};
#pragma unroll
    for (int r = 0; r < RUN; ++r) cnt[r] = d.btot[min(b0 + r, g.nt - 1)];
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        cnt[r] = b0 + r < g.nt ? cnt[r] : 0u;
        need[NC] += cnt[r];
        if (cnt[r] <= (uint32_t)ACC_EV_MIN) continue;
#pragma unroll
        for (int k = 0; k < NC; ++k) need[k] += cnt[r] > acc_events(k) ? (cnt[r] + acc_events(k) - 1) / acc_events(k) : 0u;
    }
#pragma unroll
    for (int k = 0; k <= NC; ++k) {
        const uint32_t x = wave_scan_u32(need[k]);
        if (lane_id() == 63) s_need[k][threadIdx.x >> 6] = x;
    }
    am = wave_max_u32(am);
    if (lane_id() == 63) s_need[NC + 1][threadIdx.x >> 6] = am;
    __syncthreads();
    const int wl = lane_id() < NV ? lane_id() : 0;
#pragma unroll
    for (int k = 0; k <= NC; ++k) {
        const uint32_t x = lane_id() < NV ? s_need[k][wl] : 0u;
        need[k] = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_u32(x), 63);
    }
    am = wave_max_u32(s_need[NC + 1][wl]);             // in lane 63
    int k = 0;
    while (k < NC - 1 && (need[k] > d.max_slots || need[NC] / acc_events(k) > (uint32_t)ACC_GRID)) ++k;
    const uint32_t ev = acc_events(k);
    uint32_t sum[3] = {}, ex[3], tot[3], nch[RUN];     // events, blocks, partial-sum slots
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        nch[r] = b0 + r < g.nt ? 1u : 0u;
        if (cnt[r] > ev) nch[r] = (cnt[r] + ev - 1) / ev;
        sum[0] += cnt[r];
        sum[1] += nch[r];
        sum[2] += nch[r] > 1 ? nch[r] : 0u;
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) ex[q] = block_excl_scan<uint32_t, PLAN_T>(sum[q], sh, &tot[q]);
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        const int b = b0 + r;
        if (b >= g.nt) continue;
        d.bbase[b] = ex[0];
        d.nch[b] = nch[r];
        d.chunk_base[b] = ex[1];
        d.slot_base[b] = ex[2];
        d.Dtile[b].lo = 0;
        d.Dtile[b].hi = 0;
        if (g.prec == PREC_COMP) d.Dtc[b] = ff_of(0.0f);
        ex[0] += cnt[r];
        ex[1] += nch[r];
        ex[2] += nch[r] > 1 ? nch[r] : 0u;
    }
    if (threadIdx.x == 63) d.ctl->amax_bits = am;
    if (threadIdx.x == 0) {
        d.ctl->n_cand = d.blk_cand[nb];
        d.bbase[g.nt] = tot[0];
        d.chunk_base[g.nt] = tot[1];
        d.Dtile[g.nt].lo = 0;
        d.Dtile[g.nt].hi = 0;
        d.ctl->n_events = tot[0];
        d.ctl->n_chunks = tot[1];
        d.ctl->acc_ev = ev;
        if (tot[2] > d.max_slots || tot[1] > d.max_chunks) d.ctl->bad |= 2u;   // cannot happen: sized for the worst case
    }
}

// Scatter pass: the block's events start, inside each tile's segment, at
// the slot the column pass gave it; it writes the events and the candidate
// records.
template <int SB>                            // sources per thread in flight
DEVI void k_prep_scatter_body(const Grid &g, const Dev &d, const float *A, const float *F, const float *FD, uint64_t n,
                              uint32_t *cur, uint32_t row)
{
    static_assert(PREP_SRC % (SB * WG) == 0, "whole batches");
    __shared__ uint32_t scand, cbase;
    for (int b = threadIdx.x; b < g.nt; b += WG) cur[b] = d.bbase[b] + d.boff[(size_t)row * g.nt + b];
    if (threadIdx.x == 0) {
        cbase = d.blk_cand[row];
        scand = 0;
    }
    __syncthreads();
    const int L = fx_exp(d.ctl->amax_bits, g.T);
    const uint64_t base = (uint64_t)row * d.prep_src;
    for (int r0 = 0; r0 < (int)d.prep_src / WG; r0 += SB) {
        float a[SB], f[SB], fd[SB];
        uint64_t cw[SB];                         // candidate-flag words of the sources
#pragma unroll
        for (int q = 0; q < SB; ++q) {
            const uint64_t i = base + (uint64_t)(r0 + q) * WG + threadIdx.x;
            const bool in = i < n;
            const uint64_t ic = in ? i : n - 1;        // unconditional loads: all in flight at once
            const float av = A[ic], fv = F[ic], fdv = FD[ic];
            a[q] = in ? av : 0.0f;
            f[q] = in ? fv : 1.0f;
            fd[q] = in ? fdv : 0.0f;
            cw[q] = d.cbits[ic >> 6];
        }
#pragma unroll
        for (int q = 0; q < SB; ++q) {
            pin(a[q]);
            pin(f[q]);
            pin(fd[q]);
            pin(cw[q]);
        }
#pragma unroll
        for (int q = 0; q < SB; ++q) {
            const uint64_t i = base + (uint64_t)(r0 + q) * WG + threadIdx.x;
            if (i >= n) continue;
            const Trk t = track_geom(g, a[q], f[q], fd[q]);
            if (!t.ok) continue;
            const uint64_t qfx = to_fx(t.q, L);
            if (t.live) {                  // every live source, so the counts match
                if (t.glo == t.ghi) {
                    const uint32_t p = atomicAdd(&cur[tile_of(t.glo, g.tile)], 1u);
                    d.ev_key[p] = (uint32_t)t.glo;
                    d.ev_val[p] = (int64_t)qfx;
                } else {
                    uint32_t p = atomicAdd(&cur[tile_of(t.glo, g.tile)], 1u);
                    d.ev_key[p] = (uint32_t)t.glo | 0x80000000u;
                    d.ev_val[p] = (int64_t)qfx;
                    if (t.ghi + 1 < g.B) {
                        p = atomicAdd(&cur[tile_of(t.ghi + 1, g.tile)], 1u);
                        d.ev_key[p] = (uint32_t)(t.ghi + 1) | 0x80000000u;
                        d.ev_val[p] = -(int64_t)qfx;
                    }
                }
            }
            if ((cw[q] >> (i & 63)) & 1ull) {
                const uint32_t j = cbase + atomicAdd(&scand, 1u);
                d.c_src[j] = (uint32_t)i;
                d.c_glo[j] = t.glo;
                d.c_ghi[j] = t.ghi;
                d.c_q[j] = t.q;
                d.c_qfx[j] = qfx;
                d.c_iter[j] = -1;
            }
        }
    }
}

// Blocks go round-robin over the 8 XCDs, so XCD x takes the rows [x per,
// (x + 1) per): the slots of neighbouring rows in a tile's segment are
// neighbours, and a 128-byte line is then written by one XCD's L2, not in parts
// by several (3e7 sources: 292 us, 307 with the rows dealt round-robin; more
// waves, with LDS for the grid's own tiles only, 314).
__global__ __launch_bounds__(WG) void k_prep_scatter(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const uint32_t rows = (uint32_t)((sl.n + sl.d.prep_src - 1) / sl.d.prep_src), per = (rows + 7u) / 8u;
    const uint32_t row = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per || row >= rows) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    __shared__ uint32_t cur[NBK_MAX];
    if (d.prep_src == PREP_SRC)
        k_prep_scatter_body<8>(g, d, sl.A, sl.F, sl.FD, sl.n, cur, row);
    else
        k_prep_scatter_body<4>(g, d, sl.A, sl.F, sl.FD, sl.n, cur, row);
}


DEVI void lds_add_i128(I128 *p, int64_t v)
{
    const uint64_t vlo = (uint64_t)v;
    const int64_t vhi = v < 0 ? -1 : 0;
    const uint64_t old = atomicAdd((unsigned long long *)&p->lo, (unsigned long long)vlo);
    const int64_t add_hi = vhi + (int64_t)((uint64_t)(old + vlo) < old);
    if (add_hi != 0) atomicAdd((unsigned long long *)&p->hi, (unsigned long long)add_hi);
}

DEVI void atomic_add_i128_full(I128 *p, I128 v)
{
    const uint64_t old = atomicAdd((unsigned long long *)&p->lo, (unsigned long long)v.lo);
    const int64_t add_hi = v.hi + (int64_t)((uint64_t)(old + v.lo) < old);
    if (add_hi != 0) atomicAdd((unsigned long long *)&p->hi, (unsigned long long)add_hi);
}

// Accumulation: block c sums up to ACC_EV events of one tile in LDS.  Each
// 64-bit event value v = vh 2^32 + vl (vl in [0, 2^32)) goes into two 64-bit
// LDS sums with non-returning atomics (no carry to propagate: at most ACC_EV
// events per block, so |sum vh| < 2^47 and sum vl < 2^48); the exact
// 128-bit total is sum_vh 2^32 + sum_vl.
struct SplitAcc {
    int64_t h[TILE_MAX];
    uint64_t l[TILE_MAX];
};

DEVI void split_add(SplitAcc &a, int k, int64_t v)
{
    atomicAdd((unsigned long long *)&a.h[k], (unsigned long long)(v >> 32));
    atomicAdd((unsigned long long *)&a.l[k], (unsigned long long)((uint64_t)v & 0xFFFFFFFFull));
}

DEVI I128 split_total(const SplitAcc &a, int k)
{
    const int64_t h = a.h[k];
    I128 x;
    x.lo = (uint64_t)h << 32;
    x.hi = h >> 32;
    I128 y;
    y.lo = a.l[k];
    y.hi = 0;
    return i128_add(x, y);
}

// The compensated FP32 mode's binning of the ne events from e0 on of tile b
// (chunk ci): every event's power rounded to fp32 (scaled by 2^sc), summed per bin
// in LDS by compensated atomics (xc: one-bin tracks, dc: difference array;
// TILE_MAX entries each); written to Xc, Dc and the tile sum of Dc, or to
// the chunk's partial-sum slot of a hot tile.
DEVI void accum_comp(const Grid &g, const Dev &d, int b, uint32_t ci, uint32_t e0, uint32_t ne, FF *xc, FF *dc)
{
    __shared__ FF shf[ACC_T / 64];
    const int k0 = b * g.tile;
    const int L = fx_exp(d.ctl->amax_bits, g.T);
    const int sc = f32_scale(d.ctl->amax_bits, g.T);
    for (int k = threadIdx.x; k < g.tile; k += ACC_T) {
        xc[k] = ff_of(0.0f);
        dc[k] = ff_of(0.0f);
    }
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < ne; e += ACC_T) {
        const uint32_t key = d.ev_key[e0 + e];
        const float v = (float)ldexp((double)d.ev_val[e0 + e], L + sc);
        const int k = (int)(key & 0x7FFFFFFFu) - k0;
        ff_atomic_add((key >> 31) ? &dc[k] : &xc[k], v);
    }
    __syncthreads();
    const int nbin = min(g.tile, g.B - k0);
    if (d.nch[b] == 1) {
        FF s = ff_of(0.0f);
        for (int k = threadIdx.x; k < g.tile; k += ACC_T) {
            if (k < nbin) {
                const FF x = ff_norm(xc[k].hi, xc[k].lo), y = ff_norm(dc[k].hi, dc[k].lo);
                d.Xc[k0 + k] = x;
                d.Dc[k0 + k] = y;
                s = ff_add(s, y);
            }
        }
        FF tot;
        block_excl_scan<FF, ACC_T>(s, shf, &tot);
        if (threadIdx.x == 0) d.Dtc[b] = tot;
    } else {
        FF *slot = reinterpret_cast<FF *>(d.partial + (size_t)(d.slot_base[b] + ci) * 2 * g.tile);
        for (int k = threadIdx.x; k < g.tile; k += ACC_T) {
            slot[k] = ff_norm(xc[k].hi, xc[k].lo);
            slot[g.tile + k] = ff_norm(dc[k].hi, dc[k].lo);
        }
    }
}

__global__ __launch_bounds__(ACC_T) void k_accum(const Slot *S)
{
    __shared__ SplitAcc xn, dd;
    __shared__ I128 sh[ACC_T / 64];
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;

    const uint32_t c = blockIdx.x;
    if (c >= d.ctl->n_chunks) return;
    // tile b: the last with chunk_base[b] <= c
    int lo = 0, hi = g.nt - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (d.chunk_base[mid] <= c) lo = mid; else hi = mid - 1;
    }
    const int b = lo;
    const uint32_t ci = c - d.chunk_base[b];
    const uint32_t ev = d.ctl->acc_ev;
    // this block's events, by their offset: a catalog's event numbers reach 2^32 - 2,
    // and a step past the last one would wrap
    const uint32_t e0 = d.bbase[b] + ci * ev;
    const uint32_t ne = min(ev, d.bbase[b + 1] - e0);
    const int k0 = b * g.tile;
    if (g.prec == PREC_COMP) {
        accum_comp(g, d, b, ci, e0, ne, reinterpret_cast<FF *>(xn.h), reinterpret_cast<FF *>(dd.h));
        return;
    }
    for (int k = threadIdx.x; k < g.tile; k += ACC_T) {
        xn.h[k] = 0; xn.l[k] = 0;
        dd.h[k] = 0; dd.l[k] = 0;
    }
    __syncthreads();
    // AU events per thread in flight.  A hot tile's 65536 events are the whole
    // launch of a small catalog: 25 us with 512 threads and 8 events each in
    // flight, 51 with 256 and 4 (1e7 sources 57 and 91); 1024 threads leave one
    // block per CU, 27 and 69 us
    constexpr int AU = 8;
    for (uint32_t e = threadIdx.x; e < ne; e += AU * ACC_T) {
        uint32_t key[AU];
        int64_t v[AU];
#pragma unroll
        for (int q = 0; q < AU; ++q) {
            const uint32_t ee = e0 + min(e + (uint32_t)(q * ACC_T), ne - 1u);
            key[q] = d.ev_key[ee];
            v[q] = d.ev_val[ee];
        }
#pragma unroll
        for (int q = 0; q < AU; ++q) {
            if (e + (uint32_t)(q * ACC_T) >= ne) continue;
            const int k = (int)(key[q] & 0x7FFFFFFFu) - k0;
            split_add((key[q] >> 31) ? dd : xn, k, v[q]);
        }
    }
    __syncthreads();
    const int nbin = min(g.tile, g.B - k0);
    if (d.nch[b] == 1) {
        I128 s = zero_t<I128>();
        for (int k = threadIdx.x; k < g.tile; k += ACC_T) {
            if (k < nbin) {
                const I128 dk = split_total(dd, k);
                d.Xn[k0 + k] = split_total(xn, k);
                d.D[k0 + k] = dk;
                s = i128_add(s, dk);
            }
        }
        I128 tot;
        block_excl_scan<I128, ACC_T>(s, sh, &tot);
        if (threadIdx.x == 0) d.Dtile[b] = tot;
    } else {
        I128 *slot = d.partial + (size_t)(d.slot_base[b] + ci) * 2 * g.tile;
        for (int k = threadIdx.x; k < g.tile; k += ACC_T) {
            slot[k] = split_total(xn, k);
            slot[g.tile + k] = split_total(dd, k);
        }
    }
}

// Hot tiles (several accumulation blocks): sum the partials, RED_BINS bins
// per block.
__global__ __launch_bounds__(RED_BINS) void k_accum_reduce(const Slot *S)
{
    __shared__ I128 sh[RED_BINS / 64];
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    const int per = g.tile / RED_BINS;
    const int b = blockIdx.x / per, part = blockIdx.x % per;
    if (b >= g.nt) return;
    const uint32_t nc = d.nch[b];
    if (nc <= 1) return;
    const int k = part * RED_BINS + threadIdx.x;
    const int k0 = b * g.tile;
    const int nbin = min(g.tile, g.B - k0);
    if (g.prec == PREC_COMP) {
        // the chunks' double-fp32 partials in chunk order; the block's sum
        // of Dc goes to the tile sum by a compensated atomic
        __shared__ FF shc[RED_BINS / 64];
        const FF *slot = reinterpret_cast<const FF *>(d.partial + (size_t)d.slot_base[b] * 2 * g.tile);
        FF xs = ff_of(0.0f), ys = ff_of(0.0f);
        for (uint32_t c = 0; c < nc; ++c) {
            xs = ff_add(xs, slot[(size_t)c * 4 * g.tile + k]);
            ys = ff_add(ys, slot[(size_t)c * 4 * g.tile + g.tile + k]);
        }
        if (k < nbin) {
            d.Xc[k0 + k] = xs;
            d.Dc[k0 + k] = ys;
        } else {
            ys = ff_of(0.0f);
        }
        FF tot;
        block_excl_scan<FF, RED_BINS>(ys, shc, &tot);
        if (threadIdx.x == 0) {
            ff_atomic_add(&d.Dtc[b], tot.hi);
            ff_atomic_add(&d.Dtc[b], tot.lo);
        }
        return;
    }
    I128 x = zero_t<I128>(), y = zero_t<I128>();
    const I128 *slot = d.partial + (size_t)d.slot_base[b] * 2 * g.tile;
    constexpr uint32_t U = 8;              // partial sums in flight
    for (uint32_t s = 0; s < nc; s += U) {
        I128 p[U], q[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const I128 *o = slot + (size_t)min(s + u, nc - 1) * 2 * g.tile + k;
            p[u] = o[0];
            q[u] = o[g.tile];
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (s + u >= nc) continue;
            x = i128_add(x, p[u]);
            y = i128_add(y, q[u]);
        }
    }
    I128 dsum = zero_t<I128>();
    if (k < nbin) {
        d.Xn[k0 + k] = x;
        d.D[k0 + k] = y;
        dsum = y;
    }
    // block sum of D into the tile sum (one exact 128-bit atomic per block)
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    I128 inc = wave_incl_scan(dsum);
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        I128 t = zero_t<I128>();
        for (int w = 0; w < RED_BINS / 64; ++w) t = i128_add(t, sh[w]);
        atomic_add_i128_full(&d.Dtile[b], t);
    }
}

__global__ __launch_bounds__(WG) void k_dscan(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;

    block_scan_array<I128>(d.Dtile, d.Dcarry, g.nt);
    if (g.prec == PREC_NAIVE) {
        __syncthreads();
        block_scan_array<float>(d.Dtf, d.Dcf, g.nt);
    }
}

// Naive FP32 mode: the same events summed again in fp32, in whatever order
// the atomics land (the accumulation the paper's float scatter performs).
__global__ __launch_bounds__(WG) void k_zero_f32(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active || sl.g.prec != PREC_NAIVE) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    for (int i = blockIdx.x * WG + threadIdx.x; i <= g.B; i += gridDim.x * WG) {
        if (i < g.B) d.Xf[i] = 0.0f;
        d.Df[i] = 0.0f;
        if (i <= g.nt) d.Dtf[i] = 0.0f;
    }
}

__global__ __launch_bounds__(WG) void k_accum_f32(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active || sl.g.prec != PREC_NAIVE) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    const int L = fx_exp(d.ctl->amax_bits, g.T);
    const int sc = f32_scale(d.ctl->amax_bits, g.T);
    const uint32_t ne = d.ctl->n_events;
    for (uint64_t e = blockIdx.x * WG + threadIdx.x; e < ne; e += gridDim.x * WG) {
        const uint32_t key = d.ev_key[e];
        const float v = (float)ldexp((double)d.ev_val[e], L + sc);
        const int k = (int)(key & 0x7FFFFFFFu);
        if (key >> 31) {
            atomicAdd(&d.Df[k], v);
            atomicAdd(&d.Dtf[div_p2(k, g.tile)], v);
        } else {
            atomicAdd(&d.Xf[k], v);
        }
    }
}

// ------------------------------------------------------------------ X update

// X[k] = 2^L * (Xn[k] + prefix(D)[k]) for the tiles whose X changed.  D and
// Xn are read and X written in coalesced order; the in-tile prefix runs over
// thread-contiguous runs staged in LDS (one pad entry per 8 against bank
// conflicts).
DEVI int xpad(int i) { return i + (i >> 3); }

template <int NT> DEVI void snr_tail(const Slot &sl, bool converts);

// The compensated FP32 mode's X of one tile: X = Xc + (carry + in-tile
// prefix of Dc), every sum double-fp32, rounded once to fp32 at the end.
// The carry is the sum of the tile sums of Dc before the tile (kept current
// by the subtractions), added up here in a fixed order.  `st` is LDS for the
// tile (xpad layout).
DEVI void xupdate_comp(const Grid &g, const Dev &d, int tile, int t0, int n, int R, int b, FF *st)
{
    __shared__ FF shc[WG / 64];
    const int sc = f32_scale(d.ctl->amax_bits, g.T);
    FF c = ff_of(0.0f);
    for (int j = threadIdx.x; j < tile; j += WG) c = ff_add(c, d.Dtc[j]);
    FF carry;
    block_excl_scan(c, shc, &carry);
    for (int i = threadIdx.x; i < n; i += WG) st[xpad(i)] = d.Dc[t0 + i];
    __syncthreads();
    FF s = ff_of(0.0f);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (r < R && b + r < n) {
            s = ff_add(s, st[xpad(b + r)]);
            st[xpad(b + r)] = s;
        }
    }
    FF tot;
    const FF ex = ff_add(block_excl_scan(s, shc, &tot), carry);
#pragma unroll
    for (int r = 0; r < 8; ++r)
        if (r < R && b + r < n) st[xpad(b + r)] = ff_add(st[xpad(b + r)], ex);
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += WG)
        d.X[t0 + i] = ldexp((double)ff_float(ff_add(st[xpad(i)], d.Xc[t0 + i])), -sc);
}

// The last block of the grid is the tail of the previous k_snr; the other
// blocks convert the tiles stamped with the value k_snr published.  They
// touch disjoint data: the tail reads the partials and the stamps and
// writes the control block's counters and flags, while the converting
// blocks read the accumulators, the stamps and the control fields set
// before this launch (bad, xupd, amax_bits), never the settled flag.  Past the
// settled body no k_snr runs and the accumulators stay as they are: a body
// that settles the loop subtracted nothing and stamped nothing, and after a
// max_iter stop the tiles of the last stamp are only converted again to the
// same values.
__global__ __launch_bounds__(WG) void k_xupdate(const Slot *S)
{
    __shared__ I128 sh[WG / 64];
    __shared__ I128 stage[TILE_MAX + TILE_MAX / 8];
    __shared__ float shf[WG / 64];
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    if (blockIdx.x == gridDim.x - 1) {
        // ahead of the first body: every tile, and no tail
        if (threadIdx.x == 0 && sl.d.ctl->xupd == 0) sl.d.ctl->units_x = (uint64_t)sl.g.B;
        snr_tail<WG>(sl, true);
        return;
    }
    const Grid g = sl.g;
    const Dev d = sl.d;
    if (d.ctl->bad) return;
    const int tile = blockIdx.x;
    if (tile >= g.nt || d.xstamp[tile] != d.ctl->xupd) return;
    const int L = fx_exp(d.ctl->amax_bits, g.T);
    const int t0 = tile * g.tile;
    const int n = min(g.tile, g.B - t0);
    const int R = g.tile / WG;
    const int b = (int)threadIdx.x * R;
    if (g.prec == PREC_COMP) {
        xupdate_comp(g, d, tile, t0, n, R, b, reinterpret_cast<FF *>(stage));
        return;
    }
    for (int i = threadIdx.x; i < n; i += WG) stage[xpad(i)] = d.D[t0 + i];
    __syncthreads();
    I128 s = zero_t<I128>();
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (r < R && b + r < n) {
            s = i128_add(s, stage[xpad(b + r)]);
            stage[xpad(b + r)] = s;
        }
    }
    I128 tot;
    I128 ex = block_excl_scan(s, sh, &tot);
    ex = i128_add(ex, i128_add(d.Dcarry[tile], split_sum_value(d.Dadj[tile])));
#pragma unroll
    for (int r = 0; r < 8; ++r)
        if (r < R && b + r < n) stage[xpad(b + r)] = i128_add(stage[xpad(b + r)], ex);
    __syncthreads();
    if (g.prec == PREC_FP64) {
        for (int i = threadIdx.x; i < n; i += WG)
            d.X[t0 + i] = ldexp(i128_to_double(i128_add(stage[xpad(i)], d.Xn[t0 + i])), L);
        return;
    }
    const int sc = f32_scale(d.ctl->amax_bits, g.T);
    // naive fp32: X = Xf + prefix of Df, all in fp32
    __syncthreads();
    float *fst = reinterpret_cast<float *>(stage);
    for (int i = threadIdx.x; i < n; i += WG) fst[xpad(i)] = d.Df[t0 + i];
    __syncthreads();
    float fs = 0.0f;
    float floc[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (r < R && b + r < n) fs += fst[xpad(b + r)];
        floc[r] = fs;
    }
    float ftot;
    const float fex = block_excl_scan<float>(fs, shf, &ftot) + d.Dcf[tile];
#pragma unroll
    for (int r = 0; r < 8; ++r)
        if (r < R && b + r < n) fst[xpad(b + r)] = fex + floc[r];
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += WG) d.X[t0 + i] = ldexp((double)(d.Xf[t0 + i] + fst[xpad(i)]), -sc);
}

// ------------------------------------------------------------------ running median
//
// S[k] = C * median{X[a_k .. a_k+W-1]} + S_instr[k]   (Eq. "running median").
//
// One block per tile of `tile` outputs.  The union of the tile's windows
// (tile + W - 1 bins) is loaded once into LDS and sorted there: a stable LSD
// radix sort on a per-tile 18-bit order key (the fp64 bit pattern minus the
// tile minimum, shifted), then an exact repair that orders equal keys by
// the full fp64 value.  The sorted order is cut into buckets of 32 or 64
// consecutive ranks, and a bit matrix in LDS holds, for every bucket b and
// 64-position word, which positions have a rank up to the end of bucket b,
// with the count of such positions before the word.  The median of a window
// is the h-th smallest rank among its W positions: a binary search over the
// buckets (two counts per step) gives its bucket and its index there, and
// the bucket's sorted elements are tested against the window.  Each of the
// 512 threads answers its first window so, and its other R - 1 (R = tile/512, at
// most 4) by sliding: one element leaves, one enters, and the median stays or
// moves to a neighbour in the sorted order.
// Selection is exact: no arithmetic touches X.
//
// The kernel is bound by the latency of its LDS phases (two blocks per CU in
// a full-grid launch, one block's own chain in late bodies), so each phase is
// built for few dependent steps and barriers: two 9-bit radix passes ranked by
// ballots instead of five 4-bit ones with scanned counters, ties ordered by
// counting inside their run instead of odd-even rounds, and one atomic OR per
// element with two short scans instead of a stable partition per rank bit (a
// wavelet matrix).  1e7 catalog, W = 1001: 26.4 us a launch instead of 36.5,
// 17 instead of 25 in the late bodies, of which load 1.4, sort 4.5, ties 1-4,
// matrix 2.2, selection 2.3, outputs 1.2 and the launch itself 4.5.  8-bit
// passes (16-bit keys) sort in 4.1 us, but leave more ties than they save.

constexpr int MWG = 512;                    // threads of a median block
constexpr int RMAX = TILE_MAX / MWG;        // outputs per thread, at most
constexpr int MCH = MMAX / MWG;             // union elements per thread in the sort
constexpr int DGB = 9;                      // bits of a radix digit
constexpr int NDG = 1 << DGB;               // digits: one per thread in the scan
static_assert(NDG == MWG && KEYBITS == 2 * DGB, "the sort's scan and its two passes");
constexpr int RUN_MAX = 64;                 // longest run of equal keys that the repair orders by counting
constexpr int NBK = MMAX / 64;              // rank buckets, at most
constexpr int NWD = MMAX / 64 + 1;          // 64-position words (+1: the end position)

struct MedianSmem {
    double xv[MMAX];                       // X over the union, position order
    uint32_t kp[2][MMAX];                  // sort words: key << POSBITS | position
    union {
        uint32_t hist[2][MWG / 64][NDG / 2]; // radix: per-wave digit counts, then offsets, 16 bits each
                                            // (two buffers, for the passes in turn)
        struct {                            // rows of nw | 1 words
            uint64_t bits[NBK * (NWD | 1)]; // positions with a rank up to the end of the bucket
            uint16_t cnt[NBK * (NWD | 1)];  // such positions before the word
        } bm;
        double stage[TILE_MAX];            // outputs, for coalesced stores
    } u;
    uint32_t wsc[MWG / 64];                 // cross-wave exchange of the radix sort's scan
    uint32_t red[2][MWG / 64];              // smallest and largest X of each wave (high words)
    uint64_t fix[MMAX / 64];                // elements of the runs that the repair orders
    double dsh[MWG / 64];
    int flag;
};

// Stable LSD radix sort of the M words in sm.kp[0] by bits [POSBITS, POSBITS +
// DGB*passes), DGB bits per pass; returns the buffer holding the result.  A
// wave owns a contiguous range of the current order, 64 words at a time: a
// word's rank among the wave's equal digits is the wave's count so far plus
// the lower lanes with its digit (a ballot per bit).  The lowest lane of each
// digit adds the digit's count (the adds of all words are in flight together)
// and hands the count before it to the others.  The counts, scanned over
// (digit, wave), become the offsets.  The caller's stores to kp[0] need no
// barrier of their own.
DEVI int radix_sort_tile(MedianSmem &sm, int M, int passes)
{
    constexpr int NV = MWG / 64;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int CH = (M + MWG - 1) / MWG;
    const int seg = wave * CH * 64 + lane;
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < NV * NDG / 2 / MWG; ++q) (&sm.u.hist[0][0][0])[q * MWG + tid] = 0;
    __syncthreads();
    int in = 0;
    for (int ps = 0; ps < passes; ++ps) {
        const int sh = POSBITS + DGB * ps;
        const uint32_t *kin = sm.kp[in];
        uint32_t *kout = sm.kp[in ^ 1];
        uint32_t *hist = sm.u.hist[ps & 1][wave];
        uint32_t e[MCH], lr[MCH], old[MCH];
        int first[MCH];
#pragma unroll
        for (int c = 0; c < MCH; ++c)
            if (c < CH) e[c] = kin[min(seg + c * 64, M - 1)];
#pragma unroll
        for (int c = 0; c < MCH; ++c) {
            if (c >= CH) continue;
            const bool ok = seg + c * 64 < M;
            const uint32_t dg = (e[c] >> sh) & (NDG - 1u);
            const uint64_t in = (uint64_t)__ballot(ok);
            uint32_t plo = (uint32_t)in, phi = (uint32_t)(in >> 32);
#pragma unroll
            for (int bit = 0; bit < DGB; ++bit) {
                const uint32_t sg = (uint32_t)((int32_t)(dg << (31 - bit)) >> 31);     // the bit in every bit
                const uint64_t m = (uint64_t)__ballot(sg != 0);
                plo &= ~((uint32_t)m ^ sg);
                phi &= ~((uint32_t)(m >> 32) ^ sg);
            }
            const uint64_t peers = (uint64_t)phi << 32 | plo;
            lr[c] = (uint32_t)__popcll(peers & below);
            first[c] = __ffsll((unsigned long long)peers) - 1;
            old[c] = 0;
            if (ok && lr[c] == 0)
                old[c] = atomicAdd(&hist[dg >> 1], (uint32_t)__popcll(peers) << (16 * (dg & 1u)));
        }
#pragma unroll
        for (int c = 0; c < MCH; ++c) {
            if (c >= CH) continue;
            const uint32_t dg = (e[c] >> sh) & (NDG - 1u);
            lr[c] += ((uint32_t)__shfl((int)old[c], first[c] & 63, 64) >> (16 * (dg & 1u))) & 0xFFFFu;
        }
        __syncthreads();
        // exclusive scan over (digit, wave), thread = digit
        uint16_t(*h)[NDG] = reinterpret_cast<uint16_t(*)[NDG]>(&sm.u.hist[ps & 1][0][0]);
        {
            uint32_t c[NV], s = 0;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                c[v] = h[v][tid];
                s += c[v];
            }
            const uint32_t inc = wave_scan_u32(s);
            if (lane == 63) sm.wsc[wave] = inc;
            if (ps + 1 < passes) {
#pragma unroll
                for (int q = 0; q < NV * NDG / 2 / MWG; ++q) (&sm.u.hist[(ps & 1) ^ 1][0][0])[q * MWG + tid] = 0;
            }
            __syncthreads();
            uint32_t run = inc - s;
#pragma unroll
            for (int v = 0; v < NV; ++v) run += v < wave ? sm.wsc[v] : 0u;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                h[v][tid] = (uint16_t)run;
                run += c[v];
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < MCH; ++c)
            if (c < CH && seg + c * 64 < M) kout[h[wave][(e[c] >> sh) & (NDG - 1u)] + lr[c]] = e[c];
        __syncthreads();
        in ^= 1;
    }
    return in;
}

// In-part inclusive prefix of the values st[0 .. t1-t0) of a median block
// (thread-contiguous runs of R outputs; a part is part/R threads, whole
// waves), accumulated in type A; writes the prefix back into st and the part
// sums to is_psum.  Contains one barrier.
template <typename A>
DEVI void part_prefix(double *dsh, double *st, const Grid &g, const Dev &d, int kb, int ke, int t0,
                      int t1, int R)
{
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    A loc[RMAX], s = zero_t<A>();
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        if (kb + r < ke) s += (A)st[kb + r - t0];
        loc[r] = s;
    }
    const int segw = (g.part / R) >> 6;
    const A inc = wave_incl_scan(s);
    A exw = shfl_up_t(inc, 1);
    if (lane == 0) exw = zero_t<A>();
    A *xch = reinterpret_cast<A *>(dsh);
    if (lane == 63) xch[wave] = inc;
    __syncthreads();
    const int ws0 = (wave / segw) * segw;
    A pre = zero_t<A>(), tot = zero_t<A>();
#pragma unroll
    for (int w = 0; w < MWG / 64; ++w) {
        const A x = xch[w];
        if (w >= ws0 && w < wave) pre += x;
        if (w >= ws0 && w < ws0 + segw) tot += x;
    }
    const A ex = pre + exw;
#pragma unroll
    for (int r = 0; r < RMAX; ++r)
        if (kb + r < ke) st[kb + r - t0] = (double)(ex + loc[r]);
    if ((tid & (segw * 64 - 1)) == 0) {
        const int p0 = t0 + (tid / (segw * 64)) * g.part;
        if (p0 < t1) d.is_psum[div_p2(p0, g.part)] = (double)tot;
    }
}

// part_prefix in double-fp32 (compensated FP32 mode): st[] holds fp32
// reciprocals on entry; on exit each slot holds the FF prefix (its 8 bytes),
// and is_psum the FF part sums.  Contains one barrier.
DEVI void part_prefix_ff(double *dsh, double *st, const Grid &g, const Dev &d, int kb, int ke, int t0, int t1,
                         int R)
{
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    FF loc[RMAX], s = ff_of(0.0f);
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        if (kb + r < ke) s = ff_add(s, ff_of((float)st[kb + r - t0]));
        loc[r] = s;
    }
    const int segw = (g.part / R) >> 6;
    const FF inc = wave_incl_scan(s);
    FF exw = shfl_up_t(inc, 1);
    if (lane == 0) exw = ff_of(0.0f);
    FF *xch = reinterpret_cast<FF *>(dsh);
    if (lane == 63) xch[wave] = inc;
    __syncthreads();
    const int ws0 = (wave / segw) * segw;
    FF pre = ff_of(0.0f), tot = ff_of(0.0f);
#pragma unroll
    for (int w = 0; w < MWG / 64; ++w) {
        const FF x = xch[w];
        if (w >= ws0 && w < wave) pre = ff_add(pre, x);
        if (w >= ws0 && w < ws0 + segw) tot = ff_add(tot, x);
    }
    const FF ex = ff_add(pre, exw);
    FF *stf = reinterpret_cast<FF *>(st);
#pragma unroll
    for (int r = 0; r < RMAX; ++r)
        if (kb + r < ke) stf[kb + r - t0] = ff_add(ex, loc[r]);
    if ((tid & (segw * 64 - 1)) == 0) {
        const int p0 = t0 + (tid / (segw * 64)) * g.part;
        if (p0 < t1) reinterpret_cast<FF *>(d.is_psum)[div_p2(p0, g.part)] = tot;
    }
}

// Inclusive scan of 128-bit sums across the 64 lanes of a wave: x plus the sum
// that the DPP pattern C moves in (rows outside R get zero).
template <int C, int R> DEVI uint64_t dpp_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, C, R, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), C, R, 0xF, false);
    return (uint64_t)hi << 32 | lo;
}

template <int C, int R> DEVI I128 dpp_add(I128 x)
{
    I128 y;
    y.lo = dpp_u64<C, R>(x.lo);
    y.hi = (int64_t)dpp_u64<C, R>((uint64_t)x.hi);
    return i128_add(x, y);
}

DEVI I128 wave_scan_i128(I128 x)
{
    x = dpp_add<0x111, 0xF>(x);                        // row_shr:1, 2, 4, 8
    x = dpp_add<0x112, 0xF>(x);
    x = dpp_add<0x114, 0xF>(x);
    x = dpp_add<0x118, 0xF>(x);
    x = dpp_add<0x142, 0xA>(x);                        // row_bcast:15, 31
    return dpp_add<0x143, 0xC>(x);
}

// X over the union [u0, u1] of the windows of one part straight from the
// accumulators, X = 2^L (Xn + prefix(D)), for the launches that convert and
// filter at once: xr[i] = X of bin u0 + threadIdx.x + i MWG.  The sums are
// exact integers, so one prefix from the first tile's carry serves every
// tile of the union, and a converted bin equals what k_xupdate stores.  D
// goes through `st`, LDS of FST entries that may overlap anything else (the
// last barrier is past its last read): read in bin order, summed in runs of
// consecutive bins.  A part's range from its first tile's start is at most
// tile - 1 + part + W - 1 <= MMAX - 1 + PART_MAX bins.
constexpr int FCH = (MMAX - 1 + PART_MAX + MWG - 1) / MWG;   // bins per thread, at most (odd)
constexpr int FST = MMAX + PART_MAX;
DEVI void fresh_union(const Grid &g, const Dev &d, int u0, int u1, I128 *st, double (&xr)[MCH])
{
    __shared__ I128 sh[MWG / 64];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int tl = div_p2(u0, g.tile), first = tl * g.tile, len = u1 + 1 - first;
    const int CH = ((len + MWG - 1) / MWG) | 1;             // odd: a run's reads spread over the banks
    I128 v[FCH], xn[MCH];
#pragma unroll
    for (int i = 0; i < FCH; ++i)
        if (i * MWG < len) v[i] = d.D[first + min(tid + i * MWG, len - 1)];
#pragma unroll
    for (int i = 0; i < MCH; ++i)
        if (u0 + i * MWG <= u1) xn[i] = d.Xn[min(u0 + tid + i * MWG, u1)];
    const I128 carry = i128_add(d.Dcarry[tl], split_sum_value(d.Dadj[tl]));
    const int L = fx_exp(d.ctl->amax_bits, g.T);
#pragma unroll
    for (int i = 0; i < FCH; ++i)
        if (tid + i * MWG < len) st[tid + i * MWG] = v[i];
    __syncthreads();
    const int k0 = tid * CH;
    I128 s = zero_t<I128>();
#pragma unroll
    for (int i = 0; i < FCH; ++i) {
        v[i] = zero_t<I128>();
        if (i < CH && k0 + i < len) v[i] = st[k0 + i];
        s = i128_add(s, v[i]);
    }
    const I128 inc = wave_scan_i128(s);
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    // exclusive: the waves before, and inc - s
    I128 run = carry;
#pragma unroll
    for (int w = 0; w < MWG / 64; ++w) {
        const I128 x = sh[w];
        if (w < wave) run = i128_add(run, x);
    }
    run = i128_add(run, inc);
    I128 neg;
    neg.lo = ~s.lo + 1;
    neg.hi = (int64_t)(~(uint64_t)s.hi + (neg.lo == 0));
    run = i128_add(run, neg);
#pragma unroll
    for (int i = 0; i < FCH; ++i) {
        run = i128_add(run, v[i]);
        if (i < CH && k0 + i < len) st[k0 + i] = run;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MCH; ++i) {
        const int k = u0 + tid + i * MWG;
        if (k <= u1) xr[i] = ldexp(i128_to_double(i128_add(st[k - first], xn[i])), L);
    }
    __syncthreads();
}

// X over the union from the template model's data, X = (2/T) |h|^2, as
// fresh_union; the arithmetic is k_cx_power's.
DEVI void fresh_union_cx(const Slot &sl, int u0, int u1, double (&xr)[MCH])
{
    const Grid &g = sl.g;
    const int64_t *re = sl.d.h, *im = re + (size_t)g.B;
    int64_t a[MCH], b[MCH];
#pragma unroll
    for (int i = 0; i < MCH; ++i) {
        if (u0 + i * MWG > u1) continue;
        const int k = min(u0 + (int)threadIdx.x + i * MWG, u1);
        a[i] = re[k];
        b[i] = im[k];
    }
    const int E = cx_exp(sl.d.ctl->amax_bits, (uint32_t)sl.n, g.T);
    const double s2 = 2.0 / g.T;
#pragma unroll
    for (int i = 0; i < MCH; ++i) {
        if (u0 + i * MWG > u1) continue;
        const double x = ldexp((double)a[i], -E), y = ldexp((double)b[i], -E);
        xr[i] = s2 * (x * x + y * y);
    }
}

// The largest 1/S of the wave's 64-bin segment, which starts at bin k0 < t1 (lanes
// past the outputs bring 0): the bound that the template model's SNR pass uses.
DEVI void segment_max(const Dev &d, double inv, int k0, int t1)
{
    if (!d.is_max || k0 >= t1) return;                 // wave-uniform
    const uint32_t m = wave_max_u32((uint32_t)((uint64_t)__double_as_longlong(inv) >> 32));
    if (lane_id() == 63) d.is_max[k0 >> 6] = m;
}

// Where a PSD launch takes X from: the array (converted by an earlier launch),
// the accumulators, or the template model's data.
enum XSource { X_ARRAY, X_ACCUM, X_CX };

// The work of one tile (or part) of a PSD launch.  When X is converted here,
// the block stores the bins of its own outputs where their tile's X has changed.
template <XSource SRC>
DEVI void median_work(MedianSmem &sm, const Slot *slp, int blk, int span)
{
    const Grid g = slp->g;
    const Dev d = slp->d;
    const int tid = threadIdx.x;
    const int B = g.B, W = g.W, h = g.h;
    const int t0 = blk * span;
    const int t1 = min(t0 + span, B);
    const bool whole = B < W;
    const int u0 = whole ? 0 : win_start(t0, B, W, h);
    const int u1 = whole ? B - 1 : win_start(t1 - 1, B, W, h) + W - 1;
    const int M = u1 - u0 + 1;

    // ---- load the union and the outputs' S_instr (all loads in flight
    // together); bounds of the positive values, from the high words of the
    // fp64 patterns
    double xr[MCH], sxr[RMAX];
#pragma unroll
    for (int r = 0; r < RMAX; ++r) sxr[r] = d.sx[min(t0 + tid + r * MWG, t1 - 1)];
    if constexpr (SRC != X_ARRAY) {
        static_assert(FST * sizeof(I128) <= sizeof(MedianSmem), "fresh_union's LDS");
        const bool store = d.xstamp[div_p2(t0, g.tile)] == d.ctl->xupd;
        if constexpr (SRC == X_ACCUM)
            fresh_union(g, d, u0, u1, reinterpret_cast<I128 *>(&sm), xr);
        else
            fresh_union_cx(*slp, u0, u1, xr);
#pragma unroll
        for (int i = 0; i < MCH; ++i) {
            const int k = u0 + tid + i * MWG;
            if (store && k >= t0 && k < t1) d.X[k] = xr[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < MCH; ++i) {
            const int p = tid + i * MWG;
            xr[i] = p < M ? d.X[u0 + p] : 0.0;
        }
    }
    uint32_t mn32 = ~0u, mx32 = 0;
#pragma unroll
    for (int i = 0; i < MCH; ++i) {
        const int p = tid + i * MWG;
        if (p < M) {
            sm.xv[p] = xr[i];
            const uint64_t b = (uint64_t)__double_as_longlong(xr[i]);
            const uint32_t hi = (uint32_t)(b >> 32);
            mn32 = b != 0 ? min(mn32, hi) : mn32;
            mx32 = max(mx32, hi);
        }
    }
    mn32 = wave_min_u32(mn32);
    mx32 = wave_max_u32(mx32);
    if (lane_id() == 63) {
        sm.red[0][tid >> 6] = mn32;
        sm.red[1][tid >> 6] = mx32;
    }
    if (tid < MMAX / 64) sm.fix[tid] = 0;
    if (tid == 0) sm.flag = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < MWG / 64; ++w) {
        mn32 = min(w == 0 ? ~0u : mn32, sm.red[0][w]);
        mx32 = max(w == 0 ? 0u : mx32, sm.red[1][w]);
    }
    // order key: 0 for an empty bin, 1 + (bits - lower bound) >> shift
    // otherwise (X >= 0, so the fp64 bit patterns are in value order); empty
    // bins do not stretch the key range of the occupied ones
    const uint64_t mn = (uint64_t)mn32 << 32, mx = (uint64_t)mx32 << 32 | 0xFFFFFFFFull;
    const uint64_t vspan = mx > mn ? mx - mn : 0;
    const int span_bits = vspan ? 64 - __clzll(vspan) : 0;
    const int shift = span_bits > KEYBITS ? span_bits - KEYBITS : 0;
    constexpr uint64_t KMAX = (1ull << KEYBITS) - 1ull;
    auto key_of = [&](uint64_t b) -> uint32_t {       // the two largest keys share the last value
        const uint64_t k = 1ull + ((b - mn) >> shift);
        return b ? (uint32_t)(k < KMAX ? k : KMAX) : 0u;
    };
#pragma unroll
    for (int i = 0; i < MCH; ++i) {
        const int p = tid + i * MWG;
        if (p < M) sm.kp[0][p] = (key_of((uint64_t)__double_as_longlong(xr[i])) << POSBITS) | (uint32_t)p;
    }

    // ---- sort
    uint32_t *sw = sm.kp[radix_sort_tile(sm, M, 2)];

    // ---- repair key ties: order equal keys by (fp64 value, position).  A
    // neighbouring pair out of order marks its run of equal keys; the
    // elements of a marked run then find their places by counting.  (Long
    // runs are common where wide tracks leave plateaus of equal values, but
    // those are in order.)  A marked run of more than RUN_MAX elements
    // (an outlier can stretch the key range that far) has the tile sorted
    // again by all its bits, KEYBITS at a time from the lowest.
    {
        constexpr int U = 4;                           // words looked at together
        auto bits_of = [&](uint32_t w) { return (uint64_t)__double_as_longlong(sm.xv[w & 0xFFFu]); };
        uint32_t mine[MCH];
        int todo = 0;
#pragma unroll
        for (int j = 0; j < MCH; ++j) {
            const int i = tid + j * MWG;
            mine[j] = sw[min(i, M - 1)];
            const uint32_t nx = sw[min(i + 1, M - 1)];
            if (i + 1 < M && ((mine[j] ^ nx) >> POSBITS) == 0 && bits_of(mine[j]) > bits_of(nx)) todo |= 1 << j;
        }
        for (int j = 0; todo >> j; ++j) {
            if (!((todo >> j) & 1)) continue;
            const int i = tid + j * MWG;
            const uint32_t key = sw[i] >> POSBITS;
            int l = i, r = i + 1;                      // the run's ends, U words ahead at a time
            for (bool on = true; on && r - l < RUN_MAX;) {
                uint32_t w[U];
#pragma unroll
                for (int u = 0; u < U; ++u) w[u] = sw[max(l - 1 - u, 0)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    on = on && l > 0 && (w[u] >> POSBITS) == key;
                    l -= on;
                }
            }
            for (bool on = true; on && r - l < RUN_MAX;) {
                uint32_t w[U];
#pragma unroll
                for (int u = 0; u < U; ++u) w[u] = sw[min(r + 1 + u, M - 1)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    on = on && r + 1 < M && (w[u] >> POSBITS) == key;
                    r += on;
                }
            }
            atomicOr(&sm.flag, r - l >= RUN_MAX ? 2 : 1);
            if (r - l >= RUN_MAX) break;
            const uint64_t ones = (2ull << (r - l)) - 1ull;
            atomicOr((unsigned long long *)&sm.fix[l >> 6], ones << (l & 63));
            if ((l >> 6) != (r >> 6)) atomicOr((unsigned long long *)&sm.fix[r >> 6], ones >> (64 - (l & 63)));
        }
        __syncthreads();
        const int flag = sm.flag;
        if (flag == 1) {                               // places by counting
            int at[MCH];
#pragma unroll
            for (int j = 0; j < MCH; ++j) {
                const int i = tid + j * MWG;
                at[j] = -1;
                if (i >= M || !((sm.fix[i >> 6] >> (i & 63)) & 1ull)) continue;
                const uint32_t key = mine[j] >> POSBITS;
                const uint64_t b = bits_of(mine[j]);
                int n = i;
                for (int l = i - 1, on = 1; on; l -= U) {
                    uint32_t w[U];
                    uint64_t x[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        w[u] = sw[max(l - u, 0)];
                        x[u] = bits_of(w[u]);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        on = on && l - u >= 0 && (w[u] >> POSBITS) == key;
                        n -= on && x[u] > b;
                    }
                }
                for (int r = i + 1, on = 1; on; r += U) {
                    uint32_t w[U];
                    uint64_t x[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        w[u] = sw[min(r + u, M - 1)];
                        x[u] = bits_of(w[u]);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        on = on && r + u < M && (w[u] >> POSBITS) == key;
                        n += on && x[u] < b;
                    }
                }
                at[j] = n;
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < MCH; ++j)
                if (at[j] >= 0) sw[at[j]] = mine[j];
            __syncthreads();
        } else if (flag) {
            for (int p = tid; p < M; p += MWG) sw[p] = (uint32_t)p;
            for (int lev = (shift + KEYBITS - 1) / KEYBITS; lev >= 0; --lev) {
                __syncthreads();
                const int top = lev ? shift - KEYBITS * (lev - 1) : 0, lo = top > KEYBITS ? top - KEYBITS : 0;
                uint32_t w[MCH];
#pragma unroll
                for (int i = 0; i < MCH; ++i) {
                    const uint32_t q = sw[min(tid + i * MWG, M - 1)] & 0xFFFu;
                    const uint64_t bp = (uint64_t)__double_as_longlong(sm.xv[q]);
                    const uint64_t v = lev ? ((bp - mn) >> lo) & ((1ull << (top - lo)) - 1ull)
                                           : 1ull + ((bp - mn) >> shift);      // KEYBITS + 1 bits
                    w[i] = ((bp ? (uint32_t)v : 0u) << POSBITS) | q;
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < MCH; ++i)
                    if (tid + i * MWG < M) sm.kp[0][tid + i * MWG] = w[i];
                sw = sm.kp[radix_sort_tile(sm, M, lev ? 2 : 3)];
            }
        }
    }

    const int R = (span + MWG - 1) / MWG;
    const int kb = t0 + tid * R;
    const int ke = min(kb + R, t1);
    double med[RMAX];
    if (whole) {
        const double m = sm.xv[sw[(B + 1) / 2 - 1] & 0xFFFu];
#pragma unroll
        for (int r = 0; r < RMAX; ++r) med[r] = m;
    } else {
        // ---- bit matrix of the sorted order: buckets of 2^WB ranks (32 in
        // split mode, whose unions are short enough)
        constexpr int NV = MWG / 64;
        const int lane = lane_id();
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int WB = M <= 32 * NBK ? 5 : 6;
        const int nb = (M + (1 << WB) - 1) >> WB;
        const int nw = (M >> 6) + 1;                   // with the word of the end position
        const int rw = nw | 1;                         // odd rows: a column's words spread over the banks
        uint64_t *const bits = sm.u.bm.bits;
        uint16_t *const cnt = sm.u.bm.cnt;
        for (int i = tid; i < nb * rw; i += MWG) bits[i] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < MCH; ++j) {
            const int i = j * MWG + tid;
            if (i >= M) continue;
            const uint32_t q = sw[i] & 0xFFFu;
            atomicOr((unsigned long long *)&bits[(i >> WB) * rw + (int)(q >> 6)], 1ull << (q & 63u));
        }
        __syncthreads();
        // each word's bits over the buckets (lane = bucket): the rows are
        // disjoint, so the sums of the halves are their ORs
        constexpr int NC = (NWD + NV - 1) / NV;        // columns per wave, at most
        {
            uint64_t v[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q)
                v[q] = wave + q * NV < nw && lane < nb ? bits[lane * rw + wave + q * NV] : 0ull;
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                const int w = wave + q * NV;
                if (w >= nw) continue;
                const uint64_t c = (uint64_t)wave_scan_u32((uint32_t)(v[q] >> 32)) << 32 | wave_scan_u32((uint32_t)v[q]);
                if (lane < nb) {
                    bits[lane * rw + w] = c;
                    cnt[lane * rw + w] = (uint16_t)__popcll(c);
                }
            }
        }
        __syncthreads();
        {
            constexpr int NR = (NBK + NV - 1) / NV;    // rows per wave, at most (lane = word)
            uint32_t c[NR];
#pragma unroll
            for (int q = 0; q < NR; ++q)
                c[q] = wave + q * NV < nb && lane < nw ? cnt[(wave + q * NV) * rw + lane] : 0u;
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                const uint32_t inc = wave_scan_u32(c[q]);
                if (wave + q * NV < nb && lane < nw) cnt[(wave + q * NV) * rw + lane] = (uint16_t)(inc - c[q]);
            }
        }
        __syncthreads();

        // ---- median of each window: the h-th smallest rank (0-based) among
        // positions [a, a + W) of the union.  A thread's first window: the
        // matrix gives its bucket and its index among the window's elements
        // in the bucket; the bucket's sorted elements are then tested
        // against the window.  Each next window of the thread is the
        // previous one moved by one position (or the same one, at a grid
        // edge): one element leaves, one enters, and the median stays or
        // becomes the nearest element above or below it in sorted order
        // whose position lies in the new window, found by walking the
        // sorted words (at most SLIDE_MAX steps, else the matrix again).
        // The sorted order is (fp64 value, position) in lexicographic
        // order, so comparisons with the median need no ranks.
        auto query = [&](int a) -> int {               // sorted index of the median of [a, a + W)
            const int wa = a >> 6, we = (a + W) >> 6;
            const uint64_t ma = (1ull << (a & 63)) - 1ull, me = (1ull << ((a + W) & 63)) - 1ull;
            auto upto = [&](int b) -> int {            // the window's elements up to the end of bucket b
                const int r = b * rw;
                return (int)cnt[r + we] + __popcll(bits[r + we] & me) - (int)cnt[r + wa] - __popcll(bits[r + wa] & ma);
            };
            int lo = 0, hi = nb - 1, kk = h;           // the first bucket with more than h up to its end
            while (lo < hi) {
                const int mid = (lo + hi) >> 1, c = upto(mid);
                if (c > h) {
                    hi = mid;
                } else {
                    lo = mid + 1;
                    kk = h - c;
                }
            }
            const int base = lo << WB;                 // 2^WB words: inside kp (MMAX is a multiple of 64)
            uint64_t mask = 0;
            for (int i0 = 0; i0 < (1 << WB); i0 += 4) {
                const uint4 q4 = *reinterpret_cast<const uint4 *>(&sw[base + i0]);
                const uint32_t qq[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool act = base + i0 + c < M && (qq[c] & 0xFFFu) - (uint32_t)a < (uint32_t)W;
                    mask |= (uint64_t)act << (i0 + c);
                }
            }
            // position of the (kk+1)-th set bit
            int pos = 0;
#pragma unroll
            for (int wdt = 32; wdt >= 1; wdt >>= 1) {
                const int c = __popcll(mask & ((1ull << wdt) - 1ull));
                if (kk >= c) {
                    kk -= c;
                    mask >>= wdt;
                    pos += wdt;
                }
            }
            return base + pos;
        };
        // (value bits, position) of union position p before that of q
        auto before = [&](int p, int q) -> bool {
            const uint64_t bp = (uint64_t)__double_as_longlong(sm.xv[p]);
            const uint64_t bq = (uint64_t)__double_as_longlong(sm.xv[q]);
            return bp < bq || (bp == bq && p < q);
        };
        constexpr int SLIDE_MAX = 16, SLIDE_U = 4;
        int qm[RMAX];
        int ap = kb < ke ? win_start(min(kb, ke - 1), B, W, h) - u0 : 0;
        qm[0] = query(ap);
#pragma unroll
        for (int r = 1; r < RMAX; ++r) {
            if (r >= R) break;                          // R is the same for the whole block
            const int k = min(kb + r, ke - 1);          // past the run: repeat its last window
            const int a = kb < ke ? win_start(k, B, W, h) - u0 : 0;
            int m = qm[r - 1];
            if (a != ap) {                              // a == ap + 1: ap leaves, ap + W enters
                const int pm = (int)(sw[m] & 0xFFFu);
                const int po = ap, pi = ap + W;
                int dir = 0;                            // +1: the next element above; -1: below
                if (po == pm) {
                    dir = before(pi, pm) ? -1 : 1;
                } else {
                    const bool ob = before(po, pm), ib = before(pi, pm);
                    if (ob != ib) dir = ob ? 1 : -1;
                }
                if (dir != 0) {
                    // an element on that side lies in the new window (the one
                    // that entered, or the one below or above that took the
                    // median's place), so the walk stays inside [0, M)
                    int c = m, found = -1;
                    for (int st = 0; st < SLIDE_MAX && found < 0; st += SLIDE_U, c += SLIDE_U * dir) {
                        uint32_t w[SLIDE_U];           // past the ends: repeated, never taken
#pragma unroll
                        for (int u = 0; u < SLIDE_U; ++u) w[u] = sw[min(max(c + (u + 1) * dir, 0), M - 1)];
#pragma unroll
                        for (int u = SLIDE_U - 1; u >= 0; --u)
                            if ((w[u] & 0xFFFu) - (uint32_t)a < (uint32_t)W) found = c + (u + 1) * dir;
                    }
                    m = found >= 0 ? found : query(a);
                }
            }
            qm[r] = m;
            ap = a;
        }
#pragma unroll
        for (int r = 0; r < RMAX; ++r) med[r] = (kb + r < ke && r < R) ? sm.xv[sw[qm[r]] & 0xFFFu] : 0.0;
    }

    // ---- S = C med + S_instr; in-part prefix of 1/S and the part sums.  With
    // one output per thread, from registers
    if (R == 1 && g.prec == PREC_FP64) {
        const int lane = lane_id(), wave = tid >> 6;
        const bool on = kb < ke;
        const double Sk = g.C * med[0] + sxr[0], inv = on ? 1.0 / Sk : 0.0;
        if (on) d.S[kb] = Sk;
        segment_max(d, inv, t0 + wave * 64, t1);
        const double inc = wave_incl_scan(inv);
        double exw = __shfl_up(inc, 1, 64);
        if (lane == 0) exw = 0.0;
        if (lane == 63) sm.dsh[wave] = inc;
        __syncthreads();
        double pre = 0.0, tot = 0.0;                   // span is one part here
#pragma unroll
        for (int w = 0; w < MWG / 64; ++w) {
            const double x = sm.dsh[w];
            if (w < wave) pre += x;
            if (w < span / 64) tot += x;
        }
        if (on) d.is_pre[kb] = (pre + exw) + inv;
        if (tid == 0) d.is_psum[div_p2(t0, g.part)] = tot;
        return;
    }
    // the outputs pass through LDS so that global loads and stores are coalesced
    __syncthreads();                       // the bit matrix is dead: reuse it
    double *st = sm.u.stage;
    const int sc = g.prec == PREC_FP64 ? 0 : f32_scale(d.ctl->amax_bits, g.T);
    const int n = t1 - t0;
#pragma unroll
    for (int r = 0; r < RMAX; ++r)
        if (kb + r < ke) st[kb + r - t0] = med[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        const int i = tid + r * MWG;
        double inv = 0.0;
        if (i < n) {
            double Sk;
            if (g.prec == PREC_FP64) {
                Sk = g.C * st[i] + sxr[r];
                inv = 1.0 / Sk;
            } else {                       // S and 1/S in fp32, scaled by 2^sc
                const float sf = (float)g.C * (float)ldexp(st[i], sc) + (float)ldexp(sxr[r], sc);
                Sk = ldexp((double)sf, -sc);
                inv = (double)(1.0f / sf);
            }
            d.S[t0 + i] = Sk;
            st[i] = inv;
        }
        segment_max(d, inv, t0 + (i & ~63), t1);
    }
    __syncthreads();
    // prefix of 1/S restarted at every part: fp64 sums, double-fp32 sums in
    // the compensated FP32 mode, plain fp32 sums in the naive one
    if (g.prec == PREC_NAIVE)
        part_prefix<float>(sm.dsh, st, g, d, kb, ke, t0, t1, R);
    else if (g.prec == PREC_COMP)
        part_prefix_ff(sm.dsh, st, g, d, kb, ke, t0, t1, R);
    else
        part_prefix<double>(sm.dsh, st, g, d, kb, ke, t0, t1, R);
    __syncthreads();
    for (int i = tid; i < n; i += MWG) d.is_pre[t0 + i] = st[i];
}

// One block per tile, or (split mode, chosen by the previous body's SNR
// launch when few tiles are dirty) one block per part: more, shorter
// blocks; a block whose tile is clean exits.  The launch of one slot.
__global__ __launch_bounds__(MWG, 2) void k_median(const Slot *S)
{
    __shared__ MedianSmem sm;
    const Slot &sl = S[blockIdx.y];
    if (!sl.active || sl.g.est != 0) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    if (d.ctl->done || d.ctl->bad) return;
    const bool split = d.ctl->med_split != 0;
    const int span = split ? g.part : g.tile;
    const int blk = blockIdx.x;
    const int tile = split ? blk / g.np : blk;
    if (tile >= g.nt || blk * span >= g.B || d.sstamp[tile] != d.ctl->iter) return;
    median_work<X_ARRAY>(sm, &sl, blk, span);
}

// A body's X update, PSD and the previous body's tail in one launch (one FP64
// slot, or the template model's two channels; few dirty tiles): block 0 is the tail of the k_snr before it,
// the others take a part each, convert its union from the accumulators and
// filter it.  They touch disjoint data: the blocks read the accumulators, the
// stamps and the control fields set before the launch (xupd, the stamp of this
// body, among them) and write X, S and the prefixes of their own parts; the
// tail reads the partials and stamps and writes the counters, flags and list.
// Past the settled body no tile carries the stamp.  An empty launch costs
// 4.5 us and k_xupdate's late ones 9.5; the conversion adds 3 us to a part's
// chain, so a late body of the 1e7 catalog takes 29 us instead of 35 (median
// 17, SNR 8.5, X update 9.5), and one of the running mean 19 instead of 26.  A
// part reads 32 bytes of accumulators per bin, from its first tile's start,
// where the two launches read 8 of X; taken while the dirty tiles of the body
// before fit the split budget (pace_two; at most one wave of part-sized blocks on
// the chip), where the launch is latency, not traffic.  Runs of the 1e7
// catalog, 7 full and 15 late bodies: 1557 us by the rule, 1629 with three
// launches always, 1840 with two always (40 us more a full body); running mean
// 1218, 1340 and 1374; template model 3302, 3419 and 3908.  (Template model: X
// needs no prefix, and the X update and tail launches it saves took 7.4 and 6.1
// us a body.)
//
// Blocks and parts.  One slot: a block per part of the grid, and those of clean
// tiles exit (7372 blocks, 7.5 us when all do, 5 with the 512 of the split
// budget).  Two channels: twice the blocks (14 us), so the blocks, one per part
// of the budget, look their parts up among the stamps (the list is not made
// yet); should a body have more entries than blocks, they stride over them.
// The lookup takes 1.5 us of a block's chain: late launches of the 1e7 catalogs
// 20 us with it instead of 24 for two channels, 21 instead of 20 for one slot
// (running mean 13 instead of 11).
template <int NT> DEVI void snr_tail(const Slot &sl, bool converts);
template <int NT> DEVI void cx_tail(const Slot &sl);

// The n-th tile (from 0, in tile order) whose stamp is val (-1: there are not as
// many), and the number of such tiles.  Blocks of MWG threads; contains barriers.
DEVI int nth_stamped(const Grid &g, const uint32_t *stamp, uint32_t val, int n, int *total)
{
    constexpr int NV = MWG / 64, TW = 4;
    __shared__ int s_cnt[2][NV];
    __shared__ int s_tile;
    const int tid = threadIdx.x, wave = tid >> 6;
    int seen = 0;                                      // block-uniform
    if (tid == 0) s_tile = -1;
    for (int base = 0, rd = 0; base < g.nt; base += MWG * TW, rd ^= 1) {
        const int t0 = base + tid * TW;
        uint32_t st[TW];
#pragma unroll
        for (int q = 0; q < TW; ++q) st[q] = stamp[min(t0 + q, g.nt - 1)];
        uint32_t mask = 0;
#pragma unroll
        for (int q = 0; q < TW; ++q) mask |= (t0 + q < g.nt && st[q] == val ? 1u : 0u) << q;
        const int own = __popc(mask), inc = (int)wave_scan_u32((uint32_t)own);
        if (lane_id() == 63) s_cnt[rd][wave] = inc;
        __syncthreads();
        int at = seen + inc - own;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int x = s_cnt[rd][v];
            at += v < wave ? x : 0;
            seen += x;
        }
        if (n >= at && n < at + own) {
            for (int q = at; q < n; ++q) mask &= mask - 1;
            s_tile = t0 + __builtin_ctz(mask);
        }
    }
    __syncthreads();
    *total = seen;
    return s_tile;
}

// The part of entry e of the body stamped xupd (-1: past its last), and the
// number of its entries.
DEVI int next_part(const Grid &g, const Dev &d, int e, int *n)
{
    int tiles;
    const int tile = nth_stamped(g, d.sstamp, d.ctl->xupd, e / g.np, &tiles);
    *n = tiles * g.np;
    return tile < 0 ? -1 : tile * g.np + e % g.np;
}

// A block's entries beyond its first (rare: not inlined, so that the loop does
// not cost the first one registers).
template <typename M, typename W> __device__ __noinline__ void next_entries(M &sm, const Slot *slp, int e, W work)
{
    for (int n;;) {
        e += (int)gridDim.x - 1;
        __syncthreads();                               // LDS is reused by the next entry
        const int blk = next_part(slp->g, slp->d, e, &n);
        if (blk < 0) return;
        if (blk * slp->g.part < slp->g.B) work(sm, slp, blk);
    }
}

template <XSource SRC> __global__ __launch_bounds__(MWG, 4) void k_median_next(const Slot *S)
{
    __shared__ MedianSmem sm;
    const Slot &sl = S[blockIdx.y];
    if (blockIdx.x == 0) {
        if constexpr (SRC == X_CX) {
            if (blockIdx.y == 0) cx_tail<MWG>(sl);
        } else {
            snr_tail<MWG>(sl, false);
        }
        return;
    }
    if (sl.d.ctl->bad) return;
    const Grid g = sl.g;
    const int e = (int)blockIdx.x - 1;
    if constexpr (SRC == X_CX) {
        int n;
        const int blk = next_part(g, sl.d, e, &n);
        if (blk < 0) return;
        if (blk * g.part < g.B) median_work<SRC>(sm, &sl, blk, g.part);
        if (e + (int)gridDim.x - 1 >= n) return;
        next_entries(sm, &sl, e, [](MedianSmem &m, const Slot *p, int k) { median_work<SRC>(m, p, k, p->g.part); });
    } else if (sl.d.sstamp[e / g.np] == sl.d.ctl->xupd) {
        median_work<SRC>(sm, &sl, e, g.part);
    }
}

// The launch of several slots (batches, the template model's two channels):
// the dirty tiles come listed in tile order by the previous body's tail
// (every tile for the first body) and each block takes an entry, so the
// working blocks are dispatched first and a slot's clean tiles cost few
// blocks: the grid holds the longest list a body can have, Dims::maxlist.
// (A grid of 2048 blocks striding over the list had to call the work as a
// function, with spilled registers: 42.7 instead of 39.3 us a launch of the
// template model's 1e7 run.)
__global__ __launch_bounds__(MWG, 2) void k_median_listed(const Slot *S)
{
    __shared__ MedianSmem sm;
    const Slot &sl = S[blockIdx.y];
    if (!sl.active || sl.g.est != 0) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    if (d.ctl->done || d.ctl->bad) return;
    const bool split = d.ctl->med_split != 0;
    const int span = split ? g.part : g.tile;
    const int e = blockIdx.x;
    if (e >= (int)d.ctl->n_sdl * (split ? g.np : 1)) return;
    const int tile = (int)d.sdl[split ? e / g.np : e];
    const int blk = split ? tile * g.np + e % g.np : tile;
    if (blk * span < g.B) median_work<X_ARRAY>(sm, &sl, blk, span);
}

// ------------------------------------------------------------------ running mean
//
// S[k] = (1/W) sum_{j in window(k)} (X[j] + S_instr[j])   (the mean form of the
// PSD estimate, as printed: S_instr inside the sum).  Same tiles, parts,
// dirty stamps and outputs as the median; the window sums are differences of
// an in-LDS prefix over the block's union, so no sum runs across the grid.

struct MeanSmem {
    double v[MMAX];                        // X + S_instr over the union, then its inclusive prefix
    double stage[TILE_MAX];                // outputs, for coalesced stores
    double dsh[MWG / 64];
};

// The work of one tile (or part) of a PSD launch.
template <XSource SRC>
DEVI void mean_work(MeanSmem &sm, const Slot *slp, int blk, int span, I128 *st = nullptr)
{
    const Grid g = slp->g;
    const Dev d = slp->d;
    const int tid = threadIdx.x;
    const int B = g.B, W = g.W, h = g.h;
    const int t0 = blk * span;
    const int t1 = min(t0 + span, B);
    const bool whole = B < W;
    const int u0 = whole ? 0 : win_start(t0, B, W, h);
    const int u1 = whole ? B - 1 : win_start(t1 - 1, B, W, h) + W - 1;
    const int M = u1 - u0 + 1;

    if constexpr (SRC != X_ARRAY) {
        const bool store = d.xstamp[div_p2(t0, g.tile)] == d.ctl->xupd;
        double xr[MCH];
        if constexpr (SRC == X_ACCUM)
            fresh_union(g, d, u0, u1, st, xr);
        else
            fresh_union_cx(*slp, u0, u1, xr);
#pragma unroll
        for (int i = 0; i < MCH; ++i) {
            const int p = tid + i * MWG;
            if (p >= M) continue;
            sm.v[p] = xr[i] + d.sx[u0 + p];
            if (store && u0 + p >= t0 && u0 + p < t1) d.X[u0 + p] = xr[i];
        }
    } else {
        for (int p = tid; p < M; p += MWG) sm.v[p] = d.X[u0 + p] + d.sx[u0 + p];
    }
    __syncthreads();
    // inclusive prefix over the union: thread-contiguous runs
    const int ch = (M + MWG - 1) / MWG;
    const int pb = tid * ch;
    double loc[MCH], s = 0.0;
#pragma unroll
    for (int i = 0; i < MCH; ++i) {
        if (i < ch && pb + i < M) s += sm.v[pb + i];
        loc[i] = s;
    }
    double tot;
    const double ex = block_excl_scan<double, MWG>(s, sm.dsh, &tot);
#pragma unroll
    for (int i = 0; i < MCH; ++i)
        if (i < ch && pb + i < M) sm.v[pb + i] = ex + loc[i];
    __syncthreads();
    const int n = t1 - t0;
    for (int i = tid; i - lane_id() < n; i += MWG) {   // whole waves
        const int k = t0 + i;
        double inv = 0.0;
        if (i < n) {
            double sum, len;
            if (whole) {
                sum = sm.v[M - 1];
                len = (double)B;
            } else {
                const int a = win_start(k, B, W, h) - u0;
                sum = sm.v[a + W - 1] - (a > 0 ? sm.v[a - 1] : 0.0);
                len = (double)W;
            }
            const double Sk = sum / len;
            d.S[k] = Sk;
            inv = 1.0 / Sk;
            sm.stage[i] = inv;
        }
        segment_max(d, inv, t0 + (i & ~63), t1);
    }
    __syncthreads();
    const int R = (span + MWG - 1) / MWG;
    const int kb = t0 + tid * R;
    const int ke = min(kb + R, t1);
    part_prefix<double>(sm.dsh, sm.stage, g, d, kb, ke, t0, t1, R);
    __syncthreads();
    for (int i = tid; i < n; i += MWG) d.is_pre[t0 + i] = sm.stage[i];
}

// One block per tile, or (split mode, chosen by the previous body's SNR
// launch when few tiles are dirty) one block per part: more, shorter
// blocks; a block whose tile is clean exits.  The launch of one slot.
__global__ __launch_bounds__(MWG) void k_mean(const Slot *S)
{
    __shared__ MeanSmem sm;
    const Slot &sl = S[blockIdx.y];
    if (!sl.active || sl.g.est != 1) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    if (d.ctl->done || d.ctl->bad) return;
    const bool split = d.ctl->med_split != 0;
    const int span = split ? g.part : g.tile;
    const int blk = blockIdx.x;
    const int tile = split ? blk / g.np : blk;
    if (tile >= g.nt || blk * span >= g.B || d.sstamp[tile] != d.ctl->iter) return;
    mean_work<X_ARRAY>(sm, &sl, blk, span);
}

// As k_median_next.
template <XSource SRC> __global__ __launch_bounds__(MWG, 4) void k_mean_next(const Slot *S)
{
    __shared__ union {
        MeanSmem mean;
        I128 st[SRC == X_ACCUM ? FST : 1];
    } sm;
    const Slot &sl = S[blockIdx.y];
    if (blockIdx.x == 0) {
        if constexpr (SRC == X_CX) {
            if (blockIdx.y == 0) cx_tail<MWG>(sl);
        } else {
            snr_tail<MWG>(sl, false);
        }
        return;
    }
    if (sl.d.ctl->bad) return;
    const Grid g = sl.g;
    const int e = (int)blockIdx.x - 1;
    if constexpr (SRC == X_CX) {
        int n;
        const int blk = next_part(g, sl.d, e, &n);
        if (blk < 0) return;
        if (blk * g.part < g.B) mean_work<SRC>(sm.mean, &sl, blk, g.part, sm.st);
        if (e + (int)gridDim.x - 1 >= n) return;
        next_entries(sm, &sl, e, [](auto &m, const Slot *p, int k) { mean_work<SRC>(m.mean, p, k, p->g.part, m.st); });
    } else if (sl.d.sstamp[e / g.np] == sl.d.ctl->xupd) {
        mean_work<SRC>(sm.mean, &sl, e, g.part, sm.st);
    }
}

// The launch of several slots, as k_median_listed.
__global__ __launch_bounds__(MWG) void k_mean_listed(const Slot *S)
{
    __shared__ MeanSmem sm;
    const Slot &sl = S[blockIdx.y];
    if (!sl.active || sl.g.est != 1) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    if (d.ctl->done || d.ctl->bad) return;
    const bool split = d.ctl->med_split != 0;
    const int span = split ? g.part : g.tile;
    const int e = blockIdx.x;
    if (e >= (int)d.ctl->n_sdl * (split ? g.np : 1)) return;
    const int tile = (int)d.sdl[split ? e / g.np : e];
    const int blk = split ? tile * g.np + e % g.np : tile;
    if (blk * span < g.B) mean_work<X_ARRAY>(sm, &sl, blk, span);
}

// ------------------------------------------------------------------ SNR, decisions, subtraction

// Sum of 1/S over bins lo..hi from the in-part prefixes of 1/S and `mid`,
// the sum of the part sums of the parts plo .. phi-1 (plo, phi: the parts
// of lo and hi); short tracks are summed bin by bin in ascending order.
DEVI double track_inv_sum(const double *v, const double *pre, int lo, int hi, int part, double mid)
{
    if (hi - lo + 1 <= NARROW) {
        double s = 0.0;
        for (int k = lo; k <= hi; k += 4) {            // four bins' loads at a time, summed in order
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = v[min(k + u, hi)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k + u <= hi) s += 1.0 / x[u];
        }
        return s;
    }
    const double below = mod_p2(lo, part) == 0 ? 0.0 : pre[lo - 1];
    if (div_p2(lo, part) == div_p2(hi, part)) return pre[hi] - below;
    return (mid - below) + pre[hi];
}

// rho^2 in fp32 (the FP32 precision modes): 4 q sum 1/S with the sum in
// fp32.  Compensated: Kahan over short tracks, and for longer ones
// double-fp32 differences of the double-fp32 in-part prefixes plus midc, the
// double-fp32 sum of the part sums in between.  Naive: plain fp32 (bin by
// bin, or the fp32 in-part prefixes and the fp32 sum `mid` of the part sums).
DEVI double snr2_f32(const Grid &g, const Dev &d, double qd, int lo, int hi, double mid, FF midc)
{
    // q and S scaled by 2^sc; the prefix tables already hold 1/(2^sc S)
    const int sc = f32_scale(d.ctl->amax_bits, g.T);
    const float q = (float)ldexp(qd, sc);
    float sum;
    if (hi - lo + 1 <= NARROW) {
        float s = 0.0f, c = 0.0f;
        for (int k = lo; k <= hi; ++k) {
            const float x = 1.0f / (float)ldexp(d.S[k], sc);
            if (g.prec == PREC_COMP) {         // Kahan
                const float y = x - c;
                const float t = s + y;
                c = (t - s) - y;
                s = t;
            } else {
                s += x;
            }
        }
        sum = s;
    } else if (g.prec == PREC_COMP) {
        const FF *pre = reinterpret_cast<const FF *>(d.is_pre);
        const FF below = mod_p2(lo, g.part) == 0 ? ff_of(0.0f) : pre[lo - 1];
        const FF top = pre[hi];
        const FF r = div_p2(lo, g.part) == div_p2(hi, g.part) ? ff_add(top, ff_neg(below))
                                                              : ff_add(ff_add(midc, ff_neg(below)), top);
        sum = ff_float(r);
    } else {
        const float below = mod_p2(lo, g.part) == 0 ? 0.0f : (float)d.is_pre[lo - 1];
        sum = div_p2(lo, g.part) == div_p2(hi, g.part) ? (float)d.is_pre[hi] - below
                                                         : ((float)mid - below) + (float)d.is_pre[hi];
    }
    return (double)((4.0f * q) * sum);
}

// Removes a resolved source's power from the exact accumulators: its one
// bin of Xn, or the two entries of the difference array D (X = Xn + prefix of
// D, with the prefix split into a carry per tile and a sum inside the tile;
// mark_track adds to the carries).
DEVI void subtract_track(const Grid &g, const Dev &d, int glo, int ghi, int64_t v)
{
    if (glo == ghi) {
        atomic_add_i128(&d.Xn[glo], -v);
        return;
    }
    atomic_add_i128(&d.D[glo], -v);
    if (ghi + 1 < g.B) atomic_add_i128(&d.D[ghi + 1], v);
}

// What a resolved track changes besides its own bins, by n threads (this one
// is the i-th): the carries into the tiles that start inside (glo, ghi + 1]
// (v: its power; not where the carries are float sums), and the stamps of
// the tiles the next body must convert (the track) and filter (every output
// whose window holds a bin of the track).
DEVI void mark_track(const Grid &g, const Dev &d, int glo, int ghi, int64_t v, uint32_t nxt, int i, int n)
{
    const int ta = div_p2(glo, g.tile), tb = div_p2(ghi, g.tile);
    if (v && glo != ghi) {
        const int te = min(div_p2(ghi + 1, g.tile), g.nt - 1);
        for (int tl = ta + 1 + i; tl <= te; tl += n) split_sum_add(&d.Dadj[tl], -v);
    }
    for (int tl = ta + i; tl <= tb; tl += n) d.xstamp[tl] = nxt;
    int sa, sb;
    window_reach(g, glo, ghi, &sa, &sb);
    for (int tl = div_p2(sa, g.tile) + i; tl <= div_p2(sb, g.tile); tl += n) d.sstamp[tl] = nxt;
}

// The same subtraction in fp32 (naive FP32 mode), vf = the power as a float:
// the fp32 difference array and its per-tile sums (k_snr_tail rescans the
// tile sums into the carries in fp32 every body).
DEVI void subtract_track_f32(const Grid &g, const Dev &d, int glo, int ghi, float vf)
{
    if (glo == ghi) {
        atomicAdd(&d.Xf[glo], -vf);
        return;
    }
    atomicAdd(&d.Df[glo], -vf);
    atomicAdd(&d.Dtf[div_p2(glo, g.tile)], -vf);
    if (ghi + 1 < g.B) {
        atomicAdd(&d.Df[ghi + 1], vf);
        atomicAdd(&d.Dtf[div_p2(ghi + 1, g.tile)], vf);
    }
}

// The same subtraction in the compensated FP32 mode (double-fp32
// accumulators, compensated atomics), vf = the power as a float.
DEVI void subtract_track_comp(const Grid &g, const Dev &d, int glo, int ghi, float vf)
{
    if (glo == ghi) {
        ff_atomic_add(&d.Xc[glo], -vf);
        return;
    }
    ff_atomic_add(&d.Dc[glo], -vf);
    ff_atomic_add(&d.Dtc[div_p2(glo, g.tile)], -vf);
    if (ghi + 1 < g.B) {
        ff_atomic_add(&d.Dc[ghi + 1], vf);
        ff_atomic_add(&d.Dtc[div_p2(ghi + 1, g.tile)], vf);
    }
}

// True when S^t may differ from S^{t-1} somewhere on tiles lo/tile ..
// hi/tile: one of them was refiltered in body t (stamp t), or was stamped
// for body t + 1 by a writer of this same launch, which may have replaced a
// stamp t (every stamp is at most t + 1).  Tracks over more than SKIP_TILES
// tiles count as changed without looking.
constexpr int SKIP_TILES = 4;
DEVI bool track_refiltered(const uint32_t *stamp, const Grid &g, int lo, int hi, uint32_t first, uint32_t last,
                           uint32_t t)          // first, last: the stamps of the end tiles
{
    const int a = div_p2(lo, g.tile), b = div_p2(hi, g.tile);
    if (b - a >= SKIP_TILES) return true;
    auto is = [&](uint32_t s) { return s == t || s == t + 1; };
    bool r = is(first) || is(last);
    for (int tl = a + 1; tl < b; ++tl) r |= is(stamp[tl]);
    return r;
}

// rho^2 = 4 q sum_{k in track} 1/S^t[k] for every unsubtracted candidate
// (Eq. "SNR inner product" in the sky-averaged power form); rho^2 >
// rho_th^2 subtracts the source from the binned power at once (appendix
// "Subtraction algorithm", steps 6-9: the data X^{t+1} no longer holds it)
// and stamps the tiles the next body must convert (the track) and filter
// (every output whose window holds a bin of the track, window_reach).  A candidate whose track lies in
// tiles the median left alone this body sees the same S as at its last
// evaluation, so its stored rho^2 stands (it was not above threshold then,
// or it would have been subtracted); body 0 filters every tile.  Per-block
// counts go to b_part for the tail (snr_tail).
__global__ __launch_bounds__(WG) void k_snr(const Slot *S)
{
    constexpr int NW = WG / 64;
    __shared__ uint32_t s_red[3][NW];     // new, near, evals
    __shared__ double s_min[NW];
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Grid g = sl.g;
    const Dev d = sl.d;
    if (d.ctl->done || d.ctl->bad) return;
    const int t = (int)d.ctl->iter;
    const uint32_t nxt = (uint32_t)t + 1;
    const uint32_t nc = d.ctl->n_cand;
    const bool naive = g.prec == PREC_NAIVE;
    const bool comp = g.prec == PREC_COMP;
    const FF *psum_ff = reinterpret_cast<const FF *>(d.is_psum);
    const int lane = lane_id();
    uint32_t my_new = 0, near = 0, evals = 0;         // at most one each per candidate
    double minm = INFINITY;
    // the wave walks its candidates together (uniform trip count), so that
    // all its lanes can sum the part sums under a wide track
    const uint32_t stride = gridDim.x * WG;
    // SU candidates per thread at a time: their records, then the stamps under
    // their tracks, then the evaluations.  In late bodies nearly every
    // candidate stops at the stamps, and the launch is the latency of these
    // two rounds of loads: 10.3 us a body on the 1e7 catalog
    constexpr int SU = 2;
    for (uint32_t jb0 = blockIdx.x * WG + (threadIdx.x & ~63u); jb0 < nc; jb0 += SU * stride) {
        int it_[SU], lo_[SU], hi_[SU];
        double r2_[SU];
        uint32_t sa_[SU], sb_[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const uint32_t j = min(jb0 + (uint32_t)u * stride + (uint32_t)lane, nc - 1u);
            it_[u] = d.c_iter[j];
            lo_[u] = d.c_glo[j];
            hi_[u] = d.c_ghi[j];
            r2_[u] = d.c_rho2[j];
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const bool on = it_[u] < 0;
            sa_[u] = on ? d.sstamp[div_p2(lo_[u], g.tile)] : 0u;
            sb_[u] = on ? d.sstamp[div_p2(hi_[u], g.tile)] : 0u;
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const uint32_t j = jb0 + (uint32_t)u * stride + (uint32_t)lane;
            const bool live = j < nc && it_[u] < 0;
            if (!__ballot(live)) continue;
            const int glo = live ? lo_[u] : 0, ghi = live ? hi_[u] : 0;
            const bool eval = live && (t == 0 || track_refiltered(d.sstamp, g, glo, ghi, sa_[u], sb_[u], (uint32_t)t));
            double r2 = r2_[u];
            // sum of the part sums of 1/S over the parts strictly before the
            // track's last part: a loop for tracks over a few parts, all lanes
            // of the wave together for wider ones, one track at a time
            const int plo = div_p2(glo, g.part), phi = div_p2(ghi, g.part);
            const bool need = eval && ghi - glo + 1 > NARROW && phi > plo;
            const bool wide = need && phi - plo > COOP_PARTS;
            double mid = 0.0;
            FF midc = ff_of(0.0f);
            if (need && !wide) {
                if (naive) {
                    float m = 0.0f;
                    for (int pp = plo; pp < phi; ++pp) m += (float)d.is_psum[pp];
                    mid = (double)m;
                } else if (comp) {
                    for (int pp = plo; pp < phi; ++pp) midc = ff_add(midc, psum_ff[pp]);
                } else {
                    double x[COOP_PARTS];              // at most COOP_PARTS, all loads in flight
#pragma unroll
                    for (int q = 0; q < COOP_PARTS; ++q) x[q] = d.is_psum[min(plo + q, phi - 1)];
#pragma unroll
                    for (int q = 0; q < COOP_PARTS; ++q)
                        if (plo + q < phi) mid += x[q];
                }
            }
            for (uint64_t wm = (uint64_t)__ballot(wide); wm; wm &= wm - 1) {
                const int L = __builtin_ctzll(wm);
                const int a = __builtin_amdgcn_readlane(plo, L), b = __builtin_amdgcn_readlane(phi, L);
                double sum = 0.0;
                FF sumc = ff_of(0.0f);
                if (naive) {
                    float m = 0.0f;
                    for (int pp = a + lane; pp < b; pp += 64) m += (float)d.is_psum[pp];
                    for (int o = 32; o >= 1; o >>= 1) m += __shfl_xor(m, o, 64);
                    sum = (double)m;
                } else if (comp) {
                    FF m = ff_of(0.0f);
                    for (int pp = a + lane; pp < b; pp += 64) m = ff_add(m, psum_ff[pp]);
                    for (int o = 32; o >= 1; o >>= 1) {
                        FF y;
                        y.hi = __shfl_xor(m.hi, o, 64);
                        y.lo = __shfl_xor(m.lo, o, 64);
                        m = ff_add(m, y);
                    }
                    sumc = m;
                } else {
                    // a 1.5M-bin track has 46 rounds of 64 parts: eight
                    // rounds' loads at a time
                    constexpr int PU = 8;
                    double m = 0.0;
                    for (int pp = a + lane; pp < b; pp += PU * 64) {
                        double x[PU];
#pragma unroll
                        for (int q = 0; q < PU; ++q) x[q] = d.is_psum[min(pp + q * 64, b - 1)];
#pragma unroll
                        for (int q = 0; q < PU; ++q)
                            if (pp + q * 64 < b) m += x[q];
                    }
                    sum = wave_sum(m);
                }
                if (lane == L) {
                    mid = sum;
                    midc = sumc;
                }
            }
            if (eval) {
                ++evals;
                const double q = d.c_q[j];
                r2 = g.prec == PREC_FP64 ? (4.0 * q) * track_inv_sum(d.S, d.is_pre, glo, ghi, g.part, mid)
                                         : snr2_f32(g, d, q, glo, ghi, mid, midc);
                d.c_rho2[j] = r2;
            }
            // a stored rho^2 has been in the margin's minimum since its
            // evaluation; it counts as near again in every body
            if (eval || (live && fabs(r2 - g.rth2) <= 1e-5 * g.rth2)) {
                const double rel = fabs(sqrt(r2) / g.rth - 1.0);
                minm = fmin(minm, rel);
                near += rel <= 1e-6;
            }
            const bool hit = live && r2 > g.rth2;
            int64_t v = 0;                             // for the exact carries
            if (hit) {
                d.c_iter[j] = t;
                ++my_new;
                v = (int64_t)d.c_qfx[j];
                if (v) {
                    const float vf = (float)ldexp((double)v, fx_exp(d.ctl->amax_bits, g.T) +
                                                                 f32_scale(d.ctl->amax_bits, g.T));
                    if (comp) {
                        subtract_track_comp(g, d, glo, ghi, vf);
                    } else {
                        subtract_track(g, d, glo, ghi, v);
                        if (naive) subtract_track_f32(g, d, glo, ghi, vf);
                    }
                }
                if (comp) v = 0;
            }
            // the tiles of a wide track (up to 735) by the whole wave: with one
            // thread each the first body took 46 us, with this 28
            const bool many = hit && div_p2(ghi, g.tile) - div_p2(glo, g.tile) >= SKIP_TILES;
            if (hit && !many) mark_track(g, d, glo, ghi, v, nxt, 0, 1);
            for (uint64_t wm = (uint64_t)__ballot(many); wm; wm &= wm - 1) {
                const int L = __builtin_ctzll(wm);
                const uint32_t vl = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, L);
                const uint32_t vh = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), L);
                mark_track(g, d, __builtin_amdgcn_readlane(glo, L), __builtin_amdgcn_readlane(ghi, L),
                           (int64_t)((uint64_t)vh << 32 | vl), nxt, lane, 64);
            }
        }
    }
    my_new = wave_scan_u32(my_new);
    near = wave_scan_u32(near);
    evals = wave_scan_u32(evals);
    for (int s = 32; s >= 1; s >>= 1) minm = fmin(minm, __shfl_xor(minm, s, 64));
    const int w = threadIdx.x >> 6;
    if (lane == 63) {
        s_red[0][w] = my_new;
        s_red[1][w] = near;
        s_red[2][w] = evals;
        s_min[w] = minm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (blockIdx.x == 0) {
            d.ctl->xupd = nxt;
            d.ctl->tail_due = 1;
        }
        for (int v = 1; v < NW; ++v) {
            for (int r = 0; r < 3; ++r) s_red[r][0] += s_red[r][v];
            s_min[0] = fmin(s_min[0], s_min[v]);
        }
        SnrPart p;
        p.n_new = s_red[0][0];
        p.near = s_red[1][0];
        p.evals = s_red[2][0];
        p.pad = 0;
        p.minm = s_min[0];
        d.b_part[blockIdx.x] = p;
    }
}

// Counts the tiles stamped for body nxt (the thread's share of the X stamps to
// *nx) and lists those to filter in tile order; returns the list's length.
// One block of NT threads: rounds of TW tiles per thread, all stamps of a round
// loaded together.  One tile per thread and round, with two barriers each,
// were 8 rounds of load latency for 1843 tiles and 15 for 3686: the launch
// took 10.8 and 14 us a body instead of 9.9 and 11.3.
template <int NT>
DEVI uint32_t list_stamped(const Grid &g, const Dev &d, uint32_t nxt, uint32_t (&s_wl)[2][NT / 64], uint32_t *nx)
{
    constexpr int TW = 2048 / NT;
    const int w = threadIdx.x >> 6;
    uint32_t listed = 0;                  // block-uniform
    for (int base = 0, rd = 0; base < g.nt; base += NT * TW, rd ^= 1) {
        const int t0 = base + (int)threadIdx.x * TW;
        uint32_t xs[TW], ss[TW];
#pragma unroll
        for (int q = 0; q < TW; ++q) {
            const int tl = min(t0 + q, g.nt - 1);
            xs[q] = d.xstamp[tl];
            ss[q] = d.sstamp[tl];
        }
        uint32_t mask = 0;
#pragma unroll
        for (int q = 0; q < TW; ++q) {
            if (t0 + q >= g.nt) continue;
            *nx += xs[q] == nxt;
            mask |= (ss[q] == nxt ? 1u : 0u) << q;
        }
        const uint32_t own = (uint32_t)__popc(mask), inc = wave_scan_u32(own);
        if (lane_id() == 63) s_wl[rd][w] = inc;
        __syncthreads();
        uint32_t at = listed + inc - own;
#pragma unroll
        for (int v = 0; v < NT / 64; ++v) {
            const uint32_t x = s_wl[rd][v];
            at += v < w ? x : 0u;
            listed += x;
        }
        for (; mask; mask &= mask - 1) d.sdl[at++] = (uint32_t)(t0 + __builtin_ctz(mask));
    }
    return listed;
}

// The tail of a loop body, run by one block of NT threads once k_snr has
// ended: combines the per-block partials, counts the tiles stamped for the
// next body, takes the stop decision (nothing new subtracted, or max_iter)
// and whether the next median runs in split mode.  It runs at most once per
// k_snr (tail_due).  converts: the next body's X is k_xupdate's to convert.
template <int NT> DEVI void snr_tail(const Slot &sl, bool converts)
{
    constexpr int NW = NT / 64;
    constexpr int NR = 4;                 // new, near, evals, X tiles
    constexpr int NP = SNR_BLOCKS / NT;
    __shared__ uint32_t s_red[NR][NW];
    __shared__ uint32_t s_wl[2][NW];
    __shared__ double s_min[NW];
    const Grid g = sl.g;
    const Dev d = sl.d;
    Ctl *c = d.ctl;
    const Ctl k = *c;                     // every field read once, ahead of the stores
    if (!k.tail_due || k.done || k.bad) return;
    if (g.prec == PREC_NAIVE) block_scan_array<float, NT>(d.Dtf, d.Dcf, g.nt);
    const uint32_t nxt = k.iter + 1;
    const uint32_t lx = d.xstamp[g.nt - 1], ls = d.sstamp[g.nt - 1];
    const int w = threadIdx.x >> 6;
    SnrPart p[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) p[i] = d.b_part[threadIdx.x + i * NT];
    uint32_t nx = 0;
    const uint32_t listed = list_stamped<NT>(g, d, nxt, s_wl, &nx);
    uint32_t red[NR] = {0, 0, 0, nx};
    double minm = INFINITY;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        red[0] += p[i].n_new;
        red[1] += p[i].near;
        red[2] += p[i].evals;
        minm = fmin(minm, p[i].minm);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const uint32_t x = wave_scan_u32(red[r]);
        if (lane_id() == 63) s_red[r][w] = x;
    }
    for (int s = 32; s >= 1; s >>= 1) minm = fmin(minm, __shfl_xor(minm, s, 64));
    if (lane_id() == 0) s_min[w] = minm;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int v = 1; v < NW; ++v) {
        for (int r = 0; r < NR; ++r) s_red[r][0] += s_red[r][v];
        s_min[0] = fmin(s_min[0], s_min[v]);
    }
    // bins of the stamped tiles: the last tile may be short
    const uint32_t pad = (uint32_t)(g.nt * g.tile - g.B);
    const uint64_t ux = (uint64_t)s_red[3][0] * (uint32_t)g.tile - (lx == nxt ? pad : 0u);
    const uint64_t us = (uint64_t)listed * (uint32_t)g.tile - (ls == nxt ? pad : 0u);
    const uint32_t n_new = s_red[0][0];
    c->tail_due = 0;
    c->med_split = listed <= g.split_tiles;
    c->n_sdl = listed;
    if (k.iter < (uint32_t)NEW_CAP) d.n_new[k.iter] = n_new;
    c->n_resolved = k.n_resolved + n_new;
    c->n_near = k.n_near + s_red[1][0];
    c->units_snr = k.units_snr + s_red[2][0];
    if (s_min[0] < __longlong_as_double((long long)k.min_margin))
        c->min_margin = (uint64_t)__double_as_longlong(s_min[0]);
    const uint32_t mi = g.max_iter ? g.max_iter : k.n_cand + 1;
    uint32_t done = 0;
    if (n_new == 0) {
        done = 1;
        c->n_iter = nxt;
    } else if (nxt >= mi) {
        done = 1;                    // the loop did not settle within max_iter bodies
        c->status = 6;
        c->n_iter = nxt;
    } else {
        c->iter = nxt;
        if (converts) c->units_x = k.units_x + ux;
        c->units_med = k.units_med + us;
    }
    c->done = done;
    // progress for the host that paces the launches
    if (sl.prog)
        __hip_atomic_store(sl.prog, pace_word(nxt, done, listed <= g.split_tiles, k.med_split), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

// The template model's tail, run by one block of NT threads once k_cx_snr has
// ended: the stop decision, the split mode of the next PSD launch, the list of
// its tiles, and the progress word for the host.  It runs at most once per
// k_cx_snr (tail_due); an invalid catalog settles at once.
template <int NT> DEVI void cx_tail(const Slot &sl)
{
    __shared__ uint32_t s_wl[2][NT / 64];
    __shared__ uint32_t s_nx;
    const Grid g = sl.g;
    const Dev d = sl.d;
    Ctl *c = d.ctl;
    const Ctl k = *c;
    if (k.done || !(k.tail_due || k.bad)) return;
    const uint32_t nxt = k.iter + 1;
    const uint32_t lx = d.xstamp[g.nt - 1], ls = d.sstamp[g.nt - 1];
    if (threadIdx.x == 0) s_nx = 0;
    __syncthreads();
    uint32_t nx = 0;
    const uint32_t listed = list_stamped<NT>(g, d, nxt, s_wl, &nx);
    nx = wave_scan_u32(nx);
    if (lane_id() == 63 && nx) atomicAdd(&s_nx, nx);
    __syncthreads();
    if (threadIdx.x != 0) return;
    uint32_t done = 0;
    c->tail_due = 0;
    c->margin = k.min_margin;
    if (k.bad) {
        done = 1;
        c->n_iter = k.iter;
    } else {
        const uint32_t pad = (uint32_t)(g.nt * g.tile - g.B);      // the last tile may be short
        const uint32_t n_new = k.n_new_body;
        c->n_new_body = 0;
        c->n_resolved = k.n_resolved + n_new;
        const uint32_t mi = g.max_iter ? g.max_iter : k.cand_cursor + 1;
        if (n_new == 0) {
            done = 1;
            c->n_iter = nxt;
        } else if (nxt >= mi) {
            done = 1;
            c->status = 6;
            c->n_iter = nxt;
        } else {
            c->iter = nxt;
            c->med_split = listed <= g.split_tiles;
            c->n_sdl = listed;
            c->x_next = s_nx * (uint32_t)g.tile - (lx == nxt ? pad : 0u);
            c->units_med = k.units_med + (uint64_t)listed * (uint32_t)g.tile - (ls == nxt ? pad : 0u);
        }
    }
    c->n_cand = k.cand_cursor;
    c->done = done;
    if (sl.prog)
        __hip_atomic_store(sl.prog, pace_word(nxt, done, listed <= g.split_tiles, k.med_split), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(WG) void k_cx_tail(const Slot *S) { cx_tail<WG>(*S); }

// The tail as a kernel of its own, ahead of k_xupdate: the naive FP32 mode
// rescans the fp32 tile sums into the carries that k_xupdate reads.
__global__ __launch_bounds__(SNR_BLOCKS) void k_snr_tail(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    snr_tail<SNR_BLOCKS>(sl, true);
}

// ------------------------------------------------------------------ outputs

// ids of the candidates (the catalog is not retained after the run) and the
// resolved list, unsorted.
__global__ __launch_bounds__(WG) void k_cand_ids(const Slot *S)
{
    const Slot &sl = S[blockIdx.y];
    if (!sl.active) return;
    const Dev d = sl.d;
    const uint32_t *ids = sl.ids;
    list_resolved(d.ctl->n_cand, d.c_iter, d.c_id, reinterpret_cast<uint64_t *>(d.ev_val), &d.ctl->res_cursor,
                  [&](uint32_t j) { return ids[d.c_src[j]]; });
    if (sl.host_ctl && blockIdx.x == gridDim.x - 1) put_host(sl.host_ctl, d.ctl, threadIdx.x);
}

// ------------------------------------------------------------------ launchers

hipError_t launch_grid_tables(const Slot *ds, const Dims &dm, hipStream_t st)
{
    k_sinstr<<<dim3((dm.maxB + WG - 1) / WG, dm.ns), WG, 0, st>>>(ds);
    k_inv_prefix<<<dim3(dm.maxnt, dm.ns), WG, 0, st>>>(ds);
    k_sx_scan<<<dim3(1, dm.ns), WG, 0, st>>>(ds);
    const int nseg = (dm.maxB + SEG_BINS - 1) / SEG_BINS;
    k_isx_seg<<<dim3((nseg + WG / 64 - 1) / (WG / 64), dm.ns), WG, 0, st>>>(ds);
    return hipGetLastError();
}

hipError_t launch_reset(Slot *ds, const Slot &slot, hipStream_t st)
{
    k_reset<<<(slot.g.nt + WG - 1) / WG, WG, 0, st>>>(slot, ds);
    if (slot.g.prec == PREC_NAIVE) k_zero_f32<<<1024, WG, 0, st>>>(ds);
    return hipGetLastError();
}

hipError_t launch_prep(const Slot *ds, const Dims &dm, hipStream_t st)
{
    if (dm.prep_blocks > 0) k_prep_count<<<dim3(dm.prep_blocks, dm.ns), WG, 0, st>>>(ds);
    k_prep_colscan<<<dim3((dm.maxnt + CS_COL - 1) / CS_COL, dm.ns), CS_WG, 0, st>>>(ds);
    k_prep_plan<<<dim3(1, dm.ns), PLAN_T, 0, st>>>(ds);
    if (dm.prep_blocks > 0) k_prep_scatter<<<dim3((dm.prep_blocks + 7) / 8 * 8, dm.ns), WG, 0, st>>>(ds);
    k_accum<<<dim3(dm.accum_blocks, dm.ns), ACC_T, 0, st>>>(ds);
    // a tile is hot from more than ACC_EV_MIN events on; a source has two at most
    if (2 * dm.max_n > (uint64_t)ACC_EV_MIN)
        k_accum_reduce<<<dim3(dm.maxnt * (dm.maxtile / RED_BINS), dm.ns), RED_BINS, 0, st>>>(ds);
    if (dm.naive) k_accum_f32<<<dim3(2048, dm.ns), WG, 0, st>>>(ds);
    k_dscan<<<dim3(1, dm.ns), WG, 0, st>>>(ds);
    return hipGetLastError();
}

// One kernel of the loop body; with events, the dispatch itself records its
// start (ea) and end (eb), which adds no work to the stream.
hipError_t go(const void *kernel, dim3 grid, dim3 block, hipStream_t st, hipEvent_t ea, hipEvent_t eb,
              const Slot *ds)
{
    void *args[] = {(void *)&ds};
    if (!ea && !eb) return hipLaunchKernel(kernel, grid, block, args, 0, st);
    return hipExtLaunchKernel(kernel, grid, block, args, 0, st, ea, eb, 0);
}

hipError_t launch_xupdate(const Slot *ds, const Dims &dm, hipStream_t st, hipEvent_t ea, hipEvent_t eb)
{
    return go((const void *)k_xupdate, dim3(dm.maxnt + 1, dm.ns), dim3(WG), st, ea, eb, ds);
}

hipError_t launch_median(const Slot *ds, const Dims &dm, hipStream_t st, hipEvent_t ea, hipEvent_t eb)
{
    const bool med = dm.est_mask & 1u, mean = dm.est_mask & 2u;
    hipError_t e = hipSuccess;
    // one slot: a block per part; several: the listed launch
    const bool listed = dm.ns > 1;
    const unsigned gx = (unsigned)(listed ? dm.maxlist : dm.maxparts);
    const void *km = listed ? (const void *)k_median_listed : (const void *)k_median;
    const void *kn = listed ? (const void *)k_mean_listed : (const void *)k_mean;
    if (med) e = go(km, dim3(gx, dm.ns), dim3(MWG), st, ea, mean ? nullptr : eb, ds);
    if (mean && e == hipSuccess) e = go(kn, dim3(gx, dm.ns), dim3(MWG), st, med ? nullptr : ea, eb, ds);
    return e;
}

hipError_t launch_next(const Slot *ds, const Dims &dm, hipStream_t st, hipEvent_t ea, hipEvent_t eb)
{
    const bool mean = dm.est_mask & 2u, cx = dm.ns == 2;
    const void *k = mean ? (cx ? (const void *)k_mean_next<X_CX> : (const void *)k_mean_next<X_ACCUM>)
                         : (cx ? (const void *)k_median_next<X_CX> : (const void *)k_median_next<X_ACCUM>);
    return go(k, dim3((cx ? dm.split_parts : dm.maxparts) + 1, dm.ns), dim3(MWG), st, ea, eb, ds);
}

hipError_t launch_cx_tail(const Slot *ds, hipStream_t st)
{
    k_cx_tail<<<1, WG, 0, st>>>(ds);
    return hipGetLastError();
}

hipError_t launch_snr(const Slot *ds, const Dims &dm, hipStream_t st, hipEvent_t ea, hipEvent_t eb)
{
    if (!dm.naive) return go((const void *)k_snr, dim3(SNR_BLOCKS, dm.ns), dim3(WG), st, ea, eb, ds);
    hipError_t e = go((const void *)k_snr, dim3(SNR_BLOCKS, dm.ns), dim3(WG), st, ea, nullptr, ds);
    if (e != hipSuccess) return e;
    return go((const void *)k_snr_tail, dim3(1, dm.ns), dim3(SNR_BLOCKS), st, nullptr, eb, ds);
}

// ------------------------------------------------------------------ coarse-graining
//
// Sec. "Coarse-graining of the data": the spectrum averaged over logarithmic
// frequency bins, and the mean frequency of each bin.  A bin is a contiguous
// range of grid samples [i0, i1) (found by the host), shared by `ns` blocks
// (the host adds their sums in order).  The last bins of a logarithmic grid
// hold most samples (5 % of a 4-year grid each), so one block of 256 threads
// per bin waited for 225 loads in a row: 83 us at 3.8e6 bins, 9 us with CT
// threads and the bin shared (25 and 7 us at 3.1e5 bins), next to the 4.5 us
// of an empty launch.
constexpr int CT = 512;

__global__ __launch_bounds__(CT) void k_coarse(const double *S, const double *sx, const double *X, int kind,
                                               int64_t k0, int B, double T, CoarseEdges ed, int n_out, int ns,
                                               CoarseSum *out)
{
    __shared__ double sf[CT / 64], sv[CT / 64];
    __shared__ CoarseSum sum;
    const int kb = blockIdx.x, part = blockIdx.y;
    const int i0 = ed.i[kb], i1 = ed.i[kb + 1];
    const int n = max(i1 - i0, 0), share = (n + ns - 1) / ns;
    const int b0 = i0 + min(part * share, n), b1 = i0 + min((part + 1) * share, n);
    constexpr int U = 4;
    double af = 0.0, av = 0.0;
    for (int i = b0 + (int)threadIdx.x; i < b1; i += U * CT) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(i + u * CT, b1 - 1);
            v[u] = kind == 0 ? S[j] : kind == 1 ? X[j] : kind == 2 ? S[j] - sx[j] : sx[j];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u * CT >= b1) continue;
            af += (double)(k0 + i + u * CT) / T;
            av += v[u];
        }
    }
    af = wave_sum(af);
    av = wave_sum(av);
    if (lane_id() == 0) {
        sf[threadIdx.x >> 6] = af;
        sv[threadIdx.x >> 6] = av;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < CT / 64; ++w) {
            af += sf[w];
            av += sv[w];
        }
        sum = {af, av, (double)(b1 - b0)};
    }
    __syncthreads();
    put_host(out + (size_t)kb * ns + part, &sum, threadIdx.x);
}

hipError_t launch_coarse(const double *S, const double *sx, const double *X, int kind, int64_t k0, int B,
                         double T, const CoarseEdges &ed, int n_out, int ns, CoarseSum *out, hipStream_t st)
{
    k_coarse<<<dim3(n_out, ns), CT, 0, st>>>(S, sx, X, kind, k0, B, T, ed, n_out, ns, out);
    return hipGetLastError();
}

hipError_t launch_outputs(const Slot *ds, const Dims &dm, hipStream_t st)
{
    k_cand_ids<<<dim3(SNR_BLOCKS, dm.ns), WG, 0, st>>>(ds);
    return hipGetLastError();
}

}  // namespace gbs
