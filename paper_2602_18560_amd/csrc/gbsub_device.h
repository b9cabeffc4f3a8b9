// gbsub_device.h -- device helpers shared by the kernel files of libgbsub
// (grid tables, windows and dirty-tile stamps); not part of the public ABI.
#pragma once

#include "gbsub_internal.h"

namespace gbs {

#ifndef DEVI
#define DEVI __device__ __forceinline__
#endif

// x / p and x % p for x >= 0 and p a power of two (tile and part sizes).
DEVI int div_p2(int x, int p) { return x >> __builtin_ctz((unsigned)p); }
DEVI int mod_p2(int x, int p) { return x & (p - 1); }

// Window start of output k (clamped full window), grid of B >= W bins.
DEVI int win_start(int k, int B, int W, int h)
{
    int a = k - h;
    a = a < 0 ? 0 : a;
    return a > B - W ? B - W : a;
}

// Strain-equivalent SciRDv1 A-channel noise: S_AA(f) / R_AA(f) with
//   P_OMS = (P pm)^2 [1 + (2 mHz/f)^4] (2 pi f/c)^2,
//   P_TM  = (A fm)^2 [1 + (0.4 mHz/f)^2][1 + (f/8 mHz)^4] (2 pi f)^-4 (2 pi f/c)^2,
//   S_AA  = 8 sin^2 u {4 [1 + cos u + cos^2 u] P_TM + [2 + cos u] P_OMS},
//   R_AA  = 16 sin^2 u u^2 (9/20) / (1 + 0.7 u^2),  u = f/f*, f* = c/(2 pi L)
// (appendices "LISA instrumental noise" and "Characteristic strain").
DEVI double sinstr_dev(double f, double oms_pm, double tm_fm, double arm_m)
{
    const double c = 299792458.0;
    const double two_pi = 6.283185307179586;
    const double u = f / (c / (two_pi * arm_m));
    const double w = two_pi * f;
    const double wc = w / c;
    const double oms = oms_pm * 1e-12, tm = tm_fm * 1e-15;
    const double a = 2e-3 / f, b = 4e-4 / f, e = f / 8e-3;
    const double p_oms = (oms * oms) * (1.0 + a * a * a * a) * (wc * wc);
    const double p_tm = (tm * tm) * (1.0 + b * b) * (1.0 + e * e * e * e) / (w * w * w * w) * (wc * wc);
    double s, co;
    sincos(u, &s, &co);
    const double saa = 8.0 * (s * s) * (4.0 * (1.0 + co + co * co) * p_tm + (2.0 + co) * p_oms);
    const double raa = 16.0 * (s * s) * (u * u) * (0.45 / (1.0 + 0.7 * (u * u)));
    return saa / raa;
}

DEVI void stamp_tiles(uint32_t *stamp, const Grid &g, int lo, int hi, uint32_t nxt)
{
    for (int tl = div_p2(lo, g.tile); tl <= div_p2(hi, g.tile); ++tl) stamp[tl] = nxt;
}

// Outputs whose window holds a bin of [lo, hi] (Eq. "running median" with the
// window shifted inward at the grid edges): [lo - h, hi + h] in the interior;
// every output of the lower edge (window [0, W-1]) once lo <= W-1, every
// output of the upper edge (window [B-W, B-1]) once hi >= B-W, and the whole
// grid when it is shorter than the window.
DEVI void window_reach(const Grid &g, int lo, int hi, int *a, int *b)
{
    const bool whole = g.B < g.W;
    *a = (whole || lo <= g.W - 1) ? 0 : lo - g.h;
    *b = (whole || hi >= g.B - g.W) ? g.B - 1 : hi + g.h;
}

// Fixed-point exponent E of the template model's data: every template
// component is at most A T / 2, so with m = max(n, 4096) sources the sum of the
// n components of one word stays below 2^62 and a single component below 2^50
// (which the rounding of fxm needs).
DEVI int cx_exp(uint32_t amax_bits, uint32_t n, double T)
{
    const double v = (double)max(n, 4096u) * (double)__uint_as_float(amax_bits) * (T * 0.5);
    if (!(v > 0.0)) return 0;
    return 61 - ilogb(v);
}

// A record to host-mapped memory, in 8-byte words: lane w of the calling threads
// stores word w (lane: 0, 1, .. at least the record's words).
template <typename T> DEVI void put_host(T *dst, const T *src, int lane)
{
    static_assert(sizeof(T) % 8 == 0, "copied in 8-byte words");
    if (lane < (int)(sizeof(T) / 8))
        __hip_atomic_store(reinterpret_cast<uint64_t *>(dst) + lane, reinterpret_cast<const uint64_t *>(src)[lane],
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The ids of candidates 0 .. nc-1 (id_of(j): that of candidate j) into c_id,
// and the resolved ones (iter >= 0) as words id << 32 | j into `list`, in any
// order: each block takes a contiguous share of at least LR_MIN candidates,
// counts its resolved ones and reserves their entries with one atomic (one
// block per 305 candidates spent 10 us on the 1024 same-address atomics).
// Blocks of WG threads; contains barriers.
constexpr uint32_t LR_U = 4, LR_MIN = LR_U * WG;
template <typename F>
DEVI void list_resolved(uint32_t nc, const int32_t *iter, uint32_t *c_id, uint64_t *list, uint32_t *cursor, F id_of)
{
    __shared__ uint32_t s_n, s_base;
    const uint32_t share = max((nc + gridDim.x - 1) / gridDim.x, LR_MIN);
    const uint32_t j0 = min(blockIdx.x * share, nc), j1 = min(j0 + share, nc);
    if (j0 >= j1) return;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    uint32_t mine = 0;
    for (uint32_t j = j0 + threadIdx.x; j < j1; j += LR_U * WG) {
        int32_t t[LR_U];
#pragma unroll
        for (uint32_t u = 0; u < LR_U; ++u) t[u] = iter[min(j + u * WG, j1 - 1)];
#pragma unroll
        for (uint32_t u = 0; u < LR_U; ++u) mine += j + u * WG < j1 && t[u] >= 0 ? 1u : 0u;
    }
    for (int o = 32; o >= 1; o >>= 1) mine += (uint32_t)__shfl_xor((int)mine, o, 64);
    if (__lane_id() == 0 && mine) atomicAdd(&s_n, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        s_base = s_n ? atomicAdd(cursor, s_n) : 0u;
        s_n = 0;
    }
    __syncthreads();
    for (uint32_t j = j0 + threadIdx.x; j < j1; j += LR_U * WG) {
        uint32_t id[LR_U];
        int32_t t[LR_U];
#pragma unroll
        for (uint32_t u = 0; u < LR_U; ++u) {
            const uint32_t q = min(j + u * WG, j1 - 1);
            id[u] = id_of(q);
            t[u] = iter[q];
        }
#pragma unroll
        for (uint32_t u = 0; u < LR_U; ++u) {
            const uint32_t q = j + u * WG;
            if (q >= j1) continue;
            c_id[q] = id[u];
            if (t[u] >= 0) list[s_base + atomicAdd(&s_n, 1u)] = (uint64_t)id[u] << 32 | q;
        }
    }
}

}  // namespace gbs
