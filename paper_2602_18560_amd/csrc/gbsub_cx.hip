// gbsub_cx.hip -- the complex-template data model of libgbsub.
//
// The data is one complex frequency series per TDI channel, h_A and h_E (the
// T channel is insensitive: Sec. "Simulations"), holding the sum of the
// 128-sample frequency-domain templates of every source (Sec. "Simulations";
// appendix "Subtraction algorithm").  Resolved sources are scattered out of
// h at their template's bins (Eq. "vectorized-subtraction").  The template
// of a source (A, f, fdot) and its channel phases (phi_A, phi_E) is
//
//   q = floor((f + fdot T/2) T + 1/2), delta = f T - q, d = fdot T^2,
//   s_n = (A/2) exp(2 pi i (delta x + d x^2 / 2)), x = n/128,
//   U_j = (T/128) DFT_128(s)_m, m = j mod 128, j = -64 .. 63, at bin q + j - k0,
//   H_c,j = exp(i phi_c) U_j,
//
// the slowly varying factor of the signal once the carrier q/T is taken
// out, sampled 128 times over T (a fast/slow template of our own
// sky-averaged model; the paper's templates come from gbgpu).  Then per
// channel X_c = (2/T)|h_c|^2, S_c = C median_W(X_c) + S_instr (or the running
// mean), and rho^2 = (4/T) sum_j |U_j|^2 (1/S_A + 1/S_E) over the grid bins.
//
// Design for gfx950:
//  * A template is one wave's work: two samples per lane, the first radix-2
//    stage inside the lane, then two 64-point FFTs across the lanes.  The
//    exchanges run on the VALU, not through the LDS crossbar: row swaps
//    (v_permlane32_swap, v_permlane16_swap) of the two FFTs' registers for
//    spans 32 and 16, after which each lane computes whole butterflies, and
//    DPP moves for spans 8 .. 1 (the lanes hold their positions permuted so
//    that span 4 is one half-row mirror).  exp(2 pi i t) is a 16-entry LDS
//    table (one bank row: no conflicts) times short Taylor polynomials;
//    twiddles and signs are lane constants in registers.  Templates are
//    recomputed wherever they are needed (injection, every SNR evaluation,
//    subtraction) instead of stored (2 KB per candidate, 20 GB for 1e7
//    sources): about 240 VALU instructions of one wave per template.
//  * h is exact fixed point (int64, unit 2^-E with E from the largest
//    amplitude and the source count), so injection and subtraction are
//    order-independent integer adds and a subtracted template cancels to the
//    last bit: h always equals the sum of the (rounded) templates of the
//    candidates left plus the fixed sum of the sources that can never be
//    candidates.
//  * Injection.  Most sources of a large catalog are too faint to be
//    candidates and share their centre bin with many others: the moment path
//    (k_cx_faint) sums the Taylor coefficients of their samples per centre, in
//    integers, and transforms once per centre and channel.  The others take
//    the direct path (k_cx_inject): sources are grouped by 1024-bin tile (LDS
//    histograms, one scan, a scatter with per-block range reservations); each
//    block accumulates a chunk of one tile's sources into an LDS window of
//    the tile plus the template reach on each side (even and odd bins apart:
//    the lanes of one atomic add hit pairs of neighbouring words), then adds
//    the window to h with one global atomic per touched word.  Each wave
//    takes an equal share of the chunk, 64 sources at a time: their constants
//    are computed one per lane and broadcast by readlane while the wave
//    synthesises one template after the other.
//  * The per-channel PSD is the power model's median (or mean) kernel, run
//    over a two-slot descriptor table (A and E), with the same dirty-tile
//    stamps; a body is X update, PSD, SNR + subtraction, and a one-block tail, or,
//    while few tiles are dirty, PSD (with the X update and the tail of the body
//    before) and SNR.

#include "gbsub_internal.h"
#include "gbsub_device.h"

#include <climits>
#include <math.h>

namespace gbs {

namespace {

constexpr int NF = CX_NF;
constexpr int HALO = NF / 2;                  // template reach on each side of its centre
constexpr int CXW = CX_TILE + NF;             // LDS window of an injection block
constexpr int SRC_PB = 4096;                  // sources per block of the count and scatter passes
constexpr int CH = 8192;                      // sources per injection block at most
constexpr int CH_MIN = 32;                    // and at least (a block's four waves take a quarter each)
constexpr int CH_GRID = 2048;                 // injection blocks that fill the chip
constexpr uint32_t KEY_NONE = 0xFFFFFFFFu;    // source key: no template on the grid
constexpr uint32_t KEY_FAINT = 0x80000000u;   // source key: the moment path takes it
constexpr uint32_t FAINT_MIN_N = 1u << 16;    // smallest catalog with a moment path
constexpr double FAINT_MAX_D = 0.25 * 4.0 / 3.141592653589793;   // its largest |fdot| T^2 (|b| <= 1/4)
constexpr int NMOM = 28;                      // moments per centre
constexpr int FB_MAX = 16384;                 // faint buckets at most
constexpr int FB_SRC = 16384;                 // sources per block of the faint passes
constexpr int FB_SRC_MIN = 4096;              // and in catalogs of up to FB_SMALL sources
constexpr uint64_t FB_SMALL = 1u << 20;
constexpr int FB_T = 1024;                    // threads of those blocks
constexpr int MOM_MIN = 12;                   // fewer faint sources of a centre: one template each
constexpr int MOM_COOP = 2048;                // more: all waves of the block share the centre
constexpr int SNR_GRID = 2048;                // blocks of the SNR launch
constexpr int GRP = 4;                        // consecutive candidates of a wave in it
constexpr uint32_t BOUND_MIN_N = 1u << 14;    // smallest catalog whose candidates are tested by a bound first

struct KArgs {
    Grid g;
    CxDev d;
    CxIn in;
};

__device__ __forceinline__ int lane() { return __lane_id(); }

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// Exchanges between lanes without the LDS crossbar.
//  * Row swaps (gfx950): v_permlane32_swap(P, Q) leaves P = [P lanes 0-31,
//    Q lanes 0-31] and Q = [P lanes 32-63, Q lanes 32-63];
//    v_permlane16_swap(P, Q) does the same on rows of 16 lanes, P = [P row 0,
//    Q row 0, P row 2, Q row 2] and Q = [P row 1, Q row 1, P row 3, Q row 3].
//  * DPP moves within rows of 16 lanes: lane l reads lane l ^ 8 (row rotate
//    by 8), l ^ 7 (half-row mirror), l ^ 2 and l ^ 1 (quad permutes).
template <int SPAN> __device__ __forceinline__ void row_swap(double *P, double *Q)
{
    static_assert(SPAN == 32 || SPAN == 16, "row-swap spans");
    const long long bp = __double_as_longlong(*P), bq = __double_as_longlong(*Q);
    const unsigned plo = (unsigned)(bp & 0xffffffffll), phi = (unsigned)(bp >> 32);
    const unsigned qlo = (unsigned)(bq & 0xffffffffll), qhi = (unsigned)(bq >> 32);
    unsigned p0, q0, p1, q1;
    if constexpr (SPAN == 32) {
        const auto rl = __builtin_amdgcn_permlane32_swap(plo, qlo, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(phi, qhi, false, false);
        p0 = rl[0]; q0 = rl[1]; p1 = rh[0]; q1 = rh[1];
    } else {
        const auto rl = __builtin_amdgcn_permlane16_swap(plo, qlo, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(phi, qhi, false, false);
        p0 = rl[0]; q0 = rl[1]; p1 = rh[0]; q1 = rh[1];
    }
    *P = __longlong_as_double(((long long)p1 << 32) | p0);
    *Q = __longlong_as_double(((long long)q1 << 32) | q0);
}

// DPP patterns: 8 = l ^ 8, 7 = l ^ 7, 2 = l ^ 2, 1 = l ^ 1.  Every lane of
// the wave is active and every source lane is in range: the moves need no
// old value (bound_ctrl).
template <int PAT> __device__ __forceinline__ int dpp_move(int v)
{
    static_assert(PAT == 8 || PAT == 7 || PAT == 2 || PAT == 1, "DPP patterns");
    if constexpr (PAT == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);   // row_ror:8
    else if constexpr (PAT == 7) return __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true); // row_half_mirror
    else if constexpr (PAT == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);  // quad_perm [2,3,0,1]
    else return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);                        // quad_perm [1,0,3,2]
}

template <int PAT> __device__ __forceinline__ double partner(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = dpp_move<PAT>((int)(b & 0xffffffffll)), hi = dpp_move<PAT>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int PAT> __device__ __forceinline__ double2 partner2(double2 v)
{
    return make_double2(partner<PAT>(v.x), partner<PAT>(v.y));
}

// Sum over the wave, the same value on every lane: a butterfly over lane
// pairs that differ in bit 5, bit 4, bit 3, bits 0-2, bit 1 and bit 0 (both
// lanes of a pair add the same two values).
__device__ __forceinline__ double wave_sum(double v)
{
    double w = v;
    row_swap<32>(&v, &w);
    v += w;
    w = v;
    row_swap<16>(&v, &w);
    v += w;
    v += partner<8>(v);
    v += partner<7>(v);
    v += partner<2>(v);
    v += partner<1>(v);
    return v;
}


// v (already in units of 2^-E, |v| < 2^51) rounded to the nearest integer,
// ties to even: v + 1.5 2^52 lies in [2^52, 2^53), where the spacing of
// doubles is 1, so the addition rounds v and its low mantissa bits hold the
// integer plus 2^51.
__device__ __forceinline__ long long fxm(double v)
{
    return __double_as_longlong(v + 6755399441055744.0) - 0x4338000000000000ll;
}

// Central DFT index q, delta = f T - q and d = fdot T^2 (the operations of
// the definition, in this order); false if the source has no template
// (|d| >= 2^20 or |q| >= 2^52: its phases would lose their fraction).
__device__ __forceinline__ bool cx_centre(double f, double fd, double T, double *qd, double *delta, double *d)
{
    const double x = (f + (fd * T) * 0.5) * T + 0.5;
    const double dd = (fd * T) * T;
    if (!(fabs(x) < 4503599627370496.0) || !(fabs(dd) < 1048576.0)) return false;
    *qd = floor(x);
    *delta = f * T - *qd;
    *d = dd;
    return true;
}

constexpr int NEX = 16;                        // entries of the exp(2 pi i k / NEX) table

// ex[k] = exp(2 pi i k / 16), set by the block's first threads.  The 16
// entries fill one row of LDS banks: the lanes of a wave read them without
// bank conflicts.
__device__ __forceinline__ void set_cis_table(double2 *ex)
{
    if (threadIdx.x < NEX) {
        double s, c;
        sincospi((double)threadIdx.x / (NEX / 2), &s, &c);
        ex[threadIdx.x] = make_double2(c, s);
    }
}

// exp(2 pi i t) for |t| < 2^26 turns: t = k/16 + r with k = rint(16 t) and
// |r| <= 1/32 (both exact), the table entry of k mod 16 times the Taylor
// polynomials of cos and sin at x = 2 pi r (|x| <= pi/16; the first omitted
// terms are below 2e-19).
__device__ __forceinline__ double2 cis_turns(double t, const double2 *ex)
{
    const double kd = rint(t * (double)NEX);
    const double r = fma(kd, -1.0 / NEX, t);
    const double2 e = ex[(int)kd & (NEX - 1)];
    const double x = r * 6.283185307179586;
    const double z = x * x;
    double c = fma(z, 1.0 / 479001600.0, -1.0 / 3628800.0);
    c = fma(z, c, 1.0 / 40320.0);
    c = fma(z, c, -1.0 / 720.0);
    c = fma(z, c, 1.0 / 24.0);
    c = fma(z, c, -0.5);
    c = fma(z, c, 1.0);
    double p = fma(z, -1.0 / 39916800.0, 1.0 / 362880.0);
    p = fma(z, p, -1.0 / 5040.0);
    p = fma(z, p, 1.0 / 120.0);
    p = fma(z, p, -1.0 / 6.0);
    const double sn = fma(x * z, p, x);
    return make_double2(fma(c, e.x, -(sn * e.y)), fma(c, e.y, sn * e.x));
}

__device__ __forceinline__ double2 cmulf(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

// The wave FFT.  Lane l holds the samples n = ell and ell + 64, where ell is
// l with its low three bits b mapped to b ^ 3 when b >= 4 (an involution):
// then the lanes that hold the positions ell and ell ^ 4 are l and l ^ 7,
// one DPP move apart, while positions ell ^ 8, ell ^ 2 and ell ^ 1 stay at
// l ^ 8, l ^ 2 and l ^ 1.
__device__ __forceinline__ int lane_pos(int l) { return l ^ ((l & 4) ? 3 : 0); }

// A lane's constants: its sample times x = n/128 with their squares, the
// twiddles of the in-lane stage (128 points), of the two row-swap stages
// (64 and 32 points, full butterflies in every lane) and of the spans 8
// and 4 (1 on the lane of the pair's first element), and the signs of the
// spans 8 .. 1 (+1 on the first element's lane, -1 on the other).
struct LaneFft {
    double x0, x0q, x1, x1q;
    double2 w1, wa, wb, w8, w4;
    double sg8, sg4, sg2, sg1;
};

__device__ __forceinline__ double2 twiddle(int m)   // exp(-2 pi i m / 128)
{
    double s, c;
    sincospi((double)m / (NF / 2), &s, &c);
    return make_double2(c, -s);
}

__device__ __forceinline__ LaneFft lane_fft()
{
    LaneFft L;
    const int e = lane_pos(lane()), u = e & 15;
    L.x0 = (double)e / NF;
    L.x1 = (double)(e + NF / 2) / NF;
    L.x0q = L.x0 * L.x0;
    L.x1q = L.x1 * L.x1;
    L.w1 = twiddle(e);                       // W_128^e
    L.wa = twiddle(2 * (e & 31));            // W_64^(e mod 32)
    L.wb = twiddle(4 * u);                   // W_32^(e mod 16)
    L.w8 = (u & 8) ? twiddle(8 * (u & 7)) : make_double2(1.0, 0.0);    // W_16
    L.w4 = (u & 4) ? twiddle(16 * (u & 3)) : make_double2(1.0, 0.0);   // W_8
    L.sg8 = (u & 8) ? -1.0 : 1.0;
    L.sg4 = (u & 4) ? -1.0 : 1.0;
    L.sg2 = (u & 2) ? -1.0 : 1.0;
    L.sg1 = (u & 1) ? -1.0 : 1.0;
    return L;
}

// The lane constants in LDS (18 values per lane, one row of doubles each), for
// kernels that need their registers between transforms.
constexpr int LFW = sizeof(LaneFft) / sizeof(double);

__device__ __forceinline__ void keep_fft(const LaneFft &L, double (*s)[64])
{
    const double *v = reinterpret_cast<const double *>(&L);
#pragma unroll
    for (int i = 0; i < LFW; ++i) s[i][lane()] = v[i];
}

__device__ __forceinline__ LaneFft kept_fft(const double (*s)[64])
{
    LaneFft L;
    double *v = reinterpret_cast<double *>(&L);
#pragma unroll
    for (int i = 0; i < LFW; ++i) v[i] = s[i][lane()];
    return L;
}

// Per-source constants of a template: index, centre bin, the phase
// delta x + dh x^2 in turns (dh = d/2), the scale sc = (A/2) (T/128) 2^E of
// the samples, and the channel rotations exp(i phi_A) = (ca, sa) and
// exp(i phi_E) = (ce, se); need: the template may reach the candidate cut
// (injection).
struct SrcConsts {
    uint32_t i;
    int qb;
    int need;
    double delta, dh, sc, ca, sa, ce, se;
};

// The 128-point DFT of the samples a (n = ell) and b (n = ell + 64) of each
// lane, by the whole wave: on return each lane holds two of its values, at
// the offsets lane_offsets gives.  Decimation in frequency: the first stage (n, n + 64)
// inside the lane gives the even and odd outputs as two 64-point DFTs a and
// b (registers P = a, Q = b).  The spans 32 and 16 are row swaps of P with
// Q, after which every lane holds both elements of one butterfly (of a or
// of b) and computes both outputs; the spans 8 .. 1 exchange within each
// register (the partner's value p and the own v give p + sg v, times the
// twiddle, so the first lane gets the sum and the second the difference).
__device__ __forceinline__ void wave_fft(double2 a, double2 b, const LaneFft &L, double2 *ue, double2 *uo)
{
    double2 P = cadd(a, b);
    double2 Q = cmulf(csub(a, b), L.w1);
    // span 32, then 16: full butterflies (twiddle 1 on the sum)
    row_swap<32>(&P.x, &Q.x);
    row_swap<32>(&P.y, &Q.y);
    {
        const double2 t = cadd(P, Q);
        Q = cmulf(csub(P, Q), L.wa);
        P = t;
    }
    row_swap<16>(&P.x, &Q.x);
    row_swap<16>(&P.y, &Q.y);
    {
        const double2 t = cadd(P, Q);
        Q = cmulf(csub(P, Q), L.wb);
        P = t;
    }
    // spans 8 and 4 (the latter between lanes l and l ^ 7)
    {
        const double2 p0 = partner2<8>(P), p1 = partner2<8>(Q);
        const double sg = L.sg8;
        P = cmulf(make_double2(fma(sg, P.x, p0.x), fma(sg, P.y, p0.y)), L.w8);
        Q = cmulf(make_double2(fma(sg, Q.x, p1.x), fma(sg, Q.y, p1.y)), L.w8);
    }
    {
        const double2 p0 = partner2<7>(P), p1 = partner2<7>(Q);
        const double sg = L.sg4;
        P = cmulf(make_double2(fma(sg, P.x, p0.x), fma(sg, P.y, p0.y)), L.w4);
        Q = cmulf(make_double2(fma(sg, Q.x, p1.x), fma(sg, Q.y, p1.y)), L.w4);
    }
    // span 2: twiddles 1 and -i (a swap and a sign); span 1: twiddle 1
    {
        const double2 p0 = partner2<2>(P), p1 = partner2<2>(Q);
        const double sg = L.sg2;
        const double2 d0 = make_double2(fma(sg, P.x, p0.x), fma(sg, P.y, p0.y));
        const double2 d1 = make_double2(fma(sg, Q.x, p1.x), fma(sg, Q.y, p1.y));
        const bool rot = (lane_pos(lane()) & 3) == 3;
        P = rot ? make_double2(d0.y, -d0.x) : d0;
        Q = rot ? make_double2(d1.y, -d1.x) : d1;
    }
    {
        const double2 p0 = partner2<1>(P), p1 = partner2<1>(Q);
        const double sg = L.sg1;
        *ue = make_double2(fma(sg, P.x, p0.x), fma(sg, P.y, p0.y));
        *uo = make_double2(fma(sg, Q.x, p1.x), fma(sg, Q.y, p1.y));
    }
}

// The template of one source, by the whole wave: 2^E U (U itself when sc =
// (A/2)(T/128)).  The phase is the definition's operations in their order
// (delta x, (d/2) x^2, their sum), so it is the same double as in a plain
// evaluation.
__device__ __forceinline__ void wave_template(const SrcConsts &c, const LaneFft &L, const double2 *ex,
                                              double2 *ue, double2 *uo)
{
    const double2 e0 = cis_turns(c.delta * L.x0 + c.dh * L.x0q, ex);
    const double2 e1 = cis_turns(c.delta * L.x1 + c.dh * L.x1q, ex);
    wave_fft(make_double2(c.sc * e0.x, c.sc * e0.y), make_double2(c.sc * e1.x, c.sc * e1.y), L, ue, uo);
}

// The value of a channel with rotation (c, s) = exp(i phi_c): exp(i phi_c) v.
__device__ __forceinline__ double2 rot(double2 v, double c, double s)
{
    return cmulf(v, make_double2(c, s));
}

// Template offsets j (in -64 .. 63) of a lane's two values.  After the
// FFT, register P of lane l (row r = l / 16) holds DFT a (rows 0, 1) or b
// (rows 2, 3) at position i = 32 (r mod 2) + (ell mod 16), and Q the same DFT
// at i + 16; position i of a 64-point decimation-in-frequency output is
// frequency bitrev6(i), and a and b are the even and odd outputs.
__device__ __forceinline__ void lane_offsets(int *je, int *jo)
{
    const int l = lane(), r = l >> 4;
    const int ip = 32 * (r & 1) + (lane_pos(l) & 15), iq = ip + 16;
    const int odd = r >= 2 ? 1 : 0;
    const int mp = 2 * (int)(__brev((unsigned)ip) >> 26) + odd, mq = 2 * (int)(__brev((unsigned)iq) >> 26) + odd;
    *je = mp < NF / 2 ? mp : mp - NF;
    *jo = mq < NF / 2 ? mq : mq - NF;
}

// A source's entry: valid (finite A >= 0, f > 0, finite fdot and phases).
__device__ __forceinline__ bool entry_ok(float A, float f, float fd, float pa, float pe)
{
    return isfinite(A) && A >= 0.0f && isfinite(f) && f > 0.0f && isfinite(fd) && isfinite(pa) && isfinite(pe);
}

// Grid bin of the centre, or INT_MIN when no bin of the template is on the grid.
__device__ __forceinline__ int centre_bin(const Grid &g, float f, float fd, double *delta, double *d)
{
    double qd;
    if (!cx_centre((double)f, (double)fd, g.T, &qd, delta, d)) return INT_MIN;
    const double qb = qd - (double)g.k0;
    if (qb + (HALO - 1) < 0.0 || qb - HALO > (double)(g.B - 1)) return INT_MIN;
    return (int)qb;
}

// Binning tile of a source centred at grid bin qb (clamped to the grid).
__device__ __forceinline__ int bin_tile(const Grid &g, int qb)
{
    const int k = qb < 0 ? 0 : (qb > g.B - 1 ? g.B - 1 : qb);
    return k / CX_TILE;
}

// ------------------------------------------------------------------ prep

// Clears the run's state and fills the grid tables: S_instr, 1/S_instr and its
// maximum over each 128-bin segment (a wave per segment).  (One launch: the
// tables in two of their own took 10 us more at 1e4 sources.)
__global__ __launch_bounds__(WG) void k_cx_reset(KArgs a)
{
    const Grid &g = a.g;
    const CxDev &d = a.d;
    const size_t stride = (size_t)gridDim.x * WG;
    const size_t i0 = (size_t)blockIdx.x * WG + threadIdx.x;
    const int nseg = (g.B + NF - 1) / NF;
    for (int seg = (int)(i0 >> 6); seg < nseg; seg += (int)(stride >> 6)) {
        double m = 0.0;
        for (int k = seg * NF + lane(); k < min((seg + 1) * NF, g.B); k += 64) {
            const double v = sinstr_dev((double)(g.k0 + k) / g.T, g.oms_pm, g.tm_fm, g.arm_m), i = 1.0 / v;
            d.sx[k] = v;
            d.isx[k] = i;
            m = fmax(m, i);
        }
        for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
        if (lane() == 0) d.isx_max[seg] = m;
    }
    for (size_t k = i0; k < 4 * (size_t)g.B; k += stride) d.h[k] = 0;
    for (size_t k = i0; k <= (size_t)d.ntc; k += stride) {
        d.tcnt[k] = 0;
        d.fcnt[k] = 0;
    }
    for (size_t k = i0; k < (size_t)g.nt; k += stride) {
        d.xstamp[k] = 0;
        d.sstamp[k] = 0;
        d.sdl[k] = (uint32_t)k;
    }
    if (i0 < 2) {                          // the A and E channels as two descriptors of the PSD kernels
        Slot sl{};
        sl.g = g;
        sl.d.sx = d.sx;
        sl.d.X = d.X + i0 * (size_t)g.B;
        sl.d.h = d.h + 2 * i0 * (size_t)g.B;
        sl.d.S = d.S + i0 * (size_t)g.B;
        sl.d.is_pre = d.is_pre + i0 * (size_t)g.B;
        sl.d.is_psum = d.is_psum + i0 * (size_t)g.nparts;
        sl.d.is_max = d.is_max + i0 * (size_t)((g.B + 63) / 64);
        sl.d.xstamp = d.xstamp;
        sl.d.sstamp = d.sstamp;
        sl.d.sdl = d.sdl;
        sl.d.ctl = d.ctl;
        sl.n = a.in.n;
        sl.active = 1;
        sl.prog = a.in.prog;
        d.slots[i0] = sl;
    }
    if (i0 == 0) {
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
        c->min_margin = c->margin = 0x7FF0000000000000ull;   // +inf
        c->units_x = 0;
        c->x_next = (uint32_t)g.B;
        c->units_med = (uint64_t)g.B;
        c->units_snr = 0;
        c->status = 0;
        c->med_split = (uint32_t)g.nt <= g.split_tiles;
        c->n_sdl = (uint32_t)g.nt;
        c->xupd = 0;
        c->tail_due = 0;
        c->n_new_body = 0;
        c->res_cursor = 0;
    }
}

// Whether the moment path takes a source (the "faint" sources, see
// k_cx_faint): centred on the grid, a chirp inside the range of its
// polynomial, and a lone SNR that cannot reach the candidate cut.  The last
// by Parseval (sum_j |U_j|^2 = T^2 A^2 / 4): rho_0^2 <= 2 T A^2 max 1/S_instr
// over the template's (at most two) segments.  With a cut above 1 the bound
// stays 1, so the data a set of sources gives do not depend on the
// thresholds.
__device__ __forceinline__ double lone_bound(const Grid &g, const double *isx_max, double A, int qb)
{
    const int g0 = max(qb - HALO, 0) / NF, g1 = min(qb + HALO - 1, g.B - 1) / NF;
    return 2.0 * g.T * (A * A) * fmax(isx_max[g0], isx_max[g1]) * (1.0 + 1e-9);
}

__device__ __forceinline__ bool is_faint(const Grid &g, const CxDev &d, float A, int qb, double dd)
{
    if (qb < 0 || qb >= g.B || !(fabs(dd) <= FAINT_MAX_D)) return false;
    return lone_bound(g, d.isx_max, (double)A, qb) < fmin(g.cut2, 1.0);
}

// One pass over the catalog: validity, the largest amplitude of the valid
// entries (it sets the fixed-point unit, a function of the catalog's size
// and amplitudes only), each source's key (its centre bin clamped to the
// grid and whether the moment path takes it) and the sources per binning
// tile, those of the moment path apart (LDS histogram per block, the two
// counts as 16-bit halves of a word).  Eight sources per thread in flight.
__global__ __launch_bounds__(WG) void k_cx_count(KArgs a)
{
    __shared__ uint32_t hist[CX_NTC_MAX];
    __shared__ uint32_t s_amax;
    const Grid &g = a.g;
    const CxDev &d = a.d;
    const CxIn &in = a.in;
    for (int t = threadIdx.x; t < d.ntc; t += WG) hist[t] = 0;
    if (threadIdx.x == 0) s_amax = 0;
    __syncthreads();
    const uint32_t b0 = blockIdx.x * (uint32_t)SRC_PB;
    const bool faint_n = in.n >= FAINT_MIN_N;
    uint32_t amax = 0, bad = 0;
    constexpr int U = 8;
    for (int r0 = 0; r0 < SRC_PB / WG; r0 += U) {
        float A[U], f[U], fd[U], pa[U], pe[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint32_t i = min(b0 + (uint32_t)((r0 + q) * WG) + threadIdx.x, in.n - 1u);
            A[q] = in.A[i];
            f[q] = in.F[i];
            fd[q] = in.FD[i];
            pa[q] = in.PA[i];
            pe[q] = in.PE[i];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint32_t i = b0 + (uint32_t)((r0 + q) * WG) + threadIdx.x;
            if (i >= in.n) continue;
            uint32_t key = KEY_NONE;
            if (!entry_ok(A[q], f[q], fd[q], pa[q], pe[q])) {
                bad = 1;
            } else {
                amax = max(amax, __float_as_uint(A[q]));
                double delta, dd;
                const int qb = centre_bin(g, f[q], fd[q], &delta, &dd);
                if (qb != INT_MIN) {
                    const bool faint = faint_n && is_faint(g, d, A[q], qb, dd);
                    key = (uint32_t)min(max(qb, 0), g.B - 1);
                    atomicAdd(&hist[key / CX_TILE], faint ? 0x10000u : 1u);
                    key |= faint ? KEY_FAINT : 0u;
                }
            }
            d.key[i] = key;
        }
    }
    if (bad) atomicOr(&d.ctl->bad, 1u);
    for (int o = 32; o >= 1; o >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, o, 64));
    if (lane() == 0) atomicMax(&s_amax, amax);
    __syncthreads();
    for (int t = threadIdx.x; t < d.ntc; t += WG) {
        const uint32_t h = hist[t];
        if (h & 0xFFFFu) atomicAdd(&d.tcnt[t], h & 0xFFFFu);
        if (h >> 16) atomicAdd(&d.fcnt[t], h >> 16);
    }
    if (threadIdx.x == 0 && s_amax) atomicMax(&d.ctl->amax_bits, s_amax);
}

// Exclusive prefix over the block's PLAN_T threads of three counts per
// thread; *tot gets their totals.  Contains two barriers.
struct Cnt3 {
    uint32_t a, b, c;
};

__device__ __forceinline__ Cnt3 plan_scan(Cnt3 x, Cnt3 *sw, Cnt3 *tot)
{
    const int l = lane(), w = threadIdx.x >> 6;
    Cnt3 i = x;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t ya = (uint32_t)__shfl_up((int)i.a, o, 64), yb = (uint32_t)__shfl_up((int)i.b, o, 64),
                       yc = (uint32_t)__shfl_up((int)i.c, o, 64);
        if (l >= o) {
            i.a += ya;
            i.b += yb;
            i.c += yc;
        }
    }
    __syncthreads();
    if (l == 63) sw[w] = i;
    __syncthreads();
    Cnt3 p = {i.a - x.a, i.b - x.b, i.c - x.c}, t = {0, 0, 0};
    for (int v = 0; v < PLAN_T / 64; ++v) {
        const Cnt3 y = sw[v];
        if (v < w) {
            p.a += y.a;
            p.b += y.b;
            p.c += y.c;
        }
        t.a += y.a;
        t.b += y.b;
        t.c += y.c;
    }
    *tot = t;
    return p;
}

// One block: the direct sources' tile offsets (tcnt becomes its exclusive
// prefix, tcnt[ntc] the total), scatter cursors and injection chunks per tile
// (cbase); and the faint buckets of each tile (fbb, exclusive prefix).
//
// Chunks: a tile's sources in blocks of `chunk`, the total over CH_GRID
// blocks rounded up to a power of two within [CH_MIN, CH].  A wave takes
// ~1.2 us per template, so a tile of 1000 sources in one chunk kept four
// waves busy for 300 us with the rest of the chip idle (1e4 sources, T = 1
// yr); past CH_GRID full chunks the fewer window flushes pay.
//
// Buckets: a tile's 1024 centres are cut into a power of two of equal ranges
// so that a bucket's estimated work, in wave instructions (a centre's
// moments ~1300, or its few templates ~240 each, and 16 per faint source), is
// at most the larger of 2^16 and a 3072nd of the catalog's.
__device__ __forceinline__ uint32_t faint_cost(uint32_t cnt)
{
    return min(240u * min(cnt, 1u << 20), 1300u * CX_TILE) / 64u + min(cnt, 1u << 28) / 4u;   // in units of 64
}

__global__ __launch_bounds__(PLAN_T) void k_cx_plan(KArgs a)
{
    constexpr int RUN = CX_NTC_MAX / PLAN_T;
    __shared__ Cnt3 sw[PLAN_T / 64];
    const CxDev &d = a.d;
    const int ntc = d.ntc;
    const int t0 = (int)threadIdx.x * RUN;
    uint32_t cnt[RUN], fc[RUN];
    Cnt3 s = {0, 0, 0}, tot;
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        cnt[r] = t0 + r < ntc ? d.tcnt[t0 + r] : 0u;
        fc[r] = t0 + r < ntc ? d.fcnt[t0 + r] : 0u;
        s.a += cnt[r];
        s.b += fc[r] ? faint_cost(fc[r]) : 0u;
    }
    (void)plan_scan(s, sw, &tot);
    const uint32_t want = (tot.a + CH_GRID - 1) / CH_GRID;
    uint32_t chunk = CH_MIN;
    while (chunk < want && chunk < (uint32_t)CH) chunk <<= 1;
    const uint32_t cap = max(1024u, tot.b / 3072u);
    uint32_t lb[RUN];
    s = {0, 0, 0};
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        s.a += cnt[r];
        s.b += (cnt[r] + chunk - 1) / chunk;
        lb[r] = 0;
        if (fc[r]) {
            const uint32_t c = faint_cost(fc[r]);
            while (lb[r] < 10u && (c >> lb[r]) > cap) ++lb[r];
            s.c += 1u << lb[r];
        }
    }
    Cnt3 p = plan_scan(s, sw, &tot);
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        if (t0 + r >= ntc) continue;
        d.tcnt[t0 + r] = p.a;
        d.tcur[t0 + r] = p.a;
        d.cbase[t0 + r] = p.b;
        d.fbb[t0 + r] = p.c;
        p.a += cnt[r];
        p.b += (cnt[r] + chunk - 1) / chunk;
        p.c += fc[r] ? 1u << lb[r] : 0u;
    }
    if (threadIdx.x == 0) {
        d.tcnt[ntc] = tot.a;
        d.cbase[ntc] = tot.b;
        d.fbb[ntc] = tot.c;
        d.ctl->n_chunks = chunk;
        d.ctl->n_events = tot.c;
        if (tot.c > (uint32_t)FB_MAX) d.ctl->bad |= 2u;    // cannot happen: ntc + 2 x 3072 at most
    }
}

// Groups the direct sources by binning tile: per block, an LDS count per
// tile, one global reservation of each tile's range, then LDS cursors in it.
__global__ __launch_bounds__(FB_T) void k_cx_scatter(KArgs a)
{
    __shared__ uint32_t cur[CX_NTC_MAX];
    const CxDev &d = a.d;
    const CxIn &in = a.in;
    for (int t = threadIdx.x; t < d.ntc; t += FB_T) cur[t] = 0;
    __syncthreads();
    const uint32_t b0 = blockIdx.x * (uint32_t)FB_SRC;
    int tile[FB_SRC / FB_T];
#pragma unroll
    for (int r = 0; r < FB_SRC / FB_T; ++r) {
        const uint32_t i = b0 + (uint32_t)(r * FB_T) + threadIdx.x;
        const uint32_t k = d.key[min(i, in.n - 1u)];
        tile[r] = i >= in.n || (k & KEY_FAINT) ? -1 : (int)(k / CX_TILE);      // KEY_NONE has the bit set
    }
#pragma unroll
    for (int r = 0; r < FB_SRC / FB_T; ++r)
        if (tile[r] >= 0) atomicAdd(&cur[tile[r]], 1u);
    __syncthreads();
    for (int t = threadIdx.x; t < d.ntc; t += FB_T)
        if (cur[t]) cur[t] = atomicAdd(&d.tcur[t], cur[t]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < FB_SRC / FB_T; ++r)
        if (tile[r] >= 0) d.order[atomicAdd(&cur[tile[r]], 1u)] = b0 + (uint32_t)(r * FB_T) + threadIdx.x;
}

// ---- the faint sources by bucket (catalogs of at least FAINT_MIN_N sources)
//
// As the power model's binning: a count pass writes each block's sources per
// bucket, a column pass turns them into offsets, and after a scan of the
// totals the scatter pass copies the records (amplitude, frequency,
// derivative, centre in the tile; phases) to their buckets, so that the
// moment blocks read contiguous memory instead of gathering five columns of
// a catalog in random order (64 bytes of HBM per 4-byte value).  A record has
// 24 bytes in one place, and the blocks of one XCD take
// neighbouring rows, whose slots of a bucket are neighbours: with a store per
// column and the rows dealt round-robin, a 128-byte line was written in
// parts by several XCDs' L2s (845 us for 1e7 sources).

// Row of the faint passes taken by this block: blocks go round-robin over
// the 8 XCDs, so XCD x gets the rows [x per, (x + 1) per).
__device__ __forceinline__ uint32_t faint_row(uint32_t rows)
{
    const uint32_t per = (rows + 7u) / 8u;
    return (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
}

// Bucket of a faint source and the tile map in LDS: word t holds the first
// bucket of tile t << 4 | log2(buckets of t).
__device__ __forceinline__ void load_bucket_map(const CxDev &d, uint32_t *map)
{
    for (int t = threadIdx.x; t < d.ntc; t += FB_T) {
        const uint32_t b = d.fbb[t], m = d.fbb[t + 1] - b;
        map[t] = (b << 4) | (m > 1u ? 31u - (uint32_t)__clz((int)m) : 0u);
    }
}

__device__ __forceinline__ uint32_t bucket_of(const uint32_t *map, uint32_t key)
{
    const uint32_t k = key & ~KEY_FAINT, w = map[k / CX_TILE];
    return (w >> 4) + ((k % CX_TILE) >> (10u - (w & 15u)));
}

template <int SRC> __global__ __launch_bounds__(FB_T) void k_cx_fcount(KArgs a)
{
    __shared__ uint32_t map[CX_NTC_MAX];
    __shared__ uint32_t hist[FB_MAX / 2];           // 16-bit counts
    const CxDev &d = a.d;
    const uint32_t nbk = d.ctl->n_events;
    if (d.ctl->bad) return;
    load_bucket_map(d, map);
    for (uint32_t b = threadIdx.x; b < (nbk + 1) / 2; b += FB_T) hist[b] = 0;
    __syncthreads();
    const uint32_t b0 = blockIdx.x * (uint32_t)SRC;
    uint32_t key[SRC / FB_T];
#pragma unroll
    for (int r = 0; r < SRC / FB_T; ++r) {
        const uint32_t i = b0 + (uint32_t)(r * FB_T) + threadIdx.x;
        key[r] = d.key[min(i, a.in.n - 1u)];
        if (i >= a.in.n) key[r] = KEY_NONE;
    }
#pragma unroll
    for (int r = 0; r < SRC / FB_T; ++r) {
        if (key[r] == KEY_NONE || !(key[r] & KEY_FAINT)) continue;
        const uint32_t b = bucket_of(map, key[r]);
        atomicAdd(&hist[b >> 1], 1u << (16 * (b & 1u)));
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nbk; b += FB_T)
        d.fmat[(size_t)blockIdx.x * nbk + b] = (hist[b >> 1] >> (16 * (b & 1u))) & 0xFFFFu;
}

// Column pass, in place: the sources of the blocks before, per bucket, and
// the bucket totals.  64 buckets per block, one per lane; the waves split
// the rows.
template <int SRC> __global__ __launch_bounds__(FB_T) void k_cx_fcols(KArgs a)
{
    constexpr int NV = FB_T / 64, U = 8;
    __shared__ uint32_t part[NV][64];
    const CxDev &d = a.d;
    const uint32_t nbk = d.ctl->n_events;
    if (blockIdx.x * 64u >= nbk || d.ctl->bad) return;
    const int l = lane(), w = threadIdx.x >> 6;
    const uint32_t b = blockIdx.x * 64u + (uint32_t)l;
    const bool ok = b < nbk;
    const uint32_t col = ok ? b : nbk - 1u;
    const uint32_t rows = (a.in.n + SRC - 1) / SRC, per = (rows + NV - 1) / NV;
    const uint32_t r0 = min(w * per, rows), r1 = min(r0 + per, rows);
    uint32_t sum = 0;
    for (uint32_t r = r0; r < r1; r += U) {
        uint32_t c[U];
#pragma unroll
        for (int q = 0; q < U; ++q) c[q] = d.fmat[(size_t)min(r + q, r1 - 1) * nbk + col];
#pragma unroll
        for (int q = 0; q < U; ++q) sum += r + q < r1 ? c[q] : 0u;
    }
    part[w][l] = sum;
    __syncthreads();
    uint32_t run = 0, tot = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const uint32_t x = part[v][l];
        run += v < w ? x : 0u;
        tot += x;
    }
    if (w == 0 && ok) d.ftot[b] = tot;
    for (uint32_t r = r0; r < r1; r += U) {
        uint32_t c[U];
#pragma unroll
        for (int q = 0; q < U; ++q) c[q] = d.fmat[(size_t)min(r + q, r1 - 1) * nbk + col];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (r + q >= r1) continue;
            if (ok) d.fmat[(size_t)(r + q) * nbk + b] = run;
            run += c[q];
        }
    }
}

// Bucket bases: ftot becomes its exclusive prefix, ftot[nbk] the total.
__global__ __launch_bounds__(PLAN_T) void k_cx_fscan(KArgs a)
{
    constexpr int RUN = FB_MAX / PLAN_T;
    __shared__ Cnt3 sw[PLAN_T / 64];
    const CxDev &d = a.d;
    const uint32_t nbk = d.ctl->n_events;
    if (d.ctl->bad) return;
    const uint32_t t0 = threadIdx.x * RUN;
    uint32_t c[RUN];
    Cnt3 s = {0, 0, 0}, tot;
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        c[r] = t0 + r < nbk ? d.ftot[t0 + r] : 0u;
        s.a += c[r];
    }
    Cnt3 p = plan_scan(s, sw, &tot);
#pragma unroll
    for (int r = 0; r < RUN; ++r) {
        if (t0 + r < nbk) d.ftot[t0 + r] = p.a;
        p.a += c[r];
    }
    if (threadIdx.x == 0) d.ftot[nbk] = tot.a;
}

// The faint sources' records by bucket.  A row has one or two sources for a
// bucket, so the records go to scattered lines that leave the caches partly
// filled: one record of 24 bytes per source, not two arrays.  9.4e6 sources:
// 267 us (two arrays 332 us).
template <int SRC> __global__ __launch_bounds__(FB_T) void k_cx_fscatter(KArgs a)
{
    __shared__ uint32_t map[CX_NTC_MAX];
    __shared__ uint32_t cur[FB_MAX];
    const CxDev &d = a.d;
    const CxIn &in = a.in;
    const uint32_t nbk = d.ctl->n_events;
    const uint32_t rows = (in.n + SRC - 1) / SRC, row = faint_row(rows);
    if (d.ctl->bad || row >= rows) return;
    load_bucket_map(d, map);
    for (uint32_t b = threadIdx.x; b < nbk; b += FB_T) cur[b] = d.ftot[b] + d.fmat[(size_t)row * nbk + b];
    __syncthreads();
    const uint32_t b0 = row * (uint32_t)SRC;
    constexpr int U = 4;
    for (int r0 = 0; r0 < SRC / FB_T; r0 += U) {
        uint32_t key[U];
        float A[U], f[U], fd[U], pa[U], pe[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint32_t i = b0 + (uint32_t)((r0 + q) * FB_T) + threadIdx.x, ic = min(i, in.n - 1u);
            key[q] = d.key[ic];
            A[q] = in.A[ic];
            f[q] = in.F[ic];
            fd[q] = in.FD[ic];
            pa[q] = in.PA[ic];
            pe[q] = in.PE[ic];
            if (i >= in.n) key[q] = KEY_NONE;
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (key[q] == KEY_NONE || !(key[q] & KEY_FAINT)) continue;
            const uint32_t p = atomicAdd(&cur[bucket_of(map, key[q])], 1u);
            d.frec[p] = FaintRec{A[q], f[q], fd[q], (key[q] & ~KEY_FAINT) % CX_TILE, {pa[q], pe[q]}};
        }
    }
}

// The channel rotations of source i.
__device__ __forceinline__ void rotations(const CxIn &in, uint32_t i, SrcConsts *c)
{
    sincos((double)in.PA[i], &c->sa, &c->ca);
    sincos((double)in.PE[i], &c->se, &c->ce);
}

// The constants of source i (one source per lane) with fixed-point
// exponent E; the channel rotations only when rot.
__device__ __forceinline__ SrcConsts src_consts(const Grid &g, const CxIn &in, uint32_t i, int E, bool rot)
{
    SrcConsts c;
    double d;
    c.i = i;
    c.need = 1;
    c.qb = centre_bin(g, in.F[i], in.FD[i], &c.delta, &d);
    c.dh = d * 0.5;
    c.sc = ldexp(((double)in.A[i] * 0.5) * (g.T / NF), E);
    c.ca = c.sa = c.ce = c.se = 0.0;
    if (rot) rotations(in, i, &c);
    return c;
}

// Lane k's constants (k wave-uniform), on every lane.
__device__ __forceinline__ double rl(double v, int k)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), k);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ SrcConsts bcast(const SrcConsts &c, int k)
{
    SrcConsts r;
    r.i = (uint32_t)__builtin_amdgcn_readlane((int)c.i, k);
    r.qb = __builtin_amdgcn_readlane(c.qb, k);
    r.need = __builtin_amdgcn_readlane(c.need, k);
    r.delta = rl(c.delta, k);
    r.dh = rl(c.dh, k);
    r.sc = rl(c.sc, k);
    r.ca = rl(c.ca, k);
    r.sa = rl(c.sa, k);
    r.ce = rl(c.ce, k);
    r.se = rl(c.se, k);
    return r;
}

// ---- the moment path
//
// The templates of all sources with the same centre bin share their bins,
// and the DFT is linear: their samples are summed first and transformed
// once per centre and channel.  The sum itself costs less than a sample per
// source.  Around mid-observation (z = 2x - 1) a source's samples are
// w exp(i (a z + b z^2)), a = pi (delta + d/2), |a| <= pi/2 (delta + d/2 is
// the distance of the mid-frequency from its bin), b = pi d/4, |b| <= 1/4 by
// the choice of the faint sources, w = (A/2)(T/128) exp(i (phi_c + 2 pi
// (delta/2 + d/8))).  The Taylor coefficients G_k i^k in z follow
//   G_0 = w, G_1 = a w, G_{k+1} = (a G_k - 2 i b G_{k-1}) / (k + 1),
// and NMOM = 28 of them give the exponential on |z| <= 1 to 2e-15 at the
// worst (|a| = pi/2 and |b| = 1/4; 2e-17 for |b| <= 0.14).  So a source costs
// 28 short steps in one lane, where its template took the whole wave ~240
// instructions.  The sums over a centre's sources are the samples' polynomial.
//
// The coefficients are summed as integers (unit 2^-E7, E7 from the largest
// amplitude: every coefficient stays below 2^50, and centres with more than
// 4096 sources take a coarser unit so that no sum leaves 64 bits): the sum
// does not depend on the order of a centre's sources, which the grouping
// leaves open.  A coefficient's unit reaches a value of the template 2^7 times
// (the DFT's 128 samples): with v = A T/2 of the loudest source it is 2^-48 v
// there, and 2^-(59 - k) v for a centre of more than 4096 sources, at least 2^k of
// them; h, and a template rounded on its own, has 2^-(61 - log2 n) v, 2^-45 v or
// more.  So the unit is the finer one unless a centre holds more than a quarter
// of the catalog, and at most four times the other then.  h is rounded once per
// centre.
//
// Only sources that can never be candidates are taken, so none is ever
// subtracted: h stays the same integer whatever subset of the candidates is
// left.

// Unit of a centre's coefficients.
__device__ __forceinline__ int moment_exp(uint32_t amax_bits, uint32_t cnt, double T)
{
    const double v = (double)__uint_as_float(amax_bits) * (T * 0.5);
    if (!(v > 0.0)) return 0;
    return 55 - ilogb(v) - (cnt > 4096u ? 20 - __clz((int)cnt) : 0);
}

// u64 lane exchanges as for doubles above.
template <int SPAN> __device__ __forceinline__ uint64_t swap_add(uint64_t p, uint64_t q)
{
    double P = __longlong_as_double((long long)p), Q = __longlong_as_double((long long)q);
    row_swap<SPAN>(&P, &Q);
    return (uint64_t)__double_as_longlong(P) + (uint64_t)__double_as_longlong(Q);
}

template <int PAT> __device__ __forceinline__ uint64_t fold_add(uint64_t lo, uint64_t hi, bool up)
{
    const uint64_t keep = up ? hi : lo, send = up ? lo : hi;
    return keep + (uint64_t)__double_as_longlong(partner<PAT>(__longlong_as_double((long long)send)));
}

// exp(i phi): phases of a few turns through the table (phi/(2 pi) as the
// rounded product plus its error), others by the library's reduction.
__device__ __forceinline__ double2 phase_factor(float phi, const double2 *ex)
{
    if (__builtin_expect(fabsf(phi) <= 8.0f, 1)) {
        const double p = (double)phi, t = p * 0.15915494309189535;
        const double e = fma(p, 0.15915494309189535, -t) - p * 9.839338337591009e-18;
        return cis_turns(t + e, ex);
    }
    double sp, cp;
    sincos((double)phi, &sp, &cp);
    return make_double2(cp, sp);
}

// Integer sums of the coefficients over the sources order[o], o = o0 + l,
// o0 + l + step, ... < o1, l = lane mod 32: each half of the wave sums one
// channel, lane k of half ch gets Re G_k and Im G_k of channel ch (wrapping
// 64-bit sums; lanes k >= NMOM get 0).  A value is rounded to its unit by
// adding 1.5 2^52 and its bits are added as they are; the constant part of the
// bits leaves at the end.
// Channels by halves: one fold of 56 sums for both channels where a wave per
// channel folded twice, and most centres have fewer than 32 sources, which
// left half of such a wave idle.
__device__ __forceinline__ void moment_sums(const KArgs &a, uint32_t o0, uint32_t o1, uint32_t step, int E7,
                                            const double2 *ex, uint64_t *re, uint64_t *im)
{
    const CxDev &d = a.d;
    const double T = a.g.T, scale = ldexp(T / NF * 0.5, E7);
    const int ch = lane() >> 5;
    uint64_t sr[NMOM], si[NMOM];
#pragma unroll
    for (int k = 0; k < NMOM; ++k) sr[k] = si[k] = 0;
    uint32_t turns = 0;
    // the next turn's record is loaded while this one's coefficients are
    // summed, and its place in the order one turn before that
    const uint32_t last = o1 - 1u, l = (uint32_t)lane() & 31u;
    uint32_t p = 0, pn = 0;
    float rA = 0.0f, rf = 0.0f, rd = 0.0f, ph = 0.0f;
    auto load = [&](uint32_t q) {
        const FaintRec &r = d.frec[q];
        rA = r.A;
        rf = r.f;
        rd = r.fd;
        ph = r.ph[ch];
    };
    if (o0 < o1) {
        p = d.forder[min(o0 + l, last)];
        pn = d.forder[min(o0 + step + l, last)];
        load(p);
    }
    for (uint32_t o = o0; o < o1; o += step, ++turns) {
        const bool in = o + l < o1;
        const float cA = rA, cf = rf, cd = rd, cph = ph;
        load(pn);
        pn = d.forder[min(o + 2u * step + l, last)];
        double qd, delta, dd;
        cx_centre((double)cf, (double)cd, T, &qd, &delta, &dd);
        const double al = 3.141592653589793 * (delta + 0.5 * dd);
        const double be2 = 1.5707963267948966 * dd;                       // 2b = pi d / 2
        // w = (A/2)(T/128) 2^E7 exp(i (phi + 2 pi (delta/2 + d/8)))
        const double sc = in ? (double)cA * scale : 0.0;
        double2 r = cis_turns(0.5 * delta + 0.125 * dd, ex);
        r = cmulf(r, phase_factor(cph, ex));
        r = make_double2(sc * r.x, sc * r.y);
        double gr = r.x, gi = r.y, hr = 0.0, hi = 0.0;                    // G_k, G_{k-1}
#pragma unroll
        for (int k = 0; k < NMOM; ++k) {
            sr[k] += (uint64_t)__double_as_longlong(gr + 6755399441055744.0);
            si[k] += (uint64_t)__double_as_longlong(gi + 6755399441055744.0);
            if (k + 1 < NMOM) {
                const double ak = al * (1.0 / (k + 1)), bk = be2 * (1.0 / (k + 1));
                const double nr = fma(ak, gr, bk * hi), ni = fma(ak, gi, -(bk * hr));
                hr = gr;
                hi = gi;
                gr = nr;
                gi = ni;
            }
        }
    }
    // lane l of a half ends with the sums of values 2l and 2l + 1: halves of
    // the values change places between the half's rows, then within the rows
    static_assert(NMOM == 28, "56 values: the folds below");
    uint64_t v[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const int m = j + 32;                                             // values 56 .. 63 are zero
        v[j] = swap_add<16>(j & 1 ? si[j / 2] : sr[j / 2], m < 2 * NMOM ? (j & 1 ? si[m / 2] : sr[m / 2]) : 0ull);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = fold_add<8>(v[j], v[j + 16], lane() & 8);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = fold_add<7>(v[j], v[j + 8], lane() & 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = fold_add<2>(v[j], v[j + 4], lane() & 2);
#pragma unroll
    for (int j = 0; j < 2; ++j) v[j] = fold_add<1>(v[j], v[j + 2], lane() & 1);
    const uint64_t base = (uint64_t)turns * 32ull * 0x4338000000000000ull;
    *re = l < (uint32_t)NMOM ? v[0] - base : 0ull;
    *im = l < (uint32_t)NMOM ? v[1] - base : 0ull;
}

// One block per bucket: the bucket's sources are ordered by centre (LDS
// counts; centres with fewer than MOM_MIN sources last, their sources take
// one template each), then every centre is a wave's task: the moment sums of
// both channels, and per channel the polynomial at the wave's 128 sample times
// (Horner, the coefficients broadcast by readlane), one FFT, and the values
// into the window.  A centre of more than MOM_COOP sources is shared by the block's
// waves.
// Bound by VALU issue and the dependent steps of a task (two waves per SIMD:
// 56 sums of 64 bits per lane).  1e7 sources on the 4-yr grid: 590 us for the
// 9.4e6 faint ones (690 us with a wave per channel of a centre), plus 380 us of
// grouping and 300 us for the others' templates, against 6500 us (and 110 us
// of grouping) with one template per source.  MOM_MIN: a centre's sums cost
// about 1800 wave instructions for both channels and up to 32 sources (turn
// 450, folds 330, two times Horner, FFT and rounding 500), 2600 with a wave per
// channel, a template 240; 8 and 6 measure the same as 12 within 1 % (4.1e5
// and 1e7 sources).
__global__ __launch_bounds__(WG, 2) void k_cx_faint(KArgs a)
{
    constexpr int NW = WG / 64;
    __shared__ long long acc[4][2][CXW / 2];
    __shared__ uint32_t cnt[CX_TILE], beg[CX_TILE];
    __shared__ double2 ex[NEX];
    __shared__ double lf[LFW][64];
    __shared__ unsigned long long msum[2][64];
    __shared__ uint64_t sw[NW];
    const Grid &g = a.g;
    const CxDev &d = a.d;
    const uint32_t b = blockIdx.x;
    if (d.ctl->bad || b >= d.ctl->n_events) return;
    const uint32_t m0 = d.ftot[b], m1 = d.ftot[b + 1];
    if (m0 == m1) return;
    int lo = 0, hi = d.ntc - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (d.fbb[mid] <= b) lo = mid; else hi = mid - 1;
    }
    const int tile = lo;
    const int width = CX_TILE / (int)(d.fbb[tile + 1] - d.fbb[tile]);
    const int c0 = tile * CX_TILE + (int)(b - d.fbb[tile]) * width;       // the bucket's first centre
    const int nwin = width + NF, w0 = c0 - HALO;
    for (int k = threadIdx.x; k < 4 * CXW; k += WG) (&acc[0][0][0])[k] = 0;
    for (int k = threadIdx.x; k < width; k += WG) cnt[k] = 0;
    if (threadIdx.x < 128) (&msum[0][0])[threadIdx.x] = 0;
    set_cis_table(ex);
    if (threadIdx.x < 64) keep_fft(lane_fft(), lf);
    auto centre = [&](uint32_t p) { return (int)d.frec[p].centre & (width - 1); };
    __syncthreads();
    for (uint32_t p = m0 + threadIdx.x; p < m1; p += WG) atomicAdd(&cnt[centre(p)], 1u);
    __syncthreads();
    // offsets: the centres of at least MOM_MIN sources in order, then the others
    uint32_t nbig;
    {
        constexpr int R = CX_TILE / WG;
        uint64_t own = 0;
        for (int r = 0; r < R; ++r) {
            const int c = (int)threadIdx.x * R + r;
            const uint64_t x = c < width ? cnt[c] : 0u;
            own += x >= (uint64_t)MOM_MIN ? x << 32 : x;
        }
        uint64_t inc = own;
        for (int o = 1; o < 64; o <<= 1) {
            const uint64_t y = (uint64_t)__shfl_up((long long)inc, o, 64);
            if (lane() >= o) inc += y;
        }
        if (lane() == 63) sw[threadIdx.x >> 6] = inc;
        __syncthreads();
        uint64_t run = inc - own, tot = 0;
        for (int v = 0; v < NW; ++v) {
            run += v < (int)(threadIdx.x >> 6) ? sw[v] : 0ull;
            tot += sw[v];
        }
        nbig = (uint32_t)(tot >> 32);
        for (int r = 0; r < R; ++r) {
            const int c = (int)threadIdx.x * R + r;
            if (c >= width) break;
            const uint64_t x = cnt[c];
            const bool big = x >= (uint64_t)MOM_MIN;
            beg[c] = big ? (uint32_t)(run >> 32) : nbig + (uint32_t)run;
            run += big ? x << 32 : x;
        }
        __syncthreads();
    }
    for (uint32_t p = m0 + threadIdx.x; p < m1; p += WG)
        d.forder[m0 + atomicAdd(&beg[centre(p)], 1u)] = p;
    __syncthreads();                                  // beg: now the end of each centre's range

    const int E = cx_exp(d.ctl->amax_bits, a.in.n, g.T);
    const uint32_t amax = d.ctl->amax_bits;
    const int wave = (int)(threadIdx.x >> 6);
    int je, jo;
    lane_offsets(&je, &jo);
    auto put = [&](int bin, int word, long long v) {
        atomicAdd((unsigned long long *)&acc[word][(bin - w0) & 1][(bin - w0) >> 1], (unsigned long long)v);
    };
    auto unit = [&](uint64_t sum, int E7) { return ldexp((double)(long long)sum, E - E7); };
    // the transform of a centre's sums of channel ch (lane k: Re G_k, Im G_k)
    auto transform = [&](double vr, double vi, int c, int ch) {
        const LaneFft L = kept_fft(lf);
        const double z0 = 2.0 * L.x0 - 1.0, z1 = 2.0 * L.x1 - 1.0;
        double2 p0 = make_double2(0.0, 0.0), p1 = p0;
#pragma unroll
        for (int k = NMOM - 1; k >= 0; --k) {
            const double mr = rl(vr, k), mi = rl(vi, k);
            const double cx = k % 4 == 0 ? mr : k % 4 == 1 ? -mi : k % 4 == 2 ? -mr : mi;     // i^k G_k
            const double cy = k % 4 == 0 ? mi : k % 4 == 1 ? mr : k % 4 == 2 ? -mi : -mr;
            p0 = make_double2(fma(p0.x, z0, cx), fma(p0.y, z0, cy));
            p1 = make_double2(fma(p1.x, z1, cx), fma(p1.y, z1, cy));
        }
        double2 ue, uo;
        wave_fft(p0, p1, L, &ue, &uo);
        put(c0 + c + je, 2 * ch, __double2ll_rn(ue.x));
        put(c0 + c + je, 2 * ch + 1, __double2ll_rn(ue.y));
        put(c0 + c + jo, 2 * ch, __double2ll_rn(uo.x));
        put(c0 + c + jo, 2 * ch + 1, __double2ll_rn(uo.y));
    };
    for (int c = wave; c < width; c += NW) {
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)cnt[c]);
        if (n < (uint32_t)MOM_MIN || n > (uint32_t)MOM_COOP) continue;
        const uint32_t e = m0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)beg[c]);
        const int E7 = moment_exp(amax, n, g.T);
        uint64_t re, im;
        moment_sums(a, e - n, e, 32u, E7, ex, &re, &im);
        double vr = unit(re, E7), vi = unit(im, E7);
#pragma unroll 1
        for (int ch = 0;; ++ch) {
            transform(vr, vi, c, ch);
            if (ch == 1) break;
            double t = vr, u = vi;
            row_swap<32>(&t, &vr);                    // both halves: the second channel
            row_swap<32>(&u, &vi);
        }
    }
    if (m1 - m0 > (uint32_t)MOM_COOP) {               // block-uniform
        for (int c = 0; c < width; ++c) {
            const uint32_t n = cnt[c];
            if (n <= (uint32_t)MOM_COOP) continue;
            const uint32_t e = m0 + beg[c];
            const int E7 = moment_exp(amax, n, g.T);
            uint64_t re, im;
            moment_sums(a, e - n + 32u * (uint32_t)wave, e, 32u * NW, E7, ex, &re, &im);
            atomicAdd(&msum[0][lane()], (unsigned long long)re);
            atomicAdd(&msum[1][lane()], (unsigned long long)im);
            __syncthreads();
            if (wave < 2) {
                const int k = 32 * wave + (lane() & 31);
                transform(unit(msum[0][k], E7), unit(msum[1][k], E7), c, wave);
                msum[lane() >> 5][k] = 0;
            }
            __syncthreads();
        }
    }
    // the others: one template each
    const uint32_t s0 = m0 + nbig, share = (m1 - s0 + NW - 1) / NW;
    const uint32_t v0 = min(s0 + (uint32_t)wave * share, m1), v1 = min(v0 + share, m1);
    const LaneFft L = kept_fft(lf);
    for (uint32_t base = v0; base < v1; base += 64u) {
        const uint32_t p = d.forder[min(base + (uint32_t)lane(), v1 - 1u)];
        SrcConsts mine{};
        double dd;
        const FaintRec rec = d.frec[p];
        mine.qb = centre_bin(g, rec.f, rec.fd, &mine.delta, &dd);
        mine.dh = dd * 0.5;
        mine.sc = ldexp(((double)rec.A * 0.5) * (g.T / NF), E);
        const double2 ra = phase_factor(rec.ph[0], ex), re = phase_factor(rec.ph[1], ex);
        mine.ca = ra.x;
        mine.sa = ra.y;
        mine.ce = re.x;
        mine.se = re.y;
        const int n = (int)min(64u, v1 - base);
        for (int k = 0; k < n; ++k) {
            const SrcConsts c = bcast(mine, k);
            double2 ue, uo;
            wave_template(c, L, ex, &ue, &uo);
            const double2 ae = rot(ue, c.ca, c.sa), ee = rot(ue, c.ce, c.se);
            const double2 ao = rot(uo, c.ca, c.sa), eo = rot(uo, c.ce, c.se);
            put(c.qb + je, 0, fxm(ae.x));
            put(c.qb + je, 1, fxm(ae.y));
            put(c.qb + je, 2, fxm(ee.x));
            put(c.qb + je, 3, fxm(ee.y));
            put(c.qb + jo, 0, fxm(ao.x));
            put(c.qb + jo, 1, fxm(ao.y));
            put(c.qb + jo, 2, fxm(eo.x));
            put(c.qb + jo, 3, fxm(eo.y));
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nwin; k += WG) {
        const int bin = w0 + k;
        if (bin < 0 || bin >= g.B) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const long long v = acc[c][k & 1][k >> 1];
            if (v) atomicAdd((unsigned long long *)&d.h[(size_t)c * g.B + bin], (unsigned long long)v);
        }
    }
}

// Direct injection: h += every template of the sources the moment path does
// not take (both channels), and the candidate cut
// rho_0^2 = (8/T) sum_j |U_j|^2 / S_instr >= (kappa rho_th)^2.  One block per
// chunk of sources of one binning tile (k_cx_plan); each wave takes 64
// sources at a time, their constants computed one per lane, then one
// template after the other by the whole wave.  The batch's candidates are
// recorded together: lane k keeps rho_0^2 of source k, one reservation for
// all (one same-address atomic per batch instead of one per candidate).
__global__ __launch_bounds__(WG) void k_cx_inject(KArgs a)
{
    // per channel word, the window's even bins then its odd bins (w0 is
    // even): the lanes of one atomic add hit pairs of neighbouring words
    __shared__ long long acc[4][2][CXW / 2];
    __shared__ double2 ex[NEX];
    const Grid &g = a.g;
    const CxDev &d = a.d;
    const CxIn &in = a.in;
    const uint32_t b = blockIdx.x;
    if (b >= d.cbase[d.ntc]) return;
    // the tile of this chunk: the last t with cbase[t] <= b
    int lo = 0, hi = d.ntc - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (d.cbase[mid] <= b) lo = mid; else hi = mid - 1;
    }
    const int tile = lo;
    const uint32_t chunk = d.ctl->n_chunks;
    const uint32_t s0 = d.tcnt[tile] + (b - d.cbase[tile]) * chunk;
    const uint32_t s1 = min(s0 + chunk, d.tcnt[tile + 1]);
    for (int k = threadIdx.x; k < 4 * CXW; k += WG) (&acc[0][0][0])[k] = 0;
    set_cis_table(ex);
    const LaneFft L = lane_fft();
    __syncthreads();
    const int E = cx_exp(d.ctl->amax_bits, in.n, g.T);
    const int w0 = tile * CX_TILE - HALO;        // grid bin of the window's first bin
    int je, jo;
    lane_offsets(&je, &jo);
    const double cut2 = g.cut2, T = g.T;
    // rho_0^2 of the 2^E-scaled values: (8/T) 2^-2E sum
    const double r0s = ldexp(8.0 / T, -2 * E);
    // each wave takes an equal share of the chunk, 64 sources at a time
    const uint32_t wave = threadIdx.x >> 6, share = (s1 - s0 + WG / 64 - 1) / (WG / 64);
    const uint32_t v0 = s0 + wave * share, v1 = min(v0 + share, s1);
    for (uint32_t base = v0; base < v1; base += 64u) {
        const uint32_t s = base + (uint32_t)lane();
        SrcConsts mine = src_consts(g, in, d.order[s < v1 ? s : v0], E, true);
        {
            // below the candidate cut by the bound: no exact sum
            mine.need = lone_bound(g, d.isx_max, (double)in.A[mine.i], mine.qb) >= cut2;
        }
        double myr0 = -1.0;                      // rho_0^2 of this lane's source (none: below the cut)
        // the candidate cut and the template's values into the window
        auto add = [&](const SrcConsts &c, int k, const double2 &ue, const double2 &uo) {
            const int be = c.qb + je, bo = c.qb + jo;
            const bool ine = be >= 0 && be < g.B, ino = bo >= 0 && bo < g.B;
            if (c.need) {
                const double pe = ue.x * ue.x + ue.y * ue.y, po = uo.x * uo.x + uo.y * uo.y;
                double r = (ine ? pe * d.isx[be] : 0.0) + (ino ? po * d.isx[bo] : 0.0);
                const double r0 = r0s * wave_sum(r);
                if (lane() == k) myr0 = r0;
            }
            if (ine) {
                const double2 va = rot(ue, c.ca, c.sa), ve = rot(ue, c.ce, c.se);
                unsigned long long *p = (unsigned long long *)&acc[0][(be - w0) & 1][(be - w0) >> 1];
                atomicAdd(p, (unsigned long long)fxm(va.x));
                atomicAdd(p + CXW, (unsigned long long)fxm(va.y));
                atomicAdd(p + 2 * CXW, (unsigned long long)fxm(ve.x));
                atomicAdd(p + 3 * CXW, (unsigned long long)fxm(ve.y));
            }
            if (ino) {
                const double2 va = rot(uo, c.ca, c.sa), ve = rot(uo, c.ce, c.se);
                unsigned long long *p = (unsigned long long *)&acc[0][(bo - w0) & 1][(bo - w0) >> 1];
                atomicAdd(p, (unsigned long long)fxm(va.x));
                atomicAdd(p + CXW, (unsigned long long)fxm(va.y));
                atomicAdd(p + 2 * CXW, (unsigned long long)fxm(ve.x));
                atomicAdd(p + 3 * CXW, (unsigned long long)fxm(ve.y));
            }
        };
        const int cnt = (int)min(64u, v1 - base);
        for (int k = 0; k < cnt; ++k) {
            const SrcConsts c = bcast(mine, k);
            double2 ue, uo;
            wave_template(c, L, ex, &ue, &uo);
            add(c, k, ue, uo);
        }
        const bool cand = lane() < cnt && mine.need && myr0 >= cut2;
        const uint64_t m = (uint64_t)__ballot(cand);
        if (m) {
            uint32_t slot = 0;
            if (lane() == 0) slot = atomicAdd(&d.ctl->cand_cursor, (uint32_t)__popcll(m));
            slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
            if (cand) {
                slot += (uint32_t)__popcll(m & ((1ull << lane()) - 1ull));
                d.c_src[slot] = mine.i;
                d.c_iter[slot] = -1;
                d.c_rho2[slot] = myr0;
                d.c_qb[slot] = mine.qb;
                d.c_amp[slot] = in.A[mine.i];
            }
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < CXW; k += WG) {
        const int bin = w0 + k;
        if (bin < 0 || bin >= g.B) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const long long v = acc[c][k & 1][k >> 1];
            if (v) atomicAdd((unsigned long long *)&d.h[(size_t)c * g.B + bin], (unsigned long long)v);
        }
    }
}

// ------------------------------------------------------------------ loop body

// X_c = (2/T) |h_c|^2 on the tiles stamped for this body.
__global__ __launch_bounds__(WG) void k_cx_power(KArgs a)
{
    const Grid &g = a.g;
    const CxDev &d = a.d;
    Ctl *c = d.ctl;
    if (c->done || c->bad) return;
    const int tile = blockIdx.x;
    if (tile == 0 && threadIdx.x == 0) c->units_x += c->x_next;
    if (tile >= g.nt || d.xstamp[tile] != c->iter) return;
    const int E = cx_exp(c->amax_bits, a.in.n, g.T);
    const double s2 = 2.0 / g.T;
    const int t0 = tile * g.tile, t1 = min(t0 + g.tile, g.B);
    const size_t B = (size_t)g.B;
    for (int k = t0 + (int)threadIdx.x; k < t1; k += WG) {
        const double ra = ldexp((double)d.h[k], -E), ia = ldexp((double)d.h[B + k], -E);
        const double re = ldexp((double)d.h[2 * B + k], -E), ie = ldexp((double)d.h[3 * B + k], -E);
        d.X[k] = s2 * (ra * ra + ia * ia);
        d.X[B + k] = s2 * (re * re + ie * ie);
    }
}

// rho^2 of every unsubtracted candidate whose template meets a tile
// refiltered in this body (or stamped for the next one by a subtraction of
// this launch: re-evaluating against an unchanged S gives the same value, so
// only the count of evaluations may differ between two runs);
// rho^2 > rho_th^2 subtracts its templates from h at once and stamps the
// tiles whose X and S change.  Each wave takes 64 candidates at a time: the
// lanes find which need an evaluation and their constants, then the wave
// evaluates them one after the other (0.9 us each).  The candidates of one
// region follow each other in slot order (injection chunks), so a wave takes
// groups of GRP consecutive ones from places all over the list: with 64
// consecutive ones, a late body's few dirty tiles kept a few waves busy for
// 64 evaluations in a row while the others had none (SNR of the 1e4 catalog
// 30 us a run instead of 169, of the 1e7 catalog 1.68 ms instead of 2.13).
//
// Most candidates cannot reach the threshold: by Parseval (sum_j |U_j|^2 = T^2
// A^2 / 4) rho^2 <= T A^2 (max 1/S_A + max 1/S_E) over the template's bins, and
// the PSD launches leave the maxima of every 64-bin segment.  From the second
// body on, a candidate whose bound stays below the threshold by more than
// the smallest margin of the bodies before (and the 1e-6 that counts as near;
// not the running body's, which its waves lower at their own times) is not
// evaluated: it is not resolved, and neither the margin nor the near count
// would change.  Its rho^2 is marked stale (-1) and computed after the loop
// (FINAL: S on its bins is still that of its last body; its evaluations are
// counted only for the kernel statistics, where one same-address atomic per
// wave costs 50 us at 1e7 sources).  SNR of the 1e7 catalog 1.01 ms a run, the
// last pass's 0.08 included, 1.66 with every candidate evaluated; 4.1e5 sources (2
// yr, mean) 102 and 123 us.  Whole runs of small catalogs (1 yr), with and without
// the bound: 2e3 sources 250 and 236 us, 8e3 268 and 261, 1.6e4 292 and 287,
// 2.4e4 346 and 340, 3.2e4 361 and 363, 6.5e4 441 and 463.  Below BOUND_MIN_N
// the evaluations fit one round of waves and the last pass's 5 to 14 us is all it
// changes; from there to 3e4 the two are within 2 %.
template <bool FINAL, bool COUNT>
__global__ __launch_bounds__(WG, 4) void k_cx_snr(KArgs a)
{
    __shared__ double2 ex[NEX];
    const Grid &g = a.g;
    const CxDev &d = a.d;
    const CxIn &in = a.in;
    Ctl *c = d.ctl;
    set_cis_table(ex);
    __syncthreads();
    if (c->bad || (!FINAL && c->done)) return;
    const uint32_t t = c->iter, nxt = t + 1;
    const uint32_t nc = c->cand_cursor;
    const double margin = fmax(__longlong_as_double((long long)c->margin), 2e-6);
    const double skip2 = margin < 1.0 ? g.rth2 * (1.0 - margin) * (1.0 - margin) * (1.0 - 1e-9) : 0.0;
    const int E = cx_exp(c->amax_bits, in.n, g.T);
    const double T = g.T;
    // rho^2 of the 2^E-scaled values: (4/T) 2^-2E sum
    const double rs = ldexp(4.0 / T, -2 * E);
    const size_t B = (size_t)g.B;
    int je, jo;
    lane_offsets(&je, &jo);
    const uint32_t waves = gridDim.x * (WG / 64), wave = blockIdx.x * (WG / 64) + (threadIdx.x >> 6);
    uint32_t my_new = 0, my_near = 0, evals = 0;
    double minm = INFINITY;
    // lane l of wave w looks at candidate (w + (l / GRP) waves) GRP + l % GRP
    const uint32_t per = waves * 64u;
    for (uint32_t base = wave * GRP; base < nc; base += per) {
        const uint32_t j = base + (uint32_t)(lane() / GRP) * waves * GRP + (uint32_t)(lane() % GRP);
        bool need = j < nc && d.c_iter[j] < 0;
        if (FINAL) {
            need = need && d.c_rho2[j] < 0.0;
        } else if (need && t > 0) {
            const int qb = d.c_qb[j];
            const int lo = max(qb - HALO, 0), hi = min(qb + HALO - 1, g.B - 1);
            bool changed = false;
            for (int tl = div_p2(lo, g.tile); tl <= div_p2(hi, g.tile); ++tl) changed |= d.sstamp[tl] >= t;
            need = changed;
            if (need && in.n >= BOUND_MIN_N) {
                const uint32_t *ma = d.is_max, *me = d.is_max + (g.B + 63) / 64;
                uint32_t xa = 0, xe = 0;
                for (int sg = lo >> 6; sg <= hi >> 6; ++sg) {
                    xa = max(xa, ma[sg]);
                    xe = max(xe, me[sg]);
                }
                auto above = [](uint32_t x) { return __longlong_as_double((long long)(((uint64_t)x + 1) << 32)); };
                const double A = (double)d.c_amp[j];
                if (T * (A * A) * (above(xa) + above(xe)) < skip2) {
                    need = false;
                    d.c_rho2[j] = -1.0;
                }
            }
        }
        // the constants only of the candidates evaluated
        SrcConsts mine{};
        if (need) mine = src_consts(g, in, d.c_src[j], E, false);
        uint64_t todo = (uint64_t)__ballot(need);
        if (!todo) continue;
        // the FFT's lane constants only for waves with evaluations (in late
        // bodies most have none)
        const LaneFft L = lane_fft();
        while (todo) {
            const int k = (int)__builtin_ctzll(todo);
            todo &= todo - 1;
            const SrcConsts cs = bcast(mine, k);
            const uint32_t jk = (uint32_t)__builtin_amdgcn_readlane((int)j, k);
            ++evals;
            const int be = cs.qb + je, bo = cs.qb + jo;
            const bool ine = be >= 0 && be < g.B, ino = bo >= 0 && bo < g.B;
            // the PSD under the template, loaded before the synthesis hides
            // their latency (off-grid lanes read bin 0 and drop it)
            const int bec = ine ? be : 0, boc = ino ? bo : 0;
            const double sAe = d.S[bec], sEe = d.S[B + bec], sAo = d.S[boc], sEo = d.S[B + boc];
            double2 ue, uo;
            wave_template(cs, L, ex, &ue, &uo);
            const double pe = ue.x * ue.x + ue.y * ue.y, po = uo.x * uo.x + uo.y * uo.y;
            double r = 0.0;
            if (ine) r += pe * ((sAe + sEe) / (sAe * sEe));
            if (ino) r += po * ((sAo + sEo) / (sAo * sEo));
            const double r2 = rs * wave_sum(r);
            if (lane() == 0) d.c_rho2[jk] = r2;
            if (FINAL) continue;
            const double rel = fabs(sqrt(r2) / g.rth - 1.0);
            minm = fmin(minm, rel);
            my_near += rel <= 1e-6;
            if (!(r2 > g.rth2)) continue;
            ++my_new;
            if (lane() == 0) d.c_iter[jk] = (int32_t)t;
            SrcConsts rc;
            rotations(in, cs.i, &rc);
            if (ine) {
                const double2 va = rot(ue, rc.ca, rc.sa), ve = rot(ue, rc.ce, rc.se);
                unsigned long long *p = (unsigned long long *)&d.h[be];
                atomicAdd(p, (unsigned long long)-fxm(va.x));
                atomicAdd(p + B, (unsigned long long)-fxm(va.y));
                atomicAdd(p + 2 * B, (unsigned long long)-fxm(ve.x));
                atomicAdd(p + 3 * B, (unsigned long long)-fxm(ve.y));
            }
            if (ino) {
                const double2 va = rot(uo, rc.ca, rc.sa), ve = rot(uo, rc.ce, rc.se);
                unsigned long long *p = (unsigned long long *)&d.h[bo];
                atomicAdd(p, (unsigned long long)-fxm(va.x));
                atomicAdd(p + B, (unsigned long long)-fxm(va.y));
                atomicAdd(p + 2 * B, (unsigned long long)-fxm(ve.x));
                atomicAdd(p + 3 * B, (unsigned long long)-fxm(ve.y));
            }
            if (lane() == 0) {
                const int lo = max(cs.qb - HALO, 0), hi = min(cs.qb + HALO - 1, g.B - 1);
                stamp_tiles(d.xstamp, g, lo, hi, nxt);
                int sa_, sb_;
                window_reach(g, lo, hi, &sa_, &sb_);
                stamp_tiles(d.sstamp, g, sa_, sb_, nxt);
            }
        }
    }
    if (FINAL) {
        if (COUNT && lane() == 0 && evals) atomicAdd((unsigned long long *)&c->units_snr, (unsigned long long)evals);
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        c->xupd = nxt;
        c->tail_due = 1;
    }
    if (lane() == 0) {
        if (my_new) atomicAdd(&c->n_new_body, my_new);
        if (my_near) atomicAdd((unsigned long long *)&c->n_near, (unsigned long long)my_near);
        if (evals) atomicAdd((unsigned long long *)&c->units_snr, (unsigned long long)evals);
        if (minm < INFINITY)
            atomicMin((unsigned long long *)&c->min_margin, (unsigned long long)__double_as_longlong(minm));
    }
}

// ------------------------------------------------------------------ outputs

__global__ __launch_bounds__(WG) void k_cx_ids(KArgs a)
{
    const CxDev &d = a.d;
    list_resolved(d.ctl->cand_cursor, d.c_iter, d.c_id, d.rlist, &d.ctl->res_cursor,
                  [&](uint32_t j) { return a.in.ids[d.c_src[j]]; });
    if (blockIdx.x == gridDim.x - 1) put_host(a.in.host_ctl, d.ctl, threadIdx.x);
}

__global__ __launch_bounds__(WG) void k_cx_hout(KArgs a, int ch, double *out)
{
    const CxDev &d = a.d;
    const size_t B = (size_t)a.g.B;
    const int E = cx_exp(d.ctl->amax_bits, a.in.n, a.g.T);
    const int64_t *re = d.h + (size_t)(2 * ch) * B, *im = re + B;
    for (size_t k = (size_t)blockIdx.x * WG + threadIdx.x; k < B; k += (size_t)gridDim.x * WG) {
        out[2 * k] = ldexp((double)re[k], -E);
        out[2 * k + 1] = ldexp((double)im[k], -E);
    }
}

// Templates of n sources (one wave each): q (INT64_MIN if none) and U in
// offset order j = -64 .. 63.
__global__ __launch_bounds__(WG) void k_cx_templates(Grid g, const float *A, const float *F, const float *FD,
                                                     uint32_t n, int64_t *q, double *U)
{
    __shared__ double2 ex[NEX];
    set_cis_table(ex);
    const LaneFft L = lane_fft();
    __syncthreads();
    int je, jo;
    lane_offsets(&je, &jo);
    const uint32_t waves = gridDim.x * (WG / 64);
    for (uint32_t i = blockIdx.x * (WG / 64) + (threadIdx.x >> 6); i < n; i += waves) {
        double qd, dd;
        SrcConsts c{};
        const bool ok = cx_centre((double)F[i], (double)FD[i], g.T, &qd, &c.delta, &dd);
        double2 ue = make_double2(0.0, 0.0), uo = ue;
        if (ok) {
            c.dh = dd * 0.5;
            c.sc = ((double)A[i] * 0.5) * (g.T / NF);
            wave_template(c, L, ex, &ue, &uo);
        }
        if (lane() == 0) q[i] = ok ? (int64_t)qd : INT64_MIN;
        double *u = U + (size_t)i * 2 * NF;
        u[2 * (je + HALO)] = ue.x;
        u[2 * (je + HALO) + 1] = ue.y;
        u[2 * (jo + HALO)] = uo.x;
        u[2 * (jo + HALO) + 1] = uo.y;
    }
}

KArgs args_of(const Grid &g, const CxDev &d, const CxIn &in) { return KArgs{g, d, in}; }

// The faint sources' records by bucket, SRC sources per block.
template <int SRC> void faint_group(const KArgs &a, hipStream_t st)
{
    const uint32_t rows = (a.in.n + SRC - 1) / SRC;
    k_cx_fcount<SRC><<<rows, FB_T, 0, st>>>(a);
    k_cx_fcols<SRC><<<FB_MAX / 64, FB_T, 0, st>>>(a);
    k_cx_fscan<<<1, PLAN_T, 0, st>>>(a);
    k_cx_fscatter<SRC><<<(rows + 7) / 8 * 8, FB_T, 0, st>>>(a);
}

}  // namespace

uint64_t cx_carve(const Grid &g, uint64_t n, char *base, CxDev *out)
{
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) -> char * {
        char *p = base ? base + off : nullptr;
        off = (off + (bytes ? bytes : 1) + 255) & ~uint64_t(255);
        return p;
    };
    const uint64_t B = (uint64_t)g.B, nt = (uint64_t)g.nt, nn = n ? n : 1;
    CxDev d{};
    d.ntc = (int32_t)((B + CX_TILE - 1) / CX_TILE);
    d.slots = (Slot *)take(2 * sizeof(Slot));
    d.ctl = (Ctl *)take(sizeof(Ctl));
    d.sx = (double *)take(B * 8);
    d.isx = (double *)take(B * 8);
    d.isx_max = (double *)take(((B + CX_NF - 1) / CX_NF) * 8);
    const uint64_t x0 = off;
    d.X = (double *)take(2 * B * 8);
    d.S = (double *)take(2 * B * 8);
    d.is_pre = (double *)take(2 * B * 8);
    const uint64_t spectra = off - x0;
    d.is_psum = (double *)take(2 * (uint64_t)g.nparts * 8);
    d.h = (int64_t *)take(4 * B * 8);
    d.xstamp = (uint32_t *)take(nt * 4);
    d.sstamp = (uint32_t *)take(nt * 4);
    d.sdl = (uint32_t *)take(nt * 4);
    d.tcnt = (uint32_t *)take(((uint64_t)d.ntc + 1) * 4);
    d.tcur = (uint32_t *)take((uint64_t)d.ntc * 4);
    d.cbase = (uint32_t *)take(((uint64_t)d.ntc + 1) * 4);
    d.order = (uint32_t *)take(nn * 4);
    d.c_src = (uint32_t *)take(nn * 4);
    d.c_iter = (int32_t *)take(nn * 4);
    d.c_id = (uint32_t *)take(nn * 4);
    d.c_rho2 = (double *)take(nn * 8);
    d.rlist = (uint64_t *)take(nn * 16);                                  // next to c_rho2: see frec
    d.c_qb = (int32_t *)take(nn * 4);
    d.c_amp = (float *)take(nn * 4);
    d.is_max = (uint32_t *)take(2 * ((B + 63) / 64) * 4);
    d.rs_hist = (uint32_t *)take(resolved_scratch_words(nn) * 4);
    const bool faint = n >= FAINT_MIN_N;
    d.fcnt = (uint32_t *)take(((uint64_t)d.ntc + 1) * 4);
    d.fbb = (uint32_t *)take(((uint64_t)d.ntc + 1) * 4);
    d.ftot = (uint32_t *)take(faint ? (FB_MAX + 1) * 4 : 0);
    // blocks of the faint passes: 16384 sources leave most of the chip idle in
    // small catalogs; smaller ones make more rows of the matrix, which lies
    // in the spectra (first written by the first body) if these are large
    // enough, and otherwise has 16384 sources a row.  4.1e5 sources, count,
    // columns and scatter: 22 us with 4096, 45 us with 16384.  Whole runs (4 yr)
    // with rows of 4096 and 16384: 2e5 sources 778 and 802 us, 1e6 1171 and 1190,
    // 1.5e6 1403 and 1416, 2e6 1525 and 1532, 4e6 2011 and 2004, 8e6 2901 and 2915:
    // from FB_SMALL on the two are within 1 %, and the longer rows write less.
    auto matrix = [&](uint32_t src) { return (n + src - 1) / src * (uint64_t)FB_MAX * 4; };
    d.fsrc = n <= FB_SMALL && matrix(FB_SRC_MIN) <= spectra ? FB_SRC_MIN : FB_SRC;
    d.fmat = matrix(d.fsrc) <= spectra ? (uint32_t *)d.X : (uint32_t *)take(faint ? matrix(d.fsrc) : 0);
    // binning scratch in memory that is written only later: the candidate
    // records by the direct injection (after the moment path has ended), the
    // ids and the resolved-list buffers after the run; frec lies over c_rho2
    // and the list behind it, 24 bytes a source
    static_assert(sizeof(FaintRec) == 24, "c_rho2 and rlist together");
    d.key = d.c_src;
    d.frec = (FaintRec *)d.c_rho2;
    d.forder = d.c_id;
    if (out) *out = d;
    return off;
}

hipError_t cx_launch_prep(const Grid &g, const CxDev &d, const CxIn &in, hipStream_t st)
{
    const KArgs a = args_of(g, d, in);
    k_cx_reset<<<1024, WG, 0, st>>>(a);
    const uint32_t nb = (in.n + SRC_PB - 1) / SRC_PB;
    if (nb) k_cx_count<<<nb, WG, 0, st>>>(a);
    k_cx_plan<<<1, PLAN_T, 0, st>>>(a);
    if (nb) k_cx_scatter<<<(in.n + FB_SRC - 1) / FB_SRC, FB_T, 0, st>>>(a);
    if (in.n >= FAINT_MIN_N) {
        if (d.fsrc == (uint32_t)FB_SRC_MIN)
            faint_group<FB_SRC_MIN>(a, st);
        else
            faint_group<FB_SRC>(a, st);
        k_cx_faint<<<FB_MAX, WG, 0, st>>>(a);
    }
    // chunks: at most one partial chunk per tile beyond the full ones (the
    // chunk is CH, or at least a CH_GRID'th of the direct sources)
    const uint32_t chunks = max(in.n / CH, (uint32_t)CH_GRID) + (uint32_t)d.ntc;
    if (in.n) k_cx_inject<<<chunks, WG, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t cx_launch_power(const Grid &g, const CxDev &d, const CxIn &in, hipStream_t st)
{
    k_cx_power<<<g.nt, WG, 0, st>>>(args_of(g, d, in));
    return hipGetLastError();
}

namespace {
Dims channel_dims(const Grid &g)
{
    Dims dm{};
    dm.ns = 2;
    dm.maxB = g.B;
    dm.maxnt = g.nt;
    dm.maxtile = g.tile;
    dm.maxparts = g.nparts;
    dm.maxlist = list_entries(g);
    dm.split_parts = split_parts(g);
    dm.est_mask = 1u << g.est;
    return dm;
}
}  // namespace

hipError_t cx_launch_psd(const Grid &g, const CxDev &d, hipStream_t st, hipEvent_t ea, hipEvent_t eb)
{
    return launch_median(d.slots, channel_dims(g), st, ea, eb);
}

hipError_t cx_launch_next(const Grid &g, const CxDev &d, hipStream_t st, hipEvent_t ea, hipEvent_t eb)
{
    return launch_next(d.slots, channel_dims(g), st, ea, eb);
}

hipError_t cx_launch_snr(const Grid &g, const CxDev &d, const CxIn &in, hipStream_t st)
{
    k_cx_snr<false, true><<<SNR_GRID, WG, 0, st>>>(args_of(g, d, in));
    return hipGetLastError();
}

bool cx_bounded(uint32_t n) { return n >= BOUND_MIN_N; }

hipError_t cx_launch_final(const Grid &g, const CxDev &d, const CxIn &in, bool count, hipStream_t st)
{
    if (count)
        k_cx_snr<true, true><<<SNR_GRID, WG, 0, st>>>(args_of(g, d, in));
    else
        k_cx_snr<true, false><<<SNR_GRID, WG, 0, st>>>(args_of(g, d, in));
    return hipGetLastError();
}

hipError_t cx_launch_outputs(const Grid &g, const CxDev &d, const CxIn &in, hipStream_t st)
{
    k_cx_ids<<<256, WG, 0, st>>>(args_of(g, d, in));
    return hipGetLastError();
}

hipError_t cx_launch_h(const Grid &g, const CxDev &d, uint32_t n, int ch, double *out, hipStream_t st)
{
    CxIn in{};
    in.n = n;
    k_cx_hout<<<1024, WG, 0, st>>>(args_of(g, d, in), ch, out);
    return hipGetLastError();
}

hipError_t cx_launch_templates(const Grid &g, const float *A, const float *F, const float *FD, uint32_t n,
                               int64_t *q, double *U, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const uint32_t blocks = min((n + WG / 64 - 1) / (WG / 64), 4096u);
    k_cx_templates<<<blocks, WG, 0, st>>>(g, A, F, FD, n, q, U);
    return hipGetLastError();
}

}  // namespace gbs
