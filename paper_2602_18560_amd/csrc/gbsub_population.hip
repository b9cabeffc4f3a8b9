// gbsub_population.hip -- synthetic galactic-binary catalogs drawn on the
// GPU from the population model of Sec. "Population model" (Table "priors",
// appendix "Copulas").
//
// Per source i (one thread each, no communication):
//   * four 53-bit uniforms from two Philox4x32-10 blocks (Salmon et al.,
//     SC 2011) with key = the 64-bit seed and counter = (i, block);
//   * three standard normals by Box-Muller; (z1, z2) = (n1, rho n1 +
//     sqrt(1 - rho^2) n2) is the Gaussian copula pair;
//   * f = inverse CDF of the power law f^alpha_PL on [f_lo, f_hi] at Phi(z1);
//   * log10(fdot) - mu_Gamma = inverse CDF of Gamma(alpha_Gamma, rate
//     beta_Gamma) at Phi(z2);
//   * log10(f^(-2/3) A) - mu = exp(sigma n3) (log-normal, shape sigma).
// Outputs are the fp32 catalog columns the subtraction reads.
#include "gbsub_internal.h"

#include <math.h>

namespace gbs {

namespace {

struct Philox4 {
    uint32_t v[4];
};

__device__ __forceinline__ Philox4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                            uint32_t k1)
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;   // round multipliers
    constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;   // key increments
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = static_cast<uint64_t>(M0) * c0, p1 = static_cast<uint64_t>(M1) * c2;
        const uint32_t n0 = static_cast<uint32_t>(p1 >> 32) ^ c1 ^ k0, n2 = static_cast<uint32_t>(p0 >> 32) ^ c3 ^ k1;
        c0 = n0;
        c1 = static_cast<uint32_t>(p1);
        c2 = n2;
        c3 = static_cast<uint32_t>(p0);
        k0 += W0;
        k1 += W1;
    }
    return {{c0, c1, c2, c3}};
}

__device__ __forceinline__ double unit53(uint32_t hi, uint32_t lo)
{
    const uint64_t b = ((static_cast<uint64_t>(hi) << 32) | lo) >> 11;
    return (static_cast<double>(b) + 0.5) * 0x1.0p-53;
}

// ---- the two inverse CDFs as local power series in the normal variate
//
// f = F^{-1}(Phi(z1)) and y = G^{-1}(Phi(z2)) (G: Gamma(a, 1)) are analytic in
// z, and every z that Box-Muller can return from 53-bit uniforms lies within
// sqrt(2 * 54 ln 2) = 8.652 of zero.  A block lays NODE expansion points over
// that range (spacing H) in LDS and each source evaluates one polynomial per
// marginal, instead of inverting the incomplete gamma function on its own: a
// node needs P(a, y) one to three times in the prior's range (up to 7 for
// shapes of 1e-3; the node is put at the z that belongs to its y, so Newton steps
// need only come within H/4 of its place), and its coefficients follow from the
// differential equations of the two maps.
//   Truncation: log f(z) has its nearest singularities where the power-law
// argument vanishes, at a distance of at least about 0.87 from the real axis
// for the model's two decades of f (pi/8 at 1e15 in f^e), y(z) at the zeros of
// erfc, 2.8 away; with |dz| <= H/2 + H/4 the first term left out is below 1e-17.
// A Newton iteration on P per source (a series or a continued fraction of
// divisions at every step) took 13.0 ms for 7.5e6 sources and 0.313 ms for
// 20,011; the nodes take 0.162 ms (120 MB written; bound by the fp64 and
// integer instructions of the random numbers and the exponentials) and
// 0.018 ms (the latency of one node).
constexpr int GT = 512;              // threads of a block: a node of y or of log f each
constexpr int NODE = GT / 2;
constexpr double ZMAX = 8.66;
constexpr double H = 2.0 * ZMAX / (NODE - 1);
constexpr int NY = 9, NF_ = 12;      // coefficients of y and of log f
constexpr int GEN_GRID = 768;        // three blocks per CU (LDS), each striding over the catalog

struct GenTables {
    double yz[NODE], yc[NY][NODE];   // centres and coefficients of y(z) / beta_Gamma
    double fc[NF_][NODE];            // of log f(z), centred at -ZMAX + j H
};

__device__ __forceinline__ double norm_lower(double z) { return 0.5 * erfc(-z * 0.7071067811865476); }
__device__ __forceinline__ double norm_pdf(double z) { return 0.3989422804014327 * exp(-0.5 * z * z); }

// z with Phi(z) = p, 0 < p <= 1/2, to the last bits (one Newton step on the
// library's quantile).
__device__ double norm_quantile(double p)
{
    const double z = normcdfinv(p);
    return z > -37.0 ? z - (norm_lower(z) - p) / norm_pdf(z) : z;
}

// The normal variate of y = exp(w) under Gamma(a, 1): z with Phi(z) = P(a, y),
// from the series of P up to zt <= ZSPLIT (zt: where the caller looks for it) and
// the continued fraction of Q beyond, so that each tail keeps its relative
// precision.  lga = ln Gamma(a).
//   The fraction needs about 81/y terms below y ~ 1, and y is far below that
// beyond ZSPLIT when a is small (6e-5 at z = 1.7 for a = 0.005), so the series also
// takes y < a + 1: at most 210 terms a node for a from 1e-6 to 0.1, where
// the fraction by z alone ended after GAMMA_TERMS without having converged, up
// to 64 times a node, and left fdot off by up to 1.4e-5 for a below 0.01 (now
// below 1e-12 from a = 1e-3 on; 6e-11 at 1e-4 and 4e-9 at 1e-6, by the rounding of
// 1 - P).  For a >= 1 the two rules are the same beyond ZSPLIT.
constexpr double ZSPLIT = 1.5;
constexpr int GAMMA_TERMS = 1 << 15;
__device__ double gamma_normal(double a, double lga, double w, double zt)
{
    const double y = exp(w);
    if (zt <= ZSPLIT || y < a + 1.0) {
        const double pre = exp(a * w - y - lga);
        double t = 1.0 / a, s = t;
        for (int k = 1; k < GAMMA_TERMS; ++k) {
            t *= y / (a + k);
            s += t;
            if (t < s * 0x1.0p-56) break;
        }
        const double p = s * pre;
        return p <= 0.5 ? norm_quantile(p) : -norm_quantile(1.0 - p);
    }
    constexpr double TINY = 1e-300;
    const double pre = exp(a * w - y - lga);
    double b = y + 1.0 - a;
    b = fabs(b) < TINY ? TINY : b;
    double c = 1.0 / TINY, d = 1.0 / b, h = d;
    for (int k = 1; k < GAMMA_TERMS; ++k) {
        const double an = -k * (k - a);
        b += 2.0;
        d = an * d + b;
        d = fabs(d) < TINY ? TINY : d;
        c = b + an / c;
        c = fabs(c) < TINY ? TINY : c;
        d = 1.0 / d;
        const double r = d * c;
        h *= r;
        if (fabs(r - 1.0) <= 4e-16) break;
    }
    const double q = pre * h;
    return q <= 0.5 ? -norm_quantile(q) : norm_quantile(1.0 - q);
}

// Node j of y(z).  w = ln y starts from Wilson-Hilferty (or, where that is not
// positive, from the leading term of P at small y) and takes Newton steps in
// (z, w), in which the map is nearly straight, until its own z lies within
// H/4 of the node's place; that z is the node.  With w' = phi(z) Gamma(a) e^y /
// y^a = exp(g), g = -z^2/2 - a w + y + const and y' = w' y, the coefficients are
// those of the products of power series.
__device__ void gamma_node(GenTables &t, int j, double a, double beta, double lga)
{
    const double zt = -ZMAX + j * H;
    constexpr double LOG_SQRT_2PI = 0.9189385332046727;
    double w;
    {
        const double c = 1.0 - 1.0 / (9.0 * a) + zt / (3.0 * sqrt(a));
        // below a/8 the leading term (y^a / Gamma(a + 1)) is the better start
        w = c > 0.5 ? log(a) + 3.0 * log(c) : (log(norm_lower(zt)) + lga + log(a)) / a;
    }
    double z = zt;
    if (a <= 1e6)                       // beyond, Wilson-Hilferty is closer than the sums
        for (int it = 0; it < 64; ++it) {
            z = gamma_normal(a, lga, w, zt);
            if (fabs(z - zt) <= 0.25 * H) break;
            const double slope = exp(-0.5 * z * z - LOG_SQRT_2PI - a * w + exp(w) + lga);
            const double dw = fabs(z) < 37.0 ? (zt - z) * slope : zt - z;
            w += fabs(dw) < 2.0 ? dw : copysign(2.0, zt - z);
        }
    const double y0 = exp(w);
    double W[NY], E[NY], G[NY], g[NY];
    W[0] = w;
    E[0] = y0;
    g[0] = -0.5 * z * z - LOG_SQRT_2PI - a * w + y0 + lga;
    G[0] = exp(g[0]);
#pragma unroll
    for (int n = 1; n < NY; ++n) {
        W[n] = G[n - 1] / n;
        double e = 0.0;
#pragma unroll
        for (int k = 1; k <= n; ++k) e = fma(k * W[k], E[n - k], e);
        E[n] = e / n;
        g[n] = (n == 1 ? -z : n == 2 ? -0.5 : 0.0) - a * W[n] + E[n];
        double x = 0.0;
#pragma unroll
        for (int k = 1; k <= n; ++k) x = fma(k * g[k], G[n - k], x);
        G[n] = x / n;
    }
    t.yz[j] = z;
#pragma unroll
    for (int n = 0; n < NY; ++n) t.yc[n][j] = E[n] / beta;
}

// Node j of log f(z) = log(x) / e, x = lo + Phi(z) (hi - lo) with lo = f_lo^e and
// hi = f_hi^e (from the nearer end, so that nothing cancels).
__device__ void freq_node(GenTables &t, int j, double e, double lo, double hi)
{
    const double z = -ZMAX + j * H, D = hi - lo;
    double ph[NF_], X[NF_], l[NF_];
    X[0] = z < 0.0 ? lo + norm_lower(z) * D : hi - norm_lower(-z) * D;
    l[0] = log(X[0]);
    ph[0] = norm_pdf(z);
#pragma unroll
    for (int n = 1; n < NF_; ++n) {
        X[n] = D * ph[n - 1] / n;
        ph[n] = -fma(z, ph[n - 1], n > 1 ? ph[n - 2] : 0.0) / n;
        double s = n * X[n];
#pragma unroll
        for (int k = 1; k < n; ++k) s = fma(-k * l[k], X[n - k], s);
        l[n] = s / (n * X[0]);
    }
#pragma unroll
    for (int n = 0; n < NF_; ++n) t.fc[n][j] = l[n] / e;
}

// Nearest node of z.
__device__ __forceinline__ int node_of(double z)
{
    return min(max((int)((z + ZMAX) * (1.0 / H) + 0.5), 0), NODE - 1);
}

__global__ __launch_bounds__(GT) void k_generate(PopParams pp, uint64_t seed, uint64_t first, uint64_t n, float *A,
                                                 float *F, float *FD, uint32_t *id)
{
    __shared__ GenTables t;
    if (threadIdx.x < NODE) {
        gamma_node(t, threadIdx.x, pp.alpha_g, pp.beta_g, lgamma(pp.alpha_g));
    } else {
        const double e = pp.alpha_pl + 1.0;
        freq_node(t, threadIdx.x - NODE, e, pow(pp.f_lo_hz, e), pow(pp.f_hi_hz, e));
    }
    __syncthreads();
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    const double rc = sqrt(1.0 - pp.rho * pp.rho);
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * GT + threadIdx.x; i < n;
         i += static_cast<uint64_t>(gridDim.x) * GT) {
        const uint64_t s = first + i;
        const uint32_t s0 = static_cast<uint32_t>(s), s1 = static_cast<uint32_t>(s >> 32);
        const Philox4 r = philox10(s0, s1, 0u, 0u, k0, k1);
        const Philox4 q = philox10(s0, s1, 1u, 0u, k0, k1);
        const double u1 = unit53(r.v[0], r.v[1]), u2 = unit53(r.v[2], r.v[3]);
        const double u3 = unit53(q.v[0], q.v[1]), u4 = unit53(q.v[2], q.v[3]);
        const double rad = sqrt(-2.0 * log(u1));
        double sn, cs;
        sincospi(2.0 * u2, &sn, &cs);
        const double z1 = rad * cs, n2 = rad * sn;
        const double n3 = sqrt(-2.0 * log(u3)) * cospi(2.0 * u4);
        const double z2 = pp.rho * z1 + rc * n2;
        const int j1 = node_of(z1), j2 = node_of(z2);
        const double d1 = z1 - (-ZMAX + j1 * H), d2 = z2 - t.yz[j2];
        double lf = t.fc[NF_ - 1][j1], y = t.yc[NY - 1][j2];
#pragma unroll
        for (int k = NF_ - 2; k >= 0; --k) lf = fma(lf, d1, t.fc[k][j1]);
#pragma unroll
        for (int k = NY - 2; k >= 0; --k) y = fma(y, d2, t.yc[k][j2]);
        const double at = exp(pp.sigma * n3);
        A[i] = static_cast<float>(exp10(at + pp.mu) * exp(lf * (2.0 / 3.0)));
        F[i] = static_cast<float>(exp(lf));
        FD[i] = static_cast<float>(exp10(y + pp.mu_g));
        if (id) id[i] = static_cast<uint32_t>(s);
    }
}

}  // namespace

hipError_t launch_generate(const PopParams &pp, uint64_t seed, uint64_t first, uint64_t n, float *A, float *F,
                           float *FD, uint32_t *id, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const uint64_t blocks = (n + GT - 1) / GT;
    const unsigned grid = static_cast<unsigned>(blocks < GEN_GRID ? blocks : GEN_GRID);
    k_generate<<<grid, GT, 0, st>>>(pp, seed, first, n, A, F, FD, id);
    return hipGetLastError();
}

}  // namespace gbs
