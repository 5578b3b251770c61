// gf_site.h -- the per-site bodies shared by the single-lattice and the
// batched kernels of libgf: the overrelaxation / heat-bath site update and the
// per-site gauge-condition terms.
//
// One site update (Sec. 2 of arXiv:1412.3655): K(x) = sum_mu [U_mu(x) +
// U_mu(x-mu^)^dag] (Eq. localfunctional); for the SU(2) subgroups (0,1),
// (0,2), (1,2) the maximiser of the SU(2)-span projection of the 2x2 block of
// K is raised to the power omega (or, for the annealing prelude, a heat-bath
// element is drawn) and rotates K and the accumulated G; finally U_mu(x) <-
// G U_mu(x) and U_mu(x-mu^) <- U_mu(x-mu^) G^dag (the gauge transformation of
// Sec. 2 with g(x) = G and g = 1 elsewhere).  Rotating K by the subgroup
// element equals recomputing it from the rotated links (forward links become
// S U, backward links U S^dag, so K -> S K).
//
// Work split (Sec. 3.2 and 4.2 of the paper use 8 or 4 threads per site):
// TPS lanes of one wavefront share a site, lane r owning the 8/TPS links with
// leaf index r*(8/TPS) .. (r+1)*(8/TPS)-1 in the leaf order U_0(x),
// U_0(x-0^)^dag, U_1(x), U_1(x-1^)^dag, ...  Each lane sums its leaves in the
// fixed pairwise tree ((L0+L1)+(L2+L3))+((L4+L5)+(L6+L7)) and the lanes finish
// the same tree with DPP butterflies (no LDS), so K is bitwise the same for
// every TPS.  The subgroup algebra then runs redundantly in every lane of the
// group, and each lane applies G to the links it loaded and stores them.
#pragma once

#include <type_traits>

#include "gf_device.h"
#include "gf_min8.h"

namespace gf {

constexpr int OR_EXACT = 0;
constexpr int HEATBATH = 2;

// Parameters of the subgroup rule: omega and, for the exact float64 power, its
// coefficients for overrelaxation; temperature T, Philox key and sweep counter
// for the heat bath.
template <typename R>
struct Rule;
template <>
struct Rule<double> {
    double omega, T;
    uint32_t key0, key1, sweep;
    OrPower power;
};
template <>
struct Rule<float> {
    float omega, T;
    uint32_t key0, key1, sweep;
    float power;  // omega
};

// The overrelaxation rule of an omega, the heat-bath rule of a temperature, key and sweep.
template <typename R>
__host__ __device__ __forceinline__ Rule<R> or_rule(double omega, const OrPower& power)
{
    if constexpr (sizeof(R) == 8)
        return Rule<R>{omega, 1.0, 0u, 0u, 0u, power};
    else
        return Rule<R>{(float)omega, 1.0f, 0u, 0u, 0u, (float)omega};
}

template <typename R>
__host__ __device__ __forceinline__ Rule<R> hb_rule(R T, uint32_t key0, uint32_t key1, uint32_t sweep)
{
    return Rule<R>{R(1), T, key0, key1, sweep, {}};
}

// Squares below this leave the range of rsqrt_of.
constexpr double kTinySquare = 0x1p-960;

// The principal power of a float64 quaternion (see or_element) without its angle
// (see OrPower): sin^2 psi comes straight from a, so y has a small relative
// error and no cancellation.  A block with 0 <= phi <= pi/4, which is every
// block of a configuration near its maximum, needs one reciprocal square root,
// one reciprocal and the two polynomials; phi in (pi/4, 3pi/4] is measured from
// pi/2 and phi > 3pi/4 from pi, in a branch that a wave skips when no lane needs
// it.  Against atan2 and sincos of the device library a wave of the sweep at 4
// lanes per site issues 811 vector instructions instead of about 1400; the 8^4
// sweep, which a chain of dependent operations bounds, went from 11.8 to 10.0
// us, 16^4 from 20.0 to 17.7.  The error against values of higher precision is
// no larger at any angle (rms, in 2^-53: 0.3 and 0.3 near the maximum, 1.2 and
// 1.3 over random blocks; atan2 and sincos second).
__device__ __forceinline__ Quat<double> or_power(const Quat<double>& a, const OrPower& w)
{
    Quat<double> b;
    double a0 = a.b0, x1 = a.b1, x2 = a.b2, x3 = a.b3;
    double v2 = fmad(x1, x1, fmad(x2, x2, x3 * x3));
    double a02 = a0 * a0;
    double n2 = a02 + v2;
    if (n2 < kTinySquare) {  // b does not depend on the scale of a
        constexpr double up = 0x1p+600;
        a0 *= up;
        x1 *= up;
        x2 *= up;
        x3 *= up;
        v2 = fmad(x1, x1, fmad(x2, x2, x3 * x3));
        a02 = a0 * a0;
        n2 = a02 + v2;
    }
    const double rn = rsqrt_of(n2);
    const bool near = a0 > 0.0 && a02 >= v2;
    bool identity = false;
    // psi is the angle of (big, small): cos psi = big rn, sin psi = small rn
    double big = a0, small = 0.0, small2 = v2, c = 1.0, s = 0.0, iv = 0.0;
    if (!near) {
        double v;
        if (v2 >= kTinySquare) {
            iv = rsqrt_of(v2);
            v = v2 * iv;
        } else {
            identity = !(v2 > 0.0);
            v = sqrt(v2);
            iv = 1.0 / v;
        }
        const bool mid = v2 > a02;
        big = mid ? v : -a0;
        small = mid ? a0 : v;
        small2 = mid ? a02 : v2;
        c = mid ? w.c_mid : w.c_far;
        s = mid ? w.s_mid : w.s_far;
    }
    const double y = (small2 * rn) * (rn * recip(fmad(big, rn, 1.0)));
    double p = w.p[OrPower::N - 1], q = w.q[OrPower::N - 1];
#pragma unroll
    for (int k = OrPower::N - 2; k >= 0; --k) {
        p = fmad(p, y, w.p[k]);
        q = fmad(q, y, w.q[k]);
    }
    const double cw = fmad(-y, p, 1.0);  // cos(omega psi)
    const double sw = q * rn;            // sin(omega psi) / small
    double f = -sw;
    b.b0 = cw;
    if (!near) {
        const double sn = sw * small;
        b.b0 = fmad(c, cw, s * sn);
        f = -(fmad(s, cw, -(c * sn)) * iv);
        if (identity) {
            b.b0 = a.b0 < 0.0 ? -1.0 : 1.0;
            f = x1 = x2 = x3 = 0.0;
        }
    }
    b.b1 = f * x1;
    b.b2 = f * x2;
    b.b3 = f * x3;
    return b;
}

// The same through the device library's float32 functions.  (The polynomials
// would save a float32 sweep of 8-real links about 10 % of its instructions, but
// they round most elements otherwise, and float32 results would move by their own
// error, which rough inputs amplify up to 1e-3 at single sites within ten sweeps.
// The bits of float32 results are not promised from build to build, but so broad
// a change is not made for that gain.)
__device__ __forceinline__ Quat<float> or_power(const Quat<float>& a, float omega)
{
    Quat<float> b;
    const float v2 = fmad(a.b1, a.b1, fmad(a.b2, a.b2, a.b3 * a.b3));
    if (v2 > 0.0f) {
        const float v = sqrt(v2);
        const float phi = atan2(v, a.b0);
        float s, c;
        sin_cos(omega * phi, &s, &c);
        const float f = -s / v;
        b.b0 = c;
        b.b1 = f * a.b1;
        b.b2 = f * a.b2;
        b.b3 = f * a.b3;
    } else {
        b.b0 = a.b0 < 0.0f ? -1.0f : 1.0f;
        b.b1 = 0.0f;
        b.b2 = 0.0f;
        b.b3 = 0.0f;
    }
    return b;
}

// The SU(2) element applied for the projected block quaternion a (unnormalised,
// a0 + i(a1 s1 + a2 s2 + a3 s3)): the maximiser b = (a0, -a1, -a2, -a3)/|a|
// raised to the power omega.  EXACT: with phi = atan2(|a_vec|, a0), b^omega =
// (cos(omega phi), -sin(omega phi) a_vec/|a_vec|).  BINOMIAL1: normalise
// (1 - omega) + omega b.  |a_vec| = 0 (EXACT) or |a| = 0 leaves the subgroup
// alone (up to the sign of a0).
template <int MODE, typename R>
__device__ __forceinline__ Quat<R> or_element(const Quat<R>& a, const Rule<R>& rule)
{
    if constexpr (MODE == OR_EXACT) {
        return or_power(a, rule.power);
    } else {
        Quat<R> b;
        const R omega = rule.omega;
        const R n2 = fmad(a.b0, a.b0, fmad(a.b1, a.b1, fmad(a.b2, a.b2, a.b3 * a.b3)));
        if (n2 > R(0)) {
            const R inv = R(1) / sqrt(n2);
            const R t0 = fmad(omega, a.b0 * inv, R(1) - omega);
            const R t1 = -omega * (a.b1 * inv);
            const R t2 = -omega * (a.b2 * inv);
            const R t3 = -omega * (a.b3 * inv);
            const R tn = R(1) / sqrt(fmad(t0, t0, fmad(t1, t1, fmad(t2, t2, t3 * t3))));
            b.b0 = t0 * tn;
            b.b1 = t1 * tn;
            b.b2 = t2 * tn;
            b.b3 = t3 * tn;
        } else {
            b.b0 = R(1);
            b.b1 = R(0);
            b.b2 = R(0);
            b.b3 = R(0);
        }
        return b;
    }
}


// ------------------------------------------------------------- heat bath --
//
// Simulated-annealing prelude (named in the abstract of arXiv:1412.3655; the
// paper gives no algorithm).  Each subgroup element is drawn from
// exp(Re tr[g k]/T) dHaar(g).  With q = n qhat the SU(2)-span projection of
// the block (n = |a|/2 for the quaternion a of block_quaternion) the new
// element is g = w qhat^dag where w = (r0, sqrt(1-r0^2) e), e uniform on S^2
// and r0 has density sqrt(1-r0^2) exp(kappa r0), kappa = 2n/T: Creutz's
// exponential proposal below kappa = 2, Kennedy-Pendleton from 2 on, at most
// 128 attempts (then r0 = 1).  Random numbers: Philox4x32-10 (Salmon et al.,
// SC'11) keyed by the seed, counter (lexicographic site, sweep,
// subgroup<<16 | call, 0x48420000); float64 uniforms take 27+26 bits of two
// words, float32 ones 24 bits of one word.

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t out[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0), n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c0 = n0;
        c1 = (uint32_t)p1;
        c2 = n2;
        c3 = (uint32_t)p0;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

constexpr uint32_t HB_STREAM_TAG = 0x48420000u;
constexpr int HB_MAX_ATTEMPTS = 128;

__device__ __forceinline__ void uniform_pair(const uint32_t w[4], double* a, double* b)
{
    *a = ((double)(w[0] >> 5) * 67108864.0 + (double)(w[1] >> 6) + 0.5) * (1.0 / 9007199254740992.0);
    *b = ((double)(w[2] >> 5) * 67108864.0 + (double)(w[3] >> 6) + 0.5) * (1.0 / 9007199254740992.0);
}

__device__ __forceinline__ void uniform_pair(const uint32_t w[4], float* a, float* b)
{
    *a = ((float)(w[0] >> 8) + 0.5f) * (1.0f / 16777216.0f);
    *b = ((float)(w[2] >> 8) + 0.5f) * (1.0f / 16777216.0f);
}

__device__ __forceinline__ double hb_log1p(double x) { return log1p(x); }
__device__ __forceinline__ float hb_log1p(float x) { return log1pf(x); }
__device__ __forceinline__ double hb_expm1(double x) { return expm1(x); }
__device__ __forceinline__ float hb_expm1(float x) { return expm1f(x); }
__device__ __forceinline__ double hb_log(double x) { return log(x); }
__device__ __forceinline__ float hb_log(float x) { return logf(x); }
__device__ __forceinline__ double hb_cos(double x) { return cos(x); }
__device__ __forceinline__ float hb_cos(float x) { return cosf(x); }
__device__ __forceinline__ double hb_sqrt(double x) { return sqrt(x); }
__device__ __forceinline__ float hb_sqrt(float x) { return sqrtf(x); }

template <typename R>
struct HBStream {
    uint32_t key0, key1, site, sweep, subgroup, call;

    __device__ __forceinline__ void draw2(R* a, R* b)
    {
        uint32_t w[4];
        philox4x32_10(site, sweep, (subgroup << 16) | call, HB_STREAM_TAG, key0, key1, w);
        ++call;
        uniform_pair(w, a, b);
    }
};

template <typename R>
__device__ __forceinline__ R hb_sample_r0(HBStream<R>& st, R kappa)
{
    const R two_pi = R(6.283185307179586476925286766559);
    for (int attempt = 0; attempt < HB_MAX_ATTEMPTS; ++attempt) {
        if (kappa < R(2)) {
            R u1, u2;
            st.draw2(&u1, &u2);
            const R r0 = kappa == R(0) ? R(2) * u1 - R(1)
                                       : R(1) + hb_log1p((R(1) - u1) * hb_expm1(R(-2) * kappa)) / kappa;
            if (u2 * u2 <= R(1) - r0 * r0) return r0;
        } else {
            R u1, u2, u3, u4;
            st.draw2(&u1, &u2);
            st.draw2(&u3, &u4);
            const R c = hb_cos(two_pi * u2);
            const R lam2 = -(hb_log(u1) + c * c * hb_log(u3)) / (R(2) * kappa);
            if (u4 * u4 <= R(1) - lam2) return R(1) - R(2) * lam2;
        }
    }
    return R(1);
}

template <typename R>
__device__ __forceinline__ Quat<R> hb_element(const Quat<R>& a, const Rule<R>& rule, uint32_t lex, uint32_t sg)
{
    const R two_pi = R(6.283185307179586476925286766559);
    HBStream<R> st{rule.key0, rule.key1, lex, rule.sweep, sg, 0u};
    const R n2 = fmad(a.b0, a.b0, fmad(a.b1, a.b1, fmad(a.b2, a.b2, a.b3 * a.b3)));
    const R n = hb_sqrt(n2);
    const R kappa = n2 > R(0) ? n / rule.T : R(0);
    const R r0 = hb_sample_r0(st, kappa);
    R u5, u6;
    st.draw2(&u5, &u6);
    const R ct = R(2) * u5 - R(1);
    const R stt = hb_sqrt(fmax(R(0), R(1) - ct * ct));
    R sp, cp;
    sin_cos(two_pi * u6, &sp, &cp);
    const R rr = hb_sqrt(fmax(R(0), R(1) - r0 * r0));
    Quat<R> w;
    w.b0 = r0;
    w.b1 = rr * stt * cp;
    w.b2 = rr * stt * sp;
    w.b3 = rr * ct;
    if (!(n2 > R(0))) return w;
    // w o qhat^dag, qhat^dag = (a0, -a1, -a2, -a3)/|a|; (p o q) = (p0 q0 - p.q, p0 q + q0 p - p x q)
    const R inv = R(1) / n;
    const R g0 = a.b0 * inv, g1 = -a.b1 * inv, g2 = -a.b2 * inv, g3 = -a.b3 * inv;
    Quat<R> b;
    b.b0 = fmad(w.b0, g0, -fmad(w.b1, g1, fmad(w.b2, g2, w.b3 * g3)));
    b.b1 = fmad(w.b0, g1, fmad(g0, w.b1, -fmad(w.b2, g3, -(w.b3 * g2))));
    b.b2 = fmad(w.b0, g2, fmad(g0, w.b2, -fmad(w.b3, g1, -(w.b1 * g3))));
    b.b3 = fmad(w.b0, g3, fmad(g0, w.b3, -fmad(w.b1, g2, -(w.b2 * g1))));
    return b;
}

template <int MODE, typename R>
__device__ __forceinline__ Quat<R> subgroup_element(const Quat<R>& a, const Rule<R>& rule, uint32_t lex, uint32_t sg)
{
    if constexpr (MODE == HEATBATH)
        return hb_element(a, rule, lex, sg);
    else
        return or_element<MODE>(a, rule);
}

// Directions summed into K(x): 4 for Landau gauge, 3 (x, y, z) for Coulomb
// gauge, whose functional is that of Sec. 2 restricted to the spatial links,
// one independent problem per timeslice.  The gauge transformation of a
// Coulomb site update still acts on all 8 links at the site.
constexpr int NDIR_LANDAU = 4;
constexpr int NDIR_COULOMB = 3;

// Leaf k of this lane: U (forward, bwd = false) or U^dagger (backward), or
// zero for a direction outside the first NDIR.  Sum of NL consecutive leaves
// in the fixed pairwise tree; the zero leaves keep the tree, and so K, the
// same bitwise for every number of lanes per site.
template <int NL, int NDIR, typename R>
__device__ __forceinline__ void leaf_tree(const M3<R>* U, const bool* bwd, const int* mu, M3<R>& out)
{
    if constexpr (NL == 1) {
        m_leaf(out, U[0], bwd[0]);
        if constexpr (NDIR < 4) {
            if (mu[0] >= NDIR) {
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        out.re[i][j] = R(0);
                        out.im[i][j] = R(0);
                    }
            }
        }
    } else {
        M3<R> right;
        leaf_tree<NL / 2, NDIR>(U, bwd, mu, out);
        leaf_tree<NL / 2, NDIR>(U + NL / 2, bwd + NL / 2, mu + NL / 2, right);
        m_add(out, right);
    }
}

// tr[Delta Delta^dag] for Delta = [(K - K^dag)/(2i)]_traceless, in float64
// from K of either precision: M = (K - K^dag)/(2i) has diagonal Im K_ii and
// off-diagonal ((Im K_ij + Im K_ji) - i (Re K_ij - Re K_ji)) / 2, and
// Delta = M - tr(M)/3 (equal to Eq. (landaugauge) with A_mu of Sec. 2, a g = 1).
template <typename T>
__device__ __forceinline__ double delta_norm2(const M3<T>& K)
{
    const double d0 = (double)K.im[0][0], d1 = (double)K.im[1][1], d2 = (double)K.im[2][2];
    const double tr3 = (d0 + d1 + d2) / 3.0;
    const double e0 = d0 - tr3, e1 = d1 - tr3, e2 = d2 - tr3;
    double off = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i + 1; j < 3; ++j) {
            const double mr = 0.5 * ((double)K.im[i][j] + (double)K.im[j][i]);
            const double mi = 0.5 * ((double)K.re[i][j] - (double)K.re[j][i]);
            off += mr * mr + mi * mi;
        }
    return e0 * e0 + e1 * e1 + e2 * e2 + 2.0 * off;
}

// Keeps the compiler from mixing the instructions before and after.  It would
// interleave the decodes (and encodes) of all links of a lane to hide their
// latencies, at the price of their temporaries all living at once; other waves
// hide them as well.  theta and F of 8 reals, whose threads do little else, then
// need 122 registers in float32 instead of 237 and run 4 waves per SIMD instead of
// 2 (float64 178 instead of 264, 2 instead of 1).  The sweeps keep their
// number of waves; float64 ones and the heat bath still gain (24^3x48 float64 62.7
// -> 60.6 us per half-sweep, the float32 heat bath of 32^4 at T = 1 72.3 -> 68.8;
// where it starts hotter, 84 to 87), float32 overrelaxation does not (48^3x96 515
// -> 522), so it goes without.
template <bool ON = true>
__device__ __forceinline__ void apart()
{
    if constexpr (ON) __builtin_amdgcn_sched_barrier(0);
}

// Has the coefficients in scalar registers here: while the links are on their way,
// neither before their addresses nor with a wait of its own at the first subgroup.
__device__ __forceinline__ void fetch(const OrPower& w)
{
    static_assert(OrPower::N == 11, "all of them");
    asm volatile("" ::"s"(w.p[0]), "s"(w.p[1]), "s"(w.p[2]), "s"(w.p[3]), "s"(w.p[4]), "s"(w.p[5]), "s"(w.p[6]),
                 "s"(w.p[7]), "s"(w.p[8]), "s"(w.p[9]), "s"(w.p[10]), "s"(w.q[0]), "s"(w.q[1]), "s"(w.q[2]),
                 "s"(w.q[3]), "s"(w.q[4]), "s"(w.q[5]), "s"(w.q[6]), "s"(w.q[7]), "s"(w.q[8]), "s"(w.q[9]),
                 "s"(w.q[10]));
}

// One site update of the site (parity, h) by lane r of its TPS-lane group.
// TRACKG (float32 mixed-precision bulk): also g(x) <- G g(x) for the float32
// gauge transformation accumulated since the original links; lane r of the
// group stores the chunks c with c % TPS == r.  NDIR: directions in K (Landau
// 4, Coulomb 3); all 8 links are transformed either way.  With est, lane 0 of
// the group returns tr[Delta Delta^dag] of the site's K before the update (the
// gauge-condition term of the configuration the site sees), every other lane
// and every call without est 0.  F: the link field, 12 reals per link
// (LinkField<R>) or 8 reals (Link8Field for float64, Link8Field32 for
// float32; decoded on load and encoded on store, in R).
template <typename R, int TPS, int MODE, bool TRACKG, int CP = 0, int NDIR = NDIR_LANDAU, typename F = LinkField<R>>
__device__ __forceinline__ double site_update(const F& f, const Geom& g, int parity, uint32_t h, int r,
                                              const Rule<R>& rule, const GField& gacc, bool est = false)
{
    constexpr bool kMin8 = Min8Of<F>::value;
    constexpr bool kApart = kMin8 && (sizeof(R) == 8 || MODE == HEATBATH);
    // 12 reals: all loads before the arithmetic on the first links, which holds the
    // last ones up otherwise (us per sweep without -> with, best block of each): float64
    // at 2 lanes and more (8^4 9.9 -> 9.2, 24^4 79.8 -> 77.8; heat bath at 2 lanes, 32^4
    // 7 %), and the float32 heat bath at one or two (32^4 156.7 -> 142.0).  Not at one
    // lane in float64 (16^3x32 28.8 -> 29.5), nor in float32 sweeps (two lanes, all
    // blocks and policies: 32^4 1.1 % and 48^3x96 1.0 % slower with it).
    constexpr bool kLoadsFirst = MODE == HEATBATH ? TPS == 2 || (TPS == 1 && sizeof(R) == 4) : sizeof(R) == 8 && TPS >= 2;
    constexpr int NL = 8 / TPS;
    const Site s = decode_site(g, parity, h);
    const uint32_t lex = 2 * h + (uint32_t)(s.x & 1);

    M3<R> U[NL];
    bool bwd[NL];
    int mu_of[NL];
    uint32_t at[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int li = r * NL + k;
        mu_of[k] = li >> 1;
        bwd[k] = (li & 1) != 0;
        at[k] = bwd[k] ? back_h(g, h, s, mu_of[k]) : h;
    }
    if constexpr (kMin8) {
        static_assert(std::is_same<R, typename Min8Of<F>::R>::value, "decoded in the field's precision");
        // every load first, then the decodes (each yields SU(3) to rounding); see apart
        typename Min8Of<F>::C raw[NL][Min8Of<F>::N];
#pragma unroll
        for (int k = 0; k < NL; ++k)
            load_min8_raw<nt_loads(CP)>(f, bwd[k] ? 1 - parity : parity, mu_of[k], at[k], raw[k]);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            apart<kApart>();
            decode_min8(raw[k], U[k]);
        }
        apart<kApart>();
    } else {
#pragma unroll
        for (int k = 0; k < NL; ++k)
            load_rows01<nt_loads(CP)>(f, bwd[k] ? 1 - parity : parity, mu_of[k], at[k], U[k]);
        apart<kLoadsFirst>();
        if constexpr (MODE == OR_EXACT && kLoadsFirst) fetch(rule.power);
        // Row 2 is rebuilt from the two stored rows, so a departure d from unitarity
        // of those rows becomes up to ~2d after an update that mixes the rows.  Every
        // heat-bath update mixes them strongly (d would grow ~1.35x per sweep), so the
        // heat bath re-orthonormalises the two rows on load.  Overrelaxation mixes
        // them little (its subgroup elements approach 1; d grows ~1.004x per sweep on
        // rough inputs) and relies on the periodic reunitarisation of the fix-until
        // loop, which keeps its register footprint (and occupancy) unchanged.
        if constexpr (MODE == HEATBATH) {
#pragma unroll
            for (int k = 0; k < NL; ++k) gram_schmidt_rows01(U[k]);
        }
#pragma unroll
        for (int k = 0; k < NL; ++k) rebuild_row2(U[k]);
    }

    M3<R> K;
    leaf_tree<NL, NDIR>(U, bwd, mu_of, K);
    if constexpr (TPS >= 2) dpp_accumulate<DPP_XOR1>(K);
    if constexpr (TPS >= 4) dpp_accumulate<DPP_XOR2>(K);
    if constexpr (TPS >= 8) dpp_accumulate<DPP_HALF_MIRROR>(K);
    const double th = (est && r == 0) ? delta_norm2(K) : 0.0;

    M3<R> G;
    {
        const Quat<R> b = subgroup_element<MODE>(block_quaternion<0, 1>(K), rule, lex, 0u);
        set_embedding<0, 1>(b, G);
        rotate_rows<0, 1>(b, K);
    }
    {
        const Quat<R> b = subgroup_element<MODE>(block_quaternion<0, 2>(K), rule, lex, 1u);
        rotate_rows<0, 2>(b, G);
        rotate_rows<0, 2>(b, K);
    }
    {
        const Quat<R> b = subgroup_element<MODE>(block_quaternion<1, 2>(K), rule, lex, 2u);
        rotate_rows<1, 2>(b, G);
    }

#pragma unroll
    for (int k = 0; k < NL; ++k) {
        apart<kApart>();
        if (bwd[k])
            right_mul_dag_rows01(G, U[k]);
        else
            left_mul_rows01(G, U[k]);
        store_link<nt_stores(CP)>(f, bwd[k] ? 1 - parity : parity, mu_of[k], at[k], U[k]);
    }

    if constexpr (TRACKG) {
        M3<R> gx;
        load_g(gacc, parity, h, gx);
        gram_schmidt_rows01(gx);  // g is only ever multiplied: keep it in SU(3) (see above)
        rebuild_row2(gx);
        left_mul_rows01(G, gx);
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (c % TPS == r) store_g_chunk(gacc, parity, h, c, gx);
    }
    return th;
}

// ------------------------------------------------------------- reductions --

template <typename R>
__device__ __forceinline__ void load_full_f64(const LinkField<R>& f, int parity, int mu, uint32_t h, M3<double>& u)
{
    M3<R> t;
    load_rows01(f, parity, mu, h, t);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            u.re[i][j] = (double)t.re[i][j];
            u.im[i][j] = (double)t.im[i][j];
        }
    rebuild_row2(u);
}

// Links read in place from the ABI's canonical float64 array
// [site][mu][row][col][re,im], lexicographic site x + Nx(y + Ny(z + Nz t)).
// The half index h of (parity, h) is lex >> 1 (Nx is even), so
// lex = 2h + (x & 1).  Rows 0 and 1 are read and row 2 is rebuilt from them,
// exactly as from the 12-real device layout, so every measurement over a
// CanonField equals the one over the packed float64 field of the same links.
struct CanonField {
    const double* base;
    Geom g;
};

__device__ __forceinline__ void load_full_f64(const CanonField& f, int parity, int mu, uint32_t h, M3<double>& u)
{
    const Site s = decode_site(f.g, parity, h);
    const size_t lex = 2 * (size_t)h + (size_t)(s.x & 1);
    const double2* p = (const double2*)(f.base + (lex * 4 + (size_t)mu) * 18);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        const double2 v = p[c];
        u.re[c / 3][c % 3] = v.x;
        u.im[c / 3][c % 3] = v.y;
    }
    rebuild_row2(u);
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// MI355X hands consecutive blocks to its 8 XCDs in turn, and each XCD has an L2
// of its own.  Kernels that read every link from both of its ends give each XCD
// a contiguous run of tiles instead, so the second read of a link (the same
// tile for x and mostly y, a few tiles on for z) finds it in that L2: logical
// block xcd_block(b, n) for the block b of n, a permutation of 0..n-1.  theta
// and F of 32^4 float64 113 -> 97 us (the links once at the rate of a large
// copy: 62 us), of 48^3x96 1212 -> 825, of SU(2) 32^3x64 80 -> 46; plaquette of
// 32^4 212 -> 172.  The partial sums keep their places, so theta and F are the
// same bits.
constexpr uint32_t kXcds = 8;

__device__ __forceinline__ uint32_t xcd_first(uint32_t x, uint32_t n)
{
    const uint32_t r = n % kXcds;
    return x * (n / kXcds) + (x < r ? x : r);
}

__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t n)
{
    return xcd_first(b % kXcds, n) + b / kXcds;
}

// Sum two values over the block; thread 0 writes them to out[0..1].
template <int NT>
__device__ __forceinline__ void block_sum2(double a, double b, double* out)
{
    __shared__ double lds[2][NT / 64];
    a = wave_sum(a);
    b = wave_sum(b);
    const int w = threadIdx.x / 64;
    if ((threadIdx.x & 63) == 0) {
        lds[0][w] = a;
        lds[1][w] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sa = 0.0, sb = 0.0;
        for (int i = 0; i < NT / 64; ++i) {
            sa += lds[0][i];
            sb += lds[1][i];
        }
        out[0] = sa;
        out[1] = sb;
    }
}

// out[k] = scale[k] * sum_i partial[2 i + k] over n pairs, summed in a fixed
// order by one block of NT threads (the caller synchronises before reading out).
template <int NT>
__device__ __forceinline__ void finalize_pairs(const double* partial, uint32_t n, double s0, double s1, double* out)
{
    // one block: the latency of its loads is all it costs, so 8 are in flight
    // (48^3x96: 67 -> 24 us); added in the order of a plain loop
    constexpr uint32_t kAhead = 8;
    const double2* pairs = (const double2*)partial;
    double a = 0.0, b = 0.0;
    uint32_t i = threadIdx.x;
    for (; i + (kAhead - 1) * NT < n; i += kAhead * NT) {
        double2 v[kAhead];
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) v[k] = pairs[i + k * NT];
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) {
            a += v[k].x;
            b += v[k].y;
        }
    }
    for (; i < n; i += NT) {
        a += pairs[i].x;
        b += pairs[i].y;
    }
    __shared__ double res[2];
    block_sum2<NT>(a, b, res);
    __syncthreads();
    if (threadIdx.x == 0) {
        out[0] = res[0] * s0;
        out[1] = res[1] * s1;
    }
}

// Gauge-condition and functional terms of the site (parity, h), float64:
// th = tr[Delta Delta^dag] with Delta = [(K - K^dag)/(2i)]_traceless (equal to
// Eq. (landaugauge) with A_mu of Sec. 2, a g = 1), fr = sum_mu Re tr U_mu(x),
// mu over the first NDIR directions (Landau 4; Coulomb 3, the spatial Delta_C
// and functional of one timeslice).
template <int NDIR = NDIR_LANDAU, typename Field>
__device__ __forceinline__ void measure_site(const Field& f, const Geom& g, int parity, uint32_t h, double& th,
                                             double& fr)
{
    const Site s = decode_site(g, parity, h);
    M3<double> K;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            K.re[i][j] = 0.0;
            K.im[i][j] = 0.0;
        }
    auto forward = [&](const M3<double>& u) {
        fr += u.re[0][0] + u.re[1][1] + u.re[2][2];
        m_add(K, u);
    };
    auto backward = [&](const M3<double>& u) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                K.re[i][j] += u.re[j][i];
                K.im[i][j] -= u.im[j][i];
            }
    };
    M3<double> u;
    if constexpr (Min8Of<Field>::value) {
        typename Min8Of<Field>::C p[2 * NDIR][Min8Of<Field>::N];
#pragma unroll
        for (int mu = 0; mu < NDIR; ++mu) {
            load_min8_raw(f, parity, mu, h, p[2 * mu]);
            load_min8_raw(f, 1 - parity, mu, back_h(g, h, s, mu), p[2 * mu + 1]);
        }
#pragma unroll
        for (int mu = 0; mu < NDIR; ++mu) {
            apart();
            decode_min8(p[2 * mu], u);
            forward(u);
            apart();
            decode_min8(p[2 * mu + 1], u);
            backward(u);
        }
    } else {
#pragma unroll
        for (int mu = 0; mu < NDIR; ++mu) {
            load_full_f64(f, parity, mu, h, u);
            forward(u);
            load_full_f64(f, 1 - parity, mu, back_h(g, h, s, mu), u);
            backward(u);
        }
    }
    th = delta_norm2(K);
}

}  // namespace gf
