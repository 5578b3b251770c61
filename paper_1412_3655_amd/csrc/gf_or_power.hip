// gf_or_power.hip -- the coefficients of the power g^omega (OrPower in
// gf_device.h), computed on the host once per omega.
#include <cmath>

#include "gf_kernels.h"

namespace gf {

namespace {

constexpr long double kPi = 3.14159265358979323846264338327950288L;

// P(y) = (1 - T_omega(1 - y)) / y and Q(y) = U_{omega-1}(1 - y) from their
// hypergeometric series 2F1(-omega, omega; 1/2; y/2) and omega 2F1(1 - omega,
// 1 + omega; 3/2; y/2), whose terms fall by y/2 <= 0.15 each.
constexpr int kTerms = 32;

struct OrSeries {
    long double c[kTerms], d[kTerms], w;

    explicit OrSeries(long double omega) : w(omega)
    {
        long double ck = 1.0L, dk = w;
        for (int k = 1; k <= kTerms; ++k) {
            c[k - 1] = ck *= ((long double)(k - 1) * (k - 1) - w * w) / ((2 * k - 1) * (long double)k);
            d[k - 1] = dk *= ((long double)k * k - w * w) / ((2 * k + 1) * (long double)k);
        }
    }

    void sum(long double y, long double* P, long double* Q) const
    {
        long double p = 0.0L, q = w, yk = 1.0L;
        for (int k = 0; k < kTerms; ++k) {
            p -= c[k] * yk;
            yk *= y;
            q += d[k] * yk;
        }
        *P = p;
        *Q = q;
    }
};

// Monomial coefficients of the interpolant through (x_i, f_i), i < N (f is
// overwritten by the divided differences).
template <int N>
void interpolate(const long double (&x)[N], long double (&f)[N], long double (&m)[N])
{
    for (int j = 1; j < N; ++j)
        for (int i = N - 1; i >= j; --i) f[i] = (f[i] - f[i - 1]) / (x[i] - x[i - j]);
    for (int k = 0; k < N; ++k) m[k] = 0.0L;
    for (int i = N - 1; i >= 0; --i) {
        for (int k = N - 1; k >= 1; --k) m[k] = m[k - 1] - x[i] * m[k];
        m[0] = f[i] - x[i] * m[0];
    }
}

// Chebyshev nodes of [0, 1 - 1/sqrt 2], y at psi = pi/4.
struct Nodes {
    long double x[OrPower::N];

    Nodes()
    {
        constexpr int N = OrPower::N;
        const long double top = 1.0L - sqrtl(0.5L);
        for (int i = 0; i < N; ++i)
            x[i] = 0.5L * top * (1.0L + cosl(kPi * (2 * i + 1) / (2 * N)));
    }
};

void make_power(long double w, OrPower* out)
{
    constexpr int N = OrPower::N;
    static const Nodes nodes;
    const OrSeries series(w);
    long double fp[N], fq[N], p[N], q[N];
    for (int i = 0; i < N; ++i) series.sum(nodes.x[i], &fp[i], &fq[i]);
    interpolate<N>(nodes.x, fp, p);
    interpolate<N>(nodes.x, fq, q);
    for (int k = 0; k < N; ++k) {
        out->p[k] = (double)p[k];
        out->q[k] = (double)q[k];
    }
    out->c_mid = (double)cosl(0.5L * kPi * w);
    out->s_mid = (double)sinl(0.5L * kPi * w);
    out->c_far = (double)cosl(kPi * w);
    out->s_far = (double)sinl(kPi * w);
}

}  // namespace

OrOmega make_or_omega(double omega)
{
    OrOmega om{};
    om.omega = omega;
    make_power(omega, &om.power);
    return om;
}

}  // namespace gf
