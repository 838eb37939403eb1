// Host tables: Gauss-Legendre latitudes and orthonormal associated Legendre
// functions (Section 3), computed in long double.
#include <cfloat>
#include <cmath>

#include "internal.hpp"

namespace rexi {

// Roots of P_nlat by Newton's method from the estimate cos(pi (i + 3/4)/(nlat + 1/2)),
// P_n by k P_k = (2k-1) x P_{k-1} - (k-1) P_{k-2}, P'_n = n (x P_n - P_{n-1})/(x^2-1);
// weights 2 / ((1 - x^2) P'_n(x)^2).  Order: descending x (north to south).
void gauss_legendre(int nlat, std::vector<double>& mu, std::vector<double>& w) {
    mu.resize(nlat);
    w.resize(nlat);
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int i = 0; i < nlat; ++i) {
        long double x = cosl(pi * (i + 0.75L) / (nlat + 0.5L));
        long double dp = 1;
        for (int it = 0; it < 100; ++it) {
            long double p0 = 1, p1 = x;
            for (int k = 2; k <= nlat; ++k) {
                const long double p2 = ((2 * k - 1) * x * p1 - (k - 1) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            if (nlat == 1) { p1 = x; p0 = 1; }
            dp = nlat * (x * p1 - p0) / (x * x - 1);
            const long double dx = p1 / dp;
            x -= dx;
            if (fabsl(dx) < 1e-19L * fmaxl(1.0L, fabsl(x))) break;
        }
        {
            long double p0 = 1, p1 = x;
            for (int k = 2; k <= nlat; ++k) {
                const long double p2 = ((2 * k - 1) * x * p1 - (k - 1) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = nlat * (x * p1 - p0) / (x * x - 1);
        }
        mu[i] = (double)x;
        w[i] = (double)(2.0L / ((1 - x * x) * dp * dp));
    }
}

// Orthonormal associated Legendre functions by the three-term recurrence in n:
//   P_m^m = (1/sqrt2) prod_{k=1}^{m} sqrt((2k+1)/(2k)) (1-mu^2)^{m/2},
//   P_n^m = (mu P_{n-1}^m - e_{n-1} P_{n-2}^m) / e_n,  e_n = sqrt((n^2-m^2)/(4n^2-1))
// (e_m = 0).  With P_n = s_n Q_n, s_m = s_{m+1} = 1 and s_n = (e_{n-1} / e_n) s_{n-2}
// it has one coefficient,
//   Q_n = c_n mu Q_{n-1} - Q_{n-2},  c_n = s_{n-1} / (e_n s_n),
// two operations per value instead of three (s_n falls from 1 to about 0.2 over
// 1024 degrees).  The device runs this recurrence itself; the host supplies c_n, s_n
// and, every `run` degrees, exact restart values of Q.
namespace {
// c_n (0 at n = m) and s_n of order m, index n - m
void order_coefs(int T, int m, std::vector<long double>& c, std::vector<long double>& s) {
    c.assign(T + 1 - m, 0.0L);
    s.assign(T + 1 - m, 1.0L);
    long double before = 0;  // e_{n-1}
    for (int n = m + 1; n <= T; ++n) {
        const long double e = sqrtl((long double)(n * n - m * m) / (4.0L * n * n - 1));
        const int k = n - m;
        if (k > 1) s[k] = before / e * s[k - 2];
        c[k] = s[k - 1] / (e * s[k]);
        before = e;
    }
}
}  // namespace

// c_n and s_n in spectral order, [nspec] each.
void legendre_coefs(int T, std::vector<double>& coef, std::vector<double>& scale) {
    coef.clear();
    scale.clear();
    std::vector<long double> c, s;
    for (int m = 0; m <= T; ++m) {
        order_coefs(T, m, c, s);
        coef.insert(coef.end(), c.begin(), c.end());
        scale.insert(scale.end(), s.begin(), s.end());
    }
}

// Restart rows for runs of `run` degrees: for every order m and run r with
// n0 = m + run r <= T, row (run_base[m] + r) holds Q_{n0-1}(mu_j) (0 at n0 = m)
// and Q_{n0}(mu_j), layout [row][2][nmu].  Long double (its exponent range
// holds the seeds down to the Gaussian latitude nearest a pole at T = 1023);
// values below 1e-300 are stored as 0.  tail: the same at the four parts of an
// order's last segment of `seg` degrees where that one is not whole, layout
// [m][4][2][nmu]: a part has 8 ceil(Ls / 32) degrees (Ls those of the segment), and
// parts past its end hold 0.
std::vector<double> legendre_restarts(int T, int run, int seg, const std::vector<double>& mu,
                                      std::vector<int>& run_base, std::vector<double>& tail) {
    const int nmu = (int)mu.size();
    tail.assign((size_t)(T + 1) * 8 * nmu, 0.0);
    run_base.assign(T + 2, 0);
    for (int m = 0; m <= T; ++m) run_base[m + 1] = run_base[m] + (T + 1 - m + run - 1) / run;
    std::vector<double> out((size_t)run_base[T + 1] * 2 * nmu, 0.0);
    auto put = [&](std::vector<double>& to, int row, int which, int j, long double v) {
        double d = (double)v;
        if (fabs(d) < 1e-300) d = 0.0;
        to[((size_t)row * 2 + which) * nmu + j] = d;
    };
    std::vector<long double> pmm(nmu, 1.0L / sqrtl(2.0L)), cosine(nmu), c, s;
    for (int j = 0; j < nmu; ++j) cosine[j] = sqrtl(fmaxl(0.0L, 1 - (long double)mu[j] * mu[j]));
    for (int m = 0; m <= T; ++m) {
        order_coefs(T, m, c, s);
        const long double up = m > 0 ? sqrtl((2.0L * m + 1) / (2.0L * m)) : 1.0L;
        const int L = T + 1 - m, t0 = L / seg * seg, part = 8 * ((L - t0 + 31) / 32);  // tail from m + t0
        for (int j = 0; j < nmu; ++j) {
            if (m > 0) pmm[j] *= up * cosine[j];
            const long double x = mu[j];
            long double q2 = 0, q1 = pmm[j];  // Q_{n-1}, Q_n at n = m
            for (int k = 0;; ++k) {
                if (k % run == 0) {
                    const int row = run_base[m] + k / run;
                    put(out, row, 0, j, q2);
                    put(out, row, 1, j, q1);
                }
                if (k >= t0 && (k - t0) % part == 0) {
                    const int row = m * 4 + (k - t0) / part;
                    put(tail, row, 0, j, q2);
                    put(tail, row, 1, j, q1);
                }
                if (k == L - 1) break;
                const long double q = c[k + 1] * x * q1 - q2;
                q2 = q1;
                q1 = q;
            }
        }
    }
    return out;
}

}  // namespace rexi
