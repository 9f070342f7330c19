#include "spectral_modes.h"

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <utility>

namespace cgd {

// QR steps with Wilkinson's shift, each a chase of the bulge that the first rotation
// makes (the method of Golub and Van Loan, "Matrix Computations", 8.3).  In
// the basis q1 = c u + s v, q2 = -s u + c v of a rotation the 2 x 2 block
// (a, b, g) has the diagonal c^2 a + 2 c s b + s^2 g, s^2 a - 2 c s b + c^2 g
// and the off-diagonal (c^2 - s^2) b + c s (g - a).
bool tridiagonal_modes(std::vector<double>& d, std::vector<double> e, std::vector<std::vector<double>>& z) {
    const int n = (int)d.size();
    z.assign(n, std::vector<double>(n, 0.0));
    for (int k = 0; k < n; ++k) z[k][k] = 1.0;
    e.resize(n, 0.0);
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(d[i]) || !std::isfinite(e[i])) return false;
    const double eps = 2.3e-16;
    int hi = n - 1;
    for (int64_t guard = 0; hi > 0; ++guard) {
        auto split = [&](int k) { return std::fabs(e[k]) <= eps * (std::fabs(d[k]) + std::fabs(d[k + 1])); };
        if (split(hi - 1)) {
            --hi;
            continue;
        }
        if (guard >= 60 * (int64_t)n) return false;
        int lo = hi - 1;
        while (lo > 0 && !split(lo - 1)) --lo;
        const double half = 0.5 * (d[hi - 1] - d[hi]), b = e[hi - 1];
        const double mu = d[hi] - b * b / (half + std::copysign(std::hypot(half, b), half));
        double x = d[lo] - mu, y = e[lo];
        for (int k = lo; k < hi; ++k) {
            const double r = std::hypot(x, y);
            if (r == 0.0) break;
            const double c = x / r, s = y / r;
            const double p = d[k], q = e[k], g = d[k + 1];
            d[k] = c * c * p + 2.0 * c * s * q + s * s * g;
            d[k + 1] = s * s * p - 2.0 * c * s * q + c * c * g;
            e[k] = (c * c - s * s) * q + c * s * (g - p);
            if (k > lo) e[k - 1] = r;
            if (k + 1 < hi) {
                y = s * e[k + 1];
                e[k + 1] *= c;
            }
            x = e[k];
            double* u = z[k].data();
            double* v = z[k + 1].data();
            for (int i = 0; i < n; ++i) {
                const double ui = u[i], vi = v[i];
                u[i] = c * ui + s * vi;
                v[i] = c * vi - s * ui;
            }
        }
    }
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(d[i])) return false;
    return true;
}

bool axis_modes(const std::vector<double>& h, bool sym, bool periodic, AxisModes* out) {
    std::vector<double> &lam = out->lam, &mats = out->mats;
    const int n = (int)h.size();
    const int hm = sym ? (n + 1) / 2 : n, ho = sym ? n / 2 : 0, mt = (hm + 15) / 16;
    std::vector<double> g(n + 1, 0.0), s(n), o(n, 0.0);
    for (int i = 1; i < n; ++i) g[i] = 2.0 / (h[i - 1] + h[i]);
    double oper = 0.0;
    if (periodic) {
        g[0] = g[n] = 2.0 / (h[0] + h[n - 1]);
        oper = -g[0] / std::sqrt(h[0] * h[n - 1]);
    }
    for (int i = 0; i < n; ++i) s[i] = (g[i] + g[i + 1]) / h[i];
    for (int i = 0; i + 1 < n; ++i) o[i] = -g[i + 1] / std::sqrt(h[i] * h[i + 1]);
    lam.assign(n, 0.0);
    const size_t frag = (size_t)mt * 4 * mt * 64;
    mats.assign(4 * frag, 0.0);
    for (int odd = 0; odd < (ho ? 2 : 1); ++odd) {
        // the half of the modes with x[n-1-m] = +-x[m], in the coordinates of
        // m < ho (times 1 / sqrt 2 in full) and, even ones of an odd n, the
        // middle cell; sign * o for the neighbour that is the mirror image
        const int nn = odd ? ho : hm;
        std::vector<double> d(s.begin(), s.begin() + nn), e(o.begin(), o.begin() + nn);
        const double sg = odd ? -1.0 : 1.0;
        if (sym) {
            d[0] += n > 1 ? sg * oper : 0.0;
            if (n % 2 == 0) d[nn - 1] += sg * o[ho - 1];
            else if (!odd && nn > 1) e[nn - 2] *= std::sqrt(2.0);
        }
        std::vector<std::vector<double>> z;
        if (!tridiagonal_modes(d, e, z)) return false;
        double* f = mats.data() + (odd ? frag : 0);
        double* inv = mats.data() + (odd ? 3 : 2) * frag;
        for (int k = 0; k < nn; ++k) {
            lam[odd ? hm + k : k] = d[k];
            for (int m = 0; m < nn; ++m) {
                const double v = z[k][m] * (sym && m < ho ? std::sqrt(0.5) : 1.0);
                // entry (row, col) of a packed matrix
                auto at = [&](int row, int col) {
                    return (((size_t)(row / 16) * 4 * mt + col / 4) * 64) + (size_t)(col % 4) * 16 + row % 16;
                };
                f[at(k, m)] = v * std::sqrt(h[m]);
                inv[at(m, k)] = v / std::sqrt(h[m]);
            }
        }
    }
    return true;
}

}  // namespace cgd
