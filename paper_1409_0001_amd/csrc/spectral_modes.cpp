#include "spectral_modes.h"

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <utility>

namespace cgd {

// QR steps with Wilkinson's shift, each a chase of the bulge that the first
// rotation makes (the method of Golub and Van Loan, "Matrix Computations",
// 8.3).  In the basis q1 = c u + s v, q2 = -s u + c v of a rotation the 2 x 2
// block (a, b, g) has the diagonal c^2 a + 2 c s b + s^2 g, s^2 a - 2 c s b +
// c^2 g and the off-diagonal (c^2 - s^2) b + c s (g - a).
bool tridiagonal_modes(std::vector<double>& d, std::vector<double> e, Rotations& rot) {
    const int n = (int)d.size();
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
        const size_t first = rot.cs.size();
        for (int k = lo; k < hi; ++k) {
            const double rr = x * x + y * y;
            // (the square root alone where the squares neither overflow nor lose bits)
            const double r = rr > 1e-280 && rr < 1e280 ? std::sqrt(rr) : std::hypot(x, y);
            if (r == 0.0) break;
            const double inv = 1.0 / r, c = x * inv, s = y * inv;
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
            rot.cs.push_back(c);
            rot.cs.push_back(s);
        }
        if (const int count = (int)((rot.cs.size() - first) / 2)) rot.sweeps.push_back({lo, count});
    }
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(d[i])) return false;
    return true;
}

void group_rotations(const Rotations& rot, RotationGroups& out) {
    constexpr int L = RotationGroups::kLanes, S = RotationGroups::kGroupSteps;
    const double* cs = rot.cs.data();
    for (size_t i = 0; i < rot.sweeps.size(); i += L) {
        const size_t n = std::min<size_t>(L, rot.sweeps.size() - i);
        int lo = rot.sweeps[i].lo, hi = lo;
        for (size_t j = 0; j < n; ++j) {
            lo = std::min(lo, rot.sweeps[i + j].lo);
            hi = std::max(hi, rot.sweeps[i + j].lo + rot.sweeps[i + j].count);
        }
        const int rows = hi - lo + 1, count = (rows + L - 1 + S - 1) / S * S;
        const size_t at = out.cs.size();
        out.groups.push_back({lo, rows, count});
        out.cs.resize(at + (size_t)count * L * 2, 0.0);
        for (size_t k = at; k < out.cs.size(); k += 2) out.cs[k] = 1.0;
        for (size_t j = 0; j < n; ++j) {
            const Rotations::Sweep& s = rot.sweeps[i + j];
            for (int k = s.lo; k < s.lo + s.count; ++k, cs += 2) {
                double* to = out.cs.data() + at + ((size_t)(k - lo + j) * L + j) * 2;
                to[0] = cs[0];
                to[1] = cs[1];
            }
        }
    }
}

bool axis_modes(const std::vector<double>& h, bool sym, bool periodic, RotationGroups rot[2], std::vector<double>& lam) {
    const int n = (int)h.size();
    const int hm = sym ? (n + 1) / 2 : n, ho = sym ? n / 2 : 0;
    std::vector<double> g(n + 1, 0.0), s(n), o(n, 0.0);
    for (int i = 1; i < n; ++i) g[i] = 2.0 / (h[i - 1] + h[i]);
    double oper = 0.0;
    if (periodic) {
        g[0] = g[n] = 2.0 / (h[0] + h[n - 1]);
        oper = -g[0] / std::sqrt(h[0] * h[n - 1]);
    }
    for (int i = 0; i < n; ++i) s[i] = (g[i] + g[i + 1]) / h[i];
    for (int i = 0; i + 1 < n; ++i) o[i] = -g[i + 1] / std::sqrt(h[i] * h[i + 1]);
    lam.clear();
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
        e.resize(std::max(0, nn - 1));
        Rotations r;
        if (!tridiagonal_modes(d, std::move(e), r)) return false;
        group_rotations(r, rot[odd]);
        lam.insert(lam.end(), d.begin(), d.end());
    }
    return true;
}

}  // namespace cgd
