// The test at the end of an adaptive window (Section 6, adaptive_solve).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

namespace amg355 {

// The factor of a window of k iterations whose residuals have the quotient q.
inline double window_factor(double q, int k) { return std::pow(q, 1.0 / (double)k); }

// The largest quotient whose factor does not exceed rho_max (-1: every one does),
// for a kernel that takes the same decisions without pow: beside rho_max^k, found
// on the bit patterns of the non-negative numbers, which the factor follows.
inline double window_limit(double rho_max, int k) {
    if (std::isnan(rho_max)) return rho_max;
    auto value = [](uint64_t u) {
        double q;
        std::memcpy(&q, &u, sizeof q);
        return q;
    };
    auto within = [&](uint64_t u) { return window_factor(value(u), k) <= rho_max; };
    const uint64_t inf = 0x7ffull << 52;
    if (!within(0)) return -1.0;
    if (within(inf)) return value(inf);
    uint64_t at = 0;
    const double guess = std::pow(rho_max, (double)k);
    std::memcpy(&at, &guess, sizeof at);
    uint64_t lo = std::min(at, inf), hi = lo;   // within(lo), !within(hi)
    uint64_t step = 1;
    if (within(lo)) {
        do {
            lo = hi;
            hi = std::min(inf, hi + step);
            step *= 2;
        } while (within(hi));
    } else {
        do {
            hi = lo;
            lo = lo > step ? lo - step : 0;
            step *= 2;
        } while (!within(lo));
    }
    while (hi - lo > 1) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (within(mid)) lo = mid;
        else hi = mid;
    }
    return value(lo);
}

}  // namespace amg355
