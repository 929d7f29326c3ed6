// window_limit (csrc/window.hpp): comparing a quotient with it decides as the factor
// of the window does, for every rho_max and k, beside the limit and far from it.
#include "window.hpp"

#include <cstdio>

int main() {
    const double inf = INFINITY, nan = NAN;
    long bad = 0, seen = 0;
    for (double rho : {-inf, -1.0, -0.0, 0.0, 1e-300, 0.01, 0.3, 0.5, 0.9, 0.999999, 1.0, 1.5, 1e10, 1e300, inf, nan})
        for (int k : {1, 2, 3, 4, 5, 7, 10, 100, 1000, 5000}) {
            const double limit = amg355::window_limit(rho, k);
            auto same = [&](double q) {
                seen += 1;
                bad += (amg355::window_factor(q, k) > rho) != (q > limit);
            };
            for (double q : {0.0, 5e-324, 1e-300, 1e-10, 0.1, 0.5, 1.0, 2.0, 1e300, inf, nan}) same(q);
            double up = std::max(limit, 0.0), down = up;
            for (int i = 0; i < 50; ++i, up = std::nextafter(up, inf), down = std::nextafter(down, 0.0)) {
                same(up);
                same(down);
            }
        }
    std::printf("%ld quotients, %ld wrong\n%s\n", seen, bad, bad ? "window_limit: wrong" : "window_limit: ok");
    return bad != 0;
}
