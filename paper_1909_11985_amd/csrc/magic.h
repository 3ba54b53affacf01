// Division of non-negative integers by a constant, as a multiplication and a shift.
#pragma once

namespace edl {

inline unsigned long long magic_of(int d) {
    if (d <= 0) return 0;
    return ((1ull << 40) + (unsigned long long)d - 1) / (unsigned long long)d;
}

// n / d == (n * magic_of(d)) >> 40 for every 0 <= n <= n_max: the error term needs n * d < 2^40 and the
// product must fit 64 bits
inline bool magic_fits(double n_max, int d) {
    if (d <= 0) return true;
    return n_max * (double)d < 1.0e12 && n_max * (double)magic_of(d) < 9.0e18;
}

}  // namespace edl
