// Integer quotients of the placement code by float products: a handful of instructions against the forty of an integer
// division, on paths that every wavefront walks between two round trips to memory.  Plain C++, so that tests on the host run it.
#pragma once

namespace kvc {

// x / d for 0 <= x < 2^30, 0 < d and a quotient below 2^20; recip within an ulp of 1 / d.  The product is off by less than one: float(x),
// recip and the product itself are off by 2^-24, 2^-23 and 2^-24 of the quotient; one correction either way makes it exact.
constexpr int quotient(int x, int d, float recip) {
    const int q = int(float(x) * recip);
    const int rem = x - q * d;
    return q + (rem >= d) - (rem < 0);
}

// The same for any quotient of 0 <= x < 2^30: the product is off by up to 2^8 steps either way, below 2^20 by one.
constexpr int quotient_wide(int x, int d, float recip) {
    int q = int(float(x) * recip);
    int rem = x - q * d;
    for (; rem < 0; rem += d) --q;
    for (; rem >= d; rem -= d) ++q;
    return q;
}

}  // namespace kvc
