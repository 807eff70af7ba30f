// The FP32 pseudo-potential deviation of the step kernels (dpsi_of of
// lb_step.hpp, compiled for the host) against expm1 in FP64: its largest error
// in units in the last place, and its values at infinite arguments.
#include "lb_step.hpp"

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

int main()
{
    double worst = 0;
    float at = 0;
    // every 101st float of both signs with 2^-30 <= |t| <= 80
    uint32_t lo, hi;
    const float a = 0x1p-30f, b = 80.0f;
    std::memcpy(&lo, &a, 4);
    std::memcpy(&hi, &b, 4);
    for (uint32_t k = lo; k <= hi; k += 101)
        for (uint32_t sign : {0u, 0x80000000u}) {
            const uint32_t bits = k | sign;
            float d;
            std::memcpy(&d, &bits, 4);
            // e = 1 and rho_0 = 1 add no rounding of their own
            const double ref = -std::expm1(-(double)d);
            const float got = lbk::dpsi_of(d, 1.0f, 1.0f);
            int ex;
            (void)std::frexp(ref, &ex);
            const double err = std::fabs((double)got - ref) / std::ldexp(1.0, ex - 24);
            if (!(err <= worst)) { worst = err; at = d; }
        }
    const float inf = INFINITY;
    std::printf("worst %.4f ulp at d = %.9g\n", worst, at);
    std::printf("+inf %g, -inf %g\n", lbk::dpsi_of(inf, 1.0f, 1.0f), lbk::dpsi_of(-inf, 1.0f, 1.0f));
    return 0;
}
