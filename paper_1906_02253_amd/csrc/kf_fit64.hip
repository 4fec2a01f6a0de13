// Fits in 64 bits of many tracks: two waves a SIMD.  A file of its own because
// it is compiled without hoisting out of loops: the compiler hoists the 64-bit
// constants of sine and cosine out of the step loop, some 70 registers of them,
// which two waves do not have, so that they left for scratch memory and were
// read back in every step.  Without hoisting nothing spills.  200,000 tracks of
// 0.3 and 100 GeV 224 us, 245 with hoisting, 254 by one wave a SIMD; 500,000
// with barrels and disks 555, 679 and 690.  The other fits have the registers
// (4,000,000 mixed fits 1499 us with hoisting, 1564 without).
#include "kf_fit.hpp"

namespace kfmi {

void launch_fit64(const FitArgs& a, dim3 g, int k0, int k1, int init, bool learn, bool field, bool map,
                  hipStream_t s)
{
    if (learn) fit_launch<double, double, double, true, kAnySteps, 2>(a, g, k0, k1, init, field, map, s);
    else fit_launch<double, double, double, false, kAnySteps, 2>(a, g, k0, k1, init, field, map, s);
}

}  // namespace kfmi
