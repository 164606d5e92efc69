// How many steps a block of hard-sphere beads may go without a scan.
//
// A block whose nearest bead is D from the tip cannot hold a bead within
// b + sigma of it before the tip has come D - (b + sigma) closer, and each
// step brings it at most b closer.  The rule works on lengths in units of b:
// the ratios are formed in binary64, so that binary32 only ever holds numbers
// of the order of N^2, whatever the bond length, and what does not fit there
// (a square that overflows or underflows binary64, or a NaN) gives no step to
// skip.  Its two factors and the 0.01 are far above the arithmetic's error
// (below 10^-6 of D, and D is at most 16384 b).
#pragma once

#include <math.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define RSAW_SKIP_FN __host__ __device__ __forceinline__
#else
#define RSAW_SKIP_FN inline
#endif

namespace rsaw {

// 1 / b^2: the factor that takes squared distances to units of b.
RSAW_SKIP_FN double skip_unit(double b) { return 1.0 / (b * b); }

// (b + sigma) / b, rounded up, from the culling bound (b + sigma)^2.
RSAW_SKIP_FN float skip_reach(double cull2, double unit) { return (float)sqrt(cull2 * unit) * 1.00001f; }

// Whole steps that may pass before the next scan, from the least squared tip
// distance of the block's beads in units of b; 0 for anything but a number of
// steps that a chain can have.
RSAW_SKIP_FN int skip_steps(float d2, float reach)
{
#ifdef __HIP_DEVICE_COMPILE__
    const float d = __builtin_amdgcn_sqrtf(d2); // to 1 ulp
#else
    const float d = sqrtf(d2);
#endif
    const float n = floorf(d * 0.99999f - reach - 0.01f);
    return n > 0.0f && n < 20000.0f ? (int)n : 0;
}

} // namespace rsaw
