// hrr_devbuild.hpp -- shared by the kernels that build a hierarchy and its
// tables on the GPU (hrr_build_device.hip, hrr_kernels.hip).
#pragma once

#include <stdint.h>

#ifndef HRR_HD   // host and device inline functions (also defined by hrr_rmq.hpp)
#if defined(__HIPCC__)
#define HRR_HD __host__ __device__ __forceinline__
#else
#define HRR_HD inline
#endif
#endif

namespace hrr {

// min / max with the host builder's tie rule (std::min / std::max keep the
// first operand unless the second is strictly smaller / larger), so that
// signed zeros come out the same: merged in sequence order, a bound is the
// first light's that attains it.
HRR_HD float min_first(float x, float y) { return y < x ? y : x; }
HRR_HD float max_first(float x, float y) { return x < y ? y : x; }

namespace devbuild {

// Morton quantisation box, lo xyz and hi xyz.
struct QBox {
    float lo[3], hi[3];
};

}  // namespace devbuild
}  // namespace hrr
