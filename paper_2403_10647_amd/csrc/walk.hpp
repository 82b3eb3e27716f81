// Where a ray's walk crosses a slab of the grid (host and device: the ray
// kernel runs it, and a host test checks its rounding).
#pragma once

#include <hip/hip_runtime.h>

namespace gb {

// The ray parameter at which coordinate om + t * dm meets the plane p: a difference
// and a quotient, one rounding each, which the margin by which the walk widens a
// slab covers.  (By a reciprocal kept for the ray it is a rounding more, and the
// distance from the box up to which the margin holds is a third less.)
__host__ __device__ inline float plane_t(float p, float om, float dm) { return (p - om) / dm; }

}  // namespace gb
