// Where a ray's walk crosses a slab of the grid (host and device: the ray
// kernel runs it, and a host test checks its rounding).
#pragma once

#include <hip/hip_runtime.h>

namespace gb {

// The ray parameters at which coordinate om + t * dm meets the slab's faces pa and
// pa + w.  Each is a difference and a quotient, one rounding each: the margin by
// which the walk widens a slab covers that.  (By a reciprocal kept for the ray it
// is a rounding more, and the distance from the box up to which the margin holds
// is a third less, for 0.6%: 1M rays over a 10M-triangle grid 2118 us against 2132.)
__host__ __device__ inline void slab_faces(float pa, float w, float om, float dm, float& ta, float& tb) {
  ta = (pa - om) / dm;
  tb = (pa + w - om) / dm;
}

}  // namespace gb
