// Launchers of the multi-grid (pyramid) passes (pyramid.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace pmk {

// A 3-D field of up to three channels, x-blocked by 8 like every mesh of the
// library, with power-of-2 dims (nx >= 8):
//   PYR_SEPARATE    p[c] + xoff(x, y, z)
//   PYR_INTERLEAVED p[0] + 3 * xoff(x, y, z) + c
// xoff(x, y, z) = (((x / 8) * ny + y) * nz + z) * 8 + x % 8, which for a cube
// is blk_real.
enum PyrKind : int { PYR_SEPARATE = 0, PYR_INTERLEAVED = 1 };

struct PyrField {
  float* p[3] = {nullptr, nullptr, nullptr};
  int kind = PYR_SEPARATE;
  int nx = 0, ny = 0, nz = 0;
};

// How a pass writes its value v to the destination.
enum PyrMode : int {
  PYR_STORE = 0,     // dst = v
  PYR_COMBINE = 1,   // dst = alpha * aux - v   (REDUCE into separate channels; aux: interleaved, dst's cube)
  PYR_ADD = 2,       // dst += v
  PYR_SUB = 3,       // dst -= v
};

// One level of REDUCE (centred stride-2 convolution with the order-6 B-spline,
// every axis halves) or of EXPAND (the transposed convolution times 8, every
// axis doubles), periodic, over ch channels (1, separate, or 3).  dst's dims
// are src's halved (8 at least) or doubled (16 at least).
void launch_pyr_level(bool expand, int ch, const PyrField& src, const PyrField& dst, int mode, const float* aux,
                      float alpha, hipStream_t s);

}  // namespace pmk
