// The FP32 screen of the structure analyses: image, squared distance and the
// bound up to which a candidate is noted.  No HIP header is needed: a test
// compiles this file for the CPU.
#pragma once

#include <math.h>

namespace mdpl {

// Folded coordinate x next to the cells beyond the lower (w < 0) or the upper
// (w > 0) face of the box edge L.
__device__ __forceinline__ float screen_image(float x, double L, int w) {
  return w < 0 ? x + (float)L : (w > 0 ? x - (float)L : x);
}

__device__ __forceinline__ float screen_d2(float ax, float ay, float az) {
  return __builtin_fmaf(az, az, __builtin_fmaf(ay, ay, ax * ax));
}

// Distance bound of the screen.  With M = 2^p above every box edge plus one
// cell (at most a third of an edge), an FP32 copy is within 2^(p-25) of the
// folded FP64 coordinate, and so is each of the two further roundings of an
// image (of L and of the sum): particle and candidate together 4 2^(p-25).
// The difference of a bond, at most rc + 2^(p-23), rounds by 2^-24 of that.
// So each component is within D = 2^(p-23) + 2^-24 (rc + 2^(p-23)) of the
// exact one, and the squared distance within
//   e = 2 sqrt(3) rc D + 3 D^2 + 4 2^-24 (rc + sqrt(3) D)^2,
// the last term for its three roundings.  Candidates up to rc^2 + 2 e are
// noted (the second e: FP64 roundings of the fold, within 2^-32 of an edge).
inline float screen_r2(const double box[3], const double side[3], double rc2) {
  double m = 0.0;
  for (int k = 0; k < 3; ++k) m = box[k] + side[k] > m ? box[k] + side[k] : m;
  const double u = 1.0 / 16777216.0, rc = sqrt(rc2);  // 2^-24
  const double x = 2.0 * u * exp2(ceil(log2(m * (1.0 + 1e-9))));
  const double d = x + u * (rc + x), r = rc + sqrt(3.0) * d;
  const double err = 2.0 * sqrt(3.0) * rc * d + 3.0 * d * d + 4.0 * u * r * r;
  return nextafterf((float)(rc2 + 2.0 * err), 3.0e38f);
}

}  // namespace mdpl
