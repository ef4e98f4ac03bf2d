// Index arithmetic of the kernels (host and device).
#pragma once

#include <hip/hip_runtime.h>

namespace msm {

// Quotient and remainder of 0 <= i < 2^22 by d > 0 with a float reciprocal
// (inv_d = 1/d rounded): (i + 1/2)/d lies at least 1/(2d) away from an integer,
// and the two roundings, of 1/d and of the product, move it by less than
// (i + 1/2)/d 2^-23 < 1/(2d), so the truncation is exact.  Replaces the long
// integer-division sequence for runtime divisors.
constexpr int kFdivMax = 1 << 22;
__host__ __device__ __forceinline__ int fdiv(int i, int d, float inv_d, int& rem) {
  const int q = (int)(((float)i + 0.5f) * inv_d);
  rem = i - q * d;
  return q;
}

// Position (m, x fastest) of node `node` in a grid of n[0] x n[1] x n[2] =
// count nodes.  A grid may have 2^28 nodes, more than fdiv is exact for (it puts
// 356 nodes of a face of 182^3 on the opposite face of the next row): above
// 2^22 nodes by integer divisions, a branch that is the same for a whole launch.
__host__ __device__ __forceinline__ void node_position(int node, const int* n, int count, int* m) {
  if (count <= kFdivMax) {
    m[2] = fdiv(fdiv(node, n[0], 1.f / (float)n[0], m[0]), n[1], 1.f / (float)n[1], m[1]);
  } else {
    const unsigned row = (unsigned)node / (unsigned)n[0];
    m[0] = node - (int)row * n[0];
    m[2] = (int)(row / (unsigned)n[1]);
    m[1] = (int)row - m[2] * n[1];
  }
}

// The images of a node i of the period [0, p) along one dimension, itself
// included, on a level with G ghost nodes to a side: i + j p for j = first ..
// first + count - 1, those in [-G, p + G).
struct ImageRange {
  int first, count;
};
__host__ __device__ __forceinline__ ImageRange image_range(int i, int p, int G) {
  const float inv_p = 1.f / (float)p;
  int rb, ra;
  int below = fdiv(i + G, p, inv_p, rb), above = fdiv(p + G - 1 - i, p, inv_p, ra);
  // a period beyond fdiv's range: the quotient is off by one at most
  below += (rb >= p) - (rb < 0);
  above += (ra >= p) - (ra < 0);
  return {-below, below + above + 1};
}

}  // namespace msm
