// growth.hpp -- a lane's account of how far visits have raised the sum of x^2
// over pixels, by which the sparse region job (sparse.hpp) tells whether a window
// below its bound may have been lifted to it.
//
// The growth since a test is kept apart from what grew before it: next to a large
// sum the small additions of a later side would be lost to rounding, and with them
// the visit of a window over its bound.  No sum takes more than 2^10 additions (the
// rounds of a side, or the sides) and none is a difference, so each is within
// 2^10 x 2^-24 of itself, the three together within 2e-4: kGrowth covers that, the
// sum over the lanes and the few roundings of an addition.
#pragma once

namespace smre {

constexpr float kGrowth = 1.001f;

struct Growth {
  float since;  // since the last test of the side visited, or since the side was begun
  float side;   // of this side before that test
  float total;  // since the test at the start of the job, up to the side visited
  __host__ __device__ __forceinline__ void add(float e) { since += e; }
  __host__ __device__ __forceinline__ void tested() {
    side += since;
    since = 0.0f;
  }
  __host__ __device__ __forceinline__ void side_done() {
    total += side + since;
    side = since = 0.0f;
  }
};

}  // namespace smre
