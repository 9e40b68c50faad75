// The byte offsets along K of gemm256_kernel's direct loads, on the device and,
// for tests, on the host.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vt {
namespace pf {

struct KWalk {
  static constexpr int kTile = 32;  // k values of a k-tile: two k-steps of A, 64 bytes of a row of B
  uint32_t a0, a1, b;               // offsets of the k-tile's two k-steps in A, and in a row of B
  uint32_t step;                    // bytes of a k-step of A
  int left;                         // k-tiles still to load

  __host__ __device__ KWalk(int kt0, int n, uint32_t kstep_bytes)
      : a0(kt0 * 2 * kstep_bytes), a1(a0 + kstep_bytes), b(kt0 * kTile * 2), step(kstep_bytes), left(n) {
    if (done()) stop();
  }
  __host__ __device__ bool done() const { return left <= 0; }
  // Past the last k-tile the ranges are empty; an offset of 0 keeps every load
  // outside them whether the hardware compares the lane's offset with the range
  // or with the range less the scalar offset (which would wrap below zero).
  __host__ __device__ void stop() { a0 = a1 = b = 0; }
  __host__ __device__ void next() {
    --left;
    a0 += 2 * step;
    a1 += 2 * step;
    b += kTile * 2;
    if (done()) stop();
  }
};

}  // namespace pf
}  // namespace vt
