// gm_lattice.h -- point counts of the paper's lattice sampler (device), for the sampler and for
// the scan over its triangles.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace gm {

// Eq. (1): points of a triangle at resolution r.
__device__ __forceinline__ int64_t lattice_points(int64_t r) { return (r + 1) * (r + 2) / 2; }

// Eq. (4): Delta = (8 k) A + 1; r = 1 below Delta = 25, else the positive root
// (sqrt(Delta) - 3) / 2 truncated to a whole resolution.
__device__ __forceinline__ int64_t lattice_resolution(double k, double A)
{
    double delta = 8.0 * k;
    delta = delta * A;
    delta = delta + 1.0;
    if (!(delta >= 25.0)) return 1;
    return (int64_t)floor((sqrt(delta) - 3.0) / 2.0);
}

__device__ __forceinline__ unsigned long long lattice_count(double k, double A)
{
    return (unsigned long long)lattice_points(lattice_resolution(k, A));
}

}  // namespace gm
