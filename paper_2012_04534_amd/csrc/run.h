// Runs of neighbouring columns: how the learned network's kernels walk a grid.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ufss {

struct Dims {
    int nx, ny, nz;
    int64_t n;
};

struct Run {
    int z, x, y;            // depth, first column of the run
    int64_t v;              // its voxel (column x + k: v + k nz)
};

// Runs of XV columns x at one (y, z) of the grid [ny][nx][nz], depths fastest.
template <int XV>
__host__ __device__ inline int64_t run_count(const Dims& d) {
    return (int64_t)d.ny * ((d.nx + XV - 1) / XV) * d.nz;
}

// Run t of them, t < 2^32: 64-bit division takes several times as long, and no grid
// of a network has more (2^32 voxels take 515 GB of its and its plan's buffers).
template <int XV>
__host__ __device__ __forceinline__ Run run_at(const Dims& d, int64_t t) {
    const int nxr = (d.nx + XV - 1) / XV;
    const int c = (int)((uint32_t)t / (uint32_t)d.nz);        // at most nx ny
    Run r;
    r.z = (int)((uint32_t)t - (uint32_t)c * (uint32_t)d.nz);
    r.y = c / nxr;
    r.x = (c - r.y * nxr) * XV;
    r.v = ((int64_t)r.y * d.nx + r.x) * d.nz + r.z;
    return r;
}

}  // namespace ufss
