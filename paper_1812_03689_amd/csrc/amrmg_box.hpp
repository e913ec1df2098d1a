// amrmg_box.hpp -- the box of cells that the stencils of some particles span
// (host and device code).
#pragma once
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>

namespace amrmg {

// a box of cells [lo, hi], x fastest, and the bricks it spans
struct CellBox {
    int lo[3], hi[3];
    int ex, ey, ez;
    int bx0, by0, bz0, nbx, nby, nbt;
    int64_t vol;
    // v: minima of i0 and of ~i1 per axis over the particles, INT_MAX where
    // there is none (then a box of no cells at 0: the extents of [INT_MAX,
    // INT_MIN] would overflow)
    __host__ __device__ __forceinline__ void set(const int *v)
    {
        const bool none = v[0] == INT_MAX;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lo[d] = none ? 0 : v[d];
            hi[d] = none ? -1 : ~v[3 + d];
        }
        ex = hi[0] - lo[0] + 1, ey = hi[1] - lo[1] + 1, ez = hi[2] - lo[2] + 1;
        vol = (int64_t)ex * ey * ez;
        bx0 = lo[0] >> 3, by0 = lo[1] >> 3, bz0 = lo[2] >> 3;
        nbx = (hi[0] >> 3) - bx0 + 1, nby = (hi[1] >> 3) - by0 + 1;
        nbt = nbx * nby * ((hi[2] >> 3) - bz0 + 1);
    }
    __host__ __device__ __forceinline__ bool empty() const { return lo[0] > hi[0]; }
};

}  // namespace amrmg
