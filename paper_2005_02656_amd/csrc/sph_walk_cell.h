// sph_walk_cell.h -- which cell of a box the group walk's q-th is: host and device
// code, so that the arithmetic can be checked on the CPU.
#pragma once

#include <hip/hip_runtime.h>

namespace sph {

// Cell q of a box of nx x ny x nz cells, x outermost and z fastest, each at most
// 512 (0 <= q < nx ny nz; past the end the indices stay bounded).  Quotients by
// reciprocals (ryz1 = 1 / (ny nz), rz1 = 1 / nz): an integer division costs some
// twenty instructions.  q needs up to 27 bits, more than FP32 holds, and its
// quotient can come out one off from 6.7 M cells on (200 x 201 x 203: the last
// cell of a slab read as the first of the next); the remainder shows it.  Below
// 2^18 (the index in a slab) the rounding is under an eighth of the distance of
// q + 1/2 from a multiple.
__host__ __device__ inline void box_cell(int q, int nx, int ny, int nz, float ryz1, float rz1,
                                         int& ix, int& iy, int& iz)
{
    const int nyz = ny * nz;
    ix = (int)(((float)q + 0.5f) * ryz1);
    ix = ix < nx - 1 ? ix : nx - 1;
    int r = q - ix * nyz;
    if (r < 0) {
        ix -= 1;
        r += nyz;
    } else if (r >= nyz && ix < nx - 1) {
        ix += 1;
        r -= nyz;
    }
    iy = (int)(((float)r + 0.5f) * rz1);
    iy = iy < ny - 1 ? iy : ny - 1;
    iz = r - iy * nz;
    iz = iz < nz - 1 ? iz : nz - 1;
}

}  // namespace sph
