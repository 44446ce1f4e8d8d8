// Host check of sph::box_cell against integer division, over every cell of boxes
// up to the largest (512 to a side) and a wavefront's cells past the end, whose
// indices must stay inside the box.  Prints "nx ny nz wrong outside" per box.
#include <stdio.h>

#include "sph_walk_cell.h"

int main()
{
    const int boxes[][3] = {{1, 1, 1},       {1, 1, 512},     {512, 1, 1},    {3, 5, 7},
                            {9, 9, 9},       {13, 11, 12},    {64, 64, 64},   {101, 103, 107},
                            {128, 128, 128}, {200, 201, 203}, {256, 256, 256}, {512, 3, 511},
                            {511, 512, 509}, {512, 512, 512}};
    int bad = 0;
    for (const auto& b : boxes) {
        const int nx = b[0], ny = b[1], nz = b[2];
        const float ryz1 = 1.0f / (float)(ny * nz), rz1 = 1.0f / (float)nz;
        const int n = nx * ny * nz;
        long wrong = 0, outside = 0;
        for (int q = 0; q < n + 64; ++q) {
            int ix, iy, iz;
            sph::box_cell(q, nx, ny, nz, ryz1, rz1, ix, iy, iz);
            outside += ix < 0 || ix >= nx || iy < 0 || iy >= ny || iz < 0 || iz >= nz;
            if (q < n) wrong += ix != q / (ny * nz) || iy != q / nz % ny || iz != q % nz;
        }
        printf("%d %d %d %ld %ld\n", nx, ny, nz, wrong, outside);
        bad += wrong != 0 || outside != 0;
    }
    return bad ? 1 : 0;
}
