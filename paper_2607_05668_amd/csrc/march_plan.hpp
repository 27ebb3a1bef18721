// Host arithmetic of the marching kernels' launches (march.hpp): strips,
// segments and the limits of a lane's addresses.  Plain C++.
#pragma once

#include <algorithm>

constexpr int kMarchLanes = 64;         // lanes of a wavefront, cells of a population tile
constexpr int kSimds = 1024;
constexpr int kLdsPerCu = 160 * 1024;

// Grids whose addresses and row numbers the marching kernels hold.  Every
// population of a row lies in the 2^31 - 1 bytes that a buffer descriptor at
// the row's first tile covers (offsets beyond are refused by its range check):
// the row begins up to 63 cells into that tile, its last cell lies in tile
// (63 + nx - 1) / 64 at most, and that tile's last population ends with the
// tile: (nx + 126) populations' bytes.  Unwrapped row numbers run past ny by
// the halo.
constexpr bool march_fits(long long nx, long long ny, int populations, int elem)
{
    return (nx + 2 * kMarchLanes) * populations * elem <= 0x7fffffff && ny <= 0x7fffffff - kMarchLanes;
}

// Segments of `rows` rows, and the row at which the one from y0 on ends.
constexpr int march_segments(int ny, int rows) { return (ny - 1) / rows + 1; }
constexpr int segment_end(int y0, int rows, int ny) { return ny - y0 < rows ? ny : y0 + rows; }

// Rows of a wavefront's segment.  A wavefront of T stages with `halo` lanes
// and rows lost at each end collides T rows + T halo rows, so few long
// segments cost least, but one wavefront a SIMD is the least that fills the
// chip; a second one hides the latencies of the first and costs 1.75 times its
// time in place of twice (up to 30 populations; 1.5 times with more).  Counts
// just above one or two wavefronts a SIMD leave a SIMD with one more than the
// others: shallow water 512^2, four stages, rows 3 / 4 / 6 (1539, 1152, 774
// wavefronts): 7.4 / 8.0 / 7.1 us per step.
inline int march_strips(int halo, int nx) { return (nx + 64 - 2 * halo - 1) / (64 - 2 * halo); }
inline int march_rows(int halo, int lds, int populations, int nx, int ny)
{
    const int strips = march_strips(halo, nx), two = std::min(2 * kSimds, kSimds / 4 * (kLdsPerCu / lds));
    auto rows_for = [&](int waves) {
        return (ny - 1) / std::max(1, waves / strips) + 1;
    };
    const int r1 = rows_for(kSimds), r2 = rows_for(two);
    const double c1 = r1 + halo, c2 = (populations <= 30 ? 1.75 : 1.5) * (r2 + halo);
    return c1 <= c2 || two <= kSimds ? r1 : r2;
}
