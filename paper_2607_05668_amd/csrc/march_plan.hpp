// Host arithmetic of the marching kernels' launches (march.hpp): strips,
// segments, the limits of a lane's addresses, and where a march pays.  Plain
// C++.
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

// ------------------------------------------------- where a march pays ----
// A march moves a state through memory once for its steps, and pays with lanes
// and rows that are computed and not stored: all of it where the grid is a few
// columns wide, much of it where the segments are a few rows long.  Its time
// against that of the single step decides.  Both are fitted to 60 grids from
// 64^2 to 2048^2, 1 x 200000 and 300000 x 5 in 47 states (2035 pairs; the march
// to 13%, the single step mostly to 15%).  Against the single step, two launches
// of a hundred end up slower, by at most 19%, on grids a few rows high; by a
// rule on rows alone a march was up to 22 times slower (200000 rows of one
// cell) and 1.2-1.4 times for binary16 at 512^2.  A moment history costs both
// about the same (1443 pairs) and decides nothing.  us per step, one step a
// launch / march: shallow water D2Q9 float 512^2 9.6 / 7.0, 200000 x 1
// 8.9 / 120; binary16 512^2 6.3 / 8.4, 2048^2 77.8 / 50.1.
struct StepState {
    int storage;                    // 0 double, 1 float, 2 binary16, 3 binary16 deviations
    int fields, velocities;
    bool two_rates;                 // two-relaxation-time collision
    bool sources;                   // coefficient or source fields are read
};
// us: a launch, a population's row (loads and stores) and stage of a wavefront
// that has its SIMD to itself, and the least time of a single step per population
struct StepCosts { double launch, row, stage, least; };
constexpr StepCosts kStepCosts[4] = {{2.0, 0.073, 0.054, 0.14}, {2.5, 0.042, 0.0146, 0.055}, {3.0, 0.024, 0.0282, 0.07},
                                     {2.3, 0.027, 0.029, 0.11}};
constexpr int kStepBytes[4] = {8, 4, 2, 2};

// bytes of both buffers through the last-level cache where they fit, or HBM
inline double memory_us(double bytes) { return bytes / (bytes < 268e6 ? 6.9e6 : 6.0e6); }

inline double state_bytes(const StepState &s, int nx, int ny)
{
    const double moments = s.storage == 3 ? 8.0 * s.fields : 0.0;
    return (2.0 * s.fields * s.velocities * kStepBytes[s.storage] + moments) * nx * ny;
}

inline double single_step_us(const StepState &s, int nx, int ny)
{
    const int n = s.fields * s.velocities;
    const double bytes = state_bytes(s, nx, ny), least = 2.0 + kStepCosts[s.storage].least * n;
    if (s.storage == 3) {           // tiles of 64 x 4 cells, partly empty on narrow grids
        const double tiles = (double)((nx - 1) / 64 + 1) * ((ny - 1) / 4 + 1);
        return 1.12 * std::max(least, 2.0 + std::max(bytes / (bytes < 268e6 ? 5.0e6 : 4.5e6), 256 * tiles * n * 0.65e-6));
    }
    return std::max(least, 1.7 + memory_us(bytes) + 0.35 * (least - 1.7));
}

// per step, of a march of T steps that loses `halo` rows and lanes at each end
inline double march_us(const StepState &s, int T, int halo, int lds, int nx, int ny)
{
    const int n = s.fields * s.velocities, rows = march_rows(halo, lds, n, nx, ny);
    const int two = std::min(2 * kSimds, kSimds / 4 * (kLdsPerCu / lds));
    const long long waves = (long long)march_strips(halo, nx) * march_segments(ny, rows);
    // a second wavefront on the SIMDs, and rounds of wavefronts beyond that
    const double share = (waves <= kSimds + kSimds / 20 ? 1.0 : 1.4) * (double)((waves - 1) / two + 1);
    const StepCosts &c = kStepCosts[s.storage];
    double work = n * (c.row * (rows + 2 * halo) + c.stage * T * (rows + halo));
    // kernels that read fields, and those of two rates (they read them too); fitted
    // to 608 grids and states each.  us per step, one step a launch / two in a
    // march: advection-diffusion D2Q9 600 x 512 with two rates in double 21.8 / 19.4
    if (s.two_rates) work *= s.storage == 1 ? 1.3 : 1.0;
    else if (s.sources) work *= s.storage < 2 ? 1.2 : 1.1;
    return (c.launch + std::max(share * work, memory_us(state_bytes(s, nx, ny)))) / T;
}

// Steps of the next launch when `want` of a run's `run` steps are left: `most`
// (LDS lds_most) or two (LDS lds_two) in a march, or one; launches of one step
// come last.  Strips less than half full never pay against the 64-cell tiles of
// the single step by much.  A run of three as two and one has to gain more: a
// march and a single step next to each other find what the other left in the L2
// of other XCDs (us per step of runs of three, double 512^2, single steps / with
// a march of two: neo-Hookean D2Q5 20.6 / 25.0, Euler D2Q9 24.1 / 28.7).
// halo(T): rows lost.
template <class Halo>
int march_steps(const StepState &s, int most, int lds_most, int lds_two, Halo &&halo, int want, int run, int nx, int ny)
{
    if (want < 2 || most < 2 || nx < 32 || !march_fits(nx, ny, s.fields * s.velocities, kStepBytes[s.storage])) return 1;
    const double single = 0.97 * single_step_us(s, nx, ny), gain = run == 3 ? 0.55 : (most > 2 ? 0.9 : 1.0);
    const bool two = march_us(s, 2, halo(2), lds_two, nx, ny) <= gain * single;
    if (most > 2 && want >= most && !(most == 3 && want == 4 && two) && march_us(s, most, halo(most), lds_most, nx, ny) <= single)
        return most;
    return two ? 2 : 1;
}
