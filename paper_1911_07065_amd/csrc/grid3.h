// Several chain steps per launch on constant-coefficient 7-point stencils of
// a 3-D grid of any sides (internal).
#pragma once

#include "grid2.h"

namespace ppg {

constexpr int kGrid3MaxSteps = 3;

// Rows are the points x + gx (y + gy z); coef: the interior row's seven
// coefficients, truncated at the grid's faces.
struct Grid3Mat {
    int gx = 0, gy = 0, gz = 0;
    const double *coef64 = nullptr;
    const float *coef32 = nullptr;
};

// Launches read a Grid2Shape: vx columns a lane, ry rows a wave, `waves`
// waves a workgroup (at most grid3_max_waves), `steps` steps at most (2 or 3).
int grid3_max_waves(int prec, int vx, int ry);
bool grid3_built(const Grid3Mat &m, int prec, const Grid2Shape &s);
// Sets the planes of a chunk (tz) for s.steps steps; false when the region
// leaves no tile.
bool grid3_fit(const Grid3Mat &m, Grid2Shape &s);
// Tile sides of a launch of n steps (chunks of s.tz planes) and their count;
// false when the region leaves no tile.
bool grid3_tiles(const Grid3Mat &m, const Grid2Shape &s, int n, int *tx, int *ty, long *tiles);

// One launch of p.n steps (2 <= p.n <= kGrid3MaxSteps), the first of them
// without an aux vector. out and acc must not alias in.
hipError_t launch_chain_grid3(const Grid3Mat &m, int prec, const Grid2Shape &s, const Grid2Ptrs &p, int remap,
                              hipStream_t st);

}  // namespace ppg
