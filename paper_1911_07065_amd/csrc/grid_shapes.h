// Which regions the multi-step grid kernels are launched with (internal):
// host arithmetic only, no device code.
#pragma once

#include <cstddef>
#include <utility>
#include <vector>

namespace ppg {

// Steps of one launch at most: they travel in the kernel's arguments
// (1.5 KB in FP64), and past 32 steps the launch itself is below 5 % of the time.
constexpr int kGrid2MaxSteps = 32;

constexpr int kGrid2MaxRows = 6;  // rows per wave of the largest built shape

// A 2-D grid stencil as far as a launch's shape depends on it: gx x gy points,
// 5 or 13 diagonals, one set of coefficients for all rows or not.
struct Grid2Form {
    int gx, gy, nd;
    bool constant;
    int rho() const { return nd == 13 ? 2 : 1; }
};

// How a launch is split: vx adjacent columns per lane and ry rows per wave,
// `waves` waves per workgroup: a region of 64 vx x waves ry points.
struct Grid2Shape {
    int vx = 0, ry = 0, waves = 0;
    int steps = 0;  // steps per launch
    int tz = 0;     // planes per chunk (3-D grids)
};

// The (vx, ry) pairs that are built for this stencil and precision (0: FP64, 1: FP32).
bool grid2_built(const Grid2Form &m, int prec, int vx, int ry);
// Tile sides and count of a launch of n steps; false when the region leaves no tile.
bool grid2_tiles(const Grid2Form &m, const Grid2Shape &s, int n, int *tx, int *ty, long *tiles);
// The shapes worth timing, each with its best number of steps, the most
// promising first by a model of one step's time fitted to a sweep of all
// shapes (50^2 to 1024^2; its four best always held one within 3 % of the
// fastest): 4.6 us a launch over its steps, then per wave of the fullest CU's
// SIMDs a fixed part and a part per point of a lane.
std::vector<Grid2Shape> grid2_shapes(const Grid2Form &m, int prec);

// Waves per workgroup of a batched launch at most (0: not built): two vectors
// of ry R values a lane, three with an accumulator, beside about 60 registers;
// 16 waves leave a lane 128, 8 waves 256.
constexpr int batch_grid_max_waves(size_t value_bytes, int R, int ry, bool acc) {
    const size_t regs = value_bytes / 4 * (size_t)(R * ry) * (acc ? 3 : 2);
    return regs <= 54 ? 16 : regs <= 96 ? 8 : 0;
}
bool batch_grid_ok(int prec, int R, int ry, int waves, int steps);
// Waves of the shape's launches with an accumulator.
int batch_grid_acc_waves(int prec, int R, int ry, int waves);
// Tile sides that a region of 64 x h points leaves exact on a gx x gy grid
// after `steps` steps; false when it leaves none.
bool batch_grid_tile(int gx, int gy, int h, int steps, int *tx, int *ty);
// The same for every grid (first: line length, second: lines), in the launches
// without and with an accumulator.
bool batch_grid_fits(int prec, int R, int ry, int waves, int steps, const std::vector<std::pair<int, int>> &grids);

// The batched kernel's shapes that fit the grids, each with its best number of
// steps, the most promising first by a model of one step: the launch's memory
// traffic (the regions read, the tiles written, at a copy's 4.5 TB/s) and 4 us
// over its steps, then the issue of the regions' operations (us in t).
struct BatchGridShape {
    double t;
    int ry, waves, steps;
};
std::vector<BatchGridShape> batch_grid_shapes(int prec, int R, const std::vector<std::pair<int, int>> &grids);

}  // namespace ppg
