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
