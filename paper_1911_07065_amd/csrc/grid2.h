// Several chain steps per launch on matrices whose rows are the points of a
// 2-D grid (internal): the launcher of the single-matrix kernel and the step
// form that it shares with the batched one.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "grid_shapes.h"

namespace ppg {

// One step of a chain on the vector S the chain is at:
//   w = a0 (A S) + a1 S [+ a2 (the vector before S)]   (kG2Aux: a conjugate
//   pair's second step);  acc += b0 S + b1 w (in launches with an accumulator).
// kG2Unit: a1 = 1 and no aux (a real root).
enum : int { kG2Aux = 1, kG2Unit = 2 };
template <typename AT>
struct Grid2Step {
    AT a0, a1, a2, b0, b1;
    int flags;
};

// The matrix as the kernel reads it: rows are the points x + gx y of a gx x
// gy grid, nd = 5 or 13 diagonals (the stencils of Grid2), no stored entry
// joins grid lines' ends. coef64/32: every row is these nd coefficients
// truncated at the grid (null: per-row values from the diagonal format,
// nd == 5 only).
struct Grid2Mat {
    int gx = 0, gy = 0, nd = 0;
    const double *coef64 = nullptr;
    const float *coef32 = nullptr;
    const double *dval64 = nullptr;
    const float *dval32 = nullptr;
    bool constant() const { return coef64 != nullptr; }
    int rho() const { return form().rho(); }
    Grid2Form form() const { return Grid2Form{gx, gy, nd, constant()}; }
};

// The shape is built for this matrix and precision (0: FP64, 1: FP32).
inline bool grid2_built(const Grid2Mat &m, int prec, int vx, int ry) {
    return (m.constant() || m.dval64) && grid2_built(m.form(), prec, vx, ry);
}

struct Grid2Ptrs {
    const void *in;
    void *out;         // null: the last vector is not stored
    void *acc;         // null: none
    int load_acc;      // 0: the accumulator starts at zero
    const void *vfin;  // out = vfin - w (null: out = w); not beside acc
    const Grid2Step<double> *steps;
    int n;
};
// One launch of p.n steps (<= kGrid2MaxSteps). out and acc must not alias in.
hipError_t launch_chain_grid2(const Grid2Mat &m, int prec, const Grid2Shape &s, const Grid2Ptrs &p, int remap,
                              hipStream_t st);

}  // namespace ppg
