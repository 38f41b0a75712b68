// Regions of the multi-step grid kernels (see grid_shapes.h).
#include "grid_shapes.h"

#include <algorithm>

namespace ppg {

bool grid2_built(const Grid2Form &m, int prec, int vx, int ry) {
    if ((prec != 0 && prec != 1) || !(m.nd == 5 || (m.nd == 13 && m.constant))) return false;
    if (vx * ry > 4 && !m.constant) return false;
    return (vx == 1 && (ry == 2 || ry == 3 || ry == 4 || ry == 6)) || (vx == 2 && (ry == 2 || ry == 3 || ry == 4));
}

bool grid2_tiles(const Grid2Form &m, const Grid2Shape &s, int n, int *tx, int *ty, long *tiles) {
    if (s.vx < 1 || s.ry < 1 || s.waves < 1 || s.waves > 16 || m.gx < 2 || m.gy < 1) return false;
    const int w = 64 * s.vx, h = s.waves * s.ry, halo = 2 * m.rho() * n;
    *tx = m.gx <= w ? m.gx : w - halo;
    *ty = m.gy <= h ? m.gy : h - halo;
    if (*tx < 1 || *ty < 1) return false;
    *tiles = (long)((m.gx + *tx - 1) / *tx) * ((m.gy + *ty - 1) / *ty);
    return true;
}

std::vector<Grid2Shape> grid2_shapes(const Grid2Form &m, int prec) {
    std::vector<std::pair<double, Grid2Shape>> all;
    const double fixed = m.nd == 13 ? 0.1 : 0.0, wave = prec == 0 ? 0.05 : 0.025;
    const double point = m.nd == 13 ? (prec == 0 ? 0.045 : 0.036) : (prec == 0 ? 0.024 : 0.017);
    for (int vx = 1; vx <= 2; ++vx)
        for (int ry = 1; ry <= kGrid2MaxRows; ++ry) {
            if (!grid2_built(m, prec, vx, ry)) continue;
            const int whole = (m.gy + ry - 1) / ry;  // waves that span the grid's rows
            for (int waves : {4, 8, 16, whole}) {
                if (waves > 16 || whole < waves) continue;
                if (waves == whole && !all.empty() && all.back().second.vx == vx && all.back().second.ry == ry &&
                    all.back().second.waves == whole)
                    continue;  // listed as one of the fixed counts
                Grid2Shape s, best;
                s.vx = vx;
                s.ry = ry;
                s.waves = waves;
                double bt = 1e30;
                for (int n = 2; n <= kGrid2MaxSteps; ++n) {
                    int tx, ty;
                    long tiles;
                    if (!grid2_tiles(m, s, n, &tx, &ty, &tiles)) break;
                    const double per_simd = (double)((tiles + 255) / 256) * std::max(1.0, waves / 4.0);
                    const double t = 4.6 / n + fixed + per_simd * (wave + point * ry * vx);
                    if (t < bt) {
                        bt = t;
                        best = s;
                        best.steps = n;
                    }
                }
                if (best.steps > 0) all.emplace_back(bt, best);
            }
        }
    std::stable_sort(all.begin(), all.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    std::vector<Grid2Shape> out;
    for (const auto &a : all) out.push_back(a.second);
    return out;
}

bool batch_grid_ok(int prec, int R, int ry, int waves, int steps) {
    const size_t vb = prec == 0 ? 8 : 4;
    return (prec == 0 || prec == 1) && (R == 1 || R == 2 || R == 4) && (ry == 2 || ry == 3 || ry == 4 || ry == 6) &&
           waves >= 1 && waves <= batch_grid_max_waves(vb, R, ry, false) && batch_grid_max_waves(vb, R, ry, true) > 0 &&
           steps >= 2 && steps <= kGrid2MaxSteps && 64 - 2 * steps >= 1;
}

int batch_grid_acc_waves(int prec, int R, int ry, int waves) {
    return std::min(waves, batch_grid_max_waves(prec == 0 ? 8 : 4, R, ry, true));
}

bool batch_grid_tile(int gx, int gy, int h, int steps, int *tx, int *ty) {
    *tx = gx <= 64 ? gx : 64 - 2 * steps;
    *ty = gy <= h ? gy : h - 2 * steps;
    return *tx >= 1 && *ty >= 1;
}

bool batch_grid_fits(int prec, int R, int ry, int waves, int steps, const std::vector<std::pair<int, int>> &grids) {
    // the accumulator's region is the lower one
    const int h = ry * batch_grid_acc_waves(prec, R, ry, waves);
    int tx, ty;
    for (const auto &g : grids)
        if (!batch_grid_tile(g.first, g.second, h, steps, &tx, &ty)) return false;
    return true;
}

std::vector<BatchGridShape> batch_grid_shapes(int prec, int R, const std::vector<std::pair<int, int>> &grids) {
    std::vector<BatchGridShape> all;
    const double vb = prec == 0 ? 8.0 : 4.0, ops = prec == 0 ? 12.0 : 8.0;
    for (int ry : {2, 3, 4, 6})
        for (int waves : {4, 8, 16}) {
            BatchGridShape best{1e30, ry, waves, 0};
            for (int n = 2; batch_grid_ok(prec, R, ry, waves, n) && batch_grid_fits(prec, R, ry, waves, n, grids); ++n) {
                double tiles = 0, pts = 0;
                for (const auto &[gx, gy] : grids) {
                    int tx, ty;
                    batch_grid_tile(gx, gy, ry * waves, n, &tx, &ty);
                    tiles += (double)((gx + tx - 1) / tx) * ((gy + ty - 1) / ty);
                    pts += (double)gx * gy;
                }
                const double region = 64.0 * ry * waves * R;
                const double mem = (tiles * region + pts * R) * vb / 4.5e6;
                const double issue = std::max(tiles / 256.0, 1.0) * (region / 64.0) * ops * 4.0 / 4.0 / 2400.0;
                const double t = (4.0 + mem) / n + 0.12 + issue;
                if (t < best.t) best = BatchGridShape{t, ry, waves, n};
            }
            if (best.steps > 0) all.push_back(best);
        }
    std::stable_sort(all.begin(), all.end(),
                     [](const BatchGridShape &a, const BatchGridShape &b) { return a.t < b.t; });
    return all;
}

}  // namespace ppg
