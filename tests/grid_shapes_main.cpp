// Checks of the multi-step kernels' shape lists (host arithmetic; run by
// test_grid_shapes.py).
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../paper_1911_07065_amd/csrc/grid_shapes.h"

using namespace ppg;

#define CHECK(c, ...)                    \
    do {                                 \
        if (!(c)) {                      \
            std::printf(__VA_ARGS__);    \
            std::printf(" [%s]\n", #c);  \
            std::exit(1);                \
        }                                \
    } while (0)

// Every shape offered for a batch leaves a tile on every system, in its
// launches without and with an accumulator.
static long batch_case(const std::vector<std::pair<int, int>> &grids) {
    long n = 0;
    for (int prec = 0; prec < 2; ++prec)
        for (int R : {1, 2, 4}) {
            double last = 0.0;
            for (const BatchGridShape &s : batch_grid_shapes(prec, R, grids)) {
                const int aw = batch_grid_acc_waves(prec, R, s.ry, s.waves);
                CHECK(batch_grid_ok(prec, R, s.ry, s.waves, s.steps) && aw >= 1 && aw <= s.waves, "prec %d R %d", prec, R);
                CHECK(s.t >= last, "order");
                last = s.t;
                for (const auto &g : grids)
                    for (int h : {s.ry * s.waves, s.ry * aw}) {
                        int tx, ty;
                        CHECK(batch_grid_tile(g.first, g.second, h, s.steps, &tx, &ty) && tx >= 1 && ty >= 1,
                              "prec %d R %d %d x %d: ry %d waves %d steps %d height %d", prec, R, g.first, g.second, s.ry,
                              s.waves, s.steps, h);
                    }
                ++n;
            }
        }
    return n;
}

// Every shape offered for a 2-D grid is built, leaves a tile and is offered once.
static long grid2_case(const Grid2Form &m) {
    long n = 0;
    for (int prec = 0; prec < 2; ++prec) {
        const std::vector<Grid2Shape> all = grid2_shapes(m, prec);
        for (size_t i = 0; i < all.size(); ++i) {
            int tx, ty;
            long tiles;
            CHECK(grid2_built(m, prec, all[i].vx, all[i].ry) && grid2_tiles(m, all[i], all[i].steps, &tx, &ty, &tiles),
                  "%d x %d", m.gx, m.gy);
            for (size_t k = 0; k < i; ++k)
                CHECK(all[i].vx != all[k].vx || all[i].ry != all[k].ry || all[i].waves != all[k].waves,
                      "%d x %d: shape %d x %d x %d twice", m.gx, m.gy, all[i].vx, all[i].ry, all[i].waves);
            ++n;
        }
    }
    return n;
}

int main() {
    long n = 0;
    for (int gy = 3; gy <= 130; ++gy)
        for (int gx : {3, 50, 64, 200, 1024})
            for (int form = 0; form < 3; ++form)
                if (form < 2 || (gx >= 5 && gy >= 5)) n += grid2_case(Grid2Form{gx, gy, form == 2 ? 13 : 5, form != 1});
    for (int count : {1, 8, 16, 32, 48, 96, 128, 256})
        for (int side = 3; side <= 260; ++side) n += batch_case({(size_t)count, {side, side}});
    std::mt19937 rng(5);
    for (int k = 0; k < 2000; ++k) {
        const int count = 4 + (int)(rng() % 45), lo = k % 2 ? 64 : 3, hi = lo + 16 + (int)(rng() % 180);
        std::vector<std::pair<int, int>> g;
        for (int i = 0; i < count; ++i) {
            const int gx = lo + (int)(rng() % (hi - lo + 1));
            g.emplace_back(gx, k % 3 ? gx : lo + (int)(rng() % (hi - lo + 1)));
        }
        n += batch_case(g);
    }
    std::printf("ok %ld\n", n);
    return 0;
}
