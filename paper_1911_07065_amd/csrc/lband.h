// Sparse products whose gathers hit LDS (internal): the copy's build on the
// GPU and the product kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace ppg {

// Columns in nb bands of W; a band of the input fits in LDS (kLbBytes), so a
// workgroup that holds it gathers there instead of in L2. Rows in windows of
// kLbRows; within a window and band the rows are sorted by their number of
// entries (most first, then by index) and cut into slices of 64, one row a
// lane, whose entries are stored two by two: slice q = (band nwin + window) 8
// + s owns pairs sptr[q] .. sptr[q + 1], pair k of lane l at (k 64 + l): two
// 16-bit columns (relative to the band) in one word of col and two values.
// perm[q 64 + l] = entries << 9 | row in the window (rows past the last one
// have no entries).
constexpr int kLbRows = 512;
constexpr int kLbBytes = 128 * 1024;  // 160 KB: no fewer launches, a longer copy (11.6 -> 11.9 us)
constexpr int kLbMaxBands = 8;    // partial sums a row: more would cost what the gathers save
constexpr int kLbMaxEntries = 127;  // of one row in one band
constexpr int kLbAhead = 3;         // pairs past the copy's end that the product may read

struct LBand {
    int nb = 0, W = 0, nwin = 0;
    int32_t *sptr = nullptr;
    uint16_t *perm = nullptr;
    uint32_t *col = nullptr;
    void *val = nullptr;       // the precision's matrix values, two per pair
    int32_t *eperm = nullptr;  // CSR position of each value (-1: padding)
    void *part = nullptr;      // nb n partial sums
    long pairs = 0;            // slots of 64 lanes
};

// Bands for n rows and vectors of elem bytes (0: more than kLbMaxBands).
int lb_bands(int n, size_t elem, int *W);
// Step 1 of the build: sorts the windows' rows (perm) and leaves the slices'
// first pairs in sptr (their number in its last entry) and in *bad 1 if a
// row has more than kLbMaxEntries entries in a band.
hipError_t launch_lb_sort(int n, const int32_t *rowptr, const int32_t *colind, const LBand &b, int *bad,
                          hipStream_t st);
// Step 2: columns and entry positions (both cleared by the kernel).
hipError_t launch_lb_fill(int n, const int32_t *rowptr, const int32_t *colind, const LBand &b, hipStream_t st);
// The values from the CSR values (binary64 or rounded to binary32).
hipError_t launch_lb_values(const LBand &b, bool f64, const double *val, hipStream_t st);
// part[band n + row] = the row's sum over the band's entries (FP64 sums for
// prec 0, else FP32).
hipError_t launch_lb_product(const LBand &b, int prec, int n, const void *in, int remap, hipStream_t st);

}  // namespace ppg
