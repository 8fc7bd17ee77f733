// rules.h -- index and size rules of the launches, in plain C++ (constexpr: the kernels and
// the host call the same functions, and a host compiler alone can check them).
#pragma once

namespace amgmi {

// Row of a thread when `lanes` neighbouring threads of a workgroup (a power of two that
// divides it) share one.  Taken block by block: the thread's number in the whole grid leaves
// 32 bits from 2^31 / lanes rows on, which a 7-point operator of less than 2^31 entries
// reaches with 8 lanes (2^28 rows, 1.9e9 entries).
constexpr int lane_row(int block, int threads, int thread, int lanes) {
    return block * (threads / lanes) + thread / lanes;
}

// Whether `rows` rows of `lanes` threads each fit one launch (its threads are counted in 32
// bits; one workgroup is left for the last, partly filled one).
constexpr bool lanes_fit_grid(long long rows, int lanes) { return rows * lanes <= (1ll << 32) - 1024; }

// Owner form of a Galerkin product with a workgroup of 256 threads per row of at most w columns:
// its 256 / lanes groups take `entries` L entries each per chunk, and two chunks of products
// (w per entry) and L values are kept in LDS, within half of the CU's 160 KiB so that a second
// workgroup has room.
constexpr int OWN_SMEM_MAX = 81920;
constexpr int own_smem(int lanes, int w, int entries, int bytes) {
    return 2 * (256 / lanes) * entries * (w + 1) * bytes;
}
// Eight entries per group (FP64 rows of 121 to 128 columns: 66048 bytes; four there took 18.6 us
// per product against 16.3), four for rows of more than 128 columns.
constexpr int own_entries(int w) { return w <= 128 ? 8 : 4; }

// Windowed kernels, symmetric values: whether half of the diagonals are read, twice each, the
// mirrored time at an odd offset.  Where all of them fit in the L2s (8 x 4 MB) the full read,
// bit for bit the same sums, is faster: 27-point Krylov SpMV 7.5 against 8.5 us at 44^3 and 9.6
// against 9.2 at 52^3 (30 MB); update and solve 1.29 against 1.31 ms at 44^3, with an FP32
// hierarchy 1.70 against 1.73 at 56^3 and 1.97 against 1.96 at 64^3 (28 MB).
constexpr long long WIN_FULL_BYTES = 28 << 20;
constexpr bool window_reads_half(int rows, int ndiag, int bytes) {
    return (long long)rows * ndiag * bytes > WIN_FULL_BYTES;
}

}  // namespace amgmi
