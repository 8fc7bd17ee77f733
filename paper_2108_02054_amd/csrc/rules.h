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
// (w per entry) and L values are kept in LDS, within the 64 KiB that leave room for a second
// workgroup on the CU.
constexpr int OWN_SMEM_MAX = 65536;
constexpr int own_smem(int lanes, int w, int entries, int bytes) {
    return 2 * (256 / lanes) * entries * (w + 1) * bytes;
}
// Eight entries per group where they fit (121 to 128 FP64 columns, and more than 128, take four).
constexpr int own_entries(int lanes, int w, int bytes) {
    return w <= 128 && own_smem(lanes, w, 8, bytes) <= OWN_SMEM_MAX ? 8 : 4;
}

}  // namespace amgmi
