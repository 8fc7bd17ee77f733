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

}  // namespace amgmi
