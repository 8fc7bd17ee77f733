// kernels_setup.hip -- AMG setup on the device (Algorithm 1, Section 2): strength of
// connection, aggregation by a distance-2 maximal independent set, smoothed prolongator,
// restriction R = P^T, Galerkin sparsity patterns, and the coarsest direct solver.
//
// The aggregation decisions are integer results driven by floating-point comparisons;
// they are made with separately rounded products (contraction off) in the same
// association as the definitions below, so that on the same input they are bit-exact
// and independent of scheduling.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/device/device_select.hpp>

#include "amg_internal.h"

#pragma clang fp contract(off)

namespace amgmi {

constexpr int TPB = 256;

static inline unsigned blocks_for(int64_t n) {
    int64_t b = (n + TPB - 1) / TPB;
    return (unsigned)(b > 0 ? b : 1);
}

// Lanes per row of the setup's row kernels: the power of two in [4, 32] at or below the
// mean row length (a row's entries are read side by side; with one thread per row they
// were read a row apart, 344 against 80 us for the strength pass of the 128^3 hierarchy).
#define AMG_ROW_LANES(A, ...)                                                               \
    do {                                                                                    \
        const double mean_ = (A).nrows > 0 ? (double)(A).nnz / (double)(A).nrows : 1.0;     \
        if (mean_ >= 32.0) { constexpr int G = 32; __VA_ARGS__; }                           \
        else if (mean_ >= 16.0) { constexpr int G = 16; __VA_ARGS__; }                      \
        else if (mean_ >= 6.0) { constexpr int G = 8; __VA_ARGS__; }                        \
        else { constexpr int G = 4; __VA_ARGS__; }                                          \
    } while (0)

// ------------------------------------------------------------------ input checks

// Rows: monotone pointers, sorted unique in-range columns, finite values and, for a
// square operator, a positive stored diagonal (diag_pos[i] = position of a_ii).  G lanes
// per row, so that a row's entries are read side by side.
template <int G>
__global__ __launch_bounds__(TPB) void k_validate(int n, int ncols, int64_t nnz, int need_diag,
                                                  const int* __restrict__ ptr, const int* __restrict__ col,
                                                  const double* __restrict__ val, int* __restrict__ diag_pos,
                                                  int* __restrict__ flags) {
    const int lane = threadIdx.x & (G - 1);
    const int i = lane_row(blockIdx.x, TPB, threadIdx.x, G);
    if (i == 0 && lane == 0 && (ptr[0] != 0 || (int64_t)ptr[n] != nnz)) atomicOr(&flags[F_ARG], 1);
    if (i >= n) return;
    const int b = ptr[i], e = ptr[i + 1];
    if (b > e || b < 0 || (int64_t)e > nnz) {
        if (lane == 0) {
            atomicOr(&flags[F_ARG], 1);
            if (need_diag) diag_pos[i] = -1;
        }
        return;
    }
    int d = -1;
    bool bad = false;
    for (int k = b + lane; k < e; k += G) {
        const int j = col[k];
        const int prev = k > b ? col[k - 1] : -1;
        if (j < 0 || j >= ncols || j <= prev) bad = true;
        if (val != nullptr && !isfinite(val[k])) bad = true;
        if (j == i) d = k;
    }
    if (bad) atomicOr(&flags[F_ARG], 1);
    if (!need_diag) return;
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) d = max(d, __shfl_xor(d, o, G));
    if (lane != 0) return;
    diag_pos[i] = d;
    if (d < 0 || (val != nullptr && !(val[d] > 0.0))) atomicOr(&flags[F_NOT_SPD], 1);
}

void launch_validate(const Csr& A, int32_t* diag_pos, int* flags, hipStream_t s) {
    const int need_diag = diag_pos != nullptr ? 1 : 0;
    AMG_ROW_LANES(A, (k_validate<G><<<blocks_for((int64_t)A.nrows * G), TPB, 0, s>>>(
                         A.nrows, A.ncols, A.nnz, need_diag, A.ptr, A.col, A.val, diag_pos, flags)));
    HIP_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ strength

// Entry k = (i,j), j != i, is strong when (a_ij * a_ji) > eps2 * |a_ii * a_jj|, with
// eps2 = eps * eps.  tpos[k] is the position of (j,i); a missing (j,i) means the pattern is
// not structurally symmetric.  A row without strong entries is isolated.
template <int G>
__global__ __launch_bounds__(TPB) void k_strength(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                                  const double* __restrict__ val, const int* __restrict__ diag_pos,
                                                  double eps2, uint8_t* __restrict__ strong, int* __restrict__ tpos,
                                                  uint8_t* __restrict__ isolated, int* __restrict__ flags) {
    const int lane = threadIdx.x & (G - 1);
    const int i = lane_row(xcd_block(), TPB, threadIdx.x, G);
    if (i >= n) return;
    const double aii = val[diag_pos[i]];
    int any = 0;
    const int e = ptr[i + 1];
    for (int k = ptr[i] + lane; k < e; k += G) {
        const int j = col[k];
        if (j == i) {
            strong[k] = 0;
            tpos[k] = k;
            continue;
        }
        int lo = ptr[j], hi = ptr[j + 1] - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (col[mid] < i)
                lo = mid + 1;
            else
                hi = mid;
        }
        if (hi < lo || col[lo] != i) {
            atomicOr(&flags[F_PATTERN], 1);
            strong[k] = 0;
            tpos[k] = k;
            continue;
        }
        tpos[k] = lo;
        const double ajj = val[diag_pos[j]];
        const double lhs = val[k] * val[lo];
        const double rhs = eps2 * fabs(aii * ajj);
        const bool s = lhs > rhs;
        strong[k] = s ? 1 : 0;
        any |= s ? 1 : 0;
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) any |= __shfl_xor(any, o, G);
    if (lane == 0) isolated[i] = any ? 0 : 1;
}

void launch_strength(const Csr& A, const int32_t* diag_pos, double eps2, uint8_t* strong, int32_t* tpos,
                     uint8_t* isolated, int* flags, hipStream_t s) {
    AMG_ROW_LANES(A, (k_strength<G><<<blocks_for((int64_t)A.nrows * G), TPB, 0, s>>>(
                         A.nrows, A.ptr, A.col, A.val, diag_pos, eps2, strong, tpos, isolated, flags)));
    HIP_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ MIS-2

// Priority of node i: the SplitMix64 finaliser (Steele, Lea, Flood 2014) of i, a
// bijection on 64-bit integers, so priorities never tie.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
    return z ^ (z >> 31);
}

enum : uint8_t { ST_UNDECIDED = 0, ST_ROOT = 1, ST_REMOVED = 2, ST_ISOLATED = 3 };

__global__ void k_mis_init(int n, const uint8_t* __restrict__ isolated, uint8_t* __restrict__ state,
                           uint64_t* __restrict__ m1, uint8_t* __restrict__ c1) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    state[i] = isolated[i] ? ST_ISOLATED : ST_UNDECIDED;
    m1[i] = 1;
    c1[i] = 0;
}

// The round's kernels take G lanes per row: one where rows are short (most rows of a round
// return at once; four lanes on 128^3 7-point rows 35 -> 58 us), and where they are long
// enough to be a serial chain of reads 8, or 32 on the small levels that leave the chip idle
// (27-point 72x61x50, rows of 27 and 64 entries: the rounds of both levels 767 -> 338 us).
template <int G>
__device__ __forceinline__ uint64_t group_max(uint64_t v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        const uint64_t w = (uint64_t)__shfl_xor((unsigned long long)v, o, G);
        v = w > v ? w : v;
    }
    return v;
}
template <typename F>
void with_round_lanes(const Csr& A, F f) {
    const double mean = A.nrows > 0 ? (double)A.nnz / (double)A.nrows : 1.0;
    if (mean < 12.0)
        f(std::integral_constant<int, 1>{});
    else if (A.nrows >= 65536)
        f(std::integral_constant<int, 8>{});
    else
        f(std::integral_constant<int, 32>{});
}
template <int G>
struct RowLanes {
    int i, lane;
    __device__ __forceinline__ RowLanes() {
        i = lane_row(xcd_block(), TPB, threadIdx.x, G);
        lane = threadIdx.x & (G - 1);
    }
};

// m1[i] = max priority of an undecided node among i and its strong neighbours (0: none, and
// then none in any later round either: the row is not read again, which leaves a few rounds'
// worth of work in six or seven).
template <int G>
__global__ __launch_bounds__(TPB) void k_mis_max1(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                           const uint8_t* __restrict__ strong, const uint8_t* __restrict__ state,
                           uint64_t* __restrict__ m1,
                           const int* __restrict__ go) {
    if (go != nullptr && *go == 0) return;
    const RowLanes<G> t;
    const int i = t.i;
    if (i >= n || m1[i] == 0) return;
    uint64_t m = state[i] == ST_UNDECIDED ? mix64((uint64_t)i) : 0;
    const int e = ptr[i + 1];
    for (int k = ptr[i] + t.lane; k < e; k += G) {
        if (!strong[k]) continue;
        const int j = col[k];
        if (state[j] == ST_UNDECIDED) {
            const uint64_t p = mix64((uint64_t)j);
            m = p > m ? p : m;
        }
    }
    m = group_max<G>(m);
    if (t.lane == 0) m1[i] = m;
}

// An undecided node whose priority is the largest among undecided nodes within strong
// distance 2 becomes a root.  (Repeating this round by round yields exactly the set a
// sequential greedy pass in decreasing priority order builds: every node of higher
// priority nearby has been decided before.)
template <int G>
__global__ __launch_bounds__(TPB) void k_mis_max2(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                           const uint8_t* __restrict__ strong, const uint64_t* __restrict__ m1,
                           uint8_t* __restrict__ state,
                           const int* __restrict__ go) {
    if (go != nullptr && *go == 0) return;
    const RowLanes<G> t;
    const int i = t.i;
    if (i >= n || state[i] != ST_UNDECIDED) return;
    uint64_t m = m1[i];
    const int e = ptr[i + 1];
    for (int k = ptr[i] + t.lane; k < e; k += G) {
        if (!strong[k]) continue;
        const uint64_t p = m1[col[k]];
        m = p > m ? p : m;
    }
    m = group_max<G>(m);
    if (t.lane == 0 && m == mix64((uint64_t)i)) state[i] = ST_ROOT;
}

// c1[i] = i is a root or has a strong root neighbour: a new root (a root outside c1, since a
// node next to an earlier one has been removed) marks itself and its neighbours; strength is
// symmetric, and no other root is near enough to write the same marks.
template <int G>
__global__ __launch_bounds__(TPB) void k_mis_cover1(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                             const uint8_t* __restrict__ strong, const uint8_t* __restrict__ state,
                             uint8_t* __restrict__ c1, const int* __restrict__ go) {
    if (go != nullptr && *go == 0) return;
    const RowLanes<G> t;
    const int i = t.i;
    if (i >= n || state[i] != ST_ROOT || c1[i]) return;  // (a group's lanes read before one writes)
    if (t.lane == 0) c1[i] = 1;
    const int e = ptr[i + 1];
    for (int k = ptr[i] + t.lane; k < e; k += G)
        if (strong[k]) c1[col[k]] = 1;
}

// Undecided nodes within strong distance 2 of a root are removed; any node still
// undecided raises the flag for another round.
template <int G>
__global__ __launch_bounds__(TPB) void k_mis_cover2(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                             const uint8_t* __restrict__ strong, const uint8_t* __restrict__ c1,
                             uint8_t* __restrict__ state, int* __restrict__ left,
                             const int* __restrict__ go) {
    if (go != nullptr && *go == 0) return;
    const RowLanes<G> t;
    const int i = t.i;
    if (i >= n || state[i] != ST_UNDECIDED) return;
    uint64_t c = c1[i];
    const int e = ptr[i + 1];
    for (int k = ptr[i] + t.lane; k < e && !c; k += G)
        if (strong[k] && c1[col[k]]) c = 1;
    c = group_max<G>(c);
    if (t.lane != 0) return;
    if (c)
        state[i] = ST_REMOVED;
    else
        left[0] = 1;
}

constexpr int MIS_BATCH = 8;

void run_mis2(const Csr& A, const uint8_t* strong, const uint8_t* isolated, uint8_t* state, hipStream_t s) {
    const int n = A.nrows;
    uint64_t* m1 = dnew<uint64_t>((size_t)n, s);
    uint8_t* c1 = dnew<uint8_t>((size_t)n, s);
    const unsigned nb = blocks_for(n);
    k_mis_init<<<nb, TPB, 0, s>>>(n, isolated, state, m1, c1);
    HIP_LAUNCH_CHECK();
    // Rounds are queued MIS_BATCH at a time and read back once: a round whose predecessor
    // left no undecided node returns at once (left[r]: round r left one), where reading the
    // flag back after every round left the device idle for each of about seven per level.
    int* left = dnew<int>(MIS_BATCH, s);
    int h_left = 0;
    for (int round = 0;; round += MIS_BATCH) {
        HIP_CHECK(hipMemsetAsync(left, 0, MIS_BATCH * sizeof(int), s));
        with_round_lanes(A, [&](auto L) {
            constexpr int G = decltype(L)::value;
            const unsigned nbg = blocks_for((int64_t)n * G);
            for (int r = 0; r < MIS_BATCH; ++r) {
                const int* go = r == 0 ? nullptr : left + r - 1;
                k_mis_max1<G><<<nbg, TPB, 0, s>>>(n, A.ptr, A.col, strong, state, m1, go);
                k_mis_max2<G><<<nbg, TPB, 0, s>>>(n, A.ptr, A.col, strong, m1, state, go);
                k_mis_cover1<G><<<nbg, TPB, 0, s>>>(n, A.ptr, A.col, strong, state, c1, go);
                k_mis_cover2<G><<<nbg, TPB, 0, s>>>(n, A.ptr, A.col, strong, c1, state, left + r, go);
            }
        });
        HIP_LAUNCH_CHECK();
        HIP_CHECK(hipMemcpyAsync(&h_left, left + MIS_BATCH - 1, sizeof(int), hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
        if (!h_left) break;
        if (round > 4096) throw Fail{AMG_ERR_HIP, "MIS-2 did not terminate"};
    }
    dfree(left, s);
    dfree(m1, s);
    dfree(c1, s);
}

// ------------------------------------------------------------------ aggregation

// Pass 1: roots and their strong neighbours take the root's id (roots are at least 3
// apart, so at most one root is adjacent).
template <int G>
__global__ __launch_bounds__(TPB) void k_agg_pass1(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                            const uint8_t* __restrict__ strong, const uint8_t* __restrict__ state,
                            const int* __restrict__ root_id, int* __restrict__ agg1) {
    const RowLanes<G> t;
    const int i = t.i;
    if (i >= n) return;
    uint64_t a = 0;  // id + 1
    if (state[i] == ST_ROOT) {
        a = (uint64_t)root_id[i] + 1;
    } else if (state[i] != ST_ISOLATED) {
        const int e = ptr[i + 1];
        for (int k = ptr[i] + t.lane; k < e; k += G)
            if (strong[k] && state[col[k]] == ST_ROOT) a = (uint64_t)root_id[col[k]] + 1;
    }
    a = group_max<G>(a);
    if (t.lane == 0) agg1[i] = (int)a - 1;
}

// Pass 2: a node left over joins the pass-1 aggregate of its strong neighbour j with the
// largest a_ij * a_ji (ties: the smaller aggregate id).
template <int G>
__global__ __launch_bounds__(TPB) void k_agg_pass2(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                                   const double* __restrict__ val, const uint8_t* __restrict__ strong,
                                                   const int* __restrict__ tpos, const uint8_t* __restrict__ state,
                                                   const int* __restrict__ agg1, int* __restrict__ agg,
                                                   int* __restrict__ flags) {
    const int lane = threadIdx.x & (G - 1);
    const int i = lane_row(xcd_block(), TPB, threadIdx.x, G);
    if (i >= n) return;
    const int a1 = agg1[i];
    if (a1 >= 0 || state[i] == ST_ISOLATED) {
        if (lane == 0) agg[i] = a1;
        return;
    }
    int best = -1;
    double best_w = 0.0;
    auto take = [&](int aj, double w) {
        if (aj >= 0 && (best < 0 || w > best_w || (w == best_w && aj < best))) {
            best = aj;
            best_w = w;
        }
    };
    const int e = ptr[i + 1];
    for (int k = ptr[i] + lane; k < e; k += G)
        if (strong[k]) take(agg1[col[k]], val[k] * val[tpos[k]]);
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        const int aj = __shfl_xor(best, o, G);
        const double w = __shfl_xor(best_w, o, G);
        take(aj, w);
    }
    if (lane != 0) return;
    if (best < 0) atomicOr(&flags[F_NOAGG], 1);
    agg[i] = best;
}

__global__ void k_is_root(int n, const uint8_t* __restrict__ state, int* __restrict__ r) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    if (i < n) r[i] = state[i] == ST_ROOT ? 1 : 0;
}

template <typename Tin, typename Tout>
static void scan_exclusive(const Tin* in, Tout* out, int64_t n, hipStream_t s) {
    size_t bytes = 0;
    HIP_CHECK(rocprim::exclusive_scan(nullptr, bytes, in, out, Tout(0), (size_t)n, rocprim::plus<Tout>(), s));
    void* tmp = dalloc(bytes, s);
    HIP_CHECK(rocprim::exclusive_scan(tmp, bytes, in, out, Tout(0), (size_t)n, rocprim::plus<Tout>(), s));
    dfree(tmp, s);
}

void exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, hipStream_t s) {
    scan_exclusive<int32_t, int32_t>(in, out, n, s);
}

void exclusive_scan_i64(const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
    scan_exclusive<int64_t, int64_t>(in, out, n, s);
}

int32_t run_aggregate(const Csr& A, const uint8_t* strong, const int32_t* tpos, const uint8_t* state, int32_t* agg,
                      int* flags, int* h_flags, hipStream_t s) {
    const int n = A.nrows;
    const unsigned nb = blocks_for(n);
    int* isr = dnew<int>((size_t)n + 1, s);
    int* id = dnew<int>((size_t)n + 1, s);
    int* agg1 = dnew<int>((size_t)n, s);
    k_is_root<<<nb, TPB, 0, s>>>(n, state, isr);
    HIP_LAUNCH_CHECK();
    HIP_CHECK(hipMemsetAsync(isr + n, 0, sizeof(int), s));
    scan_exclusive<int, int>(isr, id, n + 1, s);
    with_round_lanes(A, [&](auto L) {
        constexpr int G = decltype(L)::value;
        k_agg_pass1<G><<<blocks_for((int64_t)n * G), TPB, 0, s>>>(n, A.ptr, A.col, strong, state, id, agg1);
    });
    AMG_ROW_LANES(A, (k_agg_pass2<G><<<blocks_for((int64_t)n * G), TPB, 0, s>>>(n, A.ptr, A.col, A.val, strong, tpos,
                                                                              state, agg1, agg, flags)));
    HIP_LAUNCH_CHECK();
    int32_t nc = 0;
    HIP_CHECK(hipMemcpyAsync(&nc, id + n, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipMemcpyAsync(h_flags, flags, F_COUNT * sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    dfree(isr, s);
    dfree(id, s);
    dfree(agg1, s);
    if (h_flags[F_NOAGG]) throw Fail{AMG_ERR_PATTERN, "node left without an aggregate"};
    return nc;
}

// ------------------------------------------------------------------ block systems

// Node I owns rows I*B .. I*B+B-1.  Its rows must list the same columns, in groups of B
// consecutive columns starting at a multiple of B (full blocks); the node row then has
// one entry per group.  The input has passed k_validate, so every index is in range.
__global__ void k_node_count(int nn, int B, const int* __restrict__ ptr, const int* __restrict__ col,
                             int* __restrict__ cnt, int* __restrict__ flags) {
    const int I = xcd_block() * TPB + threadIdx.x;
    if (I >= nn) return;
    const int r0 = I * B;
    const int b0 = ptr[r0], len = ptr[r0 + 1] - b0;
    bool ok = len % B == 0;
    for (int c = 1; c < B && ok; ++c) {
        const int bc = ptr[r0 + c];
        if (ptr[r0 + c + 1] - bc != len) ok = false;
        for (int k = 0; k < len && ok; ++k)
            if (col[bc + k] != col[b0 + k]) ok = false;
    }
    for (int g = 0; g < len / B && ok; ++g) {
        const int c0 = col[b0 + g * B];
        if (c0 % B != 0) ok = false;
        for (int q = 1; q < B && ok; ++q)
            if (col[b0 + g * B + q] != c0 + q) ok = false;
    }
    if (!ok) atomicOr(&flags[F_BLOCK], 1);
    cnt[I] = ok ? len / B : 0;
}

// Entry (I, J) of the node matrix: the Frobenius norm of block (I, J), its squares summed
// over the block's rows in order and along each row in column order, then one square root.
__global__ void k_node_fill(int nn, int B, const int* __restrict__ ptr, const int* __restrict__ col,
                            const double* __restrict__ val, const int* __restrict__ Nptr, int* __restrict__ Ncol,
                            double* __restrict__ Nval) {
    const int I = xcd_block() * TPB + threadIdx.x;
    if (I >= nn) return;
    const int r0 = I * B;
    const int nb = Nptr[I], ng = Nptr[I + 1] - nb;
    for (int g = 0; g < ng; ++g) {
        Ncol[nb + g] = col[ptr[r0] + g * B] / B;
        if (val == nullptr) continue;  // the pattern only
        double ss = 0.0;
        for (int c = 0; c < B; ++c) {
            const double* v = val + ptr[r0 + c] + g * B;
            for (int q = 0; q < B; ++q) ss += v[q] * v[q];
        }
        Nval[nb + g] = sqrt(ss);
    }
}

// Unknown b of node I joins unknown b of the node's aggregate (none when the node is
// isolated); an entry of block (I, J) takes the strength flag of node entry (I, J).
__global__ void k_node_expand(int n, int B, const int* __restrict__ ptr, const int* __restrict__ Nptr,
                              const uint8_t* __restrict__ nstrong, const int* __restrict__ nagg,
                              uint8_t* __restrict__ strong, int* __restrict__ agg) {
    const int r = xcd_block() * TPB + threadIdx.x;
    if (r >= n) return;
    const int I = r / B;
    const int a = nagg[I];
    agg[r] = a >= 0 ? a * B + (r - I * B) : -1;
    const int b = ptr[r], nb = Nptr[I];
    for (int k = b; k < ptr[r + 1]; ++k) strong[k] = nstrong[nb + (k - b) / B];
}

void build_node_matrix(const Csr& A, int B, Csr& Nm, int* flags, int* h_flags, hipStream_t s) {
    if (B < 2 || A.nrows % B != 0) throw Fail{AMG_ERR_ARG, "block_size does not divide the row count"};
    const int nn = A.nrows / B;
    int* cnt = dnew<int>((size_t)nn + 1, s);
    k_node_count<<<blocks_for(nn), TPB, 0, s>>>(nn, B, A.ptr, A.col, cnt, flags);
    HIP_LAUNCH_CHECK();
    HIP_CHECK(hipMemsetAsync(cnt + nn, 0, sizeof(int), s));
    Nm.nrows = Nm.ncols = nn;
    Nm.ptr = dnew<int32_t>((size_t)nn + 1, s);
    scan_exclusive<int, int>(cnt, Nm.ptr, nn + 1, s);
    int32_t nnz = 0;
    HIP_CHECK(hipMemcpyAsync(&nnz, Nm.ptr + nn, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipMemcpyAsync(h_flags, flags, F_COUNT * sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    dfree(cnt, s);
    if (h_flags[F_BLOCK]) {
        dfree(Nm.ptr, s);
        Nm.ptr = nullptr;
        throw Fail{AMG_ERR_PATTERN, "block_size needs full blocks with the same columns in every row of a node"};
    }
    Nm.nnz = nnz;
    Nm.col = dnew<int32_t>((size_t)nnz, s);
    Nm.val = A.val != nullptr ? dnew<double>((size_t)nnz, s) : nullptr;
    k_node_fill<<<blocks_for(nn), TPB, 0, s>>>(nn, B, A.ptr, A.col, A.val, Nm.ptr, Nm.col, Nm.val);
    HIP_LAUNCH_CHECK();
}

void launch_node_expand(const Csr& A, int B, const Csr& Nm, const uint8_t* nstrong, const int32_t* nagg,
                        uint8_t* strong, int32_t* agg, hipStream_t s) {
    k_node_expand<<<blocks_for(A.nrows), TPB, 0, s>>>(A.nrows, B, A.ptr, Nm.ptr, nstrong, nagg, strong, agg);
    HIP_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ prolongator

// Filtered operator A_F (lumped): for a non-isolated row the diagonal is
// d_i = a_ii + sum of weak off-diagonal entries (column order), the strong entries are
// kept; an isolated row keeps a_ii only.  ratio_i = sum_j |aF_ij| / |d_i| (column order);
// rho = max_i ratio_i (exact, so order free) is accumulated on the IEEE bit pattern, which
// orders like the value for positive doubles.
// G lanes per row read the entries side by side; every lane then adds them all in column
// order, each passed round from the lane that read it.
template <int G>
__global__ __launch_bounds__(TPB) void k_filter(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                                const double* __restrict__ val, const uint8_t* __restrict__ strong,
                                                const int* __restrict__ diag_pos, const int* __restrict__ agg,
                                                double* __restrict__ dF, unsigned long long* __restrict__ rho_bits) {
    __shared__ unsigned long long sm[TPB / 64];
    const int lane = threadIdx.x & (G - 1);
    const int i = lane_row(xcd_block(), TPB, threadIdx.x, G);
    unsigned long long bits = 0;
    if (i < n) {
        const bool iso = agg[i] < 0;
        const int b = ptr[i], e = ptr[i + 1];
        // kind of an entry: 0 dropped, 1 weak, 2 strong, 3 diagonal
        auto kind = [&](int k) { return k >= e ? 0 : col[k] == i ? 3 : iso ? 0 : strong[k] ? 2 : 1; };
        double d = val[diag_pos[i]];
        const int k0 = b + lane, w0 = kind(k0);  // the row's first G entries, read once
        const double v0 = k0 < e ? val[k0] : 0.0;
        for (int c0 = b; c0 < e; c0 += G) {
            const int k = c0 + lane, w = c0 == b ? w0 : kind(k);
            const double v = c0 == b ? v0 : k < e ? val[k] : 0.0;
            for (int t = 0; t < min(G, e - c0); ++t) {
                const double vt = __shfl(v, t, G);
                if (__shfl(w, t, G) == 1) d += vt;
            }
        }
        double s = 0.0;
        for (int c0 = b; c0 < e; c0 += G) {
            const int k = c0 + lane, w = c0 == b ? w0 : kind(k);
            const double v = c0 == b ? v0 : k < e ? val[k] : 0.0;
            for (int t = 0; t < min(G, e - c0); ++t) {
                const double vt = __shfl(v, t, G);
                const int wt = __shfl(w, t, G);
                if (wt == 3)
                    s += fabs(d);
                else if (wt == 2)
                    s += fabs(vt);
            }
        }
        if (lane == 0) dF[i] = d;
        bits = (unsigned long long)__double_as_longlong(s / fabs(d));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long x = __shfl_xor(bits, o, 64);
        bits = x > bits ? x : bits;
    }
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = bits;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < TPB / 64; ++k) bits = sm[k] > bits ? sm[k] : bits;
        // (the cached read leaves the atomic to the few workgroups that raise the maximum)
        if (bits > __hip_atomic_load(rho_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) atomicMax(rho_bits, bits);
    }
}

// Aggregate of every entry's column among the entries A_F keeps (diagonal and strong), -1
// for the others; a row of an isolated node keeps none.
template <int G>
__global__ __launch_bounds__(TPB) void k_entry_agg(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                                   const uint8_t* __restrict__ strong, const int* __restrict__ agg,
                                                   int* __restrict__ eagg) {
    const int lane = threadIdx.x & (G - 1);
    const int i = lane_row(xcd_block(), TPB, threadIdx.x, G);
    if (i >= n) return;
    const bool iso = agg[i] < 0;
    const int e = ptr[i + 1];
    for (int k = ptr[i] + lane; k < e; k += G) {
        const int j = col[k];
        eagg[k] = !iso && (j == i || strong[k]) ? agg[j] : -1;
    }
}

// Rows of more than LONG_ROW entries per lane go through their aggregates one by one, in a pass
// over the row for each: comparing every entry with every earlier one, as short rows do, grows
// with the square of the length, while a long row (a hub: a node coupled to most others) meets
// few aggregates or, being isolated, none (a star of 8000 nodes: setup 2337 -> 18 ms).
constexpr int LONG_ROW = 16;

// The smallest v of the G lanes with its entry k, the earlier one where several lanes have it.
template <int G>
__device__ __forceinline__ void group_first(int& v, int& k) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        const int w = __shfl_xor(v, o, G), q = __shfl_xor(k, o, G);
        if (w < v || (w == v && q < k)) {
            v = w;
            k = q;
        }
    }
}
constexpr int NO_AGG = 0x7fffffff;

// Number of distinct aggregates among the columns of row i of A_F; that is the length of
// row i of A_F P_tent and of the smoothed P.  key[k] = 2 * aggregate + 1 for an aggregate's
// first entry, 2 * aggregate for its others, -1 for entries A_F drops.
template <int G>
__global__ __launch_bounds__(TPB) void k_pcount(int n, const int* __restrict__ ptr, const int* __restrict__ eagg,
                                                int* __restrict__ key, int* __restrict__ cnt) {
    const int lane = threadIdx.x & (G - 1);
    const int i = lane_row(xcd_block(), TPB, threadIdx.x, G);
    if (i >= n) return;
    const int b = ptr[i], e = ptr[i + 1];
    if (e - b > LONG_ROW * G) {
        for (int k = b + lane; k < e; k += G) key[k] = eagg[k] < 0 ? -1 : 2 * eagg[k];
        int c = 0;
        for (int last = -1;; ++c) {
            int J = NO_AGG, first = NO_AGG;
            for (int k = b + lane; k < e; k += G) {
                const int a = eagg[k];
                if (a > last && a < J) {
                    J = a;
                    first = k;
                }
            }
            group_first<G>(J, first);
            if (J == NO_AGG) break;
            if ((first - b) % G == lane) key[first] = 2 * J + 1;  // (by the lane that wrote it above)
            last = J;
        }
        if (lane == 0) cnt[i] = c;
        return;
    }
    int c = 0;
    for (int c0 = b; c0 < e; c0 += G) {
        const int k = c0 + lane;
        const int a = k < e ? eagg[k] : -1;
        bool f = a >= 0;
        for (int c1 = b; c1 <= c0; c1 += G) {  // against the entries before it
            const int aq = c1 == c0 ? a : eagg[c1 + lane];
            for (int t = 0; t < G; ++t) {
                const int at = __shfl(aq, t, G);  // (outside any condition: every lane passes its own on)
                f = f && !(at == a && c1 + t < k);
            }
        }
        if (k < e) key[k] = a < 0 ? -1 : 2 * a + (f ? 1 : 0);
        c += f ? 1 : 0;
    }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, G);
    if (lane == 0) cnt[i] = c;
}

// Row i of P = P_tent - (omega / d_i) * (A_F P_tent), omega = (4/3) / rho.  Columns are
// the distinct aggregates of the row in increasing order; for column J the sum over the
// row's entries with aggregate J is taken in column order starting from 0.  The lane of an
// aggregate's first entry forms its place (the smaller aggregates' first entries) and its
// sum from the row's entries passed round the group.
template <int G>
__global__ __launch_bounds__(TPB) void k_pfill(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                               const double* __restrict__ val, const int* __restrict__ agg,
                                               const int* __restrict__ key, const double* __restrict__ dF,
                                               const unsigned long long* __restrict__ rho_bits,
                                               const int* __restrict__ Pptr, int* __restrict__ Pcol,
                                               double* __restrict__ Pval) {
    const int lane = threadIdx.x & (G - 1);
    const int i = lane_row(xcd_block(), TPB, threadIdx.x, G);
    if (i >= n) return;
    const int ai = agg[i];
    if (ai < 0) return;
    const int p0 = Pptr[i];
    const double rho = __longlong_as_double((long long)*rho_bits);
    const double omega = (4.0 / 3.0) / rho;
    const double di = dF[i];
    const double scale = omega / di;
    const int b = ptr[i], e = ptr[i + 1];
    if (e - b > LONG_ROW * G) {
        const int shift = (threadIdx.x & 63) & ~(G - 1);
        const unsigned mask = G == 32 ? ~0u : (1u << G) - 1;
        int last = -1;
        for (int p = p0;; ++p) {
            int J = NO_AGG, first = NO_AGG;
            for (int k = b + lane; k < e; k += G) {
                const int kk = key[k];
                if (kk > 0 && (kk & 1) && (kk >> 1) > last && (kk >> 1) < J) {
                    J = kk >> 1;
                    first = k;
                }
            }
            group_first<G>(J, first);
            if (J == NO_AGG) break;
            double sJ = 0.0;  // of the entries from the first on, in order
            for (int c1 = first - (first - b) % G; c1 < e; c1 += G) {
                const int q = c1 + lane;
                const bool hit = q < e && key[q] >= 0 && (key[q] >> 1) == J;
                const double vq = hit ? (col[q] == i ? di : val[q]) : 0.0;
                for (unsigned m = (unsigned)(__ballot(hit) >> shift) & mask; m != 0; m &= m - 1)
                    sJ += __shfl(vq, __ffs(m) - 1, G);
            }
            if (lane == 0) {
                const double pt = (J == ai) ? 1.0 : 0.0;
                Pcol[p] = J;
                Pval[p] = pt - scale * sJ;
            }
            last = J;
        }
        return;
    }
    for (int c0 = b; c0 < e; c0 += G) {
        const int kk = c0 + lane < e ? key[c0 + lane] : -1;
        const bool mine = kk >= 0 && (kk & 1);
        const int J = kk >> 1;
        int r = 0;
        double sJ = 0.0;
        for (int c1 = b; c1 < e; c1 += G) {
            const int q = c1 + lane;
            const int kq = q < e ? key[q] : -1;
            const double vq = q < e ? (col[q] == i ? di : val[q]) : 0.0;
            for (int t = 0; t < min(G, e - c1); ++t) {
                const int kt = __shfl(kq, t, G);
                const double vt = __shfl(vq, t, G);
                if (kt >= 0 && (kt >> 1) == J) sJ += vt;
                r += kt >= 0 && (kt & 1) && (kt >> 1) < J ? 1 : 0;
            }
        }
        if (!mine) continue;
        const double pt = (J == ai) ? 1.0 : 0.0;
        Pcol[p0 + r] = J;
        Pval[p0 + r] = pt - scale * sJ;
    }
}

// Plain aggregation, P = P_tent: one unit entry per aggregated row.
__global__ __launch_bounds__(TPB) void k_plain_count(int n, const int* __restrict__ agg, int* __restrict__ cnt) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    if (i < n) cnt[i] = agg[i] < 0 ? 0 : 1;
}
__global__ __launch_bounds__(TPB) void k_plain_fill(int n, const int* __restrict__ agg, const int* __restrict__ Pptr,
                                                    int* __restrict__ Pcol, double* __restrict__ Pval) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    if (i >= n || agg[i] < 0) return;
    Pcol[Pptr[i]] = agg[i];
    Pval[Pptr[i]] = 1.0;
}

void build_prolongator(const Csr& A, const uint8_t* strong, const int32_t* diag_pos, const int32_t* agg, int32_t nc,
                       int plain, Csr& P, hipStream_t s) {
    const int n = A.nrows;
    const unsigned nb = blocks_for(n);
    double* dF = nullptr;
    unsigned long long* rho_bits = nullptr;
    int* eagg = nullptr;
    int* key = nullptr;
    int* cnt = dnew<int>((size_t)n + 1, s);
    if (plain) {
        k_plain_count<<<nb, TPB, 0, s>>>(n, agg, cnt);
    } else {
        dF = dnew<double>((size_t)n, s);
        rho_bits = dnew<unsigned long long>(1, s);
        eagg = dnew<int>((size_t)A.nnz, s);
        key = dnew<int>((size_t)A.nnz, s);
        HIP_CHECK(hipMemsetAsync(rho_bits, 0, sizeof(unsigned long long), s));
        AMG_ROW_LANES(A, (k_filter<G><<<blocks_for((int64_t)n * G), TPB, 0, s>>>(n, A.ptr, A.col, A.val, strong, diag_pos,
                                                                               agg, dF, rho_bits)));
        AMG_ROW_LANES(A, (k_entry_agg<G><<<blocks_for((int64_t)n * G), TPB, 0, s>>>(n, A.ptr, A.col, strong, agg, eagg)));
        AMG_ROW_LANES(A, (k_pcount<G><<<blocks_for((int64_t)n * G), TPB, 0, s>>>(n, A.ptr, eagg, key, cnt)));
    }
    HIP_LAUNCH_CHECK();
    HIP_CHECK(hipMemsetAsync(cnt + n, 0, sizeof(int), s));
    P.nrows = n;
    P.ncols = nc;
    P.ptr = dnew<int32_t>((size_t)n + 1, s);
    scan_exclusive<int, int>(cnt, P.ptr, n + 1, s);
    int32_t nnz = 0;
    HIP_CHECK(hipMemcpyAsync(&nnz, P.ptr + n, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    P.nnz = nnz;
    P.col = dnew<int32_t>((size_t)nnz, s);
    P.val = dnew<double>((size_t)nnz, s);
    if (plain)
        k_plain_fill<<<nb, TPB, 0, s>>>(n, agg, P.ptr, P.col, P.val);
    else
        AMG_ROW_LANES(A, (k_pfill<G><<<blocks_for((int64_t)n * G), TPB, 0, s>>>(
                             n, A.ptr, A.col, A.val, agg, key, dF, rho_bits, P.ptr, P.col, P.val)));
    HIP_LAUNCH_CHECK();
    dfree(cnt, s);
    for (void* q : {(void*)dF, (void*)rho_bits, (void*)eagg, (void*)key})
        if (q) dfree(q, s);
}

// ------------------------------------------------------------------ sorting helpers

template <typename K, typename V>
static void radix_sort_pairs(K* kin, K* kout, V* vin, V* vout, int64_t n, int end_bit, hipStream_t s) {
    size_t bytes = 0;
    HIP_CHECK(rocprim::radix_sort_pairs(nullptr, bytes, kin, kout, vin, vout, (size_t)n, 0u, (unsigned)end_bit, s));
    void* tmp = dalloc(bytes, s);
    HIP_CHECK(rocprim::radix_sort_pairs(tmp, bytes, kin, kout, vin, vout, (size_t)n, 0u, (unsigned)end_bit, s));
    dfree(tmp, s);
}

template <typename K>
static void radix_sort_keys(K* kin, K* kout, int64_t n, int end_bit, hipStream_t s) {
    size_t bytes = 0;
    HIP_CHECK(rocprim::radix_sort_keys(nullptr, bytes, kin, kout, (size_t)n, 0u, (unsigned)end_bit, s));
    void* tmp = dalloc(bytes, s);
    HIP_CHECK(rocprim::radix_sort_keys(tmp, bytes, kin, kout, (size_t)n, 0u, (unsigned)end_bit, s));
    dfree(tmp, s);
}

static int bits_for(uint64_t v) {
    int b = 1;
    while (b < 64 && (v >> b) != 0) ++b;
    return b;
}

// ptr[r] = number of keys (sorted, row-major key = r * ncols + c) with row < r.
__global__ void k_rowptr_from_keys(int nrows, int64_t nkeys, const uint64_t* __restrict__ keys, uint64_t ncols,
                                   int* __restrict__ ptr) {
    const int r = blockIdx.x * TPB + threadIdx.x;
    if (r > nrows) return;
    const uint64_t target = (uint64_t)r * ncols;
    int64_t lo = 0, hi = nkeys;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < target)
            lo = mid + 1;
        else
            hi = mid;
    }
    ptr[r] = (int)lo;
}

__global__ void k_cols_from_keys(int64_t nkeys, const uint64_t* __restrict__ keys, uint64_t ncols,
                                 int* __restrict__ col) {
    for (int64_t k = blockIdx.x * (int64_t)TPB + threadIdx.x; k < nkeys; k += (int64_t)gridDim.x * TPB)
        col[k] = (int)(keys[k] % ncols);
}

// ------------------------------------------------------------------ transpose

__global__ void k_transpose_keys(int n, const int* __restrict__ ptr, const int* __restrict__ col, uint64_t nrows,
                                 uint64_t* __restrict__ keys, int* __restrict__ idx) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    for (int k = ptr[i]; k < ptr[i + 1]; ++k) {
        keys[k] = (uint64_t)col[k] * nrows + (uint64_t)i;
        idx[k] = k;
    }
}

__global__ void k_gather_vals(int64_t nnz, const int* __restrict__ idx, const double* __restrict__ v,
                              double* __restrict__ out) {
    for (int64_t k = blockIdx.x * (int64_t)TPB + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * TPB)
        out[k] = v[idx[k]];
}

static unsigned gs_blocks(int64_t n) {
    int64_t b = (n + TPB - 1) / TPB;
    if (b > 16384) b = 16384;
    return (unsigned)(b > 0 ? b : 1);
}

// R = P^T (its arrays allocated) by sorting the entries by (column, row).
void transpose_sorted(const Csr& P, Csr& R, hipStream_t s) {
    const int64_t nnz = P.nnz;
    uint64_t* k0 = dnew<uint64_t>((size_t)nnz, s);
    uint64_t* k1 = dnew<uint64_t>((size_t)nnz, s);
    int* i0 = dnew<int>((size_t)nnz, s);
    int* i1 = dnew<int>((size_t)nnz, s);
    k_transpose_keys<<<blocks_for(P.nrows), TPB, 0, s>>>(P.nrows, P.ptr, P.col, (uint64_t)P.nrows, k0, i0);
    HIP_LAUNCH_CHECK();
    const int eb = bits_for((uint64_t)P.ncols * (uint64_t)P.nrows);
    if (nnz > 0) radix_sort_pairs<uint64_t, int>(k0, k1, i0, i1, nnz, eb, s);
    k_rowptr_from_keys<<<blocks_for(R.nrows + 1), TPB, 0, s>>>(R.nrows, nnz, k1, (uint64_t)P.nrows, R.ptr);
    k_cols_from_keys<<<gs_blocks(nnz), TPB, 0, s>>>(nnz, k1, (uint64_t)P.nrows, R.col);
    k_gather_vals<<<gs_blocks(nnz), TPB, 0, s>>>(nnz, i1, P.val, R.val);
    HIP_LAUNCH_CHECK();
    dfree(k0, s);
    dfree(k1, s);
    dfree(i0, s);
    dfree(i1, s);
}

// ------------------------------------------------------------------ symbolic product

// Upper bound of the length of row i of A B (sum of the B row lengths it references).
__global__ void k_spgemm_ub(int n, const int* __restrict__ Aptr, const int* __restrict__ Acol,
                            const int* __restrict__ Bptr, int64_t* __restrict__ ub) {
    const int i = xcd_block() * TPB + threadIdx.x;
    if (i > n) return;
    if (i == n) {
        ub[n] = 0;
        return;
    }
    int64_t c = 0;
    for (int k = Aptr[i]; k < Aptr[i + 1]; ++k) {
        const int j = Acol[k];
        c += Bptr[j + 1] - Bptr[j];
    }
    ub[i] = c;
}

__global__ void k_spgemm_expand(int n, const int* __restrict__ Aptr, const int* __restrict__ Acol,
                                const int* __restrict__ Bptr, const int* __restrict__ Bcol,
                                const int64_t* __restrict__ off, uint64_t ncols, uint64_t* __restrict__ keys) {
    const int i = xcd_block() * TPB + threadIdx.x;
    if (i >= n) return;
    int64_t pos = off[i];
    const uint64_t base = (uint64_t)i * ncols;
    for (int k = Aptr[i]; k < Aptr[i + 1]; ++k) {
        const int j = Acol[k];
        for (int q = Bptr[j]; q < Bptr[j + 1]; ++q) keys[pos++] = base + (uint64_t)Bcol[q];
    }
}

// Pattern of C = A B (structural: every product term creates its entry), sorted columns, for
// products with rows too long for symbolic_count's tables: expand all candidate (row,
// column) pairs, sort, and keep the unique ones.
void symbolic_sorted(const Csr& A, const Csr& B, Csr& C, hipStream_t s) {
    const int n = A.nrows;
    int64_t* ub = dnew<int64_t>((size_t)n + 1, s);
    int64_t* off = dnew<int64_t>((size_t)n + 1, s);
    k_spgemm_ub<<<blocks_for(n + 1), TPB, 0, s>>>(n, A.ptr, A.col, B.ptr, ub);
    HIP_LAUNCH_CHECK();
    scan_exclusive<int64_t, int64_t>(ub, off, n + 1, s);
    int64_t total = 0;
    HIP_CHECK(hipMemcpyAsync(&total, off + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    if (total >= ((int64_t)1 << 31)) throw Fail{AMG_ERR_ARG, "Galerkin product too large for int32 indexing"};
    C.nrows = n;
    C.ncols = B.ncols;
    C.ptr = dnew<int32_t>((size_t)n + 1, s);
    uint64_t* k0 = dnew<uint64_t>((size_t)total, s);
    uint64_t* k1 = dnew<uint64_t>((size_t)total, s);
    k_spgemm_expand<<<blocks_for(n), TPB, 0, s>>>(n, A.ptr, A.col, B.ptr, B.col, off, (uint64_t)B.ncols, k0);
    HIP_LAUNCH_CHECK();
    const int eb = bits_for((uint64_t)n * (uint64_t)B.ncols);
    if (total > 0) radix_sort_keys<uint64_t>(k0, k1, total, eb, s);
    // unique keys into k0
    int* nsel = dnew<int>(1, s);
    size_t bytes = 0;
    HIP_CHECK(rocprim::unique(nullptr, bytes, k1, k0, nsel, (size_t)total, rocprim::equal_to<uint64_t>(), s));
    void* tmp = dalloc(bytes, s);
    HIP_CHECK(rocprim::unique(tmp, bytes, k1, k0, nsel, (size_t)total, rocprim::equal_to<uint64_t>(), s));
    dfree(tmp, s);
    int nnz = 0;
    if (total > 0) {
        HIP_CHECK(hipMemcpyAsync(&nnz, nsel, sizeof(int), hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
    }
    C.nnz = nnz;
    C.col = dnew<int32_t>((size_t)nnz, s);
    k_rowptr_from_keys<<<blocks_for(n + 1), TPB, 0, s>>>(n, nnz, k0, (uint64_t)B.ncols, C.ptr);
    k_cols_from_keys<<<gs_blocks(nnz), TPB, 0, s>>>(nnz, k0, (uint64_t)B.ncols, C.col);
    HIP_LAUNCH_CHECK();
    dfree(nsel, s);
    dfree(k0, s);
    dfree(k1, s);
    dfree(ub, s);
    dfree(off, s);
}

// ------------------------------------------------------------------ coarsest level

template <typename T>
__global__ void k_densify(int n, const int* __restrict__ ptr, const int* __restrict__ col, const T* __restrict__ val,
                          double* __restrict__ D) {
    const int i = blockIdx.x;
    if (i >= n) return;
    for (int j = threadIdx.x; j < n; j += blockDim.x) D[(size_t)i * n + j] = 0.0;
    __syncthreads();
    for (int k = ptr[i] + threadIdx.x; k < ptr[i + 1]; k += blockDim.x) D[(size_t)i * n + col[k]] = (double)val[k];
}

template <typename T>
void launch_densify(const Csr& A, double* D, hipStream_t s) {
    k_densify<T><<<(unsigned)(A.nrows > 0 ? A.nrows : 1), 128, 0, s>>>(A.nrows, A.ptr, A.col, A.v<T>(), D);
    HIP_LAUNCH_CHECK();
}
template void launch_densify<double>(const Csr&, double*, hipStream_t);
template void launch_densify<float>(const Csr&, double*, hipStream_t);

// ------------------------------------------------------------------ dense inverse
//
// Inverse of the coarsest operator by Gauss-Jordan elimination without pivoting (the pivots
// are the positive LDL^T pivots of an SPD matrix; a non-positive or non-finite pivot reports
// "not SPD" in scal[S_COARSE]).  The elimination is one chain of n dependent pivots, so its
// latency bounds every form here: 16 pivots at a time are eliminated by one wavefront in
// registers (gj_inv16), everything else is 16 x 16 tile products on the FP64 matrix cores,
// and the next 16 x 16 (or 64 x 64) pivot block is inverted while the rest of the matrix is
// still being updated.
//   up to COARSE_LDS_MAX rows: one workgroup, the matrix in its LDS (k_dense_inverse);
//   above: 64 pivots per launch over the whole device (k_bgj_first, k_bgj_step).
// Measured: 112 rows 415 -> 37 us and 89 rows 215 -> 30 us against a pivot-by-pivot loop in
// LDS (two barriers and n^2 / 1024 dependent updates per pivot); 265 rows 137 -> 121 us and
// 559 rows 311 -> 260 us (beside a solve's first kernels) against two launches per 64 pivots
// (the pivot block inverted in one, the matrix updated in the other, neither beside the
// other).  Left: about 5 us per 16 pivots, 58 instructions per pivot in one wavefront.
typedef double bgj_v4 __attribute__((ext_vector_type(4)));
constexpr int GJ_XLD = 17;  // row stride of a 16 x 16 pivot-block inverse in LDS

// Value of v in lane `lane` (uniform) of the wavefront.
__device__ __forceinline__ double gj_lane(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), lane);
    const unsigned hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Value of v in lane P of this lane's row of 16 lanes (DPP row_newbcast: no LDS round trip).
template <int P>
__device__ __forceinline__ double gj_row_lane(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffff), 0x150 + P, 0xf, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + P, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Pivot P of gj_inv16 and the ones after it.
template <int P>
__device__ __forceinline__ void gj_pivots(double (&e)[4], int i, int q, bool& ok) {
    if constexpr (P < 16) {
        constexpr int QP = P / 4, RP = P % 4;
        const double piv = gj_lane(e[RP], 16 * QP + P);
        const double col = __shfl(e[RP], 16 * QP + i);  // e_iP, from the lanes that hold column P
        ok = ok && piv > 0.0 && isfinite(piv);
        const double pinv = 1.0 / piv;
        const double cf = col * pinv;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double pr = gj_row_lane<P>(e[j]);
            e[j] = i == P ? e[j] * pinv : fma(-cf, pr, e[j]);
        }
        if (q == QP) e[RP] = i == P ? pinv : -cf;
        gj_pivots<P + 1>(e, i, q, ok);
    }
}

// Inverse of the 16 x 16 tile at src (row stride ld) into X (row stride GJ_XLD), by one
// wavefront: lane l holds columns 4 (l / 16) .. + 3 of row l % 16, so that the pivot row
// reaches every lane within its own row of 16 lanes and a pivot costs one cross-row
// exchange (of the pivot column) instead of 15 broadcasts.
__device__ __forceinline__ void gj_inv16(const double* src, int ld, double* X, int* bad) {
    const int l = threadIdx.x % 64, i = l & 15, q = l >> 4;
    double e[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = src[i * ld + 4 * q + j];
    bool ok = true;
    gj_pivots<0>(e, i, q, ok);
#pragma unroll
    for (int j = 0; j < 4; ++j) X[i * GJ_XLD + 4 * q + j] = e[j];
    if (!ok && l == 0) *bad = 1;
}

// 16 x 16 tile product on the FP64 matrix cores: c + sign * (a b), a and b tiles in LDS with
// row strides lda and ldb, c and the result in the instruction's result layout (entry r of
// lane l is row l / 16 + 4 r, column l % 16).
__device__ __forceinline__ bgj_v4 gj_tile_mm(const double* a, int lda, const double* b, int ldb, bgj_v4 c,
                                             double sign) {
    const int l = threadIdx.x % 64, i = l & 15, kk = l >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(sign * a[i * lda + 4 * s + kk], b[(4 * s + kk) * ldb + i], c, 0, 0, 0);
    return c;
}

__device__ __forceinline__ bgj_v4 gj_tile_load(const double* t, int ld) {
    const int l = threadIdx.x % 64;
    bgj_v4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = t[((l >> 4) + 4 * r) * ld + (l & 15)];
    return v;
}

__device__ __forceinline__ void gj_tile_store(double* t, int ld, bgj_v4 v) {
    const int l = threadIdx.x % 64;
#pragma unroll
    for (int r = 0; r < 4; ++r) t[((l >> 4) + 4 * r) * ld + (l & 15)] = v[r];
}

// In-place inverse of the matrix of nt x nt tiles (16 x 16 each) at D in LDS (row stride LD,
// a multiple of 16 plus 4 doubles: the 16 rows that an operand read touches fall into
// different banks), by the 16 wavefronts of the workgroup.  For the tile row S, with
// X = D_SS^{-1}:
//   A: D_SJ <- X D_SJ;  B: D_IJ <- D_IJ - D_IS D_SJ;  C: D_IS <- -D_IS X, D_SS <- X
// (I, J != S).  In B wavefront 0 takes tile (S + 1, S + 1) first and inverts it while the
// others update the rest.  X2: two pivot-block inverses.  A pivot that is not positive and
// finite sets *bad; the elimination runs on (the values are then meaningless).
constexpr int GJ_THREADS = 1024;
constexpr int GJ_WAVES = GJ_THREADS / 64;
template <int LD>
__device__ void gj_invert_lds(double* D, int nt, double* X2, int* bad) {
    const int w = threadIdx.x / 64;
    const bgj_v4 zero = {0.0, 0.0, 0.0, 0.0};
    auto tile = [&](int I, int J) { return D + 16 * I * LD + 16 * J; };
    if (w == 0) gj_inv16(D, LD, X2, bad);
    __syncthreads();
    for (int S = 0; S < nt; ++S) {
        double* X = X2 + (S & 1) * 16 * GJ_XLD;
        double* Xn = X2 + ((S + 1) & 1) * 16 * GJ_XLD;
        for (int J = w; J < nt; J += GJ_WAVES)
            if (J != S) gj_tile_store(tile(S, J), LD, gj_tile_mm(X, GJ_XLD, tile(S, J), LD, zero, 1.0));
        __syncthreads();
        auto update = [&](int I, int J) {
            gj_tile_store(tile(I, J), LD,
                          gj_tile_mm(tile(I, S), LD, tile(S, J), LD, gj_tile_load(tile(I, J), LD), -1.0));
        };
        const int N = S + 1;  // the next pivot block, wavefront 0's
        if (N < nt && w == 0) {
            update(N, N);
            wave_fence();  // stored in the product's lane layout, read back in another
            gj_inv16(tile(N, N), LD, Xn, bad);
        } else {
            const int m = nt - 1;
            const int first = N < nt ? w - 1 : w, step = N < nt ? GJ_WAVES - 1 : GJ_WAVES;
            for (int u = first; u < m * m; u += step) {
                const int a = u / m, b = u % m;
                const int I = a < S ? a : a + 1, J = b < S ? b : b + 1;
                if (I == N && J == N) continue;
                update(I, J);
            }
        }
        __syncthreads();
        for (int I = w; I < nt; I += GJ_WAVES) {
            if (I != S) {
                gj_tile_store(tile(I, S), LD, gj_tile_mm(tile(I, S), LD, X, GJ_XLD, zero, -1.0));
            } else {
                const int l = threadIdx.x % 64;
#pragma unroll
                for (int j = 0; j < 4; ++j) tile(S, S)[(l & 15) * LD + 4 * (l >> 4) + j] = X[(l & 15) * GJ_XLD + 4 * (l >> 4) + j];
            }
        }
        __syncthreads();
    }
}

// Up to COARSE_LDS_MAX rows, in one workgroup: the matrix, padded to whole tiles with the
// identity, in LDS (132 x 128 FP64, 132 KiB of the 160 KiB available).
__global__ __launch_bounds__(GJ_THREADS) void k_dense_inverse(int n, double* __restrict__ Mg,
                                                              double* __restrict__ scal) {
    constexpr int LD = COARSE_LDS_MAX + 4;
    __shared__ double M[COARSE_LDS_MAX * LD];
    __shared__ double X2[2 * 16 * GJ_XLD];
    __shared__ int bad;
    const int nt = (n + 15) / 16, np = 16 * nt;
    for (int e = threadIdx.x; e < np * np; e += GJ_THREADS) {
        const int i = e / np, j = e - i * np;
        M[i * LD + j] = i < n && j < n ? Mg[(size_t)i * n + j] : (i == j ? 1.0 : 0.0);
    }
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    gj_invert_lds<LD>(M, nt, X2, &bad);
    for (int e = threadIdx.x; e < n * n; e += GJ_THREADS) {
        const int i = e / n, j = e - i * n;
        Mg[e] = M[i * LD + j];
    }
    if (threadIdx.x == 0) scal[S_COARSE] = bad ? 1.0 : 0.0;
}

// Coarsest levels of more rows: the same elimination taken a block of BGJ pivots at a time.
// With X = M_KK^{-1} for the pivot block K, one block step maps
//   M_KJ <- X M_KJ,   M_IJ <- M_IJ - M_IK X M_KJ,   M_IK <- -M_IK X,   M_KK <- X
// (I, J != K), which is the composition of the scalar steps of K's pivots.  Step K is one
// launch of one workgroup per block, from one copy of the matrix into another (every block
// is read by its whole row and column, so an in-place step would need a second launch); the
// workgroup of block (K + 1, K + 1), the first to be dispatched, goes on to invert its
// result, so that the next step starts with its X.  A workgroup's 64 x 64 x 64 products
// are split over its 16 wavefronts, one 16 x 16 tile each, 16 steps of
// V_MFMA_F64_16X16X4F64 per product.
constexpr int BGJ = 64;
constexpr int BGJ_RPT = BGJ * BGJ / GJ_THREADS;  // tile elements per thread
constexpr int BGJ_LD = BGJ + 4;

__device__ __forceinline__ int bgj_size(int n, int b) { return min(BGJ, n - b * BGJ); }

// A BGJ x BGJ tile spread over the threads: thread t holds rows t / BGJ + (GJ_THREADS /
// BGJ) m (m < BGJ_RPT) of column t % BGJ.  Every global load of a tile is issued before any
// is used.
constexpr int BGJ_RSTEP = GJ_THREADS / BGJ;

// Block (I, J) of the row-major n x n M (zero outside the matrix).
__device__ __forceinline__ void bgj_fetch(const double* __restrict__ M, int n, int I, int J, double (&v)[BGJ_RPT]) {
    const int bi = bgj_size(n, I), bj = bgj_size(n, J);
    const int r = threadIdx.x / BGJ, q = threadIdx.x % BGJ;
    const double* base = M + (size_t)(I * BGJ + r) * n + (size_t)J * BGJ + q;
#pragma unroll
    for (int m = 0; m < BGJ_RPT; ++m)
        v[m] = (r + BGJ_RSTEP * m < bi && q < bj) ? base[(size_t)(BGJ_RSTEP * m) * n] : 0.0;
}

// A tile stored densely (row stride BGJ), as X is.
__device__ __forceinline__ void bgj_fetch_dense(const double* __restrict__ X, double (&v)[BGJ_RPT]) {
#pragma unroll
    for (int m = 0; m < BGJ_RPT; ++m) v[m] = X[threadIdx.x + m * GJ_THREADS];
}

// Into LDS s (row stride BGJ_LD).
__device__ __forceinline__ void bgj_put(double* s, const double (&v)[BGJ_RPT]) {
    const int r = threadIdx.x / BGJ, q = threadIdx.x % BGJ;
#pragma unroll
    for (int m = 0; m < BGJ_RPT; ++m) s[(r + BGJ_RSTEP * m) * BGJ_LD + q] = v[m];
}

// The 16 x 16 tile of a b owned by this wave (tile row w / 4, tile column w % 4 for wave
// w), for BGJ x BGJ tiles a, b in LDS (row stride BGJ_LD).
// Lane l ends with entries (16 (w / 4) + l / 16 + 4 r, 16 (w % 4) + l % 16), r < 4 (the
// instruction's result layout: entry r of lane l is row l / 16 + 4 r, column l % 16).
__device__ __forceinline__ bgj_v4 bgj_mfma(const double* a, const double* b) {
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    const int i = 16 * (w >> 2) + (l & 15), j = 16 * (w & 3) + (l & 15), kk = l >> 4;
    bgj_v4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < BGJ / 4; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i * BGJ_LD + 4 * s + kk], b[(4 * s + kk) * BGJ_LD + j], acc, 0, 0, 0);
    return acc;
}

// Row and column of entry r of this lane's product tile.
__device__ __forceinline__ int bgj_out_row(int r) {
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    return 16 * (w >> 2) + (l >> 4) + 4 * r;
}
__device__ __forceinline__ int bgj_out_col() {
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    return 16 * (w & 3) + (l & 15);
}

// Inverse of the diagonal block K held in LDS at D (its bk rows and columns; the rest is set
// to the identity here), written densely to X; false (in every thread) if a pivot was not
// positive and finite.
__device__ bool bgj_invert_block(double* D, int bk, double* X2, int* bad, double* __restrict__ X) {
    const int r = threadIdx.x / BGJ, q = threadIdx.x % BGJ;
#pragma unroll
    for (int m = 0; m < BGJ_RPT; ++m) {
        const int i = r + BGJ_RSTEP * m;
        if (i >= bk || q >= bk) D[i * BGJ_LD + q] = i == q ? 1.0 : 0.0;
    }
    if (threadIdx.x == 0) *bad = 0;
    __syncthreads();
    gj_invert_lds<BGJ_LD>(D, (bk + 15) / 16, X2, bad);
#pragma unroll
    for (int m = 0; m < BGJ_RPT; ++m) X[threadIdx.x + m * GJ_THREADS] = D[(r + BGJ_RSTEP * m) * BGJ_LD + q];
    return *bad == 0;
}

// X of block 0.
__global__ __launch_bounds__(GJ_THREADS) void k_bgj_first(int n, const double* __restrict__ M, double* __restrict__ X,
                                                          double* __restrict__ scal) {
    __shared__ double D[BGJ * BGJ_LD];
    __shared__ double X2[2 * 16 * GJ_XLD];
    __shared__ int bad;
    double v[BGJ_RPT];
    bgj_fetch(M, n, 0, 0, v);
    bgj_put(D, v);
    __syncthreads();
    const bool ok = bgj_invert_block(D, bgj_size(n, 0), X2, &bad, X);
    if (threadIdx.x == 0) scal[S_COARSE] = ok ? 0.0 : 1.0;
}

// Block step k from M to Mo; X: the inverses of two consecutive pivot blocks.
__global__ __launch_bounds__(GJ_THREADS) void k_bgj_step(int n, int k, const double* __restrict__ M,
                                                         double* __restrict__ Mo, double* __restrict__ X,
                                                         double* __restrict__ scal) {
    __shared__ double sa[BGJ * BGJ_LD];
    __shared__ double sb[BGJ * BGJ_LD];
    __shared__ double st[BGJ * BGJ_LD];
    __shared__ double X2[2 * 16 * GJ_XLD];
    __shared__ int bad;
    const int nb = (n + BGJ - 1) / BGJ;
    // the next pivot block's workgroup is dispatched first (its place taken by block 0's)
    const int next = k + 1 < nb ? (k + 1) * nb + k + 1 : 0;
    const int id = (int)blockIdx.x == 0 ? next : (int)blockIdx.x == next ? 0 : (int)blockIdx.x;
    const int I = id / nb, J = id % nb;
    const int bi = bgj_size(n, I), bj = bgj_size(n, J), j = bgj_out_col();
    const double* Xk = X + (size_t)(k & 1) * BGJ * BGJ;
    double vx[BGJ_RPT], va[BGJ_RPT], vb[BGJ_RPT], cur[4];
    bgj_fetch_dense(Xk, vx);
    if (I != k) bgj_fetch(M, n, I, k, va);
    if (J != k) bgj_fetch(M, n, k, J, vb);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bgj_out_row(r);
        cur[r] = (I != k && J != k && i < bi && j < bj) ? M[(size_t)(I * BGJ + i) * n + (size_t)J * BGJ + j] : 0.0;
    }
    bgj_v4 out = {0.0, 0.0, 0.0, 0.0};
    bgj_put(sa, vx);
    if (J != k) {
        bgj_put(sb, vb);
        __syncthreads();
        out = bgj_mfma(sa, sb);  // T = X M_KJ
    } else {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = sa[bgj_out_row(r) * BGJ_LD + j];  // X
    }
    if (I != k) {  // M_IJ - M_IK T, or -M_IK X in column K
#pragma unroll
        for (int r = 0; r < 4; ++r) st[bgj_out_row(r) * BGJ_LD + j] = out[r];
        __syncthreads();
        bgj_put(sa, va);
        __syncthreads();
        const bgj_v4 acc = bgj_mfma(sa, st);
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = cur[r] - acc[r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = bgj_out_row(r);
        if (i < bi && j < bj) Mo[(size_t)(I * BGJ + i) * n + (size_t)J * BGJ + j] = out[r];
    }
    if (I == k + 1 && J == k + 1) {  // the next step's pivot block
#pragma unroll
        for (int r = 0; r < 4; ++r) sb[bgj_out_row(r) * BGJ_LD + j] = out[r];
        __syncthreads();
        const bool ok = bgj_invert_block(sb, bi, X2, &bad, X + (size_t)((k + 1) & 1) * BGJ * BGJ);
        if (threadIdx.x == 0 && !ok) scal[S_COARSE] = 1.0;
    }
}

size_t coarse_work_doubles(int n) { return n > COARSE_LDS_MAX ? 2 * (size_t)BGJ * BGJ + (size_t)n * n : 0; }

// An odd number of block steps starts from the scratch copy, so that the last one ends in D.
double* coarse_start(int n, double* D, double* work) {
    const int nb = (n + BGJ - 1) / BGJ;
    return n > COARSE_LDS_MAX && (nb & 1) ? work + 2 * (size_t)BGJ * BGJ : D;
}

void launch_dense_inverse(int n, double* D, double* scal, double* work, hipStream_t s) {
    if (n > COARSE_GLOBAL_MAX) throw Fail{AMG_ERR_ARG, "coarsest level too large for the dense inverse"};
    if (n <= COARSE_LDS_MAX) {
        k_dense_inverse<<<1, GJ_THREADS, 0, s>>>(n, D, scal);
        HIP_LAUNCH_CHECK();
        return;
    }
    if (work == nullptr) throw Fail{AMG_ERR_ARG, "blocked coarse inverse without its scratch"};
    const int nb = (n + BGJ - 1) / BGJ;
    double* from = coarse_start(n, D, work);
    double* to = from == D ? work + 2 * (size_t)BGJ * BGJ : D;
    k_bgj_first<<<1, GJ_THREADS, 0, s>>>(n, from, work, scal);
    HIP_LAUNCH_CHECK();
    for (int k = 0; k < nb; ++k) {
        k_bgj_step<<<nb * nb, GJ_THREADS, 0, s>>>(n, k, from, to, work, scal);
        HIP_LAUNCH_CHECK();
        std::swap(from, to);
    }
}

}  // namespace amgmi
