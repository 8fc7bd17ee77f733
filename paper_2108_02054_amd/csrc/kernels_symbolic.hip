// kernels_symbolic.hip -- patterns of the setup (Algorithm 1): the sparsity of a Galerkin
// product with its plan for the numeric phase, the transpose R = P^T, and the launch shapes
// of a matrix's row kernels.  Integer work only; every result is independent of scheduling.
#include <algorithm>

#include "amg_internal.h"

namespace amgmi {

constexpr int TPB = 256;

template <int G>
__device__ __forceinline__ int group_sum_i(int v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, G);
    return v;
}

// Raises *p to v.  Thousands of workgroups share one cell: the cached read first leaves the
// atomic to the few that raise it (a stale value only costs an atomic).
__device__ __forceinline__ void raise_max(int* p, int v) {
    if (v > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) atomicMax(p, v);
}

// ------------------------------------------------------------------ symbolic product
//
// Pattern of C = A B (structural: every product term creates its entry), sorted columns,
// and the numeric phase's plan: the position of every term's column in its C row.  A group
// of G lanes owns a row of C and collects the columns its terms reach in a hash table in
// LDS (open addressing, integer compare-and-swap).  Two passes: k_sym_count counts the
// row's entries and terms; k_sym_fill collects them again, ranks the distinct columns (the
// rank is the place in the sorted row), and writes the columns and, term by term, the
// positions.  Bound by the gathers of the B rows, read twice; nothing per term is written but
// its one- or two-byte position.  The former
// form wrote a 64-bit (row, column) key per term, radix-sorted the keys, kept the unique
// ones and found each term's position by a binary search in the finished row: 16.5 ms of
// a 128^3 setup (108 M terms at level 0).

constexpr int SYM_H_MIN = 64, SYM_H_MAX = 8192;  // table slots per row
constexpr size_t SYM_SMEM = 32768;               // LDS per workgroup aimed at

__device__ __forceinline__ unsigned sym_hash(int c, int shift) { return ((unsigned)c * 2654435761u) >> shift; }

// Inserts column c; its slot (fresh: it was not there), or -1 when the table is full.
__device__ __forceinline__ int sym_insert(int* tab, int H, int shift, int c, bool& fresh) {
    unsigned h = sym_hash(c, shift);
    fresh = false;
    for (int p = 0; p < H; ++p, h = (h + 1) & (unsigned)(H - 1)) {
        int cur = __hip_atomic_load(&tab[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        if (cur == c) return (int)h;
        if (cur == -1) {
            cur = atomicCAS(&tab[h], -1, c);
            fresh = cur == -1;
            if (fresh || cur == c) return (int)h;
        }
    }
    return -1;
}

// A row belongs to a group of G lanes or, on small levels of long rows, to W wavefronts
// (G = 64) that share its table and take a W-th of its A entries each: one wavefront per row
// left most of the chip idle (27-point 72x61x50, level 1 of 496 rows: count 64 -> 35 us, fill
// 176 -> 57).
template <int W>
__device__ __forceinline__ void row_fence() {
    if constexpr (W > 1)
        __syncthreads();
    else
        wave_fence();
}

// Sum of one value per wavefront of the row, and of those before this one (tmp: W ints).
template <int W>
__device__ __forceinline__ int row_prefix(int v, int w, int* tmp, int& before) {
    before = 0;
    if constexpr (W == 1) return v;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) tmp[w] = v;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        if (q == w) before = t;
        t += tmp[q];
    }
    return t;
}

// Walks the terms of the A row [b, e) (the first at offset carry): the group's lanes take 1 << lg lanes per B row, so
// several B rows at a time, the first term of four such steps in flight together.
// f(A entry, term within its B row, term within the row, column); entry(A entry, first
// term's offset, B row start, B row length) once per A entry, before its terms.  Returns the
// offset after the last.
template <int G, class E, class F>
__device__ __forceinline__ int sym_walk(int lane, int lg, int b, int e, int carry, const int* __restrict__ Acol,
                                        const int* __restrict__ Bptr, const int* __restrict__ Bcol, E entry, F f) {
    const int per = G >> lg, sub = lane >> lg, q0 = lane & ((1 << lg) - 1), step = 1 << lg;
    for (int c0 = b; c0 < e; c0 += G) {
        const int k = c0 + lane;
        int b0 = 0, len = 0;
        if (k < e) {
            const int j = Acol[k];
            b0 = Bptr[j];
            len = Bptr[j + 1] - b0;
        }
        int incl = len;
#pragma unroll
        for (int o = 1; o < G; o <<= 1) {
            const int t = __shfl_up(incl, o, G);
            if (lane >= o) incl += t;
        }
        const int to = carry + incl - len;
        carry += __shfl(incl, G - 1, G);
        if (k < e) entry(k, to, b0, len);
        const int nt = min(G, e - c0);
        constexpr int U = 4;
        for (int e0 = 0; e0 < nt; e0 += U * per) {
            int bb[U], ll[U], tt[U], cc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int x = e0 + u * per + sub, xs = x < G ? x : G - 1;
                bb[u] = __shfl(b0, xs, G);
                tt[u] = __shfl(to, xs, G);
                ll[u] = __shfl(len, xs, G);
                if (x >= nt) ll[u] = 0;
                if (q0 < ll[u]) cc[u] = Bcol[bb[u] + q0];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int ke = c0 + e0 + u * per + sub;
                if (q0 < ll[u]) f(ke, q0, tt[u] + q0, cc[u]);
                for (int q = q0 + step; q < ll[u]; q += step) f(ke, q, tt[u] + q, Bcol[bb[u] + q]);
            }
        }
    }
    return carry;
}

// cnt[i], terms[i] (both with a zero at n, so that exclusive scans end in the totals);
// stat: {overflow, most terms in a row, longest row, longest B row met}.
template <int G, int W>
__global__ __launch_bounds__(TPB) void k_sym_count(int n, int lg, int H, int shift, const int* __restrict__ Aptr,
                                                   const int* __restrict__ Acol, const int* __restrict__ Bptr,
                                                   const int* __restrict__ Bcol, int* __restrict__ cnt,
                                                   int64_t* __restrict__ terms, int* __restrict__ stat) {
    extern __shared__ __align__(16) unsigned char sym_smem[];
    __shared__ int tmp[W];
    const int lane = threadIdx.x & (G - 1), gi = threadIdx.x / (G * W), w = (threadIdx.x / G) % W;
    int* tab = reinterpret_cast<int*>(sym_smem) + (size_t)gi * H;
    const int row = xcd_block() * ((int)blockDim.x / (G * W)) + gi;
    if (row > n) return;  // rows leave whole
    if (row == n) {
        if (lane == 0 && w == 0) {
            cnt[n] = 0;
            terms[n] = 0;
        }
        return;
    }
    for (int s = w * G + lane; s < H; s += G * W) tab[s] = -1;
    row_fence<W>();
    const int b = Aptr[row], e = Aptr[row + 1], per = (e - b + W - 1) / W;
    int u = 0, full = 0, mb = 0, before;
    int nterm = sym_walk<G>(lane, lg, min(b + w * per, e), min(b + (w + 1) * per, e), 0, Acol, Bptr, Bcol,
                                  [&](int, int, int, int len) { mb = max(mb, len); },
                                  [&](int, int, int, int c) {
                                      if (full) return;  // (a full table is probed whole)
                                      bool fresh;
                                      full |= sym_insert(tab, H, shift, c, fresh) < 0;
                                      u += fresh;
                                  });
    u = group_sum_i<G>(u);
    full = group_sum_i<G>(full);
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) mb = max(mb, __shfl_xor(mb, o, G));
    u = row_prefix<W>(u, w, tmp, before);
    full = row_prefix<W>(full, w, tmp, before);
    nterm = row_prefix<W>(nterm, w, tmp, before);
    if (lane == 0) raise_max(&stat[3], mb);
    if (lane == 0 && w == 0) {
        cnt[row] = u;
        terms[row] = nterm;
        raise_max(&stat[0], full ? 1 : 0);
        raise_max(&stat[1], nterm);
        raise_max(&stat[2], u);
    }
}

__global__ void k_sym_totals(int n, const int* __restrict__ ptr, const int64_t* __restrict__ off,
                             const int* __restrict__ stat, int64_t* __restrict__ out) {
    out[0] = ptr[n];
    out[1] = off[n];
    for (int k = 0; k < 4; ++k) out[2 + k] = stat[k];
}

// Columns of row i of C in order, and the plan: per A entry its B row start (bst) and, with
// pos, its first term's offset and per term its column's position in the C row; with inv,
// per A entry k and position p of the C row the B row's entry there, inv[k iw + p] = entry + 1
// (inv cleared by the caller: 0 for none).
template <int G, int W, typename PT>
__global__ __launch_bounds__(TPB) void k_sym_fill(int n, int lg, int H, int shift, const int* __restrict__ Aptr,
                                                  const int* __restrict__ Acol, const int* __restrict__ Bptr,
                                                  const int* __restrict__ Bcol, const int* __restrict__ Cptr,
                                                  int* __restrict__ Ccol, const int64_t* __restrict__ off,
                                                  int* __restrict__ bst, uint16_t* __restrict__ tof,
                                                  PT* __restrict__ pos, uint8_t* __restrict__ inv, int iw) {
    extern __shared__ __align__(16) unsigned char sym_smem[];
    __shared__ int tmp[W];
    const int lane = threadIdx.x & (G - 1), gi = threadIdx.x / (G * W), w = (threadIdx.x / G) % W;
    unsigned char* base = sym_smem + (size_t)gi * 8 * H;
    int* tab = reinterpret_cast<int*>(base);
    uint16_t* rank = reinterpret_cast<uint16_t*>(base + (size_t)4 * H);  // of the column in each slot
    uint16_t* list = reinterpret_cast<uint16_t*>(base + (size_t)6 * H);  // the occupied slots
    const int row = xcd_block() * ((int)blockDim.x / (G * W)) + gi;
    if (row >= n) return;
    for (int s = w * G + lane; s < H; s += G * W) tab[s] = -1;
    row_fence<W>();
    const int rb = Aptr[row], re = Aptr[row + 1], per = (re - rb + W - 1) / W;
    const int b = min(rb + w * per, re), e = min(rb + (w + 1) * per, re);  // this wavefront's entries
    int first = 0;  // its first term's offset
    if constexpr (W > 1) {
        int mine = 0;
        for (int k = b + lane; k < e; k += G) mine += Bptr[Acol[k] + 1] - Bptr[Acol[k]];
        row_prefix<W>(group_sum_i<G>(mine), w, tmp, first);
    }
    PT* prow = pos != nullptr ? pos + off[row] : nullptr;
    // where a slot number fits a position's type the first walk leaves each term's slot in its
    // place, and the ranks replace them in a pass over contiguous memory; else the row is
    // walked again
    const bool by_slot = prow != nullptr && (sizeof(PT) > 1 || H <= 256);
    const int last = sym_walk<G>(
        lane, lg, b, e, first, Acol, Bptr, Bcol,
        [&](int k, int to, int b0, int) {
            if (bst != nullptr) bst[k] = b0;
            if (tof != nullptr) tof[k] = (uint16_t)to;
        },
        [&](int, int, int t, int c) {
            bool fresh;
            const int slot = sym_insert(tab, H, shift, c, fresh);
            if (by_slot) prow[t] = (PT)slot;
        });
    row_fence<W>();
    int u = 0;
    const int s_lo = W > 1 ? (H / W) * w : 0, s_hi = W > 1 ? s_lo + H / W : H;  // (H / W: a multiple of G)
    if constexpr (W > 1) {
        int occ = 0, before;
        for (int s0 = s_lo; s0 < s_hi; s0 += G) occ += __popcll(__ballot(tab[s0 + lane] != -1));
        row_prefix<W>(occ, w, tmp, before);
        u = before;
    }
    const int shiftg = (threadIdx.x & 63) & ~(G - 1);
    const unsigned long long mine = G == 64 ? ~0ull : ((1ull << G) - 1);
    for (int s0 = s_lo; s0 < s_hi; s0 += G) {  // H is a multiple of 64
        const bool occ = tab[s0 + lane] != -1;
        const unsigned long long m = (__ballot(occ) >> shiftg) & mine;
        if (occ) list[u + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)(s0 + lane);
        u += __popcll(m);
    }
    row_fence<W>();
    const int cb = Cptr[row], len = Cptr[row + 1] - cb;
    if constexpr (W > 1) u = len;
    for (int x0 = w * G; x0 < u; x0 += G * W) {
        const int x = x0 + lane;
        const int slot = x < u ? list[x] : 0;
        const int c = x < u ? tab[slot] : -1;
        int r = 0;
        for (int y0 = 0; y0 < u; y0 += G) {
            const int v = y0 + lane < u ? tab[list[y0 + lane]] : 0x7fffffff;
            const int ny = min(G, u - y0);
            for (int t = 0; t < ny; ++t) r += __shfl(v, t, G) < c;
        }
        if (x < u && r < len) {
            Ccol[cb + r] = c;
            rank[slot] = (uint16_t)r;
        }
    }
    if (pos == nullptr && inv == nullptr) return;
    row_fence<W>();
    if (by_slot) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // (the slots other lanes wrote)
        for (int t = first + lane; t < last; t += G) prow[t] = (PT)rank[prow[t]];
        return;
    }
    sym_walk<G>(lane, lg, b, e, first, Acol, Bptr, Bcol, [](int, int, int, int) {}, [&](int k, int q, int t, int c) {
        unsigned h = sym_hash(c, shift);
        for (int p = 0; p < H && tab[h] != c; ++p) h = (h + 1) & (unsigned)(H - 1);
        if (prow != nullptr)
            prow[t] = (PT)rank[h];
        else
            inv[(size_t)k * iw + rank[h]] = (uint8_t)(q + 1);
    });
}

static int log2_ceil(double v) {
    int l = 0;
    while (l < 30 && (double)(1 << l) < v) ++l;
    return l;
}

// Lanes per row from the mean number of terms (a lane for every four to eight of them, and
// wide groups for large tables, whose clearing and compaction they share).
static int sym_group(double mean_terms, int H) {
    int g = mean_terms <= 32.0 ? 8 : mean_terms <= 160.0 ? 16 : mean_terms <= 640.0 ? 32 : 64;
    while (g < 64 && H > 32 * g) g <<= 1;
    return g;
}

#define AMG_WITH_SYM_G(g, ...)                                              \
    do {                                                                    \
        switch (g) {                                                        \
            case 8: { constexpr int G = 8; __VA_ARGS__; } break;            \
            case 16: { constexpr int G = 16; __VA_ARGS__; } break;          \
            case 32: { constexpr int G = 32; __VA_ARGS__; } break;          \
            default: { constexpr int G = 64; __VA_ARGS__; } break;          \
        }                                                                   \
    } while (0)

// Products of at most SYM_W_ROWS rows get SYM_W wavefronts per row where a row has at least
// SYM_W_TERMS terms (fewer don't keep them busy) and a wavefront of table slots for each; the
// largest table leaves no LDS beside it.
constexpr int SYM_W = 4, SYM_W_ROWS = 2048, SYM_W_TERMS = 1024;
static bool sym_wide(int n, int g, int H, double mean_terms) {
    return g == 64 && n <= SYM_W_ROWS && H >= 64 * SYM_W && H < SYM_H_MAX && mean_terms >= SYM_W_TERMS;
}

// Threads per workgroup: whole wavefronts, as many rows as SYM_SMEM holds.
static int sym_threads(int g, size_t row_bytes) {
    int t = TPB;
    while (t > 64 && (size_t)(t / g) * row_bytes > SYM_SMEM) t >>= 1;
    return t;
}

bool symbolic_count(const Csr& A, const Csr& B, Csr& C, int64_t* off, SymSizes& z, hipStream_t s) {
    const int n = A.nrows;
    if (!lanes_fit_grid((int64_t)n + 1, 8)) return false;
    C.nrows = n;
    C.ncols = B.ncols;
    C.ptr = dnew<int32_t>((size_t)n + 1, s);
    int32_t* cnt = dnew<int32_t>((size_t)n + 1, s);
    int64_t* terms = dnew<int64_t>((size_t)n + 1, s);
    int* stat = dnew<int>(4, s);
    int64_t* tot = dnew<int64_t>(6, s);
    const double mean_b = B.nrows > 0 ? (double)B.nnz / (double)B.nrows : 0.0;
    z.mean_b = mean_b;
    z.mean_terms = n > 0 ? (double)A.nnz / (double)n * mean_b : 0.0;
    const int lg_b = std::min(log2_ceil(mean_b), 6);
    bool fits = false;
    int64_t h[6] = {0, 0, 0, 0, 0, 0};
    // rows keep a small share of their terms as distinct columns: start from half the mean
    // number of terms and enlarge the table when some row overflows it
    for (int H = std::min(SYM_H_MAX, std::max(SYM_H_MIN, 1 << log2_ceil(0.5 * z.mean_terms)));;) {
        const int g = sym_group(z.mean_terms, H), lg = std::min(lg_b, log2_ceil(g));
        const int t = sym_threads(g, (size_t)4 * H), rows = t / g, shift = 32 - log2_ceil(H);
        HIP_CHECK(hipMemsetAsync(stat, 0, 4 * sizeof(int), s));
        if (sym_wide(n, g, H, z.mean_terms))
            k_sym_count<64, SYM_W><<<(unsigned)n + 1, 64 * SYM_W, (size_t)4 * H, s>>>(n, lg, H, shift, A.ptr, A.col, B.ptr,
                                                                                     B.col, cnt, terms, stat);
        else
            AMG_WITH_SYM_G(g, (k_sym_count<G, 1><<<(unsigned)(n / rows + 1), t, (size_t)rows * 4 * H, s>>>(
                                  n, lg, H, shift, A.ptr, A.col, B.ptr, B.col, cnt, terms, stat)));
        HIP_LAUNCH_CHECK();
        exclusive_scan_i32(cnt, C.ptr, (int64_t)n + 1, s);
        exclusive_scan_i64(terms, off, (int64_t)n + 1, s);
        k_sym_totals<<<1, 1, 0, s>>>(n, C.ptr, off, stat, tot);
        HIP_LAUNCH_CHECK();
        HIP_CHECK(hipMemcpyAsync(h, tot, sizeof(h), hipMemcpyDeviceToHost, s));
        HIP_CHECK(hipStreamSynchronize(s));
        fits = h[2] == 0;
        if (fits || H == SYM_H_MAX || h[1] >= ((int64_t)1 << 31)) break;
        H = std::min(SYM_H_MAX, 4 * H);
    }
    dfree(cnt, s);
    dfree(terms, s);
    dfree(stat, s);
    dfree(tot, s);
    z.terms = h[1];
    z.max_terms = h[3];
    z.maxlen = (int)h[4];
    z.max_b = (int)h[5];
    if (z.terms >= ((int64_t)1 << 31)) {
        dfree(C.ptr, s);
        C.ptr = nullptr;
        throw Fail{AMG_ERR_ARG, "Galerkin product too large for int32 indexing"};
    }
    if (!fits) {
        dfree(C.ptr, s);
        C.ptr = nullptr;
        return false;
    }
    C.nnz = h[0];
    C.col = dnew<int32_t>((size_t)C.nnz, s);
    return true;
}

void symbolic_fill(const Csr& A, const Csr& B, const Csr& C, const GalShape& gs, const int64_t* off,
                   const SymSizes& z, hipStream_t s) {
    const int n = A.nrows;
    if (n == 0) return;
    const int H = std::min(SYM_H_MAX, std::max(SYM_H_MIN, 1 << log2_ceil(1.5 * z.maxlen)));
    if (gs.inv != nullptr) HIP_CHECK(hipMemsetAsync(gs.inv, 0, (size_t)A.nnz * gs.inv_w, s));
    const int g = sym_group(z.mean_terms, H), lg = std::min(std::min(log2_ceil(z.mean_b), 6), log2_ceil(g));
    const int t = sym_threads(g, (size_t)8 * H), rows = t / g, shift = 32 - log2_ceil(H);
    const unsigned nb = (unsigned)((n + rows - 1) / rows);
    auto fill = [&](auto* pos) {
        using PT = std::remove_pointer_t<decltype(pos)>;
        auto go = [&](auto kern, unsigned blocks, int threads, size_t bytes) {
            kern<<<blocks, threads, bytes, s>>>(n, lg, H, shift, A.ptr, A.col, B.ptr, B.col, C.ptr, C.col, off, gs.bst,
                                                gs.tof, pos, gs.inv, gs.inv_w);
        };
        if (sym_wide(n, g, H, z.mean_terms))
            go(k_sym_fill<64, SYM_W, PT>, (unsigned)n, 64 * SYM_W, (size_t)8 * H);
        else
            AMG_WITH_SYM_G(g, go(k_sym_fill<G, 1, PT>, nb, t, (size_t)rows * 8 * H));
    };
    if (gs.wide)
        fill((uint16_t*)gs.pos);
    else
        fill((uint8_t*)gs.pos);
    HIP_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ transpose
//
// R = P^T with sorted columns: the entries of each column of P are counted, scattered in
// any order into the column's row of R, and each row of R is then put in order by the rank
// of its (distinct) row indices.  Rows of R longer than TR_ROW_MAX would make the ranking
// quadratic: such a matrix is sorted as a whole.

constexpr int TR_ROW_MAX = 2048;
constexpr int64_t TR_LANES_MIN = 1 << 17;

// The rows of a workgroup name few different columns (neighbouring fine rows belong to the
// same aggregates), and one atomic per entry on a column's counter is what these two passes
// waited for: the workgroup meets its columns in a table in LDS and adds its share of each
// with one atomic (128^3 smoothed P,
// 7.2 M entries: count 211 -> 85 us, scatter 295 -> 99 us).  A column finds its place
// within TR_PROBE slots of its hash or, all of them being taken for good, stays outside the
// table, for every thread alike.
constexpr int TR_H = 1024, TR_PROBE = 16;

__device__ __forceinline__ int tr_slot(int* key, int J) {
    const unsigned h = ((unsigned)J * 2654435761u) >> 22;
    for (int p = 0; p < TR_PROBE; ++p) {
        const int q = (int)((h + p) & (TR_H - 1));
        const int old = atomicCAS(&key[q], -1, J);
        if (old == -1 || old == J) return q;
    }
    return -1;
}
static_assert(TR_H == 1 << 10, "the hash keeps ten bits");

__device__ __forceinline__ void tr_clear(int* key, int* num) {
    for (int q = threadIdx.x; q < TR_H; q += TPB) {
        key[q] = -1;
        num[q] = 0;
    }
    __syncthreads();
}

__global__ __launch_bounds__(TPB) void k_tr_count(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                                  int* __restrict__ cnt) {
    __shared__ int key[TR_H], num[TR_H];
    tr_clear(key, num);
    const int i = xcd_block() * TPB + threadIdx.x;
    const int k0 = i < n ? ptr[i] : 0, k1 = i < n ? ptr[i + 1] : 0;
    for (int k = k0; k < k1; ++k) {
        const int J = col[k], q = tr_slot(key, J);
        atomicAdd(q >= 0 ? &num[q] : &cnt[J], 1);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < TR_H; q += TPB)
        if (num[q] > 0) atomicAdd(&cnt[key[q]], num[q]);
}

// cnt holds each column's count and counts down to its first place.
__global__ __launch_bounds__(TPB) void k_tr_scatter(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                                    const int* __restrict__ Rptr, int* __restrict__ cnt,
                                                    int2* __restrict__ tmp) {
    __shared__ int key[TR_H], num[TR_H];
    tr_clear(key, num);
    const int i = xcd_block() * TPB + threadIdx.x;
    const int k0 = i < n ? ptr[i] : 0, k1 = i < n ? ptr[i + 1] : 0;
    for (int k = k0; k < k1; ++k) {
        const int q = tr_slot(key, col[k]);
        if (q >= 0) atomicAdd(&num[q], 1);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < TR_H; q += TPB)  // num: from the count to the first place
        if (num[q] > 0) num[q] = Rptr[key[q]] + atomicSub(&cnt[key[q]], num[q]) - num[q];
    __syncthreads();
    for (int k = k0; k < k1; ++k) {
        const int J = col[k], q = tr_slot(key, J);
        tmp[q >= 0 ? atomicAdd(&num[q], 1) : Rptr[J] + atomicSub(&cnt[J], 1) - 1] = make_int2(i, k);
    }
}

// Puts each row of R in order by the rank of its row indices: a group of G lanes per row
// stages them in LDS (at most TR_KEYS G of them) and every lane counts, for two of its own at
// a time, the smaller ones, four per LDS read (27-point 72x61x50: 174 -> 32 us on level
// 0, 104 -> 6 on the 496 rows of level 1, against a shuffle per comparison).
constexpr int TR_KEYS = TR_ROW_MAX / TPB;

template <int G>
__global__ __launch_bounds__(TPB) void k_tr_order(int nc, const int* __restrict__ Rptr, const int2* __restrict__ tmp,
                                                  const double* __restrict__ v, int* __restrict__ Rcol,
                                                  double* __restrict__ Rval) {
    __shared__ __align__(16) int keys[TPB / G][TR_KEYS * G];
    const int lane = threadIdx.x & (G - 1);
    const int row = lane_row(xcd_block(), TPB, threadIdx.x, G);
    int* mine = keys[threadIdx.x / G];
    const int b = row < nc ? Rptr[row] : 0, u = row < nc ? Rptr[row + 1] - b : 0;
    for (int x = lane; x < ((u + 3) & ~3); x += G) mine[x] = x < u ? tmp[b + x].x : 0x7fffffff;
    if constexpr (G > 64) {
        __syncthreads();
    } else {
        wave_fence();
    }
    for (int x = lane; x < u; x += 2 * G) {
        const int x2 = x + G < u ? x + G : x;
        const int t1 = mine[x], t2 = mine[x2];
        int r1 = 0, r2 = 0;
        for (int y = 0; y < u; y += 4) {
            const int4 w = *reinterpret_cast<const int4*>(mine + y);
            r1 += (w.x < t1) + (w.y < t1) + (w.z < t1) + (w.w < t1);
            r2 += (w.x < t2) + (w.y < t2) + (w.z < t2) + (w.w < t2);
        }
        Rcol[b + r1] = t1;
        Rval[b + r1] = v[tmp[b + x].y];
        if (x2 != x) {
            Rcol[b + r2] = t2;
            Rval[b + r2] = v[tmp[b + x2].y];
        }
    }
}

__global__ __launch_bounds__(TPB) void k_max_len(int n, const int* __restrict__ cnt, int* __restrict__ out) {
    __shared__ int sm[TPB / 64];
    const int i = blockIdx.x * TPB + threadIdx.x;
    int v = i < n ? cnt[i] : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < TPB / 64; ++k) v = max(v, sm[k]);
        raise_max(out, v);
    }
}

void build_transpose(const Csr& P, Csr& R, hipStream_t s) {
    const int64_t nnz = P.nnz;
    R.nrows = P.ncols;
    R.ncols = P.nrows;
    R.nnz = nnz;
    R.ptr = dnew<int32_t>((size_t)R.nrows + 1, s);
    R.col = dnew<int32_t>((size_t)nnz, s);
    R.val = dnew<double>((size_t)nnz, s);
    const unsigned nb = (unsigned)std::max<int64_t>(1, ((int64_t)P.nrows + TPB - 1) / TPB);
    int* cnt = dnew<int>((size_t)R.nrows + 2, s);  // counts, a zero, and the longest
    HIP_CHECK(hipMemsetAsync(cnt, 0, ((size_t)R.nrows + 2) * sizeof(int), s));
    k_tr_count<<<nb, TPB, 0, s>>>(P.nrows, P.ptr, P.col, cnt);
    k_max_len<<<(unsigned)std::max<int64_t>(1, ((int64_t)R.nrows + TPB - 1) / TPB), TPB, 0, s>>>(R.nrows, cnt,
                                                                                                  cnt + R.nrows + 1);
    HIP_LAUNCH_CHECK();
    exclusive_scan_i32(cnt, R.ptr, (int64_t)R.nrows + 1, s);
    int longest = 0;
    HIP_CHECK(hipMemcpyAsync(&longest, cnt + R.nrows + 1, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    if (longest > TR_ROW_MAX) {
        dfree(cnt, s);
        transpose_sorted(P, R, s);
        return;
    }
    int2* tmp = dnew<int2>((size_t)nnz, s);
    k_tr_scatter<<<nb, TPB, 0, s>>>(P.nrows, P.ptr, P.col, R.ptr, cnt, tmp);
    // lanes per row: about half its entries, enough LDS for the longest, and with few rows
    // more, so that the long rows of a small level don't leave the chip to a few wavefronts
    const double mean = R.nrows > 0 ? (double)nnz / R.nrows : 0.0;
    int g = mean <= 12.0 ? 8 : mean <= 24.0 ? 16 : 32;
    while (g < TPB && (TR_KEYS * g < longest || (int64_t)R.nrows * g < TR_LANES_MIN)) g <<= 1;
    auto order = [&](auto G) {
        constexpr int W = decltype(G)::value;
        k_tr_order<W><<<(unsigned)std::max<int64_t>(1, ((int64_t)R.nrows * W + TPB - 1) / TPB), TPB, 0, s>>>(
            R.nrows, R.ptr, tmp, P.val, R.col, R.val);
    };
    switch (g) {
        case 8: order(std::integral_constant<int, 8>{}); break;
        case 16: order(std::integral_constant<int, 16>{}); break;
        case 32: order(std::integral_constant<int, 32>{}); break;
        case 64: order(std::integral_constant<int, 64>{}); break;
        case 128: order(std::integral_constant<int, 128>{}); break;
        default: order(std::integral_constant<int, 256>{}); break;
    }
    HIP_LAUNCH_CHECK();
    dfree(cnt, s);
    dfree(tmp, s);
}

// ------------------------------------------------------------------ launch shapes

// most[b] is raised to the largest number of entries in 2^b consecutive rows (aligned at
// multiples of 2^b), for b = 0 .. 8.  (A thread per maximum: one thread raising them one after
// the other waited 25 to 55 us for memory, 5 to 20 now.)
static_assert(RB_THREADS == 256, "one workgroup reads the rows of the largest block");
__global__ __launch_bounds__(TPB) void k_row_blocks(int n, const int* __restrict__ ptr, int* __restrict__ most) {
    __shared__ int sp[RB_THREADS + 1];
    __shared__ int sm[TPB / 64][ROW_BLOCK_SIZES];
    int w[ROW_BLOCK_SIZES] = {};
    const int nblk = (n + RB_THREADS - 1) / RB_THREADS;
    for (int k = blockIdx.x; k < nblk; k += gridDim.x) {
        const int64_t r0 = (int64_t)k * RB_THREADS;
        for (int i = threadIdx.x; i <= RB_THREADS; i += TPB) sp[i] = ptr[r0 + i < n ? r0 + i : n];
        __syncthreads();
#pragma unroll
        for (int b = 0; b < ROW_BLOCK_SIZES; ++b)
            if ((int)threadIdx.x < (RB_THREADS >> b)) w[b] = max(w[b], sp[(threadIdx.x + 1) << b] - sp[threadIdx.x << b]);
        __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < ROW_BLOCK_SIZES; ++b) {
        int v = w[b];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
        if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6][b] = v;
    }
    __syncthreads();
    if (threadIdx.x < ROW_BLOCK_SIZES) {  // side by side: each waits for memory on its own
        int v = sm[0][threadIdx.x];
        for (int k = 1; k < TPB / 64; ++k) v = max(v, sm[k][threadIdx.x]);
        raise_max(&most[threadIdx.x], v);
    }
}

void launch_row_blocks(const Csr& A, int* most, hipStream_t s) {
    const int64_t nb = ((int64_t)A.nrows + RB_THREADS - 1) / RB_THREADS;
    k_row_blocks<<<(unsigned)std::min<int64_t>(std::max<int64_t>(1, nb), 512), TPB, 0, s>>>(A.nrows, A.ptr, most);
    HIP_LAUNCH_CHECK();
}

// One base per row block: the smallest column of its rows (rows are sorted, so the
// first entry of each); *wide = 1 when a block's columns span more than two bytes.  A
// wavefront per block.
__global__ __launch_bounds__(TPB) void k_c16_bases(int n, int rpb, const int* __restrict__ ptr,
                                                   const int* __restrict__ col, int* __restrict__ cblk,
                                                   int* __restrict__ wide) {
    const int b = lane_row(blockIdx.x, TPB, threadIdx.x, 64), lane = threadIdx.x & 63;
    const int r0 = b * rpb, r1 = min(r0 + rpb, n);
    if (r0 >= n) return;
    int lo = 0x7fffffff, hi = -1;
    for (int r = r0 + lane; r < r1; r += 64) {
        const int k0 = ptr[r], k1 = ptr[r + 1];
        if (k0 < k1) {
            lo = min(lo, col[k0]);
            hi = max(hi, col[k1 - 1]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, 64));
        hi = max(hi, __shfl_xor(hi, o, 64));
    }
    if (lane != 0) return;
    if (hi < 0) lo = hi = 0;  // no entries
    cblk[b] = lo;
    if (hi - lo > 65535) wide[0] = 1;
}

// A workgroup per row block, its entries in order.
__global__ __launch_bounds__(TPB) void k_c16_fill(int n, int rpb, const int* __restrict__ ptr,
                                                  const int* __restrict__ col, const int* __restrict__ cblk,
                                                  uint16_t* __restrict__ c16) {
    const int b = xcd_block();
    const int r0 = b * rpb, base = cblk[b], k1 = ptr[min(r0 + rpb, n)];
    for (int k = ptr[r0] + threadIdx.x; k < k1; k += TPB) c16[k] = (uint16_t)(col[k] - base);
}

void launch_c16_bases(const Csr& A, int32_t* cblk, int* wide, hipStream_t s) {
    const int64_t nb = (A.nrows + A.rpb - 1) / A.rpb;
    k_c16_bases<<<(unsigned)((nb * 64 + TPB - 1) / TPB), TPB, 0, s>>>(A.nrows, A.rpb, A.ptr, A.col, cblk, wide);
    HIP_LAUNCH_CHECK();
}
void launch_c16_fill(const Csr& A, const int32_t* cblk, uint16_t* c16, hipStream_t s) {
    k_c16_fill<<<(unsigned)((A.nrows + A.rpb - 1) / A.rpb), TPB, 0, s>>>(A.nrows, A.rpb, A.ptr, A.col, cblk, c16);
    HIP_LAUNCH_CHECK();
}

}  // namespace amgmi
