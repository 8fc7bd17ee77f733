// kernels_galerkin.hip -- numeric phase of the Galerkin product A_{l+1} = R_l (A_l P_l)
// on patterns cached at setup, and the smoother diagonal (Algorithm 4, Section 3; the
// reuse of the product's sparsity pattern is the extension proposed in Section 5).
//
// Determinism: no atomics.  Each output entry is owned by one lane, which adds its
// product terms in the order a row-by-row (Gustavson) product visits them: increasing k
// along row i of the left factor, at most one matching entry per row of the right factor.
// Products and sums are rounded separately (contraction off), so FP64 results are
// bitwise reproducible and independent of the launch shape.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "amg_internal.h"

#pragma clang fp contract(off)

namespace amgmi {

constexpr int TPB = 256;

#define AMG_WITH_G(g, ...)                                                  \
    do {                                                                    \
        switch (g) {                                                        \
            case 2: { constexpr int G = 2; __VA_ARGS__; } break;            \
            case 4: { constexpr int G = 4; __VA_ARGS__; } break;            \
            case 8: { constexpr int G = 8; __VA_ARGS__; } break;            \
            case 16: { constexpr int G = 16; __VA_ARGS__; } break;          \
            case 32: { constexpr int G = 32; __VA_ARGS__; } break;          \
            case 64: { constexpr int G = 64; __VA_ARGS__; } break;          \
            default: throw Fail{AMG_ERR_ARG, "unsupported lane group"};     \
        }                                                                   \
    } while (0)

static inline unsigned row_blocks(int64_t rows, int G) {
    int64_t b = (rows * G + TPB - 1) / TPB;
    return (unsigned)(b > 0 ? b : 1);
}

// Smoother diagonal of one level: damped Jacobi m_i = omega / a_ii, or SPAI0
// m_i = a_ii / sum_j a_ij^2 with the sum taken along the row in column order.
template <typename T>
__global__ __launch_bounds__(TPB) void k_smoother_diag(int n, const int* __restrict__ ptr,
                                                       const int* __restrict__ col, const T* __restrict__ val,
                                                       int kind, T omega, T* __restrict__ m) {
    const int i = xcd_block() * TPB + threadIdx.x;
    if (i >= n) return;
    T d = 0, s = 0;
    for (int k = ptr[i]; k < ptr[i + 1]; ++k) {
        const T a = val[k];
        if (col[k] == i) d = a;
        s = s + a * a;
    }
    m[i] = (kind == 1) ? d / s : omega / d;
}

// AP = A P into the cached pattern of AP.  A group of G lanes per row of A; each lane
// owns entries J of the AP row and scans the P rows of the row's columns for J.
template <int G, typename T>
__global__ __launch_bounds__(TPB) void k_galerkin_ap(int n, const int* __restrict__ Aptr,
                                                     const int* __restrict__ Acol, const T* __restrict__ Aval,
                                                     const int* __restrict__ Pptr, const int* __restrict__ Pcol,
                                                     const T* __restrict__ Pval, const int* __restrict__ APptr,
                                                     const int* __restrict__ APcol, T* __restrict__ APval) {
    const int lane = threadIdx.x & (G - 1);
    const int row = (xcd_block() * TPB + (int)threadIdx.x) / G;
    if (row >= n) return;
    const int ab = Aptr[row], ae = Aptr[row + 1];
    const int se = APptr[row + 1];
    for (int s = APptr[row] + lane; s < se; s += G) {
        const int J = APcol[s];
        T acc = 0;
        for (int k = ab; k < ae; ++k) {
            const int j = Acol[k];
            const int pe = Pptr[j + 1];
            for (int q = Pptr[j]; q < pe; ++q) {
                const int c = Pcol[q];
                if (c >= J) {
                    if (c == J) acc = acc + Aval[k] * Pval[q];
                    break;
                }
            }
        }
        APval[s] = acc;
    }
}

// Position of column J in the sorted, non-empty row cols[b, e), or -1.
__device__ __forceinline__ int find_sorted(const int* __restrict__ cols, int b, int e, int J) {
    int lo = b, hi = e - 1;  // the lower bound of J lies in [lo, hi]
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cols[mid] < J)
            lo = mid + 1;
        else
            hi = mid;
    }
    return cols[lo] == J ? lo : -1;
}

// A_c = R (AP) into the cached pattern of A_c.  A group of G lanes per coarse row; each
// lane owns entries J of the row and walks the R row, finding J in each AP row.
template <int G, typename T>
__global__ __launch_bounds__(TPB) void k_galerkin_rap(int nc, const int* __restrict__ Rptr,
                                                      const int* __restrict__ Rcol, const T* __restrict__ Rval,
                                                      const int* __restrict__ APptr, const int* __restrict__ APcol,
                                                      const T* __restrict__ APval, const int* __restrict__ Cptr,
                                                      const int* __restrict__ Ccol, T* __restrict__ Cval) {
    const int lane = threadIdx.x & (G - 1);
    const int row = (xcd_block() * TPB + (int)threadIdx.x) / G;
    if (row >= nc) return;
    const int rb = Rptr[row], re = Rptr[row + 1];
    const int se = Cptr[row + 1];
    for (int s = Cptr[row] + lane; s < se; s += G) {
        const int J = Ccol[s];
        T acc = 0;
        for (int q = rb; q < re; ++q) {
            const int i = Rcol[q];
            const int b = APptr[i], e = APptr[i + 1];
            if (b == e) continue;
            const int pos = find_sorted(APcol, b, e, J);
            if (pos >= 0) acc = acc + Rval[q] * APval[pos];
        }
        Cval[s] = acc;
    }
}

// ------------------------------------------------------------------ position-map form
//
// The terms of row i of C = L B are l_t * b_e for the L entries t of row i in order and,
// for each, the entries e of B row Lcol[t] in order; this is the order in which a
// row-by-row product adds them.  Which B entries a row's terms read, and the position of
// each term's column in the (cached, sorted) C row, depend on the patterns alone, so setup
// stores them once: for every L entry its B row start and the offset of its first term
// within the row's terms, and for every term its position in the C row (the position
// map).  Each numeric product then only multiplies, and adds each term into its C entry,
// kept in LDS.  A group of G lanes per row of C loads a chunk of the row's L entries
// (EPL per lane) into LDS, then walks them in order, WF_AHEAD at a time: the lanes load
// those entries' terms (G per entry per pass) together, then add them entry by entry.
// Positions within one B row are distinct, and the LDS operations of a wavefront complete
// in program order, so every entry of C receives its terms in the row-by-row order.  For
// C = A P the group also forms the smoother diagonal (the row's squares added in column
// order) and, from both, Q = (I - M A) P (the finished C row is still in LDS, so Q costs
// its write only), and can take A's values from a new FP64 array, storing the hierarchy's
// copies on the way.

constexpr int WF_LOADS = 8;            // B terms per lane loaded together
constexpr int WF_CAP_MAX = 4096;       // longest C row the form takes
constexpr int64_t WF_TERMS_MAX = 65535;  // most terms in one C row (two-byte term offsets)
constexpr size_t WF_SMEM_MAX = 65536;  // LDS per block

// One staged L entry: its B row start, first term (within the row) and term count.
struct alignas(16) WfEnt {
    int bs, to, len, pad;
};

template <typename T, int G, int EPL>
constexpr size_t wf_group_smem(int cap) {
    return (size_t)cap * sizeof(T) + (size_t)EPL * G * (sizeof(T) + sizeof(WfEnt));
}

template <typename T, int G, typename PT, int EPL, int TPL>
__global__ __launch_bounds__(TPB) void k_galerkin_pos(
    int nrows, int cap, const int* __restrict__ Lptr, const T* __restrict__ Lval, const int* __restrict__ Lbst,
    const uint16_t* __restrict__ Ltof, const T* __restrict__ Bval, const int* __restrict__ Cptr,
    T* __restrict__ Cval, const PT* __restrict__ pos, const int64_t* __restrict__ poff,
    const int* __restrict__ dpos, int kind, T omega, T* __restrict__ m, T* __restrict__ Qval,
    const double* __restrict__ lin,
    double* __restrict__ lout64, T* __restrict__ loutT, const uint8_t* __restrict__ dslot, int64_t dn,
    double* __restrict__ dout64, T* __restrict__ doutT) {
    extern __shared__ __align__(16) unsigned char wf_smem[];
    constexpr int NE = EPL * G;  // L entries per chunk
    const int g = threadIdx.x & (G - 1);
    const int gi = threadIdx.x / G;
    unsigned char* gbase = wf_smem + (size_t)gi * wf_group_smem<T, G, EPL>(cap);
    T* sacc = reinterpret_cast<T*>(gbase);
    T* elv = reinterpret_cast<T*>(gbase + (size_t)cap * sizeof(T));
    WfEnt* ent = reinterpret_cast<WfEnt*>(gbase + (size_t)cap * sizeof(T) + (size_t)NE * sizeof(T));
    const int row = (xcd_block() * TPB + (int)threadIdx.x) / G;
    if (row >= nrows) return;  // groups leave whole: G divides the wavefront
    const int sb = Cptr[row];
    const int len = min(Cptr[row + 1] - sb, cap);  // the host keeps every row within cap
    const int lb = Lptr[row], le = Lptr[row + 1];
    const int64_t p0 = poff[row];
    const int nterm = (int)(poff[row + 1] - p0);
    const int dp = m != nullptr ? dpos[row] : -1;
    const PT* prow = pos + p0;
    for (int q = g; q < len; q += G) sacc[q] = 0;
    T d = 0, ss = 0;
    for (int c0 = lb; c0 < le; c0 += NE) {
        const int nt = min(NE, le - c0);  // uniform across the group
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
            const int u = e * G + g;
            const int t = c0 + u;
            if (u < nt) {
                T lv;
                if (lin != nullptr) {
                    const double x = lin[t];
                    if (lout64 != nullptr) lout64[t] = x;
                    if (loutT != nullptr) loutT[t] = (T)x;
                    if (dslot != nullptr) {  // straight into the diagonal storage of L
                        const size_t q = (size_t)dslot[t] * (size_t)dn + (size_t)row;
                        dout64[q] = x;
                        if (doutT != nullptr) doutT[q] = (T)x;
                    }
                    lv = (T)x;
                } else {
                    lv = Lval[t];
                }
                const int to = Ltof[t];
                const int tn = t + 1 < le ? (int)Ltof[t + 1] : nterm;
                elv[u] = lv;
                WfEnt w;
                w.bs = Lbst[t];
                w.to = to;
                w.len = tn - to;
                w.pad = 0;
                ent[u] = w;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (m != nullptr)
            for (int u = 0; u < nt; ++u) {  // the row's squares in column order
                const T a = elv[u];
                if (c0 + u == dp) d = a;
                ss = ss + a * a;
            }
        // Batches of WF_AHEAD entries, double-buffered: the terms of the next batch are
        // loaded before the current batch is added.  Each lane loads TPL terms of every
        // entry of a batch (g, and g + G with TPL = 2), so B rows of up to TPL G terms
        // need no further round trip; TPL = 2 pays for it with half the entries per batch.
        constexpr int WF_AHEAD = WF_LOADS / TPL;
        int up[WF_AHEAD], ul[WF_AHEAD], uq[WF_AHEAD];
        T bv[WF_AHEAD], bw[WF_AHEAD];
        auto load = [&](int u0, int (&qp)[WF_AHEAD], int (&ql)[WF_AHEAD], T (&qv)[WF_AHEAD], int (&qq)[WF_AHEAD],
                        T (&qw)[WF_AHEAD]) {
#pragma unroll
            for (int i = 0; i < WF_AHEAD; ++i) {  // first 2G terms of each entry, in flight together
                const int u = u0 + i < nt ? u0 + i : nt - 1;
                const WfEnt w = ent[u];
                ql[i] = u0 + i < nt ? w.len : 0;
                if (g < ql[i]) {
                    qp[i] = (int)prow[w.to + g];
                    qv[i] = Bval[w.bs + g];
                }
                if (TPL > 1 && g + G < ql[i]) {
                    qq[i] = (int)prow[w.to + g + G];
                    qw[i] = Bval[w.bs + g + G];
                }
            }
        };
        load(0, up, ul, bv, uq, bw);
        for (int u0 = 0; u0 < nt; u0 += WF_AHEAD) {
            int up2[WF_AHEAD], ul2[WF_AHEAD], uq2[WF_AHEAD];
            T bv2[WF_AHEAD], bw2[WF_AHEAD];
            if (u0 + WF_AHEAD < nt) load(u0 + WF_AHEAD, up2, ul2, bv2, uq2, bw2);  // uniform across the group
#pragma unroll
            for (int i = 0; i < WF_AHEAD; ++i) {
                if (ul[i] == 0) continue;  // uniform across the group
                const T lv = elv[u0 + i];
                if (g < ul[i] && up[i] < len) sacc[up[i]] = sacc[up[i]] + lv * bv[i];
                if (TPL > 1 && g + G < ul[i] && uq[i] < len) sacc[uq[i]] = sacc[uq[i]] + lv * bw[i];
                if (ul[i] > TPL * G) {  // rows of B longer than TPL G
                    const WfEnt w = ent[u0 + i];
                    for (int k = g + TPL * G; k < ul[i]; k += G) {
                        const int p = (int)prow[w.to + k];
                        const T b = Bval[w.bs + k];
                        if (p < len) sacc[p] = sacc[p] + lv * b;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < WF_AHEAD; ++i) {
                up[i] = up2[i];
                ul[i] = ul2[i];
                bv[i] = bv2[i];
                uq[i] = uq2[i];
                bw[i] = bw2[i];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    for (int q = g; q < len; q += G) Cval[sb + q] = sacc[q];
    if (m == nullptr) return;
    const T mi = (kind == 1) ? d / ss : omega / d;
    if (g == 0) m[row] = mi;
    if (Qval == nullptr || dp < 0) return;
    // Q = P - M (A P): row i of P is the B row of the diagonal entry, whose terms' positions
    // place it in the C row
    const int dbs = Lbst[dp], dto = Ltof[dp];
    const int dlen = (dp + 1 < le ? (int)Ltof[dp + 1] : nterm) - dto;
    for (int q = g; q < len; q += G) sacc[q] = -mi * sacc[q];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int k = g; k < dlen; k += G) {
        const int p = (int)prow[dto + k];
        if (p < len) sacc[p] = sacc[p] + Bval[dbs + k];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int q = g; q < len; q += G) Qval[sb + q] = sacc[q];
}

// ------------------------------------------------------------------ owner form
//
// Small products (the coarse levels, and every level of a small problem) are bound by the
// chain of dependent steps along their longest rows, not by bytes: the position-map form
// stages a chunk of L entries, waits for a batch of B terms, and adds the terms through LDS
// one L entry after another.  Here lane g of a row's G lanes owns the positions g, g + G, ...
// of the C row: for an L entry it reads which entry of the B row falls there (one byte,
// cached at setup) and that entry's value.  Each sum takes its terms in the order of the L
// row, as the row-by-row product does.  Loads are unconditional, at clamped places: with a
// branch per load these kernels were bound by their instructions.
//   k_galerkin_own1: G lanes per row, the sums in registers.
//   k_galerkin_own: a workgroup per row.  Its S groups of G lanes form the products of U
//     entries each into LDS (0 for an absent term) and the first group adds each position's
//     in order: a sum that starts from +0 is never -0, so adding the +0 of an absent term
//     changes nothing.
// Measured (position-map form / k_galerkin_own / k_galerkin_own1): R (A P) of 102 rows 35.4 /
// 14.5 / 22.4 us, of 559 rows 48.6 / 24.5 / 32.9, of 1527 rows 40.5 / 33.8 / 34.4, of 4554
// rows 47.6 / 84.9 / 71.5; A P of 1080 rows 62.7 / 27.0 / 32.2, of 3109 rows 31.9 / 20.2 /
// 14.0, of 10086 rows 42.9 / 99 / 72.8 (times with about 5 us of event overhead).

// G lanes alone per row, their sums in registers: for rows enough to fill the device without
// splitting them.
template <typename T, int G, int K>
__global__ __launch_bounds__(TPB) void k_galerkin_own1(int nrows, int W, int last_b, const int* __restrict__ Lptr,
                                                       const T* __restrict__ Lval, const int* __restrict__ Lbst,
                                                       const T* __restrict__ Bval, const int* __restrict__ Cptr,
                                                       T* __restrict__ Cval, const uint8_t* __restrict__ inv,
                                                       const int* __restrict__ dpos, int kind, T omega,
                                                       T* __restrict__ m, T* __restrict__ Qval) {
    constexpr int U = 8;
    const int g = threadIdx.x & (G - 1);
    const int row = (xcd_block() * TPB + (int)threadIdx.x) / G;
    if (row >= nrows) return;
    const int lb = Lptr[row], nl = Lptr[row + 1] - lb;
    const int sb = Cptr[row], len = Cptr[row + 1] - sb;
    const int dp = m != nullptr ? dpos[row] - lb : -1;
    const T* Lv = Lval + lb;
    const int* Lb = Lbst + lb;
    const uint8_t* iv = inv + (size_t)lb * W;
    T acc[K], d = 0, ss = 0;
    int pos[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        acc[k] = 0;
        pos[k] = min(g + k * G, W - 1);
    }
    T lv[U];
    int bs[U], jj[U][K];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = min(c0 + u, nl - 1);
            lv[u] = Lv[t];
            bs[u] = Lb[t];
#pragma unroll
            for (int k = 0; k < K; ++k) jj[u][k] = iv[t * W + pos[k]];
        }
    };
    if (nl > 0) fetch(0);
    for (int c0 = 0; c0 < nl; c0 += U) {
        T bv[U][K], lc[U];
        bool on[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lc[u] = lv[u];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                on[u][k] = jj[u][k] > 0 && c0 + u < nl;
                bv[u][k] = Bval[min(bs[u] + max(jj[u][k] - 1, 0), last_b)];
            }
        }
        if (c0 + U < nl) fetch(c0 + U);  // in flight while this batch is added
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] = on[u][k] ? acc[k] + lc[u] * bv[u][k] : acc[k];
            if (m != nullptr && c0 + u < nl) {  // the row's squares in column order
                if (c0 + u == dp) d = lc[u];
                ss = ss + lc[u] * lc[u];
            }
        }
    }
    const T mi = (kind == 1) ? d / ss : omega / d;
    if (m != nullptr && g == 0) m[row] = mi;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = g + k * G;
        if (p >= len) continue;
        Cval[sb + p] = acc[k];
        if (m == nullptr || Qval == nullptr || dp < 0) continue;
        const int j = iv[dp * W + p];  // Q = P - M (A P): row i of P is the diagonal entry's B row
        const T q = -mi * acc[k];
        Qval[sb + p] = j > 0 ? q + Bval[Lb[dp] + j - 1] : q;
    }
}

template <typename T, int G, int K, int U>
__global__ __launch_bounds__(TPB) void k_galerkin_own(int nrows, int W, int last_b, const int* __restrict__ Lptr,
                                                      const T* __restrict__ Lval, const int* __restrict__ Lbst,
                                                      const T* __restrict__ Bval, const int* __restrict__ Cptr,
                                                      T* __restrict__ Cval, const uint8_t* __restrict__ inv,
                                                      const int* __restrict__ dpos, int kind, T omega,
                                                      T* __restrict__ m, T* __restrict__ Qval) {
    constexpr int S = TPB / G, E = S * U;  // groups, entries per chunk
    extern __shared__ __align__(16) unsigned char own_lds[];
    T* prod = reinterpret_cast<T*>(own_lds);  // two chunks of products, then of L values
    T* elv = prod + (size_t)2 * E * W;
    const int g = threadIdx.x & (G - 1), sub = threadIdx.x / G;
    const int row = blockIdx.x;
    const int lb = Lptr[row], nl = Lptr[row + 1] - lb;
    const int sb = Cptr[row], len = Cptr[row + 1] - sb;
    const int dp = m != nullptr ? dpos[row] - lb : -1;
    const T* Lv = Lval + lb;
    const int* Lb = Lbst + lb;
    const uint8_t* iv = inv + (size_t)lb * W;
    T acc[K], d = 0, ss = 0;
    int pos[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        acc[k] = 0;
        pos[k] = min(g + k * G, W - 1);
    }
    T lv[U];
    int bs[U], jj[U][K];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = min(c0 + sub * U + u, nl - 1);
            lv[u] = Lv[t];
            bs[u] = Lb[t];
#pragma unroll
            for (int k = 0; k < K; ++k) jj[u][k] = iv[t * W + pos[k]];
        }
    };
    if (nl > 0) fetch(0);
    int buf = 0;
    for (int c0 = 0; c0 < nl; c0 += E, buf ^= 1) {
        T bv[U][K], lc[U];
        bool on[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lc[u] = lv[u];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                on[u][k] = jj[u][k] > 0;
                bv[u][k] = Bval[min(bs[u] + max(jj[u][k] - 1, 0), last_b)];
            }
        }
        if (c0 + E < nl) fetch(c0 + E);  // in flight while this chunk is added
        T* pb = prod + (size_t)buf * E * W;
        T* eb = elv + buf * E;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = sub * U + u;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const T x = on[u][k] ? lc[u] * bv[u][k] : T(0);
                if (g + k * G < W) pb[e * W + g + k * G] = x;
            }
            if (m != nullptr && g == 0) eb[e] = lc[u];
        }
        __syncthreads();  // (the other buffer is written next: its readers passed this point)
        if (sub == 0) {
            const int ne = min(E, nl - c0);
            for (int e0 = 0; e0 < ne; e0 += U) {
                T x[U][K];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < K; ++k) x[u][k] = pb[(e0 + u) * W + pos[k]];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < K; ++k) acc[k] = e0 + u < ne ? acc[k] + x[u][k] : acc[k];
            }
            if (m != nullptr)
                for (int e = 0; e < ne; ++e) {  // the row's squares in column order
                    const T v = eb[e];
                    if (c0 + e == dp) d = v;
                    ss = ss + v * v;
                }
        }
    }
    if (sub != 0) return;
    const T mi = (kind == 1) ? d / ss : omega / d;
    if (m != nullptr && g == 0) m[row] = mi;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = g + k * G;
        if (p >= len) continue;
        Cval[sb + p] = acc[k];
        if (m == nullptr || Qval == nullptr || dp < 0) continue;
        const int j = iv[dp * W + p];  // Q = P - M (A P): row i of P is the diagonal entry's B row
        const T q = -mi * acc[k];
        Qval[sb + p] = j > 0 ? q + Bval[Lb[dp] + j - 1] : q;
    }
}

// Index of each row's diagonal entry (-1 if absent).
__global__ __launch_bounds__(TPB) void k_diag_index(int n, const int* __restrict__ ptr, const int* __restrict__ col,
                                                    int* __restrict__ dpos) {
    const int i = xcd_block() * TPB + threadIdx.x;
    if (i >= n) return;
    int lo = ptr[i], hi = ptr[i + 1];
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col[mid] < i)
            lo = mid + 1;
        else
            hi = mid;
    }
    dpos[i] = (lo < ptr[i + 1] && col[lo] == i) ? lo : -1;
}

bool galerkin_terms_fit(int64_t max_row) { return max_row <= WF_TERMS_MAX; }

void launch_diag_index(const Csr& A, int32_t* dpos, hipStream_t s) {
    if (A.nrows == 0) return;
    k_diag_index<<<row_blocks(A.nrows, 1), TPB, 0, s>>>(A.nrows, A.ptr, A.col, dpos);
    HIP_LAUNCH_CHECK();
}

#define AMG_WITH_GS1(g, ...)                                                \
    do {                                                                    \
        switch (g) {                                                        \
            case 4: { constexpr int GG = 4; __VA_ARGS__; } break;           \
            case 8: { constexpr int GG = 8; __VA_ARGS__; } break;           \
            case 16: { constexpr int GG = 16; __VA_ARGS__; } break;         \
            case 32: { constexpr int GG = 32; __VA_ARGS__; } break;         \
            case 64: { constexpr int GG = 64; __VA_ARGS__; } break;         \
            default: throw Fail{AMG_ERR_ARG, "unsupported Galerkin lane count"}; \
        }                                                                   \
    } while (0)

// Launch shape of the position-map form for C = L B from its sizes (rows and entries of L,
// terms, the longest C row): cap = the longest C row rounded up to a multiple of 8; TPL =
// 2 terms per lane and entry for products of at least TPL2_MIN_ROWS rows, half as many where
// the L rows are long (more rows per wavefront, fewer B rows left to a second round trip; measured at 128^3: level-0 A P
// 286 against 315 us, R (A P) 215 against 241 us), else 1 (small products want every lane
// on few rows); G = the power of two in [4, 64] nearest above the mean number of terms
// per L entry over TPL (the mean referenced B row length, so that most B rows take one
// pass of the group), or at least an eighth of the mean L row length, raised until a
// block's LDS (TPB / G rows of cap FP64 accumulators and the staged L entries) is within
// WF_SMEM_MAX.  {0, ...}: the rows are too long for the form (lane-group kernels).
// gforce and tforce force G and TPL where the LDS allows.  The position map itself is
// built by the caller.
// Long L rows gain from half as many rows on (27-point 112^3, rows of 50 entries: R (A P) of
// 49888 rows 421 -> 371 us, A_1 P_1 123 -> 96), shorter ones don't (two-fluid 72^3, 34137 rows
// of 38 and 33: 52 -> 55, 40 -> 42).
constexpr int32_t TPL2_MIN_ROWS = 1 << 16;
constexpr double TPL2_LONG = 44.0;
// Products of fewer rows (and L rows of more than a chunk) take at least 8 lanes per row: 4
// leave the device half empty (A P of 24078 rows 40 -> 25 us; of 46669 rows 47 us both ways).
constexpr int32_t LANES8_ROWS = 1 << 15;
constexpr int64_t OWN_BYTES = 64 << 20;
constexpr int OWN_LEN_MAX = 248;  // (own_smem with four entries per group: 63744 bytes in FP64)
constexpr int64_t OWN_ROWS_WG = 1024, OWN_ROWS = 4096;
GalShape pick_galerkin_shape(int32_t nrows, int64_t nnzL, int64_t terms, int maxlen, int gforce, int tforce) {
    if (maxlen > WF_CAP_MAX) return {};
    const double mean_b = nnzL > 0 ? (double)terms / (double)nnzL : 1.0;
    const int cap = std::max(8, (maxlen + 7) / 8 * 8);
    const double mean_l = nrows > 0 ? (double)nnzL / (double)nrows : 1.0;
    const int tpl = (tforce == 1 || tforce == 2) ? tforce
                    : nrows >= TPL2_MIN_ROWS || (nrows >= TPL2_MIN_ROWS / 2 && mean_l >= TPL2_LONG) ? 2 : 1;
    int G = 4;
    while (G < 64 && G * tpl < mean_b) G <<= 1;
    while (G < 64 && 8 * G <= mean_l) G <<= 1;  // long L rows: wider groups, fewer chunks
    while (G < 8 && nrows <= LANES8_ROWS && mean_l > 2.0 * G) G <<= 1;
    if (gforce == 4 || gforce == 8 || gforce == 16 || gforce == 32 || gforce == 64) G = gforce;
    const int epl = mean_l > 2.0 * G ? 4 : 2;
    auto smem = [&](int g) {
        return (size_t)(TPB / g) * ((size_t)cap * sizeof(double) + (size_t)epl * g * (sizeof(double) + sizeof(WfEnt)));
    };
    while (G < 64 && smem(G) > WF_SMEM_MAX) G <<= 1;
    if (smem(G) > WF_SMEM_MAX) return {};
    GalShape gs;
    gs.g = G;
    gs.cap = cap;
    gs.epl = epl;
    gs.wide = maxlen > 255 ? 1 : 0;
    gs.tpl = tpl;
    return gs;
}

bool pick_owner_form(int64_t nrows, int64_t nnzL, const SymSizes& z, GalShape& gs) {
    if (z.max_b > 254 || z.maxlen > OWN_LEN_MAX || z.maxlen == 0 || nrows == 0) return false;
    const int w = (z.maxlen + 7) / 8 * 8;
    int G = 8;
    while (G < 64 && G < z.maxlen) G <<= 1;
    if (nnzL * w > OWN_BYTES || nrows > OWN_ROWS) return false;
    gs.own = G;
    gs.own_rows = nrows <= OWN_ROWS_WG ? TPB : G;
    gs.inv_w = w;
    return true;
}

template <typename T>
static size_t acc_smem(const GalShape& gs) {
    return (size_t)(TPB / gs.g) * ((size_t)gs.cap * sizeof(T) + (size_t)gs.epl * gs.g * (sizeof(T) + sizeof(WfEnt)));
}

// Launches the position-map kernel for one product with the shape's template arguments.
template <typename T>
static void launch_pos(const Csr& L, const Csr& B, const Csr& C, const GalShape& gs, int kind, double omega, T* m,
                       T* q, const double* lin, double* lout64, T* loutT, hipStream_t s, const Dia* dia = nullptr) {
    const size_t sm = acc_smem<T>(gs);
    const int* dp = m != nullptr ? gs.dpos : nullptr;
    const uint8_t* dslot = dia != nullptr ? dia->slot : nullptr;
    double* d64 = dia != nullptr ? dia->val : nullptr;
    T* dT = nullptr;
    if constexpr (!std::is_same<T, double>::value)
        if (dia != nullptr) dT = dia->val32;
#define AMG_POS_LAUNCH(PT, EPL, TPL)                                                                      \
    AMG_WITH_GS1(gs.g, (k_galerkin_pos<T, GG, PT, EPL, TPL><<<row_blocks(L.nrows, GG), TPB, sm, s>>>(      \
                           L.nrows, gs.cap, L.ptr, L.v<T>(), gs.bst, gs.tof, B.v<T>(), C.ptr, C.v<T>(),     \
                           (const PT*)gs.pos, gs.off, dp, kind, (T)omega, m, q, lin, lout64, loutT, dslot,  \
                           (int64_t)L.nrows, d64, dT)))
#define AMG_POS_LAUNCH_T(PT, EPL)                  \
    do {                                           \
        if (gs.tpl == 2) AMG_POS_LAUNCH(PT, EPL, 2); \
        else AMG_POS_LAUNCH(PT, EPL, 1);           \
    } while (0)
    if (gs.wide) {
        if (gs.epl == 4) AMG_POS_LAUNCH_T(uint16_t, 4);
        else AMG_POS_LAUNCH_T(uint16_t, 2);
    } else {
        if (gs.epl == 4) AMG_POS_LAUNCH_T(uint8_t, 4);
        else AMG_POS_LAUNCH_T(uint8_t, 2);
    }
#undef AMG_POS_LAUNCH_T
#undef AMG_POS_LAUNCH
    HIP_LAUNCH_CHECK();
}

template <typename T>
static void launch_own(const Csr& L, const Csr& B, const Csr& C, const GalShape& gs, int kind, double omega, T* m,
                       T* q, hipStream_t s) {
    const int* dp = m != nullptr ? gs.dpos : nullptr;
    const int k = (gs.inv_w + gs.own - 1) / gs.own;
    auto go = [&](auto kern, unsigned nbk, size_t smem) {
        kern<<<nbk, TPB, smem, s>>>(L.nrows, gs.inv_w, (int)(B.nnz - 1), L.ptr, L.v<T>(), gs.bst, B.v<T>(), C.ptr,
                                    C.v<T>(), gs.inv, dp, kind, (T)omega, m, q);
    };
    if (gs.own_rows == TPB) {
        const int u = own_entries(gs.inv_w);
        const size_t sm = (size_t)own_smem(gs.own, gs.inv_w, u, sizeof(T));
        if (sm > OWN_SMEM_MAX) throw Fail{AMG_ERR_ARG, "row too long for the owner form"};
        const unsigned nbk = (unsigned)L.nrows;
        if (gs.own == 8) go(k_galerkin_own<T, 8, 1, 8>, nbk, sm);
        else if (gs.own == 16) go(k_galerkin_own<T, 16, 1, 8>, nbk, sm);
        else if (gs.own == 32) go(k_galerkin_own<T, 32, 1, 8>, nbk, sm);
        else if (k == 1) go(k_galerkin_own<T, 64, 1, 8>, nbk, sm);
        else if (k == 2) go(k_galerkin_own<T, 64, 2, 8>, nbk, sm);
        else go(k_galerkin_own<T, 64, 4, 4>, nbk, sm);
    } else {
        const unsigned nbk = row_blocks(L.nrows, gs.own);
        if (gs.own == 8) go(k_galerkin_own1<T, 8, 1>, nbk, 0);
        else if (gs.own == 16) go(k_galerkin_own1<T, 16, 1>, nbk, 0);
        else if (gs.own == 32) go(k_galerkin_own1<T, 32, 1>, nbk, 0);
        else if (k == 1) go(k_galerkin_own1<T, 64, 1>, nbk, 0);
        else if (k == 2) go(k_galerkin_own1<T, 64, 2>, nbk, 0);
        else go(k_galerkin_own1<T, 64, 4>, nbk, 0);
    }
    HIP_LAUNCH_CHECK();
}

template <typename T>
void launch_smoother_diag(const Csr& A, int kind, double omega, T* m, hipStream_t s) {
    k_smoother_diag<T><<<row_blocks(A.nrows, 1), TPB, 0, s>>>(A.nrows, A.ptr, A.col, A.v<T>(), kind, (T)omega, m);
    HIP_LAUNCH_CHECK();
}

// AP = A P; with m != nullptr also the smoother diagonal of A and, with q, the values of
// Q = (I - M A) P on AP's pattern; and with ain != nullptr
// the values of A are taken from ain (FP64) and stored on the way: into the diagonal
// storage `dia` when one is given (its FP64 and, in mixed precision, FP32 arrays), else
// into A's CSR value arrays.  Only the position-map form fuses these; it returns true when
// it did (m and the values written).
template <typename T>
bool launch_galerkin_ap(const Csr& A, const Csr& P, const Csr& AP, int g, GalShape gs, int kind, double omega, T* m,
                        const double* ain, hipStream_t s, const Dia* dia, T* q) {
    if (gs.own > 0) {
        if (ain != nullptr) throw Fail{AMG_ERR_ARG, "owner-form product cannot take new values of A"};
        launch_own<T>(A, P, AP, gs, kind, omega, m, q, s);
        return true;
    }
    if (gs.g > 0) {
        const bool to_dia = dia != nullptr && ain != nullptr;
        double* out64 = (!to_dia && ain != nullptr && ain != A.val) ? A.val : nullptr;
        T* outT = nullptr;
        if constexpr (!std::is_same<T, double>::value) outT = (!to_dia && ain != nullptr) ? A.v<T>() : nullptr;
        launch_pos<T>(A, P, AP, gs, kind, omega, m, q, ain, out64, outT, s, to_dia ? dia : nullptr);
        return true;
    }
    if (ain != nullptr) return false;  // the caller ingests the values first, then calls again
    AMG_WITH_G(g, k_galerkin_ap<G, T><<<row_blocks(A.nrows, G), TPB, 0, s>>>(
                      A.nrows, A.ptr, A.col, A.v<T>(), P.ptr, P.col, P.v<T>(), AP.ptr, AP.col, AP.v<T>()));
    HIP_LAUNCH_CHECK();
    return false;
}

template <typename T>
void launch_galerkin_rap(const Csr& R, const Csr& AP, const Csr& Ac, int g, GalShape gs, hipStream_t s) {
    if (gs.own > 0) {
        launch_own<T>(R, AP, Ac, gs, 0, 0.0, (T*)nullptr, (T*)nullptr, s);
        return;
    }
    if (gs.g > 0) {
        launch_pos<T>(R, AP, Ac, gs, 0, 0.0, (T*)nullptr, (T*)nullptr, nullptr, nullptr, (T*)nullptr, s);
        return;
    }
    AMG_WITH_G(g, k_galerkin_rap<G, T><<<row_blocks(R.nrows, G), TPB, 0, s>>>(
                      R.nrows, R.ptr, R.col, R.v<T>(), AP.ptr, AP.col, AP.v<T>(), Ac.ptr, Ac.col, Ac.v<T>()));
    HIP_LAUNCH_CHECK();
}

template bool launch_galerkin_ap<double>(const Csr&, const Csr&, const Csr&, int, GalShape, int, double, double*,
                                         const double*, hipStream_t, const Dia*, double*);
template bool launch_galerkin_ap<float>(const Csr&, const Csr&, const Csr&, int, GalShape, int, double, float*,
                                        const double*, hipStream_t, const Dia*, float*);
template void launch_galerkin_rap<double>(const Csr&, const Csr&, const Csr&, int, GalShape, hipStream_t);
template void launch_galerkin_rap<float>(const Csr&, const Csr&, const Csr&, int, GalShape, hipStream_t);
template void launch_smoother_diag<double>(const Csr&, int, double, double*, hipStream_t);
template void launch_smoother_diag<float>(const Csr&, int, double, float*, hipStream_t);

}  // namespace amgmi
