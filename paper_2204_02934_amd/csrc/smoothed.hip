// smoothed.hip -- smoothed aggregation on gfx950: the damped-Jacobi
// prolongator P = (I - omega D^-1 A) P_tent of an aggregation and the coarse
// operator P^T A P (the multigrid setup Section VI-E runs on these
// aggregates smooths its prolongator; the paper prints no formula).
//
// P_tent[i][agg i] = 1/sqrt(n_a) as in galerkin.hip.  Three sparse products,
// each with one fixed sequence of roundings:
//   P[i][a]  = (1{a = agg i} - (omega / d_i) * S) / sqrt(n_a), S = the sum of
//              A_ij over j in N[i] with agg j = a, from 0.0, the diagonal
//              first, then row i's entries in CSR order;
//   AP[i][b] = the sum of A_ij * P[j][b] over j in N[i] (i first, then row
//              i's entries in CSR order), from 0.0, absent P[j][b] skipped;
//   Ac[a][b] = the sum of P[i][a] * AP[i][b] over the rows i holding
//              P[i][a], in increasing i, from 0.0, absent AP[i][b] skipped.
// Patterns are structural, columns ascending: P row i = the distinct
// aggregates of N[i]; AP row i = the union of the P rows of N[i]; Ac row a =
// the union of the AP rows i with P[i][a].
//
// Structure (symbolic) kernels.  A row's columns are the distinct ones among its
// candidates: each source row's columns.  A P row of up to 16 candidates is
// sorted in registers (k_p_rows).  Other rows collect their columns in an LDS
// hash set: first a group of lanes per row with a small set (k_sym_group; 16
// lanes, four rows per wavefront, or all 64 for the coarse rows), then, for the
// rows with too many columns, one wavefront with a set for kMidMax and at last
// one for kSetMax columns (k_sym; each takes more LDS, so fewer rows are in
// flight).  Which of the later passes have anything to do is read back with a
// pass's total.
// P's rows have their place at once (a row has at most its entries and one), so
// one pass writes them to a spare buffer and they are then copied; AP and Ac
// take a count pass and, after a prefix sum, a pass that fills columns and
// values together (k_fill_values).  A row with more than kSetMax distinct
// columns sets an error flag.
// Value (numeric) kernels: P one group of lanes per row (k_p_values); the rows
// of AP and Ac past the first pass, one group per row (k_row_values).  Each
// entry folds its terms one after the other in the stated order, each term one
// rounded product (the file is compiled without contraction into fused
// multiply-adds).
#include <algorithm>

#include "internal.h"
#include "lanes.h"
#include "rowset.h"

#pragma clang fp contract(off)

namespace mis2 {

namespace {

constexpr int kSetMax = 2048;       // distinct columns a row may have
constexpr int kMidMax = 512;        // and in the second of the three sets
constexpr int kSThreads = 128;      // second and third pass: 2 wavefronts per workgroup
constexpr int kSWaves = kSThreads / 64;
constexpr int kSBlocks = 2048;      // about what is resident at once (second pass)
constexpr int kSU = 8;              // candidates per lane whose loads go out together

// most candidates of a row for a group of 16 and of 64 lanes
constexpr uint32_t kFew = 2048, kMany = 16384;
// most columns of a row whose values k_fill_values computes (AP, Ac)
constexpr uint32_t kApMost = 47, kCMost = 159;

int grid_of_s(int64_t work, int per_block, int cap) {
    const int64_t b = (work + per_block - 1) / per_block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

// The three kinds of rows.  For output row r, sources(r) gives the source
// rows in order; each source s contributes the columns col_of(s, k) for k in
// [0, len(s)).
//   kP:  sources = i, then i's neighbours; a source j contributes agg[j].
//   kAP: sources = i, then i's neighbours; a source j contributes P row j.
//   kC:  sources = the rows holding P[i][a] (members of R_a, increasing i);
//        a source i contributes AP row i.
enum { kP = 0, kAP = 1, kC = 2 };

// Classes of rows: which pass has the row.
constexpr uint8_t kClsGroup = 0, kClsMid = 1, kClsRegs = 2, kClsLarge = 3;

struct SymArgs {
    int64_t rows;
    // the graph
    const int64_t *row_ptr;
    const int32_t *col;
    const int32_t *agg;
    // source CSR (P for kAP, AP for kC)
    const int64_t *sptr;
    const int32_t *scol;
    // kC: the members of R_a as P entry indices, and the row of each P entry
    const int64_t *moff;
    const int32_t *members;
    const int32_t *prow_of;
    // output
    uint32_t *count;          // count pass
    const int64_t *out_ptr;   // fill pass
    int32_t *out_col;
    uint32_t *err;            // |= kSymBad, kSymMid, kSymLarge
    uint8_t *cls;             // [rows] kClsGroup, ...
    int32_t *spare;           // kP, count pass: row r also at spare[row_ptr[r] + r] (or null)
};

// Source rows of output row r: [first, last) of an index range, and the row
// id of source index t.
template <int K>
__device__ __forceinline__ void source_range(const SymArgs &a, int64_t r, int64_t &first,
                                             int64_t &last) {
    if (K == kC) {
        first = a.moff[r];
        last = a.moff[r + 1];
    } else {
        first = a.row_ptr[r] - 1;  // index first - 1 ... stands for r itself
        last = a.row_ptr[r + 1];
    }
}

template <int K>
__device__ __forceinline__ int64_t source_row(const SymArgs &a, int64_t r, int64_t t) {
    if (K == kC) return a.prow_of[a.members[t]];
    return t < a.row_ptr[r] ? r : (int64_t)a.col[t];
}

// Collects the columns of output row r; false when there are too many.
template <int K, int U, int G, int CAP, int LIM>
__device__ __forceinline__ bool collect(RowSet<G, CAP, LIM> &S, int lane, const SymArgs &a,
                                        int64_t r, uint32_t maxc) {
    int64_t first, last;
    source_range<K>(a, r, first, last);
    if constexpr (K == kP) {
        // one candidate per source: the row itself, then its entries
        if (lane == 0) row_put(S, a.agg[r]);
        const int64_t b = first + 1;
        return row_gather<G, CAP, LIM, U>(
            S, lane, 0, 1, maxc,
            [&](int64_t, int64_t &rs, int64_t &d) {
                rs = b;
                d = last - b;
            },
            [&](int64_t j) { return a.col[j]; }, [&](int32_t x) { return a.agg[x]; });
    } else {
        return row_gather<G, CAP, LIM, U>(
            S, lane, first, last, maxc,
            [&](int64_t t, int64_t &rs, int64_t &d) {
                const int64_t q = source_row<K>(a, r, t);
                rs = a.sptr[q];
                d = a.sptr[q + 1] - rs;
            },
            [&](int64_t j) { return a.scol[j]; }, [&](int32_t x) { return x; });
    }
}

// First pass: one group of G lanes per row, LIM - 1 columns at most.  Bound, as
// the quotient's rows, by each row's chain of dependent loads and LDS steps.
// FILL = false: a.count[r] and class kClsGroup, or kClsMid for a row of more
// than `most` columns, left to the second pass; FILL = true: the rows of class
// kClsGroup at a.out_ptr[r].
template <int K, bool FILL, int G, int CAP, int LIM, int U>
__global__ __launch_bounds__(kBlock) void k_sym_group(SymArgs a, uint32_t maxc, uint32_t most) {
    constexpr int kGroups = kBlock / G;
    __shared__ RowSet<G, CAP, LIM> sets[kGroups];
    const int grp = (int)threadIdx.x / G, lane = (int)threadIdx.x % G;
    RowSet<G, CAP, LIM> &S = sets[grp];
    row_clear(S, lane, 0u, true);
    // each XCD takes one run of the rows of a step (the grid is a multiple of 8)
    const int64_t blk = (int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    for (int64_t r = blk * kGroups + grp; r < a.rows; r += (int64_t)gridDim.x * kGroups) {
        if (K == kP && a.cls[r] == kClsRegs) continue;  // k_p_rows had it
        if (FILL && a.cls[r] != kClsGroup) continue;
        const bool whole = collect<K, U>(S, lane, a, r, maxc);
        const uint32_t m = S.num;
        const bool fits = whole && (FILL || m <= most);
        if (!FILL && lane == 0) {
            a.cls[r] = fits ? kClsGroup : kClsMid;
            if (fits) a.count[r] = m;
            else if (!(*(volatile uint32_t *)a.err & kSymMid)) atomicOr(a.err, kSymMid);
        }
        int32_t *out = FILL ? a.out_col + a.out_ptr[r]
                       : K == kP && a.spare ? a.spare + a.row_ptr[r] + r : nullptr;
        if (fits && out) row_write(S, lane, m, out);
        row_clear(S, lane, m, !whole);
    }
}

// Second and third pass: the rows of class CLS, one wavefront each with a set
// for MAX columns (64 classes read at a time over rows spread across all
// wavefronts).  A row with more goes from the second to the third pass; there it
// sets the error flag.
template <int K, bool FILL, uint8_t CLS>
__global__ __launch_bounds__(kSThreads) void k_sym(SymArgs a) {
    constexpr int MAX = CLS == kClsMid ? kMidMax : kSetMax;
    using Set = RowSet<64, 2 * MAX, MAX + 1>;
    __shared__ Set sets[kSWaves];
    Set &S = sets[threadIdx.x >> 6];
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t w0 = (int64_t)blockIdx.x * kSWaves + (threadIdx.x >> 6);
    const int64_t stride = (int64_t)gridDim.x * kSWaves;
    bool clean = false;  // the table is cleared before its first row
    for (int64_t j0 = 0; w0 + j0 * stride < a.rows; j0 += 64) {
        const int64_t v = w0 + (j0 + lane) * stride;
        uint64_t mask = __ballot(v < a.rows && a.cls[v] == CLS);
        while (mask) {
            const int q = __ffsll((unsigned long long)mask) - 1;
            mask &= mask - 1;
            const int64_t r = w0 + (j0 + q) * stride;
            if (!clean) row_clear(S, lane, 0u, true);
            clean = true;
            const bool fits = collect<K, kSU>(S, lane, a, r, kNoLimit);
            const uint32_t m = S.num;
            if (!FILL && lane == 0) {
                a.count[r] = fits ? m : 0u;
                if (!fits) {
                    if (CLS == kClsMid) a.cls[r] = kClsLarge;
                    atomicOr(a.err, CLS == kClsMid ? kSymLarge : kSymBad);
                }
            }
            int32_t *out = FILL ? a.out_col + a.out_ptr[r]
                           : K == kP && a.spare ? a.spare + a.row_ptr[r] + r : nullptr;
            if (fits && out) row_write(S, lane, m, out);
            row_clear(S, lane, m, !fits);
        }
    }
}

// The rows of P of at most G candidates (fewer than G entries), one group of G
// lanes each: lane 0 holds the row's own aggregate, lane k the k-th entry's; a
// bitonic network of register moves sorts them, and the first of each run of
// equal ones is kept.  Nothing in LDS, and no lane idle on a stencil's rows: one
// wavefront and a hash set per row took 194 + 286 us to count and to fill the
// 7-point 100^3 grid's P.
template <int J>
__device__ __forceinline__ uint32_t p_step(uint32_t x, int lane, int k) {
    const uint32_t y = lane_xor<J>(x);
    // ascending where bit k of the lane is clear
    return ((lane & J) == 0) == ((lane & k) == 0) ? min(x, y) : max(x, y);
}

template <bool FILL, int G>
__global__ __launch_bounds__(kBlock) void k_p_rows(SymArgs a) {
    static_assert(G == 8 || G == 16, "k_p_rows: 8 or 16 lanes");
    const int lane = (int)(threadIdx.x & (G - 1)), wl = (int)(threadIdx.x & 63u);
    // whole wavefronts stay in the loop together
    const int64_t w0 = (int64_t)blockIdx.x * (kBlock / G) + (threadIdx.x >> 6) * (64 / G);
    for (int64_t g0 = w0; g0 < a.rows; g0 += (int64_t)gridDim.x * (kBlock / G)) {
        const int64_t r = g0 + wl / G;
        const int64_t b = r < a.rows ? a.row_ptr[r] : 0;
        const int64_t d = r < a.rows ? a.row_ptr[r + 1] - b : G;
        const bool has = d < G && lane <= d;
        uint32_t x = 0xFFFFFFFFu;  // past every id
        if (has) x = (uint32_t)a.agg[lane ? (int64_t)a.col[b + lane - 1] : r];
        x = p_step<1>(x, lane, 2);
        x = p_step<2>(x, lane, 4);
        x = p_step<1>(x, lane, 4);
        x = p_step<4>(x, lane, 8);
        x = p_step<2>(x, lane, 8);
        x = p_step<1>(x, lane, 8);
        if constexpr (G == 16) {
            x = p_step<8>(x, lane, 16);
            x = p_step<4>(x, lane, 16);
            x = p_step<2>(x, lane, 16);
            x = p_step<1>(x, lane, 16);
        }
        const uint32_t prev = from_prev(x);
        const bool keep = x != 0xFFFFFFFFu && (lane == 0 || x != prev);
        const uint64_t heads = __ballot(keep) >> (wl & ~(G - 1)) & ((1ull << G) - 1);
        if (!FILL && lane == 0 && r < a.rows) a.cls[r] = d < G ? kClsRegs : kClsGroup;
        if (r < a.rows && d < G) {
            if (!FILL && lane == 0) a.count[r] = (uint32_t)__popcll(heads);
            int32_t *out = FILL ? a.out_col + a.out_ptr[r] : a.spare ? a.spare + b + r : nullptr;
            if (keep && out) out[__popcll(heads & ((1ull << lane) - 1))] = (int32_t)x;
        }
    }
}

// P's rows from the spare buffer (row r at row_ptr[r] + r) to their place, 8
// lanes each.
__global__ __launch_bounds__(kBlock) void k_p_copy(int64_t n, const int64_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ spare,
                                                   const int64_t *__restrict__ prow,
                                                   int32_t *__restrict__ pcol) {
    const int lane = (int)(threadIdx.x & 7u);
    for (int64_t r = (int64_t)blockIdx.x * (kBlock / 8) + (threadIdx.x >> 3); r < n;
         r += (int64_t)gridDim.x * (kBlock / 8)) {
        const int64_t d0 = prow[r], len = prow[r + 1] - d0, s0 = row_ptr[r] + r;
        for (int64_t k = lane; k < len; k += 8) pcol[d0 + k] = spare[s0 + k];
    }
}

// P values: one group of kPG lanes per row i, one lane per entry (i, a) of
// P's row (kPG at a time).  The row of A goes kPG entries at a time, each
// lane loading one entry's aggregate and value; the group then folds them in
// CSR order by shuffles, every lane adding the entries of its own aggregate.
constexpr int kPG = 8;

__global__ __launch_bounds__(kBlock) void k_p_values(int64_t n, const int64_t *__restrict__ row_ptr,
                                                     const int32_t *__restrict__ col,
                                                     const double *__restrict__ val,
                                                     const double *__restrict__ diag,
                                                     const int32_t *__restrict__ agg,
                                                     const uint32_t *__restrict__ size,
                                                     double omega, const int64_t *__restrict__ prow,
                                                     const int32_t *__restrict__ pcol,
                                                     double *__restrict__ pval,
                                                     int32_t *__restrict__ prow_of) {
    const int gl = (int)(threadIdx.x & (kPG - 1));
    const int64_t NG = (int64_t)gridDim.x * (kBlock / kPG);
    for (int64_t i = (int64_t)blockIdx.x * (kBlock / kPG) + threadIdx.x / kPG; i < n; i += NG) {
        const int64_t p0 = prow[i], pm = prow[i + 1] - p0;
        const int64_t rs = row_ptr[i], re = row_ptr[i + 1];
        const int32_t ai = agg[i];
        const double di = diag[i];
        for (int64_t s0 = 0; s0 < pm; s0 += kPG) {
            const bool mine = s0 + gl < pm;
            const int32_t a = mine ? pcol[p0 + s0 + gl] : -1;
            double sum = 0.0;
            if (ai == a) sum = sum + di;
            for (int64_t e0 = rs; e0 < re; e0 += kPG) {
                const int cnt = (int)min<int64_t>(kPG, re - e0);
                int32_t ag = -1;
                double v = 0.0;
                if (gl < cnt) {
                    ag = agg[col[e0 + gl]];
                    v = val[e0 + gl];
                }
                // every lane of the group runs the shuffles
                for (int t = 0; t < cnt; t++) {
                    const int32_t at = __shfl(ag, t, kPG);
                    const double vt = __shfl(v, t, kPG);
                    if (at == a) sum = sum + vt;
                }
            }
            if (mine) {
                const double w = omega / di;
                const double ind = ai == a ? 1.0 : 0.0;
                const double t = w * sum;
                const double r = ind - t;
                pval[p0 + s0 + gl] = r / sqrt((double)size[a]);
                prow_of[p0 + s0 + gl] = (int32_t)i;
            }
        }
    }
}

// AP and Ac values: one group of G lanes per output row (G = 32 for AP,
// whose rows are short, so a wavefront has two rows in flight; 64 for Ac).
// An output entry (r, b) is the sum, over the row's terms t in their stated
// order, of coef_t * S[src_t][b] (skipped where S has no such entry).  The
// row's columns go to LDS, G at a time (a slot pass); the terms go kVT at a
// time: each entry of the chunk's source rows finds its column's slot by
// binary search and writes its rounded product into a kVT x G table cleared
// to +0.0, and then every lane folds its slot's column of the table in term
// order.  An absent term reads +0.0, and adding +0.0 changes no sum that
// starts from +0.0 (such a sum is never -0.0), so the result is that of
// skipping it.  Entries of a term have distinct columns, so no two writes
// meet.
// terms per chunk: 12 leaves a 32-lane group's table small enough (14 KB per
// workgroup) for registers, not LDS, to set the occupancy (5 waves per SIMD
// against 4 at 16 terms); the sums are the same term by term for any chunk
constexpr int kVT = 12;
constexpr int kVU = 4;            // staged entries per lane per step
constexpr int kValThreads = 128;  // 2 wavefronts per workgroup

template <int G>
struct ValLds {
    double table[kVT][G];
    double coef[kVT];
    int64_t lo[kVT];        // first entry of each term's source row
    uint32_t pre[kVT + 1];  // prefix of the chunk's source row lengths
    int32_t outc[G];        // the slot pass's output columns
};

// Inclusive prefix sum over each aligned group of G lanes.
template <int G>
__device__ __forceinline__ uint32_t half_incl_scan(uint32_t x) {
    const int gl = (int)(threadIdx.x & (G - 1));
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
        const uint32_t y = __shfl_up(x, (unsigned)d, G);
        if (gl >= d) x += y;
    }
    return x;
}

// Terms of AP row i: (i, d_i), then (j, A_ij) for row i's entries in CSR order.
struct ApTerms {
    const int64_t *row_ptr;
    const int32_t *col;
    const double *val;
    const double *diag;
    struct Row {
        int64_t r, base, count;
    };
    __device__ Row row(int64_t r) const {
        const int64_t b = row_ptr[r];
        return {r, b, 1 + row_ptr[r + 1] - b};
    }
    __device__ void term(const Row &w, int64_t t, int64_t &src, double &coef) const {
        if (t == 0) {
            src = w.r;
            coef = diag[w.r];
        } else {
            src = col[w.base + t - 1];
            coef = val[w.base + t - 1];
        }
    }
};

// Terms of Ac row a: (i, P[i][a]) for the rows i holding P[i][a], increasing i.
struct CTerms {
    const int64_t *moff;
    const int32_t *members;
    const int32_t *prow_of;
    const double *pval;
    struct Row {
        int64_t base, count;
    };
    __device__ Row row(int64_t a) const {
        const int64_t b = moff[a];
        return {b, moff[a + 1] - b};
    }
    __device__ void term(const Row &w, int64_t t, int64_t &src, double &coef) const {
        const int32_t p = members[w.base + t];
        src = prow_of[p];
        coef = pval[p];
    }
};

// Stages one chunk of tc <= kVT terms (group lane t < tc holds term t's
// source row start lo, length len and coefficient cf) into the table and
// folds it into acc (group lanes < ns).  The group's lanes run it together;
// LDS accesses are ordered for the whole wavefront.
template <int G>
__device__ __forceinline__ void fold_chunk(ValLds<G> &sh, int gl, int tc, int64_t lo, uint32_t len,
                                           double cf, int ns, int32_t cmin, int32_t cmax,
                                           const int32_t *__restrict__ scol,
                                           const double *__restrict__ sval, double &acc) {
    const uint32_t incl = half_incl_scan<G>(len);
    const uint32_t E = (uint32_t)__shfl((int)incl, G - 1, G);
    if (gl < tc) {
        sh.lo[gl] = lo;
        sh.coef[gl] = cf;
        sh.pre[gl + 1] = incl;
    }
    if (gl == 0) sh.pre[0] = 0u;
    for (int t = 0; t < tc; t++) sh.table[t][gl] = 0.0;
    wave_sync();
    for (uint32_t k0 = 0; k0 < E; k0 += G * kVU) {
        // kVU entries per lane, every load issued before any is used (entries
        // past E reread entry E - 1 and are dropped)
        int tt[kVU];
        int32_t c[kVU];
        double v[kVU];
#pragma unroll
        for (int u = 0; u < kVU; u++) {
            const uint32_t k = k0 + (uint32_t)(u * G + gl);
            const uint32_t kk = k < E ? k : E - 1;
            int lo_t = 0, hi_t = tc - 1;  // the term of entry kk: last t with pre[t] <= kk
            while (lo_t < hi_t) {
                const int mid = (lo_t + hi_t + 1) >> 1;
                if (sh.pre[mid] <= kk) lo_t = mid; else hi_t = mid - 1;
            }
            const int64_t e = sh.lo[lo_t] + (int64_t)(kk - sh.pre[lo_t]);
            tt[u] = k < E ? lo_t : -1;
            c[u] = scol[e];
            v[u] = sval[e];
        }
#pragma unroll
        for (int u = 0; u < kVU; u++) {
            if (tt[u] >= 0 && c[u] >= cmin && c[u] <= cmax) {
                int l = 0, h = ns;  // its slot: the first output column >= c
                while (l < h) {
                    const int mid = (l + h) >> 1;
                    if (sh.outc[mid] < c[u]) l = mid + 1; else h = mid;
                }
                if (l < ns && sh.outc[l] == c[u]) sh.table[tt[u]][l] = sh.coef[tt[u]] * v[u];
            }
        }
    }
    wave_sync();
    if (gl < ns)
        for (int t = 0; t < tc; t++) acc = acc + sh.table[t][gl];
    wave_sync();
}

// (Only the rows past the first pass are left to it.)
template <int G, class Terms>
__global__ __launch_bounds__(kValThreads) void k_row_values(
    int64_t rows, const uint8_t *__restrict__ cls, Terms tm, const int64_t *__restrict__ sptr,
    const int32_t *__restrict__ scol, const double *__restrict__ sval,
    const int64_t *__restrict__ optr, const int32_t *__restrict__ ocol, double *__restrict__ oval) {
    static_assert(G == 32 || G == 64, "a group is half or all of a wavefront");
    __shared__ ValLds<G> sh_all[kValThreads / G];
    ValLds<G> &sh = sh_all[threadIdx.x / G];
    const int gl = (int)(threadIdx.x & (G - 1));
    const int64_t NG = (int64_t)gridDim.x * (kValThreads / G);
    for (int64_t r = (int64_t)blockIdx.x * (kValThreads / G) + threadIdx.x / G; r < rows;
         r += NG) {
        if (cls[r] == kClsGroup) continue;
        const int64_t o0 = optr[r], m = optr[r + 1] - o0;
        const typename Terms::Row w = tm.row(r);
        for (int64_t s0 = 0; s0 < m; s0 += G) {
            const int ns = (int)min<int64_t>(G, m - s0);
            const int32_t myc = gl < ns ? ocol[o0 + s0 + gl] : INT32_MAX;
            const int32_t cmin = __shfl(myc, 0, G), cmax = __shfl(myc, ns - 1, G);
            sh.outc[gl] = myc;
            double acc = 0.0;
            for (int64_t tb = 0; tb < w.count; tb += G) {
                // the source rows and coefficients of G terms, one per lane,
                // in one round of loads; each chunk takes its own by shuffles
                const int tn = (int)min<int64_t>(G, w.count - tb);
                int64_t my_lo = 0;
                uint32_t my_len = 0;
                double my_cf = 0.0;
                if (gl < tn) {
                    int64_t src;
                    tm.term(w, tb + gl, src, my_cf);
                    my_lo = sptr[src];
                    my_len = (uint32_t)(sptr[src + 1] - my_lo);
                }
                for (int c0 = 0; c0 < tn; c0 += kVT) {
                    const int tc = min(kVT, tn - c0);
                    // every lane of the group shuffles (a lane that is switched
                    // off in a shuffle cannot be read from), then lanes past tc
                    // drop it
                    const int from = c0 + (gl < tc ? gl : 0);
                    const int64_t lo = __shfl(my_lo, from, G);
                    const uint32_t len_from = (uint32_t)__shfl((int)my_len, from, G);
                    const double cf = __shfl(my_cf, from, G);
                    const uint32_t len = gl < tc ? len_from : 0u;
                    fold_chunk<G>(sh, gl, tc, lo, len, cf, ns, cmin, cmax, scol, sval, acc);
                }
            }
            if (gl < ns) oval[o0 + s0 + gl] = acc;
        }
    }
}

// Columns and values of the first pass's rows of AP and Ac together, one group
// of G lanes per row.  The row's columns are collected as in the count pass,
// ranked, written, and each one's rank kept beside its slot of the set; then the
// terms go FT at a time: their entries are dealt out over the lanes, each finds
// its column's rank through the set and writes its rounded product into an
// FT x G table cleared to +0.0, and every lane folds its column of the table in
// term order (G columns at a time; as in k_row_values, an absent term adds +0.0).
// Bound by each row's chain of loads and LDS steps with too few rows in flight
// to hide it, so AP's groups take sets of 64 slots and 4 terms at a time: 23 KB
// a workgroup and 7 waves per SIMD, 375 us on the 7-point 100^3 grid and 705 on
// the 27-point 90^3 (128 slots and 8 terms, 4 waves: 472 and 966).  Ac's rows
// keep 8 terms: 418 and 369 us (4 terms: 386 and 391).  A structure pass and a
// value pass of their own, the latter searching the row's columns for each
// entry, took 187 + 469 and 291 + 887 us for AP, 134 + 314 and 118 + 345 for Ac.
template <int G, int CAP, int LIM, int FT>
struct FillLds {
    RowSet<G, CAP, LIM> set;
    double table[FT][G];
    double coef[G];
    uint8_t rank[CAP];  // of the column in each slot of the set
};

template <int K, int G, int CAP, int LIM, int U, int FT, class Terms>
__global__ __launch_bounds__(kBlock) void k_fill_values(SymArgs a, uint32_t maxc, Terms tm,
                                                        const double *__restrict__ sval,
                                                        double *__restrict__ oval) {
    static_assert(LIM <= 256, "a rank fits a byte");
    constexpr int kGroups = kBlock / G;
    __shared__ FillLds<G, CAP, LIM, FT> all[kGroups];
    const int lane = (int)threadIdx.x % G;
    FillLds<G, CAP, LIM, FT> &F = all[threadIdx.x / G];
    RowSet<G, CAP, LIM> &S = F.set;
    row_clear(S, lane, 0u, true);
    const int64_t blk = (int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    for (int64_t r = blk * kGroups + threadIdx.x / G; r < a.rows; r += (int64_t)gridDim.x * kGroups) {
        if (a.cls[r] != kClsGroup) continue;
        const int64_t o = a.out_ptr[r];
        const bool fits = collect<K, U>(S, lane, a, r, maxc);  // as it did in the count pass
        const uint32_t m = S.num;
        for (uint32_t i = (uint32_t)lane; fits && i < m; i += (uint32_t)G) {
            const uint32_t x = S.list[i];
            uint32_t rank = 0;
            for (uint32_t y = 0; y < m; y++) rank += S.list[y] < x ? 1u : 0u;
            a.out_col[o + rank] = (int32_t)x;
            uint32_t h = qhash<CAP>(x);
            while (S.tab[h] != x) h = (h + 1) & (CAP - 1);
            F.rank[h] = (uint8_t)rank;
        }
        wave_sync();
        const typename Terms::Row w = tm.row(r);
        for (uint32_t s0 = 0; fits && s0 < m; s0 += (uint32_t)G) {
            double acc = 0.0;
            for (int64_t tb = 0; tb < w.count; tb += G) {
                const int tn = (int)min<int64_t>(G, w.count - tb);
                int64_t lo = 0;
                uint32_t len = 0;
                double cf = 0.0;
                if (lane < tn) {
                    int64_t src;
                    tm.term(w, tb + lane, src, cf);
                    lo = a.sptr[src];
                    len = (uint32_t)(a.sptr[src + 1] - lo);
                }
                const uint32_t incl = group_incl_scan<G>(len);
                if (lane == 0) S.off[0] = 0u;
                S.off[lane + 1] = incl;
                S.base[lane] = lo - (int64_t)(incl - len);
                F.coef[lane] = cf;
                for (int c0 = 0; c0 < tn; c0 += FT) {
                    const int tc = min(FT, tn - c0);
                    for (int t = 0; t < tc; t++) F.table[t][lane] = 0.0;
                    wave_sync();
                    const uint32_t q1 = S.off[c0], q2 = S.off[c0 + tc];
                    constexpr int kE = 2;  // entries per lane whose loads go out together
                    for (uint32_t q0 = q1 + (uint32_t)lane; q0 < q2; q0 += (uint32_t)(G * kE)) {
                        int t[kE];
                        int32_t c[kE];
                        double v[kE];
#pragma unroll
                        for (int k = 0; k < kE; k++) {
                            const uint32_t q = min(q0 + (uint32_t)(G * k), q2 - 1);
                            int z = c0;  // the last term with off[z] <= q (it is not empty)
#pragma unroll
                            for (int st = FT / 2; st > 0; st >>= 1)
                                if (S.off[z + st] <= q) z += st;
                            t[k] = z;
                            c[k] = a.scol[S.base[z] + (int64_t)q];
                            v[k] = sval[S.base[z] + (int64_t)q];
                        }
#pragma unroll
                        for (int k = 0; k < kE; k++) {
                            uint32_t h = qhash<CAP>((uint32_t)c[k]);
                            while (S.tab[h] != (uint32_t)c[k]) h = (h + 1) & (CAP - 1);
                            const uint32_t at = (uint32_t)F.rank[h] - s0;
                            if (at < (uint32_t)G && q0 + (uint32_t)(G * k) < q2)
                                F.table[t[k] - c0][at] = F.coef[t[k]] * v[k];
                        }
                    }
                    wave_sync();
                    for (int t = 0; t < tc; t++) acc = acc + F.table[t][lane];
                    wave_sync();
                }
            }
            if (s0 + (uint32_t)lane < m) oval[o + s0 + lane] = acc;
        }
        row_clear(S, lane, m, !fits);
    }
}

// Entries of P by column.  The columns of 64 consecutive entries are few (some
// dozen rows that couple to the same aggregates): one lane of each distinct
// column adds for all its entries, so one atomic serves them (one for every
// entry, in a count and again in a scatter pass, took 198 us on the 7-point 100^3 grid, this and
// the scatter 60).
__global__ __launch_bounds__(kBlock) void k_column_rank(int64_t n, const int32_t *__restrict__ key,
                                                        uint32_t *__restrict__ cnt,
                                                        int32_t *__restrict__ rank) {
    const int lane = (int)(threadIdx.x & 63u);
    for (int64_t v0 = (int64_t)blockIdx.x * kBlock + (threadIdx.x - lane); v0 < n;
         v0 += (int64_t)gridDim.x * kBlock) {
        const int64_t v = v0 + lane;
        const int32_t c = v < n ? key[v] : -1;
        uint64_t todo = __ballot(c >= 0), same = 0;
        int first = 0;
        while (todo) {
            const int l = __ffsll((unsigned long long)todo) - 1;
            const uint64_t eq = __ballot(c == __builtin_amdgcn_readlane(c, l));
            if (eq >> lane & 1u) {
                same = eq;
                first = l;
            }
            todo &= ~eq;
        }
        uint32_t base = 0;
        if (c >= 0 && first == lane) base = atomicAdd(&cnt[c], (uint32_t)__popcll(same));
        base = (uint32_t)__shfl((int)base, first, 64);
        if (c >= 0)
            rank[v] = (int32_t)(base + (uint32_t)__popcll(same & (lane ? ~0ull >> (64 - lane) : 0ull)));
    }
}

__global__ __launch_bounds__(kBlock) void k_column_scatter(int64_t n, const int32_t *__restrict__ key,
                                                           const int64_t *__restrict__ moff,
                                                           const int32_t *__restrict__ rank,
                                                           int32_t *__restrict__ members) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        members[moff[key[v]] + rank[v]] = (int32_t)v;
}

}  // namespace

hipError_t launch_smoothed_sym(int kind, bool fill, int64_t rows, int64_t nnz, const int64_t *row_ptr,
                               const int32_t *col, const int32_t *agg, const int64_t *sptr,
                               const int32_t *scol, const int64_t *moff, const int32_t *members,
                               const int32_t *prow_of, uint32_t *count, const int64_t *out_ptr,
                               int32_t *out_col, uint32_t *err, uint8_t *cls, int32_t *spare,
                               bool later, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    SymArgs a{rows, row_ptr, col, agg, sptr, scol, moff, members, prow_of, count, out_ptr,
              out_col, err, cls, spare};
    auto go = [&](auto kernel, int threads, int per, int cap, auto... more) {
        const int blocks = (grid_of_s(rows, per, cap) + 7) / 8 * 8;
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(threads), 0, s, a, more...);
    };
    if (kind == kP && !later) {
        // 8 lanes a row where rows are stencil rows of 7 entries or fewer
        if (nnz <= 7 * rows) {
            if (fill) go(k_p_rows<true, 8>, kBlock, kBlock / 8, 8192);
            else go(k_p_rows<false, 8>, kBlock, kBlock / 8, 8192);
        } else {
            if (fill) go(k_p_rows<true, 16>, kBlock, kBlock / 16, 8192);
            else go(k_p_rows<false, 16>, kBlock, kBlock / 16, 8192);
        }
    }
    auto passes = [&](auto group, int lanes, uint32_t maxc, uint32_t most, auto mid, auto large) {
        if (!later) {
            go(group, kBlock, kBlock / lanes, 8192, maxc, most);
            go(mid, kSThreads, kSWaves * 64, kSBlocks);
        } else {
            go(large, kSThreads, kSWaves * 64, kSBlocks);
        }
    };
    switch (kind * 2 + (fill ? 1 : 0)) {
        case 0:
            passes(k_sym_group<kP, false, 16, 128, 96, 4>, 16, kFew, 95u,
                   k_sym<kP, false, kClsMid>, k_sym<kP, false, kClsLarge>);
            break;
        case 1:
            passes(k_sym_group<kP, true, 16, 128, 96, 4>, 16, kFew, 95u, k_sym<kP, true, kClsMid>,
                   k_sym<kP, true, kClsLarge>);
            break;
        case 2:
            passes(k_sym_group<kAP, false, 16, 128, 96, 4>, 16, kFew, kApMost,
                   k_sym<kAP, false, kClsMid>, k_sym<kAP, false, kClsLarge>);
            break;
        case 4:
            passes(k_sym_group<kC, false, 64, 256, 160, 8>, 64, kMany, kCMost,
                   k_sym<kC, false, kClsMid>, k_sym<kC, false, kClsLarge>);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_p_copy(int64_t n, const int64_t *row_ptr, const int32_t *spare,
                         const int64_t *prow, int32_t *pcol, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_p_copy, dim3(grid_of_s(n, kBlock / 8, 8192)), dim3(kBlock), 0, s, n,
                       row_ptr, spare, prow, pcol);
    return hipGetLastError();
}

hipError_t launch_p_values(int64_t n, int64_t p_nnz, const int64_t *row_ptr, const int32_t *col,
                           const double *val, const double *diag, const int32_t *agg,
                           const uint32_t *size, double omega, const int64_t *prow,
                           const int32_t *pcol, double *pval, int32_t *prow_of, hipStream_t s) {
    if (n <= 0 || p_nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_p_values, dim3(grid_of_s(n, kBlock / kPG, 16384)), dim3(kBlock), 0, s, n,
                       row_ptr, col, val, diag, agg, size, omega, prow, pcol, pval, prow_of);
    return hipGetLastError();
}

namespace {

template <int K, int G, int CAP, int LIM, int U, int FT, int GV, class Terms>
hipError_t fill_rows(const SymArgs &a, uint32_t maxc, uint32_t flags, const Terms &tm,
                     const double *sval, double *oval, hipStream_t s) {
    if (a.rows <= 0) return hipSuccess;
    const int blocks = (grid_of_s(a.rows, kBlock / G, 8192) + 7) / 8 * 8;
    hipLaunchKernelGGL((k_fill_values<K, G, CAP, LIM, U, FT, Terms>), dim3(blocks), dim3(kBlock), 0,
                       s, a, maxc, tm, sval, oval);
    const int later = grid_of_s(a.rows, kSWaves * 64, kSBlocks);
    if (flags & kSymMid)
        hipLaunchKernelGGL((k_sym<K, true, kClsMid>), dim3(later), dim3(kSThreads), 0, s, a);
    if (flags & kSymLarge)
        hipLaunchKernelGGL((k_sym<K, true, kClsLarge>), dim3(later), dim3(kSThreads), 0, s, a);
    if (flags & (kSymMid | kSymLarge))
        hipLaunchKernelGGL((k_row_values<GV, Terms>), dim3(grid_of_s(a.rows, kValThreads / GV, 16384)),
                           dim3(kValThreads), 0, s, a.rows, (const uint8_t *)a.cls, tm, a.sptr,
                           a.scol, sval, a.out_ptr, (const int32_t *)a.out_col, oval);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ap_fill(int64_t n, const int64_t *row_ptr, const int32_t *col, const double *val,
                          const double *diag, const int64_t *prow, const int32_t *pcol,
                          const double *pval, const int64_t *aptr, int32_t *acol, double *aval,
                          uint8_t *cls, uint32_t flags, hipStream_t s) {
    const SymArgs a{n, row_ptr, col, nullptr, prow, pcol, nullptr, nullptr, nullptr, nullptr,
                    aptr, acol, nullptr, cls, nullptr};
    static_assert(kApMost < 48, "kApMost: the set's limit");
    return fill_rows<kAP, 16, 64, 48, 4, 4, 32>(a, kFew, flags, ApTerms{row_ptr, col, val, diag},
                                                pval, aval, s);
}

hipError_t launch_c_fill(int64_t n_agg, const int64_t *moff, const int32_t *members,
                         const int32_t *prow_of, const double *pval, const int64_t *aptr,
                         const int32_t *acol, const double *aval, const int64_t *crow,
                         int32_t *ccol, double *cval, uint8_t *cls, uint32_t flags, hipStream_t s) {
    const SymArgs a{n_agg, nullptr, nullptr, nullptr, aptr, acol, moff, members, prow_of, nullptr,
                    crow, ccol, nullptr, cls, nullptr};
    static_assert(kCMost < 160, "kCMost: the set's limit");
    return fill_rows<kC, 64, 256, 160, 8, 8, 64>(a, kMany, flags,
                                                 CTerms{moff, members, prow_of, pval}, aval, cval,
                                                 s);
}

hipError_t launch_column_rank(int64_t p_nnz, const int32_t *pcol, int64_t n_agg, uint32_t *cnt,
                              int32_t *rank, hipStream_t s) {
    const hipError_t e = launch_fill_u32(cnt, 0u, n_agg, s);
    if (e != hipSuccess || p_nnz <= 0) return e;
    hipLaunchKernelGGL(k_column_rank, dim3(grid_of_s(p_nnz, kBlock, 8192)), dim3(kBlock), 0, s,
                       p_nnz, pcol, cnt, rank);
    return hipGetLastError();
}

hipError_t launch_column_scatter(int64_t p_nnz, const int32_t *pcol, const int64_t *moff,
                                 const int32_t *rank, int32_t *members, hipStream_t s) {
    if (p_nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_column_scatter, dim3(grid_of_s(p_nnz, kBlock, 8192)), dim3(kBlock), 0, s,
                       p_nnz, pcol, moff, rank, members);
    return hipGetLastError();
}

}  // namespace mis2
