// galerkin.hip -- Galerkin coarse operator of an aggregation on gfx950, the
// multigrid hookup of the aggregates (Section VI-E sets up smoothed-aggregation
// multigrid on them).
//
// With the tentative prolongator for the constant near-null space,
// P[i][a] = 1/sqrt(n_a) when row i is in aggregate a (n_a members), the coarse
// operator is A_c = P^T A P:
//     (A_c)[a][b] = (sum of A[i][j] over i in a, j in b) / sqrt(n_a * n_b).
// Its off-diagonal part lives on the quotient graph (rows by aggregate,
// ascending columns, no self); its diagonal takes the fine diagonal and every
// coupling inside an aggregate.  Every sum runs over the fine rows in
// increasing id -- within a row, its diagonal first, then its entries in CSR
// order -- from 0.0, and is divided once by sqrt(n_a * n_b) (the product is
// exact), so the result is one fixed sequence of roundings.
//
// One wavefront per coarse row a.  Its members (counting-sorted by id) are
// walked in order, 64 at a time; their items (a member's diagonal, then its
// entries), in that order, are taken one per lane, some at a time.  Each lane
// finds the coarse column of its item (binary search in the coarse row; the
// member holding the item by binary search over the batch's item offsets), and
// the items are added to the row's accumulators in item order, by one of two
// ways.
//
// Aggregates of many items (more than 200 entries on average) and rows of at most
// kGSort columns: up to 256 items at a time go to LDS by column, in order, and a
// lane adds its columns' items; the diagonal's, most of them, are added 16 at a
// time by every lane (fold_members).  27-point 83x71x97 (1200 items a row) 267 us
// the other way, 192 this; elasticity 10^3 and 40^3 (6000) 576 and 946, 339 and
// 580: bound there by one wavefront's chain of LDS steps.
//
// Else 64 items at a time: the chunk is sorted by (column, lane) with a 64-lane
// bitonic network, and the first lane of each column's run adds the run's items
// one after the other (fold_row).  Accumulators (and the coarse row's columns)
// live in LDS for rows of at most kGCap columns, else in the output arrays
// themselves; two instances, as a pointer that may be either makes every access a
// flat one (2-D 5-point 1300^2, 30 items a row, 320 us with them, 278 without, 347
// by the first way; 7-point 100^3, 77 items, 165, 147 and 153).
// A final pass does the division.
#include "internal.h"
#include "lanes.h"
#include "rowset.h"

namespace mis2 {

namespace {

// coarse columns of a row held in LDS: 23 KB per 4-wave block with the members'
// tables (6 waves per SIMD; registers allow as many)
constexpr int kGCap = 255;
constexpr int kGWaves = kBlock / 64;

// Columns of a row whose items are sorted in LDS, one or two per lane.
constexpr int kGSort = 126;
constexpr int kGItems = 4;  // items per lane of a batch, at most

struct GStage {
    int32_t cols[kGCap];
    int64_t off[65];        // item offsets of a batch of 64 members
    int64_t rs[64];         // their CSR starts
    int32_t mi[64];         // their ids
    union {
        double acc[kGCap + 1];  // [0, d): the row's columns, [d]: its diagonal
        struct {
            // a batch: the diagonal's items from the front, the others from the
            // back (first in order of items, then by column)
            double item[64 * kGItems + 16];
            uint8_t col_of[64 * kGItems];
            int32_t cnt[kGSort];    // items of each column
            int32_t start[kGSort];
        };
    };
};

__device__ __forceinline__ int64_t lane_bcast64(int64_t v, int l) {
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// flag[0] = 1 when an aggregate id is outside [0, n_agg); flag[1] = 1 when a
// coarse column is.
__global__ __launch_bounds__(kBlock) void k_check_ids(int64_t n, const int32_t *__restrict__ agg,
                                                      int64_t cnnz,
                                                      const int32_t *__restrict__ ccol,
                                                      int64_t n_agg, uint32_t *flag) {
    uint32_t bad = 0;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n || v < cnnz;
         v += (int64_t)gridDim.x * kBlock) {
        if (v < n && (agg[v] < 0 || agg[v] >= n_agg)) bad |= 1u;
        if (v < cnnz && (ccol[v] < 0 || ccol[v] >= n_agg)) bad |= 2u;
    }
    if (bad & 1u) flag[0] = 1u;
    if (bad & 2u) flag[1] = 1u;
}

// The slot of coarse column b in the ascending cs[0 .. d) (top: the largest
// power of two <= d); -1, and *missing = 4, when b is not there.
__device__ __forceinline__ int coarse_slot(const int32_t *cs, int d, int top, int32_t b,
                                           uint32_t *missing) {
    int lo = 0;  // entries of cs below b
    for (int st = top; st > 0; st >>= 1)
        if (lo + st <= d && cs[lo + st - 1] < b) lo += st;
    if (lo < d && cs[lo] == b) return lo;
    *missing = 4u;
    return -1;
}

template <int K, int J>
__device__ __forceinline__ uint32_t bitonic_step(uint32_t key, int lane) {
    const uint32_t other = lane_xor<J>(key);
    const bool keep_min = ((lane & J) == 0) == ((lane & K) == 0);
    return keep_min ? (key < other ? key : other) : (key > other ? key : other);
}

template <int K, int J>
__device__ __forceinline__ uint32_t bitonic_merge(uint32_t key, int lane) {
    key = bitonic_step<K, J>(key, lane);
    if constexpr (J > 1) key = bitonic_merge<K, J / 2>(key, lane);
    return key;
}

// The 32-bit form of fold_chunk below, with register cross-lane moves.
__device__ __forceinline__ void fold_chunk32(int p, double v, int d, double *acc, double *accd,
                                             int lane) {
#pragma clang fp contract(off)
    uint32_t key = p >= 0 ? ((uint32_t)p << 6) | (uint32_t)lane : ~0u;
    key = bitonic_merge<2, 1>(key, lane);
    key = bitonic_merge<4, 2>(key, lane);
    key = bitonic_merge<8, 4>(key, lane);
    key = bitonic_merge<16, 8>(key, lane);
    key = bitonic_merge<32, 16>(key, lane);
    key = bitonic_merge<64, 32>(key, lane);
    const bool valid = key != ~0u;
    const int sp = valid ? (int)(key >> 6) : -1;
    const double sv = __shfl(v, (int)(key & 63), 64);
    const int prev = (int)from_prev((uint32_t)sp);
    const bool head = valid && (lane == 0 || prev != sp);
    const uint64_t heads = __ballot(head) | __ballot(!valid);
    const uint64_t after = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
    const int run = head ? (after ? __ffsll((unsigned long long)after) - 1 : 64) - lane : 0;
    const int longest = (int)__builtin_amdgcn_readfirstlane(group_max<64>((uint32_t)run));
    double my = head ? (sp == d ? *accd : acc[sp]) : 0.0;
    uint32_t lo = __double2loint(sv), hi = __double2hiint(sv);  // lane l: item l + j
    for (int j = 0; j < longest; j++) {
        const double sum = my + __hiloint2double((int)hi, (int)lo);
        my = j < run ? sum : my;
        lo = from_next(lo);
        hi = from_next(hi);
    }
    if (head) {
        if (sp == d) *accd = my;
        else acc[sp] = my;
    }
}

// Folds a chunk (lane q: slot p, -1 for none, d for the diagonal; value v) into
// the accumulators in lane order.  The chunk is sorted by (slot, lane) with a
// 64-lane bitonic network, so each slot's items form one run of lanes, still
// in lane order, and the run's first lane adds them one after the other.
// Key = slot * 64 + lane in a K-bit word (32 bits while d < 2^25).
template <typename K>
__device__ __forceinline__ void fold_chunk(int p, double v, int d, double *acc, double *accd,
                                           int lane) {
#pragma clang fp contract(off)
    const K none = ~(K)0;
    K key = p >= 0 ? ((K)(uint32_t)p << 6) | (K)(uint32_t)lane : none;
    for (int k = 2; k <= 64; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            const K other = __shfl_xor(key, j, 64);
            const bool keep_min = ((lane & j) == 0) == ((lane & k) == 0);
            key = keep_min ? (key < other ? key : other) : (key > other ? key : other);
        }
    const bool valid = key != none;
    const int sp = valid ? (int)(key >> 6) : -1;
    const double sv = __shfl(v, (int)(key & 63), 64);
    const int prev = __shfl_up(sp, 1, 64);
    const bool head = valid && (lane == 0 || prev != sp);
    // the run of the head at lane r ends at the next head (or the first
    // invalid lane)
    const uint64_t heads = __ballot(head) | __ballot(!valid);
    const uint64_t after = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
    const int run = head ? (after ? __ffsll((unsigned long long)after) - 1 : 64) - lane : 0;
    int longest = run;
    for (int o = 32; o > 0; o >>= 1) longest = max(longest, __shfl_xor(longest, o, 64));
    double my = head ? (sp == d ? *accd : acc[sp]) : 0.0;
    for (int j = 0; j < longest; j++) {
        const double vj = __shfl(sv, lane + j < 64 ? lane + j : 63, 64);
        const double sum = my + vj;
        my = j < run ? sum : my;
    }
    if (head) {
        if (sp == d) *accd = my;
        else acc[sp] = my;
    }
}

// Items t0 .. t0 + 64 U of a batch of members (lane l: items t0 + 64 k + l), as
// loaded: value, fine column, and which they are.
template <int U>
struct GItems {
    double v[U];
    int32_t c[U];
    int8_t kind[U];  // 0 an entry, 1 a member's diagonal, 2 none
};

template <int U>
__device__ __forceinline__ void load_items(const GStage &S, int lane, int64_t t0, int64_t total,
                                           int64_t nnz, const int32_t *__restrict__ col,
                                           const double *__restrict__ val,
                                           const double *__restrict__ diag, GItems<U> &g) {
#pragma unroll
    for (int k = 0; k < U; k++) {
        const int64_t t = t0 + 64 * k + lane, tc = t < total ? t : 0;
        int kr = 0;  // the member holding the item
#pragma unroll
        for (int st = 32; st > 0; st >>= 1)
            if (S.off[kr + st] <= tc) kr += st;
        const int64_t o = tc - S.off[kr], e = S.rs[kr] + o - 1;
        g.kind[k] = t >= total ? 2 : o == 0 ? 1 : 0;
        // (named as global memory: the choice of two pointers would be a flat load,
        // which the waits for LDS wait for as well)
        using Global = const __attribute__((address_space(1))) double *;
        g.v[k] = *(o == 0 ? (Global)(diag + S.mi[kr]) : (Global)(val + e));
        g.c[k] = nnz > 0 ? col[o == 0 ? 0 : e] : 0;
    }
}

// Folds them into the accumulators: columns lane and 64 + lane of the row, and
// the diagonal in every lane.  The diagonal's items, half of all or more, go to
// the front of the batch in LDS and 16 at a time through chain_add16; the others
// to its back, and from there each to its place by column (the column's items so
// far, and the lanes below of the same column, found by a ballot for each bit of
// the column's number), where a lane adds its columns' one after the other.
// then() runs before the additions.
template <int U, class Then>
__device__ __forceinline__ void fold_sorted(GStage &S, int lane, const GItems<U> &g,
                                            const int32_t (&b)[U], int32_t a, int d, int top,
                                            int bits, double (&acc)[2], double &accd,
                                            uint32_t *missing, Then then) {
#pragma clang fp contract(off)
    constexpr int kEnd = 64 * U - 1;
    const uint64_t lower = lane ? ~0ull >> (64 - lane) : 0ull;
    int nd = 0, nr = 0;
    int code[U];
#pragma unroll
    for (int k = 0; k < U; k++) {
        int lo = 0;  // columns of the coarse row below b
        for (int st = top; st > 0; st >>= 1)
            if (lo + st <= d && S.cols[lo + st - 1] < b[k]) lo += st;
        const bool found = lo < d && S.cols[min(lo, max(d - 1, 0))] == b[k];
        const bool other = g.kind[k] == 0 && b[k] != a;
        if (other && !found) *missing = 4u;
        code[k] = other && found ? lo : -1;
        const uint64_t mr = __ballot(other && found);
        const uint64_t md = __ballot(g.kind[k] == 1 || (g.kind[k] == 0 && b[k] == a));
        const int at = code[k] >= 0 ? kEnd - nr - __popcll(mr & lower) : nd + __popcll(md & lower);
        if ((mr | md) >> lane & 1u) S.item[at] = g.v[k];
        if (code[k] >= 0) S.col_of[at] = (uint8_t)code[k];
        nr += __popcll(mr);
        nd += __popcll(md);
    }
    wave_sync();
    double v[U];
    int place[U];
#pragma unroll
    for (int k = 0; k < U; k++) {
        if (64 * k < nr) {
            const int at = kEnd - 64 * k - lane;
            const bool in = 64 * k + lane < nr;
            v[k] = S.item[at];
            code[k] = in ? (int)S.col_of[at] : -1;
            uint64_t same = __ballot(in);
            for (int bit = 0; bit < bits; bit++) {
                const bool on = code[k] >> bit & 1;
                const uint64_t m = __ballot(on);
                same &= on ? m : ~m;
            }
            const int below = __popcll(same & lower);
            const int before = in ? S.cnt[code[k]] : 0;
            place[k] = before + below;
            wave_sync();
            if (in && below == 0) S.cnt[code[k]] = before + __popcll(same);
            wave_sync();
        }
    }
    // where each column's items begin
    const int n0 = lane < d ? S.cnt[lane] : 0;
    const int i0 = (int)wave_incl_scan((uint32_t)n0);
    const int s0 = kEnd + 1 - nr + i0 - n0;
    if (lane < d) {
        S.start[lane] = s0;
        S.cnt[lane] = 0;  // clear again for the next batch
    }
    int n1 = 0, s1 = 0;
    if (d > 64) {
        n1 = 64 + lane < d ? S.cnt[64 + lane] : 0;
        const int i1 = (int)wave_incl_scan((uint32_t)n1);
        s1 = kEnd + 1 - nr + __builtin_amdgcn_readlane(i0, 63) + i1 - n1;
        if (64 + lane < d) {
            S.start[64 + lane] = s1;
            S.cnt[64 + lane] = 0;
        }
    }
    wave_sync();
#pragma unroll
    for (int k = 0; k < U; k++)
        if (64 * k < nr && code[k] >= 0) S.item[S.start[code[k]] + place[k]] = v[k];
    wave_sync();
    then();
    auto add = [&](double my, int s, int n) {
        const int longest = (int)__builtin_amdgcn_readfirstlane(group_max<64>((uint32_t)n));
        for (int j = 0; j < longest; j += 4) {
            double x[4];
#pragma unroll
            for (int q = 0; q < 4; q++) x[q] = S.item[s + min(j + q, max(n - 1, 0))];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const double sum = my + x[q];
                my = j + q < n ? sum : my;
            }
        }
        return my;
    };
    if (nr > 0) {
        acc[0] = add(acc[0], s0, n0);
        if (d > 64) acc[1] = add(acc[1], s1, n1);
    }
    double next = S.item[lane & 15];
    for (int j = 0; j < nd; j += 16) {
        const double term = j + (lane & 15) < nd ? next : -0.0;  // x + -0.0 is x
        next = S.item[j + 16 + (lane & 15)];
        accd = chain_add16(accd, term);
    }
    wave_sync();
}

// A batch of members' items, 64 U at a time; the next ones are loaded while these
// are placed, and their aggregates while these are added.
template <int U>
__device__ __forceinline__ void fold_members(GStage &S, int lane, int64_t total, int64_t nnz,
                                             const int32_t *__restrict__ col,
                                             const double *__restrict__ val,
                                             const double *__restrict__ diag,
                                             const int32_t *__restrict__ agg, int32_t a, int d,
                                             int top, int bits, double (&acc)[2], double &accd,
                                             uint32_t *missing) {
    GItems<U> g;
    int32_t b[U];
    load_items<U>(S, lane, 0, total, nnz, col, val, diag, g);
#pragma unroll
    for (int k = 0; k < U; k++) b[k] = agg[g.c[k]];
    for (int64_t t0 = 0; t0 < total; t0 += 64 * U) {
        GItems<U> ahead = g;
        int32_t next[U] = {};
        const bool more = t0 + 64 * U < total;
        if (more) load_items<U>(S, lane, t0 + 64 * U, total, nnz, col, val, diag, ahead);
        fold_sorted<U>(S, lane, g, b, a, d, top, bits, acc, accd, missing, [&]() {
            if (!more) return;
#pragma unroll
            for (int k = 0; k < U; k++) next[k] = agg[ahead.c[k]];
        });
        g = ahead;
#pragma unroll
        for (int k = 0; k < U; k++) b[k] = next[k];
    }
}

// A batch of 64 members (lane j: the j-th), their items numbered one after the
// other.
__device__ __forceinline__ int64_t stage_members(GStage &S, int lane, int64_t k0, int64_t m1,
                                                 int64_t nnz, const int64_t *__restrict__ row_ptr,
                                                 const int32_t *__restrict__ members) {
    const bool mv = k0 + lane < m1;
    const int32_t mi = members[mv ? k0 + lane : m1 - 1];
    const int64_t rs = row_ptr[mi], re = row_ptr[mi + 1];
    const int64_t cnt_i = mv ? 1 + (re - rs) : 0;
    int64_t incl = cnt_i;
    if (nnz < 0x7FFFFFFF)
        incl = (int64_t)wave_incl_scan((uint32_t)cnt_i);
    else
        for (int dd = 1; dd < 64; dd <<= 1) {
            const int64_t o = __shfl_up(incl, dd, 64);
            if (lane >= dd) incl += o;
        }
    S.off[lane + 1] = incl;
    S.rs[lane] = rs;
    S.mi[lane] = mi;
    if (lane == 0) S.off[0] = 0;
    wave_sync();
    return lane_bcast64(incl, 63);
}

// The row's items 64 at a time, folded chunk by chunk into accumulators in LDS
// (SMALL: at most kGCap columns) or in the output arrays.
template <bool SMALL>
__device__ __forceinline__ void fold_row(GStage &S, int lane, int64_t a, int64_t c0, int d, int top,
                                         int64_t m0, int64_t m1, int64_t nnz,
                                         const int64_t *__restrict__ row_ptr,
                                         const int32_t *__restrict__ col,
                                         const double *__restrict__ val,
                                         const double *__restrict__ diag,
                                         const int32_t *__restrict__ agg,
                                         const int64_t *__restrict__ moff,
                                         const int32_t *__restrict__ members,
                                         const int32_t *__restrict__ ccol, double *cval,
                                         double *cdiag, uint32_t *missing) {
#pragma clang fp contract(off)
    double *acc, *accd;
    const int32_t *cs;
    if constexpr (SMALL) {
        acc = S.acc;
        accd = &S.acc[d];
        cs = S.cols;
    } else {
        acc = cval + c0;
        accd = cdiag + a;
        cs = ccol + c0;
    }
    for (int p = lane; p < d; p += 64) {
        if (SMALL) S.cols[p] = ccol[c0 + p];
        acc[p] = 0.0;
    }
    if (lane == 0) *accd = 0.0;
    const bool narrow = SMALL || d < (1 << 25);  // slot * 64 + lane fits 31 bits
    wave_sync();
    for (int64_t k0 = m0; k0 < m1; k0 += 64) {
        const int64_t total = stage_members(S, lane, k0, m1, nnz, row_ptr, members);
        // two chunks per step, A = items t0 .. t0+63 and B = the next 64: their
        // loads are issued together from clamped valid addresses, then A is
        // folded and B after it
        for (int64_t t0 = 0; t0 < total; t0 += 128) {
            const int64_t ta = t0 + lane, tb = t0 + 64 + lane;
            const bool ina = ta < total, inb = tb < total;
            const int64_t tac = ina ? ta : 0, tbc = inb ? tb : 0;
            int kra = 0, krb = 0;  // the members holding the items
            for (int st = 32; st > 0; st >>= 1) {
                if (S.off[kra + st] <= tac) kra += st;
                if (S.off[krb + st] <= tbc) krb += st;
            }
            const int64_t oa = tac - S.off[kra], ob = tbc - S.off[krb];
            const bool da = oa == 0, db = ob == 0;  // the member's diagonal
            const double dga = diag[S.mi[kra]], dgb = diag[S.mi[krb]];
            int pa = ina ? d : -1, pb = inb ? d : -1;  // -1: no item; d: the diagonal
            double va = dga, vb = dgb;
            if (nnz > 0) {
                const int64_t ea = ina && !da ? S.rs[kra] + oa - 1 : 0;
                const int64_t eb = inb && !db ? S.rs[krb] + ob - 1 : 0;
                const int32_t ca = col[ea], cb = col[eb];
                const double xa = val[ea], xb = val[eb];
                const int32_t ba = agg[ca], bb = agg[cb];
                if (ina && !da) {
                    va = xa;
                    if (ba != (int32_t)a) pa = coarse_slot(cs, d, top, ba, missing);
                }
                if (inb && !db) {
                    vb = xb;
                    if (bb != (int32_t)a) pb = coarse_slot(cs, d, top, bb, missing);
                }
            }
            if (narrow) fold_chunk32(pa, va, d, acc, accd, lane);
            else fold_chunk<uint64_t>(pa, va, d, acc, accd, lane);
            wave_sync();
            if (t0 + 64 < total) {
                if (narrow) fold_chunk32(pb, vb, d, acc, accd, lane);
                else fold_chunk<uint64_t>(pb, vb, d, acc, accd, lane);
                wave_sync();
            }
        }
    }
    // the division by sqrt(n_a * n_b)
    const double na = (double)(m1 - m0);
    for (int p = lane; p < d; p += 64) {
        const int32_t b = cs[p];
        const double nb = (double)(moff[b + 1] - moff[b]);
        cval[c0 + p] = acc[p] / sqrt(na * nb);
    }
    if (lane == 0) cdiag[a] = m1 > m0 ? *accd / sqrt(na * na) : *accd;
}

// flag[2] = 1 when an entry's aggregate pair is missing from the coarse row.
// SORT: rows of at most kGSort columns by fold_members.
template <bool SORT>
__global__ __launch_bounds__(kBlock, SORT ? 5 : 1) void k_galerkin(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const double *__restrict__ val, const double *__restrict__ diag,
    const int32_t *__restrict__ agg, int64_t n_agg, const int64_t *__restrict__ moff,
    const int32_t *__restrict__ members, const int64_t *__restrict__ crow,
    const int32_t *__restrict__ ccol, double *cval, double *cdiag, uint32_t *flag, int64_t nnz) {
#pragma clang fp contract(off)
    __shared__ GStage stage[kGWaves];
    const int lane = threadIdx.x & 63;
    GStage &S = stage[threadIdx.x >> 6];
    const int64_t a = (int64_t)blockIdx.x * kGWaves + (threadIdx.x >> 6);
    if (a >= n_agg) return;
    const int64_t c0 = crow[a], c1 = crow[a + 1];
    const int d = (int)(c1 - c0);
    const int64_t m0 = moff[a], m1 = moff[a + 1];
    const int top = d > 0 ? 1 << (31 - __builtin_clz((unsigned)d)) : 0;
    uint32_t missing = 0;
    if (SORT && d <= kGSort) {
        const int bits = d > 1 ? 32 - __builtin_clz((unsigned)d - 1u) : 0;  // of a column's number
        double part[2] = {0.0, 0.0}, partd = 0.0;
        for (int p = lane; p < d; p += 64) {
            S.cols[p] = ccol[c0 + p];
            S.cnt[p] = 0;
        }
        wave_sync();
        for (int64_t k0 = m0; k0 < m1; k0 += 64) {
            const int64_t total = stage_members(S, lane, k0, m1, nnz, row_ptr, members);
            if (total <= 128)
                fold_members<2>(S, lane, total, nnz, col, val, diag, agg, (int32_t)a, d, top, bits,
                                part, partd, &missing);
            else
                fold_members<kGItems>(S, lane, total, nnz, col, val, diag, agg, (int32_t)a, d, top,
                                      bits, part, partd, &missing);
            wave_sync();  // the offsets are rewritten by the next members
        }
        const double na = (double)(m1 - m0);
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int p = 64 * k + lane;
            if (p < d) {
                const int32_t b = S.cols[p];
                cval[c0 + p] = part[k] / sqrt(na * (double)(moff[b + 1] - moff[b]));
            }
        }
        if (lane == 0) cdiag[a] = m1 > m0 ? partd / sqrt(na * na) : partd;
    } else if (d <= kGCap) {
        fold_row<true>(S, lane, a, c0, d, top, m0, m1, nnz, row_ptr, col, val, diag, agg, moff,
                       members, ccol, cval, cdiag, &missing);
    } else {
        fold_row<false>(S, lane, a, c0, d, top, m0, m1, nnz, row_ptr, col, val, diag, agg, moff,
                        members, ccol, cval, cdiag, &missing);
    }
    if (missing) flag[2] = 1u;
}

int grid_for(int64_t work, int cap) {
    const int64_t g = (work + kBlock - 1) / kBlock;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

}  // namespace

hipError_t launch_check_ids(int64_t n, const int32_t *agg, int64_t cnnz, const int32_t *ccol,
                            int64_t n_agg, uint32_t *flag, hipStream_t s) {
    if (n <= 0 && cnnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_ids, dim3(grid_for(std::max(n, cnnz), 4096)), dim3(kBlock), 0, s,
                       n, agg, cnnz, ccol, n_agg, flag);
    return hipGetLastError();
}

hipError_t launch_galerkin(const int64_t *row_ptr, const int32_t *col, const double *val,
                           const double *diag, const int32_t *agg, int64_t n_agg,
                           const int64_t *moff, const int32_t *members, const int64_t *crow,
                           const int32_t *ccol, double *cval, double *cdiag, uint32_t *flag,
                           int64_t nnz, hipStream_t s) {
    if (n_agg <= 0) return hipSuccess;
    const int64_t blocks = (n_agg + kGWaves - 1) / kGWaves;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr, col, val,
                           diag, agg, n_agg, moff, members, crow, ccol, cval, cdiag, flag, nnz);
    };
    // (both sides measured: the file's head)
    if (nnz > 200 * n_agg) go(k_galerkin<true>);
    else go(k_galerkin<false>);
    return hipGetLastError();
}

}  // namespace mis2
