// quotient.hip -- coarse graph of an aggregation, for multilevel coarsening on gfx950.
//
// The paper coarsens recursively (Sections I and II) without saying how the
// next graph is formed.  Here it is the quotient graph: vertices are the
// aggregates, and a is adjacent to c iff some edge (u, w) has agg u = a,
// agg w = c and a != c.  Rows come out with ascending, distinct columns.
//
// A vertex with agg < 0 belongs to no coarse vertex (a batched run uses this
// for graphs that stop coarsening) and edges to it are dropped.
//
// Member lists are built by a counting sort (their order does not matter:
// every coarse row is a sorted set).  A coarse row's candidates are its
// members' stored entries; what it holds is their distinct aggregate ids, of
// which there are few even where the candidates are many (a 27-point mesh's
// aggregate has some 1000 candidates and 30 neighbours).  Rows go to one of
// four paths by how many distinct ids they turn out to have: a small LDS hash
// set per lane group (k_coarse_rows_group, several rows per wavefront where
// aggregates are small), a 1024-slot set per wavefront (only where an LDS
// bitmap cannot hold every coarse id), one workgroup, and for rows of more than
// kGiantCand candidates a bitmap slot that the whole grid fills.  The first two
// rank the distinct ids; a workgroup sweeps the coarse ids with an LDS bitmap
// (of as many bits as there are coarse ids, in windows of 32*kBitWords where
// that is more), which emits them in increasing
// order and, after the first window, visits only the range the row's
// candidates span.  Every path deals the members' entries out evenly over its
// lanes.  The first three write their rows to a spare buffer while they count
// them, and after the prefix sum they are only copied; what the buffer has no
// room for is gathered a second time and written then.
#include <algorithm>

#include "internal.h"
#include "lanes.h"
#include "rowset.h"

namespace mis2 {

namespace {

constexpr int kBitWords = 12288;             // most LDS bitmap words (48 KiB)
constexpr int kWaves = kBlock / 64;
constexpr int kWSlots = 1024;                // set of a wavefront row (second path)
constexpr int kWLim = 768;                   // a row with as many distinct ids goes on
constexpr uint32_t kWCand = 8192;            // or with more candidates
constexpr int kWEdges = 8;                   // entries per lane loaded together

// The spare buffer that rows are written to while they are counted.  Its first
// part has `per` entries for every member of a row; its second part takes the
// rows that need more, wherever there is room: kSpareParts regions with a cursor
// each (one address for the whole chip would serialise its atomics); a row's
// place, an index into the buffer, is kept in the row's unused slot of the first
// part.
constexpr int kSpareParts = 32;
constexpr int kSpareLine = 32;  // words per cursor (one cache line)
struct Spare {
    int32_t *buf;       // [per * n] first part, then the cursors, then the regions
    int64_t per;
    uint32_t *cursor;   // [kSpareParts][kSpareLine], zero before the count pass
    int64_t base;       // of region 0 in buf
    uint32_t cap;       // entries of a region
};

// m entries for row a in region `part`: their index in buf, or -1 when the
// region is full.  One thread calls it.
__device__ __forceinline__ int64_t spare_take(const Spare &sp, uint32_t part, uint32_t m) {
    part &= (uint32_t)(kSpareParts - 1);
    uint32_t *c = sp.cursor + part * kSpareLine;
    if (m > sp.cap || *(volatile uint32_t *)c > sp.cap - m) return -1;
    const uint32_t at = atomicAdd(c, m);
    return at <= sp.cap - m ? sp.base + (int64_t)part * sp.cap + at : -1;
}

// Notes the place of a row of class 3 with members from m0 on (per >= 2).
__device__ __forceinline__ void spare_note(const Spare &sp, int64_t m0, int64_t at) {
    sp.buf[m0 * sp.per] = (int32_t)(uint32_t)at;
    sp.buf[m0 * sp.per + 1] = (int32_t)(at >> 32);
}

// Classes of coarse rows: where the row is after the count pass.
constexpr uint8_t kInPlace = 0;  // first part of the spare buffer
constexpr uint8_t kSecond = 1;   // the second path's, to be written
constexpr uint8_t kBig = 2;      // a workgroup's or a giant row, to be written
constexpr uint8_t kSpared = 3;   // second part of the spare buffer

// First path: every coarse row, one group of G lanes each, its distinct ids
// in a CAP-slot set (LIM - 1 of them at most, MAXC candidates).  What bounds
// it is the chain of dependent loads of a row (member offsets, members, row
// extents, columns, their labels) and the LDS steps after it, so rows in
// flight count: 16 lanes per row and 128 slots where aggregates are small
// (four rows per wavefront), a wavefront and 256 slots where a row has
// hundreds of candidates.  Measured, counting and writing together, against one
// wavefront per row with a set as large as its candidates (and a workgroup's
// sort past 1024 of them), run twice: 2.5M rows of a 512-subdomain union
// (level 0: 5 members, 40 candidates) 4.0 -> 0.79 ms; 14 000 rows of 40
// members and 1000 candidates (27-point 83x71x97) 1.38 -> 0.06 ms.
// ccnt[a], the ids in increasing order in the spare buffer and cls[a] (class 0
// or 3); class `over` for a row it leaves to another path.
template <int G, int CAP, int LIM, int U>
__global__ __launch_bounds__(kBlock) void k_coarse_rows_group(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const int32_t *__restrict__ agg, int64_t n_agg, const int64_t *__restrict__ moff,
    const int32_t *__restrict__ members, uint32_t maxc, uint32_t *__restrict__ ccnt,
    Spare sp, uint8_t *__restrict__ cls, uint8_t over) {
    constexpr int kGroups = kBlock / G;
    __shared__ RowSet<G, CAP, LIM> sets[kGroups];
    const int grp = (int)threadIdx.x / G, lane = (int)threadIdx.x % G;
    RowSet<G, CAP, LIM> &S = sets[grp];
    row_clear(S, lane, 0u, true);
    // each XCD takes one run of the rows of a step (the grid is a multiple of
    // 8): neighbouring rows share columns and labels
    const int64_t blk = (int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    // small groups: the next row's members and their extents load while this row
    // is gathered and written, and the offsets of the one after it: 873 -> 794 us
    // for the 2.5M rows above.  (A wavefront per row has one row or two, and the
    // loads are in its way: 58 -> 65 us.)
    constexpr bool kAhead = G < 64;
    const int64_t stride = (int64_t)gridDim.x * kGroups, a0 = blk * kGroups + grp;
    auto offsets = [&](int64_t a, int64_t &m0, int64_t &m1) {
        const int64_t ac = min(a, n_agg - 1);
        m0 = moff[ac];
        m1 = moff[ac + 1];
    };
    // (an aggregate without members: vertex 0; members[0] is loaded, but where no
    // vertex has a label nothing has written it)
    auto member = [&](int64_t m0, int64_t m1) {
        const int32_t v = members[m1 > m0 ? min(m0 + lane, m1 - 1) : 0];
        return m1 > m0 ? v : 0;
    };
    int64_t m0, m1, n0 = 0, n1 = 0, rs0 = 0, d0 = 0;
    offsets(a0, m0, m1);
    if (kAhead) {
        offsets(a0 + stride, n0, n1);
        const int32_t v = member(m0, m1);
        rs0 = row_ptr[v];
        d0 = row_ptr[v + 1] - rs0;
    }
    for (int64_t a = a0; a < n_agg; a += stride) {
        int64_t l0 = 0, l1 = 0;
        const int32_t vn = kAhead ? member(n0, n1) : 0;
        if (kAhead) offsets(a + 2 * stride, l0, l1);
        const bool fits = row_gather<G, CAP, LIM, U>(
            S, lane, m0, m1, maxc,
            [&](int64_t i, int64_t &rs, int64_t &d) {
                if (kAhead && i - m0 < G) {
                    rs = rs0;
                    d = d0;
                    return;
                }
                const int32_t v = members[i];
                rs = row_ptr[v];
                d = row_ptr[v + 1] - rs;
            },
            [&](int64_t j) { return col[j]; },
            [&](int32_t x) {
                const int32_t c = agg[x];
                return (int64_t)c == a ? -1 : c;
            });
        if (kAhead) {
            rs0 = row_ptr[vn];
            d0 = row_ptr[vn + 1] - rs0;
        }
        const uint32_t m = S.num;
        int64_t at = m0 * sp.per;
        if (fits && (int64_t)m > (m1 - m0) * sp.per) {
            if (lane == 0) {
                at = spare_take(sp, blockIdx.x, m);
                S.base[0] = at;
                if (at >= 0) spare_note(sp, m0, at);
            }
            wave_sync();
            at = S.base[0];
        }
        const bool done = fits && at >= 0;
        if (done) row_write(S, lane, m, sp.buf + at);
        if (lane == 0) {
            ccnt[a] = m;
            cls[a] = !done ? over : at == m0 * sp.per ? kInPlace : kSpared;
        }
        row_clear(S, lane, m, !fits);
        if (kAhead) {
            m0 = n0;
            m1 = n1;
            n0 = l0;
            n1 = l1;
        } else {
            offsets(a + stride, m0, m1);
        }
    }
}

// The rows in the spare buffer to their place, 16 lanes each, four rows' loads at
// once (1.5M rows 191 -> 140 us: three loads in a row of trips to memory).
__global__ __launch_bounds__(kBlock) void k_copy_rows(int64_t n_agg, const int64_t *__restrict__ moff,
                                                      const int64_t *__restrict__ crow,
                                                      const uint8_t *__restrict__ cls, Spare sp,
                                                      int32_t *__restrict__ ccol) {
    constexpr int K = 4;
    const int lane = (int)(threadIdx.x & 15u);
    const int64_t stride = (int64_t)gridDim.x * (kBlock / 16);
    for (int64_t a0 = (int64_t)blockIdx.x * (kBlock / 16) + (threadIdx.x >> 4); a0 < n_agg;
         a0 += K * stride) {
        int64_t d0[K], len[K], s0[K];
        uint8_t c[K];
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int64_t a = min(a0 + k * stride, n_agg - 1);
            d0[k] = crow[a];
            len[k] = crow[a + 1] - d0[k];
            c[k] = cls[a];
            s0[k] = moff[a] * sp.per;
        }
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (a0 + k * stride >= n_agg || (c[k] != kInPlace && c[k] != kSpared)) len[k] = 0;
            if (len[k] > 0 && c[k] == kSpared)
                s0[k] = (int64_t)(uint32_t)sp.buf[s0[k]] |
                        (int64_t)((uint64_t)(uint32_t)sp.buf[s0[k] + 1] << 32);
        }
        int32_t x[K];
#pragma unroll
        for (int k = 0; k < K; k++) x[k] = sp.buf[lane < len[k] ? s0[k] + lane : 0];
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (lane < len[k]) ccol[d0[k] + lane] = x[k];
            for (int64_t i = lane + 16; i < len[k]; i += 16) ccol[d0[k] + i] = sp.buf[s0[k] + i];
        }
    }
}

// Second path, where there are more coarse ids than an LDS bitmap holds: the
// rows of class 1, one wavefront each with a 1024-slot set.  (With fewer ids a
// workgroup and a bitmap are faster: a set half full probes in long divergent
// runs.  Level 0 of Chung-Lu 1M, 17 000 rows of 96 or more distinct ids: 800
// us here.)  FILL = false: ccnt[a], and the row itself where the spare buffer
// has room (class 3); class 2 to the rows with kWLim or more distinct ids or
// more than kWCand candidates.  FILL = true: the rows still of class 1 to
// ccol[crow[a] ...].  Up to 64 ids are ranked by
// counting, more sorted in LDS.  Each wavefront reads 64 classes at a time,
// so the rows of class 1 stay spread over all wavefronts.
template <bool FILL>
__global__ __launch_bounds__(kBlock) void k_coarse_rows_wave(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const int32_t *__restrict__ agg, int64_t n_agg, const int64_t *__restrict__ moff,
    const int32_t *__restrict__ members, uint32_t *__restrict__ ccnt,
    const int64_t *__restrict__ crow, int32_t *__restrict__ ccol, uint8_t *__restrict__ cls,
    Spare sp) {
    constexpr uint32_t kEmpty = 0xFFFFFFFFu;
    __shared__ RowSet<64, kWSlots, kWLim> sets[kWaves];
    const int wv = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63u);
    RowSet<64, kWSlots, kWLim> &S = sets[wv];
    const int64_t nw = (int64_t)gridDim.x * kWaves;
    const int64_t w0 = (int64_t)blockIdx.x * kWaves + wv;
    row_clear(S, lane, 0u, true);
    auto row = [&](const int64_t a) {
        const int64_t m0 = moff[a], m1 = moff[a + 1];
        const bool done = row_gather<64, kWSlots, kWLim, kWEdges>(
            S, lane, m0, m1, kWCand,
            [&](int64_t i, int64_t &rs, int64_t &d) {
                const int32_t v = members[i];
                rs = row_ptr[v];
                d = row_ptr[v + 1] - rs;
            },
            [&](int64_t j) { return col[j]; },
            [&](int32_t x) {
                const int32_t c = agg[x];
                return (int64_t)c == a ? -1 : c;
            });
        const uint32_t m = S.num;
        int32_t *dst = nullptr;
        if (FILL) {
            dst = ccol + crow[a];
        } else {
            int64_t at = -1;
            if (lane == 0) {
                ccnt[a] = m;
                if (!done) {
                    cls[a] = kBig;
                } else if (m > 0) {
                    at = spare_take(sp, (uint32_t)w0, m);
                    if (at >= 0) {
                        cls[a] = kSpared;
                        spare_note(sp, m0, at);
                    }
                }
            }
            const int lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)at);
            const int hi = __builtin_amdgcn_readfirstlane((int)(at >> 32));
            if (hi >= 0) dst = sp.buf + (((int64_t)hi << 32) | (uint32_t)lo);
        }
        if (dst && m <= 64) {
            if ((uint32_t)lane < m) {
                const uint32_t x = S.list[lane];
                uint32_t rank = 0;
                for (uint32_t y = 0; y < m; y++) rank += S.list[y] < x ? 1u : 0u;
                dst[rank] = (int32_t)x;
            }
        } else if (dst) {
            // bitonic sort of a copy in the set's table, then the table is
            // cleared whole
            uint32_t *tab = S.tab;
            uint32_t P = 1;
            while (P < m) P <<= 1;
            for (uint32_t i = lane; i < P; i += 64) tab[i] = i < m ? S.list[i] : kEmpty;
            wave_sync();
            for (uint32_t k = 2; k <= P; k <<= 1) {
                for (uint32_t jj = k >> 1; jj > 0; jj >>= 1) {
                    for (uint32_t i = lane; i < P; i += 64) {
                        const uint32_t ixj = i ^ jj;
                        if (ixj > i) {
                            const uint32_t x = tab[i], y = tab[ixj];
                            const bool up = (i & k) == 0;
                            if ((x > y) == up) {
                                tab[i] = y;
                                tab[ixj] = x;
                            }
                        }
                    }
                    wave_sync();
                }
            }
            for (uint32_t i = lane; i < m; i += 64) dst[i] = (int32_t)tab[i];
        }
        wave_sync();
        row_clear(S, lane, m, !done || (dst && m > 64));
    };
    for (int64_t j0 = 0; w0 + j0 * nw < n_agg; j0 += 64) {
        const int64_t v = w0 + (j0 + lane) * nw;
        const bool mine = v < n_agg && cls[v] == kSecond;
        uint64_t mask = __ballot(mine);
        while (mask) {
            const int r = __ffsll((unsigned long long)mask) - 1;
            mask &= mask - 1;
            row(w0 + (j0 + r) * nw);
        }
    }
}

// cnt[a] = members of aggregate a; rank[v] = v's place among them (in no
// particular order).  Consecutive vertices often share their aggregate: the
// first lane of each run of equal labels adds for the run, so one atomic
// serves it, and the scatter below needs none (27-point 83x71x97, count and
// scatter: 72 -> 11 us; 15M vertices of small cubes 860 -> 275 us).
__global__ __launch_bounds__(kBlock) void k_member_rank(int64_t n, const int32_t *__restrict__ agg,
                                                        uint32_t *__restrict__ cnt,
                                                        int32_t *__restrict__ rank) {
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    // whole wavefronts stay in the loop together (the last chunk's tail lanes
    // carry no aggregate)
    for (int64_t v0 = (int64_t)blockIdx.x * kBlock + (threadIdx.x - lane); v0 < n; v0 += stride) {
        const int64_t v = v0 + lane;
        const int32_t a = v < n ? agg[v] : -1;
        const int32_t prev = (int32_t)from_prev((uint32_t)a);
        const uint64_t heads = __ballot(lane == 0 || a != prev);
        const int start = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
        const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1);
        const int len = later ? __ffsll((unsigned long long)later) : 64 - lane;
        uint32_t base = 0;
        if (start == lane && a >= 0) base = atomicAdd(&cnt[a], (uint32_t)len);
        base = (uint32_t)__shfl((int)base, start, 64);
        if (v < n) rank[v] = (int32_t)(base + (uint32_t)(lane - start));
    }
}

__global__ __launch_bounds__(kBlock) void k_member_scatter(int64_t n, const int32_t *__restrict__ agg,
                                                           const int64_t *__restrict__ moff,
                                                           const int32_t *__restrict__ rank,
                                                           int32_t *__restrict__ members) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock) {
        const int32_t a = agg[v];
        if (a >= 0) members[moff[a] + rank[v]] = (int32_t)v;
    }
}

// The same, with the offsets, for small graphs: one workgroup, the counts in LDS
// (one launch of 6 us instead of five: fill, ranks, scan, scatter).
constexpr int kFewThreads = 1024, kFewVertices = 8192;

__global__ __launch_bounds__(kFewThreads) void k_member_few(int n, const int32_t *__restrict__ agg,
                                                            int n_agg, uint32_t *__restrict__ cnt,
                                                            int64_t *__restrict__ moff,
                                                            int32_t *__restrict__ members) {
    constexpr int kPer = kFewVertices / kFewThreads;
    __shared__ uint32_t at[kFewVertices];
    __shared__ uint32_t wsum[kFewThreads / 64];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < n_agg; i += kFewThreads) at[i] = 0u;
    __syncthreads();
    int32_t a[kPer];
    uint32_t rank[kPer];
#pragma unroll
    for (int k = 0; k < kPer; k++) {
        const int v = k * kFewThreads + tid;
        a[k] = v < n ? agg[v] : -1;
    }
#pragma unroll
    for (int k = 0; k < kPer; k++)
        if (a[k] >= 0) rank[k] = atomicAdd(&at[a[k]], 1u);
    __syncthreads();
    // the offsets: kPer counts in a row per thread
    uint32_t c[kPer], mine = 0;
#pragma unroll
    for (int k = 0; k < kPer; k++) {
        const int i = tid * kPer + k;
        c[k] = i < n_agg ? at[i] : 0u;
        mine += c[k];
    }
    const uint32_t incl = wave_incl_scan(mine);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - mine;
    for (int w = 0; w < wave; w++) run += wsum[w];
#pragma unroll
    for (int k = 0; k < kPer; k++) {
        const int i = tid * kPer + k;
        if (i < n_agg) {
            at[i] = run;
            cnt[i] = c[k];
            moff[i] = (int64_t)run;
        }
        run += c[k];
    }
    if (tid == kFewThreads - 1) moff[n_agg] = (int64_t)run;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; k++)
        if (a[k] >= 0) members[at[a[k]] + rank[k]] = k * kFewThreads + tid;
}

// Sum over the workgroup (all threads must call it; result in every thread).
__device__ __forceinline__ unsigned long long block_sum(unsigned long long x,
                                                        unsigned long long *scratch) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) scratch[threadIdx.x >> 6] = x;
    __syncthreads();
    unsigned long long t = 0;
    for (int w = 0; w < kWaves; w++) t += scratch[w];
    return t;
}

// Minimum of *mn and maximum of *mx over the workgroup, in every thread (all
// threads must call it).
__device__ __forceinline__ void block_minmax(int32_t *mn, int32_t *mx, int32_t *scratch) {
    int32_t a = *mn, b = *mx;
    for (int off = 32; off > 0; off >>= 1) {
        a = min(a, __shfl_xor(a, off, 64));
        b = max(b, __shfl_xor(b, off, 64));
    }
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) {
        scratch[threadIdx.x >> 6] = a;
        scratch[kWaves + (threadIdx.x >> 6)] = b;
    }
    __syncthreads();
    for (int w = 0; w < kWaves; w++) {
        a = min(a, scratch[w]);
        b = max(b, scratch[kWaves + w]);
    }
    *mn = a;
    *mx = b;
}

// Exclusive prefix of x over the workgroup in thread order; *total gets the
// sum.  All threads must call it.
__device__ __forceinline__ uint32_t block_excl(uint32_t x, uint32_t *scratch, uint32_t *total) {
    const int wave = (int)(threadIdx.x >> 6);
    const uint32_t incl = wave_incl_scan(x);
    __syncthreads();
    if ((threadIdx.x & 63u) == 63u) scratch[wave] = incl;
    __syncthreads();
    uint32_t before = 0, t = 0;
    for (int w = 0; w < kWaves; w++) {
        if (w < wave) before += scratch[w];
        t += scratch[w];
    }
    *total = t;
    return before + incl - x;
}

__device__ __forceinline__ unsigned long long block_excl(unsigned long long x,
                                                         unsigned long long *scratch,
                                                         unsigned long long *total) {
    const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
    unsigned long long incl = x;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    __syncthreads();
    if (lane == 63) scratch[wave] = incl;
    __syncthreads();
    unsigned long long before = 0, t = 0;
    for (int w = 0; w < kWaves; w++) {
        if (w < wave) before += scratch[w];
        t += scratch[w];
    }
    *total = t;
    return before + incl - x;
}

// LDS of walk_members: the entry offsets of one chunk of kBlock members, and
// each member row's start less its offset.  Off: 32 bits unless the graph has
// 2^32 entries or more.
template <typename Off>
struct WalkLds {
    Off off[kBlock + 1];
    int64_t base[kBlock];
    Off scan[kWaves];
};

// f(c) for the coarse id c = agg[col[j]] of every entry j of every member of
// an aggregate (members[m0 .. m1)).  The members go in chunks of kBlock; the
// chunk's entries are numbered through a prefix sum of the row lengths and
// dealt out evenly, kWEdges in a row per thread loaded together.  Rows of any
// length mix keep every thread equally busy.  Several workgroups can share
// one chunk: `part` of `parts` takes every parts-th block of its entries.
// All threads must call it.
template <typename Off, typename F>
__device__ __forceinline__ void walk_members(const int64_t *__restrict__ row_ptr,
                                             const int32_t *__restrict__ col,
                                             const int32_t *__restrict__ agg,
                                             const int32_t *__restrict__ members, int64_t m0,
                                             int64_t m1, WalkLds<Off> &w, int part, int parts,
                                             F f) {
    const int tid = (int)threadIdx.x;
    for (int64_t c0 = m0; c0 < m1; c0 += kBlock) {
        const int64_t i = c0 + tid;
        int64_t rs = 0;
        Off len = 0;
        if (i < m1) {
            const int32_t v = members[i];
            rs = row_ptr[v];
            len = (Off)(row_ptr[v + 1] - rs);
        }
        Off tot;
        const Off ex = block_excl(len, w.scan, &tot);
        w.off[tid] = ex;
        w.base[tid] = rs - (int64_t)ex;
        if (tid == 0) w.off[kBlock] = tot;
        __syncthreads();
        for (Off c1 = (Off)part * (kBlock * kWEdges); c1 < tot;) {
            const Off q0 = c1 + (Off)(tid * kWEdges);
            if (q0 < tot && q0 >= c1) {
                int64_t at[kWEdges];
                walk_run<kBlock, kWEdges>(w.off, w.base, q0, tot, at);
                int32_t x[kWEdges];
#pragma unroll
                for (int k = 0; k < kWEdges; k++) x[k] = col[at[k]];
                int32_t c[kWEdges];
#pragma unroll
                for (int k = 0; k < kWEdges; k++) c[k] = agg[x[k]];
#pragma unroll
                for (int k = 0; k < kWEdges; k++)
                    if (tot - q0 > (Off)k) f(c[k]);
            }
            const Off step = (Off)(kBlock * kWEdges) * (Off)parts;
            if (tot - c1 <= step) break;  // c1 does not wrap
            c1 += step;
        }
        __syncthreads();  // the offsets are rewritten by the next chunk
    }
}

// The set bits of words [w0, w1) of buf, which stand for the ids from `id0`
// on, in increasing order to dst (nullptr: only counted).  Every thread takes
// a run of words, so one prefix sum numbers them all (runs of odd length:
// their LDS reads spread over the banks).  All threads must call it.
__device__ __forceinline__ uint32_t emit_bits(const uint32_t *buf, int w0, int w1, int64_t id0,
                                              int32_t *dst, uint32_t *scan_s) {
    const int run = ((w1 - w0 + kBlock - 1) / kBlock) | 1;
    const int b = min(w1, w0 + (int)threadIdx.x * run), e = min(w1, b + run);
    uint32_t cnt = 0;
    for (int i = b; i < e; i++) cnt += (uint32_t)__popc(buf[i]);
    uint32_t tot;
    uint32_t pos = block_excl(cnt, scan_s, &tot);
    if (dst) {
        for (int i = b; i < e; i++) {
            uint32_t word = buf[i];
            while (word) {
                const int bit = __ffs(word) - 1;
                word &= word - 1;
                dst[pos++] = (int32_t)(id0 + (int64_t)i * 32 + bit);
            }
        }
    }
    return tot;
}

// The rows of class 2, one workgroup each.  A workgroup owns the rows
// blockIdx.x, blockIdx.x + gridDim.x, ... and reads kBlock of their classes at
// a time.
// The row's ids are collected in an LDS bitmap of `words` words (all coarse
// ids, or kBitWords of them at a time); its size, and so the workgroups a
// compute unit holds, follows the number of coarse ids.
// FILL = false: ccnt[a], and the row itself where one window holds every
// coarse id and the spare buffer has room (class 3).
// FILL = true: the rows still of class 2 to ccol[crow[a] ...].
template <bool FILL, typename Off>
__global__ __launch_bounds__(kBlock) void k_coarse_rows(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const int32_t *__restrict__ agg, int64_t n_agg, const int64_t *__restrict__ moff,
    const int32_t *__restrict__ members, uint32_t *__restrict__ ccnt,
    const int64_t *__restrict__ crow, int32_t *__restrict__ ccol, uint8_t *__restrict__ cls,
    uint32_t *__restrict__ gmeta, uint32_t slots, int words, Spare sp) {
    extern __shared__ uint32_t buf[];
    __shared__ unsigned long long red[kWaves];
    __shared__ uint32_t scan_s[kWaves];
    __shared__ WalkLds<Off> walk;
    __shared__ int32_t range_s[2 * kWaves];
    __shared__ uint32_t giant_s;
    __shared__ int64_t at_s;
    const int tid = (int)threadIdx.x;
    const int64_t window = 32 * (int64_t)words;
    auto row = [&](const int64_t a) {
        const int64_t m0 = moff[a], m1 = moff[a + 1];
        if (gmeta) {
            unsigned long long cand = 0;
            for (int64_t i = m0 + tid; i < m1; i += kBlock) {
                const int32_t v = members[i];
                cand += (unsigned long long)(row_ptr[v + 1] - row_ptr[v]);
            }
            cand = block_sum(cand, red);
            if (cand > (unsigned long long)kGiantCand) {
                // a giant row: the count pass claims a bitmap slot for it (the
                // slot kernels then count and write it); without a free slot
                // it stays here
                if (tid == 0) {
                    uint32_t taken = 0;
                    if (!FILL) {
                        const uint32_t k = atomicAdd(&gmeta[3 * kGiantSlots], 1u);
                        if (k < slots) {
                            gmeta[k] = (uint32_t)a;
                            taken = 1;
                        }
                    } else {
                        const uint32_t cnt = min(gmeta[3 * kGiantSlots], slots);
                        for (uint32_t k = 0; k < cnt; k++) taken |= gmeta[k] == (uint32_t)a ? 1u : 0u;
                    }
                    giant_s = taken;
                }
                __syncthreads();
                if (giant_s) return;  // uniform; the next block_sum synchronises first
            }
        }
        // bitmap windows over the coarse id space.  The first window also
        // finds the smallest and largest candidate; later windows cover only
        // that range, and each window emits only the words inside it.  In a
        // disjoint union the candidates lie in the row's own graph, so a big
        // row never sweeps the coarse ids of the other graphs.
        uint32_t run = 0;
        int64_t hi = n_agg;
        int32_t tmin = INT32_MAX, tmax = -1;
        bool first = true;
        for (int64_t lo = 0; lo < hi;) {
            for (int i = tid; i < words; i += kBlock) buf[i] = 0u;
            __syncthreads();
            walk_members(row_ptr, col, agg, members, m0, m1, walk, 0, 1, [&](int32_t c) {
                if (c < 0 || (int64_t)c == a) return;
                if (first) {
                    tmin = min(tmin, c);
                    tmax = max(tmax, c);
                }
                const int64_t o = (int64_t)c - lo;
                if (o < 0 || o >= window) return;
                const uint32_t bit = 1u << (o & 31);
                if (!(buf[o >> 5] & bit)) atomicOr(&buf[o >> 5], bit);
            });
            __syncthreads();
            if (first) {
                block_minmax(&tmin, &tmax, range_s);
                hi = (int64_t)tmax + 1;  // no candidate at all: tmax = -1 ends the sweep
            }
            const int64_t e_lo = max(lo, (int64_t)tmin);
            const int64_t e_hi = min(lo + window, hi);
            if (e_lo < e_hi) {
                const int w0 = (int)((e_lo - lo) >> 5), w1 = (int)((e_hi - lo + 31) >> 5);
                int32_t *dst = FILL ? ccol + crow[a] + run : nullptr;
                uint32_t tot = 0;
                if (!FILL) {
                    // its size first, then a place for it
                    tot = emit_bits(buf, w0, w1, lo, nullptr, scan_s);
                    if (window >= n_agg) {
                        if (tid == 0) {
                            at_s = spare_take(sp, (uint32_t)blockIdx.x, tot);
                            if (at_s >= 0) {
                                cls[a] = kSpared;
                                spare_note(sp, m0, at_s);
                            }
                        }
                        __syncthreads();
                        if (at_s >= 0) dst = sp.buf + at_s;
                    }
                }
                if (dst) tot = emit_bits(buf, w0, w1, lo, dst, scan_s);
                run += tot;
            }
            __syncthreads();
            int64_t next = lo + window;
            if (first) {
                if ((int64_t)tmin > next) next = tmin;
                first = false;
            }
            lo = next;
        }
        if (!FILL && tid == 0) ccnt[a] = run;
        __syncthreads();
    };
    __shared__ uint64_t marks[kWaves];
    for (int64_t j0 = 0; (int64_t)blockIdx.x + j0 * gridDim.x < n_agg; j0 += kBlock) {
        const int64_t v = (int64_t)blockIdx.x + (j0 + tid) * gridDim.x;
        const uint64_t mine = __ballot(v < n_agg && cls[v] == kBig);
        __syncthreads();  // the marks before are read, and no row changes its class yet
        if ((tid & 63) == 0) marks[tid >> 6] = mine;
        __syncthreads();
        for (int w = 0; w < kWaves; w++) {
            uint64_t mask = marks[w];
            while (mask) {
                const int r = __ffsll((unsigned long long)mask) - 1;
                mask &= mask - 1;
                row((int64_t)blockIdx.x + (j0 + w * 64 + r) * gridDim.x);
            }
        }
    }
}

// Giant rows, one bitmap slot each (gmeta: rows [0, S), INT32_MAX less the
// smallest ids [S, 2S), the largest ids plus one [2S, 3S), rows claimed [3S]; all
// zero before a count pass).  Slots blockIdx.y, blockIdx.y + gridDim.y, ...; the
// workgroups of a slot share its members in chunks of kBlock, kGiantParts
// workgroups to a chunk (a chunk that holds hubs has a hundred times the entries
// of another).  Where the coarse ids fit an LDS bitmap (words > 0) a workgroup
// collects its share there and adds its set words to the slot's once; else it sets
// every bit in the slot (a plain read first skips bits it sees already set).  Most
// candidates of a giant row repeat: a row of 2.3 million candidates held 6000
// distinct ids, and setting each in global memory put every workgroup's
// atomics on the same few lines.
constexpr int kGiantParts = 8;
template <typename Off>
__global__ __launch_bounds__(kBlock) void k_giant_set(const int64_t *__restrict__ row_ptr,
                                                      const int32_t *__restrict__ col,
                                                      const int32_t *__restrict__ agg,
                                                      const int64_t *__restrict__ moff,
                                                      const int32_t *__restrict__ members,
                                                      uint32_t *__restrict__ gbits, int64_t stride,
                                                      uint32_t *__restrict__ gmeta, uint32_t slots,
                                                      int words) {
    extern __shared__ uint32_t buf[];
    __shared__ WalkLds<Off> walk;
    __shared__ int32_t range_s[2 * kWaves];
    const int used = (int)min(gmeta[3 * kGiantSlots], slots);
    const int part = (int)(blockIdx.x % kGiantParts);
    for (int slot = (int)blockIdx.y; slot < used; slot += (int)gridDim.y) {
        const int64_t a = gmeta[slot];
        const int64_t m0 = moff[a], m1 = moff[a + 1];
        if (m0 + (int64_t)(blockIdx.x / kGiantParts) * kBlock >= m1) continue;
        uint32_t *bits = gbits + (int64_t)slot * stride;
        for (int i = (int)threadIdx.x; i < words; i += kBlock) buf[i] = 0u;
        __syncthreads();
        int32_t tmin = INT32_MAX, tmax = -1;
        auto set = [&](int32_t c, uint32_t *to) {
            if (c < 0 || (int64_t)c == a) return;
            tmin = min(tmin, c);
            tmax = max(tmax, c);
            const uint32_t bit = 1u << (c & 31);
            if (!(to[c >> 5] & bit)) atomicOr(&to[c >> 5], bit);
        };
        for (int64_t c0 = m0 + (int64_t)(blockIdx.x / kGiantParts) * kBlock; c0 < m1;
             c0 += (int64_t)(gridDim.x / kGiantParts) * kBlock) {
            const int64_t c1 = min(c0 + kBlock, m1);
            if (words)
                walk_members(row_ptr, col, agg, members, c0, c1, walk, part, kGiantParts,
                             [&](int32_t c) { set(c, buf); });
            else
                walk_members(row_ptr, col, agg, members, c0, c1, walk, part, kGiantParts,
                             [&](int32_t c) { set(c, bits); });
        }
        block_minmax(&tmin, &tmax, range_s);
        if (tmax >= 0) {
            if (words)
                for (int i = (tmin >> 5) + (int)threadIdx.x; i <= tmax >> 5; i += kBlock)
                    if (buf[i]) atomicOr(&bits[i], buf[i]);
            if (threadIdx.x == 0) {
                atomicMax(&gmeta[kGiantSlots + slot], (uint32_t)(INT32_MAX - tmin));
                atomicMax(&gmeta[2 * kGiantSlots + slot], (uint32_t)(tmax + 1));
            }
        }
        __syncthreads();  // the bitmap is cleared for the next slot
    }
}

// One workgroup per giant slot: FILL = false: ccnt[a] = the bits set;
// FILL = true: their ids in increasing order to ccol[crow[a] ...].  Each
// thread takes kRun words in a row, so a prefix sum covers kRun * kBlock.
template <bool FILL>
__global__ __launch_bounds__(kBlock) void k_giant_emit(const uint32_t *__restrict__ gbits,
                                                       int64_t words,
                                                       const uint32_t *__restrict__ gmeta,
                                                       uint32_t slots, uint32_t *__restrict__ ccnt,
                                                       const int64_t *__restrict__ crow,
                                                       int32_t *__restrict__ ccol) {
    constexpr int kRun = 8;
    __shared__ uint32_t scan_s[kWaves];
    const int slot = (int)blockIdx.x;
    if ((uint32_t)slot >= min(gmeta[3 * kGiantSlots], slots)) return;
    const int64_t a = gmeta[slot];
    const int32_t lo = INT32_MAX - (int32_t)gmeta[kGiantSlots + slot];
    const int32_t hi = (int32_t)gmeta[2 * kGiantSlots + slot] - 1;
    const uint32_t *bits = gbits + (int64_t)slot * words;
    uint32_t run = 0;
    if (hi >= 0) {
        const int64_t w0 = lo >> 5, w1 = ((int64_t)hi >> 5) + 1;
        for (int64_t c0 = w0; c0 < w1; c0 += kBlock * kRun) {
            const int64_t wi = c0 + (int64_t)threadIdx.x * kRun;
            uint32_t word[kRun], cnt = 0;
#pragma unroll
            for (int k = 0; k < kRun; k++) {
                word[k] = bits[min(wi + k, w1 - 1)];
                if (wi + k >= w1) word[k] = 0u;
                cnt += (uint32_t)__popc(word[k]);
            }
            uint32_t tot;
            const uint32_t pos = block_excl(cnt, scan_s, &tot);
            if (FILL) {
                int32_t *dst = ccol + crow[a] + run + pos;
#pragma unroll
                for (int k = 0; k < kRun; k++) {
                    uint32_t wv = word[k];
                    while (wv) {
                        const int bit = __ffs(wv) - 1;
                        wv &= wv - 1;
                        *dst++ = (int32_t)((wi + k) * 32 + bit);
                    }
                }
            }
            run += tot;
        }
    }
    if (!FILL && threadIdx.x == 0) ccnt[a] = run;
}

int grid_for(int64_t work, int per_block, int cap) {
    int64_t b = (work + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

}  // namespace

namespace {

// cnt is zero already (cleared), unless the few-vertices kernel clears its own.
hipError_t member_lists(int64_t n, const int32_t *agg, int64_t n_agg, uint32_t *cnt, int64_t *moff,
                        unsigned long long *part, int32_t *rank, int32_t *members, bool cleared,
                        hipStream_t s) {
    hipError_t e;
    if (n <= kFewVertices && n_agg <= kFewVertices) {
        hipLaunchKernelGGL(k_member_few, dim3(1), dim3(kFewThreads), 0, s, (int)n, agg, (int)n_agg,
                           cnt, moff, members);
        return hipGetLastError();
    }
    if (!cleared && (e = launch_fill_u32(cnt, 0u, n_agg, s)) != hipSuccess) return e;
    const int blocks = grid_for(n, kBlock, 8192);
    if (n > 0)
        hipLaunchKernelGGL(k_member_rank, dim3(blocks), dim3(kBlock), 0, s, n, agg, cnt, rank);
    if ((e = exclusive_scan_u32_i64(cnt, n_agg, moff, part, s)) != hipSuccess) return e;
    if (n > 0)
        hipLaunchKernelGGL(k_member_scatter, dim3(blocks), dim3(kBlock), 0, s, n, agg,
                           (const int64_t *)moff, (const int32_t *)rank, members);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_member_lists(int64_t n, const int32_t *agg, int64_t n_agg, uint32_t *cnt,
                               int64_t *moff, unsigned long long *part, int32_t *rank,
                               int32_t *members, hipStream_t s) {
    return member_lists(n, agg, n_agg, cnt, moff, part, rank, members, false, s);
}

hipError_t quotient_graph(const int64_t *row_ptr, const int32_t *col, int64_t n, int64_t nnz,
                          const int32_t *agg, int64_t n_agg, int64_t *crow, int32_t *ccol,
                          const QuotientWs &q, unsigned long long *host_nnz, hipStream_t s) {
    hipError_t e;
    // no coarse row has more candidates than the fine graph has entries
    const bool giant = nnz > kGiantCand && n_agg > 0;
    const int64_t words = (int64_t)giant_words(n_agg);
    uint32_t *gmeta = giant ? q.gmeta : nullptr;
    // as many bitmap slots as the workspace's bits for n ids make
    const uint32_t slots = (uint32_t)std::min<int64_t>(
        kGiantSlots, kGiantShare * (int64_t)giant_words(n) / std::max<int64_t>(words, 1));
    // 16 lanes per row up to 256 candidates a row on average, else 64
    const bool narrow = nnz <= 256 * n_agg;
    const uint32_t maxc = narrow ? 512u : 16384u;
    const int gblocks = (grid_for(n_agg, kBlock / (narrow ? 16 : 64), 4096) + 7) / 8 * 8;
    const int wblocks = grid_for(n_agg, kWaves, 8192);
    const int bblocks = grid_for(n_agg, 1, 2048);  // about what is resident at once
    const bool hashed = words > kBitWords;         // second path between the first and a workgroup
    // the spare buffer holds 9 or more entries a vertex; nearly all aggregates
    // of a mesh have at most 6 neighbours a member
    Spare sp;
    sp.buf = q.tmp;
    sp.per = 6;
    const int64_t rest = (n * sp.per + 63) / 64 * 64;  // the cursors begin a cache line
    sp.cursor = (uint32_t *)(q.tmp + rest);
    sp.base = rest + kSpareParts * kSpareLine;
    sp.cap = (uint32_t)std::min<int64_t>(std::max<int64_t>(q.tmp_cap - sp.base, 0) / kSpareParts,
                                         (int64_t)1 << 26);
    // the LDS bitmap of a workgroup: all coarse ids if they fit
    const int bwords = (int)std::min<int64_t>(words, kBitWords);
    const bool wide = nnz > 0xFFFFFFFFll;
    {
        FillSpans f;  // all that has to be clear, in one launch
        f.add(q.cnt, 0u, n_agg);
        f.add(sp.cursor, 0u, kSpareParts * kSpareLine);
        if (giant) f.add(q.gbits, 0u, (int64_t)slots * words);
        if (giant) f.add(q.gmeta, 0u, kGiantMeta);
        if ((e = launch_fill_spans(f, s)) != hipSuccess) return e;
    }
    if ((e = member_lists(n, agg, n_agg, q.cnt, q.moff, q.part, q.rank, q.members, true, s)) !=
        hipSuccess)
        return e;
    auto group = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(gblocks), dim3(kBlock), 0, s, row_ptr, col, agg, n_agg,
                           q.moff, q.members, maxc, q.cnt, sp, q.cls,
                           hashed ? kSecond : kBig);
    };
    auto big = [&](auto kernel, const int64_t *rows, int32_t *cols) {
        hipLaunchKernelGGL(kernel, dim3(bblocks), dim3(kBlock), 4 * (size_t)bwords, s, row_ptr, col,
                           agg, n_agg, q.moff, q.members, q.cnt, rows, cols, q.cls, gmeta, slots,
                           bwords, sp);
    };
    if (n_agg > 0) {
        if (narrow)
            group(k_coarse_rows_group<16, 128, 96, 4>);
        else
            group(k_coarse_rows_group<64, 256, 160, 8>);
        if (hashed)
            hipLaunchKernelGGL(k_coarse_rows_wave<false>, dim3(wblocks), dim3(kBlock), 0, s,
                               row_ptr, col, agg, n_agg, q.moff, q.members, q.cnt,
                               (const int64_t *)nullptr, (int32_t *)nullptr, q.cls, sp);
        if (wide)
            big(k_coarse_rows<false, unsigned long long>, nullptr, nullptr);
        else
            big(k_coarse_rows<false, uint32_t>, nullptr, nullptr);
    }
    if (giant) {
        const int gwords = words <= kBitWords ? (int)words : 0;
        auto set = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(512, 8), dim3(kBlock), 4 * (size_t)gwords, s,
                               row_ptr, col, agg, q.moff, q.members, q.gbits, words, q.gmeta, slots,
                               gwords);
        };
        if (wide)
            set(k_giant_set<unsigned long long>);
        else
            set(k_giant_set<uint32_t>);
        hipLaunchKernelGGL(k_giant_emit<false>, dim3(slots), dim3(kBlock), 0, s,
                           (const uint32_t *)q.gbits, words, (const uint32_t *)q.gmeta, slots, q.cnt,
                           (const int64_t *)nullptr, (int32_t *)nullptr);
    }
    ScanHost host;
    host.word = host_nnz;
    if ((e = exclusive_scan_u32_i64(q.cnt, n_agg, crow, q.part, s, host)) != hipSuccess) return e;
    if (n_agg > 0) {
        hipLaunchKernelGGL(k_copy_rows, dim3(grid_for(n_agg, kBlock / 16, 2048)), dim3(kBlock), 0,
                           s, n_agg, q.moff, (const int64_t *)crow, (const uint8_t *)q.cls, sp,
                           ccol);
        if (hashed)
            hipLaunchKernelGGL(k_coarse_rows_wave<true>, dim3(wblocks), dim3(kBlock), 0, s, row_ptr,
                               col, agg, n_agg, q.moff, q.members, q.cnt, (const int64_t *)crow,
                               ccol, q.cls, sp);
        if (wide)
            big(k_coarse_rows<true, unsigned long long>, crow, ccol);
        else
            big(k_coarse_rows<true, uint32_t>, crow, ccol);
    }
    if (giant)
        hipLaunchKernelGGL(k_giant_emit<true>, dim3(slots), dim3(kBlock), 0, s,
                           (const uint32_t *)q.gbits, words, (const uint32_t *)q.gmeta, slots, q.cnt,
                           crow, ccol);
    return hipGetLastError();
}

}  // namespace mis2
