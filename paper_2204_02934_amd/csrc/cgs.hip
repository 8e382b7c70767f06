// cgs.hip -- cluster multicolor Gauss-Seidel (Algorithm 4, Section III-C) on gfx950.
//
// Setup colours a graph (the coarse graph of an aggregation, or the graph
// itself for point multicolor Gauss-Seidel) and orders the rows by colour,
// then by cluster, then by row id.  Apply runs, for each colour in turn, one
// wavefront per cluster: the wave updates its cluster's rows one after the
// other.  Clusters of one colour share no edge, so no wave reads a value
// another wave of the same launch writes, and the result is that of the
// sequential sweep in the same order.
//
// Colouring (the paper takes it from other work): Jones-Plassmann with fixed
// priorities, the packed tuple of h(seed, 0, v) (Sections V-A, V-C): every
// uncoloured vertex whose tuple is below those of its uncoloured neighbours
// takes the smallest colour no coloured neighbour has.  A vertex is coloured
// only after all its neighbours of lower tuple and before all those of higher
// tuple, so its colour is the smallest one its lower neighbours leave: the
// result is that of colouring the vertices one by one in tuple order, whatever
// subset of the ready ones a pass happens to colour.
#include "internal.h"
#include "lanes.h"

namespace mis2 {

namespace {

// State of a vertex: its tuple in the low word, its colour (-1: none yet) in
// the high one.
__device__ __forceinline__ unsigned long long jp_state(uint32_t tuple, int32_t color) {
    return (unsigned long long)tuple | ((unsigned long long)(uint32_t)color << 32);
}

__global__ __launch_bounds__(kBlock) void k_jp_init(int64_t n, TupleParams tp,
                                                    unsigned long long *__restrict__ st) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        st[v] = jp_state(make_tuple(tp, (uint32_t)v), -1);
}

constexpr int kJpLoads = 8;  // entries of a row loaded together

// kJpPasses passes over the uncoloured vertices.  Wavefront w owns the
// vertices [w * seg, (w + 1) * seg) and keeps those still uncoloured, in
// order, in list[w * seg ...] and their number in cnt[w] (first launch: all of
// them).  One lane per vertex; a neighbour's state is one 8-byte load, so a
// vertex either sees its colour and tuple together or finds it uncoloured
// and waits.  The loads and stores of states are relaxed atomics: they see
// what other workgroups coloured a moment ago (those of the same XCD share
// its L2, and each XCD owns one run of vertices), so one launch colours
// several links of a chain of neighbours; a colour missed is seen by the next
// launch.  *left = 1 when a vertex stays uncoloured, *maxc is raised to the
// largest colour given.
// One launch per round over every vertex, with the round of each neighbour
// and then its tuple loaded entry by entry, took 1.72 ms (21 launches of 82 us)
// on the 7-point 100^3 grid.
constexpr int kJpPasses = 4;
__global__ __launch_bounds__(kBlock) void k_jp_pass(int64_t n, const int64_t *__restrict__ row_ptr,
                                                    const int32_t *__restrict__ col,
                                                    unsigned long long *st,
                                                    int32_t *__restrict__ color, int32_t *list,
                                                    uint32_t *__restrict__ cnt, int64_t seg,
                                                    int first, uint32_t *__restrict__ left,
                                                    uint32_t *__restrict__ maxc) {
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t blk = (int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int64_t w = blk * (kBlock / 64) + (threadIdx.x >> 6);
    const int64_t base = w * seg;
    int64_t m = first ? max((int64_t)0, min(seg, n - base)) : (int64_t)cnt[w];
    int32_t best = -1;
    for (int pass = 0; pass < kJpPasses && m > 0; pass++) {
        int64_t out = 0;
        for (int64_t i0 = 0; i0 < m; i0 += 64) {
            const bool mine = i0 + lane < m;
            const int64_t at = base + (mine ? i0 + lane : i0);
            const int64_t v = first && pass == 0 ? at : (int64_t)list[at];
            const int64_t s = row_ptr[v], e = row_ptr[v + 1];
            const uint32_t pv = (uint32_t)st[v];
            bool wait = !mine;
            uint64_t used = 0;
            for (int64_t j = s; j < e && !wait; j += kJpLoads) {
                int32_t x[kJpLoads];
#pragma unroll
                for (int k = 0; k < kJpLoads; k++) x[k] = col[min(j + k, e - 1)];
                unsigned long long y[kJpLoads];
#pragma unroll
                for (int k = 0; k < kJpLoads; k++)
                    y[k] = __hip_atomic_load(&st[x[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int k = 0; k < kJpLoads; k++) {
                    const int32_t c = (int32_t)(y[k] >> 32);
                    if (c < 0 && (uint32_t)y[k] < pv) wait = true;
                    if (c >= 0 && c < 64) used |= 1ull << c;
                }
            }
            if (!wait) {
                // every neighbour of lower tuple is coloured, for good
                int32_t c = used != ~0ull ? __ffsll((unsigned long long)~used) - 1 : 64;
                for (int32_t b0 = 64; c == b0; b0 += 64) {  // all 64 colours before b0 taken
                    uint64_t u = 0;
                    for (int64_t j = s; j < e; j++) {
                        const int32_t d =
                            (int32_t)(__hip_atomic_load(&st[col[j]], __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) >> 32) - b0;
                        if (d >= 0 && d < 64) u |= 1ull << d;
                    }
                    c = u != ~0ull ? b0 + __ffsll((unsigned long long)~u) - 1 : b0 + 64;
                }
                __hip_atomic_store(&st[v], jp_state(pv, c), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                color[v] = c;
                best = max(best, c);
            }
            const uint64_t keep = __ballot(mine && wait);
            if (mine && wait)
                list[base + out + __popcll(keep & (lane ? ~0ull >> (64 - lane) : 0ull))] = (int32_t)v;
            out += __popcll(keep);
        }
        m = out;
        // this wavefront's list is read back by other lanes
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
    if (lane == 0) {
        cnt[w] = (uint32_t)m;
        if (m > 0) *left = 1u;
    }
    best = (int32_t)group_max<64>((uint32_t)(best + 1)) - 1;
    if (lane == 0 && best > (int32_t) * (volatile uint32_t *)maxc) atomicMax(maxc, (uint32_t)best);
}

// Ids in order of colour, then id: a counting sort.  cnt[c * tiles + t] = the
// ids of colour c in tile t of kColorTile ids; after a prefix sum over it,
// pos has where each run goes.
constexpr int kColorTile = 2048;
constexpr int kSortColors = 64;  // most colours
__global__ __launch_bounds__(kBlock) void k_color_count(int64_t n, const int32_t *__restrict__ color,
                                                        int32_t n_colors, int64_t tiles,
                                                        uint32_t *__restrict__ cnt) {
    __shared__ uint32_t h[kSortColors];
    if (threadIdx.x < kSortColors) h[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t t = blockIdx.x, e = min(n, (t + 1) * kColorTile);
    for (int64_t v = t * kColorTile + threadIdx.x; v < e; v += kBlock) atomicAdd(&h[color[v]], 1u);
    __syncthreads();
    if ((int)threadIdx.x < n_colors) cnt[(int64_t)threadIdx.x * tiles + t] = h[threadIdx.x];
}

// Each wavefront takes a quarter of the tile, 64 ids at a time; its lanes of
// one colour are numbered by a ballot.  first[c] = where colour c begins.
__global__ __launch_bounds__(kBlock) void k_color_scatter(int64_t n, const int32_t *__restrict__ color,
                                                          int32_t n_colors, int64_t tiles,
                                                          const int64_t *__restrict__ pos,
                                                          int32_t *__restrict__ out,
                                                          int64_t *__restrict__ first) {
    constexpr int kW = kBlock / 64, kPart = kColorTile / kW;
    __shared__ uint32_t h[kW][kSortColors];
    __shared__ int64_t at[kW][kSortColors];
    const int lane = (int)(threadIdx.x & 63u), wv = (int)(threadIdx.x >> 6);
    const int64_t t = blockIdx.x;
    const int64_t b = t * kColorTile + (int64_t)wv * kPart, e = min(n, b + kPart);
    h[wv][lane] = 0u;
    __syncthreads();
    for (int64_t v = b + lane; v < e; v += 64) atomicAdd(&h[wv][color[v]], 1u);
    __syncthreads();
    if (lane < n_colors) {
        int64_t o = pos[(int64_t)lane * tiles + t];
        if (t == 0 && wv == 0) first[lane] = o;
        for (int k = 0; k < wv; k++) o += h[k][lane];
        at[wv][lane] = o;
    }
    __syncthreads();
    for (int64_t v0 = b; v0 < e; v0 += 64) {
        const int64_t v = v0 + lane;
        const int32_t c = v < e ? color[v] : -1;
        uint64_t todo = __ballot(c >= 0);
        while (todo) {
            const int l = __ffsll((unsigned long long)todo) - 1;
            const int32_t cl = __builtin_amdgcn_readlane(c, l);
            const uint64_t same = __ballot(c == cl);
            const int64_t o = at[wv][cl];
            if (c == cl) out[o + __popcll(same & (lane ? ~0ull >> (64 - lane) : 0ull))] = (int32_t)v;
            __builtin_amdgcn_wave_barrier();  // o is read before it moves on
            if (lane == 0) at[wv][cl] = o + __popcll(same);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            todo &= ~same;
        }
    }
}

// The point plan: rows[k] (in order of colour) is the k-th cluster.
__global__ __launch_bounds__(kBlock) void k_point_plan(int64_t n, const int32_t *__restrict__ rows,
                                                       int32_t *__restrict__ pos,
                                                       int64_t *__restrict__ cluster_off) {
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k <= n;
         k += (int64_t)gridDim.x * kBlock) {
        cluster_off[k] = k;
        if (k < n) pos[rows[k]] = (int32_t)k;
    }
}

__global__ __launch_bounds__(kBlock) void k_iota(int64_t n, int32_t *__restrict__ out) {
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        out[v] = (int32_t)v;
}

// cnt[k] += the keys equal to k; one atomic for a run of equal keys.
__global__ __launch_bounds__(kBlock) void k_count_of(int64_t n, const int32_t *__restrict__ key,
                                                     uint32_t *__restrict__ cnt) {
    const int lane = (int)(threadIdx.x & 63u);
    // whole wavefronts stay in the loop together
    for (int64_t v0 = (int64_t)blockIdx.x * kBlock + (threadIdx.x - lane); v0 < n;
         v0 += (int64_t)gridDim.x * kBlock) {
        const int64_t v = v0 + lane;
        const int32_t k = v < n ? key[v] : -1;
        const int32_t prev = (int32_t)from_prev((uint32_t)k);
        const uint64_t heads = __ballot(lane == 0 || k != prev);
        const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1);
        const int len = later ? __ffsll((unsigned long long)later) : 64 - lane;
        if ((heads >> lane & 1u) && k >= 0) atomicAdd(&cnt[k], (uint32_t)len);
    }
}

// Colour histogram through a workgroup-local table (colours < kHistBins).
constexpr int kHistBins = 2048;
__global__ __launch_bounds__(kBlock) void k_color_hist(int64_t n, const int32_t *__restrict__ color,
                                                       int32_t n_colors, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[kHistBins];
    for (int k = threadIdx.x; k < n_colors; k += kBlock) h[k] = 0;
    __syncthreads();
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * kBlock)
        atomicAdd(&h[color[v]], 1u);
    __syncthreads();
    for (int k = threadIdx.x; k < n_colors; k += kBlock)
        if (h[k]) atomicAdd(&hist[k], h[k]);
}

constexpr int kSortRegs = 8;  // members per lane
constexpr int64_t kSmallCluster = 64 * kSortRegs;

// K members per lane of m in all.
template <int K>
__device__ __forceinline__ void sort_regs(int m, int32_t *members) {
    const int lane = threadIdx.x & 63;
    int32_t x[K];
    int rank[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        x[k] = k * 64 + lane < m ? members[k * 64 + lane] : 0x7fffffff;
        rank[k] = 0;
    }
#pragma unroll
    for (int q = 0; q < K; q++) {
        const int mq = m - q * 64 < 64 ? m - q * 64 : 64;
        for (int w = 0; w < mq; w++) {
            const int32_t y = __builtin_amdgcn_readlane(x[q], w);
#pragma unroll
            for (int k = 0; k < K; k++) rank[k] += y < x[k];
        }
    }
#pragma unroll
    for (int k = 0; k < K; k++)
        if (k * 64 + lane < m) members[rank[k]] = x[k];
}

// Each cluster of 2 .. kSmallCluster members: one wavefront, up to kSortRegs
// members per lane; a member's place is the number of smaller ones (ids are
// distinct), counted across the lanes.  Every member is in a register before
// any is written back.  (Clusters past 64 members sorted by a workgroup in
// global memory cost some 50 us each: a network of 28 passes and more.)
__global__ __launch_bounds__(kBlock) void k_sort_small(int64_t nc, const int64_t *__restrict__ moff,
                                                       int32_t *__restrict__ members) {
    const int lane = threadIdx.x & 63;
    const int64_t a = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (a >= nc) return;
    const int64_t s = moff[a], m = moff[a + 1] - s;
    if (m < 2 || m > kSmallCluster) return;
    if (m <= 64) {
        const int32_t x = lane < m ? members[s + lane] : 0x7fffffff;
        int rank = 0;
        for (int w = 0; w < (int)m; w++) rank += __builtin_amdgcn_readlane(x, w) < x;
        if (lane < m) members[s + rank] = x;
        return;
    }
    if (m <= 128)
        sort_regs<2>((int)m, members + s);
    else
        sort_regs<kSortRegs>((int)m, members + s);
}

// Each larger cluster: one workgroup sorts it with a bitonic network on the
// next power of two, positions past the end reading as +inf, in LDS up to
// kSortLds members, else in place.  The network's first step of every merge
// compares i with i ^ (k - 1) and the later ones i with i ^ j, always the
// smaller value to the lower index, so no real value ever moves past the end.
// A workgroup owns a run of clusters, reads kBlock of their sizes at once and
// sorts the large ones among them (reading them one after the other took 31 us
// on 14 000 clusters, 249 us on a million without a large one).
constexpr int kSortLds = 4096;

template <typename M>
__device__ __forceinline__ void sort_network(M m, int64_t size) {
    int64_t P = 1;
    while (P < size) P <<= 1;
    for (int64_t k = 2; k <= P; k <<= 1) {
        for (int64_t j = k >> 1; j > 0; j >>= 1) {
            for (int64_t i = threadIdx.x; i < P; i += kBlock) {
                const int64_t p = (j == (k >> 1)) ? (i ^ (k - 1)) : (i ^ j);
                if (p > i && p < size) {
                    const int32_t x = m[i], y = m[p];
                    if (x > y) {
                        m[i] = y;
                        m[p] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_sort_large(int64_t nc, const int64_t *__restrict__ moff,
                                                       int32_t *__restrict__ members) {
    __shared__ uint64_t large[kBlock / 64];
    __shared__ int32_t buf[kSortLds];
    const int64_t run = (nc + gridDim.x - 1) / gridDim.x;
    const int64_t last = min(nc, (blockIdx.x + 1) * run);
    for (int64_t a0 = blockIdx.x * run; a0 < last; a0 += kBlock) {
        const int64_t own = a0 + threadIdx.x;
        const uint64_t mine = __ballot(own < last && moff[own + 1] - moff[own] > kSmallCluster);
        __syncthreads();
        if ((threadIdx.x & 63u) == 0) large[threadIdx.x >> 6] = mine;
        __syncthreads();
        for (int w = 0; w < kBlock / 64; w++) {
            for (uint64_t mask = large[w]; mask; mask &= mask - 1) {
                const int64_t a = a0 + w * 64 + __ffsll((unsigned long long)mask) - 1;
                const int64_t s = moff[a], size = moff[a + 1] - s;
                if (size > kSortLds) {
                    sort_network(members + s, size);
                    continue;
                }
                for (int64_t i = threadIdx.x; i < size; i += kBlock) buf[i] = members[s + i];
                __syncthreads();
                sort_network(&buf[0], size);
                for (int64_t i = threadIdx.x; i < size; i += kBlock) members[s + i] = buf[i];
                __syncthreads();
            }
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_gather_sizes(int64_t nk, const int32_t *__restrict__ order,
                                                         const uint32_t *__restrict__ cnt,
                                                         uint32_t *__restrict__ out) {
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < nk;
         k += (int64_t)gridDim.x * kBlock)
        out[k] = cnt[order[k]];
}

// rows[cluster_off[k] ...] = the sorted members of the k-th cluster of the
// sweep order.
__global__ __launch_bounds__(kBlock) void k_place_rows(int64_t nk, const int32_t *__restrict__ order,
                                                       const int64_t *__restrict__ moff,
                                                       const int32_t *__restrict__ members,
                                                       const int64_t *__restrict__ cluster_off,
                                                       int32_t *__restrict__ rows) {
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < nk;
         k += (int64_t)gridDim.x * kBlock) {
        const int32_t a = order[k];
        const int64_t s = moff[a], e = moff[a + 1], o = cluster_off[k];
        for (int64_t t = s; t < e; t++) rows[o + t - s] = members[t];
    }
}

// One colour of a sweep: the sweep-order clusters [k0, k1), one lane each,
// rows in order (or reversed).  The update of row i is
// x_i = (b_i - sum over its off-diagonal entries of a_ij x_j) / d_i, summed
// in CSR order with separate roundings (no fused multiply-add), as the
// sequential sweep does it.
__global__ __launch_bounds__(kBlock) void k_scatter_pos(int64_t n, const int32_t *__restrict__ rows,
                                                        int32_t *__restrict__ pos) {
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * kBlock)
        pos[rows[t]] = (int32_t)t;
}

// ---- apply ----------------------------------------------------------------
//
// One wavefront per cluster.  The cluster's rows are taken in batches of at
// most 64 rows of at most 64 entries each and Cap entries in all; lane k
// holds the batch's k-th row.  The batch is staged in LDS in parallel: for
// each entry (row order, then CSR order) either the product a_ij * x_j with
// index kOne (x_j is final for this pass when j is not a row of the batch:
// another colour's x, a row of this cluster updated in an earlier batch, or
// one not yet reached, whose old value Gauss-Seidel uses), or a_ij with the
// batch index of j.  xb holds the batch's x, current as rows finish, and
// xb[kOne] = 1 (an exact product).  The chain then runs the rows in order:
// lane q forms the row's q-th term v * xb[index], and the terms are
// subtracted from b_i one by one in CSR order, read across lanes; a row of
// at most 8, 16, 32 (else 64) entries subtracts that many terms, the
// missing ones +0.0, which leaves every value unchanged, so every rounding
// is the sequential sweep's.  A row's LDS reads are issued while the row before it
// runs (its indices and values two rows ahead); the one x they cannot see,
// the previous row's, is taken from the chain directly.  A row longer than
// 64 entries is a batch of its own, read from global memory in pieces of 64
// (no row of its batch but itself, and it has no self-loop).
constexpr int kCgsWaves = kBlock / 64;
constexpr int kOne = 64;
// 256 entries per batch and 8 waves per SIMD (the most a SIMD holds): on the
// 27-point and 7-point 100^3 plans, 384, 512, 768 and 1024 entries at the
// occupancy their LDS allows (7, 6, 4, 3 waves) all sweep slower
constexpr int kCgsLaunchCap = 256;
constexpr int kCgsLaunchWaves = 8;

template <int Cap>
struct CgsStage {
    double v[Cap + 64];  // 64 spare entries: reads past a batch's end stay inside
    uint8_t tag[Cap + 64];
    double xb[65];
    int64_t rs[64];
    int32_t off[65];
};

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double lane_bcast(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ int64_t lane_bcast64(int64_t v, int l) {
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// acc minus the terms of lanes 0 .. W-1, in lane order; the lanes' values
// are read eight at a time ahead of their eight subtractions
template <int W>
__device__ __forceinline__ double chain_w(double acc, double term) {
#pragma clang fp contract(off)
#pragma unroll
    for (int g = 0; g < W; g += 8) {
        double t[8];
#pragma unroll
        for (int z = 0; z < 8; z++) t[z] = lane_bcast(term, g + z);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int z = 0; z < 8; z++) acc = acc - t[z];
        __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
}

// Cap: LDS entries per batch; MinW: waves per SIMD that the LDS of a wave
// (about 9 bytes per entry) still allows
template <int Cap, int MinW>
__global__ __launch_bounds__(kBlock, MinW) void k_cgs_cluster(const int64_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        const double *__restrict__ val,
                                                        const double *__restrict__ diag,
                                                        const double *__restrict__ b, double *x,
                                                        const int32_t *__restrict__ rows,
                                                        const int32_t *__restrict__ pos,
                                                        const int64_t *__restrict__ cluster_off,
                                                        int64_t k0, int64_t k1, int backward) {
#pragma clang fp contract(off)
    constexpr int kCgsCap = Cap, kCgsU = Cap / 64;
    __shared__ CgsStage<Cap> stage[kCgsWaves];
    const int lane = threadIdx.x & 63;
    CgsStage<Cap> &S = stage[threadIdx.x >> 6];
    const int64_t k = k0 + (int64_t)blockIdx.x * kCgsWaves + (threadIdx.x >> 6);
    if (k >= k1) return;
    const int64_t r0 = cluster_off[k], r1 = cluster_off[k + 1], m = r1 - r0;
    if (lane == 0) S.xb[kOne] = 1.0;
    S.v[kCgsCap + lane] = 0.0;
    S.tag[kCgsCap + lane] = kOne;
    for (int64_t u = 0; u < m;) {
        // the next (up to) 64 rows in visiting order, one per lane
        const int64_t cand = u + lane;
        const bool valid = cand < m;
        const int64_t t = backward ? r1 - 1 - cand : r0 + cand;
        const int32_t i = valid ? rows[t] : 0;
        const int64_t rs = valid ? row_ptr[i] : 0;
        const int64_t len = valid ? row_ptr[i + 1] - rs : 0;
        const double bi = valid ? b[i] : 0.0;
        const double di = valid ? diag[i] : 1.0;
        const double xo = valid ? x[i] : 0.0;
        // prefix of the lengths, each clamped to kCgsCap + 1: only prefixes up
        // to kCgsCap are used, and those are exact
        const int64_t incl =
            (int64_t)wave_incl_scan((uint32_t)(len < kCgsCap + 1 ? len : kCgsCap + 1));
        // rows before the first one longer than 64, within Cap entries
        const uint64_t longm = __ballot(valid && len > 64);
        const int first_long = longm ? __ffsll((unsigned long long)longm) - 1 : 64;
        int nb = __popcll(__ballot(valid && incl <= kCgsCap));
        nb = nb < first_long ? nb : first_long;
        if (nb == 0) {
            // lane 0's row alone, longer than 64 entries
            const int32_t i0 = __builtin_amdgcn_readfirstlane(i);
            const int64_t s0 = lane_bcast64(rs, 0), l0 = lane_bcast64(len, 0);
            double acc = lane_bcast(bi, 0);
            for (int64_t pc = 0; pc < l0; pc += 64) {
                const int64_t q = pc + lane;
                double term = 0.0;
                if (q < l0) {
                    const int64_t pe = s0 + q;
                    term = val[pe] * x[col[pe]];
                }
                acc = chain_w<64>(acc, term);
            }
            const double xn = acc / lane_bcast(di, 0);
            if (lane == 0) x[i0] = xn;
            wave_sync();
            u += 1;
            continue;
        }
        const int tot = (int)lane_bcast64(incl, nb - 1);
        // sweep positions of the batch: [lo, lo + nb)
        const int64_t lo = backward ? r1 - u - nb : r0 + u;
        if (lane < nb) {
            S.off[lane + 1] = (int32_t)incl;
            S.rs[lane] = rs;
            S.xb[lane] = xo;
        }
        if (lane == 0) S.off[0] = 0;
        wave_sync();
        // stage the batch's entries, all of a lane's loads in flight at once
        // (slots past tot re-read entry 0 and store nothing).  A batch with no
        // entries (rows without off-diagonal entries) loads nothing: its rows'
        // CSR starts may equal nnz, one past the last entry
        if (tot > 0) {
            int64_t pp[kCgsU];
#pragma unroll
            for (int c = 0; c < kCgsU; c++) {
                const int q = lane + 64 * c < tot ? lane + 64 * c : 0;
                int kr = 0;
                for (int st = 32; st > 0; st >>= 1)
                    if (kr + st < nb && S.off[kr + st] <= q) kr += st;
                pp[c] = S.rs[kr] + (q - S.off[kr]);
            }
            int32_t jj[kCgsU];
            double aa[kCgsU];
#pragma unroll
            for (int c = 0; c < kCgsU; c++) {
                jj[c] = col[pp[c]];
                aa[c] = val[pp[c]];
            }
#pragma unroll
            for (int c = 0; c < kCgsU; c++) {
                const int q = lane + 64 * c;
                const int64_t pj = pos[jj[c]];
                const double xj = x[jj[c]];
                const bool inb = pj >= lo && pj < lo + nb;
                if (q < tot) {
                    S.tag[q] = inb ? (uint8_t)(backward ? lo + nb - 1 - pj : pj - lo) : kOne;
                    S.v[q] = inb ? aa[c] : aa[c] * xj;
                }
            }
        }
        wave_sync();
        // the chain.  Row r's entries are [incl(r) - len(r), incl(r)); lane q
        // reads entry q of a row (past its end: a spare zero entry, or the
        // next row's, both masked out of the term)
        auto start = [&](int r) { return r == 0 ? 0 : (int)lane_bcast64(incl, r - 1); };
        const int s1 = start(1 < nb ? 1 : nb - 1);
        // (an index read past a row's end may be stale: clamp it into xb)
        double v0 = S.v[lane], v1 = S.v[s1 + lane];
        int g0 = min((int)S.tag[lane], kOne), g1 = min((int)S.tag[s1 + lane], kOne);
        double x0 = S.xb[g0];
        double xs = 0.0;  // x of the previous row
        for (int kk = 0; kk < nb; kk++) {
            const int ln = (int)lane_bcast64(incl, kk) - start(kk);
            // row kk's term; xb[kk - 1] was not yet written when x0 was read
            const double xf = g0 == kk - 1 ? xs : x0;
            const double term = lane < ln ? v0 * xf : 0.0;
            // reads for rows kk + 1 (x) and kk + 2 (values, indices)
            const double x1 = S.xb[g1];
            const int s2 = start(kk + 2 < nb ? kk + 2 : nb - 1);
            const double v2 = S.v[s2 + lane];
            const int g2 = min((int)S.tag[s2 + lane], kOne);
            double acc = lane_bcast(bi, kk);
            acc = ln <= 8    ? chain_w<8>(acc, term)
                  : ln <= 16 ? chain_w<16>(acc, term)
                  : ln <= 32 ? chain_w<32>(acc, term)
                             : chain_w<64>(acc, term);
            const double xn = acc / lane_bcast(di, kk);
            if (lane == 0) S.xb[kk] = xn;
            if (lane == kk) x[i] = xn;
            xs = xn;
            v0 = v1;
            g0 = g1;
            x0 = x1;
            v1 = v2;
            g1 = g2;
        }
        wave_sync();
        u += nb;
    }
}

// Point form (every cluster one row): the rows of one colour share no edge,
// so each reads only x of other colours and their order does not matter.
// One lane per row, R consecutive sweep positions per wavefront (fewer rows
// per wave give a small colour more waves): the wave stages the products
// a_ij * x_j of its rows' entries in LDS, kPtCap at a time, and each lane
// subtracts its own row's products in CSR order.
constexpr int kPtCap = 1024;

struct PointStage {
    double v[kPtCap];
    int64_t off[65];  // entry offsets of the wave's rows (off[64] = total)
    int64_t rs[64];
};

template <int R>
__global__ __launch_bounds__(kBlock) void k_cgs_point(const int64_t *__restrict__ row_ptr,
                                                      const int32_t *__restrict__ col,
                                                      const double *__restrict__ val,
                                                      const double *__restrict__ diag,
                                                      const double *__restrict__ b, double *x,
                                                      const int32_t *__restrict__ rows,
                                                      int64_t t0, int64_t t1) {
#pragma clang fp contract(off)
    __shared__ PointStage stage[kCgsWaves];
    const int lane = threadIdx.x & 63;
    PointStage &S = stage[threadIdx.x >> 6];
    const int64_t base = t0 + ((int64_t)blockIdx.x * kCgsWaves + (threadIdx.x >> 6)) * R;
    if (base >= t1) return;
    const int64_t t = base + lane;
    const bool valid = lane < R && t < t1;
    const int32_t i = valid ? rows[t] : 0;
    const int64_t rs = valid ? row_ptr[i] : 0;
    const int64_t len = valid ? row_ptr[i + 1] - rs : 0;
    double acc = valid ? b[i] : 0.0;
    int64_t incl = len;
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    const int64_t excl = incl - len;
    S.off[lane + 1] = incl;
    S.rs[lane] = rs;
    if (lane == 0) S.off[0] = 0;
    const int64_t tot = lane_bcast64(incl, 63);
    wave_sync();
    for (int64_t E = 0; E < tot; E += kPtCap) {
        const int64_t cnt = tot - E < kPtCap ? tot - E : kPtCap;
        constexpr int U = kPtCap / 64;
        int64_t pp[U];
#pragma unroll
        for (int c = 0; c < U; c++) {
            const int64_t e = E + (lane + 64 * c < cnt ? lane + 64 * c : 0);
            int kr = 0;
            for (int st = 32; st > 0; st >>= 1)
                if (S.off[kr + st] <= e) kr += st;
            pp[c] = S.rs[kr] + (e - S.off[kr]);
        }
        int32_t jj[U];
        double aa[U];
#pragma unroll
        for (int c = 0; c < U; c++) {
            jj[c] = col[pp[c]];
            aa[c] = val[pp[c]];
        }
#pragma unroll
        for (int c = 0; c < U; c++) {
            const double pr = aa[c] * x[jj[c]];
            if (lane + 64 * c < cnt) S.v[lane + 64 * c] = pr;
        }
        wave_sync();
        const int64_t lo = (excl > E ? excl : E) - E;
        const int64_t hi = (incl < E + cnt ? incl : E + cnt) - E;
        int64_t e = lo;
        for (; e + 4 <= hi; e += 4) {
            const double p0 = S.v[e], p1 = S.v[e + 1], p2 = S.v[e + 2], p3 = S.v[e + 3];
            acc = acc - p0;
            acc = acc - p1;
            acc = acc - p2;
            acc = acc - p3;
        }
        for (; e < hi; e++) acc = acc - S.v[e];
        wave_sync();
    }
    if (valid) x[i] = acc / diag[i];
}

int grid_of(int64_t work, int cap) {
    int64_t g = (work + kBlock - 1) / kBlock;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

}  // namespace

hipError_t launch_jp_init(int64_t n, const TupleParams &tp, unsigned long long *st,
                          hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_jp_init, dim3(grid_of(n, 8192)), dim3(kBlock), 0, s, n, tp, st);
    return hipGetLastError();
}

hipError_t launch_jp_pass(int64_t n, const int64_t *row_ptr, const int32_t *col,
                          unsigned long long *st, int32_t *color, int32_t *list, uint32_t *cnt,
                          bool first, uint32_t *left, uint32_t *maxc, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    // wavefronts of at least 64 vertices, a multiple of 8 workgroups (one run
    // of them per XCD), all resident at once
    int64_t blocks = (n + 4 * kBlock - 1) / (4 * kBlock);
    blocks = std::max<int64_t>(8, std::min<int64_t>((blocks + 7) / 8 * 8, 2048));
    const int64_t waves = blocks * (kBlock / 64);
    hipLaunchKernelGGL(k_jp_pass, dim3((unsigned)blocks), dim3(kBlock), 0, s, n, row_ptr, col, st,
                       color, list, cnt, (n + waves - 1) / waves, first ? 1 : 0, left, maxc);
    return hipGetLastError();
}

int64_t color_sort_counts(int64_t n, int32_t n_colors) {
    return n_colors <= kSortColors ? (n + kColorTile - 1) / kColorTile * n_colors : 0;
}

hipError_t launch_color_sort(int64_t n, const int32_t *color, int32_t n_colors, uint32_t *cnt,
                             int64_t *pos, unsigned long long *part, int32_t *out, int64_t *first,
                             hipStream_t s) {
    const int64_t tiles = (n + kColorTile - 1) / kColorTile;
    if (n <= 0 || n_colors > kSortColors || tiles > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_color_count, dim3((unsigned)tiles), dim3(kBlock), 0, s, n, color, n_colors,
                       tiles, cnt);
    const hipError_t e = exclusive_scan_u32_i64(cnt, tiles * n_colors, pos, part, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_color_scatter, dim3((unsigned)tiles), dim3(kBlock), 0, s, n, color,
                       n_colors, tiles, (const int64_t *)pos, out, first);
    return hipGetLastError();
}

hipError_t launch_point_plan(int64_t n, const int32_t *rows, int32_t *pos, int64_t *cluster_off,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_point_plan, dim3(grid_of(n + 1, 8192)), dim3(kBlock), 0, s, n, rows, pos,
                       cluster_off);
    return hipGetLastError();
}

hipError_t launch_iota(int64_t n, int32_t *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_iota, dim3(grid_of(n, 8192)), dim3(kBlock), 0, s, n, out);
    return hipGetLastError();
}

hipError_t launch_count_of(int64_t n, const int32_t *key, uint32_t *cnt, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_count_of, dim3(grid_of(n, 8192)), dim3(kBlock), 0, s, n, key, cnt);
    return hipGetLastError();
}

hipError_t launch_color_hist(int64_t n, const int32_t *color, int32_t n_colors, uint32_t *hist,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (n_colors > kHistBins) return launch_count_of(n, color, hist, s);
    hipLaunchKernelGGL(k_color_hist, dim3(grid_of(n, 1024)), dim3(kBlock), 0, s, n, color,
                       n_colors, hist);
    return hipGetLastError();
}

hipError_t launch_sort_members(int64_t nc, const int64_t *moff, int32_t *members, hipStream_t s) {
    if (nc <= 0) return hipSuccess;
    const int64_t sblocks = (nc + kBlock / 64 - 1) / (kBlock / 64);
    if (sblocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_sort_small, dim3((unsigned)sblocks), dim3(kBlock), 0, s, nc, moff,
                       members);
    hipLaunchKernelGGL(k_sort_large, dim3((unsigned)std::min<int64_t>(nc, 1024)), dim3(kBlock), 0,
                       s, nc, moff, members);
    return hipGetLastError();
}

hipError_t launch_gather_sizes(int64_t nk, const int32_t *order, const uint32_t *cnt,
                               uint32_t *out, hipStream_t s) {
    if (nk <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_sizes, dim3(grid_of(nk, 8192)), dim3(kBlock), 0, s, nk, order,
                       cnt, out);
    return hipGetLastError();
}

hipError_t launch_place_rows(int64_t nk, const int32_t *order, const int64_t *moff,
                             const int32_t *members, const int64_t *cluster_off, int32_t *rows,
                             hipStream_t s) {
    if (nk <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_place_rows, dim3(grid_of(nk, 8192)), dim3(kBlock), 0, s, nk, order, moff,
                       members, cluster_off, rows);
    return hipGetLastError();
}

hipError_t launch_scatter_pos(int64_t n, const int32_t *rows, int32_t *pos, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter_pos, dim3(grid_of(n, 8192)), dim3(kBlock), 0, s, n, rows, pos);
    return hipGetLastError();
}

hipError_t launch_cgs_sweep(const int64_t *row_ptr, const int32_t *col, const double *val,
                            const double *diag, const double *b, double *x, const int32_t *rows,
                            const int32_t *pos, const int64_t *cluster_off, int64_t k0, int64_t k1,
                            bool backward, hipStream_t s) {
    if (k1 <= k0) return hipSuccess;
    const int64_t blocks = (k1 - k0 + kCgsWaves - 1) / kCgsWaves;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_cgs_cluster<kCgsLaunchCap, kCgsLaunchWaves>), dim3((unsigned)blocks),
                       dim3(kBlock), 0, s, row_ptr, col, val, diag, b, x, rows, pos, cluster_off,
                       k0, k1, backward ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_cgs_point(const int64_t *row_ptr, const int32_t *col, const double *val,
                            const double *diag, const double *b, double *x, const int32_t *rows,
                            int64_t t0, int64_t t1, hipStream_t s) {
    if (t1 <= t0) return hipSuccess;
    // rows per wave: the most that still leaves 4 waves per SIMD (1024 SIMDs)
    const int64_t nr = t1 - t0;
    const int R = nr >= 64 * 4096 ? 64 : nr >= 32 * 4096 ? 32 : 16;
    const int64_t per = (int64_t)R * kCgsWaves;
    const int64_t blocks = (nr + per - 1) / per;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    if (R == 64)
        hipLaunchKernelGGL(k_cgs_point<64>, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr,
                           col, val, diag, b, x, rows, t0, t1);
    else if (R == 32)
        hipLaunchKernelGGL(k_cgs_point<32>, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr,
                           col, val, diag, b, x, rows, t0, t1);
    else
        hipLaunchKernelGGL(k_cgs_point<16>, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr,
                           col, val, diag, b, x, rows, t0, t1);
    return hipGetLastError();
}

}  // namespace mis2
