// cgs.hip -- cluster multicolor Gauss-Seidel (Algorithm 4, Section III-C) on gfx950.
//
// Setup colours a graph (the coarse graph of an aggregation, or the graph
// itself for point multicolor Gauss-Seidel) and orders the rows by colour,
// then by cluster, then by row id.  Apply runs, for each colour in turn, every
// cluster's rows one after the other, the clusters side by side.  Clusters of
// one colour share no edge, so none reads a value another one of the same launch
// writes, and the result is that of the sequential sweep in the same order.
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
#include "rowset.h"

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
// C clusters per workgroup, SL = 16, 64 or 256 lanes each to stage them and one
// wavefront to run them.  A cluster's rows are taken in batches of at most
// R = min(SL, 64) rows; staging lane k holds the batch's k-th row.  The batch is
// staged in LDS in parallel, every row in L slots (L: the longest row of the
// workgroup's batches; Cap slots in all): for each entry, in CSR order, either
// the product a_ij * x_j with index R (x_j is final for this pass when j is not a
// row of the batch: another colour's x, a row of this cluster updated in an
// earlier batch, or one not yet reached, whose old value Gauss-Seidel uses), or
// a_ij with the batch index of j; +0.0 with index R past the row's end.  xb holds
// the batch's x, current as rows finish, and xb[R] = 1 (an exact product).  One
// wavefront then runs the batches' chains side by side, a DPP row of 16 lanes for
// each: lane q forms a row's q-th term v * xb[index] (of 16 at a time), and the
// terms are subtracted from b_i one by one in CSR order, each read by all 16
// lanes of the row; the missing ones, +0.0, leave every value unchanged, so every
// rounding is the sequential sweep's.  A row's LDS reads are issued while the row
// before it runs (its indices and values two rows ahead); the one x they cannot
// see, the previous row's, is taken from the chain directly.  A row longer than
// Cap entries is a batch of its own, read from global memory by its cluster's
// lanes (no row of its batch but itself, and it has no self-loop).
//
// Bound by latency: a colour's launch lasts as long as its largest cluster, and
// that is five dependent loads a batch, then about 7.5 cycles a term and 104 a
// division.  One wavefront per cluster for both parts, a batch of 256 entries and
// the term read across the wavefront by two moves took 57 us a colour on the
// 27-point 100^3 grid (13 colours of 3400 clusters, 23 rows of 26 entries; this:
// 37, of which 11 are the chains).  Symmetric sweeps, before and now: 27-point
// 100^3 1467 and 866 us, 40^3 946 and 442; 7-point 100^3 535 and 319; 2-D 5-point
// 700 x 800 295 and 155; elasticity (80 entries a row, before past the staged
// length) 40^3 6482 and 2193.
constexpr int kCgsWaves = kBlock / 64;

// R: rows of a batch
template <int R, int Cap>
struct CgsStage {
    double v[Cap + 16];  // 16 spare slots: reads past a batch's end stay inside
    double xb[R + 1];
    union {
        struct {  // of the rows, for the staging
            int64_t rs[R];
            int32_t len[R];
        };
        struct {  // for the chains
            double b[R], d[R];
        };
    };
    int32_t nb, longest, more;
    uint8_t tag[Cap + 16];
};

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

// The largest value among the group's lanes up to this one (x >= 0).
template <int G>
__device__ __forceinline__ int group_incl_max(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true));
    if constexpr (G == 64) {
        x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false));
        x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false));
    }
    return x;
}

// The chains of the four staged batches (the whole wavefront): NB rows, each of K
// times 16 terms, the last W of them in the last step (16 (K - 1) < L <= 16 (K - 1) + W, or K = 1).
template <int C, int K, int W, int R, int Cap>
__device__ __forceinline__ void run_chains(CgsStage<R, Cap> *stage, int NB, int L) {
#pragma clang fp contract(off)
    const int lane = (int)(threadIdx.x & 63u), q = lane & 15;
    CgsStage<R, Cap> &S = stage[(lane >> 4) & (C - 1)];
    const int nbg = S.nb;
    const bool in = 16 * (K - 1) + q < L;  // the last step's lanes inside a row
    double v[K], w[K], x[K];
    int t[K], u[K];
    auto read = [&](int r, double (&rv)[K], int (&rt)[K]) {
        const int e = min(r, NB - 1) * L + q;
#pragma unroll
        for (int c = 0; c < K; c++) {
            rv[c] = S.v[e + 16 * c];
            rt[c] = (int)S.tag[e + 16 * c];
        }
        rv[K - 1] = in ? rv[K - 1] : 0.0;
        rt[K - 1] = in ? rt[K - 1] : R;
    };
    read(0, v, t);
    read(1, w, u);
#pragma unroll
    for (int c = 0; c < K; c++) x[c] = S.xb[t[c]];
    double bk = S.b[0], dk = S.d[0];
    double xs = 0.0;  // x of the previous row
    for (int kk = 0; kk < NB; kk++) {
        double term[K];
#pragma unroll
        for (int c = 0; c < K; c++)  // xb[kk - 1] was not yet written when x was read
            term[c] = v[c] * (t[c] == kk - 1 ? xs : x[c]);
        double acc = bk;
        // reads for rows kk + 1 (x, b, d) and kk + 2 (values, indices)
        const double dn = S.d[min(kk + 1, NB - 1)];
        bk = S.b[min(kk + 1, NB - 1)];
#pragma unroll
        for (int c = 0; c < K; c++) {
            x[c] = S.xb[u[c]];
            v[c] = w[c];
            t[c] = u[c];
        }
        read(kk + 2, w, u);
#pragma unroll
        for (int c = 0; c + 1 < K; c++) acc = chain_sub<16>(acc, term[c]);
        acc = chain_sub<W>(acc, term[K - 1]);
        xs = acc / dk;
        if (q == 0 && lane < 16 * C && kk < nbg) S.xb[kk] = xs;
        dk = dn;
    }
}

// The same for longer rows, 16 terms at a time.
template <int C, int R, int Cap>
__device__ __forceinline__ void run_long_chains(CgsStage<R, Cap> *stage, int NB, int L) {
#pragma clang fp contract(off)
    const int lane = (int)(threadIdx.x & 63u), q = lane & 15;
    CgsStage<R, Cap> &S = stage[(lane >> 4) & (C - 1)];
    const int nbg = S.nb;
    for (int kk = 0; kk < NB; kk++) {
        double acc = S.b[kk];
        const double dk = S.d[kk];
        for (int c = 0; c < L; c += 16) {
            const int e = kk * L + c + q;
            const bool in = c + q < L;
            const double p = S.v[e] * S.xb[in ? (int)S.tag[e] : R];
            acc = chain_sub<16>(acc, in ? p : 0.0);
        }
        const double xs = acc / dk;
        if (q == 0 && lane < 16 * C && kk < nbg) S.xb[kk] = xs;
    }
}

// The T = NB L slots of a batch's rows 0 .. NB - 1 (those past the group's own
// batch are empty), U of a lane's at once: all of their loads go out together.
template <int SL, int U, int R, int Cap>
__device__ __forceinline__ void stage_entries(CgsStage<R, Cap> &S, int lane, int T, int L,
                                              int64_t lo, int nb, int backward,
                                              const int32_t *__restrict__ col,
                                              const double *__restrict__ val, const double *x,
                                              const int32_t *__restrict__ pos) {
#pragma clang fp contract(off)
    const float per = 1.0f / (float)L;
    for (int q0 = lane; q0 - lane < T; q0 += SL * U) {
        int64_t pp[U];
        bool ok[U];
#pragma unroll
        for (int j = 0; j < U; j++) {
            const int q = min(q0 + SL * j, T - 1);
            // q / L: the product is off by less than 2^-21 of itself, and an
            // integer is at least 0.5 / (q + 0.5) of it away
            const int r = (int)(((float)q + 0.5f) * per), e = q - r * L;
            ok[j] = e < S.len[r];
            pp[j] = ok[j] ? S.rs[r] + e : 0;
        }
        int32_t jj[U];
        double aa[U];
#pragma unroll
        for (int j = 0; j < U; j++) {
            jj[j] = col[pp[j]];
            aa[j] = val[pp[j]];
        }
        int32_t pj[U];
        double xj[U];
#pragma unroll
        for (int j = 0; j < U; j++) {
            pj[j] = pos[jj[j]];
            xj[j] = x[jj[j]];
        }
#pragma unroll
        for (int j = 0; j < U; j++) {
            const int q = q0 + SL * j, at = (int)(pj[j] - lo);
            const bool inb = pj[j] >= lo && pj[j] < lo + nb;
            const int to = q < T ? q : Cap + 15;  // a spare slot
            const double p = aa[j] * (inb ? 1.0 : xj[j]);
            S.tag[to] = (uint8_t)(!inb || !ok[j] ? R : backward ? nb - 1 - at : at);
            S.v[to] = ok[j] ? p : 0.0;
        }
    }
}

template <int C, int SL, int Cap, int U, int MinW>
__global__ __launch_bounds__(C *SL, MinW) void k_cgs_cluster(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const double *__restrict__ val, const double *__restrict__ diag, const double *__restrict__ b,
    double *x, const int32_t *__restrict__ rows, const int32_t *__restrict__ pos,
    const int64_t *__restrict__ cluster_off, int64_t k0, int64_t k1, int backward) {
#pragma clang fp contract(off)
    static_assert(SL == 16 || SL == 64 || SL == 256, "a DPP row or wavefronts stage a cluster");
    constexpr int R = SL < 64 ? SL : 64;
    __shared__ CgsStage<R, Cap> stage[C];
    // the wavefronts of a group each work out its rows, and store the same
    const int lane = (int)threadIdx.x % R, grp = (int)threadIdx.x / SL;
    CgsStage<R, Cap> &S = stage[grp];
    // each XCD takes one run of the clusters (the grid is a multiple of 8)
    const int64_t blk = (int64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int64_t k = k0 + blk * C + grp;
    const int64_t r0 = k < k1 ? cluster_off[k] : 0;
    const int64_t r1 = k < k1 ? cluster_off[k + 1] : 0, m = r1 - r0;
    if (lane == 0) S.xb[R] = 1.0;
    // the rows from position u on in visiting order, one per lane (no branch
    // around a load, here and below: row 0 stands in)
    int32_t i = 0;
    int64_t rs = 0, re = 0;
    double bi = 0.0, di = 1.0, xo = 0.0;
    auto fetch = [&](int64_t u) {
        const int64_t cand = u + lane;
        i = rows[cand >= m ? 0 : backward ? r1 - 1 - cand : r0 + cand];
        rs = row_ptr[i];
        re = row_ptr[i + 1];
        bi = b[i];
        di = diag[i];
        xo = x[i];
    };
    fetch(0);
    for (int64_t u = 0;;) {
        const bool valid = u + lane < m;
        // the longest row so far, clamped past Cap; the rows that fit Cap slots
        const int len = valid ? (int)min<int64_t>(re - rs, Cap + 1) : 0;
        const int upto = group_incl_max<R>(len);
        uint64_t fit = __ballot(valid && upto * (lane + 1) <= Cap);
        if (SL == 16) fit = fit >> (grp * 16) & 0xFFFFull;
        const int mine = __popcll(fit);
        if (lane == 0) S.nb = 0;
        if (lane == 0) S.longest = 0;
        wave_sync();
        if (lane == mine - 1) {
            S.nb = mine;
            S.longest = upto;
        }
        __syncthreads();
        int L = 0;
#pragma unroll
        for (int g = 0; g < C; g++) L = max(L, stage[g].longest);
        const int room = L > 0 ? Cap / L : R;
        int NB = 0;
#pragma unroll
        for (int g = 0; g < C; g++) NB = max(NB, min(stage[g].nb, room));
        L = __builtin_amdgcn_readfirstlane(L);
        NB = __builtin_amdgcn_readfirstlane(NB);
        const int nb = min(mine, room);
        const int64_t next = u + max(nb, 1);
        __syncthreads();
        if (lane == 0) {
            S.nb = nb;
            S.more = next < m;
        }
        S.rs[lane] = rs;
        S.len[lane] = lane < nb ? len : 0;
        S.xb[lane] = xo;
        wave_sync();
        // sweep positions of the batch: [lo, lo + nb)
        const int64_t lo = backward ? r1 - u - nb : r0 + u;
        // (rows without off-diagonal entries stage nothing: there may be no entry
        // in all of the matrix)
        const int sl = (int)threadIdx.x % SL;
        if (NB * L <= SL * (U / 2) && L > 0)
            stage_entries<SL, U / 2>(S, sl, NB * L, L, lo, nb, backward, col, val, x, pos);
        else if (L > 0)
            stage_entries<SL, U>(S, sl, NB * L, L, lo, nb, backward, col, val, x, pos);
        if (mine == 0 && u < m && sl < 64) {
            // lane 0's row alone, longer than Cap entries
            const int first = SL == 16 ? (int)(threadIdx.x & 48u) : 0;
            const int32_t i0 = __shfl(i, first, 64);
            const int64_t s0 = __shfl(rs, first, 64), l0 = __shfl(re, first, 64) - s0;
            double acc = __shfl(bi, first, 64);
            const double d0 = __shfl(di, first, 64);
            for (int64_t pc = 0; pc < l0; pc += R * 4) {
                double term[4];
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    const int64_t q = pc + R * c + lane, pe = s0 + (q < l0 ? q : 0);
                    const double p = val[pe] * x[col[pe]];
                    term[c] = q < l0 ? p : 0.0;
                }
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    acc = chain_sub<16>(acc, term[c]);
                    if (R == 64) {  // on through the other rows' 16 lanes
                        acc = chain_sub<16>(lane_bcast(acc, 0), term[c]);
                        acc = chain_sub<16>(lane_bcast(acc, 16), term[c]);
                        acc = chain_sub<16>(lane_bcast(acc, 32), term[c]);
                        acc = lane_bcast(acc, 48);
                    }
                }
            }
            const double xn = acc / d0;
            if (lane == 0) x[i0] = xn;
        }
        if (SL > 64) __syncthreads();
        wave_sync();
        S.b[lane] = bi;
        S.d[lane] = lane < nb ? di : 1.0;
        const int32_t done = i;
        __syncthreads();
        int more = 0;
#pragma unroll
        for (int g = 0; g < C; g++) more |= stage[g].more;
        // the next batch's rows while the chains run (no x of theirs changes)
        if (more) fetch(next);
        if (threadIdx.x < 64u && NB > 0) {
            if (L <= 8) run_chains<C, 1, 8>(stage, NB, L);
            else if (L <= 16) run_chains<C, 1, 16>(stage, NB, L);
            else if (L <= 28) run_chains<C, 2, 12>(stage, NB, L);
            else if (L <= 32) run_chains<C, 2, 16>(stage, NB, L);
            else if (L <= 48) run_chains<C, 3, 16>(stage, NB, L);
            else if (L <= 64) run_chains<C, 4, 16>(stage, NB, L);
            else if (L <= 80) run_chains<C, 5, 16>(stage, NB, L);
            else run_long_chains<C>(stage, NB, L);
        }
        __syncthreads();
        if (lane < nb && sl < 64) x[done] = S.xb[lane];
        if (!more) break;
        if (SL > 64) __syncthreads();  // before the other wavefronts read it
        u = next;
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
                            int64_t per, bool backward, hipStream_t s) {
    if (k1 <= k0) return hipSuccess;
    const int64_t blocks = ((k1 - k0 + 3) / 4 + 7) / 8 * 8;  // 4 clusters each
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    auto go = [&](auto kernel, int lanes) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(4 * lanes), 0, s, row_ptr, col, val,
                           diag, b, x, rows, pos, cluster_off, k0, k1, backward ? 1 : 0);
        return hipGetLastError();
    };
    // Lanes to stage a cluster by its entries (per, on average): a 7-point
    // cluster has 40, so 16 lanes load it in three or four steps and one wavefront
    // takes four clusters.  A 27-point one has 560: a wavefront each, and slots
    // for 35 of its rows, the most that keep four workgroups on a compute unit
    // (768 slots: 40 us a colour, 1152: 40, with two clusters a workgroup 37, one
    // 40).  Where the workgroups are no more than the compute units, or a cluster
    // has thousands of entries, four wavefronts load each: 27-point 40^3 442 us
    // against 497 with one wavefront, elasticity 60^3 2856 against 3233; up to 2048
    // clusters instead of 1024 the 27-point 60^3 grid slows from 497 to 558.
    if (per <= 128) return go(k_cgs_cluster<4, 16, 128, 8, 4>, 16);
    if (per <= 1024 && k1 - k0 > 1024) return go(k_cgs_cluster<4, 64, 928, 8, 4>, 64);
    return go(k_cgs_cluster<4, 256, 2048, 8, 4>, 256);
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
