// aggregate.hip -- the labelling phases of Algorithm 3 (Section III-B) for gfx950.
//
// Phase 1 / phase 2 labelling push a root's aggregate id to its neighbours:
// the roots of an MIS-2 are at least three edges apart, so the written sets
// are disjoint and the order of the writes cannot matter.  The same pass
// knows each aggregate's size (the root plus the neighbours it labelled), so
// aggsize needs no histogram.  Phase 3 reads only the labels frozen after
// phase 2 (the "tentative" labels) and writes a separate output array, so
// every row is decided independently.
#include "internal.h"
#include "lanes.h"
#include "phase3.h"

namespace mis2 {

namespace {

constexpr int kLabelLanes = 16;  // lanes per root in the labelling push

__device__ __forceinline__ uint64_t lanes_below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

__device__ __forceinline__ int64_t wave_id() {
    const int64_t B = gridDim.x;
    const int64_t b = blockIdx.x;
    const int64_t lb = (B % 8 == 0) ? (b % 8) * (B / 8) + b / 8 : b;
    return lb * (kBlock / 64) + (threadIdx.x >> 6);
}

constexpr int kCoopLoads = 8;      // loads per lane per cooperative step
constexpr int64_t kHeavyRoot = 256;  // roots longer than this are pushed by the whole wavefront

// Labels the neighbours in [s, e) of a root with id (all of them, or only
// those still at -1), by the whole wavefront; returns the number labelled.
__device__ __forceinline__ int coop_label(const int32_t *__restrict__ col,
                                          int32_t *__restrict__ label, int64_t s, int64_t e,
                                          int32_t id, int only_unlabelled) {
    const int lane = (int)(threadIdx.x & 63u);
    int took = 0;
    for (int64_t b = s; b < e; b += 64 * kCoopLoads) {
        int32_t x[kCoopLoads];
#pragma unroll
        for (int k = 0; k < kCoopLoads; k++) {
            const int64_t j = b + (int64_t)k * 64 + lane;
            x[k] = col[j < e ? j : s];
        }
        int32_t old[kCoopLoads];
#pragma unroll
        for (int k = 0; k < kCoopLoads; k++) old[k] = only_unlabelled ? label[x[k]] : -1;
#pragma unroll
        for (int k = 0; k < kCoopLoads; k++) {
            if (b + (int64_t)k * 64 + lane < e && old[k] == -1) {
                label[x[k]] = id;
                took++;
            }
        }
    }
    return group_sum_i<64>(took);
}

// roots[0..*d_count) get ids base + k; their neighbours (all of them, or only
// those still at -1 when only_unlabelled) get the same id, and aggsize[id]
// becomes 1 + the number of neighbours labelled.  Groups of kLabelLanes
// lanes push ordinary roots; long rows are pushed by the whole wavefront.
__global__ __launch_bounds__(kBlock) void k_label_roots(const int64_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        const int32_t *__restrict__ roots,
                                                        const uint32_t *__restrict__ d_count,
                                                        const uint32_t *__restrict__ d_base,
                                                        int only_unlabelled,
                                                        int32_t *__restrict__ label,
                                                        int32_t *__restrict__ aggsize,
                                                        uint8_t *__restrict__ root_mark,
                                                        uint8_t mark) {
    constexpr int L = kLabelLanes, G = kBlock / L;
    const int64_t count = *d_count;
    const int32_t base = d_base ? (int32_t)*d_base : 0;
    const int lane = (int)(threadIdx.x & 63u);
    const int sub = (int)(threadIdx.x & (L - 1));
    // the loop bound is the same for the whole wavefront, so the shuffles
    // below always run with all lanes active
    const int64_t step = (int64_t)gridDim.x * G;
    const int64_t k0 = (int64_t)blockIdx.x * G + (threadIdx.x & ~63u) / L;
    for (int64_t kw = k0; kw < count; kw += step) {
        const int64_t k = kw + lane / L;
        const bool ok = k < count;
        const int32_t r = roots[ok ? k : count - 1];
        const int32_t id = base + (int32_t)k;
        int64_t s = row_ptr[r], e = row_ptr[r + 1];
        if (!ok) e = s;
        int took = 0;
        int heavy_took = 0;
        uint64_t heavy = __ballot(sub == 0 && e - s > kHeavyRoot);
        while (heavy) {
            const int src = __ffsll((unsigned long long)heavy) - 1;
            heavy &= heavy - 1;
            const int64_t hs = __shfl(s, src, 64), he = __shfl(e, src, 64);
            const int32_t hid = __shfl(id, src, 64);
            const int t = coop_label(col, label, hs, he, hid, only_unlabelled);
            if ((lane & ~(L - 1)) == (src & ~(L - 1))) {
                heavy_took = t;
                e = s;  // its group skips the row below
            }
        }
        for (int64_t j = s + sub; j < e; j += L) {
            const int32_t w = col[j];
            if (!only_unlabelled || label[w] == -1) {
                label[w] = id;
                took++;
            }
        }
        took = group_sum_i<L>(took);
        if (ok && sub == 0) {
            label[r] = id;
            aggsize[id] = 1 + took + heavy_took;
            if (root_mark) root_mark[r] = mark;
        }
    }
}

// flag[v] = 1 iff v is a root of the phase-2 MIS-2 (T_v = IN in the masked
// run) with at least two neighbours that are unlabelled after phase 1.  Each
// wavefront scans 64 vertices at a time; a candidate's row of up to
// kAcceptLane entries is counted by its own lane, longer ones by the whole
// wavefront, one row at a time.
constexpr int64_t kAcceptLane = 32;  // rows a lane counts alone in k_accept_phase2

// Buffer resource over n labels: a load whose byte offset is at or past
// 4n returns 0 without a memory access (the range check of raw buffer
// loads), which predicates a load per lane without a branch.  Word 3 is the
// gfx9 data-format word (32-bit elements).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t label_rsrc(const int32_t *label, int64_t n) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)label, (short)0, (int)(uint32_t)(4 * n),
                                             0x00020000);
}

// BUF: 4n < 2^32, so every label is reachable by a 32-bit buffer offset.
template <bool BUF>
__global__ __launch_bounds__(kBlock) void k_accept_phase2(int64_t n,
                                                          const int64_t *__restrict__ row_ptr,
                                                          const int32_t *__restrict__ col,
                                                          const uint32_t *__restrict__ T,
                                                          const int32_t *__restrict__ label,
                                                          uint8_t *__restrict__ flag) {
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t base = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * 64; base < n;
         base += waves * 64) {
        const int64_t v = base + lane;
        const bool cand = v < n && label[v] == -1 && T[v] == kIn;
        // a candidate with a row of up to kAcceptLane entries counts its own
        // row; longer rows go to the whole wavefront one at a time
        int64_t rs = 0, re = 0;
        if (cand) {
            rs = row_ptr[v];
            re = row_ptr[v + 1];
        }
        const bool own = cand && re - rs <= kAcceptLane;
        uint8_t f = 0;
        if (own) {
            // every entry of the row loads at once, then every label: two
            // dependent steps for the whole row; each load is issued only for
            // the entries the lane's row has
            const int len = (int)(re - rs);
            int32_t x[kAcceptLane];
#pragma unroll
            for (int k = 0; k < (int)kAcceptLane; k++) {
                x[k] = 0;
                if (k < len) x[k] = col[rs + k];
            }
            if constexpr (BUF) {
                const __amdgpu_buffer_rsrc_t rl = label_rsrc(label, n);
#pragma unroll
                for (int k = 0; k < (int)kAcceptLane; k++)
                    x[k] = __builtin_amdgcn_raw_buffer_load_b32(
                        rl, k < len ? (int)(4u * (uint32_t)x[k]) : (int)0xFFFFFFFCu, 0, 0);
            } else {
                // entries past the row all read label 0: one line for the wavefront
#pragma unroll
                for (int k = 0; k < (int)kAcceptLane; k++) x[k] = label[k < len ? x[k] : 0];
            }
            int cnt = 0;
#pragma unroll
            for (int k = 0; k < (int)kAcceptLane; k++) cnt += (k < len) & (x[k] == -1);
            f = cnt >= 2;
        }
        uint64_t mask = __ballot(cand && !own);
        while (mask) {
            const int t = __ffsll((unsigned long long)mask) - 1;
            mask &= mask - 1;
            const int64_t u = base + t;
            const int64_t s = row_ptr[u], e = row_ptr[u + 1];
            int cnt = 0;
            for (int64_t b = s; b < e; b += 64 * kCoopLoads) {
                int32_t x[kCoopLoads];
#pragma unroll
                for (int k = 0; k < kCoopLoads; k++) {
                    const int64_t j = b + (int64_t)k * 64 + lane;
                    x[k] = col[j < e ? j : s];
                }
                int32_t lb[kCoopLoads];
#pragma unroll
                for (int k = 0; k < kCoopLoads; k++) lb[k] = label[x[k]];
#pragma unroll
                for (int k = 0; k < kCoopLoads; k++)
                    cnt += (b + (int64_t)k * 64 + lane < e) & (lb[k] == -1);
            }
            cnt = group_sum_i<64>(cnt);
            if (lane == t) f = cnt >= 2;
        }
        if (v < n) flag[v] = f;
    }
}

// Each wavefront lists, in order, the vertices of its own range still
// unlabelled after phase 2, as its segment of io.wl_out, and copies the
// labels of its range to copy_to (the segments cover every vertex).
__global__ __launch_bounds__(kBlock) void k_list_unlabelled(int64_t n,
                                                            const int32_t *__restrict__ label,
                                                            int32_t *__restrict__ copy_to,
                                                            SegIO io) {
    const int64_t w = wave_id();
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t lo = w * io.seg, hi = min(n, lo + io.seg);
    uint32_t kept = 0;
    for (int64_t v0 = lo; v0 < hi; v0 += 64) {
        const int64_t v = v0 + lane;
        const int32_t lv = v < hi ? label[v] : 0;
        if (v < hi) copy_to[v] = lv;
        const bool keep = v < hi && lv == -1;
        const uint64_t mask = __ballot(keep);
        if (keep) io.wl_out[lo + kept + (uint32_t)__popcll(mask & lanes_below(lane))] = (int32_t)v;
        kept += (uint32_t)__popcll(mask);
    }
    if (lane == 0 && w < io.S) io.cnt_out[w] = kept;
}

__device__ __forceinline__ uint64_t lanes_below_p3(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// One group of L lanes per unaggregated row of the wavefront's segment.  Rows
// of at most K chunks of L entries are counted in registers; longer rows are
// listed, in order, in the wavefront's segment of io.wl_out for
// k_phase3_mid.  The group's best candidate is reduced with the candidate
// order above.
template <int L>
__global__ __launch_bounds__(kBlock) void k_phase3(const int64_t *__restrict__ row_ptr,
                                                   const int32_t *__restrict__ col,
                                                   const int32_t *__restrict__ label,
                                                   const int32_t *__restrict__ aggsize,
                                                   SegIO io, int32_t *__restrict__ agg_out,
                                                   uint32_t *__restrict__ err) {
    constexpr int K = L >= 32 ? 1 : (32 / L > 8 ? 8 : 32 / L);
    const int64_t w = wave_id();
    if (w >= io.S) return;
    const int64_t count = io.cnt_in[w];
    const int64_t sbase = w * io.seg;
    constexpr int G = 64 / L;
    const int lane = (int)(threadIdx.x & 63u);
    const int sub = lane & (L - 1);
    uint32_t kept = 0;
    for (int64_t i0 = 0; i0 < count; i0 += G) {
        const int64_t i = i0 + lane / L;
        const bool valid = i < count;
        int32_t v = 0;
        int64_t s = 0, e = 0;
        if (valid) {
            v = io.wl_in[sbase + i];
            s = row_ptr[v];
            e = row_ptr[v + 1];
        }
        const bool is_long = e - s > (int64_t)K * L;
        const int64_t es = is_long ? s : e;  // long rows are left to k_phase3_mid
        const int64_t wmax = group_max64<64>((es - s + L - 1) / L);
        int bc = 0, bs = 0x7FFFFFFF, ba = 0x7FFFFFFF;
        if (wmax > 0) {
            int32_t a[K], sz[K];
#pragma unroll
            for (int k = 0; k < K; k++) {
                const int64_t j = s + k * L + sub;
                a[k] = col[j < es ? j : 0];
            }
#pragma unroll
            for (int k = 0; k < K; k++) a[k] = label[a[k]];
#pragma unroll
            for (int k = 0; k < K; k++) {
                if (s + k * L + sub >= es) a[k] = kPad;
                sz[k] = aggsize[a[k] >= 0 ? a[k] : 0];
            }
            p3_count<L, K>(a, sz, bc, bs, ba);
        }
        p3_group_best<L>(bc, bs, ba);
        if (valid && sub == 0 && !is_long) {
            if (bc > 0)
                agg_out[v] = ba;
            else
                *err = 1u;
        }
        const bool keep = valid && sub == 0 && is_long;
        const uint64_t mask = __ballot(keep);
        if (keep) io.wl_out[sbase + kept + (uint32_t)__popcll(mask & lanes_below_p3(lane))] = v;
        kept += (uint32_t)__popcll(mask);
    }
    if (lane == 0) io.cnt_out[w] = kept;
}

// The rows k_phase3 listed: those of up to kP3Wave entries here, longer ones
// listed again, in order, for k_phase3_long.  `share` wavefronts take one
// segment's rows between them, so the device is full where segments are few.
// It is bound by each row's chain of loads (columns, labels, sizes); without
// LDS eight wavefronts per SIMD hide it.  Elasticity 60^3 (rows of 80): an LDS
// hash map per wavefront, 16 KiB and so two per SIMD, took 285 us.  Chung-Lu with
// 33 587, 221 710, 1 065 829 and 4M vertices: that map 9.5, 17, 33 and 85 us for
// all rows of more than 32 entries, this and k_phase3_long 13.9, 16, 31 and 74
// (rows of up to 512 here, one aggregate at a time: 28, 30 and 47 for the first
// three).
__global__ __launch_bounds__(kBlock) void k_phase3_mid(const int64_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col,
                                                       const int32_t *__restrict__ label,
                                                       const int32_t *__restrict__ aggsize,
                                                       SegIO io, int share,
                                                       int32_t *__restrict__ agg_out,
                                                       uint32_t *__restrict__ err) {
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t id = wave_id();
    const int64_t w = id / share;
    const int part = (int)(id % share);
    if (w >= io.S) return;
    const int64_t count = io.cnt_in[w], sbase = w * io.seg;
    uint32_t kept = 0;
    for (int64_t i0 = 0; i0 < count; i0 += 64) {
        const bool valid = i0 + lane < count;
        const int32_t v = valid ? io.wl_in[sbase + i0 + lane] : 0;
        const int64_t s = row_ptr[v], d = row_ptr[v + 1] - s;
        const bool longer = valid && d > kP3Wave;
        const int len = (int)min(d, kP3Wave);
        const uint64_t again = __ballot(longer);
        if (part == 0) {
            if (longer) io.wl_out[sbase + kept + (uint32_t)__popcll(again & lanes_below(lane))] = v;
            kept += (uint32_t)__popcll(again);
        }
        uint64_t todo = __ballot(valid && !longer && lane % share == part);
        while (todo) {
            const int l = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const int32_t vr = __builtin_amdgcn_readlane(v, l);
            const int lr = __builtin_amdgcn_readlane(len, l);
            const int64_t sr =
                (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(s >> 32), l) << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)s, l));
            int bc = 0, bs = 0x7FFFFFFF, ba = 0x7FFFFFFF;
            p3_mid<kP3Wave>(
                lr, [&](int j) { return col[sr + j]; }, [&](int32_t u) { return label[u]; },
                [&](int32_t y) { return aggsize[y]; }, bc, bs, ba);
            if (lane == 0) {
                if (bc > 0)
                    agg_out[vr] = ba;
                else
                    *err = 1u;
            }
        }
    }
    if (part == 0 && lane == 0) io.cnt_out[w] = kept;
}

// Rows of more than kP3Wave entries, one workgroup each: the couplings are
// counted in an LDS hash map (aggregate id -> count) of twice as many slots as
// entries, kP3Slots at most, of the
// ids in one of `parts` classes of a hash at a time, parts chosen so that a
// class is expected to fill half the map; a class that does not fit restarts
// the row with twice the classes.  The workgroup then reduces the entries with
// the candidate order.  (One wavefront that compared every label with
// the whole row took 3.7 ms for one launch on a coarse level of Chung-Lu 1M,
// rows of some 6000 entries.)  The grid is resident at once (64 KiB per
// workgroup): workgroup w takes the segments w, w + W, ..., reading kBlock
// sizes in one load.
constexpr int kP3Slots = 8192;
constexpr int kP3LongBlocks = 512;  // 2 resident workgroups on each of 256 compute units

__global__ __launch_bounds__(kBlock) void k_phase3_long(const int64_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        const int32_t *__restrict__ label,
                                                        const int32_t *__restrict__ aggsize,
                                                        SegIO io, int32_t *__restrict__ agg_out,
                                                        uint32_t *__restrict__ err) {
    constexpr uint32_t kEmpty = 0xFFFFFFFFu;
    constexpr int kBits = __builtin_ctz(kP3Slots), kLeast = 9, kWv = kBlock / 64;
    constexpr uint32_t kMost = kP3Slots * 3 / 4;  // ids in the map; each thread may add one more
    static_assert(kMost + kBlock < kP3Slots, "a probe always ends at an empty slot");
    __shared__ uint32_t keys[kP3Slots], cnts[kP3Slots];
    __shared__ uint32_t num;
    __shared__ uint64_t marks[kWv];
    __shared__ uint32_t counts[kBlock];
    __shared__ int best[kWv][3];
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    volatile uint32_t *vnum = &num;
    auto row = [&](const int32_t v) {
        const int64_t s = row_ptr[v], e = row_ptr[v + 1];
        int bc = 0, bs = 0x7FFFFFFF, ba = 0x7FFFFFFF;
        // (the map of a row of up to kP3Slots / 2 entries is never more than half
        // full, so only rows in classes restart)
        int bits = kLeast;
        while (bits < kBits && (int64_t)1 << bits < 2 * (e - s)) bits++;
        const int slots = 1 << bits;
        // (a class value is shared by some 128 ids, so doubling comes to an end)
        uint32_t parts = (uint32_t)((e - s + kP3Slots / 2 - 1) / (kP3Slots / 2));
        for (uint32_t p = 0; p < parts;) {
            for (int k = tid; k < slots; k += kBlock) {
                keys[k] = kEmpty;
                cnts[k] = 0u;
            }
            if (tid == 0) num = 0u;
            __syncthreads();
            for (int64_t j0 = s; j0 < e; j0 += kBlock * kCoopLoads) {
                int32_t a[kCoopLoads];
#pragma unroll
                for (int k = 0; k < kCoopLoads; k++) a[k] = col[min(j0 + k * kBlock + tid, e - 1)];
#pragma unroll
                for (int k = 0; k < kCoopLoads; k++) a[k] = label[a[k]];
#pragma unroll
                for (int k = 0; k < kCoopLoads; k++) {
                    if (j0 + k * kBlock + tid >= e || a[k] < 0) continue;
                    const uint32_t key = (uint32_t)a[k], h0 = key * 2654435761u;
                    // the class by other bits than the slot
                    if (((h0 & 0xFFFFu) ^ (key >> 7)) % parts != p) continue;
                    uint32_t h = h0 >> (32 - bits);
                    for (;;) {
                        uint32_t prev = keys[h];
                        if (prev == kEmpty) {
                            if (*vnum > kMost) break;  // too full: the row restarts
                            prev = atomicCAS(&keys[h], kEmpty, key);
                            if (prev == kEmpty) atomicAdd(&num, 1u);
                        }
                        if (prev == kEmpty || prev == key) {
                            atomicAdd(&cnts[h], 1u);
                            break;
                        }
                        h = (h + 1) & (uint32_t)(slots - 1);
                    }
                }
            }
            __syncthreads();
            const bool full = *vnum > kMost;
            if (!full)
                for (int k = tid; k < slots; k += kBlock) {
                    const uint32_t key = keys[k];
                    if (key == kEmpty) continue;
                    const int c = (int)cnts[k], sz = aggsize[key];
                    if (better(c, sz, (int)key, bc, bs, ba)) {
                        bc = c;
                        bs = sz;
                        ba = (int)key;
                    }
                }
            __syncthreads();  // the map is cleared next
            if (full) {
                parts *= 2;  // the candidates seen so far stay: they are whole counts
                p = 0;
            } else {
                p++;
            }
        }
        p3_group_best<64>(bc, bs, ba);
        if (lane == 0) {
            best[wv][0] = bc;
            best[wv][1] = bs;
            best[wv][2] = ba;
        }
        __syncthreads();
        if (tid == 0) {
            for (int q = 1; q < kWv; q++)
                if (better(best[q][0], best[q][1], best[q][2], bc, bs, ba)) {
                    bc = best[q][0];
                    bs = best[q][1];
                    ba = best[q][2];
                }
            if (bc > 0)
                agg_out[v] = ba;
            else
                *err = 1u;
        }
        __syncthreads();
    };
    const int64_t W = gridDim.x;
    for (int64_t w0 = blockIdx.x; w0 < io.S; w0 += kBlock * W) {
        const int64_t mine = w0 + tid * W;
        const uint32_t c = mine < io.S ? io.cnt_in[mine] : 0u;
        const uint64_t any = __ballot(c != 0u);
        __syncthreads();
        counts[tid] = c;
        if (lane == 0) marks[wv] = any;
        __syncthreads();
        for (int q = 0; q < kWv; q++) {
            for (uint64_t todo = marks[q]; todo; todo &= todo - 1) {
                const int j = q * 64 + __ffsll((unsigned long long)todo) - 1;
                const uint32_t count = counts[j];
                const int64_t sbase = (w0 + (int64_t)j * W) * io.seg;
                for (uint32_t i = 0; i < count; i++) row(io.wl_in[sbase + i]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Algorithm 2's second loop: every vertex left unaggregated by the first loop
// joins the aggregate of a neighbour -- the smallest aggregate id among its
// neighbours' first-loop labels.  The labels are read as unsigned, so -1
// (unaggregated) is above every id and never wins.  The labels read are
// the frozen first-loop ones (label); the result goes to agg_out, so rows
// are independent.
// ---------------------------------------------------------------------------

// Smallest label (as unsigned) over the column indices [s, e), by the whole
// wavefront.
__device__ __forceinline__ uint32_t coop_min_label(const int32_t *__restrict__ col,
                                                   const int32_t *__restrict__ label, int64_t s,
                                                   int64_t e) {
    const int lane = (int)(threadIdx.x & 63u);
    uint32_t m = 0xFFFFFFFFu;
    for (int64_t b = s; b < e; b += 64 * kCoopLoads) {
        int32_t x[kCoopLoads];
#pragma unroll
        for (int k = 0; k < kCoopLoads; k++) {
            const int64_t j = b + (int64_t)k * 64 + lane;
            x[k] = col[j < e ? j : s];
        }
        uint32_t a[kCoopLoads];
#pragma unroll
        for (int k = 0; k < kCoopLoads; k++) a[k] = (uint32_t)label[x[k]];
#pragma unroll
        for (int k = 0; k < kCoopLoads; k++)
            if (b + (int64_t)k * 64 + lane < e) m = min(m, a[k]);
    }
    return group_min<64>(m);
}

// One group of L lanes per row of the wavefront's segment of io.wl_in (the
// unaggregated vertices), K chunks of L column indices loaded before their
// labels are gathered; rows longer than 32 * L go to the whole wavefront.
// A vertex with no aggregated neighbour sets *err (host-pinned: a plain store).
template <int L>
__global__ __launch_bounds__(kBlock) void k_join_min(const int64_t *__restrict__ row_ptr,
                                                     const int32_t *__restrict__ col,
                                                     const int32_t *__restrict__ label,
                                                     SegIO io, int32_t *__restrict__ agg_out,
                                                     uint32_t *__restrict__ err) {
    constexpr int K = L >= 32 ? 1 : (32 / L > 8 ? 8 : 32 / L);
    constexpr int G = 64 / L;
    constexpr int64_t kLong = L >= 64 ? 1024 : (int64_t)32 * L;
    const int64_t w = wave_id();
    if (w >= io.S) return;
    const int64_t count = io.cnt_in[w];
    const int64_t sbase = w * io.seg;
    const int lane = (int)(threadIdx.x & 63u);
    const int sub = lane & (L - 1);
    for (int64_t i0 = 0; i0 < count; i0 += G) {
        const int64_t i = i0 + lane / L;
        const bool valid = i < count;
        const int32_t v = io.wl_in[sbase + (valid ? i : count - 1)];
        const int64_t s = row_ptr[v];
        int64_t e = valid ? row_ptr[v + 1] : s;
        uint32_t m = 0xFFFFFFFFu;
        uint64_t heavy = __ballot(sub == 0 && e - s > kLong);
        while (heavy) {
            const int src = __ffsll((unsigned long long)heavy) - 1;
            heavy &= heavy - 1;
            const uint32_t hm =
                coop_min_label(col, label, __shfl(s, src, 64), __shfl(e, src, 64));
            if ((lane & ~(L - 1)) == (src & ~(L - 1))) {
                m = min(m, hm);
                e = s;  // its group skips the row below
            }
        }
        const int64_t wmax = group_max64<64>(e - s);
        for (int64_t c0 = 0; c0 < wmax; c0 += (int64_t)L * K) {
            int32_t x[K];
#pragma unroll
            for (int k = 0; k < K; k++) {
                const int64_t j = s + c0 + k * L + sub;
                x[k] = col[j < e ? j : 0];
            }
            uint32_t a[K];
#pragma unroll
            for (int k = 0; k < K; k++) a[k] = (uint32_t)label[x[k]];
#pragma unroll
            for (int k = 0; k < K; k++)
                if (s + c0 + k * L + sub < e) m = min(m, a[k]);
        }
        m = group_min<L>(m);
        if (valid && sub == 0) {
            if (m == 0xFFFFFFFFu)
                *err = 2u;
            else
                agg_out[v] = (int32_t)m;
        }
    }
}

int grid_for(int64_t work, int per_block, int cap) {
    int64_t b = (work + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

}  // namespace

hipError_t launch_label_roots(int64_t n, const int64_t *row_ptr, const int32_t *col,
                              const int32_t *roots, const uint32_t *d_count,
                              const uint32_t *d_base, bool only_unlabelled, int32_t *label,
                              int32_t *aggsize, uint8_t *root_mark, uint8_t mark, hipStream_t s) {
    hipLaunchKernelGGL(k_label_roots, dim3(grid_for(n / 8 + 1, kBlock / kLabelLanes, 4096)),
                       dim3(kBlock), 0, s, row_ptr, col, roots, d_count, d_base,
                       (int)only_unlabelled, label, aggsize, root_mark, mark);
    return hipGetLastError();
}

hipError_t launch_accept_phase2(int64_t n, const int64_t *row_ptr, const int32_t *col,
                                const uint32_t *T, const int32_t *label, uint8_t *flag,
                                hipStream_t s) {
    if (4 * n < ((int64_t)1 << 32))
        hipLaunchKernelGGL(k_accept_phase2<true>, dim3(grid_for(n, kBlock, 4096)), dim3(kBlock), 0,
                           s, n, row_ptr, col, T, label, flag);
    else
        hipLaunchKernelGGL(k_accept_phase2<false>, dim3(grid_for(n, kBlock, 4096)), dim3(kBlock),
                           0, s, n, row_ptr, col, T, label, flag);
    return hipGetLastError();
}

hipError_t launch_list_unlabelled(int blocks, int64_t n, const int32_t *label, int32_t *copy_to,
                                  const SegIO &io, hipStream_t s) {
    hipLaunchKernelGGL(k_list_unlabelled, dim3(blocks), dim3(kBlock), 0, s, n, label, copy_to, io);
    return hipGetLastError();
}

#define MIS2_P3_DISPATCH(L, ...)                                                       \
    switch (L) {                                                                       \
        case 1: hipLaunchKernelGGL(k_phase3<1>, __VA_ARGS__); break;                   \
        case 2: hipLaunchKernelGGL(k_phase3<2>, __VA_ARGS__); break;                   \
        case 4: hipLaunchKernelGGL(k_phase3<4>, __VA_ARGS__); break;                   \
        case 8: hipLaunchKernelGGL(k_phase3<8>, __VA_ARGS__); break;                   \
        case 16: hipLaunchKernelGGL(k_phase3<16>, __VA_ARGS__); break;                 \
        case 32: hipLaunchKernelGGL(k_phase3<32>, __VA_ARGS__); break;                 \
        case 64: hipLaunchKernelGGL(k_phase3<64>, __VA_ARGS__); break;                 \
        default: return hipErrorInvalidValue;                                          \
    }

#define MIS2_JOIN_DISPATCH(L, ...)                                                     \
    switch (L) {                                                                       \
        case 1: hipLaunchKernelGGL(k_join_min<1>, __VA_ARGS__); break;                 \
        case 2: hipLaunchKernelGGL(k_join_min<2>, __VA_ARGS__); break;                 \
        case 4: hipLaunchKernelGGL(k_join_min<4>, __VA_ARGS__); break;                 \
        case 8: hipLaunchKernelGGL(k_join_min<8>, __VA_ARGS__); break;                 \
        case 16: hipLaunchKernelGGL(k_join_min<16>, __VA_ARGS__); break;               \
        case 32: hipLaunchKernelGGL(k_join_min<32>, __VA_ARGS__); break;               \
        case 64: hipLaunchKernelGGL(k_join_min<64>, __VA_ARGS__); break;               \
        default: return hipErrorInvalidValue;                                          \
    }

hipError_t launch_join_min(int lanes, int blocks, const int64_t *row_ptr, const int32_t *col,
                           const int32_t *label, const SegIO &io, int32_t *agg_out,
                           uint32_t *err, hipStream_t s) {
    MIS2_JOIN_DISPATCH(lanes, dim3(blocks), dim3(kBlock), 0, s, row_ptr, col, label, io, agg_out,
                       err);
    return hipGetLastError();
}

hipError_t launch_phase3(int lanes, int blocks, const int64_t *row_ptr, const int32_t *col,
                         const int32_t *label, const int32_t *aggsize, const SegIO &io,
                         const SegIO &io_mid, int64_t max_row, int32_t *agg_out, uint32_t *err,
                         hipStream_t s) {
    MIS2_P3_DISPATCH(lanes, dim3(blocks), dim3(kBlock), 0, s, row_ptr, col, label, aggsize, io,
                     agg_out, err);
    if (max_row > 32) {  // k_phase3 keeps up to 32 entries whatever its lanes
        // about 16 wavefronts per SIMD (of 1024), twice what is resident, so that a
        // segment of many hubs does not hold the launch up (Chung-Lu 1 065 829
        // vertices: 8 per SIMD 30.6 us, 16 19.8)
        const int share = (int)std::max<int64_t>(1, std::min<int64_t>(8, 16384 / io_mid.S));
        hipLaunchKernelGGL(k_phase3_mid, dim3((unsigned)(blocks * share)), dim3(kBlock), 0, s,
                           row_ptr, col, label, aggsize, io_mid, share, agg_out, err);
    }
    if (max_row > kP3Wave) {
        SegIO io_long = io_mid;
        io_long.wl_in = io_mid.wl_out;
        io_long.cnt_in = io_mid.cnt_out;
        io_long.wl_out = nullptr;
        io_long.cnt_out = nullptr;
        hipLaunchKernelGGL(k_phase3_long, dim3(std::min(blocks * 4, kP3LongBlocks)), dim3(kBlock),
                           0, s, row_ptr, col, label, aggsize, io_long, agg_out, err);
    }
    return hipGetLastError();
}

}  // namespace mis2
