// small.hip -- Algorithm 1 and Algorithm 3 of a small graph in one workgroup.
//
// On a few thousand vertices the launched form spends its time on launches:
// the 5-point 64 x 64 grid (16 128 entries) aggregates in 40 of them, 3 to 6 us
// each, every one a chain of dependent loads from memory that another launch
// has just written.  Here one workgroup of 16 wavefronts keeps the tuples, the
// minima, the worklists, the labels and the rows in LDS and
// runs every round and all three phases with workgroup barriers between them.
// Wavefront w owns the vertices [w * seg, (w + 1) * seg) and keeps its part of
// each worklist in order in its own slots, as the launched sweeps do, so there
// are no atomics, and results do not depend on the order (a minimum, any / all,
// integer sums).  One compute unit's throughput bounds the size: see the rule
// in small_fits.
#include <algorithm>

#include "internal.h"
#include "lanes.h"
#include "phase3.h"

namespace mis2 {

namespace {

constexpr int kSmThreads = 1024;
constexpr int kSmWaves = kSmThreads / 64;
constexpr int kSmRow = 128;   // longer rows: the whole wavefront
constexpr int kSmShort = 32;  // rows of phase 3 that four lanes hold
constexpr int kSmLoads = 4;   // entries of a lane's row loaded together
constexpr uint16_t kNone = 0xFFFFu;

constexpr int kSmN = 4096;   // vertices at most
constexpr int kSmZ = 32768;  // entries at most

struct SmallLds {
    uint32_t T[kSmN], M[kSmN];
    uint16_t l1[kSmN], l2[kSmN];
    uint16_t lab[kSmN], size[kSmN];
    uint32_t off[kSmN + 1];
    uint16_t col[kSmZ];
    uint32_t c1[kSmWaves], c2[kSmWaves];
    int best[kSmWaves][3];
    uint32_t err;
};

__device__ __forceinline__ uint64_t below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

__device__ __forceinline__ uint32_t sum_waves(const uint32_t (&c)[kSmWaves]) {
    uint32_t t = 0;
    for (int k = 0; k < kSmWaves; k++) t += c[k];
    return t;
}

__device__ __forceinline__ uint32_t sum_before(const uint32_t (&c)[kSmWaves], int wv) {
    uint32_t t = 0;
    for (int k = 0; k < kSmWaves; k++) t += k < wv ? c[k] : 0u;
    return t;
}

template <bool AGG>
__global__ __launch_bounds__(kSmThreads) void k_small(SmallArgs a) {
    __shared__ SmallLds S;
    const int lane = (int)(threadIdx.x & 63u), wv = (int)(threadIdx.x >> 6), tid = (int)threadIdx.x;
    const int n = (int)a.n;
    const int seg = ((n + kSmWaves - 1) / kSmWaves + 63) / 64 * 64;  // whole chunks of 64
    const int lo = min(n, wv * seg), hi = min(n, lo + seg);

    auto start = [&](int v) -> int { return (int)S.off[v]; };
    auto nb = [&](int j) -> int { return (int)S.col[j]; };
    auto params = [&](int r) {
        return TupleParams{xs64star((a.seed << 32) ^ (uint64_t)r), a.pmask, a.b, a.batch};
    };
    // f(u) for every neighbour u of each lane's row [s, e), the last one more
    // often; rows of more than kSmRow entries are left out
    auto own_row = [&](int s, int e, auto f) {
        if (e - s > kSmRow) return;
        for (int j = s; j < e; j += kSmLoads) {
            int x[kSmLoads];
#pragma unroll
            for (int k = 0; k < kSmLoads; k++) x[k] = nb(min(j + k, e - 1));
#pragma unroll
            for (int k = 0; k < kSmLoads; k++) f(x[k]);
        }
    };
    // the same for one longer row, by the whole wavefront
    auto wide_row = [&](int s, int e, auto f) {
        for (int j = s + lane; j < e; j += 64 * kSmLoads) {
            int x[kSmLoads];
#pragma unroll
            for (int k = 0; k < kSmLoads; k++) x[k] = nb(min(j + 64 * k, e - 1));
#pragma unroll
            for (int k = 0; k < kSmLoads; k++) f(x[k]);
        }
    };
    // Refresh Column of 64 entries of worklist2 from i0 on; returns those kept,
    // which go to the slots from `kept` on
    auto column = [&](int i0, int m2, int kept) {
        const bool has = i0 + lane < m2;
        const int v = S.l2[lo + (has ? i0 + lane : i0)];
        const int s = start(v), e = has ? start(v + 1) : s;
        uint32_t m = S.T[v];
        own_row(s, e, [&](int u) { m = min(m, S.T[u]); });
        for (uint64_t heavy = __ballot(e - s > kSmRow); heavy; heavy &= heavy - 1) {
            const int l = __ffsll((unsigned long long)heavy) - 1;
            uint32_t h = kOut;
            wide_row(__builtin_amdgcn_readlane(s, l), __builtin_amdgcn_readlane(e, l),
                     [&](int u) { h = min(h, S.T[u]); });
            h = group_min<64>(h);
            if (lane == l) m = min(m, h);
        }
        if (m == kIn) m = kOut;
        if (has) S.M[v] = m;
        const bool keep = has && m != kOut;
        const uint64_t mask = __ballot(keep);
        if (keep) S.l2[lo + kept + __popcll(mask & below(lane))] = (uint16_t)v;
        return (int)__popcll(mask);
    };
    // Decide Set of 64 entries of worklist1, with the next round's tuples
    auto decide = [&](const TupleParams &next, int i0, int m1, int kept) {
        const bool has = i0 + lane < m1;
        const int v = S.l1[lo + (has ? i0 + lane : i0)];
        const uint32_t t0 = S.T[v], mv = S.M[v];
        bool out = mv == kOut, eq = mv == t0;
        const int s = start(v), e = has && !out ? start(v + 1) : s;
        own_row(s, e, [&](int u) {
            const uint32_t x = S.M[u];
            out |= x == kOut;
            eq &= x == t0 || x == kAbsent;
        });
        for (uint64_t heavy = __ballot(e - s > kSmRow); heavy; heavy &= heavy - 1) {
            const int l = __ffsll((unsigned long long)heavy) - 1;
            const uint32_t ref = (uint32_t)__builtin_amdgcn_readlane((int)t0, l);
            uint32_t ho = 0, he = 1;
            wide_row(__builtin_amdgcn_readlane(s, l), __builtin_amdgcn_readlane(e, l), [&](int u) {
                const uint32_t x = S.M[u];
                ho |= x == kOut ? 1u : 0u;
                he &= x == ref || x == kAbsent ? 1u : 0u;
            });
            ho = group_or<64>(ho);
            he = group_and<64>(he);
            if (lane == l) {
                out |= ho != 0;
                eq &= he != 0;
            }
        }
        const bool stay = has && !out && !eq;
        if (has) S.T[v] = out ? kOut : eq ? kIn : make_tuple(next, (uint32_t)v);
        const uint64_t mask = __ballot(stay);
        if (stay) S.l1[lo + kept + __popcll(mask & below(lane))] = (uint16_t)v;
        return (int)__popcll(mask);
    };

    // Every round of one run.  m1 / m2: this wavefront's entries of the
    // worklists in l1 / l2 (slots from lo on).
    auto rounds = [&](int phase, int m1, int m2) {
        uint32_t *rth = a.rt_host[phase];
        int r = 0;
        for (;; r++) {
            if (lane == 0) {
                S.c1[wv] = (uint32_t)m1;
                S.c2[wv] = (uint32_t)m2;
            }
            __syncthreads();  // and T of the round before
            const uint32_t n1 = sum_waves(S.c1), n2 = sum_waves(S.c2);
            if (tid == 0) {
                rth[(size_t)r * kRoundStride] = n1;
                rth[(size_t)r * kRoundStride + 1] = n2;
            }
            if (n1 == 0u || r + 2 >= kTraceCap) break;
            int kept = 0;
            for (int i0 = 0; i0 < m2; i0 += 64) kept += column(i0, m2, kept);
            m2 = kept;
            __syncthreads();  // M is complete
            const TupleParams next = params(r + 1);
            kept = 0;
            for (int i0 = 0; i0 < m1; i0 += 64) kept += decide(next, i0, m1, kept);
            m1 = kept;
        }
        if (tid == 0)
            __hip_atomic_store(a.end_host + phase, (unsigned long long)(r + 1), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        __syncthreads();  // the counts are read
    };

    // rows, round-0 tuples and identity lists
    {
        // many loads in flight: the rows come from memory just once
        constexpr int kF = 8;
        const int nnz = (int)a.nnz;
        for (int v0 = 0; v0 <= n; v0 += kF * kSmThreads) {
            int64_t x[kF];
#pragma unroll
            for (int k = 0; k < kF; k++) x[k] = a.row_ptr[min(v0 + k * kSmThreads + tid, n)];
#pragma unroll
            for (int k = 0; k < kF; k++) S.off[min(v0 + k * kSmThreads + tid, n)] = (uint32_t)x[k];
        }
        for (int j0 = 0; j0 < nnz; j0 += kF * kSmThreads) {
            int32_t x[kF];
#pragma unroll
            for (int k = 0; k < kF; k++) x[k] = a.col[min(j0 + k * kSmThreads + tid, nnz - 1)];
#pragma unroll
            for (int k = 0; k < kF; k++)
                S.col[min(j0 + k * kSmThreads + tid, nnz - 1)] = (uint16_t)x[k];
        }
    }
    const TupleParams first = params(0);
    for (int v = lo + lane; v < hi; v += 64) {
        S.T[v] = make_tuple(first, (uint32_t)v);
        S.l1[v] = S.l2[v] = (uint16_t)v;
    }
    if (tid == 0) S.err = 0u;
    __syncthreads();
    rounds(0, hi - lo, hi - lo);

    if constexpr (!AGG) {
        int cnt = 0;
        for (int v0 = lo; v0 < hi; v0 += 64) {
            const int v = v0 + lane;
            const bool in = v < hi && S.T[v] == kIn;
            if (v < hi) a.status[v] = in ? 1 : 0;
            cnt += __popcll(__ballot(in));
        }
        if (lane == 0) S.c1[wv] = (uint32_t)cnt;
        __syncthreads();
        if (tid == 0) a.host[kS_Roots] = sum_waves(S.c1);
    } else {
        // One group of roots: numbered by increasing id from `base` on, each
        // labelled with its neighbours (those still free when only_free).
        // flags: bit k of a lane says whether vertex lo + 64 k + lane is one.
        auto label_roots = [&](uint32_t flags, uint32_t base, bool only_free, uint8_t mark,
                               int32_t *list) -> uint32_t {
            int cnt = 0;
            for (int v0 = lo, k = 0; v0 < hi; v0 += 64, k++) cnt += __popcll(__ballot(flags >> k & 1u));
            if (lane == 0) S.c1[wv] = (uint32_t)cnt;
            __syncthreads();
            const uint32_t total = sum_waves(S.c1);
            uint32_t at = sum_before(S.c1, wv);
            for (int v0 = lo, k = 0; v0 < hi; v0 += 64, k++) {
                const bool in = flags >> k & 1u;
                const uint64_t mask = __ballot(in);
                const int v = v0 + lane;
                const uint32_t rank = at + (uint32_t)__popcll(mask & below(lane));
                const uint16_t id = (uint16_t)(base + rank);
                at += (uint32_t)__popcll(mask);
                if (in && list) list[rank] = v;
                int took = 0;
                const int s = in ? start(v) : 0, e = in ? start(v + 1) : 0;
                auto push = [&](int u, uint16_t with) {
                    if (!only_free || S.lab[u] == kNone) {
                        S.lab[u] = with;
                        took++;
                    }
                };
                uint64_t heavy = __ballot(e - s > kSmRow);
                if (e - s <= kSmRow)
                    for (int j = s; j < e; j++) push(nb(j), id);
                while (heavy) {
                    const int q = __ffsll((unsigned long long)heavy) - 1;
                    heavy &= heavy - 1;
                    const int hv = __builtin_amdgcn_readlane(v, q);
                    const uint16_t hid = (uint16_t)__builtin_amdgcn_readlane((int)id, q);
                    const int he = start(hv + 1);
                    const int own = took;
                    took = 0;
                    for (int j = start(hv) + lane; j < he; j += 64) push(nb(j), hid);
                    const int all = group_sum_i<64>(took);
                    took = lane == q ? own + all : own;
                }
                if (in) {
                    S.lab[v] = id;
                    S.size[id] = (uint16_t)(1 + took);
                    if (a.roots) a.roots[v] = mark;
                }
            }
            __syncthreads();
            return total;
        };

        // phase 1
        uint32_t flags = 0;
        for (int v = lo + lane, k = 0; v < hi; v += 64, k++) {
            S.lab[v] = kNone;
            if (a.roots) a.roots[v] = 0;
            flags |= (S.T[v] == kIn ? 1u : 0u) << k;
        }
        __syncthreads();
        const uint32_t n1 = label_roots(flags, 0, false, 1, a.list1);

        // phase 2: the subgraph induced by the vertices without a label
        int m = 0;
        for (int v0 = lo; v0 < hi; v0 += 64) {
            const int v = v0 + lane;
            const bool act = v < hi && S.lab[v] == kNone;
            const uint64_t mask = __ballot(act);
            const int at = lo + m + __popcll(mask & below(lane));
            if (act) S.l1[at] = S.l2[at] = (uint16_t)v;
            m += __popcll(mask);
            if (v < hi) {
                S.T[v] = act ? make_tuple(first, (uint32_t)v) : kOut;
                S.M[v] = kAbsent;
            }
        }
        __syncthreads();
        rounds(1, m, m);
        // its roots with at least two neighbours without a label
        flags = 0;
        for (int v0 = lo, k = 0; v0 < hi; v0 += 64, k++) {
            const int v = v0 + lane;
            const bool cand = v < hi && S.lab[v] == kNone && S.T[v] == kIn;
            const int s = cand ? start(v) : 0, e = cand ? start(v + 1) : 0;
            int cnt = 0;
            uint64_t heavy = __ballot(e - s > kSmRow);
            if (e - s <= kSmRow)
                for (int j = s; j < e; j++) cnt += S.lab[nb(j)] == kNone;
            while (heavy) {
                const int q = __ffsll((unsigned long long)heavy) - 1;
                heavy &= heavy - 1;
                const int hv = __builtin_amdgcn_readlane(v, q);
                const int he = start(hv + 1);
                int c = 0;
                for (int j = start(hv) + lane; j < he; j += 64) c += S.lab[nb(j)] == kNone;
                c = group_sum_i<64>(c);
                if (lane == q) cnt = c;
            }
            flags |= (cnt >= 2 ? 1u : 0u) << k;
        }
        __syncthreads();
        const uint32_t n2 = label_roots(flags, n1, true, 2, a.list2);

        // phase 3 on the labels as they are now: 4 lanes per row of up to 32
        // entries, the wavefront for rows of up to kP3Mid, and after them the
        // workgroup for longer ones (listed in l1), with a count per aggregate
        // in M
        int longer = 0;
        auto lab = [&](int u) { return S.lab[u] == kNone ? -1 : (int)S.lab[u]; };
        for (int v0 = lo; v0 < hi; v0 += 64) {
            const int vl = v0 + lane;
            const bool left = vl < hi && S.lab[vl] == kNone;
            if (vl < hi && !left) a.agg[vl] = (int32_t)S.lab[vl];
            const int s = left ? start(vl) : 0, d = left ? start(vl + 1) - s : 0;
            uint64_t brief = __ballot(left && d <= kSmShort);
            uint64_t mid = __ballot(left && d > kSmShort && d <= kP3Mid);
            const uint64_t huge = __ballot(left && d > kP3Mid);
            if (left && d > kP3Mid) S.l1[lo + longer + __popcll(huge & below(lane))] = (uint16_t)vl;
            longer += __popcll(huge);
            // 16 short rows at a time: group g takes the g-th of those left
            while (brief) {
                uint64_t rest = brief;
                int src = -1;
                for (int g = 0; g < 16; g++) {
                    const int l = rest ? __ffsll((unsigned long long)rest) - 1 : -1;
                    if (lane >> 2 == g) src = l;
                    rest &= rest - 1;
                }
                brief = rest;
                const int v = v0 + max(src, 0);
                const int rs = start(v);
                const int len = src >= 0 ? start(v + 1) - rs : 0;
                int bc = 0, bs = 0x7FFFFFFF, ba = 0x7FFFFFFF;
                int32_t x[8], sz[8];
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const int j = 4 * k + (lane & 3);
                    x[k] = j < len ? lab(nb(rs + j)) : kPad;
                    sz[k] = (int)S.size[x[k] >= 0 ? x[k] : 0];
                }
                p3_count<4, 8>(x, sz, bc, bs, ba);
                p3_group_best<4>(bc, bs, ba);
                if (src >= 0 && (lane & 3) == 0) {
                    if (bc > 0)
                        a.agg[v] = ba;
                    else
                        S.err = 1u;
                }
            }
            while (mid) {
                const int l = __ffsll((unsigned long long)mid) - 1;
                mid &= mid - 1;
                const int v = v0 + l;
                const int rs = start(v);
                int bc = 0, bs = 0x7FFFFFFF, ba = 0x7FFFFFFF;
                p3_mid<kP3Mid>(
                    start(v + 1) - rs, [&](int j) { return nb(rs + j); }, lab,
                    [&](int y) { return (int)S.size[y]; }, bc, bs, ba);
                if (lane == 0) {
                    if (bc > 0)
                        a.agg[v] = ba;
                    else
                        S.err = 1u;
                }
            }
        }
        if (lane == 0) S.c1[wv] = (uint32_t)longer;
        __syncthreads();
        const int na = (int)(n1 + n2);
        for (int w = 0; w < kSmWaves; w++) {
            const int cnt = (int)S.c1[w];
            for (int i = 0; i < cnt; i++) {
                const int v = S.l1[min(n, w * seg) + i];
                for (int y = tid; y < na; y += kSmThreads) S.M[y] = 0u;
                __syncthreads();
                const int e = start(v + 1);
                for (int j = start(v) + tid; j < e; j += kSmThreads) {
                    const int y = lab(nb(j));
                    if (y >= 0) atomicAdd(&S.M[y], 1u);
                }
                __syncthreads();
                int bc = 0, bs = 0x7FFFFFFF, ba = 0x7FFFFFFF;
                for (int y = tid; y < na; y += kSmThreads) {
                    const int c = (int)S.M[y], sz = (int)S.size[y];
                    if (c > 0 && better(c, sz, y, bc, bs, ba)) {
                        bc = c;
                        bs = sz;
                        ba = y;
                    }
                }
                p3_group_best<64>(bc, bs, ba);
                if (lane == 0) {
                    S.best[wv][0] = bc;
                    S.best[wv][1] = bs;
                    S.best[wv][2] = ba;
                }
                __syncthreads();
                if (tid == 0) {
                    for (int q = 1; q < kSmWaves; q++)
                        if (better(S.best[q][0], S.best[q][1], S.best[q][2], bc, bs, ba)) {
                            bc = S.best[q][0];
                            bs = S.best[q][1];
                            ba = S.best[q][2];
                        }
                    if (bc > 0)
                        a.agg[v] = ba;
                    else
                        S.err = 1u;
                }
                __syncthreads();
            }
        }
        __syncthreads();
        if (tid == 0) {
            a.host[kS_Count1] = n1;
            a.host[kS_Count2] = n2;
            a.host[kS_Err] = S.err;
            if (a.scalars) {
                a.scalars[kS_Count1] = n1;
                a.scalars[kS_Count2] = n2;
            }
        }
    }
}

}  // namespace

// As far as the LDS goes.  Measured, one aggregation in this form against the
// launched one (us): 5-point 32 x 32 50 / 199 and 64 x 64 81 / 213; 7-point
// 10^3 61 / 215; 27-point 10^3 (20 952 entries) 94 / 227; Chung-Lu 2000
// (24 466) 200 / 300.  Past it the one compute unit loses: with the rows read
// from memory in place of LDS, 5-point 90 x 90 took 200 / 208, 27-point 13^3
// (48 456) 248 / 278 and 16^3 (93 240) 397 / 279.
bool small_fits(int64_t n, int64_t nnz) { return n >= 1 && n <= kSmN && nnz <= kSmZ; }

hipError_t launch_small(const SmallArgs &a, bool agg, hipStream_t s) {
    if (!small_fits(a.n, a.nnz)) return hipErrorInvalidValue;
    if (agg)
        hipLaunchKernelGGL(k_small<true>, dim3(1), dim3(kSmThreads), 0, s, a);
    else
        hipLaunchKernelGGL(k_small<false>, dim3(1), dim3(kSmThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace mis2
