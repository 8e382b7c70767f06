// rowset.h -- the distinct columns of a sparse output row (a coarse row of the
// quotient graph, a row of a product's structure), collected in LDS by a group
// of lanes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lanes.h"

namespace mis2 {

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CAP>
__device__ __forceinline__ uint32_t qhash(uint32_t c) {
    static_assert((CAP & (CAP - 1)) == 0 && CAP >= 64 && CAP <= 65536, "CAP: a power of two");
    constexpr int bits = __builtin_ctz(CAP);
    return (c * 2654435761u) >> (32 - bits);
}

// Column indices of the entries q0 .. q0 + U - 1 (the last entry again past
// tot) of R rows numbered one after the other: off[r] the number of row r's
// first entry, base[r] the column index of entry 0 counted back from it.  One
// binary search finds the first entry's row; the others follow it, so a row
// of U entries or more costs its lane two LDS reads, not a search per entry
// (which kept these kernels bound by LDS reads).
template <int R, int U, typename Off>
__device__ __forceinline__ void walk_run(const Off *off, const int64_t *base, Off q0, Off tot,
                                         int64_t (&at)[U]) {
    int r = 0;  // the last row with off[r] <= q0 (it is not empty)
#pragma unroll
    for (int st = R / 2; st > 0; st >>= 1)
        if (off[r + st] <= q0) r += st;
    Off next = off[r + 1];
    int64_t b = base[r];
#pragma unroll
    for (int k = 0; k < U; k++) {
        const Off q = tot - q0 > (Off)k ? q0 + (Off)k : tot - 1;
        while (q >= next) {  // tot is the last offset, so this ends
            r++;
            next = off[r + 1];
            b = base[r];
        }
        at[k] = b + (int64_t)q;
    }
}

// One row's distinct columns, collected in an LDS hash set (open addressing) by
// a group of G lanes; each id that enters is also appended to a list.  The
// candidates are the entries of the source rows m0 .. m1 - 1: src(i, rs, d)
// gives the i-th one's start and length, then(first(j)) the candidate of entry
// j (negative: none; two steps, so that a lane's loads of each go out
// together).  The sources go G at a time; their entries are numbered by a scan
// of the lengths within the group and dealt out evenly, U in a row per lane
// loaded together.  Most candidates repeat an id the set already holds: a
// plain read of the slot comes before the compare-and-swap.  Returns false
// when the row has LIM or more distinct ids, or more than maxc candidates or
// sources (the set is then only partly filled).
template <int G, int CAP, int LIM>
struct RowSet {
    uint32_t tab[CAP];
    uint32_t list[LIM + G];
    int64_t base[G];     // column index of a member row's first entry, less its number
    uint32_t off[G + 1];
    uint32_t num;
};

template <int G>
__device__ __forceinline__ uint32_t group_incl_scan(uint32_t x) {
    if constexpr (G == 64) {
        return wave_incl_scan(x);
    } else {
        static_assert(G == 16, "group_incl_scan: a DPP row or the wavefront");
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
        return x;
    }
}

constexpr uint32_t kNoLimit = 0x7FFFFFFEu;  // maxc: as many candidates as there are

template <int G, int CAP, int LIM>
__device__ __forceinline__ void row_put(RowSet<G, CAP, LIM> &S, int32_t c) {
    static_assert(LIM + G <= CAP, "every lane of the group may add an id past the limit");
    constexpr uint32_t kEmpty = 0xFFFFFFFFu;
    const uint32_t key = (uint32_t)c;
    uint32_t h = qhash<CAP>(key);
    for (;;) {  // at most LIM - 1 + G slots are ever taken, so this ends
        uint32_t prev = S.tab[h];
        if (prev == kEmpty) {
            if (*(volatile uint32_t *)&S.num >= (uint32_t)LIM) break;  // over the limit already
            prev = atomicCAS(&S.tab[h], kEmpty, key);
            if (prev == kEmpty) {
                S.list[atomicAdd(&S.num, 1u)] = key;
                break;
            }
        }
        if (prev == key) break;
        h = (h + 1) & (CAP - 1);
    }
}

template <int G, int CAP, int LIM, int U, typename SRC, typename LD1, typename LD2>
__device__ __forceinline__ bool row_gather(RowSet<G, CAP, LIM> &S, int lane, int64_t m0, int64_t m1,
                                           uint32_t maxc, SRC src, LD1 first, LD2 then) {
    volatile uint32_t *num = &S.num;
    uint64_t all = 0;
    bool fits = m1 - m0 <= (int64_t)maxc;
    for (int64_t c0 = m0; fits && c0 < m1; c0 += G) {
        const int64_t i = c0 + lane;
        int64_t rs = 0, d = 0;
        if (i < m1) src(i, rs, d);
        // each length clamped past the limit: the sums stay below 2^32 (without
        // a limit the callers' lengths do)
        const uint32_t len = (uint32_t)min(d, (int64_t)maxc + 1);
        const uint32_t incl = group_incl_scan<G>(len);
        if (lane == 0) S.off[0] = 0u;
        S.off[lane + 1] = incl;
        S.base[lane] = rs - (int64_t)(incl - len);
        wave_sync();
        const uint32_t tot = S.off[G];
        all += tot;
        fits = (maxc == kNoLimit || all <= maxc) && *num < (uint32_t)LIM;
        if (fits) {
            for (uint32_t c1 = 0; c1 < tot; c1 += (uint32_t)(G * U)) {
                const uint32_t q0 = c1 + (uint32_t)(lane * U);
                if (q0 < tot) {
                    int64_t at[U];
                    walk_run<G, U>(S.off, S.base, q0, tot, at);
                    int32_t x[U];
#pragma unroll
                    for (int k = 0; k < U; k++) x[k] = first(at[k]);
                    int32_t c[U];
#pragma unroll
                    for (int k = 0; k < U; k++) c[k] = then(x[k]);
#pragma unroll
                    for (int k = 0; k < U; k++)
                        if (q0 + (uint32_t)k < tot && c[k] >= 0) row_put(S, c[k]);
                }
                // over the limit: the row goes on to the next path
                if (c1 + (uint32_t)(G * U) < tot && *num >= (uint32_t)LIM) break;
            }
        }
        wave_sync();  // the offsets are rewritten by the next chunk
    }
    return fits && *num < (uint32_t)LIM;
}

// Empties the set of a row: the slot of each listed id (its probe run holds
// it exactly once; other lanes' clears only leave holes), or all of it.
template <int G, int CAP, int LIM>
__device__ __forceinline__ void row_clear(RowSet<G, CAP, LIM> &S, int lane, uint32_t m, bool whole) {
    constexpr uint32_t kEmpty = 0xFFFFFFFFu;
    if (whole) {
        for (int i = lane; i < CAP; i += G) S.tab[i] = kEmpty;
    } else {
        for (uint32_t i = (uint32_t)lane; i < m; i += (uint32_t)G) {
            const uint32_t key = S.list[i];
            uint32_t h = qhash<CAP>(key);
            while (S.tab[h] != key) h = (h + 1) & (CAP - 1);
            S.tab[h] = kEmpty;
        }
    }
    wave_sync();
    if (lane == 0) S.num = 0u;
    wave_sync();
}

// out[0 .. m) = the m ids of the list in increasing order, each ranked by
// counting the smaller ones (ids are distinct).
template <int G, int CAP, int LIM>
__device__ __forceinline__ void row_write(const RowSet<G, CAP, LIM> &S, int lane, uint32_t m,
                                          int32_t *out) {
    for (uint32_t i = (uint32_t)lane; i < m; i += (uint32_t)G) {
        const uint32_t x = S.list[i];
        uint32_t rank = 0;
        for (uint32_t y = 0; y < m; y++) rank += S.list[y] < x ? 1u : 0u;
        out[rank] = (int32_t)x;
    }
}

}  // namespace mis2
