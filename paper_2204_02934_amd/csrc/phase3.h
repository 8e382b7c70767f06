// phase3.h -- counting the couplings of one row in phase 3 of Algorithm 3
// (Section III-B): the pieces that the launched kernels and the one-workgroup
// form of small graphs share.
#pragma once

#include "lanes.h"

namespace mis2 {

// Candidate order of phase 3: larger coupling first, then smaller aggsize,
// then smaller aggregate id.  Returns true if (c1, s1, a1) beats (c2, s2, a2).
__device__ __forceinline__ bool better(int c1, int s1, int a1, int c2, int s2, int a2) {
    if (c1 != c2) return c1 > c2;
    if (s1 != s2) return s1 < s2;
    return a1 < a2;
}

// The best (coupling, size, id) candidate over each aligned group of L lanes,
// in every lane of the group.
template <int J>
__device__ __forceinline__ void p3_best_step(int &bc, int &bs, int &ba) {
    const int oc = lane_xor_i<J>(bc), os = lane_xor_i<J>(bs), oa = lane_xor_i<J>(ba);
    if (better(oc, os, oa, bc, bs, ba)) {
        bc = oc;
        bs = os;
        ba = oa;
    }
}

template <int L>
__device__ __forceinline__ void p3_group_best(int &bc, int &bs, int &ba) {
    if constexpr (L >= 64) p3_best_step<32>(bc, bs, ba);
    if constexpr (L >= 32) p3_best_step<16>(bc, bs, ba);
    if constexpr (L >= 16) p3_best_step<8>(bc, bs, ba);
    if constexpr (L >= 8) p3_best_step<4>(bc, bs, ba);
    if constexpr (L >= 4) p3_best_step<2>(bc, bs, ba);
    if constexpr (L >= 2) p3_best_step<1>(bc, bs, ba);
}

constexpr int32_t kPad = -2;  // label of a padding lane; never equals an aggregate id

// Short rows: lane j of the group holds the tent labels of neighbours
// k*L + j for k < K, and the sizes of their aggregates, all loaded before any
// is used.  Every lane broadcasts its K labels to the group once; each lane
// counts, for each of its own labels, the equal ones among all L*K (its
// coupling), and keeps its best candidate in the order above.  (Counting
// only the chunks that the wavefront's longest row reaches was measured on
// gfx950 and changed nothing: 30.7 us on the 27-point 100^3 graph, 217 us
// on Chung-Lu 4M, either way.)
template <int L, int K>
__device__ __forceinline__ void p3_count(const int32_t (&a)[K], const int32_t (&sz)[K], int &bc,
                                         int &bs, int &ba) {
    int cnt[K];
#pragma unroll
    for (int k = 0; k < K; k++) cnt[k] = 0;
#pragma unroll
    for (int t = 0; t < L; t++) {
#pragma unroll
        for (int k2 = 0; k2 < K; k2++) {
            const int32_t b = __shfl(a[k2], t, L);
#pragma unroll
            for (int k = 0; k < K; k++) cnt[k] += (b == a[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < K; k++) {
        if (a[k] >= 0 && better(cnt[k], sz[k], a[k], bc, bs, ba)) {
            bc = cnt[k];
            bs = sz[k];
            ba = a[k];
        }
    }
}

// Rows of up to kP3Mid entries, one wavefront each, K entries per lane in
// registers.  On a mesh a row couples to few aggregates (a 27-point row of three
// unknowns: 80 entries, some 6 aggregates), so they are counted one by one: the
// first lane not yet counted names its label, and ballots count it among all
// K * 64 entries, some 100 cycles an aggregate.  A hub's row may couple to as
// many aggregates as it has entries: past kP3Few of them a row of up to 128
// entries compares each label with all, as p3_count does, some 10 cycles an
// entry (Chung-Lu 33 587 vertices, k_phase3_mid 23.5 us with up to 128 aggregates
// one by one).  Returns (scalars) the best candidate in the order above.
constexpr int kP3Mid = 512;
constexpr int kP3Few = 8;
// nb(j): the row's j-th neighbour; lab(u): a vertex's label (negative: none);
// size(y): an aggregate's size.
template <int K, typename NB, typename LAB, typename SIZE>
__device__ __forceinline__ void p3_mid_row(int len, NB nb, LAB lab, SIZE size, int &bc, int &bs,
                                           int &ba) {
    constexpr bool kPairs = K <= 2;
    const int lane = (int)(threadIdx.x & 63u);
    int32_t a[K], sz[K];
#pragma unroll
    for (int k = 0; k < K; k++) a[k] = nb(min(k * 64 + lane, len - 1));
#pragma unroll
    for (int k = 0; k < K; k++) a[k] = lab(a[k]);
    uint64_t left[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        if (k * 64 + lane >= len) a[k] = kPad;
        left[k] = __ballot(a[k] >= 0);
        sz[k] = size(a[k] >= 0 ? a[k] : 0);
    }
    int found = 0;
#pragma unroll
    for (int k = 0; k < K; k++) {
        while (left[k] && (!kPairs || found < kP3Few)) {
            const int l = __ffsll((unsigned long long)left[k]) - 1;
            const int32_t y = __builtin_amdgcn_readlane(a[k], l);
            const int ysz = __builtin_amdgcn_readlane(sz[k], l);
            int c = 0;
#pragma unroll
            for (int q = k; q < K; q++) {
                const uint64_t eq = __ballot(a[q] == y);
                c += __popcll(eq);
                left[q] &= ~eq;
            }
            if (better(c, ysz, y, bc, bs, ba)) {
                bc = c;
                bs = ysz;
                ba = y;
            }
            found++;
        }
    }
    if constexpr (kPairs) {
        uint64_t rest = 0;
#pragma unroll
        for (int k = 0; k < K; k++) rest |= left[k];
        if (!rest) return;
        int cnt[K] = {}, c = 0, s = 0x7FFFFFFF, y = 0x7FFFFFFF;
#pragma unroll
        for (int q = 0; q < K; q++) {
            const int m = min(64, len - q * 64);
            for (int t = 0; t < m; t++) {
                const int32_t b = __builtin_amdgcn_readlane(a[q], t);
#pragma unroll
                for (int k = 0; k < K; k++) cnt[k] += b == a[k];
            }
        }
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (a[k] >= 0 && better(cnt[k], sz[k], a[k], c, s, y)) {
                c = cnt[k];
                s = sz[k];
                y = a[k];
            }
        }
        p3_group_best<64>(c, s, y);
        // (the aggregates counted one by one are among these)
        bc = __builtin_amdgcn_readfirstlane(c);
        bs = __builtin_amdgcn_readfirstlane(s);
        ba = __builtin_amdgcn_readfirstlane(y);
    }
}

// Rows of up to MAX entries (kP3Mid, or 128).
template <int MAX, typename NB, typename LAB, typename SIZE>
__device__ __forceinline__ void p3_mid(int len, NB nb, LAB lab, SIZE size, int &bc, int &bs,
                                       int &ba) {
    static_assert(MAX == 128 || MAX == kP3Mid, "p3_mid: two or kP3Mid / 64 entries a lane");
    if (len <= 64)
        p3_mid_row<1>(len, nb, lab, size, bc, bs, ba);
    else if (MAX == 128 || len <= 128)
        p3_mid_row<2>(len, nb, lab, size, bc, bs, ba);
    else
        p3_mid_row<kP3Mid / 64>(len, nb, lab, size, bc, bs, ba);
}

}  // namespace mis2
