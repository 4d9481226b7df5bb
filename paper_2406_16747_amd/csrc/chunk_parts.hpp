// The end of a chunk (see chunk.hip): which entries survive it, and their rows.  Device functions, because they run in launches of the
// attention where its MFMA kernels do the work, and in launches of their own elsewhere.
#pragma once
#include "common.hpp"

namespace spk {

// The survivors of one row, in position order: the last w entries, the keys still selected for the
// last prefix used so far (T = nv - 1 - w) and every other real key whose score is above that
// prefix's threshold.  The first two classes always fit; if the third does not, its oldest members
// are dropped and bit 0 of the row's flag word is set (later thresholds are then approximate).
//
// One workgroup per row, so what counts is the number of dependent round trips: a wave owns a contiguous run of positions,
// fetches 8 x 64 of them at once, whatever their class, and takes counts and ranks from ballots.  Classes are formed again
// in the second pass, from loads that are in flight together with the scores it needs anyway.
// Rows of 14336 virtual positions: 17 -> 11 us; four chunks of 8192 tokens with their attention 1626 -> 1588 us.
constexpr int RETAIN_UNR = 8;

// What a chunk adds to the launches of the attention: the lists' launch clears lifetimes and finds the survivors of every row
// (a workgroup of 1024 threads per row), the attention's moves the survivors' K and V rows (workgroups of 256).
struct ChunkTail {
    const unsigned long long* kept;   // [rows][rcap / 64]: the retained entries that may be selected (see chunk_clear_padding)
    int32_t *count, *flags;
    const float *u, *tau;
    int32_t* death;
    int rcap, clen, w;
    int32_t* map;
    float* ret_u;
    int32_t* ret_sel;
    const uint4 *k, *v;               // rows of the virtual sequence
    uint4 *ret_k, *ret_v;
    int unit;                         // 16-byte units per row
    int wgs;                          // workgroups per head that move rows

    // the lifetime of position e of a row
    __device__ __forceinline__ int lifetime(int row, int e) const
    {
        // (both loads without a condition, so that a caller's loads stay in flight together)
        const int d = death[(size_t)row * (rcap + clen) + e], c = min(e, rcap - 1);
        const unsigned word = ((const unsigned*)kept)[(size_t)row * (rcap / 32) + (c >> 5)];
        return (e >= rcap) | (word >> (c & 31) & 1) ? d : e;
    }
};

// Padding entries are never selected: death[e] = e.  The same holds for retained keys that were
// kept only because their score is above the threshold: they left the top-k in an earlier chunk, at
// a prefix whose block the mask skips, so their lifetime is still at its preset.
// Thread `first` of `threads` that clear a row.  (Whoever reads lifetimes in the same launch goes through lifetime(): a
// cleared one and one that is about to be come to the same.)
__device__ __forceinline__ void chunk_clear_padding(const ChunkTail& c, int row, int first, int threads)
{
    const unsigned long long* kept = c.kept + (size_t)row * (c.rcap / 64);
    for (int e = first; e < c.rcap; e += threads)
        if (!(kept[e >> 6] >> (e & 63) & 1)) c.death[(size_t)row * (c.rcap + c.clen) + e] = e;
}

struct RetainSmem {
    int wt[2][16];
};

// CLEARED: an earlier launch has cleared the lifetimes (9.9 us against 11.7 with lifetime(), a row of 9088 virtual positions).
template <bool CLEARED>
__device__ __forceinline__ void chunk_retain(RetainSmem& sm, const ChunkTail& c, int row)
{
    auto& wt = sm.wt;
    const int rcap = c.rcap, clen = c.clen, w = c.w;
    int32_t *count = c.count, *flags = c.flags, *map = c.map, *ret_sel = c.ret_sel;
    float* ret_u = c.ret_u;
    const float *u_v = c.u, *tau_v = c.tau;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nv = rcap + clen;
    const int pad = rcap - count[row];
    const int T = nv - 1 - w;  // last prefix any query has used
    const float* ur = u_v + (size_t)row * nv;
    const float thr = T >= pad ? tau_v[(size_t)row * nv + T] : -INFINITY;
    const int groups = (nv + 63) / 64, per = (groups + 15) / 16;
    const int g0 = min(wv * per, groups), g1 = min(g0 + per, groups);
    // class 1: mandatory (window, or selected for prefix T); class 2: other keys above the threshold
    float uu[RETAIN_UNR];
    unsigned long long m1[RETAIN_UNR], m2[RETAIN_UNR];
    auto classify = [&](int g) {
        int dd[RETAIN_UNR];
#pragma unroll
        for (int x = 0; x < RETAIN_UNR; x++) {
            const int e = min((g + x) * 64 + lane, nv - 1);
            dd[x] = CLEARED ? c.death[(size_t)row * nv + e] : c.lifetime(row, e);
            uu[x] = ur[e];
        }
#pragma unroll
        for (int x = 0; x < RETAIN_UNR; x++) {
            const int e = (g + x) * 64 + lane;
            const bool in = g + x < g1 && e >= pad && e < nv, must = e > T || dd[x] > T;
            m1[x] = __ballot(in && must);
            m2[x] = __ballot(in && !must && uu[x] > thr);
        }
    };
    int n1 = 0, n2 = 0;
    for (int g = g0; g < g1; g += RETAIN_UNR) {
        classify(g);
#pragma unroll
        for (int x = 0; x < RETAIN_UNR; x++) {
            n1 += __popcll(m1[x]);
            n2 += __popcll(m2[x]);
        }
    }
    if (lane == 0) {
        wt[0][wv] = n1;
        wt[1][wv] = n2;
    }
    __syncthreads();
    int p1 = 0, p2 = 0, t1 = 0, t2 = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        if (i < wv) {
            p1 += wt[0][i];
            p2 += wt[1][i];
        }
        t1 += wt[0][i];
        t2 += wt[1][i];
    }
    const int allowed = rcap - t1;        // >= 0: the mandatory classes hold at most k + w entries
    const int drop = t2 > allowed ? t2 - allowed : 0;  // the oldest `drop` members of class 2 go
    const unsigned long long below = (1ull << lane) - 1;
    for (int g = g0; g < g1; g += RETAIN_UNR) {
        classify(g);
#pragma unroll
        for (int x = 0; x < RETAIN_UNR; x++) {
            const bool must = m1[x] >> lane & 1, above = m2[x] >> lane & 1;
            const int before = p2 + __popcll(m2[x] & below);   // members of class 2 ahead of this entry
            if (must || (above && before >= drop)) {
                const size_t j = (size_t)row * rcap + p1 + __popcll(m1[x] & below) + max(before - drop, 0);
                map[j] = (g + x) * 64 + lane;
                ret_u[j] = uu[x];
                ret_sel[j] = must;
            }
            p1 += __popcll(m1[x]);
            p2 += __popcll(m2[x]);
        }
    }
    if (tid == 0) {  // every thread has read the old count (before the barrier)
        count[row] = t1 + t2 - drop;
        if (drop > 0) flags[row] |= 1;
    }
}

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));   // (arrays of uint4 would live in scratch memory)
// Workgroup `wg` of the c.wgs that move the surviving rows of head bh (score row `row`).
__device__ __forceinline__ void chunk_retain_rows(const ChunkTail& c, int bh, int row, int wg)
{
    const int nv = c.rcap + c.clen, unit = c.unit;
    const int total = c.count[row] * unit, step = c.wgs * 256;
    const int32_t* map = c.map + (size_t)row * c.rcap;
    const size_t src = (size_t)bh * nv * unit, dst = (size_t)bh * c.rcap * unit;
    for (int x0 = wg * 256 + threadIdx.x; x0 < total; x0 += 4 * step) {
        u32x4_t k[4], v[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int x = min(x0 + i * step, total - 1), j = x / unit, at = x - j * unit;
            const size_t from = src + (size_t)map[j] * unit + at;
            k[i] = ((const u32x4_t*)c.k)[from];
            v[i] = ((const u32x4_t*)c.v)[from];
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int x = x0 + i * step;
            if (x < total) {
                ((u32x4_t*)c.ret_k)[dst + x] = k[i];
                ((u32x4_t*)c.ret_v)[dst + x] = v[i];
            }
        }
    }
}

}  // namespace spk
