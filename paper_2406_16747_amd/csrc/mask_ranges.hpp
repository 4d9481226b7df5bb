// The fractional ranges of the score gradient: a device function, because it runs in a launch of its own or in the last
// workgroups of the attention backward's dK/dV kernel.
#pragma once
#include "common.hpp"

namespace spk {

struct RangesArgs {
    const float *u, *tau;
    int n, k, t_min;
    const int32_t* first_valid;
    int32_t* diff;   // nullptr: nothing to do
    int2* ab;
};

// What has to be cleared and filled before the score gradient's main kernel (zero == nullptr: nothing).
struct MaskBwdPrep {
    uint32_t* zero;
    size_t zero_words;
    RangesArgs ranges;
};
MaskBwdPrep mask_bwd_prep(const sparsek_cfg& c, const float* u, const float* tau, void* ws, int t_min,
                          const int32_t* first_valid);

// ---------------------------------------------------------------------------------
// Epilogue 1: per key j the range [a_j, b_j] of prefixes T with j in S*_T; difference array
// of |S*_T|.  tau is non-decreasing for T >= k-1, so both ends come from binary searches:
//   b_j = last  T in [max(j,k), n-1] with tau_T < u_j
//   a_j = first T in [max(j,k), n-1] with u_j < tau_T + 1      (compared in fp64, exact)
// A workgroup holds every stride-th threshold of its row in LDS (all of them up to n = 8192);
// a search runs on those samples first and finishes in global memory inside one stride.
// ---------------------------------------------------------------------------------
constexpr int RS_MAX = 8192;  // sampled thresholds per row held in LDS

// first T in [lo, n) with pred(tau_T), n if none; pred is monotone (false ... false true ... true)
template <typename Pred>
__device__ __forceinline__ int first_true(const float* __restrict__ tr, const float* ts, int lo, int n, int stride,
                                          int ns, Pred pred)
{
    const int ifirst = (lo + stride - 1) / stride;  // samples sit at T = i * stride
    int x = ifirst, y = ns;
    while (x < y) {
        const int m = (x + y) >> 1;
        if (pred(ts[m])) y = m;
        else x = m + 1;
    }
    int t0 = (x == ifirst) ? lo : (x - 1) * stride + 1;  // samples before x are false
    int t1 = (x < ns) ? x * stride : n;                  // sample x is true
    while (t0 < t1) {
        const int m = (t0 + t1) >> 1;
        if (pred(tr[m])) t1 = m;
        else t0 = m + 1;
    }
    return t0;
}

// Keys blk * blockDim.x .. of row `row`; ts: RS_MAX floats of LDS.
__device__ __forceinline__ void mask_bwd_ranges(const RangesArgs& A, float* ts, int blk, int row)
{
    const int n = A.n;
    // the first prefix that counts: more than k entries, and its threshold is there
    const int k = max(A.k + (A.first_valid ? A.first_valid[row] : 0), A.t_min);
    const float* tr = A.tau + (size_t)row * n;
    const int stride = (n + RS_MAX - 1) / RS_MAX;
    const int ns = (n + stride - 1) / stride;
    for (int i = threadIdx.x; i < ns; i += blockDim.x) ts[i] = tr[(size_t)i * stride];
    __syncthreads();
    const int j = blk * blockDim.x + threadIdx.x;
    int a = 1, b = 0;
    if (j < n) {
        const float uj = A.u[(size_t)row * n + j];
        const int lo = max(j, k);  // shorter prefixes have every gate at 1: S* empty
        if (lo <= n - 1) {
            b = first_true(tr, ts, lo, n, stride, ns, [&](float t) { return !(t < uj); }) - 1;
            a = first_true(tr, ts, lo, n, stride, ns, [&](float t) { return (double)uj < (double)t + 1.0; });
        }
        A.ab[(size_t)row * n + j] = make_int2(a, b);
    }
    // difference array: +1 at a_j, -1 at b_j + 1.  Two addresses collect most of the updates and
    // would serialise them: every key j <= k that is fractional from the start has a_j = k (one
    // add per wave instead), and every key still fractional at the end has b_j + 1 = n, an entry
    // the prefix sum never reads (dropped).
    const bool any = a <= b;
    int32_t* dr = A.diff + (size_t)row * (n + 1);
    const unsigned long long at_k = __ballot(any && a == k);
    if (any && a != k) atomicAdd(dr + a, 1);
    if (at_k != 0 && (threadIdx.x & 63) == 0) atomicAdd(dr + k, (int)__popcll(at_k));
    if (any && b + 1 < n) atomicAdd(dr + b + 1, -1);
}

}  // namespace spk
