// Importance scores of the key-value pairs (Sec. 3.2: scoring network with position slope;
// Sec. 3.5: score normalisation):
//     raw_t = x_t . w + t * slope                                  (t counted from 0)
//     u_t   = raw_t                                                (norm == 0)
//     u_t   = (raw_t - mean_t) / sqrt(var_t + norm_eps)            (norm == 1)
// with the running mean and population variance of raw_0 .. raw_t.
//
// scores_dot_kernel streams the hidden states once (the only traffic that matters: B*n*D elements
// against 4 bytes of output per position, roofline "hbm").  A wave owns 8 positions and walks the
// feature dimension with 16-byte loads; the scorer sits in LDS as fp64 and one read of it serves
// all 8 positions.  Products and sums are fp64 (exact products, the reduction is the only
// rounding), so the normalised scores stay accurate where early timesteps nearly cancel.
// The normalisation works on shifted scores z = raw - raw_0, which keeps E[z^2] - E[z]^2 free of
// cancellation whatever offset the scores carry.  A workgroup of the dot kernel does not know raw_0;
// it leaves the sums of its 32 positions relative to its own first score, and scores_norm_kernel
// moves them to raw_0 as it adds up what lies before its 256 positions, scans those and writes u.
// 32768 positions of 4096 bf16 features (268 MB): 67 -> 52.6 us with the normalisation; the dot kernel reads at 5.7 TB/s,
// 4.9 before.  What it took: waves that start at different features (69 -> 55 us for the whole call), loads that do not
// displace the caches (55 -> 52.6 us).  A second set of loads in flight per wave gave nothing.
#include "common.hpp"

namespace spk {

constexpr int SC_POS_PER_WAVE = 8;
constexpr int SC_POS_PER_BLOCK = 4 * SC_POS_PER_WAVE;
constexpr int SC_NORM_BLOCK = 256;

// 16 bytes of a hidden state as they lie in memory; they are used once.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Vec16 {
    static constexpr int N = 16 / sizeof(T);
    u32x4 r;
    __device__ __forceinline__ void load(const T* p) { r = __builtin_nontemporal_load((const u32x4*)p); }
    __device__ __forceinline__ float get(int i) const
    {
        if (sizeof(T) == 4) return __uint_as_float(r[i & 3]);
        return __uint_as_float(i & 1 ? r[i >> 1] & 0xFFFF0000u : r[i >> 1] << 16);
    }
};

// What a block's scores are shifted by: its first one, unless that is no number to compute with (an infinite score stays
// infinite in the sums then).
__device__ __forceinline__ double block_shift(double first) { return fabs(first) < INFINITY ? first : 0.0; }

// raw (and partial) are null when the scores are not normalised; partial[b][block] = (sum z, sum z^2) over the block's
// positions, z = raw - block_shift.
template <typename T>
__global__ __launch_bounds__(256, 4) void scores_dot_kernel(const T* __restrict__ x, const float* __restrict__ w,
                                                            int n, int D, double slope, double* __restrict__ raw,
                                                            double2* __restrict__ partial, float* __restrict__ u_out)
{
    // the scorer, widened once; element c sits at [c % E][c / E] so that the lanes of a wave,
    // which own consecutive groups of E features, read consecutive doubles (no bank conflicts)
    constexpr int P = SC_POS_PER_WAVE, E = Vec16<T>::N;
    extern __shared__ double wd[];   // max(D, SC_POS_PER_BLOCK)
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int DE = D / E, c_first = E * lane;
    const int start = blockIdx.x * SC_POS_PER_BLOCK, t0 = start + wv * P;
    const T* rows[P];
#pragma unroll
    for (int p = 0; p < P; p++) rows[p] = x + ((size_t)b * n + min(t0 + p, n - 1)) * D;
    Vec16<T> v[P];
    // The waves of the grid start at different features: rows are often a multiple of 4 KB, and waves that walk them side
    // by side would ask the same few memory channels at a time.
    const int steps = (D + 64 * E - 1) / (64 * E), rot = (4 * blockIdx.x + wv) % steps;
    auto column = [&](int i) { return 64 * E * (i + rot < steps ? i + rot : i + rot - steps) + c_first; };
    auto fetch = [&](int i) {   // (lanes beyond the last feature load that again)
        const unsigned at = min(column(i), D - E);
#pragma unroll
        for (int p = 0; p < P; p++) v[p].load(rows[p] + at);
    };
    fetch(0);   // ahead of the scorer
    for (int c = tid; c < D; c += 256) wd[(c % E) * DE + c / E] = (double)w[c];
    __syncthreads();
    double acc[P];
#pragma unroll
    for (int p = 0; p < P; p++) acc[p] = 0.0;
    auto add = [&](int i) {
        const int c = column(i);
        if (c < D) {
#pragma unroll
            for (int e = 0; e < E; e++) {
                const double we = wd[e * DE + c / E];
#pragma unroll
                for (int p = 0; p < P; p++) acc[p] = fma((double)v[p].get(e), we, acc[p]);
            }
        }
    };
    add(0);
#pragma unroll 1
    for (int i = 1; i < steps; i++) {
        fetch(i);
        add(i);
    }
    __syncthreads();
    double* rl = wd;   // the raw scores of the workgroup's positions
#pragma unroll
    for (int p = 0; p < P; p++) {
        const double s = wave_sum_f64(acc[p]);
        if (lane == 0) rl[wv * P + p] = s + (double)(t0 + p) * slope;
    }
    __syncthreads();
    if (wv > 0) return;
    const int t = start + lane;
    const bool in = lane < SC_POS_PER_BLOCK && t < n;
    const double r = in ? rl[lane] : 0.0;
    if (!raw) {
        if (in) u_out[(size_t)b * n + t] = (float)r;
        return;
    }
    if (in) raw[(size_t)b * n + t] = r;
    const double z = in ? r - block_shift(rl[0]) : 0.0;
    const double s1 = wave_sum_f64(z), s2 = wave_sum_f64(z * z);
    if (lane == 0) partial[(size_t)b * gridDim.x + blockIdx.x] = make_double2(s1, s2);
}

// Inclusive prefix sums of (a, b) over the 256 threads of a workgroup, in place; tot = block totals.
__device__ __forceinline__ void block_inclusive_scan2_256(double& a, double& b, double (*wt)[4] /* [2][4] LDS */,
                                                          double& tot_a, double& tot_b)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double ya = __shfl_up(a, o, 64), yb = __shfl_up(b, o, 64);
        if (lane >= o) { a += ya; b += yb; }
    }
    if (lane == 63) { wt[0][wv] = a; wt[1][wv] = b; }
    __syncthreads();
    tot_a = 0.0; tot_b = 0.0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (i < wv) { a += wt[0][i]; b += wt[1][i]; }
        tot_a += wt[0][i]; tot_b += wt[1][i];
    }
}

__global__ __launch_bounds__(SC_NORM_BLOCK) void scores_norm_kernel(const double* __restrict__ raw,
                                                                     const double2* __restrict__ partial, int npart, int n,
                                                                     double norm_eps, float* __restrict__ u)
{
    __shared__ double red[2][4];
    __shared__ double wt[2][4];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const double* r = raw + (size_t)b * n;
    const int start = blockIdx.x * SC_NORM_BLOCK;
    const double shift = r[0];
    // everything before this workgroup's positions
    double s1 = 0.0, s2 = 0.0;
    for (int i = tid; i < start / SC_POS_PER_BLOCK; i += SC_NORM_BLOCK) {
        const double2 p = partial[(size_t)b * npart + i];
        const double d = block_shift(r[i * SC_POS_PER_BLOCK]) - shift;
        s1 += p.x + SC_POS_PER_BLOCK * d;
        s2 += p.y + d * (2.0 * p.x + SC_POS_PER_BLOCK * d);
    }
    s1 = wave_sum_f64(s1);
    s2 = wave_sum_f64(s2);
    if (lane == 0) { red[0][wv] = s1; red[1][wv] = s2; }
    __syncthreads();
    const double before1 = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    const double before2 = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    const int t = start + tid;
    const double z = t < n ? r[t] - shift : 0.0;
    double c1 = z, c2 = z * z, tot1, tot2;
    block_inclusive_scan2_256(c1, c2, wt, tot1, tot2);
    if (t < n) {
        const double cnt = (double)(t + 1);
        const double mean = (before1 + c1) / cnt;
        const double var = fmax((before2 + c2) / cnt - mean * mean, 0.0);
        u[(size_t)b * n + t] = (float)((z - mean) / sqrt(var + norm_eps));
    }
}

static size_t scores_raw_bytes(int B, int n) { return align_up((size_t)B * n * sizeof(double), 256); }
static int scores_blocks(int n) { return (n + SC_POS_PER_BLOCK - 1) / SC_POS_PER_BLOCK; }
size_t scores_ws_bytes(int B, int n)
{
    return scores_raw_bytes(B, n) + align_up((size_t)B * scores_blocks(n) * sizeof(double2), 256);
}

int launch_scores(int B, int n, int D, int dtype, int norm, double slope, double norm_eps, const void* x,
                  const float* w, float* u, void* ws, hipStream_t st)
{
    double* raw = norm ? (double*)ws : nullptr;
    double2* partial = norm ? (double2*)((char*)ws + scores_raw_bytes(B, n)) : nullptr;
    dim3 grid(scores_blocks(n), B);
    const size_t lds = (size_t)std::max(D, SC_POS_PER_BLOCK) * sizeof(double);
    if (dtype == SPARSEK_BF16)
        hipLaunchKernelGGL(scores_dot_kernel<uint16_t>, grid, dim3(256), lds, st, (const uint16_t*)x, w, n, D, slope, raw,
                           partial, u);
    else
        hipLaunchKernelGGL(scores_dot_kernel<float>, grid, dim3(256), lds, st, (const float*)x, w, n, D, slope, raw,
                           partial, u);
    if (norm) {
        dim3 g2((n + SC_NORM_BLOCK - 1) / SC_NORM_BLOCK, B);
        hipLaunchKernelGGL(scores_norm_kernel, g2, dim3(SC_NORM_BLOCK), 0, st, raw, partial, scores_blocks(n), n, norm_eps,
                           u);
    }
    return launch_status();
}

}  // namespace spk
