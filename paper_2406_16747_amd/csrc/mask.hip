// Stages 1+2: SPARSEK thresholds tau_t for every causal prefix and per-key lifetimes.
//
// The paper evaluates the prefixes one after another with two heaps on the CPU (Sec. 3.3, incremental
// algorithm; App. B.3).  Here the sequence is cut into chunks of up to CHUNK prefixes that are solved
// independently, one workgroup each, in one launch (mask_kernel):
//   * tau_t and the k-th largest selection key never decrease once the prefix holds k entries (Sec. 3.2,
//     irreversibility), so inside a chunk only the scores between two bounds can change anything.
//     Both bounds come from one histogram of the prefix: f_t(x) = sum clip(z - x, 0, 1) is the integral
//     over [x, x + 1] of #{z > y}, so windowed sums of the bin counts bound f_t at every bin edge --
//     in integers, without a search.  A second pass adds up the scores that are saturated or fractional
//     whatever the threshold does inside the bounds and collects the few others (about 120 of 32768
//     scores of unit variance at k = 1024);
//   * every wave then solves a few consecutive prefixes: tau_t is the root of f_t(x) = k, on the linear piece between
//     the last breakpoint with f_t >= k and the next (solve_parallel); with too many breakpoints for that, by repeating
//     the closed form of the solution equation (tau from u*, w* and the fractional sum) until no breakpoint lies between
//     two iterates -- exact, not an iteration to a tolerance; a bracket guards it;
//   * key j dies at the first prefix that holds k larger keys: with c older keys above it, at the
//     (k - c)-th newcomer of the chunk that is larger -- a rank and a sum over 16 lanes per key.
// The histogram's window follows the scores, in position and in the width of its bins (next_window).  Chunks that no
// window suits (many equal scores around the threshold, thresholds of -inf, first thresholds spread over more than 2000)
// take the sorted path: the candidates above a lower bound are compacted into LDS, sorted once, and the same iteration
// runs on searches in the sorted list.
#include "common.hpp"

namespace spk {

constexpr int CHUNK = 128;        // prefixes per workgroup of the chunk kernel, at most
constexpr int NT_CHUNK = 1024;    // threads per workgroup (16 waves, up to 8 prefixes each)
constexpr int NW_CHUNK = NT_CHUNK / 64;
constexpr int CAP = 8192;         // sorted path: candidate capacity in LDS (64 KB of 64-bit keys, 8 KB of prefix sums)
constexpr int MAX_ITERS = 4096;
constexpr size_t STATUS_WORDS = 2048;   // up to this many chunks, each has a status word of its own

// Where a chunk reports that a threshold solve hit its iteration cap: a bit of a word.
struct Status {
    int* word;
    int bit;
};

static size_t mask_chunks(const sparsek_cfg& c) { return (size_t)c.B * c.Gu * (((size_t)c.n + CHUNK - 1) / CHUNK); }
static bool mask_shared_status(const sparsek_cfg& c) { return mask_chunks(c) > STATUS_WORDS; }

// The kernels need the status words alone (see mask_kernel): one for all chunks, or one each up to STATUS_WORDS chunks.
// The size asked for is never less than one bit per chunk and 4 bytes per 2048 positions of every row: earlier versions of
// the library used those, and what fits sparsek_mask_static, and what does not, stays the same.
size_t mask_ws_bytes(const sparsek_cfg& c)
{
    const size_t rows = (size_t)c.B * c.Gu, chunks = mask_chunks(c);
    const size_t bytes = align_up(rows * (((size_t)c.n + 2047) / 2048) * sizeof(float), 256) + 256 +
                         align_up((chunks + 31) / 32 * 4, 256);
    return mask_shared_status(c) ? bytes : std::max(bytes, align_up(chunks * sizeof(int), 256));
}

// ---------------------------------------------------------------------------------
// Candidate lists: compacted in LDS, or (overflow fallback) the raw prefix in global memory.
// ---------------------------------------------------------------------------------
// Sorted list: key[0, m_old) = selection keys (score, then older position) of the older
// candidates in descending order, pref[i] = sum of the scores of key[0, PSTRIDE * i) in fp64; the chunk's
// own scores live in registers, two per lane (entries `lane` and `lane + 64` of the chunk).
constexpr int PSTRIDE = 8;
struct ListSorted {
    const unsigned long long* key;
    const double* pref;
    int m_old, t0;
    float nv0, nv1;  // this lane's chunk scores (-inf beyond the chunk)
};
__device__ __forceinline__ float key_score(unsigned long long key)
{
    return __uint_as_float(score_key_inv((uint32_t)(key >> 32)));
}
__device__ __forceinline__ int key_pos(unsigned long long key) { return (int)(0xFFFFFFFFu - (uint32_t)key); }
struct ListGlobal {
    const float* u;
    int M;
    __device__ __forceinline__ float val(int i) const { return u[i]; }
    __device__ __forceinline__ int pos(int i) const { return i; }
};

// Right-limit counts of the piece of f_t that starts at x: F = #{z > x+1}, S = #{z > x},
// fsum = sum of the z in (x, x+1], minF = min{z > x+1}; over list entries at positions <= t.
template <class List>
__device__ __forceinline__ void eval_piece(const List& L, int t, double x, int lane, int& F, int& S,
                                           double& fsum, float& minF)
{
    int f = 0, s = 0;
    double sum = 0.0;
    float mf = INFINITY;
    const double x1 = x + 1.0;
    for (int i = lane; i < L.M; i += 64) {
        float v = L.val(i);
        if (L.pos(i) <= t) {
            double dv = (double)v;
            if (dv > x) {
                s++;
                if (dv > x1) { f++; mf = fminf(mf, v); }
                else sum += dv;
            }
        }
    }
    unsigned long long packed = wave_sum_u64(((unsigned long long)f << 32) | (unsigned long long)s);
    F = (int)(packed >> 32);
    S = (int)(packed & 0xFFFFFFFFull);
    fsum = wave_sum_f64(sum);
    minF = wave_min_f32(mf);
}

// The linear piece of f_t that contains x (right-limit counts), for the sorted list.
struct Piece {
    int F, S, a;      // a = older scores above x + 1
    double fsum;
    double next_old;  // smallest breakpoint of the older scores above x (+inf if none)
    double prev_old;  // largest breakpoint of the older scores at or below x (-inf if none)
};

// The fp64 thresholds are replaced by their round-down fp32 values: for an fp32 score v,
// v > x  <=>  v > rd(x).  The counts over the older scores are the results of two searches
// (32 probes a round; lanes 0..31 search x, lanes 32..63 search x + 1), their fractional sum is a
// difference of prefix sums, or a direct sum when at most 64 scores are fractional: a sum with a
// single fractional score has to stay exact, which the flat case (root exactly on a breakpoint,
// sup rule) relies on.  The chunk's own scores are added from registers.
__device__ __forceinline__ Piece eval_sorted(const ListSorted& L, int t, double x, int lane)
{
    const float xf = __double2float_rd(x), x1f = __double2float_rd(x + 1.0);
    const int hf = lane >> 5, l32 = lane & 31;
    const float thr = hf ? x1f : xf;
    int lo = 0, hi = L.m_old;  // the count lies in [lo, hi]: key[<lo] are above thr, key[>=hi] are not
    while (__any(lo < hi)) {
        const int stride = (hi - lo + 31) >> 5;
        const int p = lo + l32 * stride;
        const bool above = (p < hi) && (key_score(L.key[p]) > thr);
        const unsigned long long ball = __ballot(above);
        const int c = __popc(hf ? (unsigned)(ball >> 32) : (unsigned)ball);
        if (lo < hi) {
            if (c == 0) hi = lo;
            else {
                hi = min(hi, lo + c * stride);
                lo = lo + (c - 1) * stride + 1;
            }
        }
    }
    const int b = __builtin_amdgcn_readlane(lo, 0);   // older scores above x
    const int a = __builtin_amdgcn_readlane(lo, 32);  // older scores above x + 1
    Piece P;
    P.a = a;
    // neighbouring breakpoints of the older scores (uniform addresses: broadcast reads)
    P.next_old = INFINITY;
    P.prev_old = -INFINITY;
    if (b > 0) P.next_old = (double)key_score(L.key[b - 1]);
    if (a > 0) P.next_old = fmin(P.next_old, (double)key_score(L.key[a - 1]) - 1.0);
    if (b < L.m_old) P.prev_old = (double)key_score(L.key[b]);
    if (a < L.m_old) P.prev_old = fmax(P.prev_old, (double)key_score(L.key[a]) - 1.0);
    // the chunk's own scores inside prefix t
    const int nc = t - L.t0 + 1;
    const float v0 = (lane < nc) ? L.nv0 : -INFINITY, v1 = (lane + 64 < nc) ? L.nv1 : -INFINITY;
    const bool a0 = v0 > xf, b0 = v0 > x1f, a1 = v1 > xf, b1 = v1 > x1f;
    const int f = (b0 ? 1 : 0) + (b1 ? 1 : 0), sc = (a0 ? 1 : 0) + (a1 ? 1 : 0);
    double part = (double)((a0 && !b0) ? v0 : 0.0f) + (double)((a1 && !b1) ? v1 : 0.0f);
    double base = 0.0;
    if (b - a <= 64) {
        if (lane < b - a) part += (double)key_score(L.key[a + lane]);
    } else {
        base = L.pref[b / PSTRIDE] - L.pref[a / PSTRIDE];   // in whole strides, corrected at both ends
        if (lane < b % PSTRIDE) part += (double)key_score(L.key[b / PSTRIDE * PSTRIDE + lane]);
        if (lane < a % PSTRIDE) part -= (double)key_score(L.key[a / PSTRIDE * PSTRIDE + lane]);
    }
    const unsigned long long packed = wave_sum_u64(((unsigned long long)f << 32) | (unsigned long long)sc);
    P.F = a + (int)(packed >> 32);
    P.S = b + (int)(packed & 0xFFFFFFFFull);
    P.fsum = base + wave_sum_f64(part);
    return P;
}

// Smallest score above x + 1 in prefix t (the flat case needs it).
__device__ __forceinline__ float min_saturated(const ListSorted& L, int t, double x, int a, int lane)
{
    const float x1f = __double2float_rd(x + 1.0);
    const int nc = t - L.t0 + 1;
    const float v0 = (lane < nc) ? L.nv0 : -INFINITY, v1 = (lane + 64 < nc) ? L.nv1 : -INFINITY;
    float mf = fminf(v0 > x1f ? v0 : INFINITY, v1 > x1f ? v1 : INFINITY);
    if (a > 0) mf = fminf(mf, key_score(L.key[a - 1]));
    return wave_min_f32(mf);
}

// True if none of the chunk's own scores inside prefix t has a breakpoint (z or z - 1) in (lo, hi].
__device__ __forceinline__ bool own_piece_clear(const ListSorted& L, int t, double lo, double hi, int lane)
{
    const int nc = t - L.t0 + 1;
    const double v0 = (double)L.nv0, v1 = (double)L.nv1;
    const bool h0 = (lane < nc) && ((v0 > lo && v0 <= hi) || (v0 - 1.0 > lo && v0 - 1.0 <= hi));
    const bool h1 = (lane + 64 < nc) && ((v1 > lo && v1 <= hi) || (v1 - 1.0 > lo && v1 - 1.0 <= hi));
    return __ballot(h0 || h1) == 0ull;
}

// tau of prefix t (t+1 > k >= 1) starting from a point `start` with f_t(start) >= k.
// Repeats tau <- (fsum + F - k)/(S - F) (solution equation of Sec. 3.3 with u* = F, w* = S)
// until (F, S) at the new point equal those it was computed from; then that point is the
// exact root of its linear piece.  The step is the root of the linear piece through the current
// point, taken from whichever side of the root the point lies on (f_t is neither convex nor
// concave, so a one-sided iteration would creep); a bracket [lo_b, hi_b) of the root is kept and
// a step that leaves it is replaced by its midpoint.
template <class List>
__device__ double solve_tau(const List& L, int t, int k, double start, int lane, Status status)
{
    double lo_b = start, hi_b = INFINITY, x = start;
    int pF = -1, pS = -1;
    for (int it = 0; it < MAX_ITERS; it++) {
        int F, S;
        double fsum;
        float minF;
        eval_piece(L, t, x, lane, F, S, fsum, minF);
        if (F == pF && S == pS) return x;
        pF = pS = -1;
        const double f = (double)F + fsum - (double)(S - F) * x;
        double xn;
        bool have = false;
        if (f < (double)k) {
            hi_b = x;  // x is right of the root
            if (S > F) { xn = (fsum + (double)F - (double)k) / (double)(S - F); have = true; }
        } else {
            lo_b = x;
            if (S == F) {  // flat to the right of x, f == F there
                if (F == k || (F > k && minF == INFINITY)) return (double)minF - 1.0;  // sup of the level set; k or more of +inf
                xn = (double)minF - 1.0;                 // F > k: the next breakpoint, still left of the root
                if (xn < hi_b) { x = xn; continue; }
            } else {
                xn = (fsum + (double)F - (double)k) / (double)(S - F);
                if (!(xn > x)) return x;  // f(x) == k up to rounding
                have = true;
            }
        }
        if (have && xn > lo_b && xn < hi_b) {
            pF = F;
            pS = S;
            x = xn;
        } else {
            const double mid = 0.5 * (lo_b + hi_b);
            if (!(mid > lo_b && mid < hi_b)) return lo_b;
            x = mid;
        }
    }
    if (lane == 0) atomicOr(status.word, status.bit);
    return x;
}

// k-th largest selection key among list entries at positions < tlim (at least k of them exist;
// returns 0 otherwise).  Whole workgroup, MSB-first radix select, 8 bits a round, one 256-bin
// LDS histogram; every thread returns the same key.
template <class List>
__device__ unsigned long long block_kth_largest(const List& L, int tlim, int k, unsigned* hist, unsigned long long* bc)
{
    const int tid = threadIdx.x, lane = tid & 63;
    unsigned long long prefix = 0;  // decided high bits
    int r = k;                      // rank wanted among the entries matching the prefix
    for (int round = 0; round < 8; round++) {
        const int shift = 56 - 8 * round;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int i = tid; i < L.M; i += NT_CHUNK) {
            const int p = L.pos(i);
            if (p < tlim) {
                const unsigned long long key = sel_key(L.val(i), p);
                const bool match = (round == 0) || ((key >> (shift + 8)) == (prefix >> (shift + 8)));
                if (match) atomicAdd(&hist[(unsigned)(key >> shift) & 255u], 1u);
            }
        }
        __syncthreads();
        if (tid < 64) {  // wave 0: lane l owns bins 4l..4l+3; suffix sums from the top bin down
            const unsigned h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
            const unsigned lsum = h0 + h1 + h2 + h3;
            unsigned suf = lsum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned y = __shfl_down(suf, o, 64);
                if (lane + o < 64) suf += y;
            }
            const unsigned long long ball = __ballot(suf >= (unsigned)r);
            unsigned long long res = 0;  // digit | count << 16 | above << 32 ; 0xFFFF... = not enough entries
            if (ball == 0) res = ~0ull;
            else {
                const int ls = 63 - __builtin_clzll(ball);
                unsigned above = __shfl(suf - lsum, ls, 64);
                const unsigned b3 = __shfl(h3, ls, 64), b2 = __shfl(h2, ls, 64), b1 = __shfl(h1, ls, 64),
                               b0 = __shfl(h0, ls, 64);
                unsigned digit, cnt;
                if (above + b3 >= (unsigned)r) { digit = 4 * ls + 3; cnt = b3; }
                else if (above + b3 + b2 >= (unsigned)r) { digit = 4 * ls + 2; above += b3; cnt = b2; }
                else if (above + b3 + b2 + b1 >= (unsigned)r) { digit = 4 * ls + 1; above += b3 + b2; cnt = b1; }
                else { digit = 4 * ls; above += b3 + b2 + b1; cnt = b0; }
                res = (unsigned long long)digit | ((unsigned long long)min(cnt, 0xFFFFu) << 16) | ((unsigned long long)above << 32);
            }
            if (lane == 0) *bc = res;
        }
        __syncthreads();
        const unsigned long long res = *bc;
        if (res == ~0ull) return 0;
        r -= (int)(res >> 32);
        prefix |= (res & 0xFFull) << shift;
        if (((res >> 16) & 0xFFFFull) == 1 && shift > 0) {  // a single entry carries this prefix: fetch it
            __syncthreads();
            if (tid == 0) *bc = 0;
            __syncthreads();
            for (int i = tid; i < L.M; i += NT_CHUNK) {
                const int p = L.pos(i);
                if (p < tlim) {
                    const unsigned long long key = sel_key(L.val(i), p);
                    if ((key >> shift) == (prefix >> shift)) *bc = key;  // exactly one writer
                }
            }
            __syncthreads();
            return *bc;
        }
        __syncthreads();
    }
    return prefix;
}

// Smallest key strictly above `theta` among entries at positions < tlim (all-ones if none).
template <class List>
__device__ __forceinline__ unsigned long long succ_key(const List& L, int tlim, unsigned long long theta,
                                                        int lane)
{
    unsigned long long best = ~0ull;
    for (int i = lane; i < L.M; i += 64) {
        int p = L.pos(i);
        if (p < tlim) {
            unsigned long long key = sel_key(L.val(i), p);
            if (key > theta && key < best) best = key;
        }
    }
    return wave_min_u64(best);
}
template <class List>
__device__ __forceinline__ unsigned long long min_key(const List& L, int tlim, int lane)
{
    unsigned long long best = ~0ull;
    for (int i = lane; i < L.M; i += 64) {
        int p = L.pos(i);
        if (p < tlim) {
            unsigned long long key = sel_key(L.val(i), p);
            if (key < best) best = key;
        }
    }
    return wave_min_u64(best);
}

// Smallest score of prefix t.
template <class List>
__device__ __forceinline__ float prefix_min(const List& L, int t, int lane)
{
    float m2 = INFINITY;
    for (int i = lane; i < L.M; i += 64)
        if (L.pos(i) <= t) m2 = fminf(m2, L.val(i));
    return wave_min_f32(m2);
}
__device__ __forceinline__ float prefix_min(const ListSorted& L, int t, int lane)
{
    const int nc = t - L.t0 + 1;
    float m2 = fminf((lane < nc) ? L.nv0 : INFINITY, (lane + 64 < nc) ? L.nv1 : INFINITY);
    if (L.m_old > 0) m2 = fminf(m2, key_score(L.key[L.m_old - 1]));
    return wave_min_f32(m2);
}

// One wave, thresholds of prefixes [ta, tb) (those longer than k).
template <class List>
__device__ void wave_tau(const List& L, const float* __restrict__ ur, float* __restrict__ tr, int ta, int tb,
                         int k, float start0, int lane, Status status)
{
    const float my_u = (ta + lane < tb) ? ur[ta + lane] : 0.0f;  // tb - ta <= 64
    bool have_prev = false;
    double tau_prev = 0.0;
    for (int t = ta; t < tb; t++) {
        if (t + 1 <= k) continue;  // at most k entries: written by short_prefix_tau
        const double ut = (double)readlane_f32(my_u, t - ta);
        double tau;
        if (have_prev && !(ut > tau_prev)) {
            tau = tau_prev;  // the new score is below the threshold: nothing changes
        } else {
            double start;
            if (have_prev) start = tau_prev;
            else if (start0 > -INFINITY) start = (double)start0;
            else {  // no bound known: min(prefix) - 1 has f = t+1 >= k
                start = (double)prefix_min(L, t, lane) - 1.0;
            }
            tau = solve_tau(L, t, k, start, lane, status);
        }
        tau_prev = tau;
        have_prev = true;
        if (lane == 0) tr[t] = (float)tau;
    }
}

// The same for the sorted list, with the linear piece carried from prefix to prefix: a new score
// above the threshold changes the counts of the current piece by one, the root of that piece is
// the closed form, and it is final if no breakpoint lies between the old and the new threshold
// (the sorted neighbours and one ballot over the chunk's own scores tell).  Only otherwise the
// piece is evaluated again (eval_sorted), with the two-sided iteration of solve_tau.
__device__ void wave_tau(const ListSorted& L, const float* __restrict__ ur, float* __restrict__ tr, int ta,
                         int tb, int k, float start0, int lane, Status status)
{
    const float my_u = (ta + lane < tb) ? ur[ta + lane] : 0.0f;  // tb - ta <= 64
    bool started = false;  // x = tau of the previous prefix
    bool have = false;     // and P describes the piece of that prefix's f at x
    double x = 0.0;
    Piece P;
    for (int t = ta; t < tb; t++) {
        if (t + 1 <= k) continue;  // at most k entries: written by short_prefix_tau
        const float utf = readlane_f32(my_u, t - ta);
        const double ut = (double)utf;
        if (started && !(ut > x)) {  // the new score is below the threshold: nothing changes
            if (lane == 0) tr[t] = (float)x;
            continue;
        }
        if (have) {
            if (ut > x + 1.0) { P.F++; P.S++; }
            else { P.S++; P.fsum += ut; }
        } else {
            if (!started) {
                if (start0 > -INFINITY) x = (double)start0;
                else x = (double)prefix_min(L, t, lane) - 1.0;  // no bound known: f = t+1 >= k there
            }
            P = eval_sorted(L, t, x, lane);  // tau only rises: f_t(x) >= k at the previous tau too
            have = true;
        }
        started = true;
        // two-sided iteration on f_t from the piece P at x
        double lo_b = x, hi_b = INFINITY;
        int it = 0;
        for (; it < MAX_ITERS; it++) {
            const double f = (double)P.F + P.fsum - (double)(P.S - P.F) * x;
            double xn = 0.0;
            bool step = false;
            if (f < (double)k) {
                hi_b = x;
                if (P.S > P.F) {
                    xn = (P.fsum + (double)P.F - (double)k) / (double)(P.S - P.F);
                    // still inside the piece (it starts at the largest breakpoint <= x): exact root
                    if (xn < x && xn >= P.prev_old && own_piece_clear(L, t, xn, x, lane)) { x = xn; break; }
                    step = xn > lo_b && xn < hi_b;
                }
            } else {
                lo_b = x;
                if (P.S == P.F) {  // flat to the right of x, f == F there
                    const double nb = (double)min_saturated(L, t, x, P.a, lane) - 1.0;  // next breakpoint
                    if (P.F == k || (P.F > k && nb == INFINITY)) {  // sup of the level set, where the piece changes; k or more of +inf
                        x = nb;
                        have = false;
                        break;
                    }
                    xn = nb;  // F > k: still left of the root
                    step = xn < hi_b;
                } else {
                    xn = (P.fsum + (double)P.F - (double)k) / (double)(P.S - P.F);
                    if (!(xn > x)) break;  // f(x) == k up to rounding
                    if (xn < P.next_old && own_piece_clear(L, t, x, xn, lane)) { x = xn; break; }
                    step = xn < hi_b;
                }
            }
            if (!step) {
                const double mid = 0.5 * (lo_b + hi_b);
                if (!(mid > lo_b && mid < hi_b)) { x = lo_b; have = false; break; }
                xn = mid;
            }
            x = xn;
            P = eval_sorted(L, t, x, lane);
        }
        if (it == MAX_ITERS && lane == 0) atomicOr(status.word, status.bit);
        if (lane == 0) tr[t] = (float)x;
    }
}

// One wave, the whole chunk: theta_t = k-th largest selection key of prefix t (0 while the
// prefix is shorter than k), by "newcomer in, smallest out" starting from theta_{t0-1}.
template <class List>
__device__ void wave_theta(const List& L, const float* __restrict__ ur, int t0, int t1, int k,
                           unsigned long long theta, int lane, unsigned long long* th)
{
    for (int tb = t0; tb < t1; tb += 64) {
        const float my_u = (tb + lane < t1) ? ur[tb + lane] : 0.0f;
        for (int t = tb; t < min(t1, tb + 64); t++) {
            const int len = t + 1;
            if (len == k) {
                theta = min_key(L, t + 1, lane);
            } else if (len > k) {
                const unsigned long long e = sel_key(readlane_f32(my_u, t - tb), t);
                if (e > theta) {
                    const unsigned long long sc = succ_key(L, t, theta, lane);
                    theta = e < sc ? e : sc;
                }
            }
            if (lane == 0) th[t - t0] = theta;
        }
    }
}

// The same walk on the sorted list: `na` older keys lie above theta, so the next older key above
// theta is key[na - 1]; the chunk's own keys are compared in registers.  This walk is the one
// sequential dependency of a chunk, so it is kept short: in a chunk whose prefixes all hold more
// than k entries only the newcomers above the starting theta are visited (the others can never
// enter the top-k: theta only rises), the next two older keys are held in registers, and the
// steps in between are filled in afterwards with a prefix maximum.
__device__ void wave_theta(const ListSorted& L, const float* __restrict__ ur, int t0, int t1, int k,
                           unsigned long long theta, int lane, unsigned long long* th)
{
    const unsigned long long k0 = sel_key(L.nv0, t0 + lane), k1 = sel_key(L.nv1, t0 + lane + 64);
    if (t0 >= k) {
        __builtin_amdgcn_s_setprio(3);  // the other waves of the workgroup wait for this one
        const unsigned long long th_start = theta;
        int na = k - 1;  // theta = key[k - 1]
        unsigned long long so0 = na > 0 ? L.key[na - 1] : ~0ull, so1 = na > 1 ? L.key[na - 2] : ~0ull;
        th[lane] = 0ull;
        th[lane + 64] = 0ull;
        const int cn = t1 - t0;
        unsigned long long m[2] = {__ballot(lane < cn && k0 > th_start), __ballot(lane + 64 < cn && k1 > th_start)};
        for (int h = 0; h < 2; h++) {
            unsigned long long todo = m[h];
            while (todo) {
                const int cl = __builtin_ctzll(todo);
                todo &= todo - 1;
                const int c = 64 * h + cl;  // chunk entries 0..c-1 are inside the prefix, entry c is the newcomer
                const unsigned long long e = h ? readlane_u64(k1, cl) : readlane_u64(k0, cl);
                if (e > theta) {
                    unsigned long long sc = ~0ull;
                    if (lane < c && k0 > theta) sc = k0;
                    if (lane + 64 < c && k1 > theta && k1 < sc) sc = k1;
                    sc = wave_min_u64(sc);
                    unsigned long long nt = e < sc ? e : sc;
                    if (so0 < nt) {
                        nt = so0;
                        na--;
                        so0 = so1;
                        so1 = na > 1 ? L.key[na - 2] : ~0ull;
                    }
                    theta = nt;
                    if (lane == 0) th[c] = theta;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (lane 0 wrote some of them)
        // th[i] = max(th_start, th[0..i]): inclusive prefix maximum over the 128 entries
        unsigned long long a = th[lane], b = th[lane + 64];
        a = a > th_start ? a : th_start;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(a, o, 64);
            if (lane >= o && y > a) a = y;
        }
        const unsigned long long top = readlane_u64(a, 63);
        b = b > top ? b : top;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(b, o, 64);
            if (lane >= o && y > b) b = y;
        }
        th[lane] = a;
        th[lane + 64] = b;
        __builtin_amdgcn_s_setprio(0);
        return;
    }
    int na = 0;
    for (int t = t0; t < t1; t++) {
        const int len = t + 1, c = t - t0;  // chunk entries 0..c-1 are inside prefix t-1, entry c is the newcomer
        if (len == k) {
            // every entry of the prefix is selected: theta is the smallest key
            unsigned long long m = ~0ull;
            if (lane <= c) m = k0;
            if (lane + 64 <= c) m = k1 < m ? k1 : m;
            m = wave_min_u64(m);
            if (L.m_old > 0) m = L.key[L.m_old - 1] < m ? L.key[L.m_old - 1] : m;
            theta = m;
            na = L.m_old;
            // older keys above theta: all but the one that equals it, if that one is the minimum
            if (L.m_old > 0 && L.key[L.m_old - 1] == theta) na = L.m_old - 1;
        } else if (len > k) {
            const unsigned long long e = (c < 64) ? readlane_u64(k0, c) : readlane_u64(k1, c - 64);
            if (e > theta) {
                unsigned long long sc = ~0ull;
                if (lane < c && k0 > theta) sc = k0;
                if (lane + 64 < c && k1 > theta && k1 < sc) sc = k1;
                sc = wave_min_u64(sc);
                const unsigned long long so = (na > 0) ? L.key[na - 1] : ~0ull;
                unsigned long long nt = e < sc ? e : sc;
                if (so < nt) { nt = so; na--; }
                theta = nt;
            }
        }
        if (lane == 0) th[t - t0] = theta;
    }
}

// death of one list entry given the chunk's theta sequence (non-decreasing).  Positions count from the row's first
// valid key, lifetimes from the row's start (j0 = the difference); survivor != 0: the lifetime of a key that outlives
// the chunk (written by the row's last chunk).
__device__ __forceinline__ void write_death(unsigned long long key, int j, int t0, int t1, int k,
                                            const unsigned long long* th, unsigned long long th_start,
                                            int32_t* __restrict__ dr, int j0, int survivor)
{
    int first;
    if ((unsigned)j >= (unsigned)t1) return;   // (a key is a position of the chunk's prefix)
    if (j < t0) {
        if (t0 >= k && key < th_start) return;  // already out before this chunk
        first = t0;
    } else {
        first = j;
    }
    // first t in [first, t1) with th[t - t0] > key
    int a = first - t0, b = t1 - t0;  // answer in [a, b]
    while (a < b) {
        int m = (a + b) >> 1;
        if (th[m] > key) b = m;
        else a = m + 1;
    }
    if (a < t1 - t0) dr[j] = j0 + t0 + a;
    else if (survivor) dr[j] = survivor;
}

constexpr int NW_TAU = NW_CHUNK - 1;                     // waves solving tau; the last wave walks theta
constexpr int TPW_TAU = (CHUNK + NW_TAU - 1) / NW_TAU;   // prefixes per tau wave
constexpr int SLICE_REG = 8;                             // compaction: scores cached per lane and segment

template <class List>
__device__ void chunk_body(const List& L, const float* __restrict__ ur, float* __restrict__ tr,
                           int32_t* __restrict__ dr, int t0, int t1, int k, float lo, unsigned* hist,
                           unsigned long long* bc, unsigned long long* th, Status status, int j0, int survivor)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // theta at the chunk start, by the whole workgroup
    unsigned long long th_start = 0;
    if (t0 >= k) th_start = block_kth_largest(L, t0, k, hist, bc);
    // tau lies in [z_(k) - 1, z_(k)), and both ends only rise: theta_{t0-1} - 1 bounds every tau of the chunk
    float start0 = lo;
    if (t0 >= k) start0 = fmaxf(lo, __uint_as_float(score_key_inv((uint32_t)(th_start >> 32))) - 1.0f);
    if (wv < NW_TAU) {
        const int ta = min(t1, t0 + wv * TPW_TAU), tb = min(t1, ta + TPW_TAU);
        wave_tau(L, ur, tr, ta, tb, k, start0, lane, status);
    } else {
        wave_theta(L, ur, t0, t1, k, th_start, lane, th);
    }
    __syncthreads();
    for (int i = tid; i < L.M; i += NT_CHUNK) {
        const int p = L.pos(i);
        if (p < t1) write_death(sel_key(L.val(i), p), p, t0, t1, k, th, th_start, dr, j0, survivor);
    }
}

// The same for the sorted list: theta at the chunk start is the k-th sorted key.
__device__ void chunk_body_sorted(const ListSorted& L, const float* __restrict__ ur, float* __restrict__ tr,
                                  int32_t* __restrict__ dr, int t0, int t1, int k, float lo,
                                  unsigned long long* th, Status status, int j0, int survivor)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const unsigned long long th_start = (t0 >= k) ? L.key[k - 1] : 0ull;
    // tau lies in [z_(k) - 1, z_(k)), and both ends only rise: theta_{t0-1} - 1 bounds every tau of the chunk
    float start0 = lo;
    if (t0 >= k) start0 = fmaxf(lo, key_score(th_start) - 1.0f);
    if (wv < NW_TAU) {
        const int ta = min(t1, t0 + wv * TPW_TAU), tb = min(t1, ta + TPW_TAU);
        wave_tau(L, ur, tr, ta, tb, k, start0, lane, status);
    } else {
        wave_theta(L, ur, t0, t1, k, th_start, lane, th);
    }
    __syncthreads();
    for (int i = tid; i < L.m_old; i += NT_CHUNK) {
        const unsigned long long key = L.key[i];
        write_death(key, key_pos(key), t0, t1, k, th, th_start, dr, j0, survivor);
    }
    if (tid < t1 - t0) write_death(sel_key(ur[t0 + tid], t0 + tid), t0 + tid, t0, t1, k, th, th_start, dr, j0, survivor);
}

// Sorts key[0, m), m <= NT_CHUNK, distinct keys, in descending order by counting (a few entries: no cascade of barriers).
__device__ void rank_sort_desc(unsigned long long* key, int m)
{
    const int tid = threadIdx.x;
    const unsigned long long mine = key[min(tid, m - 1)];
    int rank = 0;
    if (tid < m)
        for (int j = 0; j < m; j++) rank += key[j] > mine ? 1 : 0;
    __syncthreads();
    if (tid < m) key[rank] = mine;
    __syncthreads();
}

constexpr int WAIT_LDS = 0xC07F;   // s_waitcnt lgkmcnt(0) alone

// Bitonic sort of key[0, N) in descending order, N a power of two >= 2048 (one or more pairs per
// thread).  Each wave owns a contiguous run of N/32 compare-exchange pairs, so passes whose
// stride fits into the wave's N/16 elements need no workgroup barrier: a wave's LDS accesses are
// performed in program order.
__device__ void bitonic_sort_desc(unsigned long long* key, int N)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int P = N / (2 * NW_CHUNK);  // pairs per wave
    for (int k2 = 2; k2 <= N; k2 <<= 1) {
        for (int j = k2 >> 1; j > 0; j >>= 1) {
            if (j > P) {
                // The compiler leaves the wait out here although the stage before, without a barrier of its own, has
                // writes under way: other waves then read what was there before them.
                __builtin_amdgcn_s_waitcnt(WAIT_LDS);
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (what other lanes wrote has to be read)
            }
            for (int m = lane; m < P; m += 64) {
                const int i = wv * P + m;
                const int a = 2 * i - (i & (j - 1)), b = a + j;
                const unsigned long long x = key[a], y = key[b];
                const bool desc = (a & k2) == 0;
                if ((x < y) == desc) {
                    key[a] = y;
                    key[b] = x;
                }
            }
            if (j > P) __syncthreads();
        }
    }
    __syncthreads();
}

// pref[i] = sum of the scores of key[0, PSTRIDE * i), i = 0..N / PSTRIDE, in fp64 (N a multiple of NT_CHUNK * 2).
// Infinite scores count as 0: they are never fractional, and a difference of two sums has to stay a number.
__device__ void sorted_prefix_sums(const unsigned long long* key, double* pref, int N, int m_old, double* wtot)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    double carry = 0.0;
    auto score = [&](int i) {
        const float z = i < m_old ? key_score(key[i]) : 0.0f;
        return fabsf(z) < INFINITY ? (double)z : 0.0;
    };
    for (int base = 0; base < N; base += NT_CHUNK * PSTRIDE) {
        double run = 0.0;
        for (int r = 0; r < PSTRIDE; r++) run += score(base + tid * PSTRIDE + r);
        // inclusive scan of the thread totals across the wave, then across the waves
        double inc = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        __syncthreads();
        if (lane == 63) wtot[wv] = inc;
        __syncthreads();
        double before = carry + inc - run;
        for (int i = 0; i < wv; i++) before += wtot[i];
        for (int i = 0; i < NW_CHUNK; i++) carry += wtot[i];
        if (base + tid * PSTRIDE <= N) pref[base / PSTRIDE + tid] = before;
    }
    if (tid == 0) pref[N / PSTRIDE] = carry;
    __syncthreads();
}

// LDS of the sorted path.
struct SortedSmem {
    unsigned long long skey[CAP];
    double pref[CAP / PSTRIDE + 1];
    unsigned long long th[CHUNK];
    unsigned hist[256];
    double wtot[NW_CHUNK];
    int count;
    unsigned long long bc;
};

// What a function that is not inlined is called with: the address spaces go along, or every access would be a flat one,
// and what is the same in every lane is moved to scalar registers, or it would not be known to be.
#define SPK_LDS __attribute__((address_space(3)))
#define SPK_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T* uniform_global(T* p)
{
    const unsigned long long x = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)x), hi = __builtin_amdgcn_readfirstlane((unsigned)(x >> 32));
    return (T*)(SPK_GLOBAL T*)((unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ int uniform_int(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ Status uniform_status(Status s) { return Status{uniform_global(s.word), uniform_int(s.bit)}; }

// A lower bound of every threshold of a chunk that starts at t0 >= k; tight: a few bins below the first one.
struct ChunkBound {
    float lo;
    bool tight;
};

// tau lies in [z_(k) - 1, z_(k)) and both ends only rise: theta_{t0-1} - 1 is such a bound.  Ends with a barrier.
__device__ float theta_bound(SortedSmem& sm, const float* __restrict__ ur, int t0, int k)
{
    __syncthreads();
    const unsigned long long th_start = block_kth_largest(ListGlobal{ur, t0}, t0, k, sm.hist, &sm.bc);
    __syncthreads();
    return __double2float_rd((double)key_score(th_start) - 1.0);
}

// One chunk by sorting its candidates (whole workgroup).  Positions count from the row's first valid key.
__device__ __noinline__ void mask_chunk_sorted(SPK_LDS SortedSmem* smem, const float* __restrict__ ur, float* __restrict__ tr,
                                  int32_t* __restrict__ dr, int t0, int t1, int k, Status status, int j0, int survivor,
                                  ChunkBound known)
{
    SortedSmem& sm = *(SortedSmem*)smem;
    ur = uniform_global(ur);
    tr = uniform_global(tr);
    dr = uniform_global(dr);
    status = uniform_status(status);
    t0 = uniform_int(t0);
    t1 = uniform_int(t1);
    k = uniform_int(k);
    j0 = uniform_int(j0);
    survivor = uniform_int(survivor);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    float lo = t0 >= k ? readlane_f32(known.lo, 0) : -INFINITY;
    bool exact = t0 < k || uniform_int(known.tight) != 0;   // no better bound is to be had
    if (!exact && !(lo > -INFINITY)) {
        lo = theta_bound(sm, ur, t0, k);
        exact = true;
    }
    // ---- compaction of {j < t0 : u_j > lo} as selection keys, in one pass: each wave owns a contiguous slice, read
    // in segments of 64*SLICE_REG scores held in registers (independent loads, one latency); a segment reserves
    // its room in the list with one LDS atomic.  The order in which the segments land does not matter: the list
    // is sorted next, and the keys are distinct.  A prefix of fewer than k keys selects all of them, scores of -inf
    // included: then every position is taken. ----
    const bool all = t0 < k;
    const int per = ((t0 + NW_CHUNK - 1) / NW_CHUNK + 63) / 64 * 64;
    const int sb = min(t0, wv * per), se = min(t0, sb + per);
    constexpr int SEGN = 64 * SLICE_REG;
    for (;;) {
        if (tid == 0) sm.count = 0;
        __syncthreads();
        for (int g0 = sb; g0 < se; g0 += SEGN) {
            float z[SLICE_REG];
    #pragma unroll
            for (int r = 0; r < SLICE_REG; r++) {
                const int i = g0 + r * 64 + lane;
                z[r] = (i < se) ? ur[i] : -INFINITY;
            }
            int seg_cnt = 0;
    #pragma unroll
            for (int r = 0; r < SLICE_REG; r++) {
                const bool p = g0 + r * 64 + lane < se && (all || z[r] > lo);
                seg_cnt += __popcll(__ballot(p));
            }
            int off = 0;
            if (lane == 0 && seg_cnt > 0) off = atomicAdd(&sm.count, seg_cnt);
            off = __builtin_amdgcn_readfirstlane(off);
    #pragma unroll
            for (int r = 0; r < SLICE_REG; r++) {
                const bool p = g0 + r * 64 + lane < se && (all || z[r] > lo);
                const unsigned long long ball = __ballot(p);
                const int pos = off + __popcll(ball & ((1ull << lane) - 1ull));
                if (p && pos < CAP) sm.skey[pos] = sel_key(z[r], g0 + r * 64 + lane);   // beyond CAP: the slow path below
                off += __popcll(ball);
            }
        }
        __syncthreads();
        if (exact || uniform_int(sm.count) <= CAP) break;
        lo = theta_bound(sm, ur, t0, k);   // a coarse bound leaves too many
        exact = true;
    }
    const int m_old = uniform_int(sm.count);
    // the list must hold the whole top-k of every prefix of the chunk (it does when lo is a lower
    // bound of tau; checked, not assumed)
    const bool fits = (m_old <= CAP) && (t0 < k || m_old >= k);
    if (fits) {
        int npad = 2 * NT_CHUNK;
        while (npad < m_old) npad <<= 1;
        for (int i = m_old + tid; i < npad; i += NT_CHUNK) sm.skey[i] = 0ull;  // below every real key
        __syncthreads();
        if (m_old > 0) {
            if (m_old <= 512) rank_sort_desc(sm.skey, m_old);
            else bitonic_sort_desc(sm.skey, npad);
            sorted_prefix_sums(sm.skey, sm.pref, npad, m_old, sm.wtot);
        }
        const int cn = t1 - t0;
        ListSorted L{sm.skey, sm.pref, m_old, t0, (lane < cn) ? ur[t0 + lane] : -INFINITY,
                     (lane + 64 < cn) ? ur[t0 + lane + 64] : -INFINITY};
        chunk_body_sorted(L, ur, tr, dr, t0, t1, k, lo, sm.th, status, j0, survivor);
    } else {
        ListGlobal L{ur, t1};
        chunk_body(L, ur, tr, dr, t0, t1, k, -INFINITY, sm.hist, &sm.bc, sm.th, status, j0, survivor);
    }
}

// ---------------------------------------------------------------------------------
// The histogram path.  With few chunks it is bounded by latency -- two passes over the prefix, a dozen workgroup barriers --
// and by the slowest chunk: 30000 cycles for 128 prefixes far into a row (histogram 2000, bounds 4300, second pass 5000,
// sorting the two short lists 6000, thresholds 8500, lifetimes 3000), 55000 around prefix k, where four times as many scores
// lie between the bounds.  With many chunks it is bounded by instruction issue (1600 vector instructions per wave and chunk,
// four fifths of the cycles of a SIMD).  One row of 32768 scores at k = 1024: 32 -> 25 us, 4096 at k = 256: 29 -> 15 us with
// chunks dealt as launch_mask says, lifetimes by 16 lanes per key and thresholds by interpolation; 32 rows of 16384: 248 ->
// 211 us.  Before the histogram, with a bracket search and a sort of all candidates per chunk: 85 us and 390 us.
// Windows that follow the scores, 32 rows of 16384, k = 1024: standard deviation 7 in 279 us, 27 in 276, 0.05 in 405, mean 20 in 297.  With
// two fixed widths of window and the sorted path for the rest: 716, 834, 3418 and 383; with every chunk sorted: 360, 369,
// 9185 and 390.  One row of 131072 at k = 16384: 314 us, 13.3 ms with the fixed width.
// ---------------------------------------------------------------------------------
constexpr int HBINS = 2048;      // bins of a window; scores below and above it count in the first and the last one
constexpr int WINDOWS = 4;       // windows tried at most
constexpr int TL_WAVE = 64;      // per wave: scores with a breakpoint between the bounds
constexpr int TL_CAP = NW_CHUNK * TL_WAVE;
constexpr int QL_CAP = 256;      // keys between the bounds of theta (each is compared with all of them)
constexpr int CP_CAP = 64 + 128 + 64;   // what is left of the last 64, two groups of a wave, slack for reads past the end
constexpr int BP_REG = 5;
constexpr int BP_CAP = 64 * BP_REG;     // breakpoints between the bounds, for the parallel solution

// A window: HBINS bins of width 1 / res from origin on.  covers: no score lies above it.  bounded: the thresholds of the
// chunk lie in [lo, hi).
struct HistWindow {
    float origin, res;
    bool covers, bounded;
    double lo, hi;
};

struct HistSmem {
    union {
        struct {
            unsigned hist[HBINS], own[HBINS];   // older scores, the chunk's own scores
            unsigned cum[2][HBINS];             // twice-cumulated counts, from the top bin down: older, all
        } h;
        struct {
            float v[NW_CHUNK][CP_CAP];          // per wave: older scores above the lower bound
            int pos[NW_CHUNK][CP_CAP];
        } c;
        struct {
            float v[TL_CAP + 64];               // the scores between the bounds and their breakpoints, unordered,
            double bp[BP_CAP];
            int tie[TL_CAP], btie[BP_CAP];      // and how many of each rank have been placed
        } s;
        double gain[NW_CHUNK][BP_CAP];          // what a wave's newcomers add to f at every breakpoint
    } x;
    float raw[NW_CHUNK][TL_WAVE];       // per wave: scores between the bounds
    float tl[TL_CAP];                   // the same in descending order
    double pref[BP_CAP + 1];            // sums of the first i of them
    double bps[BP_CAP];                 // lower bound, breakpoints, upper bound: ascending
    double bf[BP_CAP];                  // f of the prefix before the chunk there
    unsigned long long qk[QL_CAP];      // selection keys between the bounds of theta
    float own[CHUNK];
    unsigned long long ownkey[CHUNK];
    int oc[CHUNK], no;              // own keys between the bounds of theta, their number
    unsigned wscan[4][NW_CHUNK];
    float wmm[2][NW_CHUNK];
    double wsum[NW_CHUNK];
    int wF[NW_CHUNK], wC[NW_CHUNK], wM[NW_CHUNK];
    int jlo, jhi, jl, jh, upto, above, jmin, nq, nbp, full;
    HistWindow win;                     // the last window tried
    ChunkBound known;                   // for the sorted path
};

// Inclusive sum over the lanes of a wave (DPP row shifts, then the row totals are broadcast).
__device__ __forceinline__ unsigned wave_scan_u32(unsigned x)
{
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast15 into rows 1 and 3
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast31 into rows 2 and 3
    return x;
}

// Exclusive sums of two counters over the workgroup's threads; barriers inside (two arrays w, distinct per call).
__device__ __forceinline__ void block_scan2(unsigned a, unsigned b, unsigned* wa, unsigned* wb, unsigned& ea, unsigned& eb)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned ia = wave_scan_u32(a), ib = wave_scan_u32(b);
    if (lane == 63) { wa[wv] = ia; wb[wv] = ib; }
    __syncthreads();
    // lane l of every wave holds wave l's total; the sum over the waves before this one is a ballot-free wave scan
    const unsigned ta = wave_scan_u32(lane < NW_CHUNK ? wa[lane] : 0u), tb = wave_scan_u32(lane < NW_CHUNK ? wb[lane] : 0u);
    const unsigned pa = wv > 0 ? (unsigned)__builtin_amdgcn_readlane((int)ta, wv - 1) : 0u;
    const unsigned pb = wv > 0 ? (unsigned)__builtin_amdgcn_readlane((int)tb, wv - 1) : 0u;
    ea = pa + ia - a;
    eb = pb + ib - b;
}

// The scores a prefix of the chunk is made of, for thresholds between the bounds: Fb scores that are saturated and Cb
// (sum sumb) that are fractional at every such threshold, a short list in a fixed order, and the chunk's own scores, two
// per lane.  The first 64 * TL_REG entries of the list live in registers, widened once, so that a comparison with a
// threshold or a threshold + 1 is one instruction; -inf fills up.
constexpr int TL_REG = 3;
struct ListBounded {
    const float* v;
    int M, Fb, Cb;
    double sumb;
    int t0, lane;
    double own[2];
    double reg[TL_REG];
};

// A condition that is the same in every lane, as a scalar branch.
__device__ __forceinline__ bool uniform(bool c) { return __ballot(c) != 0ull; }

template <typename F>
__device__ __forceinline__ void each_bounded(const ListBounded& L, int t, F&& f)
{
#pragma unroll
    for (int r = 0; r < TL_REG; r++)
        if (64 * r < L.M) f(L.reg[r]);
    for (int i = 64 * TL_REG; i < L.M; i += 64) f(i + L.lane < L.M ? (double)L.v[i + L.lane] : -INFINITY);
    const int nc = t - L.t0 + 1;
    f(L.lane < nc ? L.own[0] : -INFINITY);
    if (nc > 64) f(L.lane + 64 < nc ? L.own[1] : -INFINITY);
}

struct PieceB {
    int F, S;
    double fsum;
};

// Right-limit counts of the linear piece of f_t that contains x.  A sum of one fractional score is exact (no
// differences of sums), which the flat case -- root exactly on a breakpoint, sup rule -- relies on.
__device__ __forceinline__ PieceB eval_bounded(const ListBounded& L, int t, double x)
{
    const double x1 = x + 1.0;
    int F = L.Fb, S = L.Fb + L.Cb;
    double part = 0.0;
    each_bounded(L, t, [&](double v) {
        const unsigned long long a = __ballot(v > x), b = __ballot(v > x1);
        S += (int)__popcll(a);
        F += (int)__popcll(b);
        part += ((a & ~b) >> L.lane) & 1ull ? v : 0.0;
    });
    return PieceB{F, S, L.sumb + wave_sum_f64(part)};
}

// True if no score of prefix t has a breakpoint (z or z - 1) in (lo, hi], both between the bounds.
__device__ __forceinline__ bool clear_bounded(const ListBounded& L, int t, double lo, double hi)
{
    const double lo1 = lo + 1.0, hi1 = hi + 1.0;
    unsigned long long hit = 0ull;
    each_bounded(L, t, [&](double v) {
        hit |= (__ballot(v > lo) & ~__ballot(v > hi)) | (__ballot(v > lo1) & ~__ballot(v > hi1));
    });
    return hit == 0ull;
}

// Smallest listed or own score above x + 1 in prefix t.
__device__ __forceinline__ double min_saturated(const ListBounded& L, int t, double x)
{
    const double x1 = x + 1.0;
    float mf = INFINITY;
    each_bounded(L, t, [&](double v) { mf = fminf(mf, v > x1 ? (float)v : INFINITY); });
    return (double)wave_min_f32(mf);
}

// One wave, thresholds of prefixes [ta, tb), tb - ta <= 64 (those longer than k), all roots in [lo, hi).  The iteration
// is that of wave_tau(ListSorted): the piece is carried from prefix to prefix and only evaluated again when a breakpoint
// was crossed; prefixes whose newcomer is not above the threshold are passed over.
__device__ __forceinline__ void wave_tau(const ListBounded& L, float* __restrict__ tr, int ta, int tb, int k, double lo,
                                         double hi, Status status)
{
    const int first = max(ta, k);   // prefixes of at most k entries: written by short_prefix_tau
    if (first >= tb) return;
    bool have = false;
    double x = lo;
    float res = 0.0f;               // lane l: threshold of prefix ta + l
    PieceB P{0, 0, 0.0};
    for (int t = first; t < tb;) {
        const int c = t - L.t0;
        if (have) {
            const float utf = c < 64 ? readlane_f32((float)L.own[0], c) : readlane_f32((float)L.own[1], c - 64);
            const double ut = (double)utf;
            P.S++;
            if (uniform(ut > x + 1.0)) P.F++;
            else P.fsum += ut;
        } else {
            P = eval_bounded(L, t, x);
            have = true;
        }
        double lo_b = x, hi_b = hi;
        int it = 0;
        for (; it < MAX_ITERS; it++) {
            const double f = (double)P.F + P.fsum - (double)(P.S - P.F) * x;
            const bool left = uniform(!(f < (double)k));
            double xn = (P.fsum + (double)P.F - (double)k) / (double)(P.S - P.F);
            bool step = false;
            if (!left) {
                hi_b = x;
                if (P.S > P.F) {
                    if (uniform(xn >= lo_b && xn < x) && clear_bounded(L, t, xn, x)) { x = xn; break; }
                    step = uniform(xn > lo_b && xn < hi_b);
                }
            } else {
                lo_b = x;
                if (P.S == P.F) {  // flat to the right of x, f == F there
                    const double nb = min_saturated(L, t, x) - 1.0;  // next breakpoint
                    if (P.F == k && uniform(nb < hi)) {  // sup of the level set f == k; the piece changes there
                        x = nb;
                        have = false;
                        break;
                    }
                    xn = nb;  // F > k: still left of the root
                } else {
                    if (!uniform(xn > x)) break;  // f(x) == k up to rounding
                    if (uniform(xn < hi_b) && clear_bounded(L, t, x, xn)) { x = xn; break; }
                }
                step = uniform(xn < hi_b);
            }
            if (!step) {
                const double mid = 0.5 * (lo_b + hi_b);
                if (!uniform(mid > lo_b && mid < hi_b)) { x = lo_b; have = false; break; }
                xn = mid;
            }
            x = xn;
            P = eval_bounded(L, t, x);
        }
        if (it == MAX_ITERS && L.lane == 0) atomicOr(status.word, status.bit);
        // the next prefix whose newcomer is above the threshold
        const int nc = t + 1 - L.t0;
        unsigned long long m0 = __ballot(L.own[0] > x), m1 = __ballot(L.own[1] > x);
        m0 = nc < 64 ? m0 >> nc << nc : 0ull;
        m1 = nc <= 64 ? m1 : nc < 128 ? m1 >> (nc - 64) << (nc - 64) : 0ull;
        const int next = min(tb, m0 ? L.t0 + __builtin_ctzll(m0) : m1 ? L.t0 + 64 + __builtin_ctzll(m1) : tb);
        res = ta + L.lane >= t && ta + L.lane < next ? (float)x : res;
        t = next;
    }
    if (ta + L.lane >= first && ta + L.lane < tb) tr[ta + L.lane] = res;
}

// Thresholds of the chunk's prefixes with at most k entries: tau_t = min(u[0..t]) - 1 (k == 0: max(u[0..t])).
// `before`: the extremum of u[0, t0).  One wave.
__device__ __forceinline__ void short_prefix_tau(float before, float nv0, float nv1, int t0, int t1, int k, int lane,
                                                 float* __restrict__ tr)
{
    const bool use_max = k == 0;
    const float none = use_max ? -INFINITY : INFINITY;
    const int cn = t1 - t0;
    float a = lane < cn ? nv0 : none, b = lane + 64 < cn ? nv1 : none;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float ya = __shfl_up(a, o, 64), yb = __shfl_up(b, o, 64);
        if (lane >= o) {
            a = use_max ? fmaxf(a, ya) : fminf(a, ya);
            b = use_max ? fmaxf(b, yb) : fminf(b, yb);
        }
    }
    const float top = readlane_f32(a, 63);
    a = use_max ? fmaxf(a, before) : fminf(a, before);
    b = use_max ? fmaxf(fmaxf(b, top), before) : fminf(fminf(b, top), before);
    const int upto = use_max ? t1 : min(t1, k);
    if (t0 + lane < upto) tr[t0 + lane] = use_max ? a : a - 1.0f;
    if (t0 + lane + 64 < upto) tr[t0 + lane + 64] = use_max ? b : b - 1.0f;
}

// f(score, position, is one) for the older scores, NT_CHUNK of them at a time in a fixed order, four groups in flight;
// after() follows every two groups.
template <typename F, typename G>
__device__ __forceinline__ void each_older(const float* __restrict__ ur, int t0, F&& f, G&& after)
{
    const int tid = threadIdx.x;
    auto get = [&](int base) { return base + tid < t0 ? ur[base + tid] : -INFINITY; };
    float z[4];
#pragma unroll
    for (int r = 0; r < 4; r++) z[r] = get(r * NT_CHUNK);
    for (int base = 0; base < t0; base += 4 * NT_CHUNK) {
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int b = base + r * NT_CHUNK;
            if (b < t0) f(z[r], b + tid, b + tid < t0);
            z[r] = get(b + 4 * NT_CHUNK);
            if (r & 1) after();
        }
    }
}

__device__ __forceinline__ int tM_before(int inclusive, int wv) { return wv > 0 ? __builtin_amdgcn_readlane(inclusive, wv - 1) : 0; }

// Inclusive sum over the lanes of a wave, fp64 (in lane order).
__device__ __forceinline__ double wave_scan_f64(double x)
{
#define SPK_SCAN_STEP(ctrl, rows)                                                                                       \
    {                                                                                                                   \
        const unsigned long long b = (unsigned long long)__double_as_longlong(x);                                       \
        const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, ctrl, rows, 0xF, rows == 0xF);                  \
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), ctrl, rows, 0xF, rows == 0xF);          \
        x += __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));                \
    }
    SPK_SCAN_STEP(0x111, 0xF)
    SPK_SCAN_STEP(0x112, 0xF)
    SPK_SCAN_STEP(0x114, 0xF)
    SPK_SCAN_STEP(0x118, 0xF)
    SPK_SCAN_STEP(0x142, 0xA)
    SPK_SCAN_STEP(0x143, 0xC)
#undef SPK_SCAN_STEP
    return x;
}

// Thresholds of all prefixes of the chunk at once (whole workgroup; wave w owns the prefixes [ta, tb), at most 64).  f_t is
// linear between neighbouring breakpoints and does not increase, so the root lies right of the last breakpoint at which
// f_t is still at least k, and f_t there and at the next one say where.  sm.bps: lo, the breakpoints, hi.
//   1. f_{t0-1} at every breakpoint: two searches in the sorted list and a difference of its prefix sums;
//   2. every wave adds up what its own newcomers contribute at every breakpoint;
//   3. every wave takes the sum over the waves before it, adds its newcomers one by one, counts the breakpoints with
//      f >= k after each and keeps f at both ends of the piece;
//   4. a lane per prefix interpolates.
// The slope of a piece is a number of scores: below one half it is none, and the root of a flat piece at k is its right
// end (sup rule).  On a flat piece f is a sum of whole numbers, hence exact.  Elsewhere f is off by about 2^-53 times the
// fractional scores' number and distance from 0 (1e-13 for a thousand around 0, 1e-8 around 1e5), as any sum of them is,
// and the root by that over the slope, but never out of its piece.  (The piece's own counts -- searches and a pass over the newcomers per prefix -- took a
// quarter of the instructions of this function.)
__device__ __forceinline__ void solve_parallel(HistSmem& sm, const ListBounded& L, float* __restrict__ tr, int ta, int tb,
                                               int k, double lo)
{
    const int tid = threadIdx.x, lane = L.lane, wv = tid >> 6;
    const int M = L.M, B = sm.nbp + 2;
    // prefix sums of the sorted list (wave 0) beside the searches of the others
    int S = 0, F = 0;
    const int bp = tid - 64;
    if (wv == 0) {
        double carry = 0.0;
        if (lane == 0) sm.pref[0] = 0.0;
        for (int m = 0; m < M; m += 64) {
            const double z = m + lane < M ? (double)sm.tl[m + lane] : 0.0;
            const double inc = wave_scan_f64(z);
            if (m + lane < M) sm.pref[m + lane + 1] = carry + inc;
            carry += __longlong_as_double((long long)readlane_u64((unsigned long long)__double_as_longlong(inc), 63));
        }
    } else if (bp < B) {
        const double x = sm.bps[bp];
        auto above = [&](double y) {   // listed scores above y
            int a = 0, b = M;
            while (a < b) {
                const int m = (a + b) >> 1;
                if ((double)sm.tl[m] > y) a = m + 1;
                else b = m;
            }
            return a;
        };
        S = above(x);
        F = above(x + 1.0);
    }
    __syncthreads();
    if (wv > 0 && bp < B) {
        const int Fa = L.Fb + F, Sa = L.Fb + L.Cb + S;
        sm.bf[bp] = (double)Fa + (L.sumb + (sm.pref[S] - sm.pref[F])) - (double)(Sa - Fa) * sm.bps[bp];
    }
    // 2. (registers: breakpoint 64 r + lane)
    double b[BP_REG];
#pragma unroll
    for (int r = 0; r < BP_REG; r++) b[r] = 64 * r + lane < B ? sm.bps[64 * r + lane] : INFINITY;
    auto clip = [](double x) { return fmin(fmax(x, 0.0), 1.0); };
    const int c0 = ta - L.t0, cn = tb - ta;
    double g[BP_REG];
#pragma unroll
    for (int r = 0; r < BP_REG; r++) g[r] = 0.0;
    for (int s = 0; s < cn; s++) {
        const double us = (double)sm.own[c0 + s];
        if (!uniform(us > lo)) continue;
#pragma unroll
        for (int r = 0; r < BP_REG; r++)
            if (64 * r < B) g[r] += clip(us - b[r]);
    }
#pragma unroll
    for (int r = 0; r < BP_REG; r++)
        if (64 * r < B) sm.x.gain[wv][64 * r + lane] = g[r];
    __syncthreads();
    // 3.
#pragma unroll
    for (int r = 0; r < BP_REG; r++) {
        g[r] = -INFINITY;      // f from here on
        if (64 * r >= B) continue;
        if (64 * r + lane < B) g[r] = sm.bf[64 * r + lane];
        for (int w = 0; w < wv; w++) g[r] += sm.x.gain[w][64 * r + lane];
    }
    int seg = 1;                       // lane p: prefix ta + p
    double f0 = 0.0, f1 = 0.0;
    int count = 0;
    double e0 = 0.0, e1 = 0.0;
    for (int s = 0; s < cn; s++) {
        const double us = (double)sm.own[c0 + s];
        const bool on = uniform(us > lo);
        if (on) {
#pragma unroll
            for (int r = 0; r < BP_REG; r++)
                if (64 * r < B) g[r] += clip(us - b[r]);
        }
        if (on || s == 0) {
            count = 0;
#pragma unroll
            for (int r = 0; r < BP_REG; r++)
                if (64 * r < B) count += (int)__popcll(__ballot(g[r] >= (double)k));
            count = min(max(count, 1), B - 1);
#pragma unroll
            for (int r = 0; r < BP_REG; r++) {
                const unsigned long long fr = (unsigned long long)__double_as_longlong(g[r]);
                if ((count - 1) >> 6 == r) e0 = __longlong_as_double((long long)readlane_u64(fr, (count - 1) & 63));
                if (count >> 6 == r) e1 = __longlong_as_double((long long)readlane_u64(fr, count & 63));
            }
        }
        if (lane == s) {
            seg = count;
            f0 = e0;
            f1 = e1;
        }
    }
    // 4.
    const double x0 = sm.bps[seg - 1], x1 = sm.bps[seg], fall = f0 - f1;
    double x = fall < 0.5 * (x1 - x0) ? x1 : x0 + (f0 - (double)k) / fall * (x1 - x0);
    x = fmin(fmax(x, x0), x1);
    if (ta + lane < tb && ta + lane >= k) tr[ta + lane] = (float)x;
}

// The window to try after sm.win, from what that one says of the thresholds and of the k-th largest score, if no more than
// "above" or "too many in a bin", and from the smallest and the largest score; false: there is none (whole workgroup).
__device__ bool next_window(HistSmem& sm, const float* __restrict__ ur, int t0, int cn, int k, int tried)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const HistWindow W = sm.win;
    const int jl = sm.jl, jh = sm.jh;
    if (tried == 1) {
        float a = INFINITY, b = -INFINITY;
        each_older(ur, t0, [&](float v, int, bool in) { a = fminf(a, in ? v : INFINITY); b = fmaxf(b, v); }, [] {});
        const float nv0 = sm.own[lane], nv1 = sm.own[lane + 64];
        a = wave_min_f32(fminf(a, fminf(lane < cn ? nv0 : INFINITY, lane + 64 < cn ? nv1 : INFINITY)));
        b = wave_max_f32(fmaxf(b, fmaxf(nv0, nv1)));
        if (lane == 0) { sm.wmm[0][wv] = a; sm.wmm[1][wv] = b; }
    }
    __syncthreads();   // (everybody has read what the next window clears)
    const float smallest = wave_min_f32(lane < NW_CHUNK ? sm.wmm[0][lane] : INFINITY);
    const float largest = wave_max_f32(lane < NW_CHUNK ? sm.wmm[1][lane] : -INFINITY);
    // From below the first threshold to the k-th largest score, and to a unit above the last threshold unless no score
    // lies there.
    const float edge = 1.0f / W.res;
    float from, to = jh >= 0 && jh < HBINS - 1 ? fminf(W.origin + (float)(jh + 1) * edge, largest) : largest;
    if (W.bounded) {
        from = __double2float_rd(W.lo);
        to = fmaxf(to, fminf(largest, __double2float_ru(W.hi + 1.0)));
    } else {
        from = (t0 < k || jl <= 0 ? smallest : fmaxf(W.origin + (float)jl * edge, smallest)) - 1.0f;
        to = fminf(largest, to + 1.0f);
    }
    const float span = to - from;
    if (smallest == largest || !(span > 0.0f && span < 1e30f)) return false;   // (one score for all, infinities)
    int e;
    frexpf((float)(HBINS - 8) / span, &e);   // 2^(e-1) <= bins per unit < 2^e
    float res = ldexpf(1.0f, min(e - 1, 15));
    while (fabsf(from) * res > 4194304.0f) res *= 0.5f;   // the origin as a number of bins has to be exact
    if ((W.bounded || tried > 1) && res < 2.0f * W.res) return false;   // as fine as it gets
    const float origin = floorf(from * res - 2.0f) / res;
    sm.win.res = res;   // (every wave writes the same)
    sm.win.origin = origin;
    sm.win.covers = fmaf(largest, res, -origin * res) < (float)HBINS;
    return true;
}

// What comes ahead of the windows: the chunk's own scores to LDS, thresholds of prefixes of at most k entries.  NEXT: its
// own scores say that [-8, 8) is not the window to start with, and sm.win is one that suits them.
enum { HIST_DONE, HIST_FIRST, HIST_NEXT, HIST_NONE };
__device__ __forceinline__ int mask_chunk_begin(HistSmem& sm, const float* __restrict__ ur, float* __restrict__ tr, int t0,
                                                int t1, int k)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int cn = t1 - t0;
    const float nv0 = lane < cn ? ur[t0 + lane] : -INFINITY, nv1 = lane + 64 < cn ? ur[t0 + lane + 64] : -INFINITY;
    if (wv == 0) {
        sm.ownkey[lane] = sel_key(nv0, t0 + lane);
        sm.ownkey[lane + 64] = sel_key(nv1, t0 + lane + 64);
        sm.own[lane] = nv0;
        sm.own[lane + 64] = nv1;
    }
    if (tid == 0) sm.known = ChunkBound{-INFINITY, false};
    if (t0 < k) {
        float mn = INFINITY;
        each_older(ur, t0, [&](float v, int, bool in) { mn = fminf(mn, in ? v : INFINITY); }, [] {});
        mn = wave_min_f32(mn);
        if (lane == 0) sm.wmm[0][wv] = mn;
        __syncthreads();
        const float before = wave_min_f32(lane < NW_CHUNK ? sm.wmm[0][lane] : INFINITY);
        if (wv == 0) short_prefix_tau(before, nv0, nv1, t0, t1, k, lane, tr);
        if (t1 <= k) return HIST_DONE;
        if (!(before > -INFINITY)) return HIST_NONE;   // (thresholds of -inf)
        __syncthreads();
    }
    auto outside = [](float v) { return v >= 8.0f || (v < -8.0f && v > -INFINITY); };
    if (!uniform(outside(nv0) || outside(nv1))) return HIST_FIRST;
    const float s0 = nv0 > -INFINITY ? nv0 : INFINITY, s1 = nv1 > -INFINITY ? nv1 : INFINITY;
    const float mn = wave_min_f32(fminf(s0, s1)), mx = wave_max_f32(fmaxf(nv0, nv1));
    if (!uniform(mx - mn < 1e30f)) return HIST_FIRST;
    float res = 128.0f;
    while (res > 1e-30f && (1.375f * (mx - mn) * res > (float)HBINS || fmaxf(fabsf(mn), fabsf(mx)) * res > 4194304.0f)) res *= 0.5f;
    sm.win.res = res;   // (every wave writes the same)
    sm.win.origin = floorf(0.5f * (mn + mx) * res - 0.5f * (float)HBINS) / res;
    sm.win.covers = false;
    return HIST_NEXT;
}

// One chunk (t0 < t1, k >= 1) by its histogram.  FIRST: in the window [-8, 8) with 128 bins per unit, which suits scores of
// about unit variance around 0; else in up to WINDOWS others, the first of them after [-8, 8) (tried = 1) or instead of it
// (tried = 0).  If not DONE, nothing has been written but lifetimes that are written again.
// UNROLL: of the loops that rank the lists; 4 where there are registers for it (with 64 of them 21 values are spilled around
// those loops, 130 MB of scratch for 32 rows of 16384).
template <bool FIRST, int UNROLL>
__device__ __forceinline__ int mask_chunk_hist(HistSmem& sm, const float* __restrict__ ur, float* __restrict__ tr,
                                               int32_t* __restrict__ dr, int t0, int t1, int k, Status status, int j0,
                                               int survivor, int tried)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int cn = t1 - t0;
    float origin = -8.0f, res = 128.0f, shift = 0.0f;
    bool covers = false;
    double lo = 0.0, hi = 0.0;
    float lof = 0.0f, hif = 0.0f, lo1f = 0.0f, hi1f = 0.0f, ql = 0.0f, qh = 0.0f;
    double csum = 0.0;
    int above = 0, nM = 0, nF = 0, nC = 0, MQ = 0;
    for (;; tried++) {
        if (!FIRST) {
            if (tried > 0 && (tried == WINDOWS || !next_window(sm, ur, t0, cn, k, tried))) return HIST_NONE;
            origin = readlane_f32(sm.win.origin, 0);
            res = readlane_f32(sm.win.res, 0);
            covers = uniform(sm.win.covers);
        }
        shift = -origin * res;      // exact: the origin is a multiple of 1 / res, and so many of them fit into 24 bits
        auto bin = [&](float v) { return (int)__builtin_amdgcn_fmed3f(fmaf(v, res, shift), 0.0f, (float)(HBINS - 1)); };
        const int R = res >= 1.0f ? (int)res : 0;   // bins of unit width together; none: the bins only find the k-th largest score
        *(uint2*)&sm.x.h.hist[2 * tid] = make_uint2(0, 0);
        *(uint2*)&sm.x.h.own[2 * tid] = make_uint2(0, 0);
        if (tid == 0) { sm.jlo = -1; sm.jhi = -1; sm.jl = t0 >= k ? -1 : 0; sm.jh = -1; sm.upto = t0; sm.above = 0; sm.jmin = 0; sm.nq = 0; sm.nbp = 0; sm.full = 0; }
        __syncthreads();
        each_older(ur, t0, [&](float v, int, bool in) { if (in) atomicAdd(&sm.x.h.hist[bin(v)], 1u); }, [] {});
        if (tid < cn) atomicAdd(&sm.x.h.own[bin(sm.own[tid])], 1u);
        __syncthreads();
        // Suffix counts N_i = #{bin >= i} of the older and of all scores: thread t owns the bins 2047 - 2t, 2046 - 2t.
        const int b0 = HBINS - 1 - 2 * tid;
        const uint2 ho = *(const uint2*)&sm.x.h.hist[b0 - 1], hn = *(const uint2*)&sm.x.h.own[b0 - 1];
        const unsigned o0 = ho.y, o1 = ho.x, a0 = o0 + hn.y, a1 = o1 + hn.x;
        unsigned eo, ea;
        block_scan2(o0 + o1, a0 + a1, sm.wscan[0], sm.wscan[1], eo, ea);
        const unsigned No0 = eo + o0, No1 = No0 + o1, Na0 = ea + a0, Na1 = Na0 + a1;
        if (No0 >= (unsigned)k && eo < (unsigned)k) { sm.jl = b0; sm.upto = (int)No0; }
        if (No1 >= (unsigned)k && No0 < (unsigned)k) { sm.jl = b0 - 1; sm.upto = (int)No1; }
        if (Na0 >= (unsigned)k && ea < (unsigned)k) { sm.jh = b0; sm.above = (int)eo; }
        if (Na1 >= (unsigned)k && Na0 < (unsigned)k) { sm.jh = b0 - 1; sm.above = (int)No0; }
        if (Na0 == (unsigned)t1 && ea < (unsigned)t1) sm.jmin = b0;
        if (Na1 == (unsigned)t1 && Na0 < (unsigned)t1) sm.jmin = b0 - 1;
        // Cumulate once more, so that windowed sums of N are differences.  Those of min(R, HBINS) counts have to stay below
        // 2^32 (2^24 scores at R = 128); beyond, the counts are scaled down (older: rounded down, all: rounded up).
        int s = 0;
        while (((unsigned long long)(t1 >> s) * (unsigned)min(R, HBINS)) > 1ull << 31) s++;
        const unsigned up = (1u << s) - 1u;
        unsigned co, ca;
        const unsigned so0 = No0 >> s, so1 = No1 >> s, sa0 = (Na0 + up) >> s, sa1 = (Na1 + up) >> s;
        block_scan2(so0 + so1, sa0 + sa1, sm.wscan[2], sm.wscan[3], co, ca);
        *(uint2*)&sm.x.h.cum[0][2 * tid] = make_uint2(co + so0, co + so0 + so1);
        *(uint2*)&sm.x.h.cum[1][2 * tid] = make_uint2(ca + sa0, ca + sa0 + sa1);
        __syncthreads();
        // f(edge_j) >= (sum of N_{j+1} .. N_{j+R} of the older scores) / R: the last j with a sum of at least
        // k * R is a lower bound of every threshold from prefix t0 - 1 on.  f(edge_j) <= (N_j + .. + N_{j+R-1}
        // of all scores) / R: the first j with a sum below k * R bounds every threshold of the chunk from above.
        // (Beyond the window N is 0 if it covers the scores; else the sums have to end inside it.)
        auto wsum = [&](int which, int d_hi, int d_lo) { return sm.x.h.cum[which][d_hi] - (d_lo >= 0 ? sm.x.h.cum[which][d_lo] : 0u); };
        const unsigned want = (unsigned)min(((unsigned long long)k * (unsigned)R + up) >> s, 0xFFFFFFFFull);
        auto low = [&](int j) { return wsum(0, HBINS - 2 - j, HBINS - 2 - R - j) >= want; };  // j <= jtop
        auto high = [&](int j) { return wsum(1, HBINS - 1 - j, HBINS - 1 - R - j) < want; };
        const int jtop = covers ? HBINS - 2 : HBINS - 1 - R;
        if (R > 0 && b0 - 1 >= 1 && b0 < jtop) {
            const bool l0 = low(b0 - 1), l1 = low(b0), l2 = low(b0 + 1);
            if (l0 && !l1) sm.jlo = b0 - 1;
            if (l1 && !l2) sm.jlo = b0;
            const bool h0 = high(b0 - 1), h1 = high(b0), h2 = high(b0 + 1);
            if (!h0 && h1) sm.jhi = b0;
            if (!h1 && h2) sm.jhi = b0 + 1;
        }
        __syncthreads();
        // the first threshold of a chunk that holds prefix k: at least the smallest score - 1
        const int jlo = t0 < k ? sm.jmin - R : sm.jlo, jhi = sm.jhi, jl = sm.jl, jh = sm.jh;
        above = sm.above;
        const double eps = 1.0 / 8192.0 / (double)res;   // bin() rounds: a score may lie half as much beyond its bin's edges
        const bool bounded = R > 0 && jhi > 0 && (t0 < k ? sm.jmin > 0 : jlo > 0);
        lo = (double)origin + (double)jlo / (double)res - eps;
        hi = (double)origin + (double)jhi / (double)res + eps;
        // What the second pass would have to list: where the bins are too wide for that, it is not worth its time.  (In the
        // first window the scores between the bounds hardly ever are too many, and counting them takes time.)
        auto N = [&](int j) -> unsigned { return j > HBINS - 1 ? 0u : wsum(0, HBINS - 1 - max(j, 0), HBINS - 2 - max(j, 0)) << s; };
        const bool worth = sm.upto - above <= QL_CAP && (FIRST || N(jlo) - N(jhi) + N(jlo + R) - N(jhi + R) <= TL_CAP);
        if (uniform(bounded && worth)) {
            // ---- second pass: count and sum what is certain between the bounds, collect what is not ----
            // (for an fp32 score v: v > x <=> v > rd(x))
            lof = __double2float_rd(lo);
            hif = __double2float_rd(hi);
            lo1f = __double2float_rd(lo + 1.0);
            hi1f = __double2float_rd(hi + 1.0);
            // bins jl .. jh as limits of the value that bin() truncates
            ql = jl == 0 ? -INFINITY : (float)jl;
            qh = jh == HBINS - 1 ? INFINITY : (float)(jh + 1);
            // nothing below this matters
            const float least = jl == 0 ? -INFINITY : __double2float_rd(fmin(lo, (double)origin + (double)jl / (double)res - eps));
            csum = 0.0;
            nM = nF = nC = 0;
            auto classify = [&](float v, int i, bool in) {
                const float tb = fmaf(v, res, shift);
                const bool sat = in && v > hi1f;
                const bool frac = in && v > hif && v <= lo1f;
                const bool open = in && v > lof && !sat && !frac;
                const bool sel = in && tb >= ql;
                const bool q = sel && tb < qh;
                nF += (int)__popcll(__ballot(sat && !frac));
                nC += (int)__popcll(__ballot(frac));
                csum += (double)(frac ? v : 0.0f);
                if (survivor && sel && !q) dr[i] = survivor;
                const unsigned long long bo = __ballot(open), bq = __ballot(q);
                const unsigned long long below = (1ull << lane) - 1ull;
                if (bo) {
                    const int at = nM + (int)__popcll(bo & below);
                    if (open && at < TL_WAVE) sm.raw[wv][at] = v;
                    nM += (int)__popcll(bo);
                }
                if (bq) {
                    int off = 0;
                    if (lane == 0) off = atomicAdd(&sm.nq, (int)__popcll(bq));
                    off = __builtin_amdgcn_readfirstlane(off) + (int)__popcll(bq & below);
                    if (q && off < QL_CAP) sm.qk[off] = sel_key(v, i);
                }
            };
            __syncthreads();  // the histograms are no longer needed
            // Only a few per cent of the scores lie above the lower bound.  Every wave collects its own and looks at them 64 at
            // a time, in an order that does not depend on timing (the sum is taken in that order).
            {
                float* const cv = sm.x.c.v[wv];
                int* const cp = sm.x.c.pos[wv];
                int have = 0;
                auto flush = [&](int least) {
                    int at = 0;
                    __builtin_amdgcn_wave_barrier();   // (a wave's LDS accesses are performed in program order)
                    while (have - at >= least && have > at) {
                        const bool in = at + lane < have;
                        classify(in ? cv[at + lane] : 0.0f, in ? cp[at + lane] : 0, in);
                        at = min(at + 64, have);
                    }
                    if (at > 0 && at < have) {   // fewer than 64 are left: to the front
                        const float v = cv[at + lane];
                        const int i = cp[at + lane];
                        __builtin_amdgcn_wave_barrier();
                        if (lane < have - at) { cv[lane] = v; cp[lane] = i; }
                    }
                    __builtin_amdgcn_wave_barrier();
                    have -= at;
                };
                each_older(ur, t0, [&](float v, int i, bool in) {
                    const bool p = in && v > least;
                    const unsigned long long m = __ballot(p);
                    const int at = have + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                    if (p) { cv[at] = v; cp[at] = i; }
                    have += (int)__popcll(m);
                }, [&] { if (have >= 64) flush(64); });
                flush(1);
            }
            if (wv == NW_CHUNK - 1) {   // own keys between the bounds of theta
                int at = 0;
                for (int c = lane; c < CHUNK; c += 64) {
                    const float tb = fmaf(sm.own[c], res, shift);
                    const bool on = c < cn && tb >= ql && tb < qh;
                    const unsigned long long m = __ballot(on);
                    if (on) sm.oc[at + (int)__popcll(m & ((1ull << lane) - 1ull))] = c;
                    at += (int)__popcll(m);
                }
                if (lane == 0) sm.no = at;
            }
            csum = wave_sum_f64(csum);
            if (lane == 0) {
                sm.wsum[wv] = csum;
                sm.wF[wv] = nF;
                sm.wC[wv] = nC;
                sm.wM[wv] = nM;
                if (nM > TL_WAVE) sm.full = 1;
            }
            __syncthreads();
            MQ = sm.nq;
            if (!sm.full && MQ <= QL_CAP) break;
        }
        // (every wave writes the same)
        sm.win = HistWindow{origin, res, covers, bounded, lo, hi};
        if (bounded) sm.known = ChunkBound{__double2float_rd(lo), true};
        else if (jl > 0 && !sm.known.tight)
            sm.known.lo = fmaxf(sm.known.lo, __double2float_rd((double)origin + (double)jl / (double)res - eps - 1.0));
        if (FIRST) return HIST_NEXT;
    }
    // totals over the waves, and this wave's place in the list
    const int tM = (int)wave_scan_u32(lane < NW_CHUNK ? (unsigned)sm.wM[lane] : 0u);
    const int M = __builtin_amdgcn_readlane(tM, NW_CHUNK - 1);
    ListBounded L;
    L.v = sm.tl;
    L.M = M;
    L.Fb = wave_sum_i32(lane < NW_CHUNK ? sm.wF[lane] : 0);
    L.Cb = wave_sum_i32(lane < NW_CHUNK ? sm.wC[lane] : 0);
    L.sumb = 0.0;
    for (int i = 0; i < NW_CHUNK; i++) L.sumb += sm.wsum[i];
    L.t0 = t0;
    L.lane = lane;
    {
        // The list in descending order, by rank (equal scores are interchangeable): sums over it then do not depend on
        // the order in which the scores arrived.  Its breakpoints (z and z - 1, where they lie between the bounds) are
        // collected at the same time, those of the chunk's own scores by waves 0 and 1, and ranked in the same way.
        if (lane < nM) sm.x.s.v[tM_before(tM, wv) + lane] = sm.raw[wv][lane];
        if (tid < 64) sm.x.s.v[M + tid] = -INFINITY;
        for (int i = tid; i < TL_CAP; i += NT_CHUNK) sm.x.s.tie[i] = 0;
        auto add = [&](bool on, double b) {
            const unsigned long long m = __ballot(on);
            if (!m) return;
            int off = 0;
            if (lane == 0) off = atomicAdd(&sm.nbp, (int)__popcll(m));
            off = __builtin_amdgcn_readfirstlane(off) + (int)__popcll(m & ((1ull << lane) - 1ull));
            if (on && off < BP_CAP) sm.x.s.bp[off] = b;
        };
        auto add_both = [&](bool real, float v) {
            add(real && v > lof && v <= hif, (double)v);
            add(real && v > lo1f && v <= hi1f, (double)v - 1.0);
        };
        if (nM > 0) add_both(lane < nM, sm.raw[wv][lane]);
        if (wv < CHUNK / 64) add_both(tid < cn, sm.own[tid]);
        if (tid < BP_CAP) sm.x.s.btie[tid] = 0;
        if (tid == 0) sm.bps[0] = lo;
        __syncthreads();
        // G lanes share the counting for one element: each takes a run of q others
        if (M > 0) {
            int G = 1;
            while (G < 16 && 2 * G * M <= NT_CHUNK) G *= 2;   // M <= NT_CHUNK: every element has its G lanes
            const int g = tid & (G - 1), e = tid / G, q = (M + 4 * G - 1) / (4 * G) * 4;
            const float v = sm.x.s.v[min(e, M - 1)];
            int rank = 0;
#pragma unroll UNROLL
            for (int j = g * q; j < min(g * q + q, M); j += 4) {
                const float4 y = *(const float4*)&sm.x.s.v[j];
                rank += (y.x > v ? 1 : 0) + (y.y > v ? 1 : 0) + (y.z > v ? 1 : 0) + (y.w > v ? 1 : 0);
            }
            for (int o = 1; o < G; o <<= 1) rank += __shfl_xor(rank, o, 64);
            if (e < M && g == 0) sm.tl[rank + atomicAdd(&sm.x.s.tie[rank], 1)] = v;
        }
    }
    const int B = sm.nbp;
    if (tid == 0 && B <= BP_CAP - 2) sm.bps[B + 1] = hi;
    if (B > 0 && B <= BP_CAP - 2) {
        int G = 1;
        while (G < 16 && 2 * G * B <= NT_CHUNK) G *= 2;
        const int g = tid & (G - 1), e = tid / G, q = (B + 2 * G - 1) / (2 * G) * 2;
        const double v = sm.x.s.bp[min(e, B - 1)];
        int rank = 0;
#pragma unroll UNROLL
        for (int j = g * q; j < min(g * q + q, B); j += 2) {
            const double2 y = *(const double2*)&sm.x.s.bp[j];
            rank += (y.x < v ? 1 : 0) + (y.y < v && j + 1 < B ? 1 : 0);
        }
        for (int o = 1; o < G; o <<= 1) rank += __shfl_xor(rank, o, 64);
        if (e < B && g == 0) sm.bps[1 + rank + atomicAdd(&sm.x.s.btie[rank], 1)] = v;
    }
    __syncthreads();
    const int TPW = (cn + NW_CHUNK - 1) / NW_CHUNK;
    const int ta = min(t1, t0 + wv * TPW), tb_ = min(t1, ta + TPW);
    if (B <= BP_CAP - 2 && M <= BP_CAP) {
        solve_parallel(sm, L, tr, ta, tb_, k, lo);
    } else {
        L.own[0] = (double)sm.own[lane];
        L.own[1] = (double)sm.own[lane + 64];
#pragma unroll
        for (int r = 0; r < TL_REG; r++) L.reg[r] = 64 * r + lane < M ? (double)sm.tl[64 * r + lane] : -INFINITY;
        wave_tau(L, tr, ta, tb_, k, lo, hi, status);
    }
    // ---- lifetimes: key j dies at the first prefix that holds k larger keys ----
    // Own keys outside the bins of theta need no counting: below them they are dead on arrival, above they outlive the chunk.
    if (wv == NW_CHUNK - 1)
        for (int c = lane; c < cn; c += 64) {
            const float tb = fmaf(sm.own[c], res, shift);
            if (tb < ql) dr[t0 + c] = j0 + t0 + c;
            else if (survivor && tb >= qh) dr[t0 + c] = survivor;
        }
    // The others, 16 lanes each: the lanes share the counting of older keys, and each looks at 8 of the chunk's own.
    // (A wave per key took 24000 cycles in the chunk of prefix k.)
    const int no = sm.no, g = tid & 15;
    for (int e = tid >> 4; e < MQ + no; e += NT_CHUNK / 16) {
        const int c = e < MQ ? -1 : sm.oc[e - MQ];
        const unsigned long long key = c < 0 ? sm.qk[e] : sm.ownkey[c];
        int older = 0;               // listed keys above this one
        for (int m = g; m < MQ; m += 16) older += sm.qk[m] > key ? 1 : 0;
        unsigned larger = 0;         // which of its own keys are above it (entries beyond the chunk are above nothing)
#pragma unroll
        for (int m = 0; m < 8; m += 2) {
            const ulonglong2 y = *(const ulonglong2*)&sm.ownkey[8 * g + m];
            larger |= (y.x > key ? 1u : 0u) << m | (y.y > key ? 2u : 0u) << m;
        }
#pragma unroll
        for (int st = 0; st < 4; st++) older += dpp_i32(older, st);
        int upto = __popc(larger);   // inclusive sum over the 16 lanes
        const int mine = upto;
        upto += SPK_DPP(upto, 0x111);
        upto += SPK_DPP(upto, 0x112);
        upto += SPK_DPP(upto, 0x114);
        upto += SPK_DPP(upto, 0x118);
        const int total = __shfl(upto, lane | 15, 64);
        const int need = k - above - older;   // the newcomer that pushes it out: the need-th larger one
        int d = -1;                           // chunk entry at which it dies
        if (need <= 0) {
            d = g == 0 ? c : -1;              // own: dead on arrival; older: out before this chunk
        } else if (need <= upto && need > upto - mine) {
            for (int x = need - (upto - mine); x > 1; x--) larger &= larger - 1u;
            d = max(8 * g + __builtin_ctz(larger), c);
        }
        const int j = key_pos(key);
        if (d >= 0) dr[j] = j0 + t0 + d;
        else if (survivor && need > total && g == 0) dr[j] = survivor;
    }
    return HIST_DONE;
}

// (not inlined: the registers of the first window stay as they are.  An instance per register budget: one for both kernels
// keeps to 64 registers in either and spills around all its loops.  us, before and with it: 32 rows of 16384 around 20 319 /
// 287, one of 32768 39.8 / 27.7, 8 of 4096 31 / 24.)
template <int OCC>
__device__ __noinline__ int mask_chunk_windows(SPK_LDS HistSmem* sm, const float* __restrict__ ur, float* __restrict__ tr,
                                               int32_t* __restrict__ dr, int t0, int t1, int k, Status status, int j0,
                                               int survivor, int tried)
{
    return mask_chunk_hist<false, OCC == 4 ? 4 : 1>(*(HistSmem*)sm, uniform_global(ur), uniform_global(tr), uniform_global(dr), uniform_int(t0),
                                  uniform_int(t1), uniform_int(k), uniform_status(status), uniform_int(j0),
                                  uniform_int(survivor), uniform_int(tried));
}

union MaskSmem {
    HistSmem h;
    SortedSmem s;
};

// What a workgroup does first: its chunk [t0, t1) of row `row`, in positions that count from the row's first valid key
// (the pointers are moved there; lifetimes count from the row's start, j0 being the difference).
struct ChunkArgs {
    const float* u;
    float* tau;
    int32_t* death;
    int n, k, t_begin;
    const int32_t* first_valid;
};
struct ChunkJob {
    const float* ur;
    float* tr;
    int32_t* dr;
    int t0, t1, j0, survivor;
};
__device__ __forceinline__ bool chunk_job(const ChunkArgs& a, int start, int len, int j0, int row, ChunkJob& J)
{
    const int t1 = min(a.n, start + len);
    if (t1 <= a.t_begin) return false;  // nobody asks for these thresholds and lifetimes
    if (j0 > start) {                   // entries before the row's start: never selected, and a finite threshold
        const int e = start + threadIdx.x;
        if (e < min(t1, j0)) {
            a.tau[(size_t)row * a.n + e] = 0.0f;
            a.death[(size_t)row * a.n + e] = e;
        }
        if (t1 <= j0) return false;
    }
    J.ur = a.u + (size_t)row * a.n + j0;
    J.tr = a.tau + (size_t)row * a.n + j0;
    J.dr = a.death + (size_t)row * a.n + j0;
    J.t0 = max(start - j0, 0);
    J.t1 = t1 - j0;
    J.j0 = j0;
    // every key's lifetime is written once: by the chunk in which it dies or, if it outlives the row, by the last chunk
    J.survivor = t1 == a.n ? a.n : 0;
    return true;
}

// k == 0 or k >= the row's length: nothing is ever selected, or nothing ever dies.  (The first chunk that is not
// skipped also writes the lifetimes of the chunks before it.)
__device__ __forceinline__ void trivial_deaths(const ChunkArgs& a, const ChunkJob& J)
{
    const int first = a.t_begin > 0 && J.t0 + J.j0 <= a.t_begin ? 0 : J.t0;
    for (int t = first + threadIdx.x; t < J.t1; t += NT_CHUNK) J.dr[t] = a.k == 0 ? J.j0 + t : a.n;
}

__device__ void window_only_chunk(float* red, const ChunkJob& J)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, cn = J.t1 - J.t0;
    float mx = -INFINITY;
    for (int i = tid; i < J.t0; i += NT_CHUNK) mx = fmaxf(mx, J.ur[i]);
    mx = wave_max_f32(mx);
    if (lane == 0) red[wv] = mx;
    __syncthreads();
    if (wv == 0)
        short_prefix_tau(wave_max_f32(lane < NW_CHUNK ? red[lane] : -INFINITY), lane < cn ? J.ur[J.t0 + lane] : -INFINITY,
                         lane + 64 < cn ? J.ur[J.t0 + lane + 64] : -INFINITY, J.t0, J.t1, 0, lane, J.tr);
}

__global__ void mask_clear_status_kernel(int* __restrict__ status) { *status = 0; }

// Rows for the attention that follows (chunked prefill).  A thread keeps its column and moves ROW_UNR rows at a time.
constexpr int ROW_UNR = 4;
__device__ void copy_rows(const RowCopy& R, int row, int wg)
{
    const int tid = threadIdx.x, per = NT_CHUNK / R.unit, col = tid % R.unit, r0 = tid / R.unit;
    if (r0 >= per) return;
    const int pad = R.rcap - R.count[row], nv = R.rcap + R.clen;
    const int first = min(pad, max(0, R.rcap - R.w - 64));
    const int step = per * ROW_UNR, runs = (nv - first + step - 1) / step;
    for (int i = wg; i < R.heads * runs; i += R.wgs) {
        const int h = i / runs, e0 = first + (i - h * runs) * step + r0;
        const size_t bh = (size_t)row * R.heads + h;
        const uint4 zero = make_uint4(0, 0, 0, 0);
        uint4 kk[ROW_UNR], vv[ROW_UNR];
#pragma unroll
        for (int x = 0; x < ROW_UNR; x++) {
            const int e = e0 + x * per;
            kk[x] = zero;
            vv[x] = zero;
            if (e < nv && e >= pad) {
                const bool own = e >= R.rcap;
                const size_t src = (own ? bh * R.clen + (e - R.rcap) : bh * R.rcap + (e - pad)) * R.unit + col;
                kk[x] = (own ? R.chunk_k : R.ret_k)[src];
                vv[x] = (own ? R.chunk_v : R.ret_v)[src];
            }
        }
#pragma unroll
        for (int x = 0; x < ROW_UNR; x++) {
            const int e = e0 + x * per;
            const size_t dst = (bh * nv + e) * R.unit + col;
            if (e < nv) {
                R.k[dst] = kk[x];
                R.v[dst] = vv[x];
            }
        }
        if (i == h * runs && first > 0 && r0 == 0) {
            R.k[bh * nv * R.unit + col] = zero;
            R.v[bh * nv * R.unit + col] = zero;
        }
    }
}

// The chunks of a row: `nchunks` of `len` prefixes each, of which `nsplit` from that of the first prefix of more than k
// entries on are dealt out in parts of `part`: thresholds move fastest there, and with them the number of scores and
// breakpoints a chunk has to look at (55000 cycles for 128 prefixes against 30000 further on).
struct ChunkDeal {
    int nchunks, len, nsplit, part;
    int shared_status;   // one status word for all chunks, cleared ahead of the kernel; else 8 bits per PART prefixes
    __host__ __device__ int most() const { return nchunks + nsplit * (len / part - 1); }   // workgroups per row
};
constexpr int PART = 32;   // lengths of chunks and parts are multiples of it
constexpr int CUS = 256;   // compute units

// OCC: waves per SIMD.  4: a compute unit's registers for one workgroup (nothing spilled); 8: two workgroups share it (76 KB
// of LDS, 64 registers).
template <int OCC>
__global__ __launch_bounds__(NT_CHUNK, OCC) void mask_kernel(ChunkArgs a, ChunkDeal deal, int* __restrict__ status, RowCopy rows)
{
    __shared__ __align__(16) MaskSmem sm;
    const int row = blockIdx.y, most = deal.most();
    if ((int)blockIdx.x >= most) {
        if ((int)blockIdx.x - most < rows.wgs) copy_rows(rows, row, blockIdx.x - most);
        return;
    }
    const int j0 = a.first_valid ? a.first_valid[row] : 0;
    int len = deal.len;
    const int parts = len / deal.part, first = min((a.k + j0) / len, deal.nchunks);
    const int nsplit = min(deal.nsplit, deal.nchunks - first);
    // Late chunks have the longest prefixes: they go first.  In a single round those of prefixes of at most k entries, which
    // end at once, make room ahead of them; in several they fill the last one.
    const int id = blockIdx.x, total = deal.nchunks + nsplit * (parts - 1), ahead = OCC == 4 ? first : 0;
    if (id >= total) return;
    const int c = id < ahead ? id : total - 1 - (id - ahead);
    int start = c * len;
    if (c >= first + nsplit * parts) {
        start = (c - nsplit * (parts - 1)) * len;
    } else if (c >= first) {
        start = first * len + (c - first) * deal.part;
        len = deal.part;
    }
    if (start >= a.n) return;   // (parts of the last chunk)
    Status st{status, 1};
    if (!deal.shared_status) {
        const int words = (a.n + CHUNK - 1) / CHUNK;
        unsigned char* const bytes = (unsigned char*)(status + (size_t)row * words);
        const int p = start / PART + threadIdx.x, end = start + len >= a.n ? words * (CHUNK / PART) : (start + len) / PART;
        if (p < end) bytes[p] = 0;
        st.word = (int*)bytes + start / CHUNK;
        st.bit = 1 << start % CHUNK / PART * 8;
    }
    ChunkJob J;
    if (!chunk_job(a, start, len, j0, row, J)) return;
    if (a.k == 0 || a.n - J.j0 <= a.k) trivial_deaths(a, J);
    if (a.k == 0) { window_only_chunk((float*)&sm, J); return; }
    int how = mask_chunk_begin(sm.h, J.ur, J.tr, J.t0, J.t1, a.k), tried = 0;
    if (how == HIST_FIRST) {
        how = mask_chunk_hist<true, OCC == 4 ? 4 : 1>(sm.h, J.ur, J.tr, J.dr, J.t0, J.t1, a.k, st, J.j0, J.survivor, 0);
        tried = 1;
    }
    if (how == HIST_NEXT)
        how = mask_chunk_windows<OCC>((SPK_LDS HistSmem*)&sm.h, J.ur, J.tr, J.dr, J.t0, J.t1, a.k, st, J.j0, J.survivor, tried);
    if (how == HIST_DONE) return;
    const ChunkBound known = sm.h.known;
    __syncthreads();
    mask_chunk_sorted((SPK_LDS SortedSmem*)&sm.s, J.ur, J.tr, J.dr, J.t0, J.t1, a.k, st, J.j0, J.survivor, known);
}

// ---------------------------------------------------------------------------------
// Short sequences.  The kernel above is a chain of a dozen dependent phases of a 1024-thread workgroup, 14 us however short
// the row.  Here a wave solves one prefix on its own, with the row's scores in LDS: a regula falsi in fp32 (a subtraction
// with clamp and an addition per score and step) ends within half a score of the root, the exact iteration finishes, and
// a key above its own threshold counts the larger ones.  One barrier.  Two prefixes or four per wave share the first part,
// but the wave is then the longer chain: one row of 1024 in 10.5, 12.7 and 16.2 us.  The work grows with the square of the
// length: see launch_mask for the line.  Both parts stop where rounding leaves nothing to gain; scores around 1e5, where fp32
// numbers lie 2^-7 apart, took 42 us for one row of 2000 and 48 for 4 of 1024 before, 14 and 12 with it (12.8 and 11.7
// around 0).
// ---------------------------------------------------------------------------------
constexpr int SMALL_WAVES = 4;
constexpr long long SMALL_WORK = 1ll << 22;   // rows times the square of their length
constexpr long long SMALL_LOAD = 20 << 10;     // rows times their length; any number of rows of up to SMALL_ROW
constexpr int SMALL_ROW = 48;
constexpr int SMALL_MAX = 2048;    // scores of a row, hence
constexpr int FALSI_ITERS = 20;
constexpr int NEWTON_ITERS = 64;   // beyond, only the middle of the bracket, which closes after some 2000 steps at most

// The scores of a prefix: positions before t0 in LDS, from t0 on one per lane.
struct ListRow {
    const float* v;
    int t0, lane;
    float own;
};

// f(four scores) for the positions before end (a multiple of 4), 256 at a time; `none` fills up.  (UNROLL 1 where f counts with
// ballots: the compiler unrolls no such loop of unknown length.)
template <int UNROLL, typename F>
__device__ __forceinline__ void each_row4(const float* v, int end, int lane, float none, F&& f)
{
    const float4* v4 = (const float4*)v;
    int i = 0;
#pragma unroll UNROLL
    for (; i + 256 <= end; i += 256) f(v4[(i >> 2) + lane]);
    if (i < end) f(i + 4 * lane < end ? v4[(i >> 2) + lane] : make_float4(none, none, none, none));
}

__device__ __forceinline__ PieceB eval_bounded(const ListRow& L, int t, double x)
{
    // (for an fp32 score v: v > x <=> v > rd(x))
    const float xf = __double2float_rd(x), x1f = __double2float_rd(x + 1.0);
    int F = 0, S = 0;
    double part = 0.0;
    auto one = [&](float v) {
        const unsigned long long a = __ballot(v > xf), b = __ballot(v > x1f);
        S += (int)__popcll(a);
        F += (int)__popcll(b);
        part += v > xf && !(v > x1f) ? (double)v : 0.0;
    };
    each_row4<1>(L.v, L.t0, L.lane, -INFINITY, [&](float4 z) { one(z.x); one(z.y); one(z.z); one(z.w); });
    one(L.lane <= t - L.t0 ? L.own : -INFINITY);
    return PieceB{F, S, wave_sum_f64(part)};
}

__device__ __forceinline__ double min_saturated(const ListRow& L, int t, double x)
{
    const float x1f = __double2float_rd(x + 1.0);
    float mf = INFINITY;
    auto one = [&](float v) { mf = fminf(mf, v > x1f ? v : INFINITY); };
    each_row4<2>(L.v, L.t0, L.lane, -INFINITY, [&](float4 z) { one(z.x); one(z.y); one(z.z); one(z.w); });
    one(L.lane <= t - L.t0 ? L.own : -INFINITY);
    return (double)wave_min_f32(mf);
}

// A point near the threshold of prefix t, between lo (f_t(lo) >= k) and hi (f_t(hi) < k); `count` scores are above lo.
__device__ __forceinline__ float near_threshold(const ListRow& L, int t, int k, int count, float lo, float hi)
{
    const float want = (float)k + 0.5f;
    float a = lo, b = hi, fa = (float)count - want, fb = -want, x = lo;
    int side = 0;
    for (int it = 0; it < FALSI_ITERS; it++) {
        x = fmaf((b - a) * fa, __builtin_amdgcn_rcpf(fa - fb), a);
        if (!uniform(x > a && x < b)) {
            x = 0.5f * a + 0.5f * b;
            if (!uniform(x > a && x < b)) break;   // no fp32 number lies between them
        }
        float s0 = L.lane <= t - L.t0 ? clip01(L.own - x) : 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
        each_row4<2>(L.v, L.t0, L.lane, -INFINITY, [&](float4 z) {
            s0 += clip01(z.x - x);
            s1 += clip01(z.y - x);
            s2 += clip01(z.z - x);
            s3 += clip01(z.w - x);
        });
        const float f = wave_sum_f32((s0 + s1) + (s2 + s3)) - want;
        if (uniform(fabsf(f) <= 0.5f)) break;
        if (uniform(f > 0.0f)) {      // (the end that stays counts half from the second time on: Illinois)
            a = x;
            fa = f;
            if (side > 0) fb *= 0.5f;
            side = 1;
        } else {
            b = x;
            fb = f;
            if (side < 0) fa *= 0.5f;
            side = -1;
        }
    }
    return x;
}

// The threshold of prefix t, in [lo, hi); x: a point to start from.  The iteration of solve_tau, with an upper end.
__device__ __forceinline__ double solve_row(const ListRow& L, int t, int k, double x, double lo, double hi)
{
    PieceB P = eval_bounded(L, t, x);
    for (int it = 0;; it++) {
        const double f = (double)P.F + P.fsum - (double)(P.S - P.F) * x;
        const bool left = uniform(!(f < (double)k));
        double xn = x;
        bool step = false, piece = false;   // take xn; xn is the root of the piece
        if (left) lo = x;
        else hi = x;
        if (P.S > P.F) {
            xn = (P.fsum + (double)P.F - (double)k) / (double)(P.S - P.F);
            if (left ? !uniform(xn > x) : !uniform(xn < x)) return x;   // f(x) == k up to rounding
            step = piece = uniform(xn >= lo && xn < hi);
        } else if (left) {                  // flat to the right of x, f == F there
            xn = min_saturated(L, t, x) - 1.0;        // the next breakpoint
            if (P.F == k && uniform(xn < hi)) return xn;   // sup of the level set f == k
            step = uniform(xn < hi);
        }
        if (!step || it >= NEWTON_ITERS) {
            xn = 0.5 * (lo + hi);
            piece = false;
            if (!uniform(xn > lo && xn < hi)) return lo;
        }
        const PieceB Q = eval_bounded(L, t, xn);
        if (piece && Q.F == P.F && Q.S == P.S) return xn;
        P = Q;
        x = xn;
    }
}

__global__ __launch_bounds__(64 * SMALL_WAVES) void mask_small_kernel(const float* __restrict__ u, float* __restrict__ tau,
                                                                      int32_t* __restrict__ death, int n, int k,
                                                                      int* __restrict__ status)
{
    __shared__ __align__(16) float row_scores[SMALL_MAX];
    const int row = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int last = (n + SMALL_WAVES - 1) / SMALL_WAVES - 1;
    if ((int)blockIdx.x > last) return;
    const int t = (last - (int)blockIdx.x) * SMALL_WAVES + wv;   // late prefixes are the longest: first
    const float* ur = u + (size_t)row * n;
    // (the status words are never set: solve_row ends by itself)
    if (t % CHUNK == 0 && lane == 0 && t < n) status[(size_t)row * ((n + CHUNK - 1) / CHUNK) + t / CHUNK] = 0;
    for (int i = tid; i < (n + 255) / 256 * 256; i += 64 * SMALL_WAVES) row_scores[i] = i < n ? ur[i] : -INFINITY;
    __syncthreads();
    if (t >= n) return;
    ListRow L;
    L.v = row_scores;
    L.t0 = t & ~3;
    L.lane = lane;
    L.own = L.t0 + lane <= t ? row_scores[L.t0 + lane] : -INFINITY;
    const bool older = L.t0 + lane < t;             // positions before t among the wave's own
    const float v = readlane_f32(L.own, t - L.t0);  // the score of position t
    // ---- threshold ----
    // of the finite scores: the smallest and the largest
    float mn = L.t0 + lane <= t ? L.own : INFINITY, mx = L.own;
    each_row4<2>(row_scores, L.t0, lane, NAN, [&](float4 z) {
        mn = fminf(mn, fminf(fminf(z.x, z.y), fminf(z.z, z.w)));
        mx = fmaxf(mx, fmaxf(fmaxf(z.x, z.y), fmaxf(z.z, z.w)));
    });
    mn = wave_min_f32(mn);
    mx = wave_max_f32(mx);
    float res = mn - 1.0f;                          // of at most k entries
    if (t >= k) {
        int count = t + 1, infs = 0;
        if (uniform(!(mn > -INFINITY && mx < INFINITY))) {
            count = 0;
            mn = INFINITY;
            mx = -INFINITY;
            auto one = [&](float z) {
                count += (int)__popcll(__ballot(z > -INFINITY));
                infs += (int)__popcll(__ballot(z == INFINITY));
                if (fabsf(z) < INFINITY) { mx = fmaxf(mx, z); mn = fminf(mn, z); }
            };
            each_row4<1>(row_scores, L.t0, lane, -INFINITY, [&](float4 z) { one(z.x); one(z.y); one(z.z); one(z.w); });
            one(L.own);
            mn = wave_min_f32(mn);
            mx = wave_max_f32(mx);
        }
        if (count < k) {          // f < k everywhere
            res = -INFINITY;
        } else if (infs >= k) {   // f >= k everywhere: the sup of all points
            res = INFINITY;
        } else {
            const float x = near_threshold(L, t, k, count, mn - 1.0f, mx);
            res = (float)solve_row(L, t, k, (double)x, (double)mn - 1.0, (double)mx);
        }
    }
    // ---- lifetime of key t ----
    // Below its own threshold it is not among the k largest on arrival: tau < z_(k).  (res is rounded to fp32: no fp32
    // number lies between it and the threshold.)
    int d = t;
    if (t < k || uniform(v >= res)) {
        int need = k - (int)__popcll(__ballot(older && L.own >= v));
        each_row4<1>(row_scores, L.t0, lane, NAN, [&](float4 z) {
            need -= (int)(__popcll(__ballot(z.x >= v)) + __popcll(__ballot(z.y >= v)) + __popcll(__ballot(z.z >= v)) +
                          __popcll(__ballot(z.w >= v)));
        });
        if (need > 0) {           // the need-th larger newcomer pushes it out
            d = n;
            for (int i = t / 256 * 256; i < n; i += 256) {
                const int j = i + 4 * lane;
                const float4 z = *(const float4*)&row_scores[j];
                const int more = (int)(__popcll(__ballot(j > t && z.x > v)) + __popcll(__ballot(j + 1 > t && z.y > v)) +
                                       __popcll(__ballot(j + 2 > t && z.z > v)) + __popcll(__ballot(j + 3 > t && z.w > v)));
                if (need > more) {
                    need -= more;
                    continue;
                }
                for (int j0 = i; j0 < i + 256; j0 += 64) {
                    const unsigned long long b = __ballot(j0 + lane > t && row_scores[j0 + lane] > v);
                    const int got = (int)__popcll(b);
                    if (need <= got) {
                        const int before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0));
                        d = j0 + (int)__builtin_ctzll(__ballot((b >> lane & 1ull) && before == need - 1));
                        break;
                    }
                    need -= got;
                }
                break;
            }
        }
    }
    if (lane == 0) {
        tau[(size_t)row * n + t] = res;
        death[(size_t)row * n + t] = d;
    }
}

// ---------------------------------------------------------------------------------
// Explicit top-k lists (verification aid): one workgroup per (prefix, row).
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void materialize_kernel(const float* __restrict__ u,
                                                          const float* __restrict__ tau,
                                                          const int32_t* __restrict__ death, int n, int k,
                                                          int t_begin, int nt, int32_t* __restrict__ idx,
                                                          float* __restrict__ gate)
{
    __shared__ int wcount[4];
    __shared__ int base;
    const int t = t_begin + blockIdx.x, row = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const float* ur = u + (size_t)row * n;
    const int32_t* dr = death + (size_t)row * n;
    const float tt = tau[(size_t)row * n + t];
    int32_t* io = idx + ((size_t)row * nt + blockIdx.x) * k;
    float* go = gate ? gate + ((size_t)row * nt + blockIdx.x) * k : nullptr;
    if (tid == 0) base = 0;
    __syncthreads();
    for (int j0 = 0; j0 <= t; j0 += 256) {
        int j = j0 + tid;
        bool p = (j <= t) && (dr[j] > t);
        unsigned long long ball = __ballot(p);
        if (lane == 0) wcount[wv] = __popcll(ball);
        __syncthreads();
        int off = base;
        for (int i = 0; i < wv; i++) off += wcount[i];
        if (p) {
            int o = off + __popcll(ball & ((1ull << lane) - 1ull));
            if (o < k) {
                io[o] = j;
                if (go) go[o] = clip01(ur[j] - tt);
            }
        }
        __syncthreads();
        if (tid == 0) base += wcount[0] + wcount[1] + wcount[2] + wcount[3];
        __syncthreads();
    }
    for (int o = base + tid; o < k; o += 256) {
        io[o] = -1;
        if (go) go[o] = 0.0f;
    }
}

// A workgroup per compute unit at a time: do they get one each, all but the first `idle` of every row, which end at once?
// Workgroups go to GROUPS groups of compute units in turn, and one too many in a group waits for a whole chunk: 9 rows of 3500
// at k = 256 take 34 us with the chunks around prefix k split and 27 without, 16 of 2048 33 with two of them split, 24 with
// one.  One that waits for an idle one starts late, which shows where rows are many or a group has nothing to spare (30 rows
// of 1024 at k = 128, 8.4 per group: 33 us, 27 with 7.5) and does not pay without a split (6 rows of 5425 at k = 256: 29 us, 26 in
// two rounds of split chunks).
constexpr int GROUPS = 32;
static bool fits_one_round(const ChunkDeal& deal, int nrows, int idle)
{
    const int per_row = deal.most();
    const long long total = (long long)nrows * per_row;
    if (total > CUS + (deal.nsplit > 0 ? CUS / 8 : 0)) return false;
    int load[GROUPS] = {}, most = 0;
    for (int r = 0; r < nrows; r++)
        for (int i = idle; i < per_row; i++) most = std::max(most, ++load[(r * per_row + i) % GROUPS]);
    return most <= CUS / GROUPS - (total > CUS + (nrows <= 16 ? CUS / 16 : 0) ? 1 : 0);
}

int launch_mask(const sparsek_cfg& c, const float* u, float* tau, int32_t* death, void* ws,
                hipStream_t st, int t_begin, const int32_t* first_valid, const RowCopy* rows)
{
    const int nrows = c.B * c.Gu;
    // us, this kernel against the chunks: one row of 500 8.5 / 14.3, of 1024 10.5 / 14.6, of 2000 13.0 / 14.6, of 3000 17.4 /
    // 14.4; four rows of 1024 12.6 / 14.6; 16 of 512 15.0 / 14.8; two of 2000 15.5 / 14.6.  Many shorter rows fill the chip (8192
    // waves) more than twice at a smaller square: 160 of 100 17.2 / 18.5, 240 22.6 / 18.4; 125 of 128 17.2 / 15.3 (k = 64: 14.7 /
    // 18.3), 187 22.6 / 20.7; 266 of 60 16.7 / 21.8, 666 32.8 / 32.3.  Up to some 48 prefixes a workgroup of 16 waves has too
    // little to do: 1333 of 30 33.3 / 47.0, 869 of 46 32.6 / 37.2.
    if (!rows && !first_valid && t_begin == 0 && c.k >= 1 && c.n > c.k && c.n <= SMALL_MAX &&
        (long long)nrows * c.n * c.n <= SMALL_WORK && (c.n <= SMALL_ROW || (long long)nrows * c.n <= SMALL_LOAD)) {
        // (an odd number of workgroups per row where not all have room at once, as below: 256 rows of 64 at k = 32 19.0 -> 14.5
        // us, 128 of 128 at k = 64 20.5 -> 14.9)
        const int quads = (c.n + SMALL_WAVES - 1) / SMALL_WAVES, odd = (long long)nrows * quads > 8 * CUS ? 1 : 0;
        hipLaunchKernelGGL(mask_small_kernel, dim3(quads | odd, nrows), dim3(64 * SMALL_WAVES), 0, st, u, tau, death, c.n, c.k,
                           (int*)ws);
        return launch_status();
    }
    const ChunkArgs a{u, tau, death, c.n, c.k, t_begin, first_valid};
    const bool shared = mask_shared_status(c);
    // With no more workgroups than compute units nothing shares a compute unit, and the time is that of the slowest chunk:
    // as short as fits (4 rows of 2000 at k = 128: chunks of 128 in 25 us, 64 in 16.4, 32 in 15.0; 2 rows of 5003: 22.8,
    // 17.5 and, beyond one round, 27).  Longer ones keep 128 prefixes, split where thresholds move fastest (8 rows of 4096:
    // 27.3 -> 22 us) while that still is one round (fits_one_round).  Workgroups of 64 registers, two per compute unit, take over where one
    // round does not do (32 rows of 16384: 211 us against 310 with one per compute unit); chunks are split there too (100
    // rows of 4000 at k = 1000: 186 -> 169 us, now 154) unless that takes the second or third round of workgroups (256 rows of 512:
    // 56 us, 66 in three) or, in more rounds, adds more than an eighth to them: there it is their number that counts (1100
    // rows of 100 at k = 12: 84 us with two parts, 64 without, 2048 of 511 at k = 64: 408 and 359).  Row copies need the rest of
    // the chip: chunks stay long beside them.
    ChunkDeal deal{0, CHUNK, 2, 64, shared ? 1 : 0};
    if (!rows && (long long)nrows * ((c.n + 31) / 32) <= CUS) deal = ChunkDeal{0, 32, 0, 32, 0};
    else if (!rows && (long long)nrows * ((c.n + 63) / 64 + 2) <= CUS) deal = ChunkDeal{0, 64, 2, 32, 0};
    deal.nchunks = (c.n + deal.len - 1) / deal.len;
    if (!first_valid) {   // no parts that hold nothing (1500 rows of 64: 73 us, 60 without)
        const int first = std::min(c.k / deal.len, deal.nchunks);
        deal.nsplit = std::min(deal.nsplit, deal.nchunks - first);
        if (deal.nsplit > 0 && first + deal.nsplit == deal.nchunks && c.n - (deal.nchunks - 1) * deal.len <= deal.part) deal.nsplit--;
    }
    const int idle = t_begin > 0 ? t_begin / deal.len : std::min(c.k, c.n) / deal.len;   // chunks that end at once
    const long long whole = (long long)nrows * (deal.nchunks - idle), split = (long long)nrows * (deal.most() - idle);
    const int asked = deal.nsplit;
    while (deal.nsplit > 0 && !fits_one_round(deal, nrows, idle)) deal.nsplit--;
    const bool one_round = fits_one_round(deal, nrows, idle);
    if (!one_round) deal.nsplit = asked;
    if (!one_round && ((whole <= 2 * CUS && split > 2 * CUS) || (whole <= 4 * CUS && split > 4 * CUS) ||
                       (whole > 4 * CUS && 8 * deal.nsplit > deal.nchunks - idle)))
        deal.nsplit = 0;
    RowCopy R{};
    if (rows) {
        // The chunks are bound by latency and, with one score row, few: the rows are moved by what is left of the chip
        // meanwhile, in pieces small enough that no compute unit is left with a long one (1024 workgroups: 32 K tokens in
        // chunks of 8192 in 1609 us, 512: 1633, 256: 1660).  With many score rows a few workgroups follow each of them.
        R = *rows;
        const int step = NT_CHUNK / R.unit * ROW_UNR;
        const long long most = (long long)R.heads * ((R.rcap + R.clen + step - 1) / step);
        const long long free = (1024 - (long long)nrows * (deal.most() - idle)) / nrows;
        R.wgs = (int)std::min(most, std::max(free, 8ll));
    }
    if (shared) hipLaunchKernelGGL(mask_clear_status_kernel, dim3(1), dim3(1), 0, st, (int*)ws);
    // Workgroups go to the chip's 8 partitions in turn, and there to 4 groups of 8 compute units: with a multiple of 4 per row
    // every partition would get the same chunks of all rows, and the dispatch, once it has to wait for room, waits for the one
    // with the long ones.  An odd number is the best of the small ones (2048 rows of 400 at k = 200 take 454 us with 4 per row,
    // 322 with 5, 350 with 6, 890 with 8), and next to a multiple of 32 the rows move on too little (150 rows of 3830 at
    // k = 821 with 30 to 34: 212, 221, 316, 244, 213).  Where all have room at once, or fill it exactly twice, empty ones would
    // only take it away (21 rows of 3000 at k = 50 with 24: 26 us, 25: 34; 256 of 512 with 4: 55, 5: 59).
    int per_row = deal.most() + R.wgs;
    const long long total = (long long)nrows * per_row, room = (one_round ? 1 : 2) * CUS;
    auto poor = [](int p) { return p < 30 ? p > 1 && p % 2 == 0 : p % 4 == 0 || (p + 1) % 32 <= 2; };
    while (total > room && (total != 2 * room || per_row >= 8) && poor(per_row)) per_row++;
    const dim3 grid(per_row, nrows);
    if (one_round) hipLaunchKernelGGL(mask_kernel<4>, grid, dim3(NT_CHUNK), 0, st, a, deal, (int*)ws, R);
    else hipLaunchKernelGGL(mask_kernel<8>, grid, dim3(NT_CHUNK), 0, st, a, deal, (int*)ws, R);
    return launch_status();
}

int mask_status(const sparsek_cfg& c, const void* ws, int32_t* host_flag, hipStream_t st)
{
    int32_t words[STATUS_WORDS];
    const size_t count = mask_shared_status(c) ? 1 : mask_chunks(c);
    if (hipMemcpyAsync(words, ws, count * sizeof(int32_t), hipMemcpyDeviceToHost, st) != hipSuccess)
        return SPARSEK_ERR_LAUNCH;
    if (hipStreamSynchronize(st) != hipSuccess) return SPARSEK_ERR_LAUNCH;
    *host_flag = 0;
    for (size_t i = 0; i < count; i++) *host_flag |= words[i] | words[i] >> 8 | words[i] >> 16 | words[i] >> 24;
    *host_flag &= 0xFF;   // (a byte per part of a chunk)
    return SPARSEK_OK;
}

int launch_materialize(const sparsek_cfg& c, const float* u, const float* tau, const int32_t* death,
                       int t_begin, int t_end, int32_t* idx, float* gate, hipStream_t st)
{
    const int rows = c.B * c.Gu;
    const int nt = t_end - t_begin;
    if (nt == 0 || c.k == 0) return SPARSEK_OK;
    hipLaunchKernelGGL(materialize_kernel, dim3(nt, rows), dim3(256), 0, st, u, tau, death, c.n, c.k,
                       t_begin, nt, idx, gate);
    return launch_status();
}

}  // namespace spk
