// Constant-memory decode step (Sec. 3.2 irreversibility, Sec. 3.3 incremental SPARSEK).
//
// State per score row (b,g): the scores of the w window keys (a ring), of the <= k selected
// keys, and of every other key still above tau (the set S of the incremental algorithm minus
// the top-k), plus tau itself in fp64.  State per head (b,h): k+w key/value slots.  A key keeps
// its slot from the moment it is appended until it is dropped; selection only changes the
// per-slot gate score (+inf = window key, gate 1; finite = selected key, gate
// clip(u - tau, 0, 1); -inf = empty), so one step moves no K/V rows except the new token's.
//
// One step = one launch.  What a step changes in a score row -- tau, the slot that becomes empty, the gate of the key that
// leaves the window, the new token's slot -- depends on earlier tokens only (w > 0), so every step finds it ready in a
// record and leaves that of the next one: the first workgroups of the grid, one per score row, update tau / top-k /
// candidates for the key that leaves the window in the step after this one (dependent loads, 7 to 20 us), while the others
// stream the k+w slots of a head (HBM-bound), or a share of them when there are few heads, and the one that holds the new
// token's slot stores its K/V rows.  No workgroup waits for one that may not have been dispatched yet: an order of dispatch
// holds within one XCD only.  Without a window (w == 0) the new token's own score decides, and the update runs ahead of
// the heads in a launch of its own.
#include "common.hpp"

namespace spk {

// What a step changes for the attention of one score row.
struct StepRecord {
    float tau;
    int evicted;      // the slot that becomes empty, -1: none
    int left;         // the slot of the key that leaves the window, -1: none,
    float left_u;     // and its gate score from now on
    int fresh;        // the new token's slot, -1: it has none,
    float fresh_u;    // and its gate score
    int pad[2];
};
struct RowSync {
    StepRecord rec[2];          // step s finds its record in rec[s & 1]
    unsigned long long step;    // steps that are over: counted by the last workgroup of the row to finish
    unsigned finished, pad;     // heads of the row, and its own workgroup, that are through with this step
    unsigned long long pad2[6];
};
static_assert(sizeof(RowSync) == 128, "one cache line per row");

struct DecodeLayout {
    int rows, NS, cap, wlen, klen;
    size_t pos, nsel, ncand, status, nfree, tau_d;
    size_t win_u, win_slot, sel_u, sel_pos, sel_slot, cand_u, slot_u, free_stack, kslots, vslots, sync, heads, part, total;
    int nsplit;
};

__host__ __device__ inline DecodeLayout decode_layout(const sparsek_decode_cfg& c)
{
    DecodeLayout L;
    L.rows = c.B * c.Gu;
    L.NS = c.k + c.w;
    L.cap = c.cand_cap > 0 ? c.cand_cap : 4 * (c.k > 16 ? c.k : 16);
    L.wlen = c.w > 0 ? c.w : 1;
    L.klen = c.k > 0 ? c.k : 1;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = (off + bytes + 255) / 256 * 256;
        return o;
    };
    const size_t r = (size_t)L.rows;
    L.pos = take(r * 4);
    L.nsel = take(r * 4);
    L.ncand = take(r * 4);
    L.status = take(r * 4);
    L.nfree = take(r * 4);
    L.tau_d = take(r * 8);
    L.win_u = take(r * L.wlen * 4);
    L.win_slot = take(r * L.wlen * 4);
    L.sel_u = take(r * L.klen * 4);
    L.sel_pos = take(r * L.klen * 4);
    L.sel_slot = take(r * L.klen * 4);
    L.cand_u = take(r * (size_t)L.cap * 4);
    L.slot_u = take(r * (size_t)L.NS * 4);
    L.free_stack = take(r * (size_t)L.NS * 4);
    const size_t esz = c.dtype == SPARSEK_BF16 ? 2 : 4;
    const size_t kv = (size_t)c.B * c.H * L.NS * c.d * esz;
    L.kslots = take(kv);
    L.vslots = take(kv);
    // A head's slots are dealt to nsplit workgroups: up to four per compute unit when there are few heads, but at least
    // 128 KB of K and V each (adding the shares up costs 3 us).
    const long long heads = (long long)c.B * c.H, bytes = 2ll * L.NS * c.d * (long long)esz;
    const long long want = (1024 + heads - 1) / heads, most = bytes >> 17 > 1 ? bytes >> 17 : 1;
    L.nsplit = (int)(want < most ? want : most);
    L.sync = take(r * sizeof(RowSync));
    L.heads = take((size_t)heads * 4);
    L.part = take(L.nsplit > 1 ? (size_t)heads * L.nsplit * (c.d + 2) * 8 : 0);
    L.total = off;
    return L;
}

size_t decode_state_bytes(const sparsek_decode_cfg& c) { return decode_layout(c).total; }

struct RowState {
    int *pos, *nsel, *ncand, *status, *nfree;
    double* tau_d;
    float* win_u;
    int* win_slot;
    float* sel_u;
    int *sel_pos, *sel_slot;
    float *cand_u, *slot_u;
    int* free_stack;
    RowSync* sync;
};

__device__ inline RowState row_state(char* st, const DecodeLayout& L, int row)
{
    RowState R;
    R.pos = (int*)(st + L.pos) + row;
    R.nsel = (int*)(st + L.nsel) + row;
    R.ncand = (int*)(st + L.ncand) + row;
    R.status = (int*)(st + L.status) + row;
    R.nfree = (int*)(st + L.nfree) + row;
    R.tau_d = (double*)(st + L.tau_d) + row;
    R.win_u = (float*)(st + L.win_u) + (size_t)row * L.wlen;
    R.win_slot = (int*)(st + L.win_slot) + (size_t)row * L.wlen;
    R.sel_u = (float*)(st + L.sel_u) + (size_t)row * L.klen;
    R.sel_pos = (int*)(st + L.sel_pos) + (size_t)row * L.klen;
    R.sel_slot = (int*)(st + L.sel_slot) + (size_t)row * L.klen;
    R.cand_u = (float*)(st + L.cand_u) + (size_t)row * L.cap;
    R.slot_u = (float*)(st + L.slot_u) + (size_t)row * L.NS;
    R.free_stack = (int*)(st + L.free_stack) + (size_t)row * L.NS;
    R.sync = (RowSync*)(st + L.sync) + row;
    return R;
}

constexpr int NT_ROW = 256;

// ---- block-wide reductions over NT_ROW threads (all threads get the result) ----
struct BlockRed {
    unsigned long long u64[NT_ROW / 64];
    double f64[NT_ROW / 64];
    float f32[NT_ROW / 64];
};

__device__ inline void block_eval(BlockRed& red, const float* a, int na, const float* b, int nb, double x, int& F, int& S,
                                  double& fsum, float& minF)
{
    // right-limit counts of the piece of f that starts at x, over a[0..na) U b[0..nb)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int f = 0, s = 0;
    double sum = 0.0;
    float mf = INFINITY;
    const double x1 = x + 1.0;
    auto add = [&](float v) {
        double dv = (double)v;
        if (dv > x) {
            s++;
            if (dv > x1) { f++; mf = fminf(mf, v); }
            else sum += dv;
        }
    };
    for (int i = tid; i < na; i += NT_ROW) add(a[i]);
    for (int i = tid; i < nb; i += NT_ROW) add(b[i]);
    unsigned long long packed = wave_sum_u64(((unsigned long long)f << 32) | (unsigned long long)s);
    double ws = wave_sum_f64(sum);
    float wm = wave_min_f32(mf);
    __syncthreads();
    if (lane == 0) { red.u64[wv] = packed; red.f64[wv] = ws; red.f32[wv] = wm; }
    __syncthreads();
    packed = 0;
    ws = 0.0;
    wm = INFINITY;
    for (int i = 0; i < NT_ROW / 64; i++) { packed += red.u64[i]; ws += red.f64[i]; wm = fminf(wm, red.f32[i]); }
    F = (int)(packed >> 32);
    S = (int)(packed & 0xFFFFFFFFull);
    fsum = ws;
    minF = wm;
}

// Same iteration as the prefill solver: tau <- (fsum + F - k)/(S - F), the root of the linear piece
// through the current point (from whichever side of the root it lies on), until (F, S) reproduce;
// a bracket of the root is kept and a step that leaves it is replaced by its midpoint.
template <typename Eval>
__device__ double solve_tau_iter(Eval&& eval, int k, double start, int* status)
{
    double lo_b = start, hi_b = INFINITY, x = start;
    int pF = -1, pS = -1;
    for (int it = 0; it < 4096; it++) {
        int F, S;
        double fsum;
        float minF;
        eval(x, F, S, fsum, minF);
        if (F == pF && S == pS) return x;
        pF = pS = -1;
        const double f = (double)F + fsum - (double)(S - F) * x;
        double xn = 0.0;
        bool have = false;
        if (f < (double)k) {
            hi_b = x;  // x is right of the root
            if (S > F) { xn = (fsum + (double)F - (double)k) / (double)(S - F); have = true; }
        } else {
            lo_b = x;
            if (S == F) {  // flat to the right of x, f == F there
                if (F == k) return (double)minF - 1.0;  // sup of the level set f == k
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
    if (threadIdx.x == 0) atomicOr(status, 2);
    return x;
}

// In-place, order-preserving removal of candidates <= tau.  Returns the new count.
__device__ int block_prune(int* scan, float* cand, int n, double tau)
{
    const int tid = threadIdx.x;
    __shared__ int base_s;
    if (tid == 0) base_s = 0;
    __syncthreads();
    for (int i0 = 0; i0 < n; i0 += NT_ROW) {
        const int i = i0 + tid;
        float v = (i < n) ? cand[i] : 0.0f;
        const bool keep = (i < n) && ((double)v > tau);
        const unsigned long long ball = __ballot(keep);
        const int lane = tid & 63, wv = tid >> 6;
        if (lane == 0) scan[wv] = __popcll(ball);
        __syncthreads();
        int off = base_s;
        for (int x = 0; x < wv; x++) off += scan[x];
        const int dst = off + __popcll(ball & ((1ull << lane) - 1ull));
        __syncthreads();  // all reads of this batch done before anyone writes (dst <= i always)
        if (keep) cand[dst] = v;
        if (tid == 0) base_s += scan[0] + scan[1] + scan[2] + scan[3];
        __syncthreads();
    }
    return base_s;
}

// ---------------------------------------------------------------------------------
// (1) per score row: the step under way appends its token to the window; the key that the next step takes out of it joins
// the SPARSEK prefix, and the next token gets the freed slot.  A chain of dependent loads on an otherwise idle workgroup, so everything that can be
// fetched before anything is known is fetched first: the selected keys and the candidates (up to SEL_REG / CAND_REG
// per thread in registers, the rest is read again where it is needed).
// ---------------------------------------------------------------------------------
constexpr int SEL_REG = 4, CAND_REG = 8;

struct RowRegs {
    float su[SEL_REG], cu[CAND_REG];
    int sp[SEL_REG];
};

// Right-limit counts of the piece of f that starts at x, over the selected keys, the candidates and z.
__device__ inline void row_eval(BlockRed& red, const RowRegs& G, const RowState& R, int nsel, int ncand, float z, double x,
                                int& F, int& S, double& fsum, float& minF)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int f = 0, s = 0;
    double sum = 0.0;
    float mf = INFINITY;
    const double x1 = x + 1.0;
    auto add = [&](float v) {
        const double dv = (double)v;
        const bool a = dv > x, b = dv > x1;
        s += a ? 1 : 0;
        f += b ? 1 : 0;
        mf = b ? fminf(mf, v) : mf;
        sum += a && !b ? dv : 0.0;
    };
#pragma unroll
    for (int r = 0; r < SEL_REG; r++) add(r * NT_ROW + tid < nsel ? G.su[r] : -INFINITY);
    for (int i = SEL_REG * NT_ROW + tid; i < nsel; i += NT_ROW) add(R.sel_u[i]);
#pragma unroll
    for (int r = 0; r < CAND_REG; r++) add(r * NT_ROW + tid < ncand ? G.cu[r] : -INFINITY);
    for (int i = CAND_REG * NT_ROW + tid; i < ncand; i += NT_ROW) add(R.cand_u[i]);
    if (tid == 0) add(z);
    unsigned long long packed = wave_sum_u64(((unsigned long long)f << 32) | (unsigned long long)s);
    double ws = wave_sum_f64(sum);
    float wm = wave_min_f32(mf);
    __syncthreads();
    if (lane == 0) { red.u64[wv] = packed; red.f64[wv] = ws; red.f32[wv] = wm; }
    __syncthreads();
    packed = 0;
    ws = 0.0;
    wm = INFINITY;
    for (int i = 0; i < NT_ROW / 64; i++) { packed += red.u64[i]; ws += red.f64[i]; wm = fminf(wm, red.f32[i]); }
    F = (int)(packed >> 32);
    S = (int)(packed & 0xFFFFFFFFull);
    fsum = ws;
    minF = wm;
}

struct UpdateSmem {
    BlockRed red;
    int scan[NT_ROW / 64];
    unsigned long long minkey[NT_ROW / 64];
    int at[4];
    float ev_u;
};

// UNDER_WAY: inside step number `sync->step`, whose token has the score u_new; prepares the one after it.  Else: prepares
// step number `sync->step` itself, ahead of it (u_new is read without a window only).
template <bool UNDER_WAY>
__device__ void decode_update(UpdateSmem& sm, const sparsek_decode_cfg& c, const DecodeLayout& L, char* st, int row,
                              const float* __restrict__ u_new)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const RowState R = row_state(st, L, row);
    const int k = c.k, w = c.w;
    // ---- everything that depends on nothing ----
    const int t_now = *R.pos, t = t_now + (UNDER_WAY ? 1 : 0);   // t: position of the step that is prepared
    int nsel = *R.nsel, ncand = *R.ncand;
    const int nfree0 = *R.nfree;
    const double tau_old = *R.tau_d;
    const float unew = UNDER_WAY || w == 0 ? u_new[row] : 0.0f;
    const int step = (int)(R.sync->step & 1);
    StepRecord now = R.sync->rec[0];
    const StepRecord odd = R.sync->rec[1];
    if (step) now = odd;
    RowRegs G;
    int ss[SEL_REG];
#pragma unroll
    for (int r = 0; r < SEL_REG; r++) {
        const int i = min(r * NT_ROW + tid, L.klen - 1);
        G.su[r] = R.sel_u[i];
        G.sp[r] = R.sel_pos[i];
        ss[r] = R.sel_slot[i];
    }
#pragma unroll
    for (int r = 0; r < CAND_REG; r++) G.cu[r] = R.cand_u[min(r * NT_ROW + tid, L.cap - 1)];
    // ---- what depends on the position and the free count alone ----
    const bool leave = (w == 0) || (t >= w);
    const int p = (w > 0) ? t - w : t;  // position joining the prefix (= prefix index T)
    float z = unew;
    int zslot = -1;
    if (leave && w > 0) {
        if (UNDER_WAY && p == t_now) zslot = now.fresh;   // (w == 1: the token of this step)
        else {
            z = R.win_u[p % w];
            zslot = R.win_slot[p % w];
        }
    }
    // Free-slot stack: at most one slot is pushed and at most one is popped per step, so the
    // step works on a local copy (count, the slot pushed in this step, the old top fetched
    // ahead) and writes the stack back once.
    int nfree = nfree0, pushed = -1;
    const int old_top = nfree0 > 0 ? R.free_stack[nfree0 - 1] : -1;
    auto pop_slot = [&]() -> int {
        if (pushed >= 0) { const int r = pushed; pushed = -1; return r; }
        nfree--;
        return old_top;
    };

    bool selected = false, evict = false;
    int e = -1;  // entry of the selected arrays that receives z
    int ev_slot = -1;
    float ev_u = 0.0f;
    double tau_new = tau_old;
    const int len = p + 1;
    if (leave) {
        // ---- (a) top-k decision ----
        if (k > 0) {
            if (nsel < k) {
                selected = true;
                e = nsel;
            } else {
                unsigned long long mk = ~0ull;
#pragma unroll
                for (int r = 0; r < SEL_REG; r++) {
                    const unsigned long long key = sel_key(G.su[r], G.sp[r]);
                    if (r * NT_ROW + tid < nsel) mk = key < mk ? key : mk;
                }
                for (int i = SEL_REG * NT_ROW + tid; i < nsel; i += NT_ROW) {
                    const unsigned long long key = sel_key(R.sel_u[i], R.sel_pos[i]);
                    mk = key < mk ? key : mk;
                }
                mk = wave_min_u64(mk);
                if (lane == 0) sm.minkey[wv] = mk;
                __syncthreads();
                mk = sm.minkey[0];
                for (int i = 1; i < NT_ROW / 64; i++) mk = sm.minkey[i] < mk ? sm.minkey[i] : mk;
                if (sel_key(z, p) > mk) {
                    selected = true;
                    evict = true;
#pragma unroll
                    for (int r = 0; r < SEL_REG; r++)
                        if (r * NT_ROW + tid < nsel && sel_key(G.su[r], G.sp[r]) == mk) {
                            sm.at[0] = r * NT_ROW + tid;
                            sm.at[3] = ss[r];
                            sm.ev_u = G.su[r];
                        }
                    for (int i = SEL_REG * NT_ROW + tid; i < nsel; i += NT_ROW)
                        if (sel_key(R.sel_u[i], R.sel_pos[i]) == mk) {
                            sm.at[0] = i;
                            sm.at[3] = R.sel_slot[i];
                            sm.ev_u = R.sel_u[i];
                        }
                    __syncthreads();
                    e = sm.at[0];
                    ev_slot = sm.at[3];
                    ev_u = sm.ev_u;
                }
            }
        }
        // ---- (b) threshold of prefix p ----
        if (k == 0) {
            tau_new = (len == 1) ? (double)z : fmax(tau_old, (double)z);
        } else if (len <= k) {
            tau_new = (len == 1) ? (double)z - 1.0 : fmin(tau_old, (double)z - 1.0);
        } else if ((double)z > tau_old) {
            tau_new = solve_tau_iter([&](double x, int& F, int& S, double& fsum, float& minF) {
                row_eval(sm.red, G, R, nsel, ncand, z, x, F, S, fsum, minF);
            }, k, tau_old, R.status);
        }
    }
    // ---- (c) slots, and the record of the step ----
    int new_slot = -1;
    int zval_slot = -1;          // the slot of the key that left the window and its gate score
    float zval = -INFINITY;
    if (leave) {
        if (selected) {
            int slot = zslot;
            if (evict) pushed = ev_slot;
            if (w == 0) new_slot = slot = pop_slot();
            zval_slot = slot;
            zval = z;
        } else if (w > 0) {
            zval_slot = zslot;
            pushed = zslot;
        }
    }
    if (w > 0) new_slot = pop_slot();
    const float new_u = w > 0 ? INFINITY : z;
    if (tid == 0)
        R.sync->rec[step ^ (UNDER_WAY ? 1 : 0)] =
            StepRecord{(float)tau_new, evict ? ev_slot : -1, zval_slot, zval, new_slot, new_u, {0, 0}};
    // ---- (d) candidates: scores above tau outside the top-k ----
    if (leave && k > 0 && len > k) {
        __syncthreads();
        // Candidates that fell to or below tau do no harm (they count nowhere); they are only
        // swept out when the set gets three quarters full, not at every rise of tau.
        if ((tau_new > tau_old && ncand + 2 > (L.cap / 4) * 3) || ncand + 2 > L.cap)
            ncand = block_prune(sm.scan, R.cand_u, ncand, tau_new);
        if (tid == 0) {
            float add[2];
            int na = 0;
            if (!selected && (double)z > tau_new) add[na++] = z;
            if (evict && (double)ev_u > tau_new) add[na++] = ev_u;
            for (int i = 0; i < na; i++) {
                if (ncand < L.cap) R.cand_u[ncand++] = add[i];
                else {  // bounded set (Sec. 3.3): drop the smallest, flag the row
                    atomicOr(R.status, 1);
                    int mi = 0;
                    for (int x = 1; x < ncand; x++) if (R.cand_u[x] < R.cand_u[mi]) mi = x;
                    if (ncand > 0 && R.cand_u[mi] < add[i]) R.cand_u[mi] = add[i];
                }
            }
        }
    }
    // ---- (e) the state ----
    if (tid == 0) {
        if (leave) {
            if (selected) {
                R.sel_u[e] = z;
                R.sel_pos[e] = p;
                R.sel_slot[e] = zval_slot;
                if (!evict) nsel++;
            }
            *R.nsel = nsel;
            *R.ncand = ncand;
            *R.tau_d = tau_new;
        }
        if (pushed >= 0) R.free_stack[nfree++] = pushed;
        *R.nfree = nfree;
        // gate scores and window of the step under way; without a window those of the step prepared, whose heads come later
        // (heads of this step read the gate scores meanwhile, and replace these three by their record)
        if (UNDER_WAY || w == 0) {
            const int gone = UNDER_WAY ? now.evicted : evict ? ev_slot : -1, left = UNDER_WAY ? now.left : zval_slot;
            if (gone >= 0) R.slot_u[gone] = -INFINITY;
            if (left >= 0) R.slot_u[left] = UNDER_WAY ? now.left_u : zval;
            *R.pos = t_now + 1;
        }
        if (UNDER_WAY) {
            R.slot_u[now.fresh] = INFINITY;
            R.win_u[t_now % w] = unew;
            R.win_slot[t_now % w] = now.fresh;
        }
    }
}

// One of the row's heads, or its own workgroup (there is one with a window), is through with this step.
__device__ __forceinline__ void report_finished(const sparsek_decode_cfg& c, RowSync* sync)
{
    const unsigned all = (c.Gu == 1 ? c.H : 1) + (c.w > 0 ? 1 : 0);
    if (__hip_atomic_fetch_add(&sync->finished, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == all) {
        __hip_atomic_store(&sync->finished, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&sync->step, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---------------------------------------------------------------------------------
// (2) attention of the one new query over the k+w slots of its head, or over one of nsplit shares of them.
// LPR lanes share a slot row (8 elements each), 64/LPR rows per wave-load.  Up to SLAB slots at a time: the dot products
// of their K rows go to LDS, one thread per slot turns them into weights, and the V rows are summed with those.
// HBM-bound with many heads (64 x 32 heads, 2048 slots of 256 bytes: 2.15 GB in 355 us = 6.0 TB/s; 376 us when the row
// updates ran in a launch of their own ahead of it), bound by latency with few (32 heads: 48 us with one workgroup per
// head, 14 us with eight; 16 and 32 shares take 16 and 25 us: the shares' partial results have to meet).
// Five workgroups per compute unit (96 registers) keep enough rows in flight; six spill.
// ---------------------------------------------------------------------------------
template <typename T>
struct Row8;
template <>
struct Row8<uint16_t> {
    uint4 r;
    __device__ __forceinline__ void load(const uint16_t* p) { r = *(const uint4*)p; }
    __device__ __forceinline__ void get(float (&x)[8]) const
    {
        x[0] = __uint_as_float(r.x << 16); x[1] = __uint_as_float(r.x & 0xFFFF0000u);
        x[2] = __uint_as_float(r.y << 16); x[3] = __uint_as_float(r.y & 0xFFFF0000u);
        x[4] = __uint_as_float(r.z << 16); x[5] = __uint_as_float(r.z & 0xFFFF0000u);
        x[6] = __uint_as_float(r.w << 16); x[7] = __uint_as_float(r.w & 0xFFFF0000u);
    }
};
template <>
struct Row8<float> {
    float4 a, b;
    __device__ __forceinline__ void load(const float* p) { a = *(const float4*)p; b = *(const float4*)(p + 4); }
    __device__ __forceinline__ void get(float (&x)[8]) const
    {
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    }
};
__device__ __forceinline__ void st1(uint16_t* p, float v) { *p = f32_to_bf16(v); }
__device__ __forceinline__ void st1(float* p, float v) { *p = v; }

constexpr int SLAB = 2048;
constexpr int SPT = SLAB / NT_ROW;   // slots per thread

template <int LPR>
struct AttnSmem {
    float w[SLAB];                            // dot products, then weights
    float part[4 * (64 / LPR)][LPR * 8];      // sums of the workgroup's streams
    float red[2][NT_ROW / 64];
    float newdot;
    int last;
};

template <int LPR>
__device__ __forceinline__ float row_sum(float x)   // over the LPR lanes of a row
{
    x += dpp_f32(x, 0);
    x += dpp_f32(x, 1);
    if (LPR >= 8) x += dpp_f32(x, 2);
    if (LPR >= 16) x += dpp_f32(x, 3);
    return x;
}

template <typename T, int LPR, int MODE>
__device__ void decode_attend(AttnSmem<LPR>& sm, const sparsek_decode_cfg& c, const DecodeLayout& L, char* st, int id,
                              const T* q_new, const T* k_new, const T* v_new, T* o)
{
    constexpr int D = LPR * 8;
    constexpr int RPW = 64 / LPR;        // rows per wave-load
    constexpr int NSTREAM = 4 * RPW;     // streams per workgroup
    constexpr int UNR = sizeof(T) == 2 ? 4 : 2;   // rows in flight per stream
    constexpr int ROW16 = sizeof(T) / 2;          // 16-byte units of a row per lane
    const int bh = id / L.nsplit, sp = id % L.nsplit;
    const int b = bh / c.H, h = bh % c.H;
    const int row = b * c.Gu + (c.Gu == 1 ? 0 : h);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int sub = lane % LPR, grp = lane / LPR;
    const int stream = wv * RPW + grp;
    RowSync* sync = (RowSync*)(st + L.sync) + row;
    const unsigned step = (unsigned)sync->step;   // (not counted before this head has reported its end)
    const float* slot_u = (const float*)(st + L.slot_u) + (size_t)row * L.NS;
    const T* ks = (const T*)(st + L.kslots) + (size_t)bh * L.NS * D;
    const T* vs = (const T*)(st + L.vslots) + (size_t)bh * L.NS * D;
    const int per = (L.NS + L.nsplit - 1) / L.nsplit;
    const int s_begin = min(L.NS, sp * per), s_end = min(L.NS, s_begin + per);
    float qf[8];
    {
        Row8<T> r;
        r.load(q_new + (size_t)bh * D + sub * 8);
        r.get(qf);
    }
    const float c2 = c.softmax_scale * 1.4426950408889634f;
#pragma unroll
    for (int e = 0; e < 8; e++) qf[e] *= c2;
    auto dot = [&](const Row8<T>& r) {
        float x[8], d = 0.0f;
        r.get(x);
#pragma unroll
        for (int e = 0; e < 8; e++) d += qf[e] * x[e];
        return row_sum<LPR>(d);
    };
    float m_run = -INFINITY, l_run = 0.0f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; e++) acc[e] = 0.0f;

    const StepRecord rec = sync->rec[step & 1];   // (the row's workgroup writes the other one meanwhile)
    const float tau = rec.tau, left_u = rec.left_u, new_u = rec.fresh_u;
    const int evicted = rec.evicted, left = rec.left, fresh = rec.fresh;
    for (int s0 = s_begin; s0 < s_end; s0 += SLAB) {
        const int sn = min(SLAB, s_end - s0);
        const T* kb = ks + (size_t)s0 * D;   // 32-bit offsets from here: a slab holds at most 1 MB
        const T* vb = vs + (size_t)s0 * D;
        auto at = [&](int i) { return (unsigned)(min(i, sn - 1) * D + sub * 8); };
        // ---- K: dot products (a slot the update is rewriting meanwhile is replaced below) ----
        if (s0 == s_begin && wv == 0) {
            Row8<T> r;
            r.load(k_new + (size_t)bh * D + sub * 8);
            const float d = dot(r);
            if (lane == 0) sm.newdot = d;
        }
#pragma unroll 1
        for (int x0 = stream; x0 < sn; x0 += NSTREAM * UNR) {
            Row8<T> r[UNR];
#pragma unroll
            for (int x = 0; x < UNR; x++) r[x].load(kb + at(x0 + x * NSTREAM));
#pragma unroll
            for (int x = 0; x < UNR; x++) {
                const float d = dot(r[x]);
                if (sub == 0 && x0 + x * NSTREAM < sn) sm.w[x0 + x * NSTREAM] = d;
            }
        }
        // the first V rows are on their way while the gates are formed
        float su[SPT];
#pragma unroll
        for (int r = 0; r < SPT; r++) su[r] = r * NT_ROW + tid < sn ? slot_u[s0 + r * NT_ROW + tid] : -INFINITY;
        Row8<T> vr[UNR];
#pragma unroll
        for (int x = 0; x < UNR; x++) vr[x].load(vb + at(stream + x * NSTREAM));
        __syncthreads();
        // ---- weights ----
        float s2[SPT], mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < SPT; r++) {
            const int s = s0 + r * NT_ROW + tid;
            float x = su[r];
            x = s == evicted ? -INFINITY : x;
            x = s == left ? left_u : x;
            x = s == fresh ? new_u : x;
            su[r] = clip01(x - tau);   // +inf (window) -> 1
            float d = -INFINITY;
            if (r * NT_ROW + tid < sn) d = s == fresh ? sm.newdot : sm.w[r * NT_ROW + tid];
            if (MODE == 0) d *= su[r];
            s2[r] = x > -INFINITY && r * NT_ROW + tid < sn ? d : -INFINITY;
            mx = fmaxf(mx, s2[r]);
        }
        mx = wave_max_f32(mx);
        if (lane == 0) sm.red[0][wv] = mx;
        __syncthreads();
        const float m_new = fmaxf(m_run, fmaxf(fmaxf(sm.red[0][0], sm.red[0][1]), fmaxf(sm.red[0][2], sm.red[0][3])));
        const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int r = 0; r < SPT; r++) {
            const float p = __builtin_amdgcn_exp2f(s2[r] - m_safe);
            l_run += p;
            if (r * NT_ROW + tid < sn) sm.w[r * NT_ROW + tid] = MODE == 2 ? p : p * su[r];
        }
        __syncthreads();
        // ---- V ----
#pragma unroll
        for (int e = 0; e < 8; e++) acc[e] *= alpha;
#pragma unroll 1
        for (int x0 = stream; x0 < sn; x0 += NSTREAM * UNR) {
            if (x0 >= NSTREAM * UNR) {
#pragma unroll
                for (int x = 0; x < UNR; x++) vr[x].load(vb + at(x0 + x * NSTREAM));
            }
#pragma unroll
            for (int x = 0; x < UNR; x++) {
                const int i = x0 + x * NSTREAM;
                if (s0 + i == fresh) vr[x].load(v_new + (size_t)bh * D + sub * 8);
                const float pw = i < sn ? sm.w[i] : 0.0f;
                float v[8];
                vr[x].get(v);
#pragma unroll
                for (int e = 0; e < 8; e++) acc[e] = fmaf(pw, i < sn ? v[e] : 0.0f, acc[e]);
            }
        }
        __syncthreads();
    }
    // The new rows move into their slot here and not in the row's workgroup: nobody outside this head's workgroups
    // reads them, so o may be the memory of q_new, k_new or v_new.  (The share's slots have been read.)
    if (fresh >= s_begin && fresh < s_end && tid < 2 * LPR * ROW16) {
        const int i = tid % (LPR * ROW16);
        const uint4* src = (const uint4*)((tid < LPR * ROW16 ? k_new : v_new) + (size_t)bh * D);
        uint4* dst = (uint4*)(st + (tid < LPR * ROW16 ? L.kslots : L.vslots)) + ((size_t)bh * L.NS + fresh) * (LPR * ROW16);
        dst[i] = src[i];
    }
    // ---- merge the streams ----
#pragma unroll
    for (int e = 0; e < 8; e++) sm.part[stream][sub * 8 + e] = acc[e];
    const float lw = wave_sum_f32(l_run);
    if (lane == 0) sm.red[1][wv] = lw;
    __syncthreads();
    const float l_tot = (sm.red[1][0] + sm.red[1][1]) + (sm.red[1][2] + sm.red[1][3]);
    float osum = 0.0f;
    if (tid < D) {
#pragma unroll
        for (int s = 0; s < NSTREAM; s++) osum += sm.part[s][tid];
    }
    bool finish = true;
    if (L.nsplit == 1) {
        if (tid < D) st1(o + (size_t)bh * D + tid, osum / l_tot);
    } else {
        // Partial results meet in memory, every value with the step's number beside it: a reader waits for the number, so
        // nothing has to be flushed or fenced.  The workgroup that arrives last adds them up, in the order of the shares;
        // what it waits for has been sent off by workgroups that arrived before it.
        const unsigned tag = step + 1u;
        unsigned long long* part = (unsigned long long*)(st + L.part) + (size_t)bh * L.nsplit * (D + 2);
        auto put = [&](int i, float x) {
            __hip_atomic_store(&part[(size_t)sp * (D + 2) + i], (unsigned long long)tag << 32 | __float_as_uint(x),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        if (tid < D) put(tid, osum);
        if (tid == 0) { put(D, m_run); put(D + 1, l_tot); }
        if (tid == 0) {
            unsigned* arrived = (unsigned*)(st + L.heads) + bh;
            const unsigned n = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sm.last = n == (unsigned)L.nsplit - 1u;
            if (sm.last) __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        finish = sm.last;
        if (finish) {
            // (maximum, sum) of every share, then this column of every share; all words are on their way at once
            auto get = [&](int s, int i) {
                unsigned long long x = 0ull;
                for (int spins = 0; spins < (1 << 20); spins++) {
                    x = __hip_atomic_load(&part[(size_t)s * (D + 2) + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((unsigned)(x >> 32) == tag) return __uint_as_float((unsigned)x);
                }
                atomicOr((int*)(st + L.status) + row, 4);   // and no result that could pass for one
                return __uint_as_float(0x7FC00000u);
            };
            for (int s = tid; s < 2 * L.nsplit; s += NT_ROW) sm.w[s] = get(s >> 1, D + (s & 1));
            __syncthreads();
            float M = -INFINITY, lsum = 0.0f;
            for (int s = 0; s < L.nsplit; s++) M = fmaxf(M, sm.w[2 * s]);
            constexpr int CG = NT_ROW / D;   // groups of threads that share the shares of a column
            float sum = 0.0f;
            for (int s = tid / D; s < L.nsplit; s += CG) {
                const float ms = sm.w[2 * s];
                const float f = ms == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ms - M);
                lsum += f * sm.w[2 * s + 1];
                sum += f * get(s, tid % D);
            }
            float* comb = &sm.part[0][0];
            comb[tid] = sum;
            comb[NT_ROW + tid] = lsum;
            __syncthreads();
            if (tid < D) {
                for (int x = 1; x < CG; x++) {
                    sum += comb[x * D + tid];
                    lsum += comb[NT_ROW + x * D + tid];
                }
                st1(o + (size_t)bh * D + tid, sum / lsum);
            }
        }
    }
    if (finish && tid == 0) report_finished(c, sync);
}

template <int LPR>
union StepSmem {
    UpdateSmem u;
    AttnSmem<LPR> a;
};

template <typename T, int LPR, int MODE>
__global__ __launch_bounds__(NT_ROW, 5) void decode_step_kernel(sparsek_decode_cfg c, DecodeLayout L, char* st,
                                                                const T* q_new, const T* k_new, const T* v_new,
                                                                const float* __restrict__ u_new, T* o)
{
    __shared__ __align__(16) StepSmem<LPR> sm;
    const int own = c.w > 0 ? L.rows : 0, id = blockIdx.x;
    if (id < own) {
        decode_update<true>(sm.u, c, L, st, id, u_new);
        if (threadIdx.x == 0) report_finished(c, (RowSync*)(st + L.sync) + id);
    } else {
        decode_attend<T, LPR, MODE>(sm.a, c, L, st, id - own, q_new, k_new, v_new, o);
    }
}

// The record of the step that comes next: of the first one after a state has been set up, without a window of every one.
__global__ __launch_bounds__(NT_ROW) void decode_update_kernel(sparsek_decode_cfg c, char* st, const float* __restrict__ u_new)
{
    __shared__ UpdateSmem sm;
    decode_update<false>(sm, c, decode_layout(c), st, blockIdx.x, u_new);
}

// ---------------------------------------------------------------------------------
// init / load
// ---------------------------------------------------------------------------------
// Empty slots are skipped through their gate score (-inf) but their rows are still streamed and
// multiplied by a zero weight, so they must hold finite numbers: clear slots [first, NS) of every head.
__global__ __launch_bounds__(256) void decode_zero_slots_kernel(sparsek_decode_cfg c, char* st, int from_state)
{
    const DecodeLayout L = decode_layout(c);
    const int bh = blockIdx.x;
    const int b = bh / c.H, h = bh % c.H;
    const int row = b * c.Gu + (c.Gu == 1 ? 0 : h);
    const int first = from_state ? L.NS - *((const int*)(st + L.nfree) + row) : 0;
    const size_t esz = c.dtype == SPARSEK_BF16 ? 2 : 4;
    const size_t row_bytes = (size_t)c.d * esz;
    uint4* kd = (uint4*)(st + L.kslots + ((size_t)bh * L.NS + first) * row_bytes);
    uint4* vd = (uint4*)(st + L.vslots + ((size_t)bh * L.NS + first) * row_bytes);
    const size_t nchunk = (size_t)(L.NS - first) * row_bytes / 16;
    for (size_t x = threadIdx.x + (size_t)blockIdx.y * 256; x < nchunk; x += (size_t)gridDim.y * 256) {
        kd[x] = make_uint4(0, 0, 0, 0);
        vd[x] = make_uint4(0, 0, 0, 0);
    }
    // The step numbers beside the partial results start again at 1: what an earlier generation (or another use of the
    // memory) left there must not pass for a result of the step of the same number.
    if (L.nsplit > 1) {
        unsigned long long* part = (unsigned long long*)(st + L.part) + (size_t)bh * L.nsplit * (c.d + 2);
        for (int x = threadIdx.x + blockIdx.y * 256; x < L.nsplit * (c.d + 2); x += gridDim.y * 256) part[x] = 0ull;
    }
}

// The records and counters of a row and the arrival counters of its heads.
__device__ __forceinline__ void clear_sync(const sparsek_decode_cfg& c, char* st, const DecodeLayout& L, const RowState& R, int row)
{
    if (threadIdx.x < sizeof(RowSync) / 8) ((unsigned long long*)R.sync)[threadIdx.x] = 0ull;
    const int nh = c.Gu == 1 ? c.H : 1, first = (row / c.Gu) * c.H + (c.Gu == 1 ? 0 : row % c.Gu);
    for (int h = threadIdx.x; h < nh; h += NT_ROW) ((unsigned*)(st + L.heads))[first + h] = 0u;
}

__global__ __launch_bounds__(NT_ROW) void decode_init_kernel(sparsek_decode_cfg c, char* st)
{
    const DecodeLayout L = decode_layout(c);
    const int row = blockIdx.x, tid = threadIdx.x;
    RowState R = row_state(st, L, row);
    for (int s = tid; s < L.NS; s += NT_ROW) {
        R.slot_u[s] = -INFINITY;
        R.free_stack[s] = L.NS - 1 - s;  // slot 0 is popped first
    }
    if (tid == 0) {
        *R.pos = 0; *R.nsel = 0; *R.ncand = 0; *R.status = 0; *R.nfree = L.NS;
        *R.tau_d = 0.0;
    }
    clear_sync(c, st, L, R, row);
}

// State after positions 0..n_ctx-1: selected = top-k of prefix T = n_ctx-1-w, window = last w.
__global__ __launch_bounds__(NT_ROW) void decode_load_kernel(sparsek_decode_cfg c, char* st, int n_ctx,
                                                             const float* __restrict__ u,
                                                             const float* __restrict__ tau,
                                                             const int32_t* __restrict__ death)
{
    __shared__ BlockRed red;
    __shared__ int scan[NT_ROW / 64];
    __shared__ int base_s[2];
    const DecodeLayout L = decode_layout(c);
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    RowState R = row_state(st, L, row);
    const int k = c.k, w = c.w;
    const float* ur = u + (size_t)row * n_ctx;
    const int32_t* dr = death + (size_t)row * n_ctx;
    const int Tp = n_ctx - 1 - w;
    const float tau_f = (Tp >= 0) ? tau[(size_t)row * n_ctx + Tp] : 0.0f;
    // start a little below the fp32 threshold, then re-solve exactly in fp64
    const double tau_lo = (double)tau_f - 1e-5 * fmax(1.0, fabs((double)tau_f));
    const bool long_prefix = (k > 0) && (Tp + 1 > k);
    for (int s = tid; s < L.NS; s += NT_ROW) R.slot_u[s] = -INFINITY;
    if (tid == 0) { base_s[0] = 0; base_s[1] = 0; *R.status = 0; }
    __syncthreads();
    // ---- selected keys (ascending position -> slots 0..nsel-1) and candidates ----
    for (int j0 = 0; j0 <= Tp; j0 += NT_ROW) {
        const int j = j0 + tid;
        const bool in = j <= Tp;
        const float uj = in ? ur[j] : 0.0f;
        const bool sel = in && k > 0 && dr[j] > Tp;
        const bool cand = in && !sel && long_prefix && ((double)uj > tau_lo);
        const unsigned long long bs = __ballot(sel), bc = __ballot(cand);
        if (lane == 0) { scan[wv] = __popcll(bs) | (__popcll(bc) << 16); }
        __syncthreads();
        int os = base_s[0], oc = base_s[1];
        for (int x = 0; x < wv; x++) { os += scan[x] & 0xFFFF; oc += scan[x] >> 16; }
        if (sel) {
            const int e = os + __popcll(bs & ((1ull << lane) - 1ull));
            R.sel_u[e] = uj; R.sel_pos[e] = j; R.sel_slot[e] = e; R.slot_u[e] = uj;
        }
        if (cand) {
            const int e = oc + __popcll(bc & ((1ull << lane) - 1ull));
            if (e < L.cap) R.cand_u[e] = uj;
        }
        __syncthreads();
        if (tid == 0) {
            for (int x = 0; x < NT_ROW / 64; x++) { base_s[0] += scan[x] & 0xFFFF; base_s[1] += scan[x] >> 16; }
        }
        __syncthreads();
    }
    const int nsel = base_s[0];
    int ncand = base_s[1];
    if (ncand > L.cap) {  // keeps the first cap in position order; tau becomes approximate
        ncand = L.cap;
        if (tid == 0) atomicOr(R.status, 1);
    }
    __syncthreads();
    // ---- exact fp64 threshold of prefix Tp ----
    double tau_d = 0.0;
    if (Tp >= 0) {
        if (k == 0) tau_d = (double)tau_f;
        else if (!long_prefix) tau_d = (double)tau_f;  // min(prefix) - 1: exact in fp32
        else
            tau_d = solve_tau_iter([&](double x, int& F, int& S, double& fsum, float& minF) {
                block_eval(red, R.sel_u, nsel, R.cand_u, ncand, x, F, S, fsum, minF);
            }, k, tau_lo, R.status);
    }
    if (long_prefix) ncand = block_prune(scan, R.cand_u, ncand, tau_d);
    // ---- window: positions max(0, n_ctx-w) .. n_ctx-1 -> slots nsel.. ----
    const int wb = max(0, n_ctx - w);
    const int nwin = n_ctx - wb;
    for (int i = tid; i < nwin; i += NT_ROW) {
        const int p = wb + i;
        R.win_u[p % w] = ur[p];
        R.win_slot[p % w] = nsel + i;
        R.slot_u[nsel + i] = INFINITY;
    }
    const int used = nsel + nwin;
    for (int s = tid; s < L.NS - used; s += NT_ROW) R.free_stack[s] = L.NS - 1 - s;  // pops `used` first
    if (tid == 0) {
        *R.pos = n_ctx; *R.nsel = nsel; *R.ncand = ncand; *R.nfree = L.NS - used;
        *R.tau_d = tau_d;
    }
    clear_sync(c, st, L, R, row);
}

// K/V rows of the loaded positions, one workgroup per head, 16-byte copies.
template <typename T>
__global__ __launch_bounds__(256) void decode_load_kv_kernel(sparsek_decode_cfg c, char* st, int n_ctx,
                                                             const T* __restrict__ kk, const T* __restrict__ vv)
{
    const DecodeLayout L = decode_layout(c);
    const int bh = blockIdx.x, tid = threadIdx.x;
    const int b = bh / c.H, h = bh % c.H;
    const int row = b * c.Gu + (c.Gu == 1 ? 0 : h);
    RowState R = row_state(st, L, row);
    const int nsel = *R.nsel;
    const int used = L.NS - *R.nfree;
    const int wb = max(0, n_ctx - c.w);
    const int cpr = c.d * (int)sizeof(T) / 16;  // 16-byte chunks per row
    const uint4* ksrc = (const uint4*)(kk + (size_t)bh * n_ctx * c.d);
    const uint4* vsrc = (const uint4*)(vv + (size_t)bh * n_ctx * c.d);
    uint4* kdst = (uint4*)((T*)(st + L.kslots) + (size_t)bh * L.NS * c.d);
    uint4* vdst = (uint4*)((T*)(st + L.vslots) + (size_t)bh * L.NS * c.d);
    for (int x = tid; x < used * cpr; x += 256) {
        const int s = x / cpr, cc = x % cpr;
        const int p = (s < nsel) ? R.sel_pos[s] : wb + (s - nsel);
        kdst[(size_t)s * cpr + cc] = ksrc[(size_t)p * cpr + cc];
        vdst[(size_t)s * cpr + cc] = vsrc[(size_t)p * cpr + cc];
    }
}

// ---------------------------------------------------------------------------------
// (the last launch of a set-up: those before it count the free slots)
static void prepare_first_step(const sparsek_decode_cfg& c, void* state, hipStream_t st)
{
    if (c.w > 0)
        hipLaunchKernelGGL(decode_update_kernel, dim3(c.B * c.Gu), dim3(NT_ROW), 0, st, c, (char*)state, (const float*)nullptr);
}

int launch_decode_init(const sparsek_decode_cfg& c, void* state, hipStream_t st)
{
    if (c.d != 32 && c.d != 64 && c.d != 128) return SPARSEK_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(decode_init_kernel, dim3(c.B * c.Gu), dim3(NT_ROW), 0, st, c, (char*)state);
    hipLaunchKernelGGL(decode_zero_slots_kernel, dim3(c.B * c.H, 4), dim3(256), 0, st, c, (char*)state, 0);
    prepare_first_step(c, state, st);
    return launch_status();
}

int launch_decode_load(const sparsek_decode_cfg& c, void* state, int n_ctx, const void* k, const void* v,
                       const float* u, const float* tau, const int32_t* death, hipStream_t st)
{
    if (c.d != 32 && c.d != 64 && c.d != 128) return SPARSEK_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(decode_load_kernel, dim3(c.B * c.Gu), dim3(NT_ROW), 0, st, c, (char*)state, n_ctx, u, tau,
                       death);
    if (c.dtype == SPARSEK_BF16)
        hipLaunchKernelGGL(decode_load_kv_kernel<uint16_t>, dim3(c.B * c.H), dim3(256), 0, st, c, (char*)state,
                           n_ctx, (const uint16_t*)k, (const uint16_t*)v);
    else
        hipLaunchKernelGGL(decode_load_kv_kernel<float>, dim3(c.B * c.H), dim3(256), 0, st, c, (char*)state,
                           n_ctx, (const float*)k, (const float*)v);
    hipLaunchKernelGGL(decode_zero_slots_kernel, dim3(c.B * c.H, 4), dim3(256), 0, st, c, (char*)state, 1);
    prepare_first_step(c, state, st);
    return launch_status();
}

template <typename T, int LPR>
static void launch_step_t(const sparsek_decode_cfg& c, void* state, const void* q, const void* k, const void* v,
                          const float* u_new, void* o, hipStream_t st)
{
    const DecodeLayout L = decode_layout(c);
    if (c.w == 0) hipLaunchKernelGGL(decode_update_kernel, dim3(L.rows), dim3(NT_ROW), 0, st, c, (char*)state, u_new);
    dim3 grid((unsigned)((c.w > 0 ? L.rows : 0) + c.B * c.H * L.nsplit));
#define SPK_STEP(MODE)                                                                                                 \
    hipLaunchKernelGGL((decode_step_kernel<T, LPR, MODE>), grid, dim3(NT_ROW), 0, st, c, L, (char*)state, (const T*)q, \
                       (const T*)k, (const T*)v, u_new, (T*)o)
    if (c.gate_mode == 0) SPK_STEP(0);
    else if (c.gate_mode == 1) SPK_STEP(1);
    else SPK_STEP(2);
#undef SPK_STEP
}

int launch_decode_step(const sparsek_decode_cfg& c, void* state, const void* q, const void* k, const void* v,
                       const float* u_new, void* o, hipStream_t st)
{
    if (c.d != 32 && c.d != 64 && c.d != 128) return SPARSEK_ERR_UNSUPPORTED;
    if (c.dtype == SPARSEK_BF16) {
        if (c.d == 128) launch_step_t<uint16_t, 16>(c, state, q, k, v, u_new, o, st);
        else if (c.d == 64) launch_step_t<uint16_t, 8>(c, state, q, k, v, u_new, o, st);
        else launch_step_t<uint16_t, 4>(c, state, q, k, v, u_new, o, st);
    } else {
        if (c.d == 128) launch_step_t<float, 16>(c, state, q, k, v, u_new, o, st);
        else if (c.d == 64) launch_step_t<float, 8>(c, state, q, k, v, u_new, o, st);
        else launch_step_t<float, 4>(c, state, q, k, v, u_new, o, st);
    }
    return launch_status();
}

int decode_status(const sparsek_decode_cfg& c, const void* state, int32_t* host_flags, hipStream_t st)
{
    const DecodeLayout L = decode_layout(c);
    if (hipMemcpyAsync(host_flags, (const char*)state + L.status, (size_t)L.rows * 4, hipMemcpyDeviceToHost, st) !=
        hipSuccess)
        return SPARSEK_ERR_LAUNCH;
    if (hipStreamSynchronize(st) != hipSuccess) return SPARSEK_ERR_LAUNCH;
    return SPARSEK_OK;
}

}  // namespace spk
