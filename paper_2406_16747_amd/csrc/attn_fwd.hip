// Stage 3: gated attention forward over top-k + sliding window (Sec. 3.2, 3.4, 3.5).
//
// Key fact used everywhere (follows from the irreversible selection, Sec. 3.2): key j is
// attended by the contiguous query range j <= i <= L_j with L_j = w - 1 + death[j]; its gate
// is 1 while i - j < w and clip(u_j - tau_{i-w}, 0, 1) afterwards.  So a block of QB
// consecutive queries starting at i0 needs
//   (a) the top-k of prefix T0 = i0 - w   (a compact list, built once per score row), and
//   (b) the contiguous keys max(0, i0-w+1) .. i0+QB-1 (window + keys that become selected
//       while the block runs),
// with a per-pair validity/gate test.  That turns the per-query sparse gather into dense
// (queries x keys) tiles.
#include "common.hpp"
#include "attn_tiles.hpp"
#include "chunk_parts.hpp"
#include <type_traits>

namespace spk {


// Workspace of the per-block top-k lists: lists [rows][nb][max(k,1)] int32, then counts [rows][nb]
// (list lengths) and stays [rows][nb] (lengths of the first partitions).
size_t block_lists_bytes(const sparsek_cfg& c, size_t* counts_offset)
{
    size_t rows = (size_t)c.B * c.Gu;
    size_t nb = nblocks(c.n);
    size_t lists = align_up(rows * nb * (size_t)(c.k > 0 ? c.k : 1) * sizeof(int32_t), 256);
    size_t counts = align_up(2 * rows * nb * sizeof(int32_t), 256);
    if (counts_offset) *counts_offset = lists;
    return lists + counts;
}

size_t attn_fwd_ws_bytes(const sparsek_cfg& c) { return block_lists_bytes(c, nullptr) + 3 * ext_array_bytes(c); }

// ---------------------------------------------------------------------------------
// Per (row, block): the positions of the top-k of prefix T0 = blk*QB - w, in two partitions:
// first the keys that stay selected for every query of the block (death >= T0 + QB, ascending),
// then, filled from the back, the keys that expire inside the block.  Only the tiles of the
// second partition need a per-pair validity test.  Each of the 16 waves owns a slice of
// [0, T0]: one counting pass, one barrier, one placement pass; up to BL_REG lifetimes per lane stay in
// registers in between.  The list is put together in LDS and written from there in order, with the
// scores fetched at that point: placing entries straight into memory made every group of 64 positions
// wait for its scores.
// A workgroup that owns several consecutive blocks scans the prefix for the first one only: the top-k of the next
// block's prefix are the keys that stayed selected, and the 128 positions in between.
// Bounded by latency for one row (18.9 -> 12.5 us at n = 32768, k = 1024), by the scans' issue for many
// (82 us, 62 us with a workgroup per block, 42 us with eight blocks per workgroup, for 32 rows of 16384).
// With xpos != nullptr the same lists are also written in the extended form described above.
// ---------------------------------------------------------------------------------
constexpr int BL_WAVES = 16;   // waves per workgroup of block_lists_kernel
constexpr int BL_LDS = 4096;   // entries put together in LDS; longer lists are placed in memory directly

struct ListSmem {
    int wstay[BL_WAVES], wgo[BL_WAVES];
    int pos[2][BL_LDS], death[2][BL_LDS];   // the list of this block, of the one before
};
struct ListOut {
    int32_t *lo, *xpos, *xdeath;
    float* xu;
};

// The lists of `cand(e)` = (position, lifetime), e = 0 .. ncand - 1, that are alive at T0, each wave owning a slice of
// the candidates, REG per lane at a time: into LDS, or into memory when there are more than BL_LDS of them.
// Returns the number of entries that stay for the whole block, cnt = entries in all.
template <int REG, typename Death, typename Pos>
__device__ __forceinline__ int block_list(ListSmem& sm, int buf, int ncand, int T0, int k, const float* __restrict__ ur,
                                          const ListOut& out, int& cnt, Death&& death_of, Pos&& pos_of)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned long long below = (1ull << lane) - 1ull;
    const int per = ((ncand + BL_WAVES - 1) / BL_WAVES + 63) / 64 * 64;
    const int e_lo = min(ncand, wv * per), e_hi = min(ncand, e_lo + per);
    const int stay_from = T0 + QB;
    int dj[REG];
    auto load = [&](int e0) {
#pragma unroll
        for (int r = 0; r < REG; r++) {
            if (e0 + 64 * r >= e_hi) break;   // (uniform)
            const int e = e0 + 64 * r + lane;
            dj[r] = e < e_hi ? death_of(e) : 0;
        }
    };
    int ns = 0, ng = 0;
    for (int e0 = e_lo; e0 < e_hi; e0 += 64 * REG) {
        load(e0);
#pragma unroll
        for (int r = 0; r < REG; r++) {
            if (e0 + 64 * r >= e_hi) break;
            const unsigned long long alive = __ballot(dj[r] > T0), stay = __ballot(dj[r] >= stay_from);
            ns += __popcll(stay);
            ng += __popcll(alive) - __popcll(stay);
        }
    }
    if (lane == 0) { sm.wstay[wv] = ns; sm.wgo[wv] = ng; }
    __syncthreads();
    int os = 0, og = 0, tot_s = 0, tot_g = 0;
    for (int i = 0; i < BL_WAVES; i++) {
        if (i < wv) { os += sm.wstay[i]; og += sm.wgo[i]; }
        tot_s += sm.wstay[i];
        tot_g += sm.wgo[i];
    }
    // min(k, T0 + 1) for a consistent death array; counted, so that every entry below cnt is written
    cnt = min(k, tot_s + tot_g);
    const bool in_lds = cnt <= BL_LDS;
    for (int e0 = e_lo; e0 < e_hi; e0 += 64 * REG) {
        if (per > 64 * REG) load(e0);
#pragma unroll
        for (int r = 0; r < REG; r++) {
            if (e0 + 64 * r >= e_hi) break;
            const unsigned long long alive = __ballot(dj[r] > T0), bs = __ballot(dj[r] >= stay_from), bg = alive & ~bs;
            if (!alive) continue;
            int o = -1;
            if (dj[r] >= stay_from) {
                o = os + __popcll(bs & below);
                if (o >= cnt) o = -1;
            } else if (dj[r] > T0) {
                o = cnt - 1 - (og + __popcll(bg & below));
            }
            if (o >= 0) {
                const int j = pos_of(e0 + 64 * r + lane);
                if (in_lds) {
                    sm.pos[buf][o] = j;
                    sm.death[buf][o] = dj[r];
                } else {
                    out.lo[o] = j;
                    if (out.xpos) {
                        out.xpos[o] = j;
                        out.xdeath[o] = dj[r];
                        out.xu[o] = ur[j];
                    }
                }
            }
            os += __popcll(bs);
            og += __popcll(bg);
        }
    }
    __syncthreads();   // the list is complete; wstay and wgo may be written again
    return tot_s;
}

// BL_REG: lifetimes per lane of a scan.  32 read a prefix of 32768 once; 8 leave room for a second workgroup on the
// compute unit.  RUNS: a workgroup owns `run` consecutive blocks, else one.  CHUNK: lifetimes are read as the end of a chunk has
// them; the first workgroup of a row finds its survivors, the others clear the lifetimes in memory when their lists are done.
template <int BL_REG, bool RUNS, bool CHUNK>
__global__ __launch_bounds__(64 * BL_WAVES, RUNS ? 8 : 4) void block_lists_kernel(
    const int32_t* __restrict__ death, int n, int k, int w, int nb, int run /* consecutive blocks per workgroup */,
    int32_t* __restrict__ lists, int32_t* __restrict__ counts, const float* __restrict__ u, int32_t* __restrict__ xpos,
    int32_t* __restrict__ xdeath, float* __restrict__ xu, int KP, int blk0, ChunkTail tail)
{
    constexpr int NT = 64 * BL_WAVES;
    union Smem {
        __device__ Smem() {}
        ListSmem l;
        RetainSmem r;
    };
    __shared__ Smem smem;
    ListSmem& sm = smem.l;
    if (CHUNK && blockIdx.x == 0) {
        chunk_retain<false>(smem.r, tail, blockIdx.y);
        return;
    }
    const int wg = CHUNK ? blockIdx.x - 1 : blockIdx.x;
    const int row = blockIdx.y, nrows = gridDim.y;
    const int tid = threadIdx.x;
    const int32_t* dr = death + (size_t)row * n;
    auto lifetime = [&](int e) { return CHUNK ? tail.lifetime(row, e) : dr[e]; };
    const float* ur = u ? u + (size_t)row * n : nullptr;
    int stayed = -1;   // entries of the list before that stayed selected; -1: no such list
    int buf = 0;
    const int b_first = blk0 + (RUNS ? wg * run : wg), b_end = RUNS ? min(nb, b_first + run) : b_first + 1;
    for (int blk = b_first; blk < b_end; blk++) {
        const int T0 = blk * QB - w;
        if (T0 < 0 || k == 0) {
            if (tid == 0) {
                counts[(size_t)row * nb + blk] = 0;
                counts[((size_t)nrows + row) * nb + blk] = 0;
            }
            continue;
        }
        const size_t xo = ((size_t)row * nb + blk) * (size_t)KP;
        const ListOut out{lists + ((size_t)row * nb + blk) * (size_t)k, xpos ? xpos + xo : nullptr, xdeath + xo, xu + xo};
        int cnt, tot_s;
        if (!RUNS || stayed < 0) {
            tot_s = block_list<BL_REG>(sm, buf, T0 + 1, T0, k, ur, out, cnt, lifetime,
                                       [](int e) { return e; });
        } else {   // what stayed, then the positions T0 - QB + 1 .. T0: ascending again
            const int* pp = sm.pos[buf ^ 1];
            const int* pd = sm.death[buf ^ 1];
            const int first = T0 - QB + 1 - stayed;
            tot_s = block_list<2>(sm, buf, stayed + QB, T0, k, ur, out, cnt,
                                  [&](int e) { return e < stayed ? pd[e] : lifetime(first + e); },
                                  [&](int e) { return e < stayed ? pp[e] : first + e; });
        }
        if (tid == 0) {
            counts[(size_t)row * nb + blk] = cnt;
            counts[((size_t)nrows + row) * nb + blk] = min(cnt, tot_s);
        }
        if (cnt <= BL_LDS) {
            for (int o = tid; o < cnt; o += NT) {
                const int j = sm.pos[buf][o];
                out.lo[o] = j;
                if (xpos) {
                    out.xpos[o] = j;
                    out.xdeath[o] = sm.death[buf][o];
                    out.xu[o] = ur[j];
                }
            }
        }
        if (xpos) {
            // padding up to the tile boundary above min(k, T0 + 1), the length the forward kernel lays its tiles out for
            const int padded = (min(k, T0 + 1) + KT - 1) / KT * KT;
            for (int o = cnt + tid; o < padded; o += NT) {
                out.xpos[o] = 0;
                out.xdeath[o] = INT32_MIN;
                out.xu[o] = 0.0f;
            }
        }
        stayed = cnt <= BL_LDS && tot_s <= cnt ? tot_s : -1;
        buf ^= 1;
    }
    if (CHUNK) chunk_clear_padding(tail, row, wg * NT + tid, (gridDim.x - 1) * NT);
}

// ---------------------------------------------------------------------------------
// Kernel for fp32 storage, and for bf16 with a head dimension the kernel below does not cover (any d <= 128 that is a
// multiple of 4): fp32 matrix instructions (v_mfma_f32_16x16x4_f32, full fp32 products and sums).  A workgroup owns 16
// queries; its four waves take the 16-key tiles of their key set in turn, each with an online softmax of its own, and
// merge through LDS.  No LDS staging: operands come from memory in the layout the instruction wants --
//   S^T = K.Q^T    lane l supplies K[key l % 16] at d = 16 x + 4 (l / 16) + {0..3}: one 16-byte load feeds four steps (the
//                  order of d inside a contraction is free, Q uses the same);
//   O^T += V^T.P^T step r contracts the keys 4 g + r, g = 0..3: exactly the P values that lane group g holds.
// Problems of this kind are small (one head of 1024 queries, k = w = 64: 31 us with a wave per query and scalar
// products), so it is built for latency: GEN_SPLIT workgroups per query block, positions one tile ahead.
// ---------------------------------------------------------------------------------
constexpr int GQ = 16;                 // queries per workgroup
constexpr int GEN_SPLIT = QB / GQ;
// Without lists (OWN) a workgroup finds the top-k of its own first prefix: one pass over up to GEN_N lifetimes, the positions in
// LDS.  The launch in between is saved, and the key set is that of 16 queries and not of 128.  An instance of its own: one kernel for
// both takes 6 to 8 registers more, and up to 32 columns that is the fifth wave of a SIMD (64 heads of 4096, k = w = 64, d = 32, prefill
// 211 us, 183 with two instances; 16 heads of 16384, which take lists, 223 and 203).
constexpr int GEN_N = 4096, GEN_K = 1024;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
// As wide as the head dimension's multiple of 4 allows, but tensors of this kernel need no more than element alignment.
typedef float f32x4_any __attribute__((__vector_size__(16), __aligned__(4)));
typedef uint32_t u32x2_any __attribute__((__vector_size__(8), __aligned__(2)));

__device__ __forceinline__ f32x4 load4(const float* p) { return *(const f32x4_any*)p; }
__device__ __forceinline__ f32x4 load4(const uint16_t* p)
{
    const u32x2_any r = *(const u32x2_any*)p;
    return f32x4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xFFFF0000u), __uint_as_float(r[1] << 16),
                 __uint_as_float(r[1] & 0xFFFF0000u)};
}
__device__ __forceinline__ float load1(const float* p) { return *p; }
__device__ __forceinline__ float load1(const uint16_t* p) { return bf16_to_f32(*p); }
__device__ __forceinline__ void store1(float* p, float v) { *p = v; }
__device__ __forceinline__ void store1(uint16_t* p, float v) { *p = f32_to_bf16(v); }

template <typename T, int DT, bool OWN>   // DT = number of 16-column blocks of the head dimension (rounded up)
__global__ __launch_bounds__(256) void attn_fwd_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ kk, const T* __restrict__ v,
    const float* __restrict__ u, const float* __restrict__ tau, const int32_t* __restrict__ death,
    const int32_t* __restrict__ lists, const int32_t* __restrict__ counts, T* __restrict__ o,
    float* __restrict__ lse, int H, int Gu, int n, int d, int k, int w, int gate_mode, float scale, int nb,
    int q_begin, const int32_t* __restrict__ first_valid, int q_rows)
{
    __shared__ float po[4][DT * 16][GQ + 1], pm[4][GQ], pl[4][GQ];
    __shared__ int own[OWN ? GEN_K : 1], wtot[4];
    const int blk = blockIdx.x / GEN_SPLIT, sub = blockIdx.x % GEN_SPLIT, bh = blockIdx.y;
    const int b = bh / H, h = bh % H;
    const int row = b * Gu + (Gu == 1 ? 0 : h);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int i0 = blk * QB, ia = i0 + GQ * sub;   // first query of the block, of this workgroup
    if (i0 + QB <= q_begin || ia >= n) return;     // queries before q_begin are not wanted (chunked prefill)
    // q and o hold q_rows rows per head starting at query q_begin (0: all n rows)
    const ptrdiff_t qo = q_rows ? (ptrdiff_t)bh * q_rows - q_begin : (ptrdiff_t)bh * n;
    const T* kh = kk + (size_t)bh * n * d;
    const T* vh = v + (size_t)bh * n * d;
    const float* ur = u + (size_t)row * n;
    const int32_t* dr = death + (size_t)row * n;
    const int32_t* list = lists + (OWN ? 0 : ((size_t)row * nb + blk) * (size_t)(k > 0 ? k : 1));
    const int T0 = (OWN ? ia : i0) - w;          // the prefix of the listed keys
    // keys before first_valid[row] (padding of a chunked prefill) are attended by nobody
    const int c0 = max(max(0, T0 + 1), first_valid ? first_valid[row] : 0);
    const int i = ia + col;                        // this lane's query
    const int iq = min(i, n - 1);
    const int Tp = i - w;
    const float tauT = (Tp >= 0 && i < n) ? tau[(size_t)row * n + Tp] : 0.0f;
    const int ib = min(ia + GQ - 1, n - 1);        // last query of the workgroup
    int nl = !OWN && ib - w >= 0 ? counts[(size_t)row * nb + blk] : 0;
    f32x4 qf[DT], acc[DT];
#pragma unroll
    for (int x = 0; x < DT; x++) {
        const int dd = 16 * x + 4 * grp;
        qf[x] = f32x4{0, 0, 0, 0};
        if (dd < d) qf[x] = load4(q + (qo + iq) * d + dd);
        acc[x] = f32x4{0, 0, 0, 0};
    }
    if (OWN && T0 >= 0) {   // (uniform)
        constexpr int REG = GEN_N / 256;
        const int per = ((T0 + 4) / 4 + 63) / 64 * 64, e_lo = wv * per, e_hi = min(T0 + 1, e_lo + per);
        int dj[REG], mine = 0;
#pragma unroll
        for (int r = 0; r < REG; r++) {
            const int e = e_lo + 64 * r + lane;
            dj[r] = e < e_hi ? dr[e] : INT32_MIN;
        }
#pragma unroll
        for (int r = 0; r < REG; r++) mine += __popcll(__ballot(dj[r] > T0));
        if (lane == 0) wtot[wv] = mine;
        __syncthreads();
        int at = 0;
#pragma unroll
        for (int x = 0; x < 4; x++) {
            if (x < wv) at += wtot[x];
            nl += wtot[x];
        }
        nl = min(nl, k);
#pragma unroll
        for (int r = 0; r < REG; r++) {
            const unsigned long long alive = __ballot(dj[r] > T0);
            const int o = at + __popcll(alive & ((1ull << lane) - 1ull));
            if (dj[r] > T0 && o < nl) own[o] = e_lo + 64 * r + lane;
            at += __popcll(alive);
        }
        __syncthreads();
    }
    const int total = nl + max(0, ib - c0 + 1);
    const float c2 = scale * 1.4426950408889634f;
    auto pos = [&](int e) { return e >= total ? -1 : e >= nl ? c0 + (e - nl) : OWN ? own[e] : list[e]; };
    float m_run = -INFINITY, l_run = 0.0f;
    // positions of this lane's K row and of its four P / V rows
    int jk = pos(16 * wv + col), jp[4];
#pragma unroll
    for (int r = 0; r < 4; r++) jp[r] = pos(16 * wv + 4 * grp + r);
    for (int e0 = 16 * wv; e0 < total; e0 += 64) {
        const T* kr = kh + (size_t)max(jk, 0) * d;
        f32x4 kf[DT];
#pragma unroll
        for (int x = 0; x < DT; x++) {
            const int dd = 16 * x + 4 * grp;
            kf[x] = f32x4{0, 0, 0, 0};
            if (dd < d) kf[x] = load4(kr + dd);
        }
        float vf[4][DT], uj[4];
        int dj[4];
        unsigned vtop = 0;   // largest magnitude among the values, as bits
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int j = max(jp[r], 0);
            uj[r] = ur[j];
            dj[r] = dr[j];
#pragma unroll
            for (int x = 0; x < DT; x++) {
                vf[r][x] = 16 * x + col < d ? load1(vh + (size_t)j * d + 16 * x + col) : 0.0f;
                vtop = max(vtop, __float_as_uint(vf[r][x]) & 0x7FFFFFFFu);
            }
        }
        const int jc[4] = {jp[0], jp[1], jp[2], jp[3]};
        jk = pos(e0 + 64 + col);
#pragma unroll
        for (int r = 0; r < 4; r++) jp[r] = pos(e0 + 64 + 4 * grp + r);
        f32x4 s = {0, 0, 0, 0};
#pragma unroll
        for (int x = 0; x < DT; x++)
#pragma unroll
            for (int e = 0; e < 4; e++) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[x][e], qf[x][e], s, 0, 0, 0);
        float s2[4], g[4], mx = -INFINITY;
        int ok = 0;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int j = jc[r];
            const bool win = i - j < w;
            // a window key (not in the future), or selected for prefix i - w
            const bool valid = j >= 0 && j <= i && (win || dj[r] > Tp);
            ok |= valid ? 1 << r : 0;
            g[r] = win ? 1.0f : clip01(uj[r] - tauT);
            s2[r] = valid ? s[r] * (gate_mode == 0 ? g[r] : 1.0f) * c2 : -INFINITY;
            mx = fmaxf(mx, s2[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
        const float corr = __builtin_amdgcn_exp2f(m_run - m_safe);
        m_run = m_new;
        l_run *= corr;
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            p[r] = __builtin_amdgcn_exp2f(s2[r] - m_safe);
            l_run += p[r];
            if (gate_mode != 2) p[r] *= g[r];
        }
#pragma unroll
        for (int x = 0; x < DT; x++) acc[x] *= corr;
        if (__any(vtop >= 0x7F800000u)) {
            // An infinity or NaN among the values reaches the queries that attend its key and no other: no zero weights.
#pragma unroll
            for (int r = 0; r < 4; r++)
#pragma unroll 1
                for (int y = 0; y < 4; y++) {
                    const float py = __shfl(p[r], 16 * y + col, 64);
                    const bool oy = __shfl(ok, 16 * y + col, 64) >> r & 1;
                    const T* vr = vh + (size_t)max(__shfl(jc[r], 16 * y, 64), 0) * d;
#pragma unroll
                    for (int x = 0; x < DT; x++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int dd = 16 * x + 4 * grp + e;
                            if (oy && dd < d) acc[x][e] += py * load1(vr + dd);
                        }
                }
            continue;
        }
#pragma unroll
        for (int x = 0; x < DT; x++)
#pragma unroll
            for (int r = 0; r < 4; r++) acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][x], p[r], acc[x], 0, 0, 0);
    }
    // ---- merge the waves: O^T rows 16 x + 4 grp + e, column col ----
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (grp == 0) { pm[wv][col] = m_run; pl[wv][col] = l_run; }
#pragma unroll
    for (int x = 0; x < DT; x++)
#pragma unroll
        for (int e = 0; e < 4; e++) po[wv][16 * x + 4 * grp + e][col] = acc[x][e];
    __syncthreads();
    for (int x = tid; x < GQ * d; x += 256) {
        const int qi = x / d, dd = x % d;
        if (ia + qi >= n || ia + qi < q_begin) continue;
        const float M = fmaxf(fmaxf(pm[0][qi], pm[1][qi]), fmaxf(pm[2][qi], pm[3][qi]));
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int y = 0; y < 4; y++) {
            const float f = pm[y][qi] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(pm[y][qi] - M);
            num += f * po[y][dd][qi];
            den += f * pl[y][qi];
        }
        store1(o + (qo + ia + qi) * d + dd, num / den);
        if (lse && dd == 0) lse[qo + ia + qi] = (M + log2f(den)) * 0.6931471805599453f;
    }
}

// ---------------------------------------------------------------------------------
// MFMA kernel (bf16 storage, D = 64 or 128).  One workgroup = 128 queries x 4 waves; each
// wave owns 32 queries and walks the block's key set in tiles of 64 keys:
//   S^T (keys x queries) = K_tile . Q^T     v_mfma_f32_32x32x16_bf16, K rows from LDS
//   online softmax down the key axis: every lane owns one query column, so row maxima and
//   sums stay inside a lane (one exchange with the lane holding the other half of the keys)
//   O^T (d x queries)   += V_tile^T . P^T   the A operand needs the key axis contiguous per
//   lane: V stays row-major in LDS and is read with the transposing LDS load
//   (ds_read_b64_tr_b16); P^T feeds the B operand straight from the accumulator layout.
// K/V rows are gathered from HBM by position straight into LDS (global_load_lds, 16 bytes per
// lane, no register staging), double-buffered, one tile ahead of the compute, one barrier per
// tile.  A wave-load moves 1 KB = RPL whole rows; tile row r goes to group r % NL, slot r / NL,
// and the groups are padded (16 bytes for K, 64 for V) so that the operand reads of 16
// consecutive lanes fall on distinct banks.
//
// The kernel is bound by vector-ALU issue (gates, masks, exponentials), not by the matrix
// cores, so inside a tile the two are interleaved by hand: the tile is split into two halves
// of 32 keys, and the instruction stream is
//   S_A | S_B + softmax(A) | O += V_A^T.P_A + softmax(B) | O += V_B^T.P_B
// with one MFMA followed by a slice of the softmax work, the slices fenced with sched_barrier
// so that the compiler keeps the order.
// ---------------------------------------------------------------------------------
// The forward's LDS: the double-buffered K and V tiles and the staged metadata.
template <int D>
struct FwdSmem : MfmaTileBufs<D, 64>, TileMeta {};
static_assert(sizeof(FwdSmem<128>) <= 80 * 1024, "two workgroups per CU");

template <int D>
__device__ __forceinline__ void rescale_o(f32x16 (&acc_o)[D / 32], float alpha)
{
    if (__any(alpha != 1.0f)) {
#pragma unroll
        for (int x = 0; x < D / 32; x++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc_o[x][r] *= alpha;
    }
}

// The reference point of the online softmax of one query: m (logit units, -inf before the
// first visible key) and mc = m * scale * log2(e) (0 while m is -inf), what the exponent subtracts.
struct SoftRef {
    float m, mc;
};

// Softmax state of one 32-key half of a tile: this lane holds 16 of its logits (4 groups of 4
// consecutive keys), their gates and lifetimes.
struct HalfState {
    float4 G[4];   // scores, overwritten by the gates
    float tmax, mc, alpha, psum;
    bf16x8 pb[2];  // P^T in operand layout
};

template <int MODE, int KIND>
__device__ __forceinline__ void load_meta(HalfState& h, const float* ju, int hf, int half)
{
    using TT = TileTraits<MODE, KIND>;
#pragma unroll
    for (int g4 = 0; g4 < 4; g4++) {
        const int kb = 32 * hf + 8 * g4 + 4 * half;
        if (TT::GATED) h.G[g4] = *(const float4*)&ju[kb];
    }
    h.tmax = -INFINITY;
    h.psum = 0.0f;
}

// Slice U of the softmax work of one half.  U = 0..3: gates and masks of key group U and the
// running maximum; after group 3 the maximum is exchanged with the partner lane and the
// reference point moves if it has to (lazily: only when the maximum grew by more than 2^8 in
// probability; softmax is shift-invariant and p stays below 2^8, harmless in fp32/bf16; this
// keeps the rescale of the output accumulator a rare event).  U = 4..7: exponentials, row sum,
// value gate and bf16 packing of key group U - 4.
template <int MODE, int KIND, int U>
__device__ __forceinline__ void softmax_slice(HalfState& h, f32x16& sv, const int32_t* jdeath, int half, int hf,
                                              int qw, int dqh, int dqw, float tau_q, float c2, SoftRef& ref)
{
    using TT = TileTraits<MODE, KIND>;
    constexpr float LAZY_LOG2 = 8.0f;
    if (U < 4) {
        constexpr int g4 = U & 3;
        float gg[4] = {h.G[g4].x, h.G[g4].y, h.G[g4].z, h.G[g4].w};
        // lifetimes are read where they are used (only the few masked tile kinds need them):
        // holding them across the tile costs more registers than the kernel has
        int4 L4 = make_int4(0, 0, 0, 0);
        if (TT::MASKL) L4 = *(const int4*)&jdeath[32 * hf + 8 * g4 + 4 * half];
        const int ll[4] = {L4.x, L4.y, L4.z, L4.w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int r = 4 * g4 + e;
            // key number within the tile minus the lane-dependent 4*half (folded into dqh, dqw so
            // that every compare below has a compile-time constant on one side)
            const int cst = 32 * hf + 8 * g4 + e;
            float s2 = sv[r];
            if (TT::GATED) {
                float g = clip01(gg[e] - tau_q);
                if (TT::SELECT) g = (cst > dqw) ? 1.0f : g;
                gg[e] = g;
                if (TT::KGATE) s2 *= g;
            }
            // key j is attended by query i while i <= w - 1 + death[j], i.e. qw = i - (w - 1) <= death[j]
            if (TT::MASKL && TT::MASKC) s2 = (cst <= dqh && qw <= ll[e]) ? s2 : -INFINITY;
            else if (TT::MASKL) s2 = (qw <= ll[e]) ? s2 : -INFINITY;
            else if (TT::MASKC) s2 = (cst <= dqh) ? s2 : -INFINITY;
            sv[r] = s2;
            h.tmax = fmaxf(h.tmax, s2);
        }
        if (TT::GATED) h.G[g4] = make_float4(gg[0], gg[1], gg[2], gg[3]);
        if (U == 3) {
            // Almost always no lane of the wave has to move its reference point: one compare and
            // a wave-uniform branch; the exchange with the partner lane, the new reference and
            // the rescale factor are computed only in the rare other case.
            const float limit = ref.m + LAZY_LOG2 / c2;
            h.alpha = 1.0f;
            if (__any(h.tmax > limit)) {
                const unsigned tb = __float_as_uint(h.tmax);
                const auto sw = __builtin_amdgcn_permlane32_swap(tb, tb, false, false);  // both halves, no LDS
                const float tq = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
                const float m_new = (tq > limit) ? tq : ref.m;
                const float m_safe = (m_new == -INFINITY) ? 0.0f : m_new;
                h.alpha = __builtin_amdgcn_exp2f((ref.m - m_safe) * c2);
                ref.mc = m_safe * c2;
                ref.m = m_new;
            }
            h.mc = ref.mc;
        }
    } else {
        constexpr int g4 = U & 3;
        const float gg[4] = {h.G[g4].x, h.G[g4].y, h.G[g4].z, h.G[g4].w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int r = 4 * g4 + e;
            const float p = __builtin_amdgcn_exp2f(fmaf(sv[r], c2, -h.mc));
            h.psum += p;
            const float pv = TT::GATED ? p * gg[e] : p;
            h.pb[r >> 3][r & 7] = (__bf16)pv;
        }
    }
}

template <int MODE, int KIND, int U0, int U1>
__device__ __forceinline__ void softmax_slices(HalfState& h, f32x16& sv, const int32_t* jdeath, int half, int hf,
                                               int qw, int dqh, int dqw, float tau_q, float c2, SoftRef& ref)
{
    if constexpr (U0 < U1) {
        softmax_slice<MODE, KIND, U0>(h, sv, jdeath, half, hf, qw, dqh, dqw, tau_q, c2, ref);
        softmax_slices<MODE, KIND, U0 + 1, U1>(h, sv, jdeath, half, hf, qw, dqh, dqw, tau_q, c2, ref);
    }
}

// One 64-key tile for one wave (see the schedule in the header comment).  The tile is a
// sequence of MFMA slots (S_A, S_B, PV_A, PV_B); the LDS operand of slot n is requested DEPTH
// slots earlier into a small register ring, so that no MFMA waits for a read it has just issued.
template <int D, int MODE, int KIND>
__device__ __forceinline__ void tile_body(FwdSmem<D>& sm, int buf, const int32_t* jdeath, const float* ju,
                                          const int32_t* jp_next, int jbase, bool more,
                                          const uint16_t* kh, const uint16_t* vh, int wv, int col, int half,
                                          int lane, int qi, int w, float tau_q, float c2,
                                          const bf16x8 (&qreg)[D / 16], f32x16 (&acc_o)[D / 32], SoftRef& ref,
                                          float& l_run)
{
    using S = FwdSmem<D>;
    constexpr int NS = D / 16;      // MFMAs per half of S^T
    constexpr int DB = D / 32;      // 32-row blocks of O^T
    constexpr int NP = 2 * DB;      // MFMAs per half of O^T += V^T.P^T
    constexpr int US = 8 / NS;      // softmax slices per MFMA of S_B
    constexpr int UP = 8 / NP;      // softmax slices per MFMA of the first PV half
    constexpr int NSLOT = 2 * NS + 2 * NP;
    constexpr int DEPTH = 2;
    constexpr int NX = S::NL / 4;   // gather steps of the next tile, one per S_A slot
    static_assert(NX <= NS, "one gather step per S_A slot");
    const unsigned char* kbuf = sm.kb[buf];
    const unsigned char* vbuf = sm.vb[buf];
    const int qw = qi - (w - 1);
    const int dqh = qi - jbase - 4 * half;  // contiguous tiles: key number cst + 4*half sits dqh - cst behind the query
    const int dqw = dqh - w;                // in the window  <=>  cst > dqw
    const unsigned char* krA = kbuf + (col % S::NL) * S::GSK + (col / S::NL) * S::RB + 16 * half;
    const unsigned char* krB = kbuf + ((32 + col) % S::NL) * S::GSK + ((32 + col) / S::NL) * S::RB + 16 * half;
    // The A operand of O^T += V^T.P^T comes through transposing LDS loads: within each group of
    // 16 lanes, lane r points at (row r/4, 4-column block r%4) of a 4-row x 16-column patch of V
    // and receives the 4 rows of column r.  MFMA g (16 keys) uses rows 16g + 4*half + {0..3}
    // (k-slots 0..3) and 16g + 8 + 4*half + {0..3} (k-slots 4..7): the key order P^T already has.
    const int r16 = lane & 15, grp2 = (lane >> 4) & 1;
    const int vcol = (16 * grp2 + 4 * (r16 & 3)) * 2;
    const int vrow = 4 * half + (r16 >> 2);
    auto v_operand = [&](int g, int x) -> bf16x8 {
        const int row0 = 16 * g + vrow;
        const int row1 = row0 + 8;
        const unsigned char* v0 = vbuf + (row0 % S::NL) * S::GSV + (row0 / S::NL) * S::RB + vcol + 64 * x;
        const unsigned char* v1 = vbuf + (row1 % S::NL) * S::GSV + (row1 / S::NL) * S::RB + vcol + 64 * x;
        const i16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3)))*)v0);
        const i16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3)))*)v1);
        const bf16x4 lo = __builtin_bit_cast(bf16x4, lo4), hi = __builtin_bit_cast(bf16x4, hi4);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto operand = [&](int n) -> bf16x8 {  // n is a compile-time constant after unrolling
        if (n < NS) return *(const bf16x8*)(krA + 32 * n);
        if (n < 2 * NS) return *(const bf16x8*)(krB + 32 * (n - NS));
        const int i = n - 2 * NS;
        return v_operand(i / DB, i % DB);
    };

    HalfState A, B;
    f32x16 sA, sB;
#pragma unroll
    for (int r = 0; r < 16; r++) { sA[r] = 0.0f; sB[r] = 0.0f; }
    bf16x8 ring[DEPTH];
#pragma unroll
    for (int n = 0; n < DEPTH; n++) ring[n] = operand(n);
    TileRows<D, 64> rows;
    if (more) rows = tile_rows<D, 64>(jp_next, wv, lane);
    load_meta<MODE, KIND>(A, ju, 0, half);
    __builtin_amdgcn_sched_barrier(0);
    // ---- S_A, then S_B with softmax(A) ----
    static_for<0, 2 * NS>([&](auto nc) {
        constexpr int n = decltype(nc)::value;
        const bf16x8 cur = ring[n % DEPTH];
        if constexpr (n < NS) sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, qreg[n], sA, 0, 0, 0);
        else sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, qreg[n - NS], sB, 0, 0, 0);
        if (n + DEPTH < NSLOT) ring[n % DEPTH] = operand(n + DEPTH);
        // the gather of the next tile rides on the S_A slots, whose issue is otherwise idle
        // (every wave is past this tile's barrier, so the other buffer is free)
        if (n < NX && more) tile_load_step<D, 64>(sm, buf ^ 1, rows, n, kh, vh, wv, lane);
        if (n >= NS) {
            constexpr int s = n >= NS ? n - NS : 0;
            softmax_slices<MODE, KIND, US * s, US * (s + 1)>(A, sA, jdeath, half, 0, qw, dqh, dqw, tau_q, c2, ref);
            if (US * (s + 1) == 4) load_meta<MODE, KIND>(B, ju, 1, half);
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    // (the empty asm uses keep the compiler from sinking the exponentials below the rescale branch)
    asm volatile("" ::"v"(A.pb[0]), "v"(A.pb[1]), "v"(A.psum));
    l_run = l_run * A.alpha + A.psum;
    rescale_o<D>(acc_o, A.alpha);
    // ---- O^T += V_A^T . P_A^T with softmax(B) ----
    static_for<0, NP>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int n = 2 * NS + i;
        const bf16x8 cur = ring[n % DEPTH];
        acc_o[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, A.pb[i / DB], acc_o[i % DB], 0, 0, 0);
        if (n + DEPTH < NSLOT) ring[n % DEPTH] = operand(n + DEPTH);
        softmax_slices<MODE, KIND, UP * i, UP * (i + 1)>(B, sB, jdeath, half, 1, qw, dqh, dqw, tau_q, c2, ref);
        __builtin_amdgcn_sched_barrier(0);
    });
    asm volatile("" ::"v"(B.pb[0]), "v"(B.pb[1]), "v"(B.psum));
    l_run = l_run * B.alpha + B.psum;
    rescale_o<D>(acc_o, B.alpha);
    // ---- O^T += V_B^T . P_B^T ----
    static_for<0, NP>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int n = 2 * NS + NP + i;
        const bf16x8 cur = ring[n % DEPTH];
        acc_o[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, B.pb[i / DB], acc_o[i % DB], 0, 0, 0);
        if (n + DEPTH < NSLOT) ring[n % DEPTH] = operand(n + DEPTH);
    });
}

// The tiles [T, T_end) of the block's key set, all of one kind.  T counts the block's tiles; tile T uses K/V buffer
// T & 1 and the metadata of segment T / TPS.
template <int D, int MODE, int KIND>
__device__ __forceinline__ void run_tiles(FwdSmem<D>& sm, const StageSrc& src, int& T, int T_end, int jbase0,
                                          const uint16_t* kh, const uint16_t* vh, int wv, int col, int half,
                                          int lane, int qi, int w, float tau_q, float c2,
                                          const bf16x8 (&qreg)[D / 16], f32x16 (&acc_o)[D / 32], SoftRef& ref,
                                          float& l_run)
{
    for (; T < T_end; T++) {
        // tile T has landed (this wave's part: vmcnt; the other waves' parts: barrier); the
        // barrier also says that everybody is done with tile T-1, whose buffer is refilled next
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const int sg = T / TPS, lt = T - sg * TPS;
        // first tile of a segment: everybody has left the segment before, so its metadata buffer takes the next one
        if (lt == 0 && (sg + 1) * TPS < src.nt) stage_meta(sm, src, sg + 1, wv, lane);
        const int sgn = (T + 1) / TPS;
        const int32_t* jp_next = sm.jpos[sgn & 1] + (T + 1 - sgn * TPS) * KT;
        const bool more = T + 1 < src.nt;
        if (KIND != TILE_SKIP)
            tile_body<D, MODE, KIND>(sm, T & 1, sm.jdeath[sg & 1] + lt * KT, sm.ju[sg & 1] + lt * KT, jp_next,
                                     jbase0 + T * KT, more, kh, vh, wv, col, half, lane, qi, w, tau_q, c2, qreg,
                                     acc_o, ref, l_run);
        else if (more)
            issue_tile_loads<D, 64>(sm, (T + 1) & 1, jp_next, kh, vh, wv, lane);
    }
}

// TAIL: workgroups behind the blocks move the rows that survive a chunk (an instance of its own: the registers are all taken).
// WGS: workgroups per compute unit.  Without gates and with 64 columns three fit at the cost of 3 spilled registers (96 heads of 4096,
// k = w = 256: 125.3 -> 114.5 us for the prefill; 64 heads of 8192 at k = 512, w = 700: 249.0 -> 232.7; see three_per_cu for where they
// lose).  With gates it takes 29 of them and loses (135 -> 199, 631 -> 766).
template <int D, int MODE, bool TAIL, int WGS>
__global__ __launch_bounds__(256, WGS) void attn_fwd_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kk, const uint16_t* __restrict__ v,
    const float* __restrict__ u, const float* __restrict__ tau, const int32_t* __restrict__ death,
    const int32_t* __restrict__ xpos, const int32_t* __restrict__ xdeath, const float* __restrict__ xu, int KP,
    const int32_t* __restrict__ counts, uint16_t* __restrict__ o,
    float* __restrict__ lse, int H, int Gu, int n, int k, int w, float scale, int nb, int BH, int nrows,
    int q_begin, const int32_t* __restrict__ first_valid, int q_rows, ChunkTail tail)
{
    __shared__ __align__(16) FwdSmem<D> sm;
    constexpr int DS = D / 16;   // MFMA k-steps over the head dim
    constexpr int DB = D / 32;   // 32-row blocks of O^T
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;

    if (TAIL && (int)blockIdx.x >= nb * BH) {
        const int id = blockIdx.x - nb * BH, bh = id % BH;
        chunk_retain_rows(tail, bh, bh / H * Gu + (Gu == 1 ? 0 : bh % H), id / BH);
        return;
    }
    // ---- block -> (head, query block): heads are dealt to the 8 XCDs so that one head's
    // blocks share an L2; late (long) blocks go first
    int bh, blk;
    deal_block(blockIdx.x, nb, BH, bh, blk);
    const int b = bh / H, h = bh % H;
    const int row = b * Gu + (Gu == 1 ? 0 : h);
    const int i0 = blk * QB;
    if (i0 + QB <= q_begin) return;  // queries before q_begin are not wanted (chunked prefill)
    // q and o hold q_rows rows per head starting at query q_begin (0: all n rows)
    const ptrdiff_t qo = q_rows ? (ptrdiff_t)bh * q_rows - q_begin : (ptrdiff_t)bh * n;
    const uint16_t* qh = q + qo * D;
    const uint16_t* kh = kk + (size_t)bh * n * D;
    const uint16_t* vh = v + (size_t)bh * n * D;
    const float* tr = tau + (size_t)row * n;
    const int nstay = counts[(size_t)nrows * nb + (size_t)row * nb + blk];
    // keys before first_valid[row] (padding of a chunked prefill) are attended by nobody
    const int c0 = max(max(0, i0 - w + 1), first_valid ? first_valid[row] : 0);
    const int c_end = min(n - 1, i0 + QB - 1);
    // The list part is laid out for min(k, T0 + 1) keys, the length of a complete top-k list (known without a load);
    // a shorter list (lifetimes cleared by a chunked prefill) ends in padding that nobody attends.
    const int T0 = i0 - w;
    const int nkl = (T0 >= 0 && k > 0) ? (min(k, T0 + 1) + KT - 1) / KT * KT : 0;   // list part, whole tiles
    const int nkc = max(0, (c_end - c0 + 1 + KT - 1) / KT * KT);                    // contiguous part, padded
    const int NT = (nkl + nkc) / KT;

    StageSrc src;
    {
        const size_t xo = ((size_t)row * nb + blk) * (size_t)KP;
        src.xpos = xpos + xo;
        src.xdeath = xdeath + xo;
        src.xu = xu + xo;
        src.dr = death + (size_t)row * n;
        src.ur = u + (size_t)row * n;
        src.nkl = nkl;
        src.c0 = c0;
        src.c_end = c_end;
        src.nt = NT;
    }

    // ---- this wave's queries ----
    const int qa = i0 + 32 * wv;          // first query of the wave
    const int qb = min(qa + 31, n - 1);   // last real query of the wave
    const int qi = qa + col;              // this lane's query
    const bool wave_live = qa < n;
    const int qrow = min(qi, n - 1);
    const float tau_q = (qi < n && qi - w >= 0) ? tr[qi - w] : 0.0f;
    bf16x8 qreg[DS];
#pragma unroll
    for (int s = 0; s < DS; s++)
        qreg[s] = *(const bf16x8*)(qh + (size_t)qrow * D + 16 * s + 8 * half);
    // the first segment of metadata: its copies need nothing that is loaded above, so they fly together
    stage_meta(sm, src, 0, wv, lane);

    // ---- the runs of tile kinds for this wave, as tile numbers (all wave-uniform) ----
    const WaveRuns wr = wave_runs(wave_live, nkl, nkc, nstay, qa, qb, w, c0);
    const int b0 = wr.b0, b1 = wr.b1, b2 = wr.b2, b3 = wr.b3, b4 = wr.b4;
    const bool narrow = wr.narrow;

    f32x16 acc_o[DB];
#pragma unroll
    for (int x = 0; x < DB; x++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc_o[x][r] = 0.0f;
    SoftRef ref{-INFINITY, 0.0f};
    float l_run = 0.0f;
    const float c2 = scale * 1.4426950408889634f;

    // The metadata copies and the tile gathers are direct-to-LDS loads that the compiler does not track.  Everything
    // it does track (the Q fragments, tau, the counts) is waited for here, ahead of the first gather: left to their
    // first use inside the tile loop, those waits would count the prefetched tile too and drain it early.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < DS; s++) asm volatile("" ::"v"(qreg[s]));
    __syncthreads();  // segment 0 of the metadata is in place
    if (NT > 0) issue_tile_loads<D, 64>(sm, 0, sm.jpos[0], kh, vh, wv, lane);
    {
        const int jbase0 = c0 - nkl;     // position of tile 0's first key if the whole key set were contiguous
        int T = 0;
#define SPK_RUN(KIND, bound)                                                                                     \
    run_tiles<D, MODE, KIND>(sm, src, T, min(NT, (bound)), jbase0, kh, vh, wv, col, half, lane, qi, w, tau_q, c2, \
                             qreg, acc_o, ref, l_run)
        SPK_RUN(TILE_LIST, b0);
        SPK_RUN(TILE_LIST_MASK, b1);
        if (narrow) SPK_RUN(TILE_CONT, b2);
        else SPK_RUN(TILE_EDGE, b2);
        SPK_RUN(TILE_FAST, b3);
        SPK_RUN(TILE_DIAG, b4);
        SPK_RUN(TILE_SKIP, NT);
#undef SPK_RUN
    }

    // ---- epilogue: O = O^T / l, lse ----
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    if (qi < n) {
        const float inv = 1.0f / l_tot;
        uint16_t* orow = o + (qo + qi) * D;
#pragma unroll
        for (int x = 0; x < DB; x++) {
#pragma unroll
            for (int g4 = 0; g4 < 4; g4++) {
                bf16x4 pk;
#pragma unroll
                for (int e = 0; e < 4; e++) pk[e] = (__bf16)(acc_o[x][4 * g4 + e] * inv);
                *(bf16x4*)(orow + 32 * x + 8 * g4 + 4 * half) = pk;
            }
        }
        if (lse && half == 0) lse[qo + qi] = (ref.m * c2 + log2f(l_tot)) * 0.6931471805599453f;
    }
}

template <typename T>
static void launch_generic(const sparsek_cfg& c, const void* q, const void* k, const void* v, const float* u,
                           const float* tau, const int32_t* death, const int32_t* lists, const int32_t* counts, void* o,
                           float* lse, int nb, int q_begin, const int32_t* first_valid, int q_rows, hipStream_t st)
{
    dim3 grid(nb * GEN_SPLIT, c.B * c.H);
#define SPK_LAUNCH_G(DT, OWN)                                                                                              \
    hipLaunchKernelGGL((attn_fwd_generic_kernel<T, DT, OWN>), grid, dim3(256), 0, st, (const T*)q, (const T*)k, (const T*)v, \
                       u, tau, death, lists, counts, (T*)o, lse, c.H, c.Gu, c.n, c.d, c.k, c.w, c.gate_mode,                 \
                       c.softmax_scale, nb, q_begin, first_valid, q_rows)
    if (lists) {
        if (c.d <= 32) SPK_LAUNCH_G(2, false);
        else if (c.d <= 64) SPK_LAUNCH_G(4, false);
        else SPK_LAUNCH_G(8, false);
    } else if (c.d <= 32) SPK_LAUNCH_G(2, true);
    else if (c.d <= 64) SPK_LAUNCH_G(4, true);
    else SPK_LAUNCH_G(8, true);
#undef SPK_LAUNCH_G
}

template <int D>
static void launch_mfma(const sparsek_cfg& c, const void* q, const void* k, const void* v, const float* u,
                        const float* tau, const int32_t* death, const ExtLists& x, const int32_t* counts,
                        void* o, float* lse, int nb, int q_begin, const int32_t* first_valid,
                        int q_rows, const ChunkTail& tail, hipStream_t st)
{
    const int BH = c.B * c.H;
    dim3 grid((nb + tail.wgs) * BH);
#define SPK_LAUNCH(MODE, TAIL, WGS)                                                                               \
    hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, MODE, TAIL, WGS>), grid, dim3(256), 0, st, (const uint16_t*)q,         \
                       (const uint16_t*)k, (const uint16_t*)v, u, tau, death, (const int32_t*)x.pos,              \
                       (const int32_t*)x.death, (const float*)x.u, x.KP, counts, (uint16_t*)o, lse, c.H, c.Gu,    \
                       c.n, c.k, c.w, c.softmax_scale, nb, BH, c.B * c.Gu, q_begin, first_valid, q_rows, tail)
    constexpr int MOST = D == 64 ? 3 : 2;
    const bool most = D == 64 && three_per_cu(c, q_begin);
    if (tail.wgs) {
        if (c.gate_mode == 0) SPK_LAUNCH(0, true, 2);
        else if (c.gate_mode == 1) SPK_LAUNCH(1, true, 2);
        else if (most) SPK_LAUNCH(2, true, MOST);
        else SPK_LAUNCH(2, true, 2);
    } else if (c.gate_mode == 0) SPK_LAUNCH(0, false, 2);
    else if (c.gate_mode == 1) SPK_LAUNCH(1, false, 2);
    else if (most) SPK_LAUNCH(2, false, MOST);
    else SPK_LAUNCH(2, false, 2);
#undef SPK_LAUNCH
}

void launch_block_lists_ext(const sparsek_cfg& c, const int32_t* death, int32_t* lists, int32_t* counts,
                            const float* u, const ExtLists& x, hipStream_t st, int q_begin, const ChunkTail* tail)
{
    const int nb = nblocks(c.n), blk0 = tail ? q_begin / QB : 0, nl = nb - blk0;
    // Up to 256 blocks: a compute unit for each.  More: two workgroups per compute unit, and runs of up to 16 blocks
    // once there are several rounds of them.
    const long long blocks = (long long)nl * c.B * c.Gu;
    const int run = (int)std::max(1ll, std::min(16ll, blocks / 512));
    const ChunkTail t = tail ? *tail : ChunkTail{};
#define SPK_LISTS(REG, RUNS, CHUNK)                                                                                       \
    hipLaunchKernelGGL((block_lists_kernel<REG, RUNS, CHUNK>), dim3((RUNS ? (nl + run - 1) / run : nl) + (CHUNK ? 1 : 0), c.B * c.Gu), \
                       dim3(64 * BL_WAVES), 0, st, death, c.n, c.k, c.w, nb, RUNS ? run : 1, lists, counts, u, x.pos, x.death, \
                       x.u, x.KP, blk0, t)
    if (blocks > 256) {
        if (tail) SPK_LISTS(8, true, true);
        else SPK_LISTS(8, true, false);
    } else {
        if (tail) SPK_LISTS(32, false, true);
        else SPK_LISTS(32, false, false);
    }
#undef SPK_LISTS
}

void launch_block_lists(const sparsek_cfg& c, const int32_t* death, int32_t* lists, int32_t* counts,
                        hipStream_t st)
{
    launch_block_lists_ext(c, death, lists, counts, nullptr, ExtLists{nullptr, nullptr, nullptr, 0}, st);
}

bool attn_fwd_mfma(const sparsek_cfg& c)
{
    return c.dtype == SPARSEK_BF16 && (c.d == 64 || c.d == 128) && (uint64_t)c.n * c.d * 2 <= 0xFFFFFFFFull;
}

static ExtLists fwd_ext_lists(const sparsek_cfg& c, char* ws, size_t lb)
{
    const size_t xb = ext_array_bytes(c);
    return ExtLists{(int32_t*)(ws + lb), (int32_t*)(ws + lb + xb), (float*)(ws + lb + 2 * xb), (int)ext_stride(c)};
}

FwdLists attn_fwd_lists(const sparsek_cfg& c, const void* ws)
{
    if (!attn_fwd_mfma(c)) return FwdLists{};
    size_t coff = 0;
    const size_t lb = block_lists_bytes(c, &coff);
    const ExtLists x = fwd_ext_lists(c, (char*)ws, lb);
    return FwdLists{(const int32_t*)ws, (const int32_t*)((const char*)ws + coff), x.pos, x.death, x.u};
}

int launch_attn_fwd(const sparsek_cfg& c, const void* q, const void* k, const void* v, const float* u,
                    const float* tau, const int32_t* death, void* o, float* lse, void* ws,
                    hipStream_t st, int q_begin, const int32_t* first_valid, int q_rows, const ChunkTail* tail)
{
    const int nb = nblocks(c.n);
    size_t coff = 0;
    const size_t lb = block_lists_bytes(c, &coff);
    int32_t* lists = (int32_t*)ws;
    int32_t* counts = (int32_t*)((char*)ws + coff);
    if (attn_fwd_mfma(c)) {
        const ExtLists x = fwd_ext_lists(c, (char*)ws, lb);
        launch_block_lists_ext(c, death, lists, counts, u, x, st, q_begin, tail);
        ChunkTail t = tail ? *tail : ChunkTail{};
        // a workgroup of the row copy takes 16 KB or more of each tensor; 2048 of them are four rounds of what the chip holds
        t.wgs = tail ? (int)std::max<long long>(1, std::min<long long>(((long long)t.rcap * t.unit + 1023) / 1024, 2048 / std::max(1, c.B * c.H))) : 0;
        if (c.d == 64) launch_mfma<64>(c, q, k, v, u, tau, death, x, counts, o, lse, nb, q_begin, first_valid, q_rows, t, st);
        else launch_mfma<128>(c, q, k, v, u, tau, death, x, counts, o, lse, nb, q_begin, first_valid, q_rows, t, st);
        return launch_status();
    }
    // The line lies where a workgroup's registers and LDS end; below it the lists were slower wherever both were timed (37 sizes of 4 to
    // 256 heads).  us with the lists / without, mask and all: one head of 1024, k = w = 64, d = 64 24.7 / 21.6; 16 heads of 2048,
    // k = w = 128, d = 64 85 / 75; the least was gained with many heads, few columns and a full scan: 256 heads of 4096, k = w = 64,
    // d = 32 705 / 666, 32 heads of 4096, k = 64, w = 1024 348 / 332, k = 1024, w = 64 374 / 338.
    if (c.n <= GEN_N && c.k <= GEN_K) lists = nullptr;
    else launch_block_lists(c, death, lists, counts, st);
    if (c.dtype == SPARSEK_F32)
        launch_generic<float>(c, q, k, v, u, tau, death, lists, counts, o, lse, nb, q_begin, first_valid, q_rows, st);
    else
        launch_generic<uint16_t>(c, q, k, v, u, tau, death, lists, counts, o, lse, nb, q_begin, first_valid, q_rows, st);
    return launch_status();
}

}  // namespace spk
