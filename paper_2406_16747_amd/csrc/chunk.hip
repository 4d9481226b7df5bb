// Chunk-wise recurrent prefill with a fixed-size scored cache (Sec. 3.4, "training with
// fixed-size truncation-free cache": attend the chunk against the cache, add the chunk's
// key-value pairs and scores, prune by score).  The result equals the unchunked computation.
//
// What must survive a chunk is decided by the SPARSEK threshold, which never decreases: a key
// whose score is not above the threshold of the last prefix used so far can neither be selected
// again nor enter the support of a later threshold.  So the state keeps, per score row and in
// position order, the scores of (a) every key older than the window that is still above that
// threshold (the top-k are among them) and (b) the last w keys, together with their K/V rows:
// at most R_cap = k + w + cand_cap entries, independent of the sequence length.
//
// A call builds a "virtual sequence"  [ padding | retained entries | chunk ]  of fixed length
// R_cap + c, runs the ordinary mask and attention kernels on it (only the chunk's queries are
// evaluated) and compacts the survivors back into the state.  Inside the virtual sequence
// distances of at most w are preserved (the last w retained entries are the true window), and
// dropped keys cannot change any threshold or selection, so every chunk query sees exactly the
// keys and gates of the unchunked run.  The mask and attention kernels are told the first real
// position: rows start there, and the padding is kept out of every query's key set (lifetimes cleared).
#include "common.hpp"

namespace spk {

struct ChunkLayout {
    int rcap;                              // capacity of the retained set (multiple of 128)
    size_t count, flags, ret_u, ret_sel, ret_k, ret_v, total;
};

static int chunk_rcap(const sparsek_chunk_cfg& c)
{
    const int cand = c.cand_cap > 0 ? c.cand_cap : 4 * (c.k > 16 ? c.k : 16);
    return (c.k + c.w + cand + 127) / 128 * 128;
}

static size_t esize(int dtype) { return dtype == SPARSEK_BF16 ? 2 : 4; }

static ChunkLayout chunk_layout(const sparsek_chunk_cfg& c)
{
    ChunkLayout L;
    L.rcap = chunk_rcap(c);
    const size_t rows = (size_t)c.B * c.Gu, BH = (size_t)c.B * c.H;
    size_t off = 0;
    L.count = off; off += align_up(rows * 4, 256);
    L.flags = off; off += align_up(rows * 4, 256);
    L.ret_u = off; off += align_up(rows * L.rcap * 4, 256);
    L.ret_sel = off; off += align_up(rows * L.rcap * 4, 256);
    L.ret_k = off; off += align_up(BH * L.rcap * c.d * esize(c.dtype), 256);
    L.ret_v = off; off += align_up(BH * L.rcap * c.d * esize(c.dtype), 256);
    L.total = off;
    return L;
}

size_t chunk_state_bytes(const sparsek_chunk_cfg& c) { return chunk_layout(c).total; }

static sparsek_cfg virtual_cfg(const sparsek_chunk_cfg& c, int nv)
{
    sparsek_cfg v;
    v.B = c.B; v.H = c.H; v.Gu = c.Gu; v.n = nv; v.d = c.d; v.k = c.k; v.w = c.w;
    v.dtype = c.dtype;
    v.gate_mode = c.gate_mode == 3 ? 2 : c.gate_mode;
    v.softmax_scale = c.softmax_scale;
    return v;
}

struct ChunkWs {
    size_t u, tau, death, map, first, lse, k, v, mask, attn, total;
};
static ChunkWs chunk_ws(const sparsek_chunk_cfg& c, int clen)
{
    const ChunkLayout L = chunk_layout(c);
    const int nv = L.rcap + clen;
    const size_t rows = (size_t)c.B * c.Gu, BH = (size_t)c.B * c.H;
    const sparsek_cfg v = virtual_cfg(c, nv);
    ChunkWs W;
    size_t off = 0;
    W.u = off; off += align_up(rows * nv * 4, 256);
    W.tau = off; off += align_up(rows * nv * 4, 256);
    W.death = off; off += align_up(rows * nv * 4, 256);
    W.map = off; off += align_up(rows * L.rcap * 4, 256);
    W.first = off; off += align_up(rows * 4, 256);
    W.lse = off; off += align_up(BH * (size_t)clen * 4, 256);
    const size_t tens = align_up(BH * nv * c.d * esize(c.dtype), 256);
    W.k = off; off += tens;
    W.v = off; off += tens;
    W.mask = off; off += align_up(mask_ws_bytes(v), 256);
    W.attn = off; off += align_up(attn_fwd_ws_bytes(v), 256);
    W.total = off;
    return W;
}
size_t chunk_ws_bytes(const sparsek_chunk_cfg& c) { return chunk_ws(c, c.chunk_max).total; }

__global__ void chunk_init_kernel(int32_t* count, int32_t* flags, int rows)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows) { count[i] = 0; flags[i] = 0; }
}

// Scores of the virtual sequence of one row: padding (-inf, nobody looks at it), retained, chunk.
__global__ __launch_bounds__(1024) void chunk_assemble_scores_kernel(const int32_t* __restrict__ count,
                                                                     const float* __restrict__ ret_u,
                                                                     const float* __restrict__ u_chunk, int rcap,
                                                                     int clen, float* __restrict__ u_v,
                                                                     int32_t* __restrict__ first_valid)
{
    const int row = blockIdx.y;
    const int pad = rcap - count[row], nv = rcap + clen;
    const int e = blockIdx.x * 1024 + threadIdx.x;
    if (e == 0) first_valid[row] = pad;
    if (e < nv)
        u_v[(size_t)row * nv + e] = e < pad ? -INFINITY : e < rcap ? ret_u[(size_t)row * rcap + (e - pad)]
                                                                   : u_chunk[(size_t)row * clen + (e - rcap)];
}

// K and V rows of the virtual sequence: moved by workgroups of the mask's launch.  (Q and O stay in the caller's chunk
// tensors: the attention kernel addresses them from its first query.)
static RowCopy chunk_rows(const sparsek_chunk_cfg& c, const ChunkLayout& L, char* state, const void* k, const void* v,
                          int clen, char* kd, char* vd)
{
    return RowCopy{(const int32_t*)(state + L.count), (const uint4*)(state + L.ret_k), (const uint4*)(state + L.ret_v),
                   (const uint4*)k, (const uint4*)v, (uint4*)kd, (uint4*)vd, c.Gu == 1 ? c.H : 1, L.rcap, clen, c.w,
                   (int)(c.d * esize(c.dtype) / 16), 0};
}

// Padding entries are never selected: death[e] = e.  The same holds for retained keys that were
// kept only because their score is above the threshold: they left the top-k in an earlier chunk, at
// a prefix whose block the mask skips, so their lifetime is still at its preset.
__global__ void chunk_clear_padding_kernel(const int32_t* __restrict__ count, const int32_t* __restrict__ ret_sel,
                                           int rcap, int nv, int32_t* __restrict__ death)
{
    const int row = blockIdx.y;
    const int pad = rcap - count[row];
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rcap) return;
    if (e < pad || !ret_sel[(size_t)row * rcap + (e - pad)]) death[(size_t)row * nv + e] = e;
}

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

__global__ __launch_bounds__(1024) void chunk_retain_kernel(int32_t* __restrict__ count, int32_t* __restrict__ flags,
                                                            const float* __restrict__ u_v,
                                                            const float* __restrict__ tau_v,
                                                            const int32_t* __restrict__ death_v, int rcap, int clen,
                                                            int w, int32_t* __restrict__ map, float* __restrict__ ret_u,
                                                            int32_t* __restrict__ ret_sel)
{
    __shared__ int wt[2][16];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nv = rcap + clen;
    const int pad = rcap - count[row];
    const int T = nv - 1 - w;  // last prefix any query has used
    const float* ur = u_v + (size_t)row * nv;
    const int32_t* dr = death_v + (size_t)row * nv;
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
            dd[x] = dr[e];
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

__global__ __launch_bounds__(256) void chunk_retain_rows_kernel(const int32_t* __restrict__ count,
                                                                const int32_t* __restrict__ map,
                                                                const uint4* __restrict__ k_v,
                                                                const uint4* __restrict__ v_v, int H, int Gu, int rcap,
                                                                int nv, int row16, uint4* __restrict__ ret_k,
                                                                uint4* __restrict__ ret_v)
{
    const int bh = blockIdx.y;
    const int b = bh / H, h = bh % H;
    const int row = b * Gu + (Gu == 1 ? 0 : h);
    const size_t total = (size_t)count[row] * row16;
    for (size_t x = (size_t)blockIdx.x * 256 + threadIdx.x; x < total; x += (size_t)gridDim.x * 256) {
        const int j = (int)(x / row16), c16 = (int)(x % row16);
        const int e = map[(size_t)row * rcap + j];
        const size_t src = ((size_t)bh * nv + e) * row16 + c16;
        const size_t dst = ((size_t)bh * rcap + j) * row16 + c16;
        ret_k[dst] = k_v[src];
        ret_v[dst] = v_v[src];
    }
}

int launch_chunk_init(const sparsek_chunk_cfg& c, void* state, hipStream_t st)
{
    const ChunkLayout L = chunk_layout(c);
    const int rows = c.B * c.Gu;
    char* s = (char*)state;
    hipLaunchKernelGGL(chunk_init_kernel, dim3((rows + 255) / 256), dim3(256), 0, st, (int32_t*)(s + L.count),
                       (int32_t*)(s + L.flags), rows);
    return launch_status();
}

int launch_chunk_prefill(const sparsek_chunk_cfg& c, void* state, int clen, const void* q, const void* k,
                         const void* v, const float* u, void* o, void* ws, hipStream_t st)
{
    const ChunkLayout L = chunk_layout(c);
    const ChunkWs W = chunk_ws(c, clen);
    const int rows = c.B * c.Gu, BH = c.B * c.H;
    const int nv = L.rcap + clen;
    const int row16 = (int)(c.d * esize(c.dtype) / 16);
    char* s = (char*)state;
    char* w = (char*)ws;
    int32_t* count = (int32_t*)(s + L.count);
    int32_t* flags = (int32_t*)(s + L.flags);
    float* ret_u = (float*)(s + L.ret_u);
    uint4* ret_k = (uint4*)(s + L.ret_k);
    uint4* ret_v = (uint4*)(s + L.ret_v);
    float* u_v = (float*)(w + W.u);
    float* tau_v = (float*)(w + W.tau);
    int32_t* death_v = (int32_t*)(w + W.death);
    int32_t* map = (int32_t*)(w + W.map);
    int32_t* first_valid = (int32_t*)(w + W.first);
    uint4* k_v = (uint4*)(w + W.k);
    uint4* v_v = (uint4*)(w + W.v);
    const sparsek_cfg cv = virtual_cfg(c, nv);

    hipLaunchKernelGGL(chunk_assemble_scores_kernel, dim3((nv + 1023) / 1024, rows), dim3(1024), 0, st, count, ret_u, u, L.rcap, clen, u_v,
                       first_valid);
    const RowCopy copy = chunk_rows(c, L, s, k, v, clen, w + W.k, w + W.v);
    // thresholds are needed from prefix R_cap - w - 1 on (the last one the previous call used)
    int rc = launch_mask(cv, u_v, tau_v, death_v, w + W.mask, st, std::max(0, L.rcap - c.w - 1), first_valid, &copy);
    if (rc) return rc;
    hipLaunchKernelGGL(chunk_clear_padding_kernel, dim3((L.rcap + 255) / 256, rows), dim3(256), 0, st, count,
                       (const int32_t*)(s + L.ret_sel), L.rcap, nv, death_v);
    rc = launch_attn_fwd(cv, q, k_v, v_v, u_v, tau_v, death_v, o, (float*)(w + W.lse), w + W.attn, st, L.rcap,
                         first_valid, clen);
    if (rc) return rc;
    hipLaunchKernelGGL(chunk_retain_kernel, dim3(rows), dim3(1024), 0, st, count, flags, u_v, tau_v, death_v, L.rcap,
                       clen, c.w, map, ret_u, (int32_t*)(s + L.ret_sel));
    const int gr = (int)std::min<size_t>(((size_t)L.rcap * row16 + 255) / 256, 2048);
    hipLaunchKernelGGL(chunk_retain_rows_kernel, dim3(gr, BH), dim3(256), 0, st, count, map, k_v, v_v, c.H, c.Gu,
                       L.rcap, nv, row16, ret_k, ret_v);
    return launch_status();
}

// Backward of one chunk with the cache's gradient stopped (training with chunk-wise recurrence, Algorithm 3):
// the gradients of L = sum(dO * O_chunk) with respect to the chunk's own q, k, v and scores, the retained keys
// being constants.  The forward call left the virtual sequence (scores, thresholds, lifetimes, K and V rows, lse)
// in its workspace; the ordinary backward kernels run on it with the queries offset to the chunk, and only
// keys from the chunk on receive dk, dv, du.
struct ChunkBwdWs {
    size_t du, attn, mask, total;
};
static ChunkBwdWs chunk_bwd_ws(const sparsek_chunk_cfg& c, int clen)
{
    const ChunkLayout L = chunk_layout(c);
    const int nv = L.rcap + clen;
    sparsek_cfg v = virtual_cfg(c, nv);
    ChunkBwdWs W;
    size_t off = 0;
    W.du = off; off += align_up((size_t)c.B * c.Gu * nv * 4, 256);
    W.attn = off; off += align_up(attn_bwd_ws_bytes(v), 256);
    v.gate_mode = c.gate_mode;
    W.mask = off; off += align_up(mask_bwd_ws_bytes(v), 256);
    W.total = off;
    return W;
}
size_t chunk_bwd_ws_bytes(const sparsek_chunk_cfg& c) { return chunk_bwd_ws(c, c.chunk_max).total; }

__global__ void chunk_slice_du_kernel(const float* __restrict__ du_v, int nv, int rcap, int clen, float* __restrict__ du)
{
    const int row = blockIdx.y;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < clen; x += gridDim.x * blockDim.x)
        du[(size_t)row * clen + x] = du_v[(size_t)row * nv + rcap + x];
}

int launch_chunk_bwd(const sparsek_chunk_cfg& c, int clen, const void* q, const void* o, const void* dO,
                     const void* fwd_ws, void* dq, void* dk, void* dv, float* du, void* ws, hipStream_t st)
{
    const ChunkLayout L = chunk_layout(c);
    const ChunkWs W = chunk_ws(c, clen);
    const ChunkBwdWs Bw = chunk_bwd_ws(c, clen);
    const int rows = c.B * c.Gu;
    const int nv = L.rcap + clen;
    const char* w = (const char*)fwd_ws;
    char* b = (char*)ws;
    const float* u_v = (const float*)(w + W.u);
    const float* tau_v = (const float*)(w + W.tau);
    const int32_t* death_v = (const int32_t*)(w + W.death);
    const int32_t* first_valid = (const int32_t*)(w + W.first);
    const float* lse = (const float*)(w + W.lse);
    const void* k_v = w + W.k;
    const void* v_v = w + W.v;
    sparsek_cfg cv = virtual_cfg(c, nv);
    cv.gate_mode = c.gate_mode;  // (the straight-through mode has its own score gradient)
    float* du_v = (float*)(b + Bw.du);
    const int rc = launch_bwd(cv, q, k_v, v_v, u_v, tau_v, death_v, o, lse, dO, dq, dk, dv, du_v, b + Bw.attn, b + Bw.mask, st,
                              L.rcap, first_valid, clen, std::max(0, L.rcap - c.w - 1));
    if (rc) return rc;
    hipLaunchKernelGGL(chunk_slice_du_kernel, dim3((clen + 255) / 256, rows), dim3(256), 0, st, du_v, nv, L.rcap, clen, du);
    return launch_status();
}

// Decode state after the tokens consumed so far: the retained entries alone (no chunk) form a
// virtual history whose last prefix has the true threshold and top-k, which is all the decode
// state is built from.  Needs at least k + w consumed tokens: with fewer, the padding would make
// a short prefix look long to the loader.
int launch_decode_load(const sparsek_decode_cfg& c, void* state, int n_ctx, const void* k, const void* v,
                       const float* u, const float* tau, const int32_t* death, hipStream_t st);

int launch_chunk_to_decode(const sparsek_chunk_cfg& c, void* state, void* ws, const sparsek_decode_cfg& dc,
                           void* dstate, hipStream_t st)
{
    const ChunkLayout L = chunk_layout(c);
    const ChunkWs W = chunk_ws(c, 0);
    const int rows = c.B * c.Gu;
    const int nv = L.rcap;
    char* s = (char*)state;
    char* w = (char*)ws;
    int32_t* count = (int32_t*)(s + L.count);
    float* u_v = (float*)(w + W.u);
    float* tau_v = (float*)(w + W.tau);
    int32_t* death_v = (int32_t*)(w + W.death);
    uint4* k_v = (uint4*)(w + W.k);
    uint4* v_v = (uint4*)(w + W.v);
    const sparsek_cfg cv = virtual_cfg(c, nv);
    hipLaunchKernelGGL(chunk_assemble_scores_kernel, dim3((nv + 1023) / 1024, rows), dim3(1024), 0, st, count, (const float*)(s + L.ret_u),
                       (const float*)nullptr, L.rcap, 0, u_v, (int32_t*)(w + W.first));
    const RowCopy copy = chunk_rows(c, L, s, nullptr, nullptr, 0, w + W.k, w + W.v);
    int rc = launch_mask(cv, u_v, tau_v, death_v, w + W.mask, st, std::max(0, L.rcap - c.w - 1), (const int32_t*)(w + W.first), &copy);
    if (rc) return rc;
    hipLaunchKernelGGL(chunk_clear_padding_kernel, dim3((L.rcap + 255) / 256, rows), dim3(256), 0, st, count,
                       (const int32_t*)(s + L.ret_sel), L.rcap, nv, death_v);
    return launch_decode_load(dc, dstate, nv, k_v, v_v, u_v, tau_v, death_v, st);
}

int chunk_status(const sparsek_chunk_cfg& c, const void* state, int32_t* host_counts, int32_t* host_flags,
                 hipStream_t st)
{
    const ChunkLayout L = chunk_layout(c);
    const size_t rows = (size_t)c.B * c.Gu;
    const char* s = (const char*)state;
    if (host_counts && hipMemcpyAsync(host_counts, s + L.count, rows * 4, hipMemcpyDeviceToHost, st) != hipSuccess)
        return SPARSEK_ERR_LAUNCH;
    if (host_flags && hipMemcpyAsync(host_flags, s + L.flags, rows * 4, hipMemcpyDeviceToHost, st) != hipSuccess)
        return SPARSEK_ERR_LAUNCH;
    return hipStreamSynchronize(st) == hipSuccess ? SPARSEK_OK : SPARSEK_ERR_LAUNCH;
}

}  // namespace spk
