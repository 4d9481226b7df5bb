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
#include "chunk_parts.hpp"

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
    size_t u, tau, death, map, first, kept, lse, k, v, mask, attn, total;
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
    W.kept = off; off += align_up(rows * (size_t)(L.rcap / 64) * 8, 256);
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

// Scores of the virtual sequence of one row: padding (-inf, nobody looks at it), retained, chunk.  kept: which of the first rcap
// positions are neither padding nor retained for their score alone (a wave looks at 64 of them, all before rcap or none).
__global__ __launch_bounds__(1024) void chunk_assemble_scores_kernel(const int32_t* __restrict__ count,
                                                                     const float* __restrict__ ret_u,
                                                                     const int32_t* __restrict__ ret_sel,
                                                                     const float* __restrict__ u_chunk, int rcap,
                                                                     int clen, float* __restrict__ u_v,
                                                                     int32_t* __restrict__ first_valid,
                                                                     unsigned long long* __restrict__ kept)
{
    const int row = blockIdx.y;
    const int pad = rcap - count[row], nv = rcap + clen;
    const int e = blockIdx.x * 1024 + threadIdx.x;
    if (e == 0) first_valid[row] = pad;
    if (e < rcap) {
        const unsigned long long m = __ballot(e >= pad && ret_sel[(size_t)row * rcap + max(e - pad, 0)] != 0);
        if ((e & 63) == 0) kept[(size_t)row * (rcap / 64) + (e >> 6)] = m;
    }
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

// The parts of a chunk's end as launches of their own.
__global__ __launch_bounds__(1024) void chunk_retain_kernel(ChunkTail c)
{
    __shared__ RetainSmem sm;
    chunk_retain<true>(sm, c, blockIdx.x);
}

__global__ __launch_bounds__(256) void chunk_retain_rows_kernel(ChunkTail c, int H, int Gu)
{
    const int bh = blockIdx.y;
    chunk_retain_rows(c, bh, bh / H * Gu + (Gu == 1 ? 0 : bh % H), blockIdx.x);
}

__global__ __launch_bounds__(1024) void chunk_clear_padding_kernel(ChunkTail c) { chunk_clear_padding(c, blockIdx.x, threadIdx.x, 1024); }

int launch_chunk_init(const sparsek_chunk_cfg& c, void* state, hipStream_t st)
{
    const ChunkLayout L = chunk_layout(c);
    const int rows = c.B * c.Gu;
    char* s = (char*)state;
    hipLaunchKernelGGL(chunk_init_kernel, dim3((rows + 255) / 256), dim3(256), 0, st, (int32_t*)(s + L.count),
                       (int32_t*)(s + L.flags), rows);
    return launch_status();
}

static ChunkTail chunk_tail(const sparsek_chunk_cfg& c, const ChunkLayout& L, const ChunkWs& W, char* s, char* w, int clen)
{
    return ChunkTail{(const unsigned long long*)(w + W.kept), (int32_t*)(s + L.count), (int32_t*)(s + L.flags),
                     (const float*)(w + W.u), (const float*)(w + W.tau), (int32_t*)(w + W.death), L.rcap, clen, c.w,
                     (int32_t*)(w + W.map), (float*)(s + L.ret_u), (int32_t*)(s + L.ret_sel), (const uint4*)(w + W.k),
                     (const uint4*)(w + W.v), (uint4*)(s + L.ret_k), (uint4*)(s + L.ret_v), 0, 0};
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
    float* u_v = (float*)(w + W.u);
    float* tau_v = (float*)(w + W.tau);
    int32_t* death_v = (int32_t*)(w + W.death);
    int32_t* first_valid = (int32_t*)(w + W.first);
    uint4* k_v = (uint4*)(w + W.k);
    uint4* v_v = (uint4*)(w + W.v);
    const sparsek_cfg cv = virtual_cfg(c, nv);

    hipLaunchKernelGGL(chunk_assemble_scores_kernel, dim3((nv + 1023) / 1024, rows), dim3(1024), 0, st, count,
                       (const float*)(s + L.ret_u), (const int32_t*)(s + L.ret_sel), u, L.rcap, clen, u_v, first_valid, (unsigned long long*)(w + W.kept));
    const RowCopy copy = chunk_rows(c, L, s, k, v, clen, w + W.k, w + W.v);
    // thresholds are needed from prefix R_cap - w - 1 on (the last one the previous call used)
    int rc = launch_mask(cv, u_v, tau_v, death_v, w + W.mask, st, std::max(0, L.rcap - c.w - 1), first_valid, &copy);
    if (rc) return rc;
    ChunkTail tail = chunk_tail(c, L, W, s, w, clen);
    tail.unit = row16;
    // Where the MFMA kernels do the attention, the rest of the chunk rides on its launches: three launches less, the survivors are
    // found beside the lists and their rows move while the attention's last blocks run.  32 heads in chunks of 8192, k = w = 1024,
    // d = 128: 397 -> 381 us a chunk; 8 heads in chunks of 512, k = w = 64: 46 -> 39.
    if (attn_fwd_mfma(cv)) {
        rc = launch_attn_fwd(cv, q, k_v, v_v, u_v, tau_v, death_v, o, (float*)(w + W.lse), w + W.attn, st, L.rcap,
                             first_valid, clen, &tail);
        return rc ? rc : launch_status();
    }
    hipLaunchKernelGGL(chunk_clear_padding_kernel, dim3(rows), dim3(1024), 0, st, tail);
    rc = launch_attn_fwd(cv, q, k_v, v_v, u_v, tau_v, death_v, o, (float*)(w + W.lse), w + W.attn, st, L.rcap,
                         first_valid, clen);
    if (rc) return rc;
    hipLaunchKernelGGL(chunk_retain_kernel, dim3(rows), dim3(1024), 0, st, tail);
    tail.wgs = (int)std::min<size_t>(((size_t)L.rcap * row16 + 1023) / 1024, 512);
    hipLaunchKernelGGL(chunk_retain_rows_kernel, dim3(tail.wgs, BH), dim3(256), 0, st, tail, c.H, c.Gu);
    return launch_status();
}

// Backward of one chunk with the cache's gradient stopped (training with chunk-wise recurrence, Algorithm 3):
// the gradients of L = sum(dO * O_chunk) with respect to the chunk's own q, k, v and scores, the retained keys
// being constants.  The forward call left the virtual sequence (scores, thresholds, lifetimes, K and V rows, lse)
// in its workspace; the ordinary backward kernels run on it with the queries offset to the chunk, and only
// keys from the chunk on receive dk, dv, du.
struct ChunkBwdWs {
    size_t attn, mask, total;
};
static ChunkBwdWs chunk_bwd_ws(const sparsek_chunk_cfg& c, int clen)
{
    const ChunkLayout L = chunk_layout(c);
    const int nv = L.rcap + clen;
    sparsek_cfg v = virtual_cfg(c, nv);
    ChunkBwdWs W;
    size_t off = 0;
    W.attn = off; off += align_up(attn_bwd_ws_bytes(v), 256);
    v.gate_mode = c.gate_mode;
    W.mask = off; off += align_up(mask_bwd_ws_bytes(v), 256);
    W.total = off;
    return W;
}
size_t chunk_bwd_ws_bytes(const sparsek_chunk_cfg& c) { return chunk_bwd_ws(c, c.chunk_max).total; }

int launch_chunk_bwd(const sparsek_chunk_cfg& c, int clen, const void* q, const void* o, const void* dO,
                     const void* fwd_ws, void* dq, void* dk, void* dv, float* du, void* ws, hipStream_t st)
{
    const ChunkLayout L = chunk_layout(c);
    const ChunkWs W = chunk_ws(c, clen);
    const ChunkBwdWs Bw = chunk_bwd_ws(c, clen);
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
    // (the forward's lists are those of the same lifetimes)
    const FwdLists lists = attn_fwd_lists(virtual_cfg(c, nv), w + W.attn);
    return launch_bwd(cv, q, k_v, v_v, u_v, tau_v, death_v, o, lse, dO, dq, dk, dv, du, b + Bw.attn, b + Bw.mask, st,
                      L.rcap, first_valid, clen, std::max(0, L.rcap - c.w - 1), lists.pos ? &lists : nullptr);
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
                       (const int32_t*)(s + L.ret_sel), (const float*)nullptr, L.rcap, 0, u_v, (int32_t*)(w + W.first),
                       (unsigned long long*)(w + W.kept));
    const RowCopy copy = chunk_rows(c, L, s, nullptr, nullptr, 0, w + W.k, w + W.v);
    int rc = launch_mask(cv, u_v, tau_v, death_v, w + W.mask, st, std::max(0, L.rcap - c.w - 1), (const int32_t*)(w + W.first), &copy);
    if (rc) return rc;
    hipLaunchKernelGGL(chunk_clear_padding_kernel, dim3(rows), dim3(1024), 0, st, chunk_tail(c, L, W, s, w, 0));
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
