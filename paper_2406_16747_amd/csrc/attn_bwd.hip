// Attention backward: gradients of L = sum(dO * O) with respect to q, k, v, the gates held fixed
// (the gradient with respect to the scores is mask_bwd.hip's).  From the selected-attention
// equations of Sec. 3.2 with the gating variants: with s_ij = scale gk_ij (q_i.k_j), p = softmax,
// o_i = sum_j p_ij gv_ij v_j and D_i = dO_i.o_i,
//     dV_j = sum_i p_ij gv_ij dO_i        dp_ij = gv_ij (dO_i.v_j)      ds_ij = p_ij (dp_ij - D_i)
//     dQ_i = sum_j ds_ij scale gk_ij k_j  dK_j  = sum_i ds_ij scale gk_ij q_i
// gk = gate in mode 0, else 1; gv = gate in modes 0 and 1, else 1; window keys carry gate 1.
// p_ij is recomputed from q, k and the forward's lse; nothing of size n x (k + w) is stored.
#include "common.hpp"
#include "attn_tiles.hpp"
#include "bwd_merge.hpp"
#include "mask_ranges.hpp"
#include <cmath>

namespace spk {

void launch_block_lists(const sparsek_cfg& c, const int32_t* death, int32_t* lists, int32_t* counts,
                        hipStream_t st);
size_t block_lists_bytes(const sparsek_cfg& c, size_t* counts_offset);

struct AbwdWs {
    size_t lists, counts, xpos, xdeath, xu, delta, lse2, elist, ecount, eslot, dk32, dv32, sk32, sv32, total;
};
static AbwdWs abwd_ws(const sparsek_cfg& c)
{
    AbwdWs W;
    size_t coff = 0;
    const size_t lb = block_lists_bytes(c, &coff);
    const size_t BH = (size_t)c.B * c.H;
    W.lists = 0;
    W.counts = coff;
    size_t off = align_up(lb, 256);
    W.xpos = off; off += ext_array_bytes(c);
    W.xdeath = off; off += ext_array_bytes(c);
    W.xu = off; off += ext_array_bytes(c);
    W.delta = off; off += align_up(BH * c.n * 4, 256);
    W.lse2 = off; off += align_up(BH * c.n * 4, 256);
    W.elist = off; off += align_up((size_t)c.B * c.Gu * c.n * 4, 256);
    W.ecount = off; off += align_up((size_t)c.B * c.Gu * 4, 256);
    W.eslot = off; off += align_up((size_t)c.B * c.Gu * c.n * 4, 256);
    W.dk32 = off; off += align_up(BH * c.n * c.d * 4, 256);
    W.dv32 = off; off += align_up(BH * c.n * c.d * 4, 256);
    W.sk32 = off; off += align_up(BH * c.n * c.d * 4, 256);
    W.sv32 = off; off += align_up(BH * c.n * c.d * 4, 256);
    W.total = off;
    return W;
}
size_t attn_bwd_ws_bytes(const sparsek_cfg& c) { return abwd_ws(c).total; }

template <typename T>
__device__ __forceinline__ float ldg(const T* p);
template <>
__device__ __forceinline__ float ldg<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ldg<uint16_t>(const uint16_t* p) { return bf16_to_f32(*p); }
template <typename T>
__device__ __forceinline__ void stg(T* p, float v);
template <>
__device__ __forceinline__ void stg<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void stg<uint16_t>(uint16_t* p, float v) { *p = f32_to_bf16(v); }

__global__ void abwd_zero_kernel(uint4* p, size_t n16)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

// delta[bh][i] = dO_i . o_i: one wave per row.
template <typename T>
__global__ __launch_bounds__(256) void abwd_delta_kernel(const T* __restrict__ o, const T* __restrict__ dO, size_t rows,
                                                         int d, float* __restrict__ delta)
{
    const size_t r = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= rows) return;
    float s = 0.0f;
    for (int c = lane; c < d; c += 64) s += ldg(o + r * d + c) * ldg(dO + r * d + c);
    s = wave_sum_f32(s);
    if (lane == 0) delta[r] = s;
}

// fp32 accumulators -> storage type
template <typename T>
__global__ void abwd_convert_kernel(const float* __restrict__ a, const float* __restrict__ b, T* __restrict__ oa,
                                    T* __restrict__ ob, size_t nelem)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nelem; i += (size_t)gridDim.x * blockDim.x) {
        stg(oa + i, a[i]);
        stg(ob + i, b[i]);
    }
}

// ---------------------------------------------------------------------------------
// Generic vector-ALU kernel (fp32 or bf16 storage, any d <= 128 that is a multiple of 4): one wave
// per query, lanes over keys for the dot products, over columns for the row updates.  dQ stays
// with the wave; dK and dV rows are accumulated in fp32 with one atomic per column.
// ---------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ kk, const T* __restrict__ v, const float* __restrict__ u,
    const float* __restrict__ tau, const int32_t* __restrict__ death, const int32_t* __restrict__ lists,
    const int32_t* __restrict__ counts, const float* __restrict__ lse, const T* __restrict__ dO,
    const float* __restrict__ delta, T* __restrict__ dq, float* __restrict__ dk32, float* __restrict__ dv32, int H,
    int Gu, int n, int d, int k, int w, int gate_mode, float scale, int nb)
{
    __shared__ float qs[4][128], ds[4][128];
    const int blk = blockIdx.x, bh = blockIdx.y;
    const int b = bh / H, h = bh % H;
    const int row = b * Gu + (Gu == 1 ? 0 : h);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i0 = blk * QB;
    const size_t hb = (size_t)bh * n * d;
    const float* ur = u + (size_t)row * n;
    const float* tr = tau + (size_t)row * n;
    const int32_t* dr = death + (size_t)row * n;
    const int32_t* list = lists + ((size_t)row * nb + blk) * (size_t)(k > 0 ? k : 1);
    const int cnt = counts[(size_t)row * nb + blk];
    const int c0 = max(0, i0 - w + 1);
    const bool gate_k = gate_mode == 0, gate_v = gate_mode == 0 || gate_mode == 1;

    for (int qi = wv; qi < QB; qi += 4) {
        const int i = i0 + qi;
        if (i >= n) break;
        for (int c = lane; c < d; c += 64) {
            qs[wv][c] = ldg(q + hb + (size_t)i * d + c);
            ds[wv][c] = ldg(dO + hb + (size_t)i * d + c);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        const int Tp = i - w;
        const float tauT = (Tp >= 0) ? tr[Tp] : 0.0f;
        const float lse_i = lse[(size_t)bh * n + i];
        const float Di = delta[(size_t)bh * n + i];
        float dq0 = 0.0f, dq1 = 0.0f;  // columns lane and lane + 64 of dQ_i
        const int n_list = (Tp >= 0) ? cnt : 0;
        const int total = n_list + (i - c0 + 1);
        for (int e0 = 0; e0 < total; e0 += 64) {
            const int e = e0 + lane;
            int j = -1;
            if (e < total) j = (e < n_list) ? list[e] : c0 + (e - n_list);
            bool valid = false;
            float gate = 1.0f;
            if (j >= 0) {
                if (i - j < w) valid = true;
                else if (dr[j] > Tp) { valid = true; gate = clip01(ur[j] - tauT); }
            }
            float pv = 0.0f, coef = 0.0f;
            if (valid) {
                float qk = 0.0f, dov = 0.0f;
                const T* kj = kk + hb + (size_t)j * d;
                const T* vj = v + hb + (size_t)j * d;
                for (int c = 0; c < d; c++) {
                    qk += qs[wv][c] * ldg(kj + c);
                    dov += ds[wv][c] * ldg(vj + c);
                }
                const float gk = gate_k ? gate : 1.0f, gv = gate_v ? gate : 1.0f;
                const float p = __expf(scale * gk * qk - lse_i);
                pv = p * gv;
                coef = p * (gv * dov - Di) * scale * gk;
            }
            unsigned long long ball = __ballot(valid);
            while (ball) {
                const int src = __builtin_ctzll(ball);
                ball &= ball - 1;
                const float ps = __shfl(pv, src, 64), cs = __shfl(coef, src, 64);
                const int js = __shfl(j, src, 64);
                const size_t ro = hb + (size_t)js * d;
                if (lane < d) {
                    dq0 += cs * ldg(kk + ro + lane);
                    unsafeAtomicAdd(dv32 + ro + lane, ps * ds[wv][lane]);
                    unsafeAtomicAdd(dk32 + ro + lane, cs * qs[wv][lane]);
                }
                if (lane + 64 < d) {
                    dq1 += cs * ldg(kk + ro + lane + 64);
                    unsafeAtomicAdd(dv32 + ro + lane + 64, ps * ds[wv][lane + 64]);
                    unsafeAtomicAdd(dk32 + ro + lane + 64, cs * qs[wv][lane + 64]);
                }
            }
        }
        if (dq) {  // null: dQ comes from the MFMA kernel
            if (lane < d) stg(dq + hb + (size_t)i * d + lane, dq0);
            if (lane + 64 < d) stg(dq + hb + (size_t)i * d + lane + 64, dq1);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
}

// ---------------------------------------------------------------------------------
// MFMA kernel for dQ (bf16, D = 64 or 128).  Same blocking and the same walk over a query block's key set as the
// forward (attn_fwd.hip): 128 queries x 4 waves, 64-key tiles (the block's top-k list, then the contiguous keys up
// to the block's last query) in runs of one kind per wave, so that only the tiles that need a test or a gate pay
// for it; metadata staged in segments, tiles gathered straight into LDS one tile ahead.  Per 32-key half:
// S^T = K.Q^T and DV^T = V.dO^T (row reads of the K and V tiles), the elementwise step to ds_ij gk_ij in bf16, then
// dQ^T += K^T.dS^T with K^T through transposing reads of the same K tile (see RowTile).  The softmax scale is
// applied once, to the finished dQ.
// ---------------------------------------------------------------------------------
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
// two floats rounded to bf16 (nearest even), the first in the low half
__device__ __forceinline__ unsigned pack_bf16x2(float a, float b)
{
    f32x2v f = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2v));
}

// A tile of 64 rows (Q or dO) in LDS serves 16-byte row reads (A operand of the contractions over the head dimension) and
// transposing 8-byte reads (A operand of the contractions over the queries).  Every row lands once, in groups of 1 KB (a
// wave-load) padded by 16 bytes; which rows share a group is chosen so that both kinds of reads touch every bank once per
// pass: 16 consecutive rows differ in (group, slot) modulo the 16 chunks of 256 bytes, and 4 consecutive ones by multiples
// of 4 chunks.  Unlike a permutation of the chunks inside a row this leaves every operand of a tile at a constant distance
// from one address per lane (two in all, one for each kind of read), so tiles can sit in a ring without code of their own.
template <int D>
struct RowTile {
    static constexpr int RB = D * 2, RPL = 1024 / RB, NL = KT / RPL;   // bytes per row, rows per group, groups
    static constexpr int GS = 1024 + 16, BYTES = NL * GS;
    // tile row r sits in group g(r), slot s(r)
    __device__ static constexpr int group(int r) { return D == 128 ? 4 * (r & 3) + ((r >> 2) & 3) : 4 * (r & 1) + ((r >> 2) & 3); }
    __device__ static constexpr int slot(int r) { return D == 128 ? r >> 4 : ((r >> 1) & 1) + 2 * (r >> 4); }
    __device__ static constexpr int row(int g, int s)   // the inverse
    {
        return D == 128 ? (g >> 2) + 4 * (g & 3) + 16 * s : (g >> 2) + 2 * (s & 1) + 4 * (g & 3) + 16 * (s >> 1);
    }
    __device__ static constexpr int offset(int r) { return group(r) * GS + slot(r) * RB; }
    static constexpr int R16 = 16 / (D == 128 ? 16 : 8) * RB;   // 16 rows on: the same group, so many bytes on
    static constexpr int R8 = 2 * GS;                           // 8 rows on, from a row of 0 .. 7 modulo 16
};

// Two tiles: the one in use and the one on its way.
template <int D>
struct DqSmem : TileMeta {
    struct Tile {
        unsigned char k[RowTile<D>::BYTES];
        unsigned char v[RowTile<D>::BYTES];
    } t[2];
};
static_assert(sizeof(DqSmem<128>) <= 80 * 1024, "two workgroups per CU");

typedef const unsigned char __attribute__((address_space(3)))* lds_bytes_t;
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(lds_void_t*)p; }
// The operands of a RowTile: a row read (16 bytes of one row), and a transposing read (8 + 8 bytes, rows 8 apart).
__device__ __forceinline__ bf16x8 row_operand(uint32_t at)
{
    return *(const bf16x8 __attribute__((address_space(3)))*)(lds_bytes_t)(uintptr_t)at;
}
template <int D>
__device__ __forceinline__ bf16x8 transposed_operand(uint32_t at)
{
    const i16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3)))*)(uintptr_t)at);
    const i16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3)))*)(uintptr_t)(at + RowTile<D>::R8));
    const bf16x4 lo = __builtin_bit_cast(bf16x4, lo4), hi = __builtin_bit_cast(bf16x4, hi4);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// Where in a tile a lane's operands start: row reads of rows 0 .. 31, chunk lane / 32 (+ 2 per step); transposing reads of rows
// 4 (lane / 32) + r16 / 4 (+ 8, + 16 per step), 8 bytes at column 16 grp2 + 4 (r16 % 4) (+ 32 per step).
template <int D>
__device__ __forceinline__ uint32_t row_lane(int lane) { return RowTile<D>::offset(lane & 31) + 16 * (lane >> 5); }
template <int D>
__device__ __forceinline__ uint32_t transposed_lane(int lane)
{
    const int half = lane >> 5, r16 = lane & 15, grp2 = (lane >> 4) & 1;
    return RowTile<D>::offset(4 * half + (r16 >> 2)) + (16 * grp2 + 4 * (r16 & 3)) * 2;
}

// What a lane of the dQ kernel keeps for the whole block.
struct DqLane {
    float tau_q, lse2, Di; // threshold of the query's prefix, lse * log2(e), dO.o
    int qi;
};

// The gather of one tile: K and V rows at the positions jp[0..63].  The wave's loads are groups whose rows are neighbours, so
// that a lane's row numbers come with one read.
template <int D>
__device__ __forceinline__ void dq_issue(typename DqSmem<D>::Tile& t, const int32_t* jp, const unsigned char* kh,
                                         const unsigned char* vh, int wv, int lane)
{
    using S = RowTile<D>;
    constexpr int NX = S::NL / 4, LPR = S::RB / 16;
    static_assert(S::row(4, 0) == 1 && (NX == 2 || S::row(8, 0) == 2), "the rows of groups wv, wv + 4, .. are neighbours");
    const int32_t* src = jp + S::row(wv, 0) + S::row(0, lane / LPR);
    int j[NX];
    if constexpr (NX == 4) {
        const int4 x = *(const int4*)src;
        j[0] = x.x; j[1] = x.y; j[2] = x.z; j[3] = x.w;
    } else {
        const int2 x = *(const int2*)src;
        j[0] = x.x; j[1] = x.y;
    }
#pragma unroll
    for (int x = 0; x < NX; x++) {
        const int L = wv + 4 * x;
        const uint32_t off = (uint32_t)j[x] * (uint32_t)S::RB + 16u * (uint32_t)(lane % LPR);
        async_load_lds16(kh, off, &t.k[L * S::GS]);
        async_load_lds16(vh, off, &t.v[L * S::GS]);
    }
}

// One 64-key tile for one wave.  jbase: position of the tile's first key if the key set were contiguous.
template <int D, int MODE, int KIND>
__device__ __forceinline__ void dq_tile_body(uint32_t rk, uint32_t tk, const int32_t* jdeath, const float* ju, int jbase,
                                             const DqLane& ln, int lane, int w, float c2,
                                             const bf16x8 (&qreg)[D / 16], const bf16x8 (&dreg)[D / 16],
                                             f32x16 (&acc_q)[D / 32])
{
    using TT = TileTraits<MODE, KIND>;
    using S = RowTile<D>;
    constexpr int DS = D / 16, DB = D / 32;
    const int half = lane >> 5;
    const int qw = ln.qi - (w - 1);
    const int dqh = ln.qi - jbase - 4 * half;  // contiguous tiles: key number cst + 4*half sits dqh - cst behind the query
    const int dqw = dqh - w;                   // in the window  <=>  cst > dqw
#pragma unroll
    for (int mb = 0; mb < 2; mb++) {
        const f32x16 zero = {0};
        f32x16 acc_s = zero, acc_d = zero;
        __builtin_amdgcn_sched_barrier(0);  // one half at a time: there are no registers for two in flight
#pragma unroll
        for (int s = 0; s < DS; s++) {
            const bf16x8 ka = row_operand(rk + 2 * mb * S::R16 + 32 * s);
            const bf16x8 va = row_operand(rk + S::BYTES + 2 * mb * S::R16 + 32 * s);
            acc_s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[s], s == 0 ? zero : acc_s, 0, 0, 0);
            acc_d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, dreg[s], s == 0 ? zero : acc_d, 0, 0, 0);
        }
        // ds_ij gk_ij without the softmax scale; a pair that is not attended gets p = 0 through the exponent
        u32x4 dsb[2];
        float hold = 0.0f;
#pragma unroll
        for (int g4 = 0; g4 < 4; g4++) {
            const int kb = 32 * mb + 8 * g4 + 4 * half;
            float4 U4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            int4 L4 = make_int4(0, 0, 0, 0);
            if (TT::GATED) U4 = *(const float4*)&ju[kb];
            if (TT::MASKL) L4 = *(const int4*)&jdeath[kb];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int r = 4 * g4 + e;
                const int cst = 32 * mb + 8 * g4 + e;  // key number in the tile minus the lane's 4 * half (folded into dqh, dqw)
                const int Lj = e == 0 ? L4.x : e == 1 ? L4.y : e == 2 ? L4.z : L4.w;
                const float uj = e == 0 ? U4.x : e == 1 ? U4.y : e == 2 ? U4.z : U4.w;
                const float qk = acc_s[r], dov = acc_d[r];
                float gate = 1.0f;
                if (TT::GATED) {
                    gate = clip01(uj - ln.tau_q);
                    if (TT::SELECT) gate = (cst > dqw) ? 1.0f : gate;
                }
                float arg = TT::KGATE ? fmaf(qk, gate * c2, -ln.lse2) : fmaf(qk, c2, -ln.lse2);
                // key j is attended by query i while j <= i and i - (w - 1) <= death[j]
                if (TT::MASKL && TT::MASKC) arg = (cst <= dqh && qw <= Lj) ? arg : -INFINITY;
                else if (TT::MASKL) arg = (qw <= Lj) ? arg : -INFINITY;
                else if (TT::MASKC) arg = (cst <= dqh) ? arg : -INFINITY;
                const float p = __builtin_amdgcn_exp2f(arg);
                float ds = p * (TT::GATED ? fmaf(gate, dov, -ln.Di) : dov - ln.Di);
                if (TT::KGATE) ds *= gate;
                if ((r & 1) == 0) hold = ds;
                else dsb[r >> 3][(r & 7) >> 1] = pack_bf16x2(hold, ds);
            }
        }
#pragma unroll
        for (int i = 0; i < 2 * DB; i++)
            acc_q[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(transposed_operand<D>(tk + (2 * mb + i / DB) * S::R16 + 64 * (i % DB)),
                                                                    __builtin_bit_cast(bf16x8, dsb[i / DB]),
                                                                    acc_q[i % DB], 0, 0, 0);
    }
}

// The tiles [T, T_end) of the block's key set, all of one kind; the metadata of tile T sits in segment T / TPS.
template <int D, int MODE, int KIND>
__device__ __forceinline__ void dq_run_tiles(DqSmem<D>& sm, const StageSrc& src, int& T, int T_end, int jbase0,
                                             const unsigned char* kh, const unsigned char* vh, int wv, int lane,
                                             const DqLane& ln, int w, float c2, const bf16x8 (&qreg)[D / 16],
                                             const bf16x8 (&dreg)[D / 16], f32x16 (&acc_q)[D / 32])
{
    const uint32_t rl = lds_address(&sm.t[0].k[0]) + row_lane<D>(lane), tl = lds_address(&sm.t[0].k[0]) + transposed_lane<D>(lane);
    for (; T < T_end; T++) {
        const int sg = T / TPS, lt = T - sg * TPS;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();  // tile T has landed; everybody is done with tile T-1 (and, at the first tile of a segment, with the segment before)
        if (lt == 0 && (sg + 1) * TPS < src.nt) stage_meta(sm, src, sg + 1, wv, lane);
        if (T + 1 < src.nt) {
            const int sn = (T + 1) / TPS;
            dq_issue<D>(sm.t[(T + 1) & 1], sm.jpos[sn & 1] + (T + 1 - sn * TPS) * KT, kh, vh, wv, lane);
        }
        if (KIND != TILE_SKIP) {
            const uint32_t tb = (uint32_t)(T & 1) * (uint32_t)sizeof(typename DqSmem<D>::Tile);
            dq_tile_body<D, MODE, KIND>(rl + tb, tl + tb, sm.jdeath[sg & 1] + lt * KT, sm.ju[sg & 1] + lt * KT, jbase0 + T * KT, ln,
                                        lane, w, c2, qreg, dreg, acc_q);
        }
    }
}

// elist: the ever-selected keys of a score row (death_j > j), ordered by death_j / bw and then by position,
// so that the 32 keys of a wave and the 128 of a block stop being attended at about the same query and the
// span of query tiles they walk is short.  eslot[j]: where key j sits in that list, -1 if it is not in it.
// A counting sort whose result does not depend on timing: every wave owns a contiguous range of positions
// and its own cursor per bucket.  One workgroup per row, at the head of the dQ kernel's grid: dK/dV, which needs the
// list, is the next launch, and a launch of its own (28 us at n = 8192) would only be waited for.
constexpr int EBK = 512;
constexpr int EW = 4;   // waves
struct ElistSmem {
    int cur[EW][EBK];
    int start[EBK];
};
__device__ void abwd_elist(ElistSmem& sm, int row, const int32_t* __restrict__ death, int n, int j_min,
                           int32_t* __restrict__ elist, int32_t* __restrict__ ecount, int32_t* __restrict__ eslot)
{
    auto& cur = sm.cur;
    auto& start = sm.start;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t* dr = death + (size_t)row * n;
    int32_t* el = elist + (size_t)row * n;
    int32_t* es = eslot + (size_t)row * n;
    const int bw = max(256, (n + EBK) / EBK);  // death <= n, so death / bw < EBK
    for (int i = tid; i < EW * EBK; i += 64 * EW) (&cur[0][0])[i] = 0;
    __syncthreads();
    const int per = ((n + EW - 1) / EW + 63) / 64 * 64;
    const int j_begin = min(n, wv * per), j_end = min(n, j_begin + per);
    for (int j0 = j_begin; j0 < j_end; j0 += 256) {   // four loads in flight
        int dj[4];
#pragma unroll
        for (int x = 0; x < 4; x++) dj[x] = j0 + 64 * x + lane < j_end ? dr[j0 + 64 * x + lane] : 0;
#pragma unroll
        for (int x = 0; x < 4; x++) {
            const int j = j0 + 64 * x + lane;
            if (j < j_end && dj[x] > j && j >= j_min) atomicAdd(&cur[wv][dj[x] / bw], 1);
        }
    }
    __syncthreads();
    for (int i = tid; i < EBK; i += 64 * EW) {  // per bucket: each wave's offset inside the bucket, and the bucket's size
        int acc = 0;
#pragma unroll
        for (int x = 0; x < EW; x++) {
            const int c = cur[x][i];
            cur[x][i] = acc;
            acc += c;
        }
        start[i] = acc;
    }
    __syncthreads();
    if (wv == 0) {  // exclusive scan of the bucket sizes, 8 buckets per lane
        int v[EBK / 64], sum = 0;
#pragma unroll
        for (int i = 0; i < EBK / 64; i++) { v[i] = start[lane * (EBK / 64) + i]; sum += v[i]; }
        int incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        int ex = incl - sum;
#pragma unroll
        for (int i = 0; i < EBK / 64; i++) { start[lane * (EBK / 64) + i] = ex; ex += v[i]; }
        if (lane == 63) ecount[row] = incl;
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    int next = j_begin + lane < j_end ? dr[j_begin + lane] : 0;
    for (int j0 = j_begin; j0 < j_end; j0 += 64) {
        const int j = j0 + lane;
        const int dj = next;
        next = j + 64 < j_end ? dr[j + 64] : 0;
        const bool sel = j < j_end && dj > j && j >= j_min;  // keys before j_min receive no gradient
        const int bkt = sel ? dj / bw : -1;
        int slot = -1;
        unsigned long long rem = __ballot(sel);
        while (rem) {  // one turn per distinct bucket among this step's lanes
            const int l = __ffsll((long long)rem) - 1;
            const int bb = __shfl(bkt, l, 64);
            const unsigned long long m = __ballot(bkt == bb);
            const int base = start[bb] + cur[wv][bb];
            if (bkt == bb) slot = base + __popcll(m & below);
            if (lane == l) cur[wv][bb] += __popcll(m);
            rem &= ~m;
        }
        if (sel) el[slot] = j;
        if (j < j_end) es[j] = slot;
    }
}

// What the first workgroups of the dQ kernel do: the lists of ever-selected keys, and clearing words for whoever asks.
struct DqAux {
    int rows, zero_blocks;
    int j_min;
    int32_t *elist, *ecount, *eslot;
    uint32_t* zero;
    size_t zero_words;
};
constexpr int ZERO_PER_BLOCK = 256 * 32;   // words

__device__ __forceinline__ void dq_aux(ElistSmem& sm, const DqAux& a, int id, const int32_t* __restrict__ death, int n)
{
    if (id < a.rows) {
        abwd_elist(sm, id, death, n, a.j_min, a.elist, a.ecount, a.eslot);
        return;
    }
    const size_t w0 = (size_t)(id - a.rows) * ZERO_PER_BLOCK;
    for (size_t i = w0 + threadIdx.x; i < min(a.zero_words, w0 + ZERO_PER_BLOCK); i += 256) a.zero[i] = 0u;
}

// WGS: workgroups per compute unit, three where the registers allow it and there are blocks for them, as in the forward (48 heads of
// 2000, k = w = 128, straight-through, forward and backward: 152.7 -> 147.7 us by this kernel, 152.1 -> 147.5 by the forward's).
template <int D, int MODE, int WGS>
__global__ __launch_bounds__(256, WGS) void attn_bwd_dq_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kk, const uint16_t* __restrict__ v,
    const float* __restrict__ u, const float* __restrict__ tau, const int32_t* __restrict__ death,
    const int32_t* __restrict__ xpos, const int32_t* __restrict__ xdeath, const float* __restrict__ xu, int KP,
    const int32_t* __restrict__ counts, const float* __restrict__ lse, const uint16_t* __restrict__ o,
    const uint16_t* __restrict__ dO, float* __restrict__ delta, float* __restrict__ lse2s, uint16_t* __restrict__ dq,
    int H, int Gu, int n, int k, int w, float scale, int nb, int BH, int nrows, int q_begin,
    const int32_t* __restrict__ first_valid, int q_rows, DqAux aux)
{
    union Smem {
        __device__ Smem() {}
        DqSmem<D> t;
        ElistSmem e;
    };
    __shared__ __align__(16) Smem smem;
    DqSmem<D>& sm = smem.t;
    constexpr int DS = D / 16, DB = D / 32;
    const int n_aux = aux.rows + aux.zero_blocks;
    if ((int)blockIdx.x < n_aux) {
        dq_aux(smem.e, aux, blockIdx.x, death, n);
        return;
    }
    int bh, blk;
    deal_block(blockIdx.x - n_aux, nb, BH, bh, blk);
    const int b = bh / H, h = bh % H;
    const int row = b * Gu + (Gu == 1 ? 0 : h);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int i0 = blk * QB;
    // queries before q_begin do not exist; q, dO, lse, delta and dq then hold q_rows rows per head from query q_begin
    if (i0 + QB <= q_begin) return;
    const ptrdiff_t qo = q_rows ? (ptrdiff_t)bh * q_rows - q_begin : (ptrdiff_t)bh * n;
    const unsigned char* kh = (const unsigned char*)(kk + (size_t)bh * n * D);
    const unsigned char* vh = (const unsigned char*)(v + (size_t)bh * n * D);
    const float* tr = tau + (size_t)row * n;
    const int nstay = counts[(size_t)nrows * nb + (size_t)row * nb + blk];
    const int c0 = max(max(0, i0 - w + 1), first_valid ? first_valid[row] : 0);
    const int c_end = min(n - 1, i0 + QB - 1);
    // the list part is laid out for min(k, T0 + 1) keys, the length of a complete top-k list (see the forward)
    const int T0 = i0 - w;
    const int nkl = (T0 >= 0 && k > 0) ? (min(k, T0 + 1) + KT - 1) / KT * KT : 0;
    const int nkc = max(0, (c_end - c0 + 1 + KT - 1) / KT * KT);
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

    const int qa = i0 + 32 * wv;
    const int qb = min(qa + 31, n - 1);
    const bool wave_live = qa < n;
    DqLane ln;
    ln.qi = qa + col;
    const int qrow = min(ln.qi, n - 1);
    ln.tau_q = (ln.qi < n && ln.qi - w >= 0) ? tr[ln.qi - w] : 0.0f;
    ln.lse2 = lse[qo + qrow] * 1.4426950408889634f;
    bf16x8 qreg[DS], dreg[DS];
    {
        // D_i = dO_i . o_i is formed here, where the dO rows are loaded anyway, and left for the kernels that follow
        // together with lse * log2(e), the form their exponents subtract
        bf16x8 oreg[DS];
#pragma unroll
        for (int s = 0; s < DS; s++) {
            const size_t off = (size_t)(qo + qrow) * D + 16 * s + 8 * half;
            qreg[s] = *(const bf16x8*)(q + off);
            dreg[s] = *(const bf16x8*)(dO + off);
            oreg[s] = *(const bf16x8*)(o + off);
        }
        float dpart = 0.0f;
#pragma unroll
        for (int s = 0; s < DS; s++)
#pragma unroll
            for (int e = 0; e < 8; e++) dpart = fmaf((float)dreg[s][e], (float)oreg[s][e], dpart);
        ln.Di = dpart + __shfl_xor(dpart, 32, 64);
        if (half == 0 && ln.qi < n) {
            delta[qo + ln.qi] = ln.Di;
            lse2s[qo + ln.qi] = ln.lse2;
        }
    }
    stage_meta(sm, src, 0, wv, lane);
    const WaveRuns wr = wave_runs(wave_live, nkl, nkc, nstay, qa, qb, w, c0);
    f32x16 acc_q[DB];
#pragma unroll
    for (int x = 0; x < DB; x++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc_q[x][r] = 0.0f;
    const float c2 = scale * 1.4426950408889634f;
    // Everything the compiler tracks must have arrived before the first untracked load (see the forward).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < DS; s++) asm volatile("" ::"v"(qreg[s]), "v"(dreg[s]));
    asm volatile("" ::"v"(ln.tau_q), "v"(ln.lse2), "v"(ln.Di));
    __syncthreads();   // segment 0 of the metadata has landed
    if (NT > 0) dq_issue<D>(sm.t[0], sm.jpos[0], kh, vh, wv, lane);
    {
        const int jbase0 = c0 - nkl;
        int T = 0;
#define SPK_RUN(KIND, bound) \
    dq_run_tiles<D, MODE, KIND>(sm, src, T, min(NT, (bound)), jbase0, kh, vh, wv, lane, ln, w, c2, qreg, dreg, acc_q)
        SPK_RUN(TILE_LIST, wr.b0);
        SPK_RUN(TILE_LIST_MASK, wr.b1);
        if (wr.narrow) SPK_RUN(TILE_CONT, wr.b2);
        else SPK_RUN(TILE_EDGE, wr.b2);
        SPK_RUN(TILE_FAST, wr.b3);
        SPK_RUN(TILE_DIAG, wr.b4);
        SPK_RUN(TILE_SKIP, NT);
#undef SPK_RUN
    }
    if (ln.qi < n) {
        uint16_t* orow = dq + (size_t)(qo + ln.qi) * D;
#pragma unroll
        for (int x = 0; x < DB; x++) {
#pragma unroll
            for (int g4 = 0; g4 < 4; g4++) {
                bf16x4 pk;
#pragma unroll
                for (int e = 0; e < 4; e++) pk[e] = (__bf16)(scale * acc_q[x][4 * g4 + e]);
                *(bf16x4*)(orow + 32 * x + 8 * g4 + 4 * half) = pk;
            }
        }
    }
}

template <int D>
static void launch_dq_mfma(const sparsek_cfg& c, const void* q, const void* k, const void* v, const float* u,
                           const float* tau, const int32_t* death, const ExtLists& x, const int32_t* counts,
                           const float* lse, const void* o, const void* dO, float* delta, float* lse2, void* dq, int nb,
                           hipStream_t st, int q_begin, const int32_t* first_valid, int q_rows, const DqAux& aux)
{
    const int BH = c.B * c.H;
    dim3 grid(nb * BH + aux.rows + aux.zero_blocks);
#define SPK_LAUNCH_DQ(MODE, WGS)                                                                                   \
    hipLaunchKernelGGL((attn_bwd_dq_kernel<D, MODE, WGS>), grid, dim3(256), 0, st, (const uint16_t*)q, (const uint16_t*)k, \
                       (const uint16_t*)v, u, tau, death, (const int32_t*)x.pos, (const int32_t*)x.death,          \
                       (const float*)x.u, x.KP, counts, lse, (const uint16_t*)o, (const uint16_t*)dO, delta, lse2, \
                       (uint16_t*)dq, c.H, c.Gu, c.n, c.k, c.w, c.softmax_scale, nb, BH, c.B * c.Gu, q_begin,      \
                       first_valid, q_rows, aux)
    if (c.gate_mode == 0) SPK_LAUNCH_DQ(0, 2);
    else if (c.gate_mode == 1) SPK_LAUNCH_DQ(1, 2);
    else if (D == 64 && three_per_cu(c, q_begin, aux.rows)) SPK_LAUNCH_DQ(2, (D == 64 ? 3 : 2));
    else SPK_LAUNCH_DQ(2, 2);
#undef SPK_LAUNCH_DQ
}

// ---------------------------------------------------------------------------------
// MFMA kernel for dK and dV (bf16, D = 64 or 128): the mirror image of the forward.  A workgroup
// owns 128 keys (4 waves x 32 keys) whose K and V fragments stay in registers, and streams 64-query
// tiles of Q and dO through LDS, so S = Q.K^T and dO.V^T land with lane = key; P and dS are then
// directly the B operands of dV^T += dO^T.P and dK^T += Q^T.dS (Q^T, dO^T through transposing LDS
// reads).  Nothing is reduced across waves and no row data goes through atomics inside the loop.
// Because a key is attended on one contiguous range of queries, two kinds of key blocks cover all
// pairs with one interval test per pair:
//   window blocks    128 consecutive positions, queries j <= i <= j + w - 1, gate 1;
//   selected blocks  128 ever-selected keys (death_j > j, listed by death, see abwd_elist), queries
//                    j + w <= i <= death_j + w - 1, gate clip(u_j - tau_{i-w}).
// Every key belongs to exactly one window block and at most one selected block, so nothing needs an
// atomic: a window block stores the final dk, dv rows of the keys that are never selected, and its
// fp32 part of the others into dk32 / dv32 by position; a selected block stores into sk32 / sv32 at
// the key's slot of the list; abwd_merge adds the two parts and rounds, in the score gradient's launch or in one of its own.
// With q_rows != 0 the queries are offset (a chunk attending retained keys): q, dO, lse, delta, dk, dv
// hold q_rows rows per head from position q_begin, and only keys from q_begin on are processed.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ int wave_max_i32(int x)
{
#pragma unroll
    for (int s = 0; s < 4; s++) x = max(x, dpp_i32(x, s));
    return max(max(__builtin_amdgcn_readlane(x, 15), __builtin_amdgcn_readlane(x, 31)),
               max(__builtin_amdgcn_readlane(x, 47), __builtin_amdgcn_readlane(x, 63)));
}
__device__ __forceinline__ int wave_min_i32(int x) { return ~wave_max_i32(~x); }

__device__ __forceinline__ int b_row(int bh, int H, int Gu) { return (bh / H) * Gu + (Gu == 1 ? 0 : bh % H); }

// S and dO.V go straight to vector registers: the compiler, given accumulation registers, puts every product there, and the
// elementwise work then reads each value with an instruction of its own (64 per tile).  It does not know the latency of these
// products (8 passes: behind the builtin form it leaves 12 states).  What keeps the distance is the schedule below: between the
// last product into a sum and its first reader lie the LEAD + 1 slots of another run, each a product of 8 passes with an LDS read,
// and the 4 states of settled(); where nothing lies between (a wave's first unit) settled() waits 24 states.  Their operands come
// from LDS and from registers that are loaded once, never from a vector instruction just ahead.  The build reads the generated
// code and refuses any in which a result is touched within 12 states or an operand within 2 (check_products), so whoever changes
// LEAD or a slot's contents finds out.  64 heads of 8192 at k = w = 512: the backward -18 us of 930.
template <bool FIRST>
__device__ __forceinline__ void mfma_v(f32x16& d, const bf16x8& a, const bf16x8& b)
{
    if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}

constexpr int DKV_NBUF = 4;  // tiles in LDS: the one the products are at, the one before it, and two on their way
template <int D>
struct DkvSmem {
    struct Tile {
        unsigned char q[RowTile<D>::BYTES];   // Q rows of a tile
        unsigned char g[RowTile<D>::BYTES];   // dO rows
    } t[DKV_NBUF];
    // per query of a tile: lse * log2(e), D_i, tau_{i-w} (and a fourth row that only keeps the loads branch-free)
    float meta[DKV_NBUF][4][KT];
    int red[2][4];
};

template <int D, int MODE>
__global__ __launch_bounds__(256, 1) void attn_bwd_dkv_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kk, const uint16_t* __restrict__ v,
    const float* __restrict__ u, const float* __restrict__ tau, const int32_t* __restrict__ death,
    const int32_t* __restrict__ elist, const int32_t* __restrict__ ecount, const float* __restrict__ lse2s,
    const uint16_t* __restrict__ dO, const float* __restrict__ delta, float* __restrict__ dk32,
    float* __restrict__ dv32, float* __restrict__ sk32, float* __restrict__ sv32, const int32_t* __restrict__ eslot,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int H, int Gu, int n, int w, float scale, int nb,
    int q_begin, int q_rows, RangesArgs ranges)
{
    union Smem {
        __device__ Smem() {}
        DkvSmem<D> t;
        float ts[RS_MAX];
    };
    __shared__ __align__(16) Smem smem;
    DkvSmem<D>& sm = smem.t;
    if ((int)blockIdx.y >= 2 * nb) {   // the last rows of the grid: the ranges of the score gradient, 256 keys each
        const int id = (blockIdx.y - 2 * nb) * gridDim.x + blockIdx.x, per_row = (n + 255) / 256;
        const int rows = gridDim.x / H * Gu;
        if (id < rows * per_row) mask_bwd_ranges(ranges, smem.ts, id % per_row, id / per_row);
        return;
    }
    using S = RowTile<D>;
    constexpr int DS = D / 16, DB = D / 32, NX = S::NL / 4, LPR = S::RB / 16, RB = S::RB;
    const int bh = blockIdx.x;
    const int b = bh / H, h = bh % H;
    const int row = b * Gu + (Gu == 1 ? 0 : h);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    // The head is the fast grid index: workgroups go to the chip's 8 partitions in turn, so each partition
    // keeps whole heads (the same mix of block lengths everywhere, and a head's rows in one L2).  Blocks of
    // selected keys come first, latest deaths (longest spans) first; the short window blocks fill the tail.
    const bool selected_kind = (int)blockIdx.y < nb;
    int kblk = blockIdx.y - nb;
    if (selected_kind) {  // y = 0 is the list's last block; the workgroups beyond the list come after it and leave at once
        const int ne_blocks = (ecount[b_row(blockIdx.x, H, Gu)] + 127) / 128;
        kblk = (int)blockIdx.y < ne_blocks ? ne_blocks - 1 - (int)blockIdx.y : nb;
    }
    const float* ur = u + (size_t)row * n;
    const float* tr = tau + (size_t)row * n;
    const int32_t* dr = death + (size_t)row * n;
    const int ne = selected_kind ? ecount[row] : n;
    if (kblk * 128 >= ne) return;  // no such block of selected keys
    // Keys before q_begin receive no gradient and queries before it do not exist (q_begin is a multiple of
    // 128); q, dO, lse, delta, dk and dv then hold q_rows rows per head from position q_begin.
    if (!selected_kind && kblk * 128 + 128 <= q_begin) return;
    const ptrdiff_t qo = q_rows ? (ptrdiff_t)bh * q_rows - q_begin : (ptrdiff_t)bh * n;

    // ---- this lane's key and the queries that attend it ----
    const int kidx = kblk * 128 + 32 * wv + col;
    const bool kreal = kidx < ne;
    const int j = !kreal ? 0 : selected_kind ? elist[(size_t)row * n + kidx] : kidx;
    int lo = 1, hi = 0;  // empty for a filler lane
    float uj = 0.0f;
    if (kreal) {
        if (selected_kind) { lo = j + w; hi = min(n - 1, dr[j] + w - 1); uj = ur[j]; }
        else { lo = j; hi = min(n - 1, j + w - 1); }
    }
    const bool kvalid = lo <= hi;
    int wlo = wave_min_i32(kvalid ? lo : 0x7fffffff);
    int whi = wave_max_i32(kvalid ? hi : -1);
    // a tile inside [wfull_lo, wfull_hi] is attended in full by every key of the wave: no interval tests there
    int wfull_lo = wave_max_i32(kvalid ? lo : 0x7fffffff);
    int wfull_hi = wave_min_i32(kvalid ? hi : -1);
    // (branches on these are kept vector branches: with scalar ones the compiler copies the 128 accumulators between the
    // alternatives of every tile)
    asm volatile("" : "+v"(wlo), "+v"(whi), "+v"(wfull_lo), "+v"(wfull_hi));
    // query i attends this lane's key iff (unsigned)(i - lo_eff) <= span (never for an empty lane)
    const int lo_eff = kvalid ? lo : 0x7fffffff;
    const unsigned span = kvalid ? (unsigned)(hi - lo) : 0u;
    if (lane == 0) { sm.red[0][wv] = wlo; sm.red[1][wv] = whi; }
    bf16x8 kreg[DS], vreg[DS];
#pragma unroll
    for (int s = 0; s < DS; s++) {
        const size_t off = ((size_t)bh * n + j) * D + 16 * s + 8 * half;
        kreg[s] = *(const bf16x8*)(kk + off);
        vreg[s] = *(const bf16x8*)(v + off);
    }
    f32x16 acc_k[DB], acc_v[DB];
#pragma unroll
    for (int x = 0; x < DB; x++)
#pragma unroll
        for (int r = 0; r < 16; r++) { acc_k[x][r] = 0.0f; acc_v[x][r] = 0.0f; }
    __syncthreads();
    const int blo = min(min(sm.red[0][0], sm.red[0][1]), min(sm.red[0][2], sm.red[0][3]));
    const int bhi = max(max(sm.red[1][0], sm.red[1][1]), max(sm.red[1][2], sm.red[1][3]));
    const int ntiles = blo > bhi ? 0 : (bhi - blo) / KT + 1;  // (uniform) 0: nothing attends these keys
    const float c2 = scale * 1.4426950408889634f;
    const unsigned char* qh = (const unsigned char*)(q + qo * D);
    const unsigned char* gh = (const unsigned char*)(dO + qo * D);

    // The gather of one tile (64 consecutive queries from i_first, clamped to the last row): load L fills group L, lane l
    // delivers chunk l % LPR of the row in slot l / LPR.  One step of it is the Q and the dO rows of one group.
    const int grow = S::row(0, lane / LPR), gchunk = 16 * (lane % LPR);
    auto issue_step = [&](int buf, int i_first, int x) {
        const int L = wv + 4 * x;
        // rows past the end of the sequence repeat the last row (their pairs are masked)
        const int i = min(i_first + S::row(L, 0) + grow, n - 1);
        const uint32_t off = (uint32_t)i * (uint32_t)RB + (uint32_t)gchunk;
        async_load_lds16(qh, off, &sm.t[buf].q[L * S::GS]);
        async_load_lds16(gh, off, &sm.t[buf].g[L * S::GS]);
    };
    // the tile's per-query values: waves 0, 1, 2 load one row each (wave 3 a copy of tau into the spare row)
    const float* msrc = wv == 0 ? lse2s + qo : wv == 1 ? delta + qo : tr;
    auto issue_meta = [&](int buf, int i_first) {
        const int i = min(i_first + lane, n - 1);
        async_load_lds4(msrc, 4u * (uint32_t)(wv >= 2 ? max(i - w, 0) : i), &sm.meta[buf][wv][0]);
    };
    constexpr int NLOADS = 2 * NX + 1;   // a wave's loads per tile
    auto issue = [&](int t) {   // tile t; past the last one its rows again, so that every tile has the same number of loads behind it
        const int i_first = blo + min(t, ntiles - 1) * KT, buf = t & (DKV_NBUF - 1);
#pragma unroll
        for (int x = 0; x < NX; x++) issue_step(buf, i_first, x);
        issue_meta(buf, i_first);
    };
    // tile t has landed (this wave's share of it; only tile t + 1 may still be under way), for every wave, and everybody is
    // done with the tile before the one before it
    auto landed = [&]() {
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NLOADS) : "memory");
    };
    // The K / V fragments must have arrived before the first load that the compiler does not know: its own wait for them would
    // otherwise sit at their first use, inside the loop, and count the loads of every iteration too.
    // (The first tiles' gather is under way beside them.)
    if (ntiles > 0) {
        issue(0);
        issue(1);
    }
#pragma unroll
    for (int s = 0; s < DS; s++) asm volatile("" ::"v"(kreg[s]), "v"(vreg[s]));
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");

    // The work on 32 queries (a unit; a tile holds two) is four runs of MFMAs: S and D = dO.V, then dV += dO^T.P and
    // dK += Q^T.dS, with the elementwise work in two parts: P from S, and dS from P and D.  One wave per SIMD has nothing else
    // to hide behind, so the runs of neighbouring units are interleaved and every run has elementwise work of another under it:
    //     S(m)          dV(m-1)        D(m)          dK(m-1)        S(m+1) ...
    //     dS(m-1)       P(m)           P(m)          dS(m)          dS(m)
    // A slot is one MFMA, the LDS read of an operand DEPTH slots on and a slice of elementwise work, fenced so that the
    // scheduler keeps the interleave.  The first LEAD slots after S and D have no elementwise work (its input is still being
    // computed); the next tile's gather sits there.  A tile's barrier lies DEPTH slots ahead of its first S, inside the tile
    // before, so that nobody waits for operands behind it.  GATED: the keys carry soft gates (selected keys, gate modes 0 and
    // 1); CHECK: some (query, key) pair of the tile may lie outside the key's interval; FIRST: nothing comes before the tile.
    // The softmax scale of dS is applied once, to the finished dK.
    constexpr int DEPTH = 4, LEAD = D == 128 ? 3 : 2, ESL = 2 * DS - LEAD;
    static_assert(DS == 2 * DB && DEPTH <= DS && DS % DEPTH == 0, "run lengths");
    static_assert(3 * LEAD >= NX + 1, "slots for the gather");
    const uint32_t lds0 = lds_address(&sm.t[0].q[0]);
    constexpr uint32_t TB = sizeof(typename DkvSmem<D>::Tile);
    const uint32_t rlane = lds0 + row_lane<D>(lane), tlane = lds0 + transposed_lane<D>(lane);
    const uint32_t mlane = lds_address(&sm.meta[0][0][0]) + 16 * half;
    constexpr uint32_t MB = 4 * KT * 4;
    uint32_t rcur = rlane, tcur = tlane, tprev = tlane, mcur = mlane, mprev = mlane;
    auto values = [&](uint32_t base, int imm) -> float4 {
        const f32x4v x = *(const f32x4v __attribute__((address_space(3)))*)(uintptr_t)(base + imm);
        return make_float4(x[0], x[1], x[2], x[3]);
    };
    // operand idx of a tile: run idx / DS in the order S, dV, D, dK of the first unit, then of the second, and S of the next tile
    auto operand = [&](auto ic) -> bf16x8 {
        constexpr int idx = decltype(ic)::value, run = idx / DS, m = idx % DS, h = run / 4, kind = run % 4;
        if constexpr (run == 8) return row_operand(rcur + 32 * m);   // (rcur is the next tile's by then)
        else if constexpr (kind == 0) return row_operand(rcur + 2 * h * S::R16 + 32 * m);
        else if constexpr (kind == 2) return row_operand(rcur + S::BYTES + 2 * h * S::R16 + 32 * m);
        else return transposed_operand<D>((h == 0 ? tprev : tcur) + (kind == 1 ? S::BYTES : 0) + ((h == 0 ? 2 : 0) + m / DB) * S::R16 + 64 * (m % DB));
    };
    struct Pipe {                       // what goes from one tile to the next
        f32x16 sacc, dacc;
        float pv[16];                   // P of the unit whose dS is next
        u32x4 pb[2][2], dsb[2][2];      // P and dS of the first / second unit of a tile as B operands
        float4 L4[2], PT4[2], D4[2], DT4[2];
        bf16x8 ring[DEPTH];
        float ds_even;
    };
    // per-query values of 4 elements: one group of 4 ahead
    auto p_values = [&](Pipe& P, auto gatedc, auto hc, auto gc) {
        constexpr int h = decltype(hc)::value, g4 = decltype(gc)::value;
        P.L4[g4 & 1] = values(mcur, 4 * (32 * h + 8 * g4));
        if constexpr (decltype(gatedc)::value) P.PT4[g4 & 1] = values(mcur, 4 * (32 * h + 8 * g4 + 2 * KT));
    };
    auto ds_values = [&](Pipe& P, auto gatedc, auto hc, auto gc, uint32_t mb) {
        constexpr int h = decltype(hc)::value, g4 = decltype(gc)::value;
        P.D4[g4 & 1] = values(mb, 4 * (32 * h + 8 * g4 + KT));
        if constexpr (decltype(gatedc)::value) P.DT4[g4 & 1] = values(mb, 4 * (32 * h + 8 * g4 + 2 * KT));
    };
    auto part = [](const float4& x, int e) { return e == 0 ? x.x : e == 1 ? x.y : e == 2 ? x.z : x.w; };
    auto p_element = [&](Pipe& P, auto gatedc, auto checkc, auto hc, auto rc, int rel0) {
        constexpr bool GATED = decltype(gatedc)::value;
        constexpr int h = decltype(hc)::value, r = decltype(rc)::value, g4 = r / 4, e = r % 4;
        if constexpr (e == 0 && g4 < 3) p_values(P, gatedc, hc, std::integral_constant<int, g4 + 1>{});
        float gate = 1.0f;
        if constexpr (GATED) gate = clip01(uj - part(P.PT4[g4 & 1], e));
        float arg = fmaf(P.sacc[r], GATED && MODE == 0 ? gate * c2 : c2, -part(P.L4[g4 & 1], e));
        if constexpr (decltype(checkc)::value) {
            const bool valid = (unsigned)(rel0 + (32 * h + 8 * g4 + e)) <= span;
            arg = valid ? arg : -INFINITY;  // p = 0, and with it dS
        }
        const float p = __builtin_amdgcn_exp2f(arg);
        P.pv[r] = GATED && MODE == 1 ? p : GATED ? p * gate : p;
        if constexpr (r & 1) {
            if constexpr (GATED && MODE == 1) {
                const float g0 = clip01(uj - part(P.PT4[g4 & 1], e - 1));
                P.pb[h][r >> 3][(r & 7) >> 1] = pack_bf16x2(P.pv[r - 1] * g0, P.pv[r] * gate);
            } else P.pb[h][r >> 3][(r & 7) >> 1] = pack_bf16x2(P.pv[r - 1], P.pv[r]);
        }
    };
    auto ds_element = [&](Pipe& P, auto gatedc, auto hc, auto rc, uint32_t mb) {
        constexpr bool GATED = decltype(gatedc)::value;
        constexpr int h = decltype(hc)::value, r = decltype(rc)::value, g4 = r / 4, e = r % 4;
        if constexpr (e == 0 && g4 < 3) ds_values(P, gatedc, hc, std::integral_constant<int, g4 + 1>{}, mb);
        float ds;
        if constexpr (GATED) ds = P.pv[r] * fmaf(clip01(uj - part(P.DT4[g4 & 1], e)), P.dacc[r], -part(P.D4[g4 & 1], e));
        else ds = P.pv[r] * (P.dacc[r] - part(P.D4[g4 & 1], e));
        if constexpr (r & 1) P.dsb[h][r >> 3][(r & 7) >> 1] = pack_bf16x2(P.ds_even, ds);
        else P.ds_even = ds;
    };
    // elements [16 e / ESL, 16 (e + 1) / ESL) in the e-th of the ESL slots of an elementwise part
    auto p_slice = [&](Pipe& P, auto gatedc, auto checkc, auto hc, auto ec, int rel0) {
        constexpr int e = decltype(ec)::value;
        static_for<16 * e / ESL, 16 * (e + 1) / ESL>([&](auto rc) { p_element(P, gatedc, checkc, hc, rc, rel0); });
    };
    auto ds_slice = [&](Pipe& P, auto gatedc, auto hc, auto ec, uint32_t mb) {   // mb: the values of the unit's tile
        constexpr int e = decltype(ec)::value;
        static_for<16 * e / ESL, 16 * (e + 1) / ESL>([&](auto rc) { ds_element(P, gatedc, hc, rc, mb); });
    };
    // the products of a run are far enough behind: LEAD + 1 slots, and 4 states more (24 where nothing lies between; see mfma_v)
    auto settled = [](f32x16& x, auto alone) {
        if constexpr (decltype(alone)::value) asm volatile("s_nop 15\n\ts_nop 7" : "+v"(x));
        else asm volatile("s_nop 3" : "+v"(x));
    };
#define SPK_I(x) std::integral_constant<int, (x)>{}
    // tile t; slot(idx) issues the product, refills the P.ring and does whatever lies under it
    auto tile = [&](Pipe& P, auto gatedc, auto checkc, auto firstc, int t) {
        constexpr bool FIRST = decltype(firstc)::value;
        const int rel0 = blo + t * KT + 4 * half - lo_eff;
        const int ni = blo + min(t + 2, ntiles - 1) * KT, nbuf = (t + 2) & (DKV_NBUF - 1);
        if constexpr (FIRST) static_for<0, DEPTH>([&](auto ic) { P.ring[decltype(ic)::value] = operand(ic); });
        static_for<0, 8 * DS>([&](auto ic) {
            constexpr int idx = decltype(ic)::value, run = idx / DS, m = idx % DS, h = run / 4, kind = run % 4;
            constexpr bool product = !(FIRST && h == 0 && (kind & 1));
            const bf16x8 cur = P.ring[idx % DEPTH];
            if constexpr (product) {
                if constexpr (kind == 0) mfma_v<m == 0>(P.sacc, cur, kreg[m]);
                else if constexpr (kind == 2) mfma_v<m == 0>(P.dacc, cur, vreg[m]);
                else if constexpr (kind == 1) acc_v[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, __builtin_bit_cast(bf16x8, P.pb[h ^ 1][m / DB]), acc_v[m % DB], 0, 0, 0);
                else acc_k[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, __builtin_bit_cast(bf16x8, P.dsb[h ^ 1][m / DB]), acc_k[m % DB], 0, 0, 0);
            }
            if constexpr (idx == 8 * DS - DEPTH) {   // the next tile's barrier; from here on its rows are read
                landed();
                rcur = rlane + (uint32_t)((t + 1) & (DKV_NBUF - 1)) * TB;
            }
            constexpr int nx = idx + DEPTH, nrun = nx / DS;
            if constexpr (!(FIRST && nrun < 4 && (nrun & 1))) P.ring[idx % DEPTH] = operand(SPK_I(nx));
            // the gather: a step per slot without elementwise work, in the runs dV, dK of the first unit and dV of the second
            if constexpr ((kind & 1) && m < LEAD) {
                constexpr int g = (run / 2) * LEAD + m;
                if constexpr (g < NX) issue_step(nbuf, ni, g);
                if constexpr (g == NX) issue_meta(nbuf, ni);
            }
            // elementwise work
            if constexpr (kind == 0 && m == DS - 2) p_values(P, gatedc, SPK_I(h), SPK_I(0));
            if constexpr (kind == 2 && m == DS - 2) ds_values(P, gatedc, SPK_I(h), SPK_I(0), mcur);
            if constexpr (kind == 1 && m == LEAD) settled(P.sacc, SPK_I(FIRST && h == 0));
            if constexpr (kind == 3 && m == LEAD) settled(P.dacc, SPK_I(FIRST && h == 0));
            if constexpr (kind == 1 && m >= LEAD) p_slice(P, gatedc, checkc, SPK_I(h), SPK_I(m - LEAD), rel0);
            if constexpr (kind == 2) p_slice(P, gatedc, checkc, SPK_I(h), SPK_I(m + DS - LEAD), rel0);
            if constexpr (kind == 3 && m >= LEAD) ds_slice(P, gatedc, SPK_I(h), SPK_I(m - LEAD), mcur);
            if constexpr (kind == 0 && !(FIRST && h == 0)) ds_slice(P, gatedc, SPK_I(h ^ 1), SPK_I(m + DS - LEAD), h == 0 ? mprev : mcur);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // what is left of the last tile: the rest of its second unit's dS, and its dV and dK
    auto finish = [&](Pipe& P, auto gatedc) {
        static_for<DS, 2 * DS>([&](auto ic) { if constexpr (decltype(ic)::value < DS + DEPTH) P.ring[decltype(ic)::value % DEPTH] = operand(ic); });
        static_for<0, DS>([&](auto mc) { ds_slice(P, gatedc, SPK_I(1), SPK_I(decltype(mc)::value + DS - LEAD), mprev); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, 2 * DS>([&](auto ic) {
            constexpr int idx = decltype(ic)::value, m = idx % DS;
            const bf16x8 cur = P.ring[(DS + idx) % DEPTH];
            if constexpr (idx < DS) acc_v[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, __builtin_bit_cast(bf16x8, P.pb[1][m / DB]), acc_v[m % DB], 0, 0, 0);
            else acc_k[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, __builtin_bit_cast(bf16x8, P.dsb[1][m / DB]), acc_k[m % DB], 0, 0, 0);
            constexpr int nx = idx + DEPTH;   // operands of dV (run 1), then of dK (run 3)
            if constexpr (nx < 2 * DS) P.ring[(DS + idx) % DEPTH] = operand(SPK_I(nx < DS ? DS + nx : 2 * DS + nx));
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto tiles = [&](auto gatedc) {
        Pipe P;
        bool prev = false;
        for (int t = 0; t <= ntiles; t++) {
            // the dK / dV accumulators stay in the accumulation registers: only MFMAs touch them until the end
#pragma unroll
            for (int x = 0; x < DB; x++) asm volatile("" : "+a"(acc_k[x]), "+a"(acc_v[x]));
            const int i_first = blo + t * KT;
            const uint32_t cb = (uint32_t)(t & (DKV_NBUF - 1));
            rcur = rlane + cb * TB;
            tprev = tcur;
            mprev = mcur;
            tcur = tlane + cb * TB;
            mcur = mlane + cb * MB;
            // some key of this wave is attended from this tile
            const bool live = t < ntiles && i_first <= whi && i_first + KT - 1 >= wlo;
            if (live) {
                const bool full = i_first >= wfull_lo && i_first + KT - 1 <= wfull_hi;
                if (!prev) tile(P, gatedc, std::true_type{}, std::true_type{}, t);
                else if (full) tile(P, gatedc, std::false_type{}, std::false_type{}, t);
                else tile(P, gatedc, std::true_type{}, std::false_type{}, t);
            } else {
                if (prev) finish(P, gatedc);
                if (t < ntiles) {
                    issue(t + 2);
                    landed();
                }
            }
            prev = live;
        }
    };
    if (selected_kind && MODE != 2) tiles(std::true_type{});
    else tiles(std::false_type{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (loads past the last tile land in LDS that is still this workgroup's)
#undef SPK_I
    // A key that is never selected gets all of its gradient here: round and store it.  The other keys' two parts
    // (window block, selected block) go to fp32 buffers and are added by abwd_merge.
    // A lane holds one key's row: stored from there, every instruction touches 32 rows, 32 bytes of each (64 such instructions a
    // wave took longer than a tile).  The rows go through LDS, a wave's 32 at a time, and are stored whole.  16 heads in chunks of
    // 4096, k = w = 512: 1455 -> 1418 us for the document's forward and backward; 48 heads of 2000, k = w = 128: 164 -> 162.7.
    constexpr int RS = D + 4;   // floats per row in LDS (16 lanes' 16-byte accesses to neighbouring rows fall on distinct banks)
    static_assert(4 * 32 * RS * sizeof(float) <= sizeof(sm.t), "the waves' rows take the tiles' place");
    __syncthreads();   // every wave's loads have landed, and nobody reads tiles any more
    const int k0 = kblk * 128 + 32 * wv;
    const unsigned final_rows = (unsigned)__ballot(kreal && !selected_kind && eslot[(size_t)row * n + j] < 0);
    float* area = (float*)&sm.t[0] + wv * 32 * RS;
    auto store = [&](const f32x16 (&acc)[DB], float factor, float* part, uint16_t* whole) {
#pragma unroll
        for (int x = 0; x < DB; x++)
#pragma unroll
            for (int g4 = 0; g4 < 4; g4++)
                *(float4*)(area + col * RS + 32 * x + 8 * g4 + 4 * half) =
                    make_float4(factor * acc[x][4 * g4], factor * acc[x][4 * g4 + 1], factor * acc[x][4 * g4 + 2], factor * acc[x][4 * g4 + 3]);
        constexpr int LPK = D / 4;   // lanes per row
        const int c = lane % LPK * 4;
#pragma unroll
        for (int r0 = 0; r0 < 32; r0 += 64 / LPK) {
            const int r = r0 + lane / LPK;
            const float4 f = *(const float4*)(area + r * RS + c);
            if (k0 + r >= ne) continue;
            if (final_rows >> r & 1) *(uint2*)(whole + (ptrdiff_t)r * D + c) = make_uint2(pack_bf16x2(f.x, f.y), pack_bf16x2(f.z, f.w));
            else *(float4*)(part + (ptrdiff_t)r * D + c) = f;
        }
    };
    const size_t po = ((size_t)bh * n + k0) * D;
    const ptrdiff_t wo = (qo + k0) * D;   // (used for window blocks only)
    store(acc_k, scale, (selected_kind ? sk32 : dk32) + po, dk + wo);
    store(acc_v, 1.0f, (selected_kind ? sv32 : dv32) + po, dv + wo);
}

__global__ __launch_bounds__(256) void abwd_merge_kernel(MergeArgs m) { abwd_merge(m, blockIdx.y, blockIdx.x); }

// Workgroups per head for the merge among the score gradient's blocks.  Each holds a place of a block for some 5 us and 12 or fewer turns
// of two units per thread: one for every four blocks, more where that many turns do not suffice for the keys that k makes selected
// (random scores), and where blocks with a gradient leave half of the chip's 512 places free as many as fill them.  Training,
// d = 128, us at a quarter of the blocks / now: 8 heads of 1000, k = 800, w = 900 149 / 118; 128 of 600, k = w = 100 229 / 216;
// 50 of 700, k = 200, w = 100 168 / 144; 32 of 2048, k = w = 1024 333 / 317.  Always 512 in all: 48 of 2000, k = w = 128, d = 64,
// straight-through 149 / 155, 12 of 8192, k = 1024, w = 64 570 / 590.
static int merge_parts(const sparsek_cfg& c, int nb, int q_begin)
{
    const double BH = (double)c.B * c.H, rows = c.n - q_begin;
    const double busy = BH * (q_begin ? nb - q_begin / QB : std::max(0, nb - (c.k + c.w) / QB));   // blocks with a gradient
    const double selected = c.k >= rows ? rows : std::min(rows, c.k * (1.0 + std::log(rows / c.k)));
    const double units = selected * c.d / 4, parts = std::max(nb / 4, (int)std::ceil(units / 6144));
    return (int)std::max(1.0, std::min(busy < 256 ? std::max(parts, (512 - busy) / BH) : parts, std::ceil(units / 512)));
}

template <int D>
static void launch_dkv_mfma(const sparsek_cfg& c, const void* q, const void* k, const void* v, const float* u,
                            const float* tau, const int32_t* death, const int32_t* elist, const int32_t* ecount,
                            const float* lse, const void* dO, const float* delta, float* dk32, float* dv32,
                            float* sk32, float* sv32, const int32_t* eslot, void* dk, void* dv, int nb, hipStream_t st,
                            int q_begin, int q_rows, const RangesArgs& ranges)
{
    // per head: (up to) nb blocks of selected keys, then the nb window blocks
    const int BH = c.B * c.H;
    const int extra = ranges.diff ? (c.B * c.Gu * ((c.n + 255) / 256) + BH - 1) / BH : 0;
    dim3 grid(BH, 2 * nb + extra);
#define SPK_LAUNCH_KV(MODE)                                                                                         \
    hipLaunchKernelGGL((attn_bwd_dkv_kernel<D, MODE>), grid, dim3(256), 0, st, (const uint16_t*)q, (const uint16_t*)k, \
                       (const uint16_t*)v, u, tau, death, elist, ecount, lse, (const uint16_t*)dO, delta, dk32, dv32,  \
                       sk32, sv32, eslot, (uint16_t*)dk, (uint16_t*)dv, c.H, c.Gu, c.n, c.w, c.softmax_scale, nb, q_begin, \
                       q_rows, ranges)
    if (c.gate_mode == 0) SPK_LAUNCH_KV(0);
    else if (c.gate_mode == 1) SPK_LAUNCH_KV(1);
    else SPK_LAUNCH_KV(2);
#undef SPK_LAUNCH_KV
}

int launch_attn_bwd(const sparsek_cfg& c, const void* q, const void* k, const void* v, const float* u,
                    const float* tau, const int32_t* death, const void* o, const float* lse, const void* dO, void* dq,
                    void* dk, void* dv, void* ws, hipStream_t st, int q_begin, const int32_t* first_valid, int q_rows,
                    const MaskBwdPrep* prep, BwdShared* shared, const FwdLists* have, MergeArgs* merge)
{
    const AbwdWs W = abwd_ws(c);
    char* base = (char*)ws;
    const int nb = (c.n + QB - 1) / QB;
    const size_t BH = (size_t)c.B * c.H, rows = BH * (q_rows ? q_rows : c.n), nelem = rows * c.d;
    int32_t* lists = (int32_t*)(base + W.lists);
    int32_t* counts = (int32_t*)(base + W.counts);
    float* delta = (float*)(base + W.delta);
    float* lse2 = (float*)(base + W.lse2);
    float* dk32 = (float*)(base + W.dk32);
    float* dv32 = (float*)(base + W.dv32);
    // (the dK/dV kernel puts 2 * nb key blocks on the grid's y axis)
    const bool mfma = c.dtype == SPARSEK_BF16 && (c.d == 64 || c.d == 128) && (uint64_t)c.n * c.d * 2 <= 0xFFFFFFFFull &&
                      2 * nb <= 65535;
    if (!mfma && (q_begin != 0 || first_valid || q_rows != 0)) return SPARSEK_ERR_UNSUPPORTED;
    if (q_begin % 128 != 0) return SPARSEK_ERR_INVALID_ARG;
    if (!mfma)  // the generic kernel accumulates dk, dv with atomics
        hipLaunchKernelGGL(abwd_zero_kernel, dim3(2048), dim3(256), 0, st, (uint4*)(base + W.dk32), (W.sk32 - W.dk32) / 16);
    ExtLists x{nullptr, nullptr, nullptr, 0};
    if (mfma) {
        x.pos = (int32_t*)(base + W.xpos);
        x.death = (int32_t*)(base + W.xdeath);
        x.u = (float*)(base + W.xu);
        x.KP = (int)ext_stride(c);
    }
    if (mfma && have) {
        lists = const_cast<int32_t*>(have->lists);
        counts = const_cast<int32_t*>(have->counts);
        x = ExtLists{const_cast<int32_t*>(have->pos), const_cast<int32_t*>(have->death), const_cast<float*>(have->u), x.KP};
    } else
        launch_block_lists_ext(c, death, lists, counts, u, x, st);
    dim3 grid(nb, c.B * c.H);
    if (c.dtype == SPARSEK_F32) {
        hipLaunchKernelGGL(abwd_delta_kernel<float>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, (const float*)o,
                           (const float*)dO, rows, c.d, delta);
        hipLaunchKernelGGL(attn_bwd_generic_kernel<float>, grid, dim3(256), 0, st, (const float*)q, (const float*)k,
                           (const float*)v, u, tau, death, lists, counts, lse, (const float*)dO, delta, (float*)dq, dk32,
                           dv32, c.H, c.Gu, c.n, c.d, c.k, c.w, c.gate_mode, c.softmax_scale, nb);
        hipLaunchKernelGGL(abwd_convert_kernel<float>, dim3(2048), dim3(256), 0, st, dk32, dv32, (float*)dk, (float*)dv,
                           nelem);
    } else {
        if (!mfma)
            hipLaunchKernelGGL(abwd_delta_kernel<uint16_t>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st,
                               (const uint16_t*)o, (const uint16_t*)dO, rows, c.d, delta);
        if (mfma) {
            int32_t* elist = (int32_t*)(base + W.elist);
            int32_t* ecount = (int32_t*)(base + W.ecount);
            int32_t* eslot = (int32_t*)(base + W.eslot);
            float* sk32 = (float*)(base + W.sk32);
            float* sv32 = (float*)(base + W.sv32);
            DqAux aux{c.B * c.Gu, 0, q_begin, elist, ecount, eslot, nullptr, 0};
            RangesArgs ranges{};
            // (the score gradient's ranges take at most nb + 1 more rows of the dK/dV kernel's grid)
            const bool share = shared && 3 * nb + 1 <= 65535;
            if (prep && prep->zero && share) {
                aux.zero = prep->zero;
                aux.zero_words = prep->zero_words;
                aux.zero_blocks = (int)((prep->zero_words + ZERO_PER_BLOCK - 1) / ZERO_PER_BLOCK);
                ranges = prep->ranges;
            }
            if (share) *shared = BwdShared{lists, counts, delta, nullptr};
            if (c.d == 64) {
                launch_dq_mfma<64>(c, q, k, v, u, tau, death, x, counts, lse, o, dO, delta, lse2, dq, nb, st, q_begin,
                                   first_valid, q_rows, aux);
                launch_dkv_mfma<64>(c, q, k, v, u, tau, death, elist, ecount, lse2, dO, delta, dk32, dv32, sk32, sv32, eslot,
                                    dk, dv, nb, st, q_begin, q_rows, ranges);
            } else {
                launch_dq_mfma<128>(c, q, k, v, u, tau, death, x, counts, lse, o, dO, delta, lse2, dq, nb, st, q_begin,
                                    first_valid, q_rows, aux);
                launch_dkv_mfma<128>(c, q, k, v, u, tau, death, elist, ecount, lse2, dO, delta, dk32, dv32, sk32, sv32, eslot,
                                     dk, dv, nb, st, q_begin, q_rows, ranges);
            }
            MergeArgs m{dk32, dv32, sk32, sv32, elist, ecount, c.H, c.Gu, c.n, c.d / 4, (uint16_t*)dk, (uint16_t*)dv, q_begin,
                        q_rows, 0};
            if (share && prep && prep->zero) {   // the score gradient's main kernel takes it along
                m.parts = merge_parts(c, nb, q_begin);
                *merge = m;
                shared->merge = merge;
            } else {
                m.parts = (int)std::min<size_t>(((size_t)c.n * m.d4 + 511) / 512, 512);
                hipLaunchKernelGGL(abwd_merge_kernel, dim3(m.parts, c.B * c.H), dim3(256), 0, st, m);
            }
        } else {
            hipLaunchKernelGGL(attn_bwd_generic_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t*)q,
                               (const uint16_t*)k, (const uint16_t*)v, u, tau, death, lists, counts, lse,
                               (const uint16_t*)dO, delta, (uint16_t*)dq, dk32, dv32, c.H, c.Gu, c.n, c.d, c.k, c.w,
                               c.gate_mode, c.softmax_scale, nb);
            hipLaunchKernelGGL(abwd_convert_kernel<uint16_t>, dim3(2048), dim3(256), 0, st, dk32, dv32, (uint16_t*)dk,
                               (uint16_t*)dv, nelem);
        }
    }
    return launch_status();
}

int launch_bwd(const sparsek_cfg& cfg, const void* q, const void* k, const void* v, const float* u, const float* tau,
               const int32_t* death, const void* o, const float* lse, const void* dO, void* dq, void* dk, void* dv, float* du,
               void* attn_ws, void* mask_ws, hipStream_t st, int q_begin, const int32_t* first_valid, int q_rows, int t_min,
               const FwdLists* lists)
{
    sparsek_cfg c = cfg;
    if (c.gate_mode == 3) c.gate_mode = 2;  // the straight-through forward has no gates on q, k, v
    const MaskBwdPrep prep = mask_bwd_prep(cfg, u, tau, mask_ws, t_min, first_valid);
    BwdShared shared{nullptr, nullptr, nullptr, nullptr};
    MergeArgs merge;
    const int rc = launch_attn_bwd(c, q, k, v, u, tau, death, o, lse, dO, dq, dk, dv, attn_ws, st, q_begin, first_valid, q_rows,
                                   &prep, &shared, lists, &merge);
    if (rc) return rc;
    return launch_mask_bwd(cfg, q, k, v, u, tau, death, o, lse, dO, du, mask_ws, st, q_begin, q_rows, t_min, first_valid,
                           shared.delta ? &shared : nullptr);
}

}  // namespace spk
