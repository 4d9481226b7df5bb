// The two parts of dK and dV of ever-selected keys added up: a device function, because it runs in a launch of its own or in workgroups
// among those of the score gradient's main kernel.
#pragma once
#include "common.hpp"

namespace spk {

// For every ever-selected key (list slot e, position j): dk_j = dk32_j + sk32_e rounded to bf16; same for dv.
struct MergeArgs {
    const float *dk32, *dv32, *sk32, *sv32;
    const int32_t *elist, *ecount;
    int H, Gu, n, d4;       // d4: units of 4 columns per row
    uint16_t *dk, *dv;
    int q_begin, q_rows;    // dk and dv hold q_rows rows per head from position q_begin (0: all n)
    int parts;              // workgroups per head (at least 1)
};

// Workgroup `part` of m.parts on head bh.  Bound by memory: two units of each of the four parts are under way per thread.
__device__ __forceinline__ void abwd_merge(const MergeArgs& m, int bh, int part)
{
    const ptrdiff_t qo = m.q_rows ? (ptrdiff_t)bh * m.q_rows - m.q_begin : (ptrdiff_t)bh * m.n;  // rows of dk, dv
    const int row = bh / m.H * m.Gu + (m.Gu == 1 ? 0 : bh % m.H);
    const int total = m.ecount[row] * m.d4, step = m.parts * 256;
    const int32_t* el = m.elist + (size_t)row * m.n;
    auto load = [](const float* p) { return *(const float4*)p; };
    for (int x0 = part * 256 + threadIdx.x; x0 < total; x0 += 2 * step) {
        float4 a[2], c[2], a2[2], c2[2];
        size_t dst[2];
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int x = min(x0 + i * step, total - 1), e = x / m.d4, c4 = x - e * m.d4, j = el[e];
            const size_t src = 4 * (((size_t)bh * m.n + j) * m.d4 + c4), s2 = 4 * (((size_t)bh * m.n + e) * m.d4 + c4);
            a[i] = load(m.dk32 + src);
            c[i] = load(m.dv32 + src);
            a2[i] = load(m.sk32 + s2);
            c2[i] = load(m.sv32 + s2);
            dst[i] = (size_t)(qo + j) * m.d4 + c4;
        }
#pragma unroll
        for (int i = 0; i < 2; i++) {
            if (x0 + i * step >= total) break;
            ushort4 oa, oc;
            oa.x = f32_to_bf16(a[i].x + a2[i].x); oa.y = f32_to_bf16(a[i].y + a2[i].y);
            oa.z = f32_to_bf16(a[i].z + a2[i].z); oa.w = f32_to_bf16(a[i].w + a2[i].w);
            oc.x = f32_to_bf16(c[i].x + c2[i].x); oc.y = f32_to_bf16(c[i].y + c2[i].y);
            oc.z = f32_to_bf16(c[i].z + c2[i].z); oc.w = f32_to_bf16(c[i].w + c2[i].w);
            ((ushort4*)m.dk)[dst[i]] = oa;
            ((ushort4*)m.dv)[dst[i]] = oc;
        }
    }
}

}  // namespace spk
