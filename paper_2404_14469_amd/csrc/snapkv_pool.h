// Pooled, group-summed scores (Sec. 4.3; Listing 1, the pool1d call) of a run of four positions, shared by the kernels
// that store them and those that select from them on the way.
#ifndef SNAPKV_POOL_H_
#define SNAPKV_POOL_H_

#include "snapkv_internal.h"

namespace snapkv {

// acc[i] = score of position j0 + i of KV head hkv (rows of votes 16-byte aligned, j0 a multiple of four; positions at
// or past G.n get what their neighbours give and are the caller's to ignore).  interior: the run and its taps, in whole
// 16-byte pieces, lie inside the row.  Taps are combined in increasing order and query heads in head order, as
// pool_group does.
template <int P>
__device__ __forceinline__ void pooled_run(const float* __restrict__ vote, const ScoreGeom& G, const int hkv,
                                           const int64_t j0, const bool interior, const int pool_kind, float (&acc)[4]) {
    constexpr int r = P / 2;
    constexpr int RQ = (r + 3) / 4;             // float4 loads on each side of the centre one
    constexpr int NV4 = 2 * RQ + 1;
    const float pad = pool_kind == 0 ? -INFINITY : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = 0.f;
    for (int h = 0; h < G.g; ++h) {
        // (a query head whose window was scored in blocks has one vote row per block: they are added,
        // in order, before pooling)
        const float* vb = vote + ((int64_t)hkv * G.NV + (int64_t)h * G.VB) * G.vpitch;
        float v[NV4 * 4];
        if (interior) {
#pragma unroll
            for (int x = 0; x < NV4; ++x) {
                const float4 q = *reinterpret_cast<const float4*>(vb + j0 + 4 * (x - RQ));
                v[4 * x] = q.x;
                v[4 * x + 1] = q.y;
                v[4 * x + 2] = q.z;
                v[4 * x + 3] = q.w;
            }
            for (int b = 1; b < G.VB; ++b) {
#pragma unroll
                for (int x = 0; x < NV4; ++x) {
                    const float4 q = *reinterpret_cast<const float4*>(vb + (int64_t)b * G.vpitch + j0 + 4 * (x - RQ));
                    v[4 * x] += q.x;
                    v[4 * x + 1] += q.y;
                    v[4 * x + 2] += q.z;
                    v[4 * x + 3] += q.w;
                }
            }
        } else {
#pragma unroll
            for (int x = 0; x < NV4 * 4; ++x) {
                const int64_t j = j0 + x - 4 * RQ;
                v[x] = pad;
                if (j >= 0 && j < G.n) {
                    v[x] = vb[j];
                    for (int b = 1; b < G.VB; ++b) v[x] += vb[(int64_t)b * G.vpitch + j];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float val = v[4 * RQ + i - r];
#pragma unroll
            for (int d = 1; d < P; ++d)
                val = pool_kind == 0 ? fmaxf(val, v[4 * RQ + i - r + d]) : val + v[4 * RQ + i - r + d];
            if (pool_kind != 0) val = val / (float)P;
            acc[i] += val;
        }
    }
}

}  // namespace snapkv
#endif
