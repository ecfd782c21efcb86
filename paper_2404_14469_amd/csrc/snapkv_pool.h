// Pooled, group-summed scores (Sec. 4.3; Listing 1, the pool1d call) of a run of four positions, shared by the kernels
// that store them and those that select from them on the way.
#ifndef SNAPKV_POOL_H_
#define SNAPKV_POOL_H_

#include "snapkv_internal.h"

namespace snapkv {

// acc[i] += the pooled value of taps v[O + i .. O + i + P - 1].  Which pooling is asked once for the run: as a choice at every tap
// both were computed, and the average's divisions with them.  Maxima do not depend on their order, so the four share the
// taps they have in common (8 instructions of two or three operands for 24 at P = 7); sums take theirs in increasing order.
template <int P, int O, int N>
__device__ __forceinline__ void add_pooled(const float (&v)[N], const int pool_kind, float (&acc)[4]) {
    static_assert(O >= 0 && O + P + 3 <= N, "taps inside the run");
    if (pool_kind == 0) {
        if constexpr (P >= 4) {
            float core = v[O + 3];
#pragma unroll
            for (int d = 4; d < P; ++d) core = fmaxf(core, v[O + d]);
            const float left = fmaxf(v[O + 1], v[O + 2]), right = fmaxf(v[O + P], v[O + P + 1]);
            acc[0] += fmaxf(fmaxf(core, v[O]), left);
            acc[1] += fmaxf(fmaxf(core, left), v[O + P]);
            acc[2] += fmaxf(fmaxf(core, v[O + 2]), right);
            acc[3] += fmaxf(fmaxf(core, right), v[O + P + 2]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float val = v[O + i];
#pragma unroll
                for (int d = 1; d < P; ++d) val = fmaxf(val, v[O + i + d]);
                acc[i] += val;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float val = v[O + i];
#pragma unroll
            for (int d = 1; d < P; ++d) val = val + v[O + i + d];
            acc[i] += val / (float)P;
        }
    }
}

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
        add_pooled<P, 4 * RQ - r>(v, pool_kind, acc);
    }
}

}  // namespace snapkv
#endif
