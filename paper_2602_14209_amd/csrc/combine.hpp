// Merge of the split-key partials of one query row of an attention call into out / lse: 256 consecutive threads = D/4
// channel quads x SG split groups.  Group g walks splits g, g+SG, ..., CH of them in flight with their statistics and
// values requested together (one round trip to memory; the maximum over all splits, which would have to come first, is
// replaced by a running one per group), then the groups are added in a fixed order through LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ids.hpp"
#include "plan.hpp"

namespace mage {

template <int D>
struct CombineLds {
    static constexpr int TPR = D / 4;                 // threads per row of channels
    static constexpr int SG = 256 / TPR;              // split groups
    float4 o[SG][TPR];
    float l[SG], m[SG];
};

// `t`: this thread's number within the row's 256 threads; `live`: the row exists (all threads of a workgroup call: barriers)
template <int D>
__device__ __forceinline__ void combine_row(const KernelArgs &a, int row, int h, int t, bool live, CombineLds<D> &lds)
{
    constexpr int TPR = CombineLds<D>::TPR, SG = CombineLds<D>::SG;
    constexpr int CH = 4;
    const int c4 = t % TPR, sg = t / TPR;
    const long long base = (long long)h * a.n_split * a.rpad + row;

    float M = -3.0e38f, lt = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live) {
        for (int s0 = sg; s0 < a.n_split; s0 += SG * CH) {
            float m[CH], l[CH];
            float4 v[CH];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int s = s0 + i * SG;
                const long long pi = base + (long long)(s < a.n_split ? s : s0) * a.rpad;
                m[i] = a.part_m[pi];
                l[i] = a.part_l[pi];
                v[i] = *reinterpret_cast<const float4 *>(a.part_o + pi * D + c4 * 4);
            }
            float top = M;
#pragma unroll
            for (int i = 0; i < CH; ++i) top = fmaxf(top, m[i]);
            const float corr = exp2f(M - top);
            M = top;
            lt *= corr;
            acc.x *= corr;
            acc.y *= corr;
            acc.z *= corr;
            acc.w *= corr;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const float w = s0 + i * SG < a.n_split ? exp2f(m[i] - M) : 0.f;
                lt = fmaf(w, l[i], lt);
                acc.x = fmaf(w, v[i].x, acc.x);
                acc.y = fmaf(w, v[i].y, acc.y);
                acc.z = fmaf(w, v[i].z, acc.z);
                acc.w = fmaf(w, v[i].w, acc.w);
            }
        }
    }
    lds.o[sg][c4] = acc;
    if (c4 == 0) {
        lds.l[sg] = lt;
        lds.m[sg] = M;
    }
    __syncthreads();
    if (sg != 0 || !live) return;
#pragma unroll
    for (int g = 1; g < SG; ++g) M = fmaxf(M, lds.m[g]);
    acc = make_float4(0.f, 0.f, 0.f, 0.f);
    lt = 0.f;
#pragma unroll
    for (int g = 0; g < SG; ++g) {
        const float4 v = lds.o[g][c4];
        const float w = exp2f(lds.m[g] - M);
        lt = fmaf(w, lds.l[g], lt);
        acc.x = fmaf(w, v.x, acc.x);
        acc.y = fmaf(w, v.y, acc.y);
        acc.z = fmaf(w, v.z, acc.z);
        acc.w = fmaf(w, v.w, acc.w);
    }
    const float inv = 1.f / lt;
    const int gl = row / a.B, qi = row - gl * a.B;
    const long long orow = (long long)qi * a.Hq + (long long)h * a.G + gl;
    *reinterpret_cast<float4 *>(a.out + orow * D + c4 * 4) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
    if (a.lse_out && c4 == 0) a.lse_out[orow] = (M + log2f(lt)) * 0.6931471805599453f;
}

}  // namespace mage
