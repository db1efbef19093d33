// Merge of the split-key partials of one query row of an attention call into out / lse: 256 consecutive threads = D/4
// channel quads x SG split groups.  Split s contributes weight exp2(m_s - M); group g walks splits g, g+SG, ... with all
// its loads in flight, then the groups are added in a fixed order through LDS.
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
    float l[SG];
    float m[4];
};

// `t`: this thread's number within the row's 256 threads; `live`: the row exists (all threads of a workgroup call: barriers)
template <int D>
__device__ __forceinline__ void combine_row(const KernelArgs &a, int row, int h, int t, bool live, CombineLds<D> &lds)
{
    constexpr int TPR = CombineLds<D>::TPR, SG = CombineLds<D>::SG;
    const int c4 = t % TPR, sg = t / TPR;
    const long long base = (long long)h * a.n_split * a.rpad + row;

    float M = -INFINITY;
    if (live)
        for (int s = t; s < a.n_split; s += 256) M = fmaxf(M, a.part_m[base + (long long)s * a.rpad]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) M = fmaxf(M, __shfl_xor(M, d));
    if ((t & 63) == 0) lds.m[t >> 6] = M;
    __syncthreads();
    M = fmaxf(fmaxf(lds.m[0], lds.m[1]), fmaxf(lds.m[2], lds.m[3]));

    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float lt = 0.f;
    if (live) {
#pragma unroll 4
        for (int s = sg; s < a.n_split; s += SG) {
            const long long pi = base + (long long)s * a.rpad;
            const float w = exp2f(a.part_m[pi] - M);
            lt = fmaf(w, a.part_l[pi], lt);
            const float4 v = *reinterpret_cast<const float4 *>(a.part_o + pi * D + c4 * 4);
            acc.x = fmaf(w, v.x, acc.x);
            acc.y = fmaf(w, v.y, acc.y);
            acc.z = fmaf(w, v.z, acc.z);
            acc.w = fmaf(w, v.w, acc.w);
        }
    }
    lds.o[sg][c4] = acc;
    if (c4 == 0) lds.l[sg] = lt;
    __syncthreads();
    if (sg != 0 || !live) return;
    acc = lds.o[0][c4];
    lt = lds.l[0];
#pragma unroll
    for (int g = 1; g < SG; ++g) {
        const float4 v = lds.o[g][c4];
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
        lt += lds.l[g];
    }
    const float inv = 1.f / lt;
    const int gl = row / a.B, qi = row - gl * a.B;
    const long long orow = (long long)qi * a.Hq + (long long)h * a.G + gl;
    *reinterpret_cast<float4 *>(a.out + orow * D + c4 * 4) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
    if (a.lse_out && c4 == 0) a.lse_out[orow] = (M + log2f(lt)) * 0.6931471805599453f;
}

}  // namespace mage
