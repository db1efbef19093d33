// Small kernels around the attention passes (gfx950):
//   combine_kernel   merges the split-key partials of an attention call into out / lse
//   lse_kernel       merges the statistics partials of selection into one log2-domain log-sum-exp per query row,
//                    where the column sums do not do it themselves (row_stats.hpp): more rows than one of their
//                    workgroups covers, or so many splits that every workgroup reading all of them costs more
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "combine.hpp"
#include "ids.hpp"
#include "plan.hpp"

namespace mage {

// One workgroup per (query row, KV head)
template <int D>
__global__ __launch_bounds__(256) void combine_kernel(const KernelArgs a)
{
    __shared__ CombineLds<D> lds;
    combine_row<D>(a, wg_x(), wg_y(), tid_x(), true, lds);
}

// lse2[h][row] = M + log2( sum_s l_s * 2^(m_s - M) ): one wavefront per row, lane s takes splits
// s, s+64, ...; the sum is accumulated in fp64 in a fixed order.
__global__ __launch_bounds__(256) void lse_kernel(const KernelArgs a, float *lse2_out)
{
    const int h = wg_y();
    const int row = wg_x() * 4 + (tid_x() >> 6);
    const int lane = tid_x() & 63;
    if (row >= a.R) return;
    float M = -INFINITY;
    for (int s = lane; s < a.n_split; s += 64) M = fmaxf(M, a.part_m[((long long)h * a.n_split + s) * a.rpad + row]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) M = fmaxf(M, __shfl_xor(M, d));
    double lt = 0.0;
    for (int s = lane; s < a.n_split; s += 64) {
        const long long pi = ((long long)h * a.n_split + s) * a.rpad + row;
        lt += (double)a.part_l[pi] * (double)exp2f(a.part_m[pi] - M);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) lt += __shfl_xor(lt, d);
    if (lane == 0) lse2_out[(long long)h * a.rpad + row] = M + (float)log2(lt);
}

hipError_t launch_combine(const KernelArgs &a, int d, hipStream_t stream)
{
    dim3 grid(a.R, a.Hkv), block(256);
    if (d == 128) hipLaunchKernelGGL((combine_kernel<128>), grid, block, 0, stream, a);
    else if (d == 64) hipLaunchKernelGGL((combine_kernel<64>), grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_lse(const KernelArgs &a, float *lse2_out, hipStream_t stream)
{
    dim3 grid((a.R + 3) / 4, a.Hkv), block(256);
    hipLaunchKernelGGL(lse_kernel, grid, block, 0, stream, a, lse2_out);
    return hipGetLastError();
}

}  // namespace mage
