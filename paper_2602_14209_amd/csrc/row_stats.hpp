// Merge of the per-split softmax statistics of selection's query rows, inside the column-sum kernels.
//
// The first pass leaves (reference, sum) per key split and row; the second needs their log-sum-exp per row before it
// can weigh a score.  A kernel of its own for that (lse_kernel: 3.9 us at 52 splits, nearly all of it launch, cold code and one
// round trip) sits between the two passes; merged by every workgroup of the second pass instead, the round trip runs
// beside the workgroup's first tile requests.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ids.hpp"
#include "lds_asm.hpp"
#include "plan.hpp"

namespace mage {

// M + log2(l) rounded once: the logarithm of the mantissa alone has an absolute error of 1e-7, whatever the size of the sum
__device__ __forceinline__ float lse2_of(float M, double l)
{
    const int e = __builtin_amdgcn_frexp_exp(l);
    const float m = (float)__builtin_amdgcn_frexp_mant(l);
    return (float)((double)M + (double)e + (double)__builtin_amdgcn_logf(m));
}

// lse2 of rows [row_lo, row_lo + rows) of KV head h into the LDS floats at `dst` (byte address).  `scratch`: 12 bytes per
// thread, 8-byte aligned.  Every thread of the workgroup (THREADS of them, rows <= THREADS) calls; the caller puts a
// barrier (LDS writes completed) between this and the first read of dst, and one before scratch is used again.
// Loads and LDS accesses are arranged so that nothing waits for tile loads the caller has in flight: issue() before
// them, finish() after.
template <int THREADS>
struct RowStats {
    static constexpr int CHUNK = 16;                  // splits a thread has in flight
    float m[CHUNK], l[CHUNK];
    int rows32, parts, part, row;
    unsigned off, step, last;                         // element offsets from (head, split 0, row 0): this thread's next split, from one to the next, the last split
    const float *pm, *pl;                             // uniform
    bool live;

    // the next CHUNK of the splits part, part + parts, ...; past the last split the last one again (weighted zero in finish)
    __device__ __forceinline__ void request()
    {
#pragma unroll
        for (int i = 0; i < CHUNK; ++i) {
            const unsigned at = off < last ? off : last;
            m[i] = pm[at];
            l[i] = pl[at];
            off += step;
        }
    }

    __device__ __forceinline__ void issue(const KernelArgs &a, int h, int row_lo, int rows)
    {
        rows32 = (rows + 31) & ~31;
        parts = __builtin_amdgcn_readfirstlane(THREADS / rows32);
        part = (int)tid_x() / rows32;
        row = (int)tid_x() - part * rows32;
        live = part < parts && row < rows;
        const long long base = (long long)h * a.stat_split * a.rpad + row_lo;
        pm = a.part_m + base;
        pl = a.part_l + base;
        const unsigned r = live ? row : 0;
        off = (unsigned)part * (unsigned)a.rpad + r;
        step = (unsigned)parts * (unsigned)a.rpad;
        last = (unsigned)(a.stat_split - 1) * (unsigned)a.rpad + r;
        request();
    }

    __device__ __forceinline__ void finish(const KernelArgs &a, unsigned dst, unsigned scratch)
    {
        float M = -3.0e38f;
        double sum = 0.0;
        for (int s0 = CHUNK * parts;; s0 += CHUNK * parts) {      // one round unless there are more than CHUNK splits per part
            float top = M;
#pragma unroll
            for (int i = 0; i < CHUNK; ++i) top = fmaxf(top, m[i]);
            sum *= (double)__builtin_amdgcn_exp2f(M - top);
            M = top;
            unsigned at = off - CHUNK * step;
#pragma unroll
            for (int i = 0; i < CHUNK; ++i) {
                const float w = l[i] * __builtin_amdgcn_exp2f(m[i] - M);
                sum += (double)(at <= last ? w : 0.f);
                at += step;
            }
            if (s0 >= a.stat_split) break;
            request();
        }
        const unsigned sum_at = scratch + (unsigned)tid_x() * 8, m_at = scratch + THREADS * 8 + (unsigned)tid_x() * 4;
        asm volatile("ds_write_b64 %0, %1\n\tds_write_b32 %2, %3" ::"v"(sum_at), "v"(sum), "v"(m_at), "v"(M) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (!live || part != 0) return;
        for (int p = 1; p < parts; ++p) {
            float mp = lds_read_f32<0>(m_at + p * rows32 * 4);
            double sp;
            asm volatile("ds_read_b64 %0, %1" : "=v"(sp) : "v"(sum_at + p * rows32 * 8));
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(mp), "+v"(sp));
            const float top = fmaxf(M, mp);
            sum = sum * (double)__builtin_amdgcn_exp2f(M - top) + sp * (double)__builtin_amdgcn_exp2f(mp - top);
            M = top;
        }
        const float v = lse2_of(M, sum);
        asm volatile("ds_write_b32 %0, %1" ::"v"(dst + (unsigned)row * 4), "v"(v) : "memory");
    }
};

}  // namespace mage
