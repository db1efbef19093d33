// fp32 kernels of the MAGE hot path for gfx950: the MAGE_F32 element type, on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, 157 TFLOP/s on the chip -- as much as the vector ALU with
// packed arithmetic, twice what it has without).
//
//   attn_f32_kernel<D,MODE,GATHER>   attention of 16-row tiles of a KV head's query rows over a share of the keys, or
//                                    (F32_STATS) only the row statistics of selection's first pass
//   colsum_f32_kernel<D>             second pass of selection: averaged probabilities per key
//
// Both work from registers: a wavefront owns 16 query rows (attention) or 32 keys (column sums) and reads its
// operands straight from memory, without LDS and without a barrier in the loop.  What makes that possible is that a
// sum over channels (scores) may take them in any order and that the output channels may be dealt to the MFMA rows
// in any order:
//   - scores: MFMA step (j, e) multiplies channels 16*j + 4*(lane/16) + e of query and key, so a lane's operands of
//     four steps are one 16-byte load of its row;
//   - P.V: MFMA step v takes keys 4*(lane/16) + v, which is the layout the scores come out in, and channels
//     64*g + 4*(lane%16) + e, so a lane's operands of four accumulators are one 16-byte load of a value row.
// A 16-key tile costs 64 MFMAs of 32 cycles per wavefront at d = 128 and 16 KB of loads, which the vector L1 (wavefronts
// of one workgroup share the keys) and the L2 serve at a fraction of their rate: the loop is bound by the matrix cores.
// Measured at 16 query heads in 4 groups, d = 128, B = 16, L = 8192: exact attention and selection 440 us with the
// vector-ALU kernels that stood here (keys through LDS in 4-byte reads, 2.4 TFLOP/s), 50 us with these; the smallest call
// (4 x 4 query rows, 64 + 4 keys, d = 64) 16.0 us in two launches, 5.7 us in one.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ids.hpp"
#include "plan.hpp"
#include "row_stats.hpp"

namespace mage {

enum { F32_ATTN = 0, F32_STATS = 1 };

typedef float f32v4_t __attribute__((ext_vector_type(4)));

constexpr int kF32Waves = 8;                // attention: wavefronts per workgroup = row tiles x key slices
constexpr int kF32Keys = 16;                // keys per tile of a wavefront

// 16 bytes of row `lane % 16` per 16 channels: the score operand (either side) of a lane
template <int D>
__device__ __forceinline__ void f32_load_row(const float *row, f32v4_t (&x)[D / 16])
{
    const float *src = row + 4 * ((tid_x() & 63) >> 4);
#pragma unroll
    for (int j = 0; j < D / 16; ++j) x[j] = *reinterpret_cast<const f32v4_t *>(src + 16 * j);
}

// scores of 16 x 16 items: c[v] belongs to item 4*(lane/16) + v of `a` and item lane%16 of `b`
template <int D>
__device__ __forceinline__ f32v4_t f32_scores(const f32v4_t (&a)[D / 16], const f32v4_t (&b)[D / 16])
{
    f32v4_t c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
            c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j][e], b[j][e], c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j][e + 1], b[j][e + 1], c1, 0, 0, 0);
        }
    return c0 + c1;
}

// address of query row `row` of KV head h's row space (row = g_local * B + q)
template <int D>
__device__ __forceinline__ const float *f32_q_row(const KernelArgs &a, int h, int row)
{
    const int gl = row / a.B, qi = row - gl * a.B;
    return static_cast<const float *>(a.q) + ((long long)qi * a.Hq + (long long)h * a.G + gl) * D;
}

// Workgroup: a.rw row tiles x kF32Waves / a.rw key slices.  The 16-key tiles (cache tiles first, then the in-block
// tiles) are dealt round-robin to the key slices of all splits.  Key slices are merged through LDS, splits by
// combine_kernel / lse_kernel.
template <int D, int MODE, bool GATHER>
__global__ __launch_bounds__(kF32Waves * 64) __attribute__((amdgpu_waves_per_eu(2))) void attn_f32_kernel(const KernelArgs a)
{
    constexpr bool WITH_V = (MODE == F32_ATTN);
    constexpr int NJ = D / 16, NG = D / 64;
    constexpr float kLazy = 8.f, kFloor = -3.0e38f;      // lazily raised softmax reference, as in the bf16 kernels
    __shared__ f32v4_t part[WITH_V ? kF32Waves * NG * 4 * 64 : 1];      // [wave][accumulator][lane]
    __shared__ float stat[kF32Waves][4][16];                            // m, l, and the same over the cache keys only

    const int h = wg_x(), split = wg_y(), rg = wg_z();
    const int lane = tid_x() & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid_x() >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int kw = kF32Waves / a.rw;                     // key slices of the workgroup
    const int rt = wave & (a.rw - 1), slice = wave / a.rw;
    const int row = (rg * a.rw + rt) * 16 + l16;

    const int nc = (int)a.nc;
    const int cache_tiles = (nc + kF32Keys - 1) / kF32Keys;
    const int ntiles = cache_tiles + (a.n_blk + kF32Keys - 1) / kF32Keys;
    const int step = a.n_split * kw;
    const int32_t *idx = GATHER ? a.idx + (long long)h * a.nc : nullptr;
    const float *kc = static_cast<const float *>(a.kc) + (long long)h * D, *vc = static_cast<const float *>(a.vc) + (long long)h * D;
    const float *kb = static_cast<const float *>(a.kblk) + (long long)h * D, *vb = static_cast<const float *>(a.vblk) + (long long)h * D;
    const unsigned stride = (unsigned)a.Hkv * D;

    // row of the cache (or of the block, for tiles past the cache) that holds this lane's key l16 of tile t
    auto entry = [&](int t) -> int {
        const bool cache = t < cache_tiles;
        int p = (cache ? t : t - cache_tiles) * kF32Keys + l16;
        const int last = (cache ? nc : a.n_blk) - 1;
        p = p < last ? p : last;                          // positions past the end repeat the last row (masked below)
        return GATHER && cache ? idx[p] : p;
    };
    auto load_k = [&](int t, int e, f32v4_t (&k)[NJ]) {
        f32_load_row<D>((t < cache_tiles ? kc : kb) + (unsigned long long)(unsigned)e * stride, k);
    };
    auto load_v = [&](int t, int e, f32v4_t (&v)[4][NG]) {
        const float *base = (t < cache_tiles ? vc : vb) + 4 * l16;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float *src = base + (unsigned long long)(unsigned)__shfl(e, 4 * lg + i) * stride;
#pragma unroll
            for (int g = 0; g < NG; ++g) v[i][g] = *reinterpret_cast<const f32v4_t *>(src + 64 * g);
        }
    };

    f32v4_t o[WITH_V ? NG * 4 : 1];
#pragma unroll
    for (int i = 0; i < (WITH_V ? NG * 4 : 1); ++i) o[i] = f32v4_t{0.f, 0.f, 0.f, 0.f};
    float m_run = kFloor, l_run = 0.f, m_pre = kFloor, l_pre = 0.f;

    const int t0 = split * kw + slice;
    int e_cur = 0, e_nxt = 0;
    f32v4_t q[NJ], ka[NJ], kn[NJ];
    if (t0 < ntiles) e_cur = entry(t0);
    if (t0 + step < ntiles) e_nxt = entry(t0 + step);
    f32_load_row<D>(f32_q_row<D>(a, h, row < a.R ? row : a.R - 1), q);        // rows past R stand in for the last and are never stored
    if (t0 < ntiles) load_k(t0, e_cur, ka);

    // one tile; the keys of the next one are requested behind this tile's values
    auto tile = [&](int t, const f32v4_t (&k)[NJ], f32v4_t (&k_next)[NJ]) {
        f32v4_t v[4][NG];
        if (WITH_V) load_v(t, e_cur, v);
        if (t + step < ntiles) load_k(t + step, e_nxt, k_next);
        e_cur = e_nxt;
        if (t + 2 * step < ntiles) e_nxt = entry(t + 2 * step);
        if (t >= cache_tiles && t - step < cache_tiles) {            // first in-block tile: freeze the prefix statistics
            m_pre = m_run;
            l_pre = l_run;
        }
        f32v4_t s = f32_scores<D>(k, q);                             // s[i]: key 4*lg + i, query row l16
        const int valid = t < cache_tiles ? nc - t * kF32Keys : a.n_blk - (t - cache_tiles) * kF32Keys;
        if (valid < kF32Keys) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * lg + i >= valid) s[i] = -INFINITY;
        }
        float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * a.scale_log2;
        if (__any(mx > m_run + kLazy)) {
            const float m_new = fmaxf(m_run, ceilf(mx));        // whole numbers: the fp64 split merge of near-ties scales by exact powers of two
            const float corr = exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= corr;
            if (WITH_V) {
#pragma unroll
                for (int i = 0; i < NG * 4; ++i) o[i] *= corr;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[i] = exp2f(fmaf(s[i], a.scale_log2, -m_run));
            l_run += s[i];
        }
        if (WITH_V) {
            // o[4*g + e][v]: channel 64*g + 4*(4*lg + v) + e of query row l16
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int g = 0; g < NG; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[4 * g + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][g][e], s[i], o[4 * g + e], 0, 0, 0);
        }
    };
    for (int t = t0; t < ntiles; t += 2 * step) {
        tile(t, ka, kn);
        if (t + step < ntiles) tile(t + step, kn, ka);
    }

    // merge of the key slices
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    l_pre += __shfl_xor(l_pre, 16);
    l_pre += __shfl_xor(l_pre, 32);
    {   // last tile of this slice; no in-block tile among its tiles: everything seen was prefix
        const int t_last = t0 < ntiles ? t0 + (ntiles - 1 - t0) / step * step : -1;
        if (t_last < cache_tiles) {
            m_pre = m_run;
            l_pre = l_run;
        }
    }
    if (lg == 0) {
        stat[wave][0][l16] = m_run;
        stat[wave][1][l16] = l_run;
        stat[wave][2][l16] = m_pre;
        stat[wave][3][l16] = l_pre;
    }
    if (WITH_V) {
#pragma unroll
        for (int i = 0; i < NG * 4; ++i) part[(wave * NG * 4 + i) * 64 + lane] = o[i];
    }
    __syncthreads();
    float M = kFloor, Mp = kFloor;
    for (int s = 0; s < kw; ++s) {
        M = fmaxf(M, stat[s * a.rw + rt][0][l16]);
        Mp = fmaxf(Mp, stat[s * a.rw + rt][2][l16]);
    }
    float lt = 0.f, lp = 0.f;
    for (int s = 0; s < kw; ++s) {
        const int w = s * a.rw + rt;
        lt = fmaf(exp2f(stat[w][0][l16] - M), stat[w][1][l16], lt);
        lp = fmaf(exp2f(stat[w][2][l16] - Mp), stat[w][3][l16], lp);
    }
    if (row >= a.R) return;
    const long long pi = ((long long)h * a.n_split + split) * a.rpad + row;
    const bool scalars = slice == 0 && lg == 0;
    if (WITH_V && a.stat_m != nullptr && scalars) {
        a.stat_m[pi] = Mp;
        a.stat_l[pi] = lp;
    }
    const bool direct = WITH_V && a.n_split == 1;
    if (!direct && scalars) {
        a.part_m[pi] = M;
        a.part_l[pi] = lt;
    }
    if (!WITH_V) return;
    const float inv = direct ? 1.f / lt : 1.f;
    float *dst;
    if (direct) {
        const int gl = row / a.B, qi = row - gl * a.B;
        const long long orow = (long long)qi * a.Hq + (long long)h * a.G + gl;
        dst = a.out + orow * D;
        if (a.lse_out && scalars) a.lse_out[orow] = (M + log2f(lt)) * 0.6931471805599453f;
    } else {
        dst = a.part_o + pi * D;
    }
    // 16-byte pieces (g, v) of the row: channels 64*g + 16*lg + 4*v .. +3; the key slices take turns
    for (int c = slice; c < NG * 4; c += kw) {
        const int g = c >> 2, v = c & 3;
        f32v4_t acc = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < kw; ++s) {
            const int w = s * a.rw + rt;
            const float wgt = exp2f(stat[w][0][l16] - M);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[e] = fmaf(wgt, reinterpret_cast<const float *>(&part[(w * NG * 4 + 4 * g + e) * 64 + lane])[v], acc[e]);
        }
        *reinterpret_cast<f32v4_t *>(dst + 64 * g + 16 * lg + 4 * v) = acc * inv;
    }
}

// Second pass of selection (Eq. 5): alpha[h,j] = 1/(G*B) * sum_rows exp2(score2 - lse2[row]).  A wavefront holds 32 keys
// in registers and walks the query rows 16 at a time (they are the same few KB for everyone: L1 / L2 hits), so a
// sum over rows never leaves the wavefront.  Also leaves the maxima over 16 consecutive keys for the top-k filter.
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void colsum_f32_kernel(const KernelArgs a)
{
    constexpr int NJ = D / 16;
    // one grid column per KV head (all G*B rows, Eq. 5), or with head_rows = B per QUERY head (its B rows, Eq. 2)
    const int hy = wg_x(), split = wg_y();
    const bool per_head = a.head_rows > 0;
    const int h = per_head ? hy / a.G : hy;
    const int row_lo = per_head ? (hy % a.G) * a.B : 0;
    const int row_end = per_head ? row_lo + a.head_rows : a.R;
    const int lane = tid_x() & 63, wave = __builtin_amdgcn_readfirstlane(tid_x() >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const float *kc = static_cast<const float *>(a.kc) + (long long)h * D;
    const unsigned stride = (unsigned)a.Hkv * D;
    __shared__ float lse_lds[kMergeRows];
    __shared__ __attribute__((aligned(8))) unsigned char scratch[256 * 12];
    const float *lse2 = a.lse2 + (long long)h * a.rpad;            // by row of the KV head
    if (a.lse2 == nullptr) {
        RowStats<256> stats;
        stats.issue(a, h, row_lo, row_end - row_lo);
        stats.finish(a, lds_addr(lse_lds), lds_addr(scratch));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
    }
    const long long n_groups = (a.L + kGroupKeys - 1) / kGroupKeys;
    const int units = (int)((a.L + 31) / 32);

    for (int u = split * 4 + wave; u < units; u += a.n_split * 4) {
        f32v4_t k[2][NJ];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const long long j = (long long)u * 32 + 16 * b + l16;
            f32_load_row<D>(kc + (unsigned long long)(unsigned)(j < a.L ? j : a.L - 1) * stride, k[b]);
        }
        f32v4_t q[NJ];
        auto load_q = [&](int r0) {
            const int r = r0 + l16;
            f32_load_row<D>(f32_q_row<D>(a, h, r < row_end ? r : row_end - 1), q);
        };
        load_q(row_lo);
        float col[2] = {0.f, 0.f};
        for (int r0 = row_lo; r0 < row_end; r0 += 16) {
            float ls[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = r0 + 4 * lg + v;
                const bool in = r < row_end;                         // exp2(-inf) = 0 for rows outside the sum
                ls[v] = a.lse2 == nullptr ? (in ? lse_lds[r - row_lo] : INFINITY) : (in ? lse2[r] : INFINITY);
            }
            const f32v4_t s0 = f32_scores<D>(q, k[0]), s1 = f32_scores<D>(q, k[1]);      // query r0 + 4*lg + v, key l16
            if (r0 + 16 < row_end) load_q(r0 + 16);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                col[0] += exp2f(fmaf(s0[v], a.scale_log2, -ls[v]));
                col[1] += exp2f(fmaf(s1[v], a.scale_log2, -ls[v]));
            }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float c = col[b];
            c += __shfl_xor(c, 16);
            c += __shfl_xor(c, 32);
            c *= a.inv_rows;
            const long long j = (long long)u * 32 + 16 * b + l16;
            if (lg == 0 && j < a.L) a.alpha[(long long)hy * a.L + j] = c;
            if (a.gmax != nullptr) {
                static_assert(kGroupKeys == kF32Keys, "a group of the filter is one 16-key half of a unit");
                float g = j < a.L ? c : 0.f;
#pragma unroll
                for (int d = 1; d < 16; d <<= 1) g = fmaxf(g, __shfl_xor(g, d));
                const long long gi = (long long)u * 2 + b;
                if (lane == 0 && gi < n_groups) a.gmax[(long long)hy * n_groups + gi] = g;
            }
        }
    }
}

hipError_t f32_attn(const KernelArgs &a, int d, int row_groups, bool gather, hipStream_t stream)
{
    if (a.rw != 1 && a.rw != 2) return hipErrorInvalidValue;
    dim3 grid(a.Hkv, a.n_split, row_groups), block(kF32Waves * 64);
    if (d == 128) {
        if (gather) hipLaunchKernelGGL((attn_f32_kernel<128, F32_ATTN, true>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((attn_f32_kernel<128, F32_ATTN, false>), grid, block, 0, stream, a);
    } else if (d == 64) {
        if (gather) hipLaunchKernelGGL((attn_f32_kernel<64, F32_ATTN, true>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((attn_f32_kernel<64, F32_ATTN, false>), grid, block, 0, stream, a);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t f32_stats(const KernelArgs &a, int d, int row_groups, hipStream_t stream)
{
    if (a.rw != 1 && a.rw != 2) return hipErrorInvalidValue;
    dim3 grid(a.Hkv, a.n_split, row_groups), block(kF32Waves * 64);
    if (d == 128) hipLaunchKernelGGL((attn_f32_kernel<128, F32_STATS, false>), grid, block, 0, stream, a);
    else if (d == 64) hipLaunchKernelGGL((attn_f32_kernel<64, F32_STATS, false>), grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t f32_colsum(const KernelArgs &a, int d, hipStream_t stream)
{
    dim3 grid(a.head_rows > 0 ? a.Hq : a.Hkv, a.n_split), block(256);
    if (d == 128) hipLaunchKernelGGL((colsum_f32_kernel<128>), grid, block, 0, stream, a);
    else if (d == 64) hipLaunchKernelGGL((colsum_f32_kernel<64>), grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace mage
