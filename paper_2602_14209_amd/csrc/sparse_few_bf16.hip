// Batched sparse step for few sequences (gfx950): the variant of sparse_batch_bf16.hip for calls whose (sequence, KV
// head) units do not fill the chip with 128-row workgroups.
//
// There a workgroup's time is its chain of 32-key tiles (about 1 us each: barrier, fragment reads, scores, softmax, P.V), and most
// compute units have no workgroup at all.  Here the eight wavefronts of a workgroup are RW row tiles x KP = 8 / RW key
// parts: every iteration takes KP tiles, one per key part, so the chain is KP times shorter, and there are 8 / RW times as
// many workgroups.  The price is that every workgroup of a unit fetches the unit's rows (from the XCD's L2, which the row
// groups of a unit share) and that the key parts are merged through LDS at the end.  The ring takes 136 KB, one
// workgroup per CU: this kernel is for calls that leave CUs idle (sparse_few_row_tiles); the smallest calls go to
// sparse_bf16.hip, one 16-row tile per workgroup (sparse_takes_sequences).
// Measured at 28 query heads in 4 groups, B = 32, k = 300: 12 sequences 14.7 us with 128-row workgroups (96 of them), 11.7 us
// with 64-row ones (192).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sparse_batch.hpp"

namespace mage {

template <int D, int RW>
__global__ __launch_bounds__(SB_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void sparse_few_kernel(const BatchArgs a)
{
    constexpr int NW = SB_WAVES, TK = SB_TK, KP = NW / RW, NBUF = 8;
    constexpr int KS = D / 32;                           // MFMA k-steps of the score product
    constexpr int DT = D / 16;                           // 16-channel tiles of O^T
    constexpr int ROW_BYTES = D * 2, CH = D / 8;
    constexpr int MAT_BYTES = TK * ROW_BYTES;            // one 32-key K (or V) tile
    constexpr int RPI = 1024 / ROW_BYTES;                // rows covered by one wavefront-wide load
    constexpr int MAT_UNITS = MAT_BYTES / 1024;          // wavefront-wide loads per matrix
    constexpr int UPW = 2 * MAT_UNITS / NW;              // ... per wavefront and tile (K and V together)
    constexpr int BUF_BYTES = 2 * MAT_BYTES;             // K tile, then V tile
    constexpr int BLK = 16 * ROW_BYTES;
    constexpr int PART_BYTES = NW * DT * 64 * 16;
    static_assert(NBUF % KP == 0 && NBUF * UPW < 64, "whole iterations in the ring; outstanding loads fit the counter");
    static_assert(PART_BYTES + 2 * NW * 16 * 4 <= NBUF * BUF_BYTES, "the merge fits in the ring");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NBUF * BUF_BYTES];
    __shared__ int32_t idx_lds[SB_IDX_TILES * TK];

    // Workgroup id -> (unit, row group), as in sparse_batch_kernel: the row groups of a unit share an XCD
    const int blk = wg_z() * SB_GRID_Y + wg_y(), within = wg_x();
    const int unit = blk * 8 + (within & 7), rg = within >> 3;
    if (unit >= a.n_units) return;                       // uniform
    const int zi = a.Hkv == 1 ? unit : (int)(((unsigned long long)(unsigned)unit * a.inv_Hkv) >> 32);
    const int h = unit - zi * a.Hkv;
    const long long z = zi;
    const int lane = tid_x() & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid_x() >> 6);
    const int rw = wave % RW, kp = wave / RW;            // row tile and key part of this wavefront
    const int l16 = lane & 15, lg4 = lane >> 4;
    const int row0 = (rg * RW + rw) * 16, row = row0 + l16;
    const bool wave_active = row0 < a.R;

    const int nk = a.nk, n_keys = nk + a.n_blk;
    const int ntiles = __builtin_amdgcn_readfirstlane((n_keys + TK - 1) / TK);
    const unsigned stride_bytes = (unsigned)(a.Hkv * D) * 2u;
    const u16 *kc = static_cast<const u16 *>(a.kc) + z * a.seq_kv + (long long)h * D;
    const u16 *vc = static_cast<const u16 *>(a.vc) + z * a.seq_kv + (long long)h * D;
    const u16 *kb = static_cast<const u16 *>(a.kblk) + z * a.seq_blk + (long long)h * D;
    const u16 *vb = static_cast<const u16 *>(a.vblk) + z * a.seq_blk + (long long)h * D;
    const int32_t *idx = a.idx + z * a.seq_idx + (long long)h * nk;

    // index entries of key positions [t0*TK, (t0 + SB_IDX_TILES)*TK) -> LDS
    int idx_t0 = 0;
    constexpr int PER = SB_IDX_TILES * TK / (NW * 64);
    auto load_idx = [&](int t0) {
        int e[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int p = t0 * TK + i * NW * 64 + (int)tid_x();
            e[i] = p < nk ? idx[p] : 0;
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) idx_lds[i * NW * 64 + tid_x()] = e[i];
        idx_t0 = t0;
    };
    const unsigned idx_addr = lds_addr(idx_lds);
    // this wavefront's share of a tile: units n*NW + wave of the K matrix, then the V matrix (1 KB = RPI rows each)
    const unsigned char *unit_src[UPW], *unit_blk[UPW];  // cache / block base + swizzled source chunk
    int unit_row[UPW];
#pragma unroll
    for (int n = 0; n < UPW; ++n) {
        const int u = n * NW + wave;
        const bool is_v = u >= MAT_UNITS;                // uniform
        unit_row[n] = (u % MAT_UNITS) * RPI + lane / CH;
        const unsigned chunk = (unsigned)(((lane % CH) ^ (sb_swz(unit_row[n]) & (CH - 1))) * 16);
        unit_src[n] = reinterpret_cast<const unsigned char *>(is_v ? vc : kc) + chunk;
        unit_blk[n] = reinterpret_cast<const unsigned char *>(is_v ? vb : kb) + chunk;
    }
    const unsigned lds_wave = __builtin_amdgcn_readfirstlane(lds_addr(smem) + wave * 1024);
    // request the rows of `count` tiles from t on (those that exist); their entries are read from LDS together
    auto issue = [&](int t, auto COUNT) {
        constexpr int count = decltype(COUNT)::value;
        float ent[count][UPW];
        static_for<count>([&](auto JI) {
            constexpr int j = decltype(JI)::value;
            static_for<UPW>([&](auto NI) {
                constexpr int n = decltype(NI)::value;
                int p = (t + j) * TK + unit_row[n];
                p = (p < nk ? p : nk - 1) - idx_t0 * TK;     // in-block positions read some entry and ignore it
                p = p < 0 ? 0 : (p < SB_IDX_TILES * TK ? p : SB_IDX_TILES * TK - 1);
                ent[j][n] = lds_read_f32<0>(idx_addr + (unsigned)p * 4);
            });
        });
        static_for<count>([&](auto JI) {
            constexpr int j = decltype(JI)::value;
            static_for<UPW>([&](auto NI) { lds_wait<(count - 1 - j) * UPW + UPW - 1 - decltype(NI)::value>(ent[j][decltype(NI)::value]); });
            if (t + j < ntiles) {                        // uniform
                const unsigned dst = lds_wave + (unsigned)((t + j) % NBUF) * BUF_BYTES;
                static_for<UPW>([&](auto NI) {
                    constexpr int n = decltype(NI)::value;
                    int p = (t + j) * TK + unit_row[n];
                    p = p < n_keys ? p : n_keys - 1;     // positions past the last key repeat it (masked below)
                    const bool cache = p < nk;
                    const unsigned src_row = cache ? (unsigned)__builtin_bit_cast(int, ent[j][n]) : (unsigned)(p - nk);
                    const unsigned char *src = (cache ? unit_src[n] : unit_blk[n]) + (unsigned long long)src_row * stride_bytes;
                    __builtin_amdgcn_global_load_lds(MAGE_GLOBAL_PTR(src), MAGE_LDS_ADDR(dst + n * NW * 1024), 16, 0, 0);
                });
            }
        });
    };

    load_idx(0);
    // query fragment (B operand): row l16 of this wavefront's 16 rows, channels 32*ks + 8*lg4 .. +7
    bf16x8_t qf[KS];
    {
        const int rq = row < a.R ? row : a.R - 1;         // rows past R re-read the last row and are never stored
        const int gl = a.B == 1 ? rq : (int)(((unsigned long long)(unsigned)rq * a.inv_B) >> 32), qi = rq - gl * a.B;
        const u16 *src = static_cast<const u16 *>(a.q) + z * a.seq_q + ((long long)qi * a.Hq + (long long)h * a.G + gl) * D + 8 * lg4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(src + ks * 32));
    }
    __syncthreads();
    constexpr int STEP = KP < 4 ? KP : 4;                // tiles whose entries are in flight together
#pragma clang loop unroll(disable)
    for (int j = 0; j < NBUF && j < ntiles; j += STEP) issue(j, std::integral_constant<int, STEP>{});

    // fragment read addresses: a lane constant plus the ring slot's offset (see sparse_batch_kernel)
    const unsigned smem_addr = lds_addr(smem);
    unsigned kaddr[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        kaddr[ks] = smem_addr + (((unsigned)(l16 * ROW_BYTES) | (unsigned)(((lg4 ^ sb_swz(l16)) & (CH - 1)) << 4)) ^ (unsigned)(ks << 6));
    const int jj = l16 >> 2, q4 = l16 & 3;
    const int vr = 4 * lg4 + jj;
    unsigned vaddr[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        vaddr[dt] = smem_addr + (((unsigned)(vr * ROW_BYTES + 8 * (q4 & 1)) | (unsigned)((((q4 >> 1) ^ sb_swz(vr)) & (CH - 1)) << 4)) ^ (unsigned)(dt << 5));

    f32x4_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    constexpr float kLazy = 8.f, kFloor = -3.0e38f;      // lazily raised softmax reference (see sparse_batch_kernel)
    float m_run = kFloor, l_run = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" ::"v"(qf[ks]));

    auto step = [&](int t) {                              // this wavefront's tile of an iteration, in ring slot t % NBUF
        const unsigned koff = (unsigned)(t % NBUF) * BUF_BYTES, voff = koff + MAT_BYTES;
        u32x4_t kf[KS][2];
        static_for<KS>([&](auto S) {
            constexpr int i = decltype(S)::value;
            kf[i][0] = lds_read_b128<0>(kaddr[i] + koff);
            kf[i][1] = lds_read_b128<BLK>(kaddr[i] + koff);
        });
        // scores: sc[b][v] = S^T(key 16*b + 4*lg4 + v of the tile, query row l16)
        f32x4_t sc[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
        static_for<KS>([&](auto S) {
            constexpr int i = decltype(S)::value;
            static_for<2>([&](auto BI) {
                constexpr int b = decltype(BI)::value;
                lds_wait<2 * KS - 1 - (2 * i + b)>(kf[i][b]);
                sc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kf[i][b]), qf[i], sc[b], 0, 0, 0);
            });
        });
        constexpr int kPre = DT < 4 ? DT : 4;             // V^T fragments that travel while the softmax runs
        u32x2_t lo[DT], hi[DT];
        static_for<kPre>([&](auto T) {
            constexpr int dt = decltype(T)::value;
            lo[dt] = lds_read_tr16_b64<0>(vaddr[dt] + voff);
            hi[dt] = lds_read_tr16_b64<BLK>(vaddr[dt] + voff);
        });
        const int valid = n_keys - t * TK;                // >= 1
        if (valid < TK) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (16 * b + 4 * lg4 + v >= valid) sc[b][v] = -INFINITY;
        }
        float mx = fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3]));
        mx = fmaxf(mx, fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
        {   // the other keys of this query row sit in the three other 16-lane rows of the wavefront
            float x0, x1;
            lane_rows16(mx, x0, x1);
            mx = fmaxf(x0, x1);
            lane_halves(mx, x0, x1);
            mx = fmaxf(x0, x1) * a.scale_log2;
        }
        if (__any(mx > m_run + kLazy)) {
            const float m_new = fmaxf(m_run, mx);
            const float corr = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= corr;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
        }
        bf16x8_t pf;
        float psum = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float p = __builtin_amdgcn_exp2f(fmaf(sc[b][v], a.scale_log2, -m_run));
                psum += p;
                pf[4 * b + v] = (__bf16)p;
            }
        l_run += psum;
        static_for<DT>([&](auto T) {
            constexpr int dt = decltype(T)::value;
            constexpr int younger = ((dt + kPre < DT ? dt + kPre : DT) - dt - 1) * 2;
            lds_wait<younger>(lo[dt], hi[dt]);
            const u32x4_t both = {lo[dt][0], lo[dt][1], hi[dt][0], hi[dt][1]};
            o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, both), pf, o[dt], 0, 0, 0);
            if constexpr (dt + kPre < DT) {
                lo[dt + kPre] = lds_read_tr16_b64<0>(vaddr[dt + kPre] + voff);
                hi[dt + kPre] = lds_read_tr16_b64<BLK>(vaddr[dt + kPre] + voff);
            }
        });
    };

    // Iteration: tiles t0 .. t0 + KP - 1.  All slots are requested up front; from the second iteration on the slots of the
    // iteration before are refilled, after the barrier that says everyone has left them.
#pragma clang loop unroll(disable)
    for (int t0 = 0; t0 < ntiles; t0 += KP) {
        const int tn = t0 - KP + NBUF;                    // what goes into the slots of the iteration before
        auto refill = [&] {
            if (t0 == 0 || tn >= ntiles) return;
            if (tn + KP > idx_t0 + SB_IDX_TILES && tn * TK < nk) {                // uniform; rare (k > 2048)
                load_idx(tn);
                __syncthreads();
            }
            issue(tn, std::integral_constant<int, STEP>{});
            if constexpr (KP > STEP) issue(tn + STEP, std::integral_constant<int, STEP>{});
        };
        if constexpr (NBUF > KP) {
            // landed: everything but the NBUF - 2 * KP tiles behind this iteration's (all NBUF - KP of them in the first one)
            if (t0 > 0 && t0 + NBUF - KP <= ntiles) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NBUF - 2 * KP) * UPW) : "memory");
            else if (t0 == 0 && NBUF <= ntiles) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NBUF - KP) * UPW) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __syncthreads();
            refill();
        } else {
            if (t0 > 0) {
                __syncthreads();
                refill();
            }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __syncthreads();
        }
        if (wave_active && t0 + kp < ntiles) step(t0 + kp);
    }

    // ---- merge of the key parts through LDS; each of them finishes some of the channel tiles ----
    float l_w = l_run + __shfl_xor(l_run, 16);
    l_w += __shfl_xor(l_w, 32);
    float (*ml)[NW][16] = reinterpret_cast<float (*)[NW][16]>(smem + PART_BYTES);
    f32x4_t *part = reinterpret_cast<f32x4_t *>(smem);    // [wave][dt][lane]
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();                                      // every wavefront is done with the ring
    if (lg4 == 0) {
        ml[0][wave][l16] = m_run;
        ml[1][wave][l16] = l_w;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) part[(wave * DT + dt) * 64 + lane] = o[dt];
    __syncthreads();
    float M = kFloor;
#pragma unroll
    for (int s = 0; s < KP; ++s) M = fmaxf(M, ml[0][s * RW + rw][l16]);
    float wgt[KP], lt = 0.f;
#pragma unroll
    for (int s = 0; s < KP; ++s) {
        wgt[s] = __builtin_amdgcn_exp2f(ml[0][s * RW + rw][l16] - M);
        lt = fmaf(wgt[s], ml[1][s * RW + rw][l16], lt);
    }
    if (row >= a.R) return;
    const int gl = a.B == 1 ? row : (int)(((unsigned long long)(unsigned)row * a.inv_B) >> 32), qi = row - gl * a.B;
    const long long orow = (long long)qi * a.Hq + (long long)h * a.G + gl;
    float *dst = a.out + z * a.seq_out + orow * D;
    const float inv = 1.f / lt;
    for (int dt = kp; dt < DT; dt += KP) {
        f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KP; ++s) acc += part[((s * RW + rw) * DT + dt) * 64 + lane] * wgt[s];
        *reinterpret_cast<f32x4_t *>(dst + 16 * dt + 4 * lg4) = acc * inv;
    }
    if (a.lse_out && kp == 0 && lg4 == 0) a.lse_out[z * a.seq_lse + orow] = (M + log2f(lt)) * 0.6931471805599453f;
}

// As few row tiles per workgroup, two or four, as still give every workgroup a compute unit of its own (ids come in blocks of 8
// units; calls that could have one are sparse_bf16.hip's).
// (With 320 .. 512 workgroups of 4 row tiles and a ring of half the size, two per CU: 32 heads, k = 300, 24 sequences 17.8 us
// against 16.4 with 128-row workgroups; no gain.)  Units that fill the chip one each anyway and are long are bound by
// the gather's bandwidth, which the other kernel's continuous stream of requests uses better than whole iterations at a
// time (256 units, k = 1000: 29.4 against 31.6 us; k = 100: 8.2 against 7.5 us).
int sparse_few_row_tiles(long long n_units, int R, int n_keys)
{
    const long long ids = (n_units + 7) / 8 * 8;
    if (ids * ((R + 127) / 128) >= 256 && n_keys > 512) return 0;
    for (int rw = 2; rw <= 4; rw *= 2)
        if (ids * ((R + 16 * rw - 1) / (16 * rw)) <= 256) return rw;
    return 0;
}

template <int D>
static hipError_t launch_few(const BatchArgs &a, int row_tiles, hipStream_t stream)
{
    const int row_groups = (a.R + 16 * row_tiles - 1) / (16 * row_tiles);
    dim3 grid(8 * row_groups, (a.n_units + 7) / 8), block(SB_WAVES * 64);
    if (row_tiles == 2) hipLaunchKernelGGL((sparse_few_kernel<D, 2>), grid, block, 0, stream, a);
    else if (row_tiles == 4) hipLaunchKernelGGL((sparse_few_kernel<D, 4>), grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_sparse_few(const BatchArgs &a, int d, int row_tiles, hipStream_t stream)
{
    if (d == 128) return launch_few<128>(a, row_tiles, stream);
    if (d == 64) return launch_few<64>(a, row_tiles, stream);
    return hipErrorInvalidValue;
}

}  // namespace mage
