// Host-side launch plans and workspace layout for the MAGE kernels (gfx950).
//
// A plan is a pure function of the problem geometry, so mage_workspace_bytes() and the
// launchers always agree.  Partial results of split attention live in the caller's workspace:
//   part_o [Hkv][n_split][rpad][d] fp32  unnormalised weighted value sums
//   part_m [Hkv][n_split][rpad]    fp32  running maximum of the log2-scaled logits
//   part_l [Hkv][n_split][rpad]    fp32  sum of exp2(logit2 - part_m)
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "../../include/mage.h"

namespace mage {

constexpr int kBf16Tile = 64;   // keys per LDS tile, MFMA path
constexpr int kF32Workgroups = 256;      // fp32 path, attention and statistics: one 8-wavefront workgroup per CU (registers)
constexpr int kF32ColsumWorkgroups = 512;   // fp32 path, column sums: two 4-wavefront workgroups per CU
constexpr int kBf16Workgroups = 256;     // MFMA path: one 8-wavefront workgroup per CU (its tile ring fills the LDS)

struct SplitPlan {
    int R;            // query rows sharing one KV head: G*B
    int rows_per_wg;  // rows one workgroup covers
    int row_groups;   // workgroups along the row axis
    int rpad;         // row_groups * rows_per_wg
    int waves;        // wavefronts per workgroup of the column-sum pass (one per 32 rows; MFMA path)
    int tile;         // keys per tile (fp32: keys a workgroup covers per round, 16 per key slice)
    int rw;           // fp32: 16-row tiles per workgroup (1 or 2); its 8 wavefronts are rw row tiles x 8/rw key slices
    int kps;          // cache keys per split (multiple of tile)
    int n_split;      // splits along the key axis, including a block-only split if any
    int n_cyc;        // splits that own cache keys (the first n_cyc)
    int blk_split;    // split that also attends the in-block keys
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// 16-key tiles of the fp32 kernels: those of the cache, then those of the block, which no tile mixes
inline int64_t f32_key_tiles(int64_t cache_keys, int block_keys) { return (cache_keys + 15) / 16 + (block_keys + 15) / 16; }

// `keys`: cache keys of the pass.  fp32: a workgroup with two row tiles reads its keys once for both; four would leave two key
// slices, twice the splits for the same number of workgroups and twice the partial results (B*G = 64, L = 16384, d = 128: 34.6 against
// 33.4 us; 224 rows: 95.6 against 86.4, 14 row tiles being no multiple of four).  One row tile and eight key slices while all
// of that fits the chip in one round, where only the length of the round counts (k = 200, B*G = 64: 12.3 us; 17.3 with two
// row tiles, 20.9 with four).
inline void plan_rows(const mage_shape &s, SplitPlan &p, int64_t keys)
{
    p.R = (s.Hq / s.Hkv) * s.B;
    if (s.dtype == MAGE_BF16) {
        p.rows_per_wg = 128;
        p.waves = p.R > 128 ? 8 : 4;
        p.tile = kBf16Tile;
    } else {
        p.waves = 4;
        const int64_t one_round = (int64_t)s.Hkv * ceil_div(p.R, 16) * ((keys + 127) / 128);
        p.rw = p.R > 16 && one_round > kF32Workgroups ? 2 : 1;
        p.rows_per_wg = 16 * p.rw;
        p.tile = 16 * (8 / p.rw);
    }
    p.row_groups = ceil_div(p.R, p.rows_per_wg);
    p.rpad = p.row_groups * p.rows_per_wg;
}

// Dense pass over all L cache keys, cut into at most `target_workgroups`.  A CU that holds one workgroup more than the
// others ends that much later, so the count stays at or below a multiple of 256: with tiles of 64 keys, 33 splits of 8 heads (264
// workgroups of 2 tiles) measured 16.5 us where 22 splits (176 of 3 tiles) take 12.9.  Every workgroup pays a fixed 4 to
// 5 us (cold code, first tile, merge), so up to 64 tiles go one per split (L = 1500, B = 8, 16 heads: 11.0 us against 13.2
// with at least four); beyond that a split has at least two, because exact attention pays a [rows x d] partial per split.  The
// fp32 kernels pay 1.9 us (d = 128) per round of tiles, more than a partial costs (B*G = 16, L = 1024: 12.9 us with one round,
// 16.0 with two, 21.4 with four).
inline SplitPlan plan_dense(const mage_shape &s, int target_workgroups = 0, bool rows_in_one_workgroup = false)
{
    SplitPlan p{};
    plan_rows(s, p, s.L);
    if (target_workgroups == 0) target_workgroups = s.dtype == MAGE_BF16 ? kBf16Workgroups : kF32Workgroups;
    const int64_t tiles = (s.L + p.tile - 1) / p.tile;
    const int64_t per_split = (int64_t)s.Hkv * (rows_in_one_workgroup ? 1 : p.row_groups);   // workgroups per key split
    const int64_t target = target_workgroups / per_split > 0 ? target_workgroups / per_split : 1;
    int64_t tps = (tiles + target - 1) / target;     // tiles per split
    const int64_t min_tps = s.dtype == MAGE_BF16 && tiles > 64 ? 2 : 1;
    if (tps < min_tps) tps = min_tps;
    p.n_split = (int)((tiles + tps - 1) / tps);
    p.kps = (int)(tps * p.tile);
    p.blk_split = p.n_split - 1;
    p.n_cyc = p.n_split;
    return p;
}

// Selection, first pass (row statistics).  Two workgroups fit a CU.  With few query rows they are worth having (memory
// latency: B*G = 32, L = 32768: 35.0 against 35.8 us for the selection); with more than 64 the vector ALU is busy with one, and
// half as many splits are half as many statistics to merge (B*G = 224, L = 32768: 37.1 against 40.7 us).
inline SplitPlan plan_stats(const mage_shape &s)
{
    const int R = (s.Hq / s.Hkv) * s.B;
    return plan_dense(s, s.dtype == MAGE_BF16 ? (R > 64 ? 1 : 2) * kBf16Workgroups : kF32Workgroups);
}

// Selection, second pass (column sums).  The MFMA kernel parks the sums of up to kColsumTiles tiles
// in LDS and writes them out together.  Like the statistics pass it wants long splits (every
// workgroup pays a pipeline fill) and a power-of-two number of them.
constexpr int kColsumTiles = 8;
constexpr int kGroupKeys = 16;           // keys per group maximum handed from the column sums to the top-k filter
// The MFMA kernel keeps all rows of a KV head in one workgroup.  4 wavefronts: three workgroups fit a CU; at d = 64
// three are the fastest, at d = 128 two (L = 32768: 40.1 against 41.8 us).  8 wavefronts: one per CU while its tiles fit the
// ring of finished sums (L = 16411: 33.0 us for the selection against 35.2 with 260 workgroups), then two.
inline SplitPlan plan_colsum(const mage_shape &s)
{
    if (s.dtype != MAGE_BF16) {
        // a workgroup's four wavefronts take 32 keys each per round
        SplitPlan p{};
        plan_rows(s, p, s.L);
        p.tile = 128;
        const int64_t tiles = (s.L + p.tile - 1) / p.tile;
        const int64_t target = kF32ColsumWorkgroups / s.Hkv > 0 ? kF32ColsumWorkgroups / s.Hkv : 1;
        const int64_t tps = (tiles + target - 1) / target;
        p.n_split = (int)((tiles + tps - 1) / tps);
        p.kps = (int)(tps * p.tile);
        p.blk_split = p.n_split - 1;
        p.n_cyc = p.n_split;
        return p;
    }
    const int R = (s.Hq / s.Hkv) * s.B;
    if (R <= 128) return plan_dense(s, (s.d == 64 ? 3 : 2) * kBf16Workgroups, true);
    const SplitPlan one = plan_dense(s, kBf16Workgroups, true);
    return one.kps <= kColsumTiles * one.tile ? one : plan_dense(s, 2 * kBf16Workgroups, true);
}

// Do the column sums merge the row statistics themselves (row_stats.hpp)?  Every one of their workgroups then reads the
// statistics of all splits: 1 us of L2 time at 128 splits of 128 rows, still less than the launch it saves.
constexpr int kMergeSplits = 128, kMergeRows = 256;
inline bool colsum_merges_stats(int rows, int n_split) { return rows <= kMergeRows && n_split <= kMergeSplits; }

// Sparse step: k gathered cache keys and the block's own.  The bf16 kernels merge on chip (one split).  fp32: a second launch
// costs what two rounds of tiles cost at d = 128 and three at d = 64 (k = 200, one row tile: 12.1 us either way; 7.7 against
// 9.6); up to that many stay in one split, whose key slices are merged on chip.
inline SplitPlan plan_sparse(const mage_shape &s)
{
    SplitPlan p{};
    plan_rows(s, p, s.k);
    const bool f32 = s.dtype != MAGE_BF16;
    const int64_t slices = p.tile / 16;
    const int64_t tiles = (f32_key_tiles(s.k, s.B) + slices - 1) / slices;
    const int64_t per_split = (int64_t)s.Hkv * p.row_groups;
    const int64_t target = kF32Workgroups / per_split > 0 ? kF32Workgroups / per_split : 1;
    const int64_t tps = !f32 || tiles <= (s.d == 64 ? 3 : 2) ? tiles : (tiles + target - 1) / target;
    p.n_split = (int)((tiles + tps - 1) / tps);
    p.kps = (int)(tps * p.tile);
    p.n_cyc = p.n_split;
    p.blk_split = p.n_split - 1;
    return p;
}

inline size_t partial_bytes(const mage_shape &s, const SplitPlan &p)
{
    const size_t rows = (size_t)s.Hkv * p.n_split * p.rpad;
    return align_up(rows * s.d * sizeof(float), 256) + 2 * align_up(rows * sizeof(float), 256);
}

struct SelectLayout {
    size_t part_m, part_l, lse2, alpha, gmax, bytes;
};

inline SelectLayout select_layout(const mage_shape &s, const SplitPlan &p)
{
    SelectLayout l{};
    const size_t rows = (size_t)s.Hkv * p.n_split * p.rpad;
    size_t off = 0;
    l.part_m = off; off += align_up(rows * sizeof(float), 256);
    l.part_l = off; off += align_up(rows * sizeof(float), 256);
    l.lse2 = off;   off += align_up((size_t)s.Hkv * p.rpad * sizeof(float), 256);
    l.alpha = off;  off += align_up((size_t)s.Hkv * (size_t)s.L * sizeof(float), 256);
    l.gmax = off;   off += align_up((size_t)s.Hkv * (size_t)((s.L + kGroupKeys - 1) / kGroupKeys) * sizeof(float), 256);
    l.bytes = off;
    return l;
}

// Fused step 1 (exact attention that also feeds selection): the attention partials, then the
// prefix statistics per attention split, then selection's lse2 and alpha.
struct Step1Layout {
    size_t partials, stat_m, stat_l, lse2, alpha, gmax, bytes;
};

inline Step1Layout step1_layout(const mage_shape &s, const SplitPlan &attn)
{
    Step1Layout l{};
    const size_t rows = (size_t)s.Hkv * attn.n_split * attn.rpad;
    size_t off = 0;
    l.partials = off; off += partial_bytes(s, attn);
    l.stat_m = off;   off += align_up(rows * sizeof(float), 256);
    l.stat_l = off;   off += align_up(rows * sizeof(float), 256);
    l.lse2 = off;     off += align_up((size_t)s.Hkv * attn.rpad * sizeof(float), 256);
    l.alpha = off;    off += align_up((size_t)s.Hkv * (size_t)s.L * sizeof(float), 256);
    l.gmax = off;     off += align_up((size_t)s.Hkv * (size_t)((s.L + kGroupKeys - 1) / kGroupKeys) * sizeof(float), 256);
    l.bytes = off;
    return l;
}

// Arguments shared by the attention / statistics / column-sum kernels of both element types.
struct KernelArgs {
    const void *q, *kc, *vc, *kblk, *vblk;
    const int32_t *idx;      // gather indices [Hkv][nc] or nullptr
    float *out, *lse_out;    // final outputs (used directly when n_split == 1)
    float *part_o, *part_m, *part_l;
    float *stat_m, *stat_l;  // exact attention, optional: prefix-only (cache keys) statistics per split, as part_m/part_l
    const float *lse2;       // column-sum pass: per-row log2-domain log-sum-exp [Hkv][rpad]; nullptr: merged there from part_m / part_l
    int stat_split;          // ... of this many splits
    float *alpha;            // column-sum pass: [Hkv][L] (or [Hq][L] with head_rows)
    int head_rows;           // column-sum pass: 0, or B = one grid row per QUERY head, summing that head's B rows only (Eq. 2 per head)
    float *gmax;             // column-sum pass, optional: [Hkv][ceil(L / kGroupKeys)] maxima of alpha over groups of consecutive keys
    int B, Hq, Hkv, G, R, rpad;
    int rw;                  // fp32 path: row tiles per workgroup (SplitPlan::rw)
    long long L;             // rows in the cache
    long long nc;            // cache keys attended: L (dense) or k (gather)
    int kps, n_split, blk_split, n_blk;
    int n_cyc;               // MFMA path: split s < n_cyc owns the cache tiles s, s + n_cyc, s + 2*n_cyc, ...
    // batched launches (grid z = sequence): element strides between consecutive sequences, 0 when not batched
    long long seq_q, seq_kv, seq_idx, seq_blk, seq_out, seq_lse;
    float scale_log2;        // log2(e) / sqrt(d)
    float inv_rows;          // 1 / (G*B)
    // worked out on the host so that the bf16 kernels start without a division (fill_split_consts):
    int tiles_q, tiles_r;    // ceil(nc / 64) cache tiles = tiles_q * n_cyc + tiles_r
    unsigned inv_B;          // ceil(2^32 / B) for B >= 2: row / B == (row * inv_B) >> 32 while row * B < 2^32
};

// What the top-k kernel needs to re-score the few candidates whose fp32 alpha lies within `eps`
// (relative) of the k-th value in fp64 from the inputs (see topk.hip); q == nullptr switches it off.
struct RescoreArgs {
    const void *q, *kc;              // queries [B,Hq,d], keys [L,Hkv,d]
    const float *stat_m, *stat_l;    // row statistics per key split [Hkv][n_split][rpad], log2 domain
    int esz;                         // bytes per element of q / kc: 2 (bf16) or 4 (fp32)
    int d, Hq, Hkv, G, B, R, n_split, rpad;
    float scale_log2;                // the factor the statistics were taken with
    int split_q;                     // q has d / 2 channels, to be split by sign into [max(q, 0) | min(q, 0)]
    double inv_rows;                 // 1 / (R * key weight)
    float eps;
};

}  // namespace mage
