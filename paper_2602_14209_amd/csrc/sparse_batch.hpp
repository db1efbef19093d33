// What the two kernels of the batched sparse step share (sparse_batch_bf16.hip, sparse_few_bf16.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ids.hpp"
#include "lds_asm.hpp"
#include "plan.hpp"

namespace mage {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

constexpr int SB_WAVES = 8;
constexpr int SB_TK = 32;                    // keys per tile (two 16-key MFMA blocks)
constexpr int SB_IDX_TILES = 64;             // tiles whose index entries LDS holds at a time (2048 entries)

// What the kernel needs of a call, packed: the kernel arguments arrive through scalar loads that the very
// first instructions wait for, so they are few and adjacent, and what the host can work out is worked out
// there (the divisions by Hkv and B become a multiply-high).
struct BatchArgs {
    const void *q, *kc, *vc, *kblk, *vblk;
    const int32_t *idx;
    float *out, *lse_out;
    long long seq_q, seq_kv, seq_idx, seq_blk, seq_out, seq_lse;   // element strides between sequences
    int B, Hq, Hkv, G, R;
    int nk, n_blk;               // selected cache rows, the block's own rows (0 = none)
    int n_units;                 // n_seq * Hkv
    unsigned inv_Hkv;            // ceil(2^32 / Hkv) for Hkv >= 2: unit / Hkv == mulhi(unit, inv_Hkv) while unit * Hkv < 2^32
    unsigned inv_B;              // the same for B (row * B < 2^32)
    float scale_log2;
};

constexpr int SB_GRID_Y = 32768;            // workgroup id: x = place inside a block of ids, (z, y) = block (y < SB_GRID_Y)

// XOR swizzle of the 16-byte chunk index of tile row r (taken modulo 16): the 16 rows of a K fragment
// read and the 8 rows of one phase of a transposing V read land on distinct LDS banks.
__device__ __forceinline__ int sb_swz(int r) { return ((r & 7) << 1) | ((r >> 3) & 1); }

// The kernel for few units: 0 = the call has enough of them for sparse_batch_kernel, otherwise the row tiles per workgroup
int sparse_few_row_tiles(long long n_units, int R, int n_keys);
hipError_t launch_sparse_few(const BatchArgs &a, int d, int row_tiles, hipStream_t stream);

}  // namespace mage
