// The projection GEMMs on smaller output tiles (k_gemm_tiles.hip): what k_gemm_bf16.hip's choice
// of kernels needs to know about them.
#pragma once
#include "kernels.h"

namespace ppk {

// C[M, N] = A B^T, or the QKV outputs; mtile_m0: a plan's row-tile list, or null for every row.
struct GemmArgs {
    const void* A;
    int64_t lda;
    const void* B;
    int64_t ldb;
    void* C;
    int64_t ldc;
    int M, N, K;
    const int32_t* mtile_m0;
    QkvOut qkv;
};

// CUs of the GPU, rounded down to a multiple of 8 so that every XCD runs the same number of workgroups.
int cu_count();

// Tile sizes (rows x columns) and the measured time in us of a tile's K-step of 64, a CU's tiles
// one after another (two workgroups of a CU together: per tile).  Each step moves (rows +
// columns) x 128 bytes into LDS, at about 60 GB/s per CU for all of them (weights in the Infinity Cache).
constexpr int kGemmTiles = 5;
constexpr int kTileRows[kGemmTiles] = {32, 64, 128, 128, 128};
constexpr int kTileCols[kGemmTiles] = {64, 64, 64, 128, 256};
constexpr float kTileStep[kGemmTiles] = {0.18f, 0.23f, 0.38f, 0.55f, 0.84f};

// Entries mt_first .. mt_first + n_mt - 1 of the row-tile list (without one: of the 256-row tiles
// of M) on tile size `tile`.  n_cu: a multiple of 8.
// kPartial: K in `splits` pieces of whole steps, C = part[splits][M][ldc] float32.
void gemm_tiles(int epi, int tile, const GemmArgs& g, int mt_first, int n_mt, int n_cu, hipStream_t s, int splits = 1);

// The LM head of k prompts (hl [k, d], W [V, d], any V, d % 64 == 0) on 128 x 256 tiles: float32
// logits [k, V] unless null, and the best (logit, lowest id) of prompt m among vocabulary rows
// 128 b .. + 127 to part[m n_blocks + b] (an ArgMax; n_blocks = ceil(V / 128)).
void lm_head_tiles(const void* hl, int k, const void* W, int V, int d, float* logits, void* part, int n_blocks,
                   hipStream_t s);

}  // namespace ppk
