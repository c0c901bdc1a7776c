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

// Tile sizes (rows x columns) and the measured time in us of a tile's K-step of 64, a CU's tiles
// one after another (two workgroups of a CU together: per tile).  Each step moves (rows +
// columns) x 128 bytes into LDS, at about 60 GB/s per CU for all of them.
constexpr int kGemmTiles = 5;
constexpr int kTileRows[kGemmTiles] = {32, 64, 128, 128, 128};
constexpr int kTileCols[kGemmTiles] = {64, 64, 64, 128, 256};
constexpr float kTileStep[kGemmTiles] = {0.18f, 0.23f, 0.38f, 0.55f, 0.84f};

// Entries mt_first .. mt_first + n_mt - 1 of the row-tile list (without one: of the 256-row tiles
// of M) on tile size `tile`.  n_cu: a multiple of 8.
// kPartial: K in `splits` pieces of whole steps, C = part[splits][M][ldc] float32.
void gemm_tiles(int epi, int tile, const GemmArgs& g, int mt_first, int n_mt, int n_cu, hipStream_t s, int splits = 1);

}  // namespace ppk
