// Host side of the small-tile FFN kernels (ffn_tile.hip).
#pragma once

#include "common.hpp"

namespace fm {

// Which kernels run a layer's products over T tokens, top-k: the large-tile
// bf16 kernels of ffn.hip or one of the small tiles.  A pure function of the
// layer's shape, T and k (the bucket sizes are only known on the device).
struct TilePlan {
  enum Rows { LARGE_ROWS, ROWS_32, ROWS_64, ROWS_128 } rows;   // gate-up, down, dH, dX
  enum Dw { LARGE_DW, SMALL_DW } dw;                           // dW_gate/up, dW_down
};
TilePlan tile_plan(const moe_layer* L, int T, int k);
// The tile of a small-tile weight gradient: 64 x 32 with k split (fp32), 64 x 64 (fp32)
// or 64 x 128 (bf16), 128 x 128 (bf16).
enum DwTile { DW_SPLIT_K, DW_64, DW_128 };
DwTile dw_tile(const moe_layer* L, int T, int k, bool gate_up);
// Columns of I per partial of the utility's row norms (the dH column tile).
int tile_norm_cols(const moe_layer* L, const TilePlan& p);
constexpr int NORM_COLS_MIN = 64;   // the fewest that any plan takes

void tile_fwd(const TilePlan& p, const moe_layer* L, const void* X, const void* Xp, const int32_t* offsets, int T,
              int k, void* Ag, void* Au, void* H, void* O, hipStream_t st);
// dAg, dAu: [rows, ldA] scratch; norms: per row and dH column tile (sum dA^2, sum h^2).
void tile_dh(const TilePlan& p, const moe_layer* L, const int32_t* offsets, int T, int k, const void* Ag,
             const void* Au, const void* dO, void* dAg, void* dAu, int ldA, float2* norms, hipStream_t st);
void tile_dw(const moe_layer* L, const void* X, const void* Xp, const int32_t* offsets, int T, int k, const void* H,
             const void* dO, const void* dAg, const void* dAu, int ldA, int accumulate, hipStream_t st);
void tile_dx(const TilePlan& p, const moe_layer* L, const int32_t* offsets, int T, int k, const void* dAg,
             const void* dAu, int ldA, void* dXp, hipStream_t st);

// Rows of the int8 forward's row tile: 32, 64, 128, or 256 (the kernels of ffn.hip).
int q8_tile(const moe_layer_q8* L, int T, int k);
// The int8 forward on a tile of fewer than 256 rows.
void tile_fwd_q8(const moe_layer_q8* L, const void* X, const void* Xp, const int32_t* offsets, int T, int k, void* H,
                 void* O, hipStream_t st);

// One block per compute unit, rounded to the XCD count.
int persistent_blocks();

}  // namespace fm
