// The expert computation's form for few rows (ffn_thin.hip), as ffn.hip sees it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe {

struct TileTableHeader;
struct TileEntry;

constexpr int kThinRows = 64;  // rows of a row tile

// The tables hold one entry per row tile.
void launch_thin_gate_up(const uint16_t *A, int64_t M, int64_t H, int64_t F, const uint16_t *W_gate, const uint16_t *W_up,
                         uint16_t *a, TileTableHeader *hdr, const TileEntry *table, int row_tiles, int out_cols,
                         const int32_t *gather_rows, int gather_div, uint32_t gather_bytes, hipStream_t st);
// scatter_w != nullptr: `y` is the fp32 sums that the weighted rows are added to (see GEMM's kScatter)
void launch_thin_down(const uint16_t *a, int64_t M, int64_t H, int64_t F, const uint16_t *W_down, void *y,
                      TileTableHeader *hdr, const TileEntry *table, int row_tiles, int out_cols, const int32_t *row_of_slot, int K,
                      const float *scatter_w, hipStream_t st);

}  // namespace moe
