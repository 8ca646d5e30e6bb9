// Weight gradient on the sparsity pattern: the product's tables, made once per handle, and its launch (sprnn_wgrad.hip), and
// the kernel that keeps one sum per lane and nonzero (sprnn_wgrad_lanes.hip).  sprnn_wgrad_rule.h says which is taken when.
#ifndef SPRNN_WGRAD_H_
#define SPRNN_WGRAD_H_

#include <hip/hip_runtime.h>

#include <cstdint>

#include "sprnn_wgrad_rule.h"

namespace sprnn {

// starts[t * rows + r] = CSR position of row r's first nonzero at or beyond column t * tile_cols, t = 0 .. column tiles.
hipError_t launch_tile_starts(const int32_t* row_ptr, const int32_t* col, int rows, int cols, int tile_cols, int32_t* starts,
                              hipStream_t stream);

// dU[p] = sum_m a[m][row(p)] * b[m][col(p)] over all stored nonzeros p, m = 0 .. vectors - 1 (time x batch).
struct WGradOperand {
  const float* x = nullptr;          // [vectors][ld]
  const float* first = nullptr;      // shifted operands: the first `shift` vectors, [shift][ld], or null (zeros)
  int ld = 0;
  int shift = 0;                     // 0, or batch: vector m is first[m] for m < shift, x[m - shift] beyond
};
struct WGradArgs {
  WGradOperand a, b;                 // row side (ld = rows of the matrix), column side (ld = its columns)
  const float* gate = nullptr;       // where set: columns from gate_from on are b[m][c] * gate[m][c - gate_from] (rounded once),
  int gate_from = 0, gate_ld = 0;    // ... [vectors][gate_ld] (no shift on the column side then)
  const int32_t* col;                // CSR column indices
  const int32_t* starts;             // from launch_tile_starts
  float* dU;
  int vectors, nnz;
};
hipError_t launch_weight_gradient(const WGradArgs& args, WGradTile tile, hipStream_t stream);
hipError_t prepare_weight_gradient(WGradTile tile, bool gated);   // once per device before the first launch (with gate set)

// The lane sums: same sums, in time order, on the forward mapping.
struct LaneSumsArgs {
  const uint32_t* words;             // the handle's packed words (only the column offsets are used)
  const int32_t* lane_row;           // [grid][block]
  const int32_t* wave_words;         // [grid][waves]
  const int32_t* word_src;           // [grid][NW][block] CSR position of each packed word, -1 for padding
  const float* delta;                // [T][B][rows]
  const float* h_fwd;                // [T][B][H] forward outputs h_1..h_T
  const float* h0;                   // [B][H] or null (zeros)
  float* dU;                         // [nnz] CSR order
  int hidden, T, index_shift;
  int rows;                          // rows of the matrix: hidden, or 3 or 4 times as many for the gated cells
};
const void* lane_sums_kernel_for(int batch, int template_words);

}  // namespace sprnn
#endif
