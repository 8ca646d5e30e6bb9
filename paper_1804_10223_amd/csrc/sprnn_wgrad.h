// Weight gradient on the sparsity pattern: tables made once per handle and the launch (see sprnn_wgrad.hip).
#ifndef SPRNN_WGRAD_H_
#define SPRNN_WGRAD_H_

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sprnn {

struct WGradTile {
  int rows = 0, cols = 0;            // shape of one workgroup's part of the dense product
};
// The tile shape for a matrix of this size on a device with this many CUs.
WGradTile choose_weight_gradient_tile(int rows, int cols, int num_cus);

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
  const int32_t* col;                // CSR column indices
  const int32_t* starts;             // from launch_tile_starts
  float* dU;
  int vectors, nnz;
};
hipError_t launch_weight_gradient(const WGradArgs& args, WGradTile tile, hipStream_t stream);
hipError_t prepare_weight_gradient(WGradTile tile);   // once per device before the first launch

}  // namespace sprnn
#endif
