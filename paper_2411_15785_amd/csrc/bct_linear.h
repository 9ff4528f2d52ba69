// What the projection kernels' files share: the outputs of a projection and the tiled activation layout.
#ifndef BCT_LINEAR_H
#define BCT_LINEAR_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bct {

// Up to three row-major outputs side by side along N: output i takes the features [start[i], start[i + 1]).
struct LinearOut {
  uint16_t* ptr[3];
  uint32_t start[4];
};

// Tiled activations: rows in groups of 32, inputs in groups of 32; group (r / 32, k / 32) is 2 KB, two A
// operands of v_mfma_f32_16x16x32_bf16 (rows 0-15 and 16-31 of the group), each 64 lanes x 16 bytes with
// lane 16 * ((k % 32) / 8) + r % 16 holding the inputs k % 8 = 0..7.  Returns the 16-byte chunk index.
__device__ __forceinline__ size_t tiled_chunk(uint32_t r, uint32_t k, uint32_t K) {
  return ((((size_t)(r / 32) * (K / 32) + k / 32) * 2 + (r % 32) / 16) * 64) + 16 * ((k % 32) / 8) + r % 16;
}

// What a projection launch gives each workgroup: rows x features (SwiGLU: of the product), and in how many parts K is
// summed (each a chain of its own, the parts added in order).
struct LinearTile {
  uint32_t rows, features, k_parts;
};

// The tile of launch_linear_rows for a shape: host logic, what that launch itself goes by.
LinearTile linear_rows_tile(uint32_t rows, uint32_t K, uint32_t N, bool swiglu, bool x_tiled);

// The matrix-core projection of many rows (bct_linear_rows.hip).  w2 non-null: SwiGLU of w and w2.  x_tiled /
// out_tiled: activations in the tiled order.  N is a multiple of 16 (out_tiled: 32), K of 32.
hipError_t launch_linear_rows(const void* x, const void* w, const void* w2, const void* residual, const LinearOut& dst,
                              uint32_t rows, uint32_t K, uint32_t N, bool x_tiled, bool out_tiled, hipStream_t s);

}  // namespace bct

#endif
