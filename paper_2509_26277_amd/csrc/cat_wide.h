// Fused inference for shapes whose centroid operand no wave can hold (cat_wide_kernel.h).
#pragma once
#include "cat_tile.h"

namespace cat {

// Whether the kernel has an instance for the shape: rows of at most 4 KB (more than 128 clusters: 3 KB), K <= 256, and none of
// the row-tile kernel's that cat_apply always prefers.
bool wide_supported(int64_t N, int64_t D, int32_t K, cat_dtype dt);
// Cluster tiles of its operand (0: no instance).
int wide_cluster_tiles(int64_t D, int32_t K, cat_dtype dt);
// Nearest centroid and affine map in one pass (gamma, beta: K x D with the blending coefficient folded in); assign nullable;
// fold as in infer_apply.
cat_status wide_apply(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, const float* cent, const float* gamma,
                      const float* beta, void* corrected, int32_t* assign, const TileWs& ws, hipStream_t st,
                      const FoldAlpha* fold = nullptr);

}  // namespace cat
