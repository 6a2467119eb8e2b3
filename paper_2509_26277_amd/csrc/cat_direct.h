// Fused inference for few rows in one launch (cat_direct.hip).
#pragma once
#include "cat_tile.h"

namespace cat {

// Whether the call is small enough for it to be the faster one.
bool direct_apply_pays(int64_t N, int64_t D, int32_t K, cat_dtype dt);
// corrected = x + alpha (gamma[a] x + beta[a] - x), a = nearest centroid of x; gamma, beta: K x D as fitted; assign nullable.
cat_status direct_apply(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, const float* cent, const float* gamma,
                        const float* beta, float alpha, void* corrected, int32_t* assign, hipStream_t st);

}  // namespace cat
