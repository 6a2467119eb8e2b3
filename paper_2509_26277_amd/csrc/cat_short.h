// Inference over short rows (cat_short.hip): interface to the host driver.
#pragma once
#include "cat_common.h"

namespace cat {

// whether the kernel takes this shape and is the fastest there
bool short_apply_pays(int64_t N, int64_t D, int32_t K, cat_dtype dt);
// cat_apply; needs no scratch
cat_status short_apply(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, const float* cent, const float* gamma,
                       const float* beta, float alpha, void* corrected, int32_t* assign, hipStream_t st);

}  // namespace cat
