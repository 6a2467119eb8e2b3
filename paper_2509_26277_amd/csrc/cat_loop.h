// The whole Lloyd loop of a small fit in one launch (cat_loop.hip): interface to the host driver.
#pragma once
#include "cat_tile.h"

namespace cat {

// Whether the loop in one launch takes this shape, and whether it is the faster one there.
bool loop_pays(int64_t N, int64_t D, int32_t K, int32_t iters, cat_dtype dt);
// tile_lloyd without distance bounds, same outputs: iterates in place in cent_io and stops once the partition repeats.  sums is 3 x K x D
// doubles of scratch; lw.sort_ws and lw.list serve as scratch too.  skipped (nullable) receives the number of passes left out.
cat_status loop_lloyd(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, int32_t iters, float* cent_io, double* sums,
                      int32_t* assign, int32_t* counts, double* inertia, unsigned long long* rep, int32_t* skipped,
                      const LloydWs& lw, hipStream_t st);

}  // namespace cat
