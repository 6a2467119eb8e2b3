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

// The passes 3 .. iters of tile_lloyd with bounds (record), once pass 2 has evaluated every row: sums holds the cluster sums before
// that pass's list (K x D doubles, twice as many of scratch behind them), cent_io that pass's centroids.  Same outputs.
struct LoopBounds {
    double* expire;              // as pass 2 left it
    int32_t* rows;               // N + 63
    const uint32_t* list_count;  // rows that changed cluster in pass 2 (lw.list)
    const int32_t* counts;       // rows per cluster in pass 2
};
bool loop_bounds_pays(int64_t N, int64_t D, int32_t K, int32_t iters, cat_dtype dt);
cat_status loop_lloyd_bounds(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, int32_t iters, float* cent_io, double* sums,
                             int32_t* assign, int32_t* counts, double* inertia, unsigned long long* rep, const LloydWs& lw,
                             const LoopBounds& lb, hipStream_t st);

}  // namespace cat
