// What the kernels share in which clusters are the M dimension of the products (cat_loop.hip, cat_short.hip): lanes n, n + 16, n + 32
// and n + 48 hold the values of row n of a tile, each for a quarter of the clusters.
#pragma once
#include "cat_common.h"

namespace cat {

// the values of a lane and of its partner 16 or 32 lanes on, lower one first: the same pair in both
__device__ __forceinline__ void halves16(uint32_t v, uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void halves32(uint32_t v, uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ float sum_groups(float v) {  // over the four lanes of a row
    uint32_t a, b;
    halves16(__float_as_uint(v), a, b);
    halves32(__float_as_uint(__uint_as_float(a) + __uint_as_float(b)), a, b);
    return __uint_as_float(a) + __uint_as_float(b);
}
// the least score f1 of the four lanes of a row, its cluster i1 (the lowest one on ties) and the second least f2, in all of them
__device__ __forceinline__ void best_two_groups(float& f1, int& i1, float& f2) {
#pragma unroll
    for (int o = 0; o < 2; o++) {
        uint32_t a1, c1, a2, c2, ai, ci;
        if (o == 0) {
            halves16(__float_as_uint(f1), a1, c1);
            halves16(__float_as_uint(f2), a2, c2);
            halves16((uint32_t)i1, ai, ci);
        } else {
            halves32(__float_as_uint(f1), a1, c1);
            halves32(__float_as_uint(f2), a2, c2);
            halves32((uint32_t)i1, ai, ci);
        }
        const float x1 = __uint_as_float(a1), y1 = __uint_as_float(c1);
        const bool take = y1 < x1 || (y1 == x1 && (int)ci < (int)ai);
        f1 = take ? y1 : x1;
        i1 = take ? (int)ci : (int)ai;
        f2 = fminf(fminf(__uint_as_float(a2), __uint_as_float(c2)), take ? x1 : y1);
    }
}
// The error bound of the split arithmetic: tau |x| |c| + tau2 |c|^2 for n_acc accumulations of products of two bf16 parts each
// (rows of bf16: exact, one part), as in the tile kernels (cat_tile.hip: base_params).
inline float split_tau(cat_dtype dt, int n_acc) { return (dt == CAT_BF16 ? 3.1e-5f : 9.4e-5f) + 4.f * (float)n_acc * 5.96e-8f; }
constexpr float kSplitTau2 = 4.0e-7f;

}  // namespace cat
