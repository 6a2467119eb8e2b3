// Leading eigenpairs of a symmetric matrix (cat_eig.hip), for the PCA front-end.
#pragma once
#include "cat_common.h"

namespace cat {

constexpr int kEigMaxD = 2048;  // a step of the tridiagonalisation keeps 8 x 256 columns in registers at most
constexpr int kEigMaxP = 256;   // vectors (one workgroup makes them orthogonal, one after the other)

// doubles of scratch beside the two D x ld matrices
static inline size_t eig_scratch_doubles(int64_t D) { return 6 * (size_t)D; }

// The p largest eigenvalues (descending) of the symmetric D x D matrix W (both triangles, rows ld apart) and their unit
// eigenvectors, the entry of largest magnitude (the first such) positive: comps p x D float, evals p doubles (nullable).
// W and V (D x ld each) are overwritten.  1 <= p <= min(D, kEigMaxP), D <= kEigMaxD.
cat_status launch_eig_leading(double* W, double* V, int64_t ld, int32_t D, int32_t p, double* scratch, float* comps,
                              double* evals, hipStream_t st);

// Where in V (bytes) a word of 32 bits says afterwards how the columns were done (CAT_PCA_*); 0: nowhere, a launch each.  V comes
// as an identity matrix or with zeros there.
size_t eig_route_at(int64_t ld, int64_t D);

}  // namespace cat
