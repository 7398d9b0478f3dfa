// Nearest-centroid assignment (assign.hip), used by encoding and training.
#pragma once

#include "common.h"

namespace dcpq {

// labels[i][j] = nearest centroid of sub-vector j of point i (labels of 1, 2 or 4 bytes), dist NULL or [n][m]
int launch_assign(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int ncent, void *labels,
                  int label_bytes, float *dist, hipStream_t st);

// The same by the filters, sub-vectors of up to 16, 32 and 128 components; dp: dsub rounded up to a multiple of 4
int launch_assign_short(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent, void *labels,
                        int label_bytes, float *dist, hipStream_t st);
int launch_assign_middle(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent, void *labels,
                         int label_bytes, float *dist, hipStream_t st);
int launch_assign_long(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent, void *labels,
                       int label_bytes, float *dist, hipStream_t st);

}  // namespace dcpq
