// Small unprotected problems: assignment and Lloyd iteration in one launch each (see ftk_small.hip).
#pragma once

#include "ftk_internal.h"

namespace ftk {

bool small_assign_pays(ftk_dtype dtype, int64_t N, int D, int K);
// what it can take at all
bool small_assign_fits(ftk_dtype dtype, int64_t N, int D, int K);
ftk_status launch_small_assign(const AssignCall &c, hipStream_t st);

bool small_fit_pays(ftk_dtype dtype, int64_t N, int D, int K);
size_t small_fit_bytes(int D, int K);  // 0: never
// iters >= 1; C_first: the initial centroids (may be C_cur or C_out); C_cur is used up; partials: 1024 doubles;
// absmax is found on the way
ftk_status launch_small_fit(ftk_dtype dtype, const void *X, int64_t N, int D, int K, int iters, const void *C_first, void *C_cur,
                            void *C_out, int32_t *labels, int32_t *counts, double *absmax, double *inertia, double *partials,
                            void *scratch, hipStream_t st);

}  // namespace ftk
