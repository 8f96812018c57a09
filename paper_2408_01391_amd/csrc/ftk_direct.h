// Unprotected assignment in one launch, every distance in double (see ftk_direct.hip).
#pragma once

#include "ftk_internal.h"

namespace ftk {

struct DirectPlan {
    int lanes;    // that share the features of a row
    int kg;       // centroids of a lane at a time
    int tc_log2;  // groups of lanes with different centroids of the same points
};
bool direct_pays(ftk_dtype dtype, int64_t N, int D, int K);
// the cut: distances depend on it in the last place (fp64), so parts of a problem take that of the whole
DirectPlan cut_direct(ftk_dtype dtype, int64_t N, int D, int K);
ftk_status launch_direct_assign(const AssignCall &c, const DirectPlan &p, hipStream_t st);

}  // namespace ftk
