// Re-packing of a basis into the layouts the plan's kernels read: every layout is a job, and one
// launch runs all of a plan's jobs, each on every n_jobs-th workgroup.  (A training step replaces
// the basis before every forward: four kernels of 4-5 us each, and the copy, became one.)
#pragma once
#include "fwd_common.h"

namespace melt {

enum PackKind { PACK_COPY, PACK_F32, PACK_H16, PACK_PLANES, PACK_DX, PACK_DX_PLANES };
struct PackJob {
    PackKind kind;
    void *out;
    const int *seg, *col;      // segment and first column of each k-group (forward layouts)
    int NG, tiles;             // k-groups (of G rows for PACK_DX_PLANES: per hop segment); row tiles
    int form;                  // PACK_H16: 0 bf16, 1 fp16, 2 / 3 their split low parts; planes: count, + 8 binary16
};
struct PackJobs {
    static constexpr int kMax = 6;
    int n = 0;
    PackJob job[kMax];
    void add(const PackJob &j) { job[n++] = j; }
};
// the layout of the backward's dx (bwd: melt_bwd.hip), added to the jobs
melt_status pack_dx_job(Plan &p, PackJobs &jobs);

}  // namespace melt
