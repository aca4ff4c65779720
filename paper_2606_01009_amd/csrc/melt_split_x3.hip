// The split precisions (BF16X3, FP16X3) on hi and lo planes.
#include "melt_split.h"

namespace melt {
melt_status launch_melt_split_x3(Plan &p, const FwdTask &t) {
    return prec_f16(p) ? launch_split_forward<Split2F16>(p, t) : launch_split_forward<Split2BF16>(p, t);
}
}  // namespace melt
