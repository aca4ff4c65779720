// The FP32 projection on three bfloat16 planes per operand.
#include "melt_split.h"

namespace melt {
melt_status launch_melt_split_f32(Plan &p, const FwdTask &t) { return launch_split_forward<Split3BF16>(p, t); }
}  // namespace melt
