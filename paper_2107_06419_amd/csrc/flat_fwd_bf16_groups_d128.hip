// Key-group forms of the fused bf16 kernel, d = 96, 128 and 256: 32 or 64 rows over four groups, 64 or 128 rows over two
// (chosen by predicted time in flat_plan.hip).
#include "flat_fwd_bf16_kernel.hpp"

namespace flat {

FLAT_INSTANTIATE_BF16_GROUPS(96, 1, 4, 2, 128, 4)
FLAT_INSTANTIATE_BF16_GROUPS(96, 1, 8, 2, 128, 4)
FLAT_INSTANTIATE_BF16_GROUPS(96, 1, 4, 2, 64, 2)
FLAT_INSTANTIATE_BF16_GROUPS(96, 1, 8, 2, 64, 2)
FLAT_INSTANTIATE_BF16_GROUPS(128, 1, 4, 2, 128, 4)
FLAT_INSTANTIATE_BF16_GROUPS(128, 1, 8, 2, 128, 4)
FLAT_INSTANTIATE_BF16_GROUPS(128, 1, 4, 2, 64, 2)
FLAT_INSTANTIATE_BF16_GROUPS(128, 1, 8, 2, 64, 2)
FLAT_INSTANTIATE_BF16_GROUPS(256, 1, 4, 2, 64, 2)

}  // namespace flat
