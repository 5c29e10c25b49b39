// FP64 passes of small instances in one launch.
#include "kernel_list.h"

namespace opo {
OPO_TEAM_KERNELS_F64(template)
} // namespace opo
