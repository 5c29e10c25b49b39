// FP32 passes of small instances in one launch.
#include "kernel_list.h"

namespace opo {
OPO_TEAM_KERNELS(template, float)
} // namespace opo
