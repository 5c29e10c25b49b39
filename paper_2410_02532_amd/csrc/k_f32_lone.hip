// FP32 interior steps of handles too small to fill the chip.
#include "kernel_list.h"

namespace opo {
OPO_LONE_KERNELS(template, float)
} // namespace opo
