// FP64 interior launches of batches.
#include "kernel_list.h"

namespace opo {
OPO_MID_KERNELS(template, double)
} // namespace opo
