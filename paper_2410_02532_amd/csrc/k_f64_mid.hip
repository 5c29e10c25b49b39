// FP64 interior launches of batches.
#include "kernel_list.h"

namespace opo {
OPO_MID_KERNELS_F64(template)
} // namespace opo
