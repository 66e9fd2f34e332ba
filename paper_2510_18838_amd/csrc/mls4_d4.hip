// 4-D neighbour-list and transfer kernels with four lanes per target (see kernels.h).
#include "kernels.h"

namespace pcms {
PCMS_DEFINE_DIM_KERNELS(4, kQuad)
}  // namespace pcms
