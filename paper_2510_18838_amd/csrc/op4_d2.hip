// 2-D operator-emission kernels with four lanes per target (see kernels.h).
#include "kernels.h"

namespace pcms {
PCMS_DEFINE_DIM_OPERATOR(2, kQuad)
}  // namespace pcms
