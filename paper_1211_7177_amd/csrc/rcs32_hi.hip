// Matrix-core translation kernels, FP32 (rcs_kernel.h): part of the orders.
#include "rcs_kernel.h"

namespace fmb {
RCS_ORDERS32_HI(RCS_INSTANTIATE)
}
