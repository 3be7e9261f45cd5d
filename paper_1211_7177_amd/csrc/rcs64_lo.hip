// Matrix-core translation kernels, FP64 (rcs_kernel.h): part of the orders.
#include "rcs_kernel.h"

namespace fmb {
RCS_ORDERS64_LO(RCS_INSTANTIATE)
}
