// Quad solver kernels: see quad_kernel.hpp.
#include "quad_launch.hpp"

namespace mcc {
MCC_QUAD_DEFINE(2, 32, 1, 16, 1)
MCC_QUAD_DEFINE(2, 32, 2, 16, 1)
}  // namespace mcc
