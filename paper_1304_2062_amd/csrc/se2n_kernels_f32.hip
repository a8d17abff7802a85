// Kernels of the five passes, float.
#include "se2n_kernels.hpp"

namespace se2n {
SE2N_KERNELS_INSTANTIATE(float)
}  // namespace se2n
