// Kernels of the five passes, double.
#include "se2n_kernels.hpp"

namespace se2n {
SE2N_KERNELS_INSTANTIATE(double)
}  // namespace se2n
