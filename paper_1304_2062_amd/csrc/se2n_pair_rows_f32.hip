// Row kernels of the pair path, float.
#include "se2n_pair_rows.hpp"

namespace se2n {
SE2N_PAIR_ROWS_INSTANTIATE(float)
}  // namespace se2n
