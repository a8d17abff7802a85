// Row kernels of the pair path, double.
#include "se2n_pair_rows.hpp"

namespace se2n {
SE2N_PAIR_ROWS_INSTANTIATE(double)
}  // namespace se2n
