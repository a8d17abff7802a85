// Middle pass of the pair path, double.
#include "se2n_pair_mid.hpp"

namespace se2n {
SE2N_PAIR_MID_INSTANTIATE(double)
}  // namespace se2n
