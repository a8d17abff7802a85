// Middle pass of the pair path, float.
#include "se2n_pair_mid.hpp"

namespace se2n {
SE2N_PAIR_MID_INSTANTIATE(float)
}  // namespace se2n
