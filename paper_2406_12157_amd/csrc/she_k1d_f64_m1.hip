// Explicit 1D step kernels: state type double, mode 1, every wave its own numbers.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_t<double, 1, false>(const Launch1D &);
}  // namespace she
