// Explicit 1D step kernels: state type double, mode 4, every wave its own numbers.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_t<double, 4, false>(const Launch1D &);
}  // namespace she
