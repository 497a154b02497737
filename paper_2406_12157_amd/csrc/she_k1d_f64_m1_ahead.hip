// Explicit 1D step kernels: state type double, mode 1, numbers drawn ahead.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_t<double, 1, true>(const Launch1D &);
}  // namespace she
