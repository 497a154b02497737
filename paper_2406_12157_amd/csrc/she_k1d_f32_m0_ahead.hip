// Explicit 1D step kernels: state type float, mode 0, numbers drawn ahead.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_t<float, 0, true>(const Launch1D &);
}  // namespace she
