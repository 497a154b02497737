// Explicit 1D step kernels: state type float, mode 4, numbers drawn ahead.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_t<float, 4, true>(const Launch1D &);
}  // namespace she
