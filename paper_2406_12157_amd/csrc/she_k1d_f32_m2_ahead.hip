// 1D step kernels of batches with implicit rods: state type float.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_t<float, 2, true>(const Launch1D &);
}  // namespace she
