// 1D step kernels of batches with implicit rods, no material coefficients: state type double.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_t<double, 6, true>(const Launch1D &);
}  // namespace she
