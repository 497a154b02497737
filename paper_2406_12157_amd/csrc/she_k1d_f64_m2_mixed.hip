// 1D step kernels of batches whose implicit rods have different cells per lane, with material coefficients: state type double.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_mixed_t<double, 2>(const Launch1D &);
}  // namespace she
