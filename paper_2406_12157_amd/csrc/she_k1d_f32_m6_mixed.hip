// 1D step kernels of batches whose implicit rods have different cells per lane: state type float.
#include "she_step_1d.hpp"

namespace she {
template hipError_t rods_mixed_t<float, 6>(const Launch1D &);
}  // namespace she
