// Instantiations of the register-tile passes: float, Chebyshev form, fixed counts.
#include "k2r_impl.h"

namespace mx {
namespace reg2d {
template hipError_t launch<float, FM_CHEB, false>(const Coef<float> &, int, int, int, const RegArgs<float> &, hipStream_t, int *);
}  // namespace reg2d
}  // namespace mx
