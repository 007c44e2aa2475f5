// Instantiations of the register-tile passes: double, tolerance solves, Chebyshev form.
#include "k2r_impl.h"

namespace mx {
namespace reg2d {
template hipError_t launch<double, FM_CHEB, true>(const Coef<double> &, int, int, int, const RegArgs<double> &, hipStream_t, int *);
}  // namespace reg2d
}  // namespace mx
