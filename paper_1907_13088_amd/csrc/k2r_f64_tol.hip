// Instantiations of the register-tile passes: double, tolerance solves, standard and delta forms.
#include "k2r_impl.h"

namespace mx {
namespace reg2d {
template hipError_t launch<double, FM_STD, true>(const Coef<double> &, int, int, int, const RegArgs<double> &, hipStream_t, int *);
template hipError_t launch<double, FM_DELTA, true>(const Coef<double> &, int, int, int, const RegArgs<double> &, hipStream_t, int *);
}  // namespace reg2d
}  // namespace mx
