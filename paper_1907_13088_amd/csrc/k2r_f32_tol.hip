// Instantiations of the register-tile passes: float, tolerance solves, standard and delta forms.
#include "k2r_impl.h"

namespace mx {
namespace reg2d {
template hipError_t launch<float, FM_STD, true>(const Coef<float> &, int, int, int, const RegArgs<float> &, hipStream_t, int *);
template hipError_t launch<float, FM_DELTA, true>(const Coef<float> &, int, int, int, const RegArgs<float> &, hipStream_t, int *);
}  // namespace reg2d
}  // namespace mx
