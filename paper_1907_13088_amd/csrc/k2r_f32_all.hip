// Instantiations of the register-tile passes: float, TE and TM blocks together.
#include "k2r_impl.h"

namespace mx {
namespace reg2d {
template hipError_t launch<float, 3>(const Coef<float> &, int, int, const RegArgs<float> &, hipStream_t);
}  // namespace reg2d
}  // namespace mx
