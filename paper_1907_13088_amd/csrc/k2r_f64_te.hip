// Instantiations of the register-tile passes: double, TE block.
#include "k2r_impl.h"

namespace mx {
namespace reg2d {
template hipError_t launch<double, 1>(const Coef<double> &, int, int, const RegArgs<double> &, hipStream_t);
}  // namespace reg2d
}  // namespace mx
