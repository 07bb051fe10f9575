// The fused product pass along x, float.
#include "ps_launch_impl.hpp"

namespace ps {
template bool mhd_supported<float>(int);
template hipError_t launch_x_prod<float>(int, bool, bool, int, XArgs<float>, hipStream_t);
}  // namespace ps
