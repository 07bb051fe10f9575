// The fused product pass along x, double.
#include "ps_launch_impl.hpp"

namespace ps {
template bool mhd_supported<double>(int);
template hipError_t launch_x_prod<double>(int, bool, bool, int, XArgs<double>, hipStream_t);
}  // namespace ps
