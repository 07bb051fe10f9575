// Fused inverse y / product / forward y passes of LDS-resident planes, double.
#include "ps_plane_impl.hpp"

namespace ps {
template bool plane_fits<double>(int, int, bool, bool, bool);
template hipError_t launch_plane<double>(int, bool, bool, bool, bool, PlaneArgs<double>, hipStream_t);
}  // namespace ps
