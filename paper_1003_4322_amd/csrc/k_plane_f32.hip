// Fused inverse y / product / forward y passes of LDS-resident planes, float.
#include "ps_plane_impl.hpp"

namespace ps {
template bool plane_fits<float>(int, int, bool, bool, bool);
template hipError_t launch_plane<float>(int, bool, bool, bool, bool, PlaneArgs<float>, hipStream_t);
}  // namespace ps
