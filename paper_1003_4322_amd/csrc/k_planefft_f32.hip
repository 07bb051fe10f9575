// Plain real transforms: x passes, and whole LDS-resident planes, float.
#include "ps_planefft_impl.hpp"

namespace ps {
template bool planefft_fits<float>(int, int);
template hipError_t launch_planefft<float>(int, int, PlaneFftArgs<float>, hipStream_t);
template hipError_t launch_xfft<float>(int, int, XFftArgs<float>, hipStream_t);
}  // namespace ps
