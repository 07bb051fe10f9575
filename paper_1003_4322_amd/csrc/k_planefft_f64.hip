// Plain real transforms: x passes, and whole LDS-resident planes, double.
#include "ps_planefft_impl.hpp"

namespace ps {
template bool planefft_fits<double>(int, int);
template hipError_t launch_planefft<double>(int, int, PlaneFftArgs<double>, hipStream_t);
template hipError_t launch_xfft<double>(int, int, XFftArgs<double>, hipStream_t);
}  // namespace ps
