// Fused forward z pass + dealias / projection / induction / RK2 epilogue, double.
#include "ps_launch_impl.hpp"

namespace ps {
template hipError_t launch_z_epi<double>(int, bool, bool, int, ZEpiArgs<double>, const DiskTiles*, hipStream_t);
template unsigned z_epi_widths<double>(int);
}  // namespace ps
