// Field-parallel z passes of small boxes, double.
#include "ps_zfield_impl.hpp"

namespace ps {
template hipError_t launch_z_curl_field<double>(int, bool, bool, ZCurlArgs<double>, const DiskTiles*, hipStream_t);
template hipError_t launch_z_epi_field<double>(int, bool, bool, ZEpiArgs<double>, const DiskTiles*, hipStream_t);
}  // namespace ps
