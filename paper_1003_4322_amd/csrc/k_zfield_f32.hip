// Field-parallel z passes of small boxes, float.
#include "ps_zfield_impl.hpp"

namespace ps {
template hipError_t launch_z_curl_field<float>(int, bool, bool, ZCurlArgs<float>, const DiskTiles*, hipStream_t);
template hipError_t launch_z_epi_field<float>(int, bool, bool, ZEpiArgs<float>, const DiskTiles*, hipStream_t);
}  // namespace ps
