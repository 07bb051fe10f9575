// ps_launch.hpp -- host-side launchers of the gfx950 kernels (internal).
// Each launcher picks the compiled configuration for the length N of the axis
// its pass transforms (z passes: nz, y passes: ny, x passes: nx) and the
// requested variant, fills in the tile counts and enqueues one kernel.
#pragma once

#include <hip/hip_runtime.h>

#include "ps_kernels.hpp"
#include "ps_plane.hpp"
#include "ps_planefft.hpp"
#include "ps_xfft.hpp"
#include "ps_spectrum.hpp"

namespace ps {

bool size_supported(int N);
template <typename T>
bool mhd_supported(int N);

// number of variants of a pass kind at size N ("y", "z", "z_curl", "z_epi", "x_prod")
int variant_count(const char* kind, int N, bool mhd);

template <typename T>
hipError_t launch_strided(int N, int dir, int var, StridedArgs<T> a, hipStream_t s);
// Tiles of a z pass whose first column meets the dealiasing disk
// Grid::disk(kx, ky), one device list per tile width (entries
// tile | ky << 16, ky-major).
struct DiskTiles {
  static constexpr int MAXTX = 16;
  const int* list[MAXTX + 1] = {};
  int count[MAXTX + 1] = {};
};
// grid of a z pass: every tile, or only those in the disk list
template <int TX>
long z_grid(int ny, int ntile, int nb, bool listed, const DiskTiles* dt, const int*& tiles, int& ntl) {
  static_assert(TX <= DiskTiles::MAXTX, "disk tile lists cover widths up to 16");
  if (listed && dt && dt->list[TX]) {
    tiles = dt->list[TX];
    ntl = dt->count[TX];
    return (long)ntl * nb;
  }
  tiles = nullptr;
  ntl = 0;
  return (long)ntile * ny * nb;
}

// f(b0, n) for the boxes [0, nb) in runs [b0, b0 + n) whose launches, of
// per_box workgroups of nt threads a box, stay below the 2^32 threads a launch
// may have (one run but for ensembles of millions of small boxes)
template <class F>
hipError_t by_launch(int nb, long per_box, int nt, F&& f) {
  const long most = 0xffffffffL / (per_box * nt);
  for (long b0 = 0; b0 < nb; b0 += most) {
    const hipError_t e = f((int)b0, (int)(nb - b0 < most ? nb - b0 : most));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// tile widths a length's z-pass variants use (bit w: width w)
template <typename T>
unsigned z_curl_widths(int N);
template <typename T>
unsigned z_epi_widths(int N);

// els: MHD in the Elsasser (divergence) form -- z_curl transforms z+- without
// a curl, x_prod forms the products z+_i z-_j (less z+_2 z-_2 on the diagonal,
// eight fields), z_epi takes their divergence
template <typename T>
hipError_t launch_z_curl(int N, bool mhd, bool els, int var, ZCurlArgs<T> a, const DiskTiles* dt,
                         hipStream_t s);
template <typename T>
hipError_t launch_z_epi(int N, bool mhd, bool els, int var, ZEpiArgs<T> a, const DiskTiles* dt,
                        hipStream_t s);
template <typename T>
hipError_t launch_x_prod(int N, bool mhd, bool els, int var, XArgs<T> a, hipStream_t s);
// Inverse y pass, products and forward y pass of whole z-planes in one kernel:
// plane_fits says whether a (kx, ky) plane of the form's fields fits in LDS;
// many: more planes in the class than the chip has CUs.
template <typename T>
bool plane_fits(int nx, int ny, bool mhd, bool els, bool prune);
template <typename T>
hipError_t launch_plane(int N, bool mhd, bool els, bool prune, bool many, PlaneArgs<T> a, hipStream_t s);
// z passes with the fields of a column tile side by side, for launches whose
// column tiles alone leave the chip idle; columns: those the pass transforms
// in all boxes of the class (launch times, us, one field after another against
// side by side).  The inverse pass gains up to 96 points: for the divergence
// forms up to 32768 columns (MHD 16 points FP32, 12312 columns 21 to 20, 24768
// 26 to 27); for the rotational forms, whose fields read their inputs two to
// four times, as long as these come from the caches: FP64 up to 32768 (512 x 384
// x 8 MHD 896 to 313; NS from 64 points on to 16384: 64 points, 12800 columns 54 to
// 49, 25344 119 to 137), FP32 up to 5120 (NS 64 points 4800 columns 25 to 23, 9600
// 26 to 31; MHD 25344 132 to 238), further where few threads share a column (48
// points, MHD 24: 14976 columns 93 to 73) and at 96 (NS 24768 columns 87 to 79, MHD
// 14112 160 to 168).
constexpr int ZCURL_FIELD_MAXN = 96;
inline bool z_curl_by_field(int nz, long columns, bool f32, bool mhd, bool els) {
  if (nz > ZCURL_FIELD_MAXN) return false;
  if (els) return columns <= 32768;
  if (!f32) return columns <= (nz >= 64 && !mhd ? 16384 : 32768);
  if (nz == 48 || (nz == 24 && mhd) || (nz == 96 && !mhd)) return columns <= 32768;
  return columns <= (nz == 96 ? 16384 : 5120);
}
// the epilogue gains at every count up to 64 points (MHD 64^3 103 to 79; 48
// boxes of 64^3 646 to 611) and up to 128 points while the columns are few
// (steps: NS 96^3 122 to 104, 1608 columns; NS 96^3 FP64, 4704 columns, 198 to 213;
// launches at 128 points: FP32 2903 columns 32 to 25, 3264 40 to 47; FP64 1600 35 to
// 33, 2496 38 to 48).
// (48 boxes of NS 64^3: k_z_epi_tile ties with it, 365 us a step; 200 of 32^3:
// 201 against 194.)
inline bool z_epi_by_field(int nz, long columns, bool f32) {
  return nz <= 64 || (nz <= 128 && columns <= (nz == 96 ? 4096 : f32 ? 3000 : 1600));
}
template <typename T>
hipError_t launch_z_curl_field(int N, bool mhd, bool els, ZCurlArgs<T> a, const DiskTiles* dt, hipStream_t s);
template <typename T>
hipError_t launch_z_epi_field(int N, bool mhd, bool els, ZEpiArgs<T> a, const DiskTiles* dt, hipStream_t s);
// x and y passes of the plain transforms (dir FWD: r2c, INV: c2r) in one kernel,
// where one field's plane fits in LDS
template <typename T>
bool planefft_fits(int nx, int ny);
template <typename T>
hipError_t launch_planefft(int N, int dir, PlaneFftArgs<T> a, hipStream_t s);
// the x pass alone
template <typename T>
hipError_t launch_xfft(int N, int dir, XFftArgs<T> a, hipStream_t s);
// Bytes of the library-held device scratch of ps_energy_spectrum_static:
// the partials of one box, nz * nshell * 2 + nz doubles (14.6 MB at
// 1024^3, the largest supported grid).
constexpr size_t SPEC_SCRATCH_BYTES = size_t(16) << 20;
// Device address of the current device's copy of that scratch (looked up
// once per device; call with `device` current).
hipError_t spectrum_scratch(int device, double** ptr);

// mhd: Eu(s), Eb(s), Hc(s) of an Elsasser state instead of E(s) (and Z, maxdiv)
template <typename T>
hipError_t launch_spectrum(SpecArgs<T> a, bool mhd, double* spec, double* totals, hipStream_t s);

}  // namespace ps
