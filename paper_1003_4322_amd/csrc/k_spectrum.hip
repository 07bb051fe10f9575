// Deterministic FP64 shell spectra (energy and enstrophy; MHD energies and
// cross-helicity).
#include <cstring>
#include <map>
#include <mutex>

#include "ps_config.hpp"
#include "ps_launch.hpp"

namespace ps {

// Library-held scratch of the allocation-free spectrum entry point
// (ps_energy_spectrum_static): the per-plane partials of one box at a time.
// Each device the library runs on holds its own copy until the process
// ends.  Host code never passes the array's name to a kernel (on the host it
// is only a stand-in for the symbol): it uses the device address that
// spectrum_scratch() looked up with the device current.
static __device__ __align__(256) double scratch[SPEC_SCRATCH_BYTES / sizeof(double)];

hipError_t spectrum_scratch(int device, double** ptr) {
  static std::mutex mu;
  static std::map<int, double*> addr;  // device -> address of its copy
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find(device);
  if (it != addr.end()) {
    *ptr = it->second;
    return hipSuccess;
  }
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // the current device's copy
  if (e != hipSuccess) return e;
  addr[device] = static_cast<double*>(p);
  *ptr = static_cast<double*>(p);
  return hipSuccess;
}

bool size_supported(int N) {
  switch (N) {
#define PS_CASE(NN) case NN:
    PS_FOR_EACH_N(PS_CASE)
#undef PS_CASE
    return true;
    default:
      return false;
  }
}

int variant_count(const char* kind, int N, bool mhd) {
  (void)mhd;
  if (!has_variants(N)) return 1;
  if (!strcmp(kind, "z_curl")) return NZCURL;
  if (!strcmp(kind, "z_epi")) return NZEPI;
  if (!strcmp(kind, "y") || !strcmp(kind, "z")) return NSTR;
  if (!strcmp(kind, "x_prod")) return NXPROD;
  return 1;
}

// Second stage: per-shell sums over the plane pairs, then the totals over the
// shells, all Neumaier-compensated and in a fixed order.  Q = 2 (energy):
// spec[s] = E(s), totals = [sum E, sum Z, max of pmax]; Q = 3 (MHD):
// spec[q nshell + s] = quantity q of shell s, totals[q] = its sum.
constexpr int FIN_S = 32, FIN_G = 32;  // shells and plane groups of a workgroup

// totals of the per-shell sums part[s Q + q] (one workgroup of FIN_S * FIN_G
// threads): wave q adds the shells of quantity q, a lane's own in order, then
// the lanes' pairs (value, compensation) in a tree; the other waves find the
// maximum.  One barrier: a small box's spectrum is a chain of latencies (NS
// FP64, whole spectra: 32^3 11.1 us, 64^3 15.0; with a tree of all threads and 30
// barriers, the values alone 11.9 and 16.7, the pairs 12.9 and 17.9).
template <int Q>
__device__ void spec_totals(const double* part, const double* pmax, int npm, int nshell, double* totals,
                            double* red) {
  constexpr int NT = FIN_S * FIN_G;
  const int t = threadIdx.x, lane = t % 64, wv = t / 64;
  if (wv < Q) {
    NSum v{0, 0};
#pragma unroll 4
    for (int s = lane; s < nshell; s += 64) nadd(v, part[(long)s * Q + wv]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) nadd(v, NSum{__shfl_down(v.s, d, 64), __shfl_down(v.c, d, 64)});
    if (lane == 0) totals[wv] = v.s + v.c;
  }
  if constexpr (Q == 2) {
    double m = 0;
    if (wv >= Q)
      for (int i = t - Q * 64; i < npm; i += NT - Q * 64) m = fmax(m, pmax[i]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m = fmax(m, __shfl_down(m, d, 64));
    if (lane == 0) red[wv] = m;
    __syncthreads();
    if (t == 0) {
      for (int w = Q; w < NT / 64; ++w) m = fmax(m, red[w]);
      totals[2] = m;
    }
  }
}

// Workgroup b takes the shell blocks b, b + gridDim.x, ...; each thread adds
// the planes g, g + FIN_G, ... of one shell, then the groups' pairs are added in
// order.  The sums go to spec and (every q) to the first plane's place in part,
// which only this workgroup has read; a launch of one workgroup also forms
// the totals.
template <int Q>
__global__ __launch_bounds__(FIN_S* FIN_G) void k_spec_final(double* part, const double* pmax, int npm,
                                                             int nplanes, int nshell, double* spec,
                                                             double* totals) {
  __shared__ NSum sh[Q][FIN_G][FIN_S];
  const int l = threadIdx.x % FIN_S, g = threadIdx.x / FIN_S;
  const int nblk = (nshell + FIN_S - 1) / FIN_S;
  for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int s = b * FIN_S + l;
    NSum e[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) e[q] = NSum{0, 0};
    if (s < nshell)
      for (int p = g; p < nplanes; p += FIN_G)
#pragma unroll
        for (int q = 0; q < Q; ++q) nadd(e[q], part[((long)p * nshell + s) * Q + q]);
#pragma unroll
    for (int q = 0; q < Q; ++q) sh[q][g][l] = e[q];
    __syncthreads();
    if (g < Q && s < nshell) {
      NSum sum{0, 0};
      for (int i = 0; i < min(FIN_G, nplanes); ++i) nadd(sum, sh[g][i][l]);
      const double v = sum.s + sum.c;
      part[(long)s * Q + g] = v;
      if (Q == 3 || g == 0) spec[g * nshell + s] = v;
    }
    __syncthreads();
  }
  if (gridDim.x == 1) spec_totals<Q>(part, pmax, npm, nshell, totals, &sh[0][0][0].s);
}
template <int Q>
__global__ __launch_bounds__(FIN_S* FIN_G) void k_spec_totals(const double* part, const double* pmax, int npm,
                                                              int nshell, double* totals) {
  __shared__ double red[FIN_S * FIN_G / 64];
  spec_totals<Q>(part, pmax, npm, nshell, totals, red);
}

template <typename T>
hipError_t launch_spectrum(SpecArgs<T> a, bool mhd, double* spec, double* totals, hipStream_t s) {
  const int nwin = spec_windows(a.nshell), nplanes = a.nz / 2 + 1, npm = nplanes * nwin;
  // at most SPEC_MAXWIN windows (squares of 2 nshell stay below 2^24), at
  // most SPEC_NF fields
  if (nwin > SPEC_MAXWIN || a.nf > SPEC_NF) return hipErrorInvalidValue;
  const dim3 grid(npm), block(SPEC_ROWS * 64);
  if (mhd)
    k_spec_planes<T, true, 6, true><<<grid, block, 0, s>>>(a);
  else if (a.nf == 3)
    k_spec_planes<T, false, 3, true><<<grid, block, 0, s>>>(a);
  else if (a.nf == 6)
    k_spec_planes<T, false, 6, true><<<grid, block, 0, s>>>(a);
  else
    k_spec_planes<T, false, 6, false><<<grid, block, 0, s>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // few partials: one workgroup adds them and the totals in one launch
  const int nblk = (long)nplanes * a.nshell <= 8192 ? 1 : (a.nshell + FIN_S - 1) / FIN_S;
  const dim3 fb(FIN_S * FIN_G);
  auto finish = [&](auto q) -> hipError_t {
    constexpr int Q = decltype(q)::value;
    k_spec_final<Q><<<dim3(nblk), fb, 0, s>>>(a.part, a.pmax, npm, nplanes, a.nshell, spec, totals);
    hipError_t er = hipGetLastError();
    if (er != hipSuccess || nblk == 1) return er;
    k_spec_totals<Q><<<dim3(1), fb, 0, s>>>(a.part, a.pmax, npm, a.nshell, totals);
    return hipGetLastError();
  };
  return mhd ? finish(std::integral_constant<int, 3>{}) : finish(std::integral_constant<int, 2>{});
}

template hipError_t launch_spectrum<float>(SpecArgs<float>, bool, double*, double*, hipStream_t);
template hipError_t launch_spectrum<double>(SpecArgs<double>, bool, double*, double*, hipStream_t);

}  // namespace ps
