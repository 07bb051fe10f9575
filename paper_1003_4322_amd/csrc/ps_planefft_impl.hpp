// ps_planefft_impl.hpp -- launchers of the plain real transforms along x and of
// whole planes, included by one translation unit per dtype
// (k_planefft_<dtype>.hip).
#pragma once

#include "ps_launch.hpp"
#include "ps_planefft.hpp"
#include "ps_xfft.hpp"

namespace ps {

template <class F>
bool planefft_pick(int N, F&& f) {
  switch (N) {
#define PS_CASE(NN)                            \
  case NN:                                     \
    f(std::integral_constant<int, NN>{});      \
    return true;
    PS_FOR_EACH_PLANEFFT_N(PS_CASE)
#undef PS_CASE
  }
  return false;
}

template <typename T>
bool planefft_fits(int nx, int ny) {
  bool fits = false;
  if (nx == ny) planefft_pick(nx, [&](auto n) { fits = PlaneFftCfg<T, decltype(n)::value>::FITS; });
  return fits;
}

template <typename T>
hipError_t launch_planefft(int N, int dir, PlaneFftArgs<T> a, hipStream_t s) {
  hipError_t r = hipErrorInvalidValue;
  const long per_box = (long)a.nz * a.nf;
  if (per_box <= 0 || a.nb <= 0) return hipSuccess;
  planefft_pick(N, [&](auto n) {
    constexpr int N_ = decltype(n)::value;
    using P = PlaneFftCfg<T, N_>;
    if constexpr (P::FITS)
      r = by_launch(a.nb, per_box, P::NT, [&](int b0, int nb) {
        PlaneFftArgs<T> b = a;
        b.cplx += b0 * a.bs;
        b.real += b0 * per_box * N_ * N_;
        b.nb = nb;
        const dim3 grid((unsigned)(per_box * nb));
        if (dir == INV)
          k_plane_c2r<T, N_><<<grid, dim3(P::NT), 0, s>>>(b);
        else
          k_plane_r2c<T, N_><<<grid, dim3(P::NT), 0, s>>>(b);
        return hipGetLastError();
      });
  });
  return r;
}

template <typename T>
hipError_t launch_xfft(int N, int dir, XFftArgs<T> a, hipStream_t s) {
  const unsigned long total = (unsigned long)a.pairs * a.nf * a.nb;
  if (total == 0) return hipSuccess;
  if (total >= 0xffffffffUL) return hipErrorInvalidValue;  // the kernels number row pairs in 32 bits
  switch (N) {
#define PS_CASE(NN)                                                        \
  case NN: {                                                               \
    using X = XFftCfg<T, NN>;                                              \
    const dim3 grid((unsigned)((total + X::G - 1) / X::G)), block(X::NT);  \
    if (dir == INV)                                                        \
      k_x_c2r<T, NN><<<grid, block, 0, s>>>(a);                            \
    else                                                                   \
      k_x_r2c<T, NN><<<grid, block, 0, s>>>(a);                            \
    return hipGetLastError();                                              \
  }
    PS_FOR_EACH_N(PS_CASE)
#undef PS_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace ps
