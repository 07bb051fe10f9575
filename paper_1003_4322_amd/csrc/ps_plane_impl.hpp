// ps_plane_impl.hpp -- launcher of k_plane, included by one translation unit
// per dtype (k_plane_<dtype>.hip).
#pragma once

#include "ps_config.hpp"
#include "ps_launch.hpp"
#include "ps_plane.hpp"

namespace ps {

// f(integral N, MHD, ELS, PR) for the runtime values, where N has a plane
// schedule; false otherwise
template <class F>
bool plane_pick(int N, bool mhd, bool els, bool pr, F&& f) {
  using t_ = std::true_type;
  using f_ = std::false_type;
  auto forms = [&](auto n) {
    auto with = [&](auto m, auto e) {
      if (pr)
        f(n, m, e, t_{});
      else
        f(n, m, e, f_{});
    };
    if (mhd && els) with(t_{}, t_{});
    if (mhd && !els) with(t_{}, f_{});
    if (!mhd && els) with(f_{}, t_{});
    if (!mhd && !els) with(f_{}, f_{});
  };
  switch (N) {
#define PS_CASE(NN)                               \
  case NN:                                        \
    forms(std::integral_constant<int, NN>{});     \
    return true;
    PS_FOR_EACH_PLANE_N(PS_CASE)
#undef PS_CASE
  }
  return false;
}

// Which kernel takes a form's planes: 2 k_plane_field, 1 k_plane, 0 neither.
// k_plane_field wins wherever its plane fits in LDS (three passes against it:
// MHD 32^3 FP64 114 to 102 us a step, 300 boxes of NS 16^3 FP32 285 to 121, 16
// boxes of MHD 64^3 FP32 pruned 385 to 267), except where NS planes in the
// divergence form let two workgroups of k_plane share a CU and there are more
// planes than CUs (48 boxes of 64^3: 467 with k_plane_field, 402 with k_plane;
// one box 49 against 55).  NS planes too large for it (64^2 in FP64, pruned)
// fit k_plane (16 boxes 350 to 261); MHD planes that fit k_plane only are no
// faster than the three passes (MHD 48^3 FP64 pruned 70 to 83).
template <typename T, int N, bool MHD, bool ELS, bool PR>
constexpr int plane_kernel(bool many) {
  using P = PlaneCfg<T, N, MHD, ELS, PR>;
  using PF = PlaneFieldCfg<T, N, MHD, ELS, PR>;
  if (!MHD && P::FITS) {
    if (!PF::FITS) return 1;
    if (many && P::FIN == 3 && P::LDS <= 81920 && PF::LDS > 81920) return 1;
  }
  return PF::FITS ? 2 : 0;
}

template <typename T>
bool plane_fits(int nx, int ny, bool mhd, bool els, bool prune) {
  bool fits = false;
  if (nx == ny)
    plane_pick(nx, mhd, els, prune, [&](auto n, auto m, auto e, auto p) {
      fits = plane_kernel<T, decltype(n)::value, decltype(m)::value, decltype(e)::value, decltype(p)::value>(
                 false) != 0;
    });
  return fits;
}

template <typename T>
hipError_t launch_plane(int N, bool mhd, bool els, bool prune, bool many, PlaneArgs<T> a, hipStream_t s) {
  hipError_t r = hipErrorInvalidValue;
  if (a.g.nx != N || a.g.ny != N) return r;
  if (a.nz <= 0 || a.nb <= 0) return hipSuccess;
  plane_pick(N, mhd, els, prune, [&](auto n, auto m, auto e, auto p) {
    constexpr int N_ = decltype(n)::value;
    constexpr bool M_ = decltype(m)::value, E_ = decltype(e)::value, P_ = decltype(p)::value;
    const int k = plane_kernel<T, N_, M_, E_, P_>(many);
    auto go = [&](auto kernel, int nt) {
      r = by_launch(a.nb, a.nz, nt, [&](int b0, int nb) {
        PlaneArgs<T> b = a;
        b.work += b0 * a.bs;
        b.nb = nb;
        kernel<<<dim3((unsigned)((long)a.nz * nb)), dim3(nt), 0, s>>>(b);
        return hipGetLastError();
      });
    };
    if constexpr (plane_kernel<T, N_, M_, E_, P_>(true) == 1) {
      if (k == 1) go(k_plane<T, N_, M_, E_, P_>, PlaneCfg<T, N_, M_, E_, P_>::NW * 64);
    }
    if constexpr (plane_kernel<T, N_, M_, E_, P_>(false) == 2) {
      if (k == 2) go(k_plane_field<T, N_, M_, E_, P_>, PlaneFieldCfg<T, N_, M_, E_, P_>::NW * 64);
    }
  });
  return r;
}

}  // namespace ps
