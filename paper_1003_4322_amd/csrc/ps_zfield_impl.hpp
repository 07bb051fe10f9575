// ps_zfield_impl.hpp -- launchers of the field-parallel z passes, included by
// one translation unit per dtype (k_zfield_<dtype>.hip).
#pragma once

#include "ps_config.hpp"
#include "ps_launch.hpp"
#include "ps_zfield.hpp"

namespace ps {

template <typename T, int N>
struct ZFieldCfg {
  static constexpr int TQ = LenCfg<N>::TQ;
  // columns per tile of the epilogue: 8, or 16 (128-byte row pieces) where
  // FP32 columns of 128 points fill the workgroup anyway (MHD 128^3 FP32 step,
  // pruned: 201 us with 8, 189 with 16; at 96 points 16 is the slower)
  static constexpr int TXC = 8, TXE = sizeof(T) == 4 && N >= 128 ? 16 : 8;
  // field groups of the epilogue: as many as 1024 threads hold
  static constexpr int ng(int np) {
    const int most = 1024 / (TXE * TQ);
    return cdiv(np, cdiv(np, most));
  }
  static constexpr int epi_lds(int np) { return (np * (pad8(N - 1) + 1) * TXE + N) * 2 * (int)sizeof(T); }
};

#define PS_FOR_EACH_ZFIELD_N(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128)

// f(integral N, MHD, ELS) for the runtime values
template <class F>
hipError_t zfield_pick(int N, bool mhd, bool els, F&& f) {
  using t_ = std::true_type;
  using f_ = std::false_type;
  auto forms = [&](auto n) {
    if (mhd && els) return f(n, t_{}, t_{});
    if (mhd) return f(n, t_{}, f_{});
    if (els) return f(n, f_{}, t_{});
    return f(n, f_{}, f_{});
  };
  switch (N) {
#define PS_CASE(NN) \
  case NN:          \
    return forms(std::integral_constant<int, NN>{});
    PS_FOR_EACH_ZFIELD_N(PS_CASE)
#undef PS_CASE
  }
  return hipErrorInvalidValue;
}

// Tiles of a field-parallel launch: a launch large enough to be spread over
// the XCDs tile range by tile range (from remap on) takes the pruned tiles from the
// disk list, so that no XCD's range is empty; a small one finds them from its
// block index, which spares it a dependent load.
template <int TX>
long zfield_grid(unsigned remap, int ny, int ntile, int nb, int fields, bool pruned, const DiskTiles* dt,
                 const int*& tiles, int& ntl) {
  const long all = (long)ntile * ny * nb * fields;
  if (all >= (long)remap) return z_grid<TX>(ny, ntile, nb, pruned, dt, tiles, ntl) * fields;
  tiles = nullptr;
  ntl = 0;
  return all;
}

template <typename T>
hipError_t launch_z_curl_field(int N, bool mhd, bool els, ZCurlArgs<T> a, const DiskTiles* dt, hipStream_t s) {
  if (a.g.nz != N) return hipErrorInvalidValue;
  return zfield_pick(N, mhd, els, [&](auto n, auto m, auto e) -> hipError_t {
    constexpr int N_ = decltype(n)::value;
    constexpr bool M_ = decltype(m)::value, E_ = decltype(e)::value;
    using Z = ZFieldCfg<T, N_>;
    if constexpr (N_ > ZCURL_FIELD_MAXN) {
      return hipErrorInvalidValue;
    } else {
      a.ntile = cdiv(a.g.nx / 2 + 1, Z::TXC);
      const long grid =
          zfield_grid<Z::TXC>(ZREMAP_CURL, a.g.ny, a.ntile, a.nb, xprod_fin(M_, E_), a.prune != 0, dt, a.tiles, a.ntl);
      k_z_curl_field<T, N_, Z::TQ, Z::TXC, typename LenCfg<N_>::RL, M_, E_>
          <<<dim3((unsigned)grid), dim3(Z::TXC * Z::TQ), 0, s>>>(a);
      return hipGetLastError();
    }
  });
}

template <typename T>
hipError_t launch_z_epi_field(int N, bool mhd, bool els, ZEpiArgs<T> a, const DiskTiles* dt, hipStream_t s) {
  if (a.g.nz != N) return hipErrorInvalidValue;
  return zfield_pick(N, mhd, els, [&](auto n, auto m, auto e) -> hipError_t {
    constexpr int N_ = decltype(n)::value;
    constexpr bool M_ = decltype(m)::value, E_ = decltype(e)::value;
    using Z = ZFieldCfg<T, N_>;
    constexpr int NP = xprod_fout(M_, E_), NG = Z::ng(NP);
    static_assert(Z::epi_lds(NP) <= 163840, "the tile of every product fits in LDS");
    a.ntile = cdiv(a.g.nx / 2 + 1, Z::TXE);
    const long grid = zfield_grid<Z::TXE>(ZREMAP_EPI, a.g.ny, a.ntile, a.nb, 1, a.prune && a.mode != 0, dt, a.tiles, a.ntl);
    k_z_epi_field<T, N_, Z::TQ, Z::TXE, typename LenCfg<N_>::RL, M_, E_, NG>
        <<<dim3((unsigned)grid), dim3(NG * Z::TXE * Z::TQ), 0, s>>>(a);
    return hipGetLastError();
  });
}

}  // namespace ps
