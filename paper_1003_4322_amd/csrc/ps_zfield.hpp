// ps_zfield.hpp -- z passes that transform the fields of a column tile side by
// side instead of one after another.
#pragma once

#include "ps_config.hpp"
#include "ps_kernels.hpp"

namespace ps {

// Workgroups from which neighbouring tiles go to one XCD (they share cache
// lines); fewer are spread over all XCDs.  An inverse pass has several fields'
// workgroups to a tile, an epilogue one (from 2048 -> from 512, us: MHD 48 x 384 x
// 64 FP32, 1536 workgroups, 107 -> 53; three boxes of NS 96^3 in the divergence
// form 117 -> 60; NS 192 x 192 x 128 129 -> 98).
constexpr unsigned ZREMAP_CURL = 2048, ZREMAP_EPI = 512;

// Inverse z pass + curl (k_z_curl's outputs), one output field per workgroup:
// the field's inputs are read straight from the state (a base field's one or,
// MHD, two; a curl's two or four), so every field of every tile is in flight
// at once.  Bound by latency (one memory round trip and one transform); with
// one field after another, MHD 32^3 FP64 spent 17 us here, now 8.6 (a third of
// the step's time at both ends).
template <typename T, int L, int TQ, int TX, class RL, bool MHD, bool ELS>
__global__ __launch_bounds__(TX* TQ) void k_z_curl_field(ZCurlArgs<T> a) {
  using E = Stockham<T, L, TQ, INV, RL>;
  using CT = ColTile<T, L, TX, 0>;
  constexpr int NT = TX * TQ;
  constexpr int NPHYS = ELS ? (MHD ? 6 : 3) : (MHD ? 12 : 6);
  __shared__ C2<T> smem[CT::ROWS * TX + L];
  C2<T>* const tws = smem + CT::ROWS * TX;
  const int tid = threadIdx.x, c = tid % TX, q = tid / TX;
  const int blk = gridDim.x >= ZREMAP_CURL ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
  const int fo = blk % NPHYS;
  const Grid& g = a.g;
  const ZTile zt = z_tile(blk / NPHYS, a.ntile, g.ny, a.tiles, a.ntl);
  const int col = zt.tile * TX + c, ky = zt.ky, kyw = wav(ky, g.ny);
  if (a.prune && !g.disk(zt.tile * TX, kyw)) return;  // tile outside the disk
  const bool ok = col < g.nx / 2 + 1 && (!a.prune || g.disk(col, kyw));
  const long in_es = (long)g.ny * a.in_pitch, out_es = (long)g.ny * a.out_pitch;
  const C2<T>* in = a.in + zt.box * a.in_bs + ky * a.in_pitch + col;
  C2<T>* out = a.out + zt.box * a.out_bs + fo * a.out_fs + ky * a.out_pitch + col;
  const int kperp2 = g.perp(col, kyw);
  TwFill<T, L, NT, RL> fill;
  fill.load(a.tw, tid);
  // base fields u (MHD: (z+ + z-)/2) and b ((z+ - z-)/2, sign -1); curl
  // component comp = ka g(ca) - kb g(cb), with kz in one of ka, kb.  All loads
  // come before any arithmetic on them.
  const int grp = fo / 3, comp = fo % 3;
  const bool curl = !ELS && (grp & 1) != 0;
  const T sign = MHD && grp >= 2 ? T(-1) : T(1);
  const int ca = comp == 0 ? 2 : comp == 1 ? 0 : 1, cb = comp == 0 ? 1 : comp == 1 ? 2 : 0;
  constexpr int NL = ELS ? 1 : MHD ? 4 : 2;  // loads a value may need
  C2<T> ld[NL][E::FIRST_SLOTS];
  auto load = [&](C2<T>(&dst)[E::FIRST_SLOTS], int f) {
#pragma unroll
    for (int s = 0; s < E::FIRST_SLOTS; ++s) {
      const int kzi = E::first_index(q, s);
      const bool live = E::first_valid(q, s) && ok && (!a.prune || g.keep_p(kperp2, wav(kzi, L)));
      dst[s] = live ? in[f * a.in_fs + (long)kzi * in_es] : zero2<T>();
    }
  };
  const int fa = ELS ? fo : curl ? ca : comp;
  load(ld[0], fa);
  if constexpr (!ELS) {
    if constexpr (MHD) load(ld[2], 3 + fa);
    if (curl) {
      load(ld[1], cb);
      if constexpr (MHD) load(ld[3], 3 + cb);
    }
  }
  fill.store(tws, tid);
  const T kx = a.sx * (T)dwavx(col, g.nx), kyd = a.sy * (T)dwav(ky, g.ny);
  const T kA = comp == 0 ? kyd : kx, kB = comp == 1 ? kx : kyd;
  C2<T> v[E::SLOTS];
  // the first stage's barrier orders the twiddles before their first use
  E::template run_tw<typename CT::Lay>(v, smem + c, TX, q, TwStaged<T>{tws}, [&](int s, int kzi) -> C2<T> {
    if constexpr (ELS) {
      return ld[0][s];
    } else {
      C2<T> u = ld[0][s];
      if constexpr (MHD) u = T(0.5) * (u + sign * ld[2][s]);
      if (!curl) return u;
      C2<T> w = ld[1][s];
      if constexpr (MHD) w = T(0.5) * (w + sign * ld[3][s]);
      const T kz = a.sz * (T)dwav(kzi, L);
      return mul_i((comp == 1 ? kz : kA) * u - (comp == 0 ? kz : kB) * w);
    }
  });
#pragma unroll
  for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
    if (ok && E::last_valid(q, s)) out[E::last_index(q, s) * out_es] = v[s];
}

// Forward z pass + epilogue (k_z_epi's outputs and modes), the NP product
// fields of a column tile side by side: NG groups of TX x TQ threads, group
// grp transforming fields grp, grp + NG, ... in LDS tiles of their own.  The
// transforms end in LDS, and each thread then finishes the modes (c, kz) with
// kz = tid / TX, + NT / TX, ...: it gathers the NP values of a mode from LDS and
// updates the state, whose values it has loaded before the transforms.  All of
// a tile's loads (products, state, twiddles) are in flight together, where one
// field after another waits for memory NP times: MHD 64^3 FP32 (8 products, 72
// busy tiles) 19.5 -> 7.3 us, NS 32^3 FP64 10.0 -> 5.6 us.
template <typename T, int L, int TQ, int TX, class RL, bool MHD, bool ELS, int NG>
__global__ __launch_bounds__(NG* TX* TQ) void k_z_epi_field(ZEpiArgs<T> a) {
  using E = Stockham<T, L, TQ, FWD, RL>;
  constexpr int NF = MHD ? 6 : 3;                             // state fields
  constexpr int NP = xprod_fout(MHD, ELS), NR = cdiv(NP, NG);  // products, rounds
  constexpr int NT = NG * TX * TQ, NO = E::LAST_NB * E::RL_;
  constexpr int PTS = cdiv(L * TX, NT);
  using Lay = LayColPad8;
  constexpr int ROWS = pad8(L - 1) + 1, TILE = ROWS * TX;
  __shared__ C2<T> smem[NP * TILE + L];
  C2<T>* const tws = smem + NP * TILE;
  const int tid = threadIdx.x, c = tid % TX, q = tid / TX % TQ, grp = tid / (TX * TQ);
  const Grid& g = a.g;
  const int blk = gridDim.x >= ZREMAP_EPI ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
  const ZTile zt = z_tile(blk, a.ntile, g.ny, a.tiles, a.ntl);
  const int col = zt.tile * TX + c, ky = zt.ky, kyw = wav(ky, g.ny);
  if (a.prune && a.mode != 0 && !g.disk(zt.tile * TX, kyw)) return;
  const bool ok = col < g.nx / 2 + 1;
  const bool disk = ok && (!a.prune || g.disk(col, kyw));
  const long in_es = (long)g.ny * a.in_pitch, out_es = (long)g.ny * a.out_pitch;
  const C2<T>* in = a.in + zt.box * a.in_bs + ky * a.in_pitch + col;
  TwFill<T, L, NT, RL> fill;
  fill.load(a.tw, tid);
  C2<T> x[NR][E::FIRST_SLOTS];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int s = 0; s < E::FIRST_SLOTS; ++s) {
      const int f = grp + r * NG;
      x[r][s] = f < NP && disk && E::first_valid(q, s) ? in[f * a.in_fs + E::first_index(q, s) * in_es] : zero2<T>();
    }
  // the state: zz the fields the viscous term acts on, z0 the ones updated
  const int kperp2 = g.perp(col, kyw);
  const long base = zt.box * a.out_bs + ky * a.out_pitch + col;
  C2<T> zz[PTS][NF], z0[PTS][NF];
  auto touched = [&](int i) {  // point i of this thread is a mode the call writes
    const int kzi = tid / TX + i * (NT / TX);
    return ok && ((L * TX) % NT == 0 || kzi < L) && (a.mode == 0 || !a.prune || g.keep_p(kperp2, wav(kzi, L)));
  };
  if (a.mode != 0) {
    const C2<T>* zv = a.mode == 1 ? a.st0 : a.st1;
#pragma unroll
    for (int i = 0; i < PTS; ++i) {
      const bool t = touched(i);
      const long pos = base + (tid / TX + i * (NT / TX)) * out_es;
#pragma unroll
      for (int f = 0; f < NF; ++f) zz[i][f] = t ? zv[f * a.out_fs + pos] : zero2<T>();
      if (a.mode == 2) {
#pragma unroll
        for (int f = 0; f < NF; ++f) z0[i][f] = t ? a.st0[f * a.out_fs + pos] : zero2<T>();
      }
    }
  }
  fill.store(tws, tid);
  C2<T> v[NR][E::SLOTS];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int f = grp + r * NG;
    E::template run_tw<Lay>(v[r], smem + (f < NP ? f : 0) * TILE + c, TX, q, TwStaged<T>{tws},
                            [&](int s, int) { return x[r][s]; }, f < NP);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int f = grp + r * NG;
    if (f < NP) {
#pragma unroll
      for (int s = 0; s < NO; ++s)
        if (E::last_valid(q, s)) smem[f * TILE + c + Lay::off(E::last_index(q, s), TX)] = v[r][s];
    }
  }
  __syncthreads();
  const T kx = a.sx * (T)col, ky_ = a.sy * (T)kyw;
  const T kxd = a.sx * (T)dwavx(col, g.nx), kyd = a.sy * (T)dwav(ky, g.ny);
#pragma unroll
  for (int i = 0; i < PTS; ++i) {
    if (!touched(i)) continue;
    const int kzi = tid / TX + i * (NT / TX), ikz = wav(kzi, L);
    const bool zero_mode = col == 0 && kyw == 0 && ikz == 0;
    const bool keep = !zero_mode && g.keep_p(kperp2, ikz);
    // physical wavenumber (projector, |k|^2) and derivative wavenumber
    const T kz = a.sz * (T)ikz, kzd = a.sz * (T)dwav(kzi, L);
    const T k2 = kx * kx + ky_ * ky_ + kz * kz;
    auto at = [&](int f) -> C2<T> { return a.scale * smem[f * TILE + c + Lay::off(kzi, TX)]; };
    C2<T> nh[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) nh[f] = zero2<T>();
    if (keep) {
      const T ik2 = T(1) / k2;
      auto project = [&](C2<T>& n0, C2<T>& n1, C2<T>& n2) {  // P(k) n
        const C2<T> kn = kx * n0 + ky_ * n1 + kz * n2;
        n0 = n0 - (kx * ik2) * kn;
        n1 = n1 - (ky_ * ik2) * kn;
        n2 = n2 - (kz * ik2) * kn;
      };
      if constexpr (ELS && MHD) {
        // a_i = sum_j k_j T_ij, c_j = sum_i k_i T_ij, T_ij field 3 i + j, T_22 = 0
        C2<T> t[9];
#pragma unroll
        for (int f = 0; f < 8; ++f) t[f] = at(f);
        t[8] = zero2<T>();
        const T k[3] = {kxd, kyd, kzd};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          nh[d] = k[0] * t[3 * d] + k[1] * t[3 * d + 1] + k[2] * t[3 * d + 2];
          nh[3 + d] = k[0] * t[d] + k[1] * t[3 + d] + k[2] * t[6 + d];
        }
      } else if constexpr (ELS) {
        // S_00 - S_22, S_11 - S_22, S_01, S_02, S_12
        const C2<T> s00 = at(0), s11 = at(1), s01 = at(2), s02 = at(3), s12 = at(4);
        nh[0] = kxd * s00 + kyd * s01 + kzd * s02;
        nh[1] = kxd * s01 + kyd * s11 + kzd * s12;
        nh[2] = kxd * s02 + kyd * s12;
      } else {
#pragma unroll
        for (int f = 0; f < 3; ++f) nh[f] = at(f);
      }
      project(nh[0], nh[1], nh[2]);
      if constexpr (ELS && MHD) project(nh[3], nh[4], nh[5]);
      if constexpr (ELS) {
#pragma unroll
        for (int f = 0; f < NF; ++f) nh[f] = mul_mi(nh[f]);
      } else if constexpr (MHD) {
        const C2<T> e0 = at(3), e1 = at(4), e2 = at(5);
        const C2<T> c0 = mul_i(kyd * e2 - kzd * e1), c1 = mul_i(kzd * e0 - kxd * e2), c2 = mul_i(kxd * e1 - kyd * e0);
        nh[3] = nh[0] - c0;
        nh[4] = nh[1] - c1;
        nh[5] = nh[2] - c2;
        nh[0] = nh[0] + c0;
        nh[1] = nh[1] + c1;
        nh[2] = nh[2] + c2;
      }
    }
    const long pos = base + kzi * out_es;
    if (a.mode == 0) {
#pragma unroll
      for (int f = 0; f < NF; ++f) a.out[f * a.out_fs + pos] = nh[f];
      continue;
    }
    C2<T>* dst = a.mode == 1 ? a.out : const_cast<C2<T>*>(a.st0);
    C2<T> cor[3] = {zero2<T>(), zero2<T>(), zero2<T>()};
    if (a.rot && !zero_mode) {
      C2<T> u[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) u[d] = MHD ? T(0.5) * (zz[i][d] + zz[i][(d + 3) % NF]) : zz[i][d];
      const C2<T> w0 = a.w2y * u[2] - a.w2z * u[1];
      const C2<T> w1 = a.w2z * u[0] - a.w2x * u[2];
      const C2<T> w2 = a.w2x * u[1] - a.w2y * u[0];
      const C2<T> kw = (T(1) / k2) * (kx * w0 + ky_ * w1 + kz * w2);
      cor[0] = w0 - kx * kw;
      cor[1] = w1 - ky_ * kw;
      cor[2] = w2 - kz * kw;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      C2<T> vis = (a.nua * k2) * zz[i][f];
      if constexpr (MHD) vis = vis + (a.nub * k2) * zz[i][(f + 3) % NF];
      vis = vis + cor[f % 3];
      const C2<T> old = a.mode == 1 ? zz[i][f] : z0[i][f];
      dst[f * a.out_fs + pos] = old + a.h * (nh[f] - vis);
    }
  }
}

// Forward z pass + epilogue (k_z_epi's outputs and modes) with the fields of a
// column tile combined before the transform and in LDS side by side.
//
// A column's (kx, ky) is fixed, so with k = (kx, ky, kz), kp = |(kx, ky)| and the
// horizontal unit vectors eL = (kx, ky) / kp = (cx, cy) and eT = (-cy, cx) (eL =
// (1, 0) where kp = 0), linear combinations over the horizontal indices may be
// taken before the transform along z.  The projection keeps a vector's eT
// component and, of its (eL, ez) part, the component across k:
//   P(k) a = aT eT + s (-kz eL + kp ez),  s = (kp az - kz aL) / k^2.
// For the divergence forms, a_i = sum_j k_j T_ij, this needs from T = z+ z- (and
// its transpose for z-) only
//   T0+ = eT T eL, T0- = eL T eT, Q = eL T eL, T1+ = eT T ez, B = eL T ez,
//   T1- = ez T eT, A = ez T eL   (T less its isotropic part, T_zz = 0):
//   aT+- = kp T0+- + kz T1+-, aL+ = kp Q + kz B, az+ = kp A, aL- = kp Q + kz A,
//   az- = kp B:
// seven transforms instead of eight (MHD), and for the symmetric u u (T1+ = T1-,
// A = B, T0+ = T0-) four instead of five (NS).  The rotational forms transform
// their three or six fields as they are.
//
// Tiles: PH = 1 keeps all of them in LDS at once; PH = 2 does the two groups
// {T0, Q} and {T1, A, B} (MHD rotational: u x w + j x b, then u x b) one after
// the other, half the LDS.  Every thread first loads its elements of the
// group's input fields and writes their combinations to the tiles (the second
// group's and the state's loads are in flight during the first transforms);
// TX x TQ threads then transform each tile, all tiles at once; and each thread
// finishes the modes (c, kz) of its elements from LDS.
//
// Bound by memory (64-byte pieces of rows a plane apart) and the exchanges.
// One barrier-separated transform of a whole group, a seventh or a fifth fewer
// transforms and no accumulators held across them, against k_z_epi, launch
// times, us: MHD Elsasser 384^3 FP32 522 -> 384, FP64 1099 -> 757, 512^3 FP32 971
// -> 900, FP64 1820 -> 1650, 192^3 FP64 136 -> 82, 8 boxes of 96^3 FP32 73 -> 47;
// NS divergence form, 48 boxes of 64^3 FP32 61 -> 40, 16 of 96^3 53 -> 37, 4 of
// 128^3 33 -> 29.  It loses where k_z_epi's registers suffice (NS 256^3 FP32 55
// -> 70, MHD 256^3 FP32 123 -> 134) and, by its extra pass through LDS, to
// k_z_epi_field where a launch is one round of latency (NS 64^3 5.6 -> 6.3).
template <bool MHD, bool ELS>
struct EpiGroups {
  static constexpr int in0 = ELS ? (MHD ? 4 : 3) : 3, in1 = ELS ? (MHD ? 4 : 2) : MHD ? 3 : 0;
  static constexpr int out0 = ELS ? (MHD ? 3 : 2) : 3, out1 = ELS ? (MHD ? 4 : 2) : MHD ? 3 : 0;
  // input field i of group g
  static constexpr int field(int g, int i) {
    if (ELS && MHD) return g == 0 ? (i < 2 ? i : i + 1) : (i == 0 ? 2 : 4 + i);  // 00 01 10 11; 02 12 20 21
    return g == 0 ? i : in0 + i;                                               // NS: 00 11 01; 02 12
  }
  static constexpr int nin(int g) { return g == 0 ? in0 : in1; }
  static constexpr int nout(int g) { return g == 0 ? out0 : out1; }
  // tiles that are in LDS together
  static constexpr int tiles(int ph) { return ph == 1 ? out0 + out1 : out0 > out1 ? out0 : out1; }
  // tile t of group g from the group's inputs
  template <typename T>
  __device__ __forceinline__ static C2<T> tile(int g, int t, const C2<T>* x, T cx, T cy) {
    if constexpr (!ELS) {
      return x[t];
    } else if (g == 0) {
      if constexpr (MHD) {
        const C2<T> d = (cx * cy) * (x[3] - x[0]);
        if (t == 0) return (cx * cx) * x[2] + d - (cy * cy) * x[1];  // T0+
        if (t == 1) return (cx * cx) * x[1] + d - (cy * cy) * x[2];  // T0-
        return (cx * cx) * x[0] + (cx * cy) * (x[1] + x[2]) + (cy * cy) * x[3];
      } else {
        if (t == 0) return (cx * cx - cy * cy) * x[2] + (cx * cy) * (x[1] - x[0]);
        return (cx * cx) * x[0] + (T(2) * cx * cy) * x[2] + (cy * cy) * x[1];
      }
    } else {
      if (t == 0) return cx * x[1] - cy * x[0];  // T1+
      if (t == 1) return cx * x[0] + cy * x[1];  // B
      if constexpr (MHD) {
        if (t == 2) return cx * x[3] - cy * x[2];  // T1-
        return cx * x[2] + cy * x[3];              // A
      }
      return zero2<T>();
    }
  }
};

template <typename T, int L, int TQ, int TX, bool MHD, bool ELS, int PH>
struct EpiTileCfg {
  using G = EpiGroups<MHD, ELS>;
  static constexpr int TILES = G::tiles(PH), ROWS = pad8(L - 1) + 1;
  // thread groups: one per tile, fewer where 1024 threads do not hold them
  static constexpr int NG = [] {
    const int most = 1024 / (TX * TQ) < 1 ? 1 : 1024 / (TX * TQ);
    return cdiv(TILES, cdiv(TILES, most));
  }();
  static constexpr int NT = NG * TX * TQ;
  static constexpr int LDS = (TILES * ROWS * TX + L) * (int)sizeof(C2<T>);
  static constexpr bool FITS = LDS <= 163840 && NT <= 1024;
};

template <typename T, int L, int TQ, int TX, class RL, bool MHD, bool ELS, int PH>
__global__ __launch_bounds__((EpiTileCfg<T, L, TQ, TX, MHD, ELS, PH>::NT)) void k_z_epi_tile(ZEpiArgs<T> a) {
  using E = Stockham<T, L, TQ, FWD, RL>;
  using Cfg = EpiTileCfg<T, L, TQ, TX, MHD, ELS, PH>;
  using G = EpiGroups<MHD, ELS>;
  constexpr int NF = MHD ? 6 : 3;  // state fields
  constexpr int NG = Cfg::NG, NT = Cfg::NT, NO = E::LAST_NB * E::RL_;
  constexpr int PTS = cdiv(L * TX, NT);
  constexpr bool EXACT = (L * TX) % NT == 0;
  using Lay = LayColPad8;
  constexpr int TILE = Cfg::ROWS * TX;
  // the second group's and the state's loads go out before a transform, unless
  // its registers leave no room for them (16 values a thread, the first group's
  // results and the state of a long column: 971 us at 512 FP32 with spills,
  // 1045 without this line; 384 FP32 405 without the early loads, 384 with)
  constexpr bool AHEAD = L < 512;
  __shared__ C2<T> smem[Cfg::TILES * TILE + L];
  C2<T>* const tws = smem + Cfg::TILES * TILE;
  const int tid = threadIdx.x, c = tid % TX, q = tid / TX % TQ, grp = tid / (TX * TQ);
  const Grid& g = a.g;
  const int blk = gridDim.x >= ZREMAP_EPI ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
  const ZTile zt = z_tile(blk, a.ntile, g.ny, a.tiles, a.ntl);
  const int col = zt.tile * TX + c, ky = zt.ky, kyw = wav(ky, g.ny);
  if (a.prune && a.mode != 0 && !g.disk(zt.tile * TX, kyw)) return;
  const bool ok = col < g.nx / 2 + 1;
  const bool disk = ok && (!a.prune || g.disk(col, kyw));
  const long in_es = (long)g.ny * a.in_pitch, out_es = (long)g.ny * a.out_pitch;
  const C2<T>* in = a.in + zt.box * a.in_bs + ky * a.in_pitch + col;
  // element i of this thread: column c, row (grid plane, then kz) zi(i)
  auto zi = [&](int i) { return tid / TX + i * (NT / TX); };
  auto inside = [&](int i) { return EXACT || zi(i) < L; };
  const T kx = a.sx * (T)col, ky_ = a.sy * (T)kyw;
  const T kp2 = kx * kx + ky_ * ky_, kp = sqrt(kp2);
  const T ikp = kp2 > T(0) ? T(1) / kp : T(0);
  const T cx = kp2 > T(0) ? kx * ikp : T(1), cy = ky_ * ikp;
  TwFill<T, L, NT, RL> fill;
  fill.load(a.tw, tid);
  auto load0 = [&](C2<T>(&x)[PTS][G::in0]) {
#pragma unroll
    for (int i = 0; i < PTS; ++i)
#pragma unroll
      for (int f = 0; f < G::in0; ++f)
        x[i][f] = disk && inside(i) ? in[G::field(0, f) * a.in_fs + zi(i) * in_es] : zero2<T>();
  };
  constexpr int IN1 = G::in1 > 0 ? G::in1 : 1;
  auto load1 = [&](C2<T>(&x)[PTS][IN1]) {
#pragma unroll
    for (int i = 0; i < PTS; ++i)
#pragma unroll
      for (int f = 0; f < G::in1; ++f)
        x[i][f] = disk && inside(i) ? in[G::field(1, f) * a.in_fs + zi(i) * in_es] : zero2<T>();
  };
  // tiles [t0, t0 + nout) of LDS from a group's inputs
  auto put = [&](auto gc, int t0, const auto& x) {
    constexpr int gi = decltype(gc)::value;
#pragma unroll
    for (int i = 0; i < PTS; ++i)
      if (inside(i)) {
#pragma unroll
        for (int t = 0; t < G::nout(gi); ++t)
          smem[(t0 + t) * TILE + c + Lay::off(zi(i), TX)] = G::template tile<T>(gi, t, x[i], cx, cy);
      }
  };
  // transform the first n tiles in place (every thread takes part in the barriers)
  auto transform = [&](auto nc) {
    constexpr int n = decltype(nc)::value, NR = cdiv(n, NG);
    C2<T> v[NR][E::SLOTS];
    __syncthreads();  // the tiles (and the staged twiddles) are written
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int t = grp + r * NG;
      C2<T>* tile = smem + (t < n ? t : 0) * TILE + c;
      E::template run_tw<Lay>(v[r], tile, TX, q, TwStaged<T>{tws},
                              [&](int, int idx) { return tile[Lay::off(idx, TX)]; }, t < n);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int t = grp + r * NG;
      if (t < n) {
#pragma unroll
        for (int s = 0; s < NO; ++s)
          if (E::last_valid(q, s)) smem[t * TILE + c + Lay::off(E::last_index(q, s), TX)] = v[r][s];
      }
    }
    __syncthreads();
  };
  const int kperp2 = g.perp(col, kyw);
  const long base = zt.box * a.out_bs + ky * a.out_pitch + col;
  auto touched = [&](int i) {  // element i is a mode the call writes
    return ok && inside(i) && (a.mode == 0 || !a.prune || g.keep_p(kperp2, wav(zi(i), L)));
  };
  // the state: zz the fields the viscous term acts on
  C2<T> zz[PTS][NF];
  auto load_state = [&] {
    if (a.mode == 0) return;
    const C2<T>* zv = a.mode == 1 ? a.st0 : a.st1;
#pragma unroll
    for (int i = 0; i < PTS; ++i) {
      const bool t = touched(i);
#pragma unroll
      for (int f = 0; f < NF; ++f) zz[i][f] = t ? zv[f * a.out_fs + base + zi(i) * out_es] : zero2<T>();
    }
  };
  C2<T> h0[PTS][G::out0];  // the first group's results (PH = 2)
  using g0_ = std::integral_constant<int, 0>;
  using g1_ = std::integral_constant<int, 1>;
  {
    C2<T> x0[PTS][G::in0], x1[PTS][IN1];
    load0(x0);
    if constexpr (PH == 1) {
      load1(x1);
      load_state();
      fill.store(tws, tid);
      put(g0_{}, 0, x0);
      if constexpr (G::in1 > 0) put(g1_{}, G::out0, x1);
      transform(std::integral_constant<int, Cfg::TILES>{});
    } else {
      fill.store(tws, tid);
      put(g0_{}, 0, x0);
      if constexpr (AHEAD) load1(x1);
      transform(std::integral_constant<int, G::out0>{});
#pragma unroll
      for (int i = 0; i < PTS; ++i)
#pragma unroll
        for (int t = 0; t < G::out0; ++t)
          h0[i][t] = inside(i) ? smem[t * TILE + c + Lay::off(zi(i), TX)] : zero2<T>();
      __syncthreads();
      if constexpr (!AHEAD) load1(x1);
      put(g1_{}, 0, x1);
      if constexpr (AHEAD) load_state();
      transform(std::integral_constant<int, G::out1>{});
      if constexpr (!AHEAD) load_state();
    }
  }
#pragma unroll
  for (int i = 0; i < PTS; ++i) {
    if (!touched(i)) continue;
    const int kzi = zi(i), ikz = wav(kzi, L);
    const bool zero_mode = col == 0 && kyw == 0 && ikz == 0;
    const bool keep = !zero_mode && g.keep_p(kperp2, ikz);
    const T kz = a.sz * (T)ikz, k2 = kp2 + kz * kz;
    auto lds = [&](int t) -> C2<T> { return smem[t * TILE + c + Lay::off(kzi, TX)]; };
    auto at0 = [&](int t) -> C2<T> { return a.scale * (PH == 1 ? lds(t) : h0[i][t]); };
    auto at1 = [&](int t) -> C2<T> { return a.scale * lds(PH == 1 ? G::out0 + t : t); };
    const long pos = base + kzi * out_es;
    C2<T> z0[NF];
    if (a.mode == 2) {
#pragma unroll
      for (int f = 0; f < NF; ++f) z0[f] = a.st0[f * a.out_fs + pos];
    }
    C2<T> nh[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) nh[f] = zero2<T>();
    if (keep) {
      const T ik2 = T(1) / k2;
      if constexpr (ELS) {
        // -i P(k) a from its eT component and s
        auto put3 = [&](C2<T>* n, C2<T> aT, C2<T> s) {
          const C2<T> h = kz * s;
          n[0] = mul_mi(zero2<T>() - (cy * aT + cx * h));
          n[1] = mul_mi(cx * aT - cy * h);
          n[2] = mul_mi(kp * s);
        };
        if constexpr (MHD) {
          const C2<T> Q = kp * at0(2), t1p = at1(0), B = at1(1), t1m = at1(2), A = at1(3);
          put3(nh, kp * at0(0) + kz * t1p, ik2 * (kp2 * A - kz * (Q + kz * B)));
          put3(nh + 3, kp * at0(1) + kz * t1m, ik2 * (kp2 * B - kz * (Q + kz * A)));
        } else {
          const C2<T> B = at1(1);
          put3(nh, kp * at0(0) + kz * at1(0), ik2 * (kp2 * B - kz * (kp * at0(1) + kz * B)));
        }
      } else {
        C2<T> n0 = at0(0), n1 = at0(1), n2 = at0(2);
        const C2<T> kn = kx * n0 + ky_ * n1 + kz * n2;
        nh[0] = n0 - (kx * ik2) * kn;
        nh[1] = n1 - (ky_ * ik2) * kn;
        nh[2] = n2 - (kz * ik2) * kn;
        if constexpr (MHD) {
          // kept modes have no Nyquist index: derivatives use k itself
          const C2<T> e0 = at1(0), e1 = at1(1), e2 = at1(2);
          const C2<T> c0 = mul_i(ky_ * e2 - kz * e1), c1 = mul_i(kz * e0 - kx * e2), c2 = mul_i(kx * e1 - ky_ * e0);
          nh[3] = nh[0] - c0;
          nh[4] = nh[1] - c1;
          nh[5] = nh[2] - c2;
          nh[0] = nh[0] + c0;
          nh[1] = nh[1] + c1;
          nh[2] = nh[2] + c2;
        }
      }
    }
    if (a.mode == 0) {
#pragma unroll
      for (int f = 0; f < NF; ++f) a.out[f * a.out_fs + pos] = nh[f];
      continue;
    }
    C2<T>* dst = a.mode == 1 ? a.out : const_cast<C2<T>*>(a.st0);
    C2<T> cor[3] = {zero2<T>(), zero2<T>(), zero2<T>()};
    if (a.rot && !zero_mode) {
      C2<T> u[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) u[d] = MHD ? T(0.5) * (zz[i][d] + zz[i][(d + 3) % NF]) : zz[i][d];
      const C2<T> w0 = a.w2y * u[2] - a.w2z * u[1];
      const C2<T> w1 = a.w2z * u[0] - a.w2x * u[2];
      const C2<T> w2 = a.w2x * u[1] - a.w2y * u[0];
      const C2<T> kw = (T(1) / k2) * (kx * w0 + ky_ * w1 + kz * w2);
      cor[0] = w0 - kx * kw;
      cor[1] = w1 - ky_ * kw;
      cor[2] = w2 - kz * kw;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      C2<T> vis = (a.nua * k2) * zz[i][f];
      if constexpr (MHD) vis = vis + (a.nub * k2) * zz[i][(f + 3) % NF];
      vis = vis + cor[f % 3];
      dst[f * a.out_fs + pos] = (a.mode == 1 ? zz[i][f] : z0[f]) + a.h * (nh[f] - vis);
    }
  }
}

}  // namespace ps
