// ps_plane.hpp -- one z-plane's inverse y pass, product pass and forward y pass
// in one kernel, for boxes whose (ky, kx) plane of fields fits in LDS.
#pragma once

#include "ps_config.hpp"
#include "ps_kernels.hpp"

namespace ps {

// Schedules of the rows per length: XI / XF, inverse and forward.  The last
// radix of XI is the first of XF, so the thread that ends an inverse transform
// holding points q + TQ b + m (N / R) starts the forward one from the same
// points, and the products need no exchange.  V8: about eight values per thread;
// V4: four (more threads, fewer registers), at 64 points only, where k_plane
// takes six FP64 fields.
template <int N>
struct PlaneLen;
template <int TQ_, class XI_, class XF_>
struct PlaneX {
  static constexpr int TQ = TQ_;
  using XI = XI_;
  using XF = XF_;
};
#define PS_R(...) Radices<__VA_ARGS__>
#define PS_PLANE(N_, TQ8, XI8, XF8)   \
  template <>                         \
  struct PlaneLen<N_> {               \
    using V8 = PlaneX<TQ8, XI8, XF8>; \
    using V4 = V8;                    \
  };
PS_PLANE(8, 1, PS_R(8), PS_R(8))
PS_PLANE(12, 3, PS_R(3, 4), PS_R(4, 3))
PS_PLANE(16, 4, PS_R(4, 4), PS_R(4, 4))
PS_PLANE(24, 3, PS_R(3, 8), PS_R(8, 3))
PS_PLANE(32, 4, PS_R(4, 8), PS_R(8, 4))
PS_PLANE(48, 6, PS_R(3, 4, 4), PS_R(4, 4, 3))
template <>
struct PlaneLen<64> {
  using V8 = PlaneX<8, PS_R(8, 8), PS_R(8, 8)>;
  using V4 = PlaneX<16, PS_R(4, 4, 4), PS_R(4, 4, 4)>;
};
#undef PS_PLANE
#undef PS_R
#define PS_FOR_EACH_PLANE_N(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64)

template <typename T>
struct PlaneArgs {
  C2<T>* work;      // field f, plane z: work + box bs + f fs + z N pitch
  const C2<T>* tw;  // exp(-2 pi i e / N), e < N
  long fs, pitch, bs;
  int z0, nz, nb;  // planes [z0, z0 + nz) of every box
  Grid g;
};

template <typename T, int N, bool MHD, bool ELS, bool PR>
struct PlaneCfg {
  static constexpr int FIN = xprod_fin(MHD, ELS), FOUT = xprod_fout(MHD, ELS);
  static constexpr int F = FIN > FOUT ? FIN : FOUT;
  static constexpr int K = PR ? (N - 1) / 3 + 1 : N / 2 + 1;  // kx columns kept
  static constexpr int W = 256 / (int)sizeof(C2<T>);          // elements one LDS cycle serves
  using YC = LenCfg<N>;
  static constexpr int TQY = YC::TQ, CG = 64 / TQY;  // columns a wave transforms at a time
  // eight values per thread while the physical values of all input fields
  // fit in about 96 registers
  static constexpr bool EIGHT = FIN * 8 * (int)sizeof(C2<T>) / 4 <= 96;
  using XC = std::conditional_t<EIGHT, typename PlaneLen<N>::V8, typename PlaneLen<N>::V4>;
  static constexpr int TQX = XC::TQ, GX = 64 / TQX;  // row pairs a wave transforms at a time
  using EI = Stockham<T, N, TQX, INV, typename XC::XI>;
  using EF = Stockham<T, N, TQX, FWD, typename XC::XF>;
  static constexpr int YT1 = cdiv(FIN * K, CG), YT3 = cdiv(FOUT * K, CG), XT = cdiv(N / 2, GX);
  static constexpr int NW0 = YT3 > YT1 ? (YT3 > XT ? YT3 : XT) : (YT1 > XT ? YT1 : XT);
  static constexpr int NW = NW0 < 8 ? NW0 : 8;  // waves
  static constexpr int EXS = EI::EX_SLOTS > EF::EX_SLOTS ? EI::EX_SLOTS : EF::EX_SLOTS;
  static constexpr int lds(int kp, int nxw) {
    return (F * N * kp + nxw * GX * EXS + 3 * N) * (int)sizeof(C2<T>);
  }
  // pitch of an LDS row: odd (the first column stage writes rows 8 q + m), and
  // where the room is there away from multiples of W (columns of different
  // rows are read together)
  static constexpr int KP = [] {
    for (int p = K | 1; p < (K | 1) + 8; p += 2)
      if (p % W >= W / 4 - 1 && p % W <= 3 * W / 4 + 1 && lds(p, 4) <= 163840) return p;
    return K | 1;
  }();
  // waves that transform rows: as many as have some and find exchange space
  static constexpr int NXW = [] {
    int n = XT < NW ? XT : NW;
    while (n > 1 && lds(KP, n) > 163840) --n;
    return n;
  }();
  static constexpr int PLANE = F * N * KP, SCR = NXW * GX * EXS;
  static constexpr int LDS = lds(KP, NXW);
  static constexpr bool FITS = LDS <= 163840;
  // waves per SIMD asked of the register allocator: two workgroups per CU
  // where few fields leave the registers for it
  static constexpr int MINW = EIGHT && FIN == 3 && sizeof(T) == 4 && LDS <= 81920 && NW >= 2 ? NW / 2 : cdiv(NW, 4);
};

// One workgroup per (box, z-plane).  The plane of F fields x N x K kept columns
// lives in LDS between the three transforms: columns inverse (global -> LDS),
// rows inverse, products in registers, rows forward (LDS -> LDS, two real rows
// per complex transform), columns forward (LDS -> global), so the two passes
// over memory between them are gone.  A column's and a row pair's threads lie
// in one wave, so only the three phases are separated by workgroup barriers.
// Bound by LDS and vector issue, about equally.  48 boxes of NS 64^3 FP32 in the
// divergence form, pruned (3072 planes, two workgroups per CU): 113 us where
// the three passes took 115 + 45 + 71.
template <typename T, int N, bool MHD, bool ELS, bool PR>
__global__ __launch_bounds__((PlaneCfg<T, N, MHD, ELS, PR>::NW * 64), (PlaneCfg<T, N, MHD, ELS, PR>::MINW)) void
k_plane(PlaneArgs<T> a) {
  using P = PlaneCfg<T, N, MHD, ELS, PR>;
  constexpr int FIN = P::FIN, FOUT = P::FOUT, K = P::K, KP = P::KP, NW = P::NW;
  __shared__ C2<T> smem[P::PLANE + P::SCR + 3 * N];
  C2<T>* const twy = smem + P::PLANE + P::SCR;
  C2<T>* const twi = twy + N;
  C2<T>* const twf = twi + N;
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int box = blockIdx.x / a.nz, z = a.z0 + blockIdx.x % a.nz;
  C2<T>* const w = a.work + box * a.bs + (long)z * N * a.pitch;
  using YI = Stockham<T, N, P::TQY, INV, typename P::YC::RL>;
  using YF = Stockham<T, N, P::TQY, FWD, typename P::YC::RL>;
  using EI = typename P::EI;
  using EF = typename P::EF;
  fill_staged<T, N>(twy, a.tw, 1, tid, NW * 64, typename P::YC::RL{});
  fill_staged<T, N>(twi, a.tw, 1, tid, NW * 64, typename P::XC::XI{});
  fill_staged<T, N>(twf, a.tw, 1, tid, NW * 64, typename P::XC::XF{});
  __syncthreads();
  auto in_disk = [&](int col, int idx) { return !PR || a.g.disk(col, wav(idx, N)); };
  const int yc = lane % P::CG, yq = lane / P::CG;
  // ---- columns, inverse: memory -> the plane in LDS
  for (int t = wv; t < P::YT1; t += NW) {
    const int id = t * P::CG + yc, f = id / K, c = id % K;
    const bool act = yq < P::TQY && id < FIN * K;
    const C2<T>* in = w + f * a.fs + c;
    C2<T>* col = smem + f * N * KP + c;
    C2<T> v[YI::SLOTS];
    YI::template run_tw<LayStride, 2>(
        v, col, KP, yq, TwStaged<T>{twy},
        [&](int, int idx) { return in_disk(c, idx) ? in[idx * a.pitch] : zero2<T>(); }, act);
    wave_lds_sync();
    if (act) {
#pragma unroll
      for (int s = 0; s < YI::LAST_NB * YI::RL_; ++s)
        if (YI::last_valid(yq, s)) col[YI::last_index(yq, s) * KP] = v[s];
    }
  }
  __syncthreads();
  // ---- rows: two grid rows y = 2 pair, 2 pair + 1 of a field per transform
  {
    static_assert(EI::RL_ == EF::R1, "products are formed where the inverse transform left its points");
    constexpr int NP = EI::LAST_NB * EI::RL_;
    constexpr unsigned ZIN = PR ? xpk_mid_slots<N, EI::R1, P::TQX, (N - 1) / 3>() : 0u;
    const int g = lane / P::TQX, q = lane % P::TQX;
    for (int t = wv; t < P::XT && wv < P::NXW; t += P::NXW) {
      const int pair = t * P::GX + g;
      const bool act = g < P::GX && pair < N / 2;
      C2<T>* const buf = smem + P::PLANE + (wv * P::GX + g) * P::EXS;
      C2<T>* const rows = smem + 2 * pair * KP;
      C2<T> ph[FIN][NP];  // (x, y): the field on the two rows
#pragma unroll
      for (int f = 0; f < FIN; ++f) {
        const C2<T>* sx = rows + f * N * KP;
        C2<T> v[EI::SLOTS];
        EI::template run_ex<2>(
            v, buf, q, TwStaged<T>{twi},
            ld_zero<ZIN>([&](int, int k) -> C2<T> {
              // Z = X + i Y of the half spectra; only the real parts of the
              // kx = 0 and N/2 bins (the pass-order convention)
              const bool up = k > N / 2;
              const int kk = up ? N - k : k;
              const bool real_bin = kk == 0 || 2 * kk == N;
              const bool live = kk < K;
              const C2<T> x = live ? sx[kk] : zero2<T>(), y = live ? sx[KP + kk] : zero2<T>();
              const T xi = real_bin ? T(0) : (up ? -x.y : x.y);
              const T yi = real_bin ? T(0) : (up ? -y.y : y.y);
              return C2<T>{x.x - yi, xi + y.x};
            }),
            act);
#pragma unroll
        for (int s = 0; s < NP; ++s) ph[f][s] = v[s];
      }
#pragma unroll
      for (int fo = 0; fo < FOUT; ++fo) {
        C2<T> v[EF::SLOTS];
        EF::template run_ex<2>(
            v, buf, q, TwStaged<T>{twf},
            [&](int s, int) -> C2<T> {
              C2<T> acc = zero2<T>();
              bool first = true;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const PTerm pt = prod_def(MHD, ELS, fo).t[i];
                if (pt.s == 0) continue;
                const C2<T> x = ph[pt.a][s], y = ph[pt.b][s];
                const C2<T> xy{x.x * y.x, x.y * y.y};
                acc = first ? xy : pt.s > 0 ? acc + xy : acc - xy;  // the first term's sign is +
                first = false;
              }
              return acc;
            },
            act);
        wave_lds_sync();
        if (act) {
#pragma unroll
          for (int s = 0; s < EF::LAST_NB * EF::RL_; ++s)
            if (EF::last_valid(q, s)) buf[EF::last_index(q, s)] = v[s];
        }
        wave_lds_sync();
        // the two spectra, over the rows of input field fo (already read)
        if (act) {
          C2<T>* dst = rows + fo * N * KP;
          for (int k = q; k < K; k += P::TQX) {
            const C2<T> zk = buf[k], zm = conj(buf[k == 0 ? 0 : N - k]);
            dst[k] = T(0.5) * (zk + zm);
            dst[KP + k] = T(0.5) * mul_mi(zk - zm);
          }
        }
      }
    }
  }
  __syncthreads();
  // ---- columns, forward: the plane -> memory
  for (int t = wv; t < P::YT3; t += NW) {
    const int id = t * P::CG + yc, f = id / K, c = id % K;
    const bool act = yq < P::TQY && id < FOUT * K;
    C2<T>* col = smem + f * N * KP + c;
    C2<T>* out = w + f * a.fs + c;
    C2<T> v[YF::SLOTS];
    YF::template run_tw<LayStride, 2>(v, col, KP, yq, TwStaged<T>{twy}, [&](int, int idx) { return col[idx * KP]; },
                                      act);
    if (act) {
#pragma unroll
      for (int s = 0; s < YF::LAST_NB * YF::RL_; ++s) {
        const int idx = YF::last_index(yq, s);
        if (YF::last_valid(yq, s) && in_disk(c, idx)) out[idx * a.pitch] = v[s];
      }
    }
  }
}

// The same passes for few planes, where one plane's latency counts: the fields
// go over the waves in every phase (a wave transforms one field's columns, then
// one field's row pairs, then one product's), so each wave's chain is a few
// transforms long; the physical rows stay in the plane's own rows in LDS.  For
// one small box it is bound by latency: step times with the three passes and
// with this kernel: NS 32^3 FP64 55 and 42 us, MHD 64^3 FP32 pruned 72 and 64.
template <typename T, int N, bool MHD, bool ELS, bool PR>
struct PlaneFieldCfg {
  static constexpr int FIN = xprod_fin(MHD, ELS), FOUT = xprod_fout(MHD, ELS);
  static constexpr int F = FIN > FOUT ? FIN : FOUT;
  static constexpr int K = PR ? (N - 1) / 3 + 1 : N / 2 + 1;
  static constexpr int W = 256 / (int)sizeof(C2<T>);
  using YC = LenCfg<N>;
  static constexpr int TQY = YC::TQ, CG = 64 / TQY;
  using XC = typename PlaneLen<N>::V8;
  static constexpr int TQX = XC::TQ, GX = 64 / TQX, XG = cdiv(N / 2, GX);  // pair groups of a field
  using EI = Stockham<T, N, TQX, INV, typename XC::XI>;
  using EF = Stockham<T, N, TQX, FWD, typename XC::XF>;
  static constexpr int EXS = EI::EX_SLOTS > EF::EX_SLOTS ? EI::EX_SLOTS : EF::EX_SLOTS;
  // a pair's two rows hold one transform's exchanges (EXS slots)
  static constexpr int KMIN = (K > (EXS + 1) / 2 ? K : (EXS + 1) / 2) | 1;
  static constexpr int lds(int kp) { return (F * N * kp + 3 * N) * (int)sizeof(C2<T>); }
  static constexpr int KP = [] {
    for (int p = KMIN; p < KMIN + 8; p += 2)
      if (p % W >= W / 4 - 1 && p % W <= 3 * W / 4 + 1 && lds(p) <= 163840) return p;
    return KMIN;
  }();
  static constexpr int LDS = lds(KP);
  static constexpr bool FITS = LDS <= 163840;
  static constexpr int YT1 = cdiv(FIN * K, CG), YT3 = cdiv(FOUT * K, CG);
  static constexpr int most(int a, int b) { return a > b ? a : b; }
  static constexpr int NW0 = most(most(YT1, YT3), F * XG);
  static constexpr int NW = NW0 < 16 ? NW0 : 16;
  static constexpr int R2 = cdiv(FOUT * XG, NW);  // products a wave transforms
};

template <typename T, int N, bool MHD, bool ELS, bool PR>
__global__ __launch_bounds__((PlaneFieldCfg<T, N, MHD, ELS, PR>::NW * 64)) void k_plane_field(PlaneArgs<T> a) {
  using P = PlaneFieldCfg<T, N, MHD, ELS, PR>;
  constexpr int FIN = P::FIN, FOUT = P::FOUT, K = P::K, KP = P::KP, NW = P::NW, NT = NW * 64;
  __shared__ C2<T> smem[P::F * N * KP + 3 * N];
  C2<T>* const twy = smem + P::F * N * KP;
  C2<T>* const twi = twy + N;
  C2<T>* const twf = twi + N;
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int box = blockIdx.x / a.nz, z = a.z0 + blockIdx.x % a.nz;
  C2<T>* const w = a.work + box * a.bs + (long)z * N * a.pitch;
  using YI = Stockham<T, N, P::TQY, INV, typename P::YC::RL>;
  using YF = Stockham<T, N, P::TQY, FWD, typename P::YC::RL>;
  using EI = typename P::EI;
  using EF = typename P::EF;
  auto in_disk = [&](int col, int idx) { return !PR || a.g.disk(col, wav(idx, N)); };
  const int yc = lane % P::CG, yq = lane / P::CG;
  // ---- columns, inverse; the first columns' loads are in flight together
  // with the twiddles'
  TwFill<T, N, NT, typename P::YC::RL> fy;
  TwFill<T, N, NT, typename P::XC::XI> fi;
  TwFill<T, N, NT, typename P::XC::XF> ff;
  fy.load(a.tw, tid);
  fi.load(a.tw, tid);
  ff.load(a.tw, tid);
  auto fetch = [&](int t, C2<T>(&x)[YI::FIRST_SLOTS]) {
    const int id = t * P::CG + yc, f = id / K, c = id % K;
    const bool act = yq < P::TQY && id < FIN * K;
    const C2<T>* in = w + f * a.fs + c;
#pragma unroll
    for (int s = 0; s < YI::FIRST_SLOTS; ++s) {
      const int idx = YI::first_index(yq, s);
      x[s] = act && YI::first_valid(yq, s) && in_disk(c, idx) ? in[idx * a.pitch] : zero2<T>();
    }
  };
  C2<T> x[YI::FIRST_SLOTS];
  fetch(wv, x);
  fy.store(twy, tid);
  fi.store(twi, tid);
  ff.store(twf, tid);
  __syncthreads();
  for (int t = wv; t < P::YT1; t += NW) {
    const int id = t * P::CG + yc;
    const bool act = yq < P::TQY && id < FIN * K;
    C2<T>* col = smem + (id / K) * N * KP + id % K;
    if (t != wv) fetch(t, x);
    C2<T> v[YI::SLOTS];
    YI::template run_tw<LayStride, 2>(v, col, KP, yq, TwStaged<T>{twy}, [&](int s, int) { return x[s]; }, act);
    wave_lds_sync();
    if (act) {
#pragma unroll
      for (int s = 0; s < YI::LAST_NB * YI::RL_; ++s)
        if (YI::last_valid(yq, s)) col[YI::last_index(yq, s) * KP] = v[s];
    }
  }
  __syncthreads();
  const int g = lane / P::TQX, q = lane % P::TQX;
  // ---- rows, inverse, in place: rows 2 pair and 2 pair + 1 of field f become
  // the N values (x, y) of the physical rows
  for (int t = wv; t < FIN * P::XG; t += NW) {
    constexpr unsigned ZIN = PR ? xpk_mid_slots<N, EI::R1, P::TQX, (N - 1) / 3>() : 0u;
    const int f = t / P::XG, pair = t % P::XG * P::GX + g;
    const bool act = g < P::GX && pair < N / 2;
    C2<T>* const buf = smem + (f * N + 2 * pair) * KP;
    C2<T> v[EI::SLOTS];
    EI::template run_ex<2>(
        v, buf, q, TwStaged<T>{twi},
        ld_zero<ZIN>([&](int, int k) -> C2<T> {
          const bool up = k > N / 2;
          const int kk = up ? N - k : k;
          const bool real_bin = kk == 0 || 2 * kk == N;  // real parts only (the pass-order convention)
          const bool live = kk < K;
          const C2<T> xr = live ? buf[kk] : zero2<T>(), yr = live ? buf[KP + kk] : zero2<T>();
          const T xi = real_bin ? T(0) : (up ? -xr.y : xr.y);
          const T yi = real_bin ? T(0) : (up ? -yr.y : yr.y);
          return C2<T>{xr.x - yi, xi + yr.x};
        }),
        act);
    wave_lds_sync();
    if (act) {
#pragma unroll
      for (int s = 0; s < EI::LAST_NB * EI::RL_; ++s)
        if (EI::last_valid(q, s)) buf[EI::last_index(q, s)] = v[s];
    }
  }
  __syncthreads();
  // ---- products, all read before any row is overwritten
  C2<T> p[P::R2][EF::FIRST_SLOTS];
#pragma unroll
  for (int r = 0; r < P::R2; ++r) {
    const int t = wv + r * NW, fo = t / P::XG, pair = t % P::XG * P::GX + g;
    const bool act = t < FOUT * P::XG && g < P::GX && pair < N / 2;
#pragma unroll
    for (int s = 0; s < EF::FIRST_SLOTS; ++s) {
      p[r][s] = zero2<T>();
      if (act && EF::first_valid(q, s)) {
        const int n = 2 * pair * KP + EF::first_index(q, s);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const PTerm pt = prod_def(MHD, ELS, fo).t[i];
          if (pt.s != 0) {
            const C2<T> xa = smem[pt.a * N * KP + n], xb = smem[pt.b * N * KP + n];
            p[r][s] = C2<T>{p[r][s].x + T(pt.s) * xa.x * xb.x, p[r][s].y + T(pt.s) * xa.y * xb.y};
          }
        }
      }
    }
  }
  __syncthreads();
  // ---- rows, forward, in place over input field fo's rows
#pragma unroll
  for (int r = 0; r < P::R2; ++r) {
    const int t = wv + r * NW, fo = t / P::XG, pair = t % P::XG * P::GX + g;
    if (t >= FOUT * P::XG) break;  // uniform over the wave
    const bool act = g < P::GX && pair < N / 2;
    C2<T>* const buf = smem + (fo * N + 2 * pair) * KP;
    C2<T> v[EF::SLOTS];
    EF::template run_ex<2>(v, buf, q, TwStaged<T>{twf}, [&](int s, int) { return p[r][s]; }, act);
    wave_lds_sync();
    if (act) {
#pragma unroll
      for (int s = 0; s < EF::LAST_NB * EF::RL_; ++s)
        if (EF::last_valid(q, s)) buf[EF::last_index(q, s)] = v[s];
    }
    wave_lds_sync();
    constexpr int NK = cdiv(K, P::TQX);
    C2<T> o0[NK], o1[NK];
    if (act) {
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        const int k = q + i * P::TQX, kc = k < K ? k : K - 1;
        const C2<T> zk = buf[kc], zm = conj(buf[kc == 0 ? 0 : N - kc]);
        o0[i] = T(0.5) * (zk + zm);
        o1[i] = T(0.5) * mul_mi(zk - zm);
      }
    }
    wave_lds_sync();
    if (act) {
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        const int k = q + i * P::TQX;
        if (k < K) {
          buf[k] = o0[i];
          buf[KP + k] = o1[i];
        }
      }
    }
  }
  __syncthreads();
  // ---- columns, forward: the plane -> memory
  for (int t = wv; t < P::YT3; t += NW) {
    const int id = t * P::CG + yc, f = id / K, c = id % K;
    const bool act = yq < P::TQY && id < FOUT * K;
    C2<T>* col = smem + f * N * KP + c;
    C2<T>* out = w + f * a.fs + c;
    C2<T> v[YF::SLOTS];
    YF::template run_tw<LayStride, 2>(v, col, KP, yq, TwStaged<T>{twy}, [&](int, int idx) { return col[idx * KP]; },
                                      act);
    if (act) {
#pragma unroll
      for (int s = 0; s < YF::LAST_NB * YF::RL_; ++s) {
        const int idx = YF::last_index(yq, s);
        if (YF::last_valid(yq, s) && in_disk(c, idx)) out[idx * a.pitch] = v[s];
      }
    }
  }
}

}  // namespace ps
