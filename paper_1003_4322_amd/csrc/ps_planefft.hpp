// ps_planefft.hpp -- the x and y passes of the plain 3D transforms in one
// kernel, for boxes whose z-plane of one field fits in LDS.
#pragma once

#include "ps_config.hpp"
#include "ps_kernels.hpp"

namespace ps {

#define PS_FOR_EACH_PLANEFFT_N(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96)

template <typename T, int N>
struct PlaneFftCfg {
  using C = LenCfg<N>;
  static constexpr int K = N / 2 + 1, TQ = C::TQ;
  using EI = Stockham<T, N, TQ, INV, typename C::RL>;
  using EF = Stockham<T, N, TQ, FWD, typename C::RL>;
  static constexpr int EXS = EI::EX_SLOTS > N ? EI::EX_SLOTS : N;
  // LDS row pitch: odd, and a pair of rows holds one transform's exchanges
  static constexpr int KP = (K > (EXS + 1) / 2 ? K : (EXS + 1) / 2) | 1;
  static constexpr int NTC = K * TQ, NTR = N / 2 * TQ;  // threads of the columns, of the row pairs
  static constexpr int NT = ((NTC > NTR ? NTC : NTR) + 63) / 64 * 64;
  static constexpr int LDS = (N * KP + N) * (int)sizeof(C2<T>);
  // two workgroups per CU: an FP64 plane of 96 x 96 leaves one, and separate
  // passes are faster (c2r of three fields 34 us with the plane kernel, 28.5
  // without; at 128 the two tie in FP32, 31.4 against 30.4)
  static constexpr bool FITS = LDS <= 81920 && NT <= 1024;
};

template <typename T>
struct PlaneFftArgs {
  const C2<T>* tw;  // exp(-2 pi i e / N), e < N
  C2<T>* cplx;      // half spectra along x and y: plane p of set f at f fs + p N pitch
  T* real;          // real planes, N reals a row, dense
  long fs, pitch;   // field stride and row pitch of cplx
  long bs;          // box stride of cplx
  int nz, nf, nb;   // planes a field, fields a box, boxes
};

// One workgroup per plane of one field, the plane in LDS between the two
// transforms: K = N/2 + 1 columns along y, and two real rows per complex
// transform along x (Z = X + i Y of their half spectra).  Against separate x
// and y passes the plane is read and written once instead of twice.
//   c2r: inverse columns, then rows (the real parts of the kx = 0 and N/2 bins
//        only, the pass-order convention); r2c: rows, then forward columns.
// Whole transforms of three fields with it and with separate x and y passes:
// 48^3 FP32 c2r 11.7 us against 14.6, 64^3 FP64 r2c 13.3 against 17.1.
template <typename T, int N>
__global__ __launch_bounds__((PlaneFftCfg<T, N>::NT)) void k_plane_c2r(PlaneFftArgs<T> a) {
  using P = PlaneFftCfg<T, N>;
  using E = typename P::EI;
  constexpr int K = P::K, KP = P::KP, TQ = P::TQ, NT = P::NT;
  __shared__ C2<T> smem[N * KP + N];
  C2<T>* const tws = smem + N * KP;
  const int tid = threadIdx.x;
  const int z = blockIdx.x % a.nz, fb = blockIdx.x / a.nz;
  const C2<T>* in = a.cplx + (fb / a.nf) * a.bs + (fb % a.nf) * a.fs + (long)z * N * a.pitch;
  T* out = a.real + (long)blockIdx.x * N * N;
  TwFill<T, N, NT, typename P::C::RL> fill;
  fill.load(a.tw, tid);
  C2<T> v[E::SLOTS];
  {
    const int c = tid % K, q = tid / K;
    const bool act = q < TQ;
    C2<T> x[E::FIRST_SLOTS];
#pragma unroll
    for (int s = 0; s < E::FIRST_SLOTS; ++s)
      x[s] = act && E::first_valid(q, s) ? in[E::first_index(q, s) * a.pitch + c] : zero2<T>();
    fill.store(tws, tid);
    E::template run_tw<LayStride>(v, smem + c, KP, q, TwStaged<T>{tws}, [&](int s, int) { return x[s]; }, act);
    __syncthreads();
    if (act) {
#pragma unroll
      for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
        if (E::last_valid(q, s)) smem[E::last_index(q, s) * KP + c] = v[s];
    }
  }
  __syncthreads();
  {
    const int pair = tid / TQ, q = tid % TQ;
    const bool act = pair < N / 2;
    C2<T>* const buf = smem + 2 * pair * KP;
    E::template run_ex<0>(
        v, buf, q, TwStaged<T>{tws},
        [&](int, int k) -> C2<T> {
          const bool up = k > N / 2, real_bin = k == 0 || 2 * k == N;
          const int kk = up ? N - k : k;
          const C2<T> xr = buf[kk], yr = buf[KP + kk];
          const T xi = real_bin ? T(0) : (up ? -xr.y : xr.y);
          const T yi = real_bin ? T(0) : (up ? -yr.y : yr.y);
          return C2<T>{xr.x - yi, xi + yr.x};
        },
        act);
    __syncthreads();
    if (act) {
#pragma unroll
      for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
        if (E::last_valid(q, s)) buf[E::last_index(q, s)] = v[s];
    }
  }
  __syncthreads();
  // rows 2 p and 2 p + 1, two reals a thread
  for (int i = tid; i < N / 2 * (N / 2); i += NT) {
    const int p = i / (N / 2), n = 2 * (i % (N / 2));
    const C2<T> z0 = smem[2 * p * KP + n], z1 = smem[2 * p * KP + n + 1];
    C2<T>* row = reinterpret_cast<C2<T>*>(out + (long)2 * p * N + n);
    row[0] = C2<T>{z0.x, z1.x};
    row[N / 2] = C2<T>{z0.y, z1.y};
  }
}

template <typename T, int N>
__global__ __launch_bounds__((PlaneFftCfg<T, N>::NT)) void k_plane_r2c(PlaneFftArgs<T> a) {
  using P = PlaneFftCfg<T, N>;
  using E = typename P::EF;
  constexpr int K = P::K, KP = P::KP, TQ = P::TQ, NT = P::NT;
  __shared__ C2<T> smem[N * KP + N];
  C2<T>* const tws = smem + N * KP;
  const int tid = threadIdx.x;
  const int z = blockIdx.x % a.nz, fb = blockIdx.x / a.nz;
  const T* in = a.real + (long)blockIdx.x * N * N;
  C2<T>* out = a.cplx + (fb / a.nf) * a.bs + (fb % a.nf) * a.fs + (long)z * N * a.pitch;
  TwFill<T, N, NT, typename P::C::RL> fill;
  fill.load(a.tw, tid);
  for (int i = tid; i < N / 2 * (N / 2); i += NT) {
    const int p = i / (N / 2), n = 2 * (i % (N / 2));
    const C2<T>* row = reinterpret_cast<const C2<T>*>(in + (long)2 * p * N + n);
    const C2<T> x = row[0], y = row[N / 2];
    smem[2 * p * KP + n] = C2<T>{x.x, y.x};
    smem[2 * p * KP + n + 1] = C2<T>{x.y, y.y};
  }
  fill.store(tws, tid);
  __syncthreads();
  C2<T> v[E::SLOTS];
  {
    const int pair = tid / TQ, q = tid % TQ;
    const bool act = pair < N / 2;
    C2<T>* const buf = smem + 2 * pair * KP;
    E::template run_ex<0>(v, buf, q, TwStaged<T>{tws}, [&](int, int n) { return buf[n]; }, act);
    __syncthreads();
    if (act) {
#pragma unroll
      for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
        if (E::last_valid(q, s)) buf[E::last_index(q, s)] = v[s];
    }
    __syncthreads();
    // the two rows' spectra, in place of the pair's transform
    constexpr int NK = cdiv(K, TQ);
    C2<T> o0[NK], o1[NK];
    if (act) {
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        const int k = q + i * TQ, kc = k < K ? k : K - 1;
        const C2<T> zk = buf[kc], zm = conj(buf[kc == 0 ? 0 : N - kc]);
        o0[i] = T(0.5) * (zk + zm);
        o1[i] = T(0.5) * mul_mi(zk - zm);
      }
    }
    __syncthreads();
    if (act) {
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        const int k = q + i * TQ;
        if (k < K) {
          buf[k] = o0[i];
          buf[KP + k] = o1[i];
        }
      }
    }
  }
  __syncthreads();
  const int c = tid % K, q = tid / K;
  const bool act = q < TQ;
  E::template run_tw<LayStride>(v, smem + c, KP, q, TwStaged<T>{tws},
                                [&](int, int idx) { return smem[idx * KP + c]; }, act);
  if (act) {
#pragma unroll
    for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
      if (E::last_valid(q, s)) out[E::last_index(q, s) * a.pitch + c] = v[s];
  }
}

}  // namespace ps
