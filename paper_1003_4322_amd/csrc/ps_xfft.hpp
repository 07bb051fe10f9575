// ps_xfft.hpp -- plain real transforms along x (contiguous rows).
#pragma once

#include "ps_config.hpp"
#include "ps_kernels.hpp"

namespace ps {

// Two real rows X, Y of one field per complex transform of the full length N
// (z = x + i y), TQ threads each, G transforms a workgroup.  Rows go straight
// between memory and the first or last stage's registers (STAGE: by way of LDS);
// else only the exchanges (and, forward, the upper half of the spectrum the
// split needs) use LDS.
// Bound by memory: against half-length transforms with their rows staged in
// LDS and twiddles read from memory, three fields take (whole transforms) 964 ->
// 860 us (r2c 384^3 FP32), 2475 -> 1968 (r2c 512^3 FP32), 4498 -> 4006 (c2r 512^3
// FP64), 34 -> 28.5 (c2r 96^3 FP64).
template <typename T, int N>
struct XFftCfg {
  using C = LenCfg<N>;
  static constexpr int TQ = C::TQ;
  using EI = Stockham<T, N, TQ, INV, typename C::RL>;
  using EF = Stockham<T, N, TQ, FWD, typename C::RL>;
  static constexpr bool XW = TQ <= 64 && 64 % TQ == 0;  // a transform lies in one wave
  static constexpr int EXS = EI::EX_SLOTS;
  static constexpr int G = 256 / TQ < 1 ? 1 : 256 / TQ;
  static constexpr int NT = G * TQ;
  // rows staged in LDS where one thread has the whole transform and would touch
  // a row of its own in each access (8 x 1024 x 384, whole transforms of six FP32
  // fields: r2c 190 -> 145 us, c2r 306 -> 257); three threads and more lose by the
  // two barriers (24 x 64 x 96 c2r 16.6 -> 19.9, 48 x 256 x 192 r2c 66 -> 75)
  static constexpr int K = N / 2 + 1;
  static constexpr bool STAGE = TQ == 1;
  static_assert(!STAGE || NT == G, "staged copies take whole rounds of the workgroup");
  // LDS slots of a transform (odd: neighbours in different banks)
  static constexpr int S = STAGE ? (EXS > 2 * K ? EXS : 2 * K) | 1 : EXS;
};

template <typename T>
struct XFftArgs {
  const C2<T>* tw;  // exp(-2 pi i e / N), e < N
  C2<T>* cplx;      // half spectra: row r of field f of box b at b bs + f fs + r pitch
  T* real;          // dense rows of N reals
  long fs, pitch, bs;
  unsigned pairs;  // row pairs a field (ny nz / 2)
  int nf, nb;
};

// the transform's row pair: its two rows in both arrays
template <typename T, int N>
struct XFftRows {
  C2<T>* c[2];
  T* r[2];
  bool ok;
  __device__ __forceinline__ XFftRows(const XFftArgs<T>& a, unsigned id) {
    ok = id < a.pairs * (unsigned)(a.nf * a.nb);
    const unsigned fb = ok ? id / a.pairs : 0, p = ok ? id - fb * a.pairs : 0;
    const unsigned b = fb / (unsigned)a.nf, f = fb - b * (unsigned)a.nf;
    c[0] = a.cplx + (long)b * a.bs + (long)f * a.fs + (long)(2 * p) * a.pitch;
    c[1] = c[0] + a.pitch;
    r[0] = a.real + ((long)fb * a.pairs + p) * 2 * N;
    r[1] = r[0] + N;
  }
};

template <typename T, int N>
__global__ __launch_bounds__((XFftCfg<T, N>::NT)) void k_x_c2r(XFftArgs<T> a) {
  using X = XFftCfg<T, N>;
  using E = typename X::EI;
  constexpr int K = X::K;
  __shared__ C2<T> smem[X::G * X::S + N];
  C2<T>* const tws = smem + X::G * X::S;
  const int tid = threadIdx.x, c = tid / X::TQ, q = tid % X::TQ;
  const unsigned first = (unsigned)xcd_remap(blockIdx.x, gridDim.x) * X::G;
  const XFftRows<T, N> rows(a, first + c);
  C2<T>* const buf = smem + c * X::S;
  TwFill<T, N, X::NT, typename X::C::RL> fill;
  fill.load(a.tw, tid);
  C2<T> x[E::FIRST_SLOTS], y[E::FIRST_SLOTS];
  if constexpr (X::STAGE) {
    C2<T> ld[2 * K];  // (a workgroup has as many threads as transforms)
#pragma unroll
    for (int j = 0; j < 2 * K; ++j) {
      const int i = tid + j * X::NT, e = i % (2 * K);
      const XFftRows<T, N> row(a, first + i / (2 * K));
      ld[j] = row.ok ? row.c[e / K][e % K] : zero2<T>();
    }
#pragma unroll
    for (int j = 0; j < 2 * K; ++j) {
      const int i = tid + j * X::NT;
      smem[i / (2 * K) * X::S + i % (2 * K)] = ld[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int s = 0; s < E::FIRST_SLOTS; ++s) {
    const int k = E::first_index(q, s), kk = k > N / 2 ? N - k : k;
    const bool live = rows.ok && E::first_valid(q, s);
    x[s] = live ? (X::STAGE ? buf[kk] : rows.c[0][kk]) : zero2<T>();
    y[s] = live ? (X::STAGE ? buf[K + kk] : rows.c[1][kk]) : zero2<T>();
  }
  fill.store(tws, tid);
  C2<T> v[E::SLOTS];
  // the first stage's barrier orders the twiddles before their first use
  E::template run_ex<X::XW>(v, buf, q, TwStaged<T>{tws}, [&](int s, int k) -> C2<T> {
    // Z = X + i Y; only the real parts of the kx = 0 and N/2 bins
    const bool up = k > N / 2, real_bin = k == 0 || 2 * k == N;
    const T xi = real_bin ? T(0) : (up ? -x[s].y : x[s].y);
    const T yi = real_bin ? T(0) : (up ? -y[s].y : y[s].y);
    return C2<T>{x[s].x - yi, xi + y[s].x};
  });
  if constexpr (X::STAGE) {
    __syncthreads();
#pragma unroll
    for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
      if (E::last_valid(q, s)) buf[E::last_index(q, s)] = v[s];
    __syncthreads();
    // the real rows of all pairs follow one another
    T* const out = a.real + (long)first * 2 * N;
#pragma unroll
    for (int j = 0; j < 2 * N; ++j) {
      const int i = tid + j * X::NT, t = i / (2 * N), e = i % (2 * N);
      const C2<T> z = smem[t * X::S + e % N];
      if (first + t < a.pairs * (unsigned)(a.nf * a.nb)) out[i] = e < N ? z.x : z.y;
    }
    return;
  }
  if (!rows.ok) return;
#pragma unroll
  for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
    if (E::last_valid(q, s)) {
      rows.r[0][E::last_index(q, s)] = v[s].x;
      rows.r[1][E::last_index(q, s)] = v[s].y;
    }
}

template <typename T, int N>
__global__ __launch_bounds__((XFftCfg<T, N>::NT)) void k_x_r2c(XFftArgs<T> a) {
  using X = XFftCfg<T, N>;
  using E = typename X::EF;
  constexpr int K = X::K;
  __shared__ C2<T> smem[X::G * X::S + N];
  C2<T>* const tws = smem + X::G * X::S;
  const int tid = threadIdx.x, c = tid / X::TQ, q = tid % X::TQ;
  const unsigned first = (unsigned)xcd_remap(blockIdx.x, gridDim.x) * X::G;
  const XFftRows<T, N> rows(a, first + c);
  C2<T>* const buf = smem + c * X::S;
  TwFill<T, N, X::NT, typename X::C::RL> fill;
  fill.load(a.tw, tid);
  C2<T> x[E::FIRST_SLOTS];
  if constexpr (X::STAGE) {
    // the real rows of all pairs follow one another
    const T* const in = a.real + (long)first * 2 * N;
    T ld[2 * N];  // (a workgroup has as many threads as transforms)
#pragma unroll
    for (int j = 0; j < 2 * N; ++j) {
      const int i = tid + j * X::NT;
      ld[j] = first + i / (2 * N) < a.pairs * (unsigned)(a.nf * a.nb) ? in[i] : T(0);
    }
#pragma unroll
    for (int j = 0; j < 2 * N; ++j) {
      const int i = tid + j * X::NT, t = i / (2 * N), e = i % (2 * N);
      reinterpret_cast<T*>(smem + t * X::S + e % N)[e / N] = ld[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int s = 0; s < E::FIRST_SLOTS; ++s) {
    const int n = E::first_index(q, s);
    const bool live = rows.ok && E::first_valid(q, s);
    if constexpr (X::STAGE)
      x[s] = live ? buf[n] : zero2<T>();
    else
      x[s] = live ? C2<T>{rows.r[0][n], rows.r[1][n]} : zero2<T>();
  }
  fill.store(tws, tid);
  C2<T> v[E::SLOTS];
  E::template run_ex<X::XW>(v, buf, q, TwStaged<T>{tws}, [&](int s, int) { return x[s]; });
  auto own_sync = [] {
    if constexpr (X::XW)
      wave_lds_sync();
    else
      __syncthreads();
  };
  auto split = [&](int k, C2<T> zk, C2<T> zm) {  // Z[k] and conj Z[N - k]
    rows.c[0][k] = T(0.5) * (zk + zm);
    rows.c[1][k] = T(0.5) * mul_mi(zk - zm);
  };
  if constexpr (X::STAGE) {
    __syncthreads();
#pragma unroll
    for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
      if (E::last_valid(q, s)) buf[E::last_index(q, s)] = v[s];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2 * K; ++j) {
      const int i = tid + j * X::NT, t = i / (2 * K), e = i % (2 * K), k = e % K;
      const XFftRows<T, N> row(a, first + t);
      if (!row.ok) continue;
      const C2<T> zk = smem[t * X::S + k], zm = conj(smem[t * X::S + (k == 0 ? 0 : N - k)]);
      row.c[e / K][k] = e < K ? T(0.5) * (zk + zm) : T(0.5) * mul_mi(zk - zm);
    }
    return;
  }
  own_sync();
  if constexpr ((N / E::RL_) % X::TQ == 0) {
    // the thread holds Z[q + TQ j], j < J: only the upper half goes through LDS
    constexpr int J = N / X::TQ, NB = E::LAST_NB;
    auto slot = [](int j) constexpr { return (j % NB) * E::RL_ + j / NB; };
#pragma unroll
    for (int j = J / 2; j < J; ++j) buf[q + X::TQ * j] = v[slot(j)];
    own_sync();
    if (!rows.ok) return;
#pragma unroll
    for (int j = 0; j <= J / 2; ++j) {
      const int k = q + X::TQ * j;
      if (k > N / 2) continue;
      const C2<T> zk = v[slot(j)];
      split(k, zk, conj(k == 0 ? zk : buf[N - k]));
    }
  } else {
#pragma unroll
    for (int s = 0; s < E::LAST_NB * E::RL_; ++s)
      if (E::last_valid(q, s)) buf[E::last_index(q, s)] = v[s];
    own_sync();
    if (!rows.ok) return;
    for (int k = q; k <= N / 2; k += X::TQ) split(k, buf[k], conj(buf[k == 0 ? 0 : N - k]));
  }
}

}  // namespace ps
