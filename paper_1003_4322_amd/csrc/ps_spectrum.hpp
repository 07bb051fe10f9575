// ps_spectrum.hpp -- deterministic FP64 shell spectra (energy, enstrophy and
// divergence; MHD energies and cross-helicity).
#pragma once

#include "ps_device.hpp"

namespace ps {

// ---------------------------------------------------------------------------
// Kernel 1 (k_spec_planes): the four rows (+-ky, +-kz) of a row orbit have the
// same shells at every kx, so a mode's terms are first added over the orbit's
// rows (at most four, fewer on the planes 0 and N/2 that are their own mirror
// image) and the shell sums are formed once per orbit.  The shells are cut
// into windows of 64; a workgroup owns one window on one plane pair +-kz, and
// its SPEC_ROWS waves share the window's orbits: wave r visits ky = r,
// r + SPEC_ROWS, ... up to NY/2.  The modes of a row whose shells fall in the
// window form one contiguous kx range (the shell of (kx, ky, kz) does not
// decrease with kx); the wave reads it in chunks of 64 consecutive kx, one
// mode per lane, sums each shell's run by a segmented scan across the lanes
// (DPP moves), and the last lane of a run adds it to the shell's
// Neumaier-compensated sums in LDS.  The waves' partial sums of a shell are
// added in wave order.  Kernel 2 (k_spec_final) adds the plane pairs: 32
// groups of planes, each in plane order, then the groups in order, and the
// totals from the shells, as compensated pairs throughout.  Every
// shell's terms are thus added in one fixed order without atomics, so results
// are bitwise reproducible.
//   energy (Q = 2): E(s) = 1/2 sum w |f|^2 and Z(s) = 1/2 sum w |k|^2 |f|^2
//                   over nf fields, plus max |k_d . f|;
//   MHD    (Q = 3): with u = (z+ + z-)/2, b = (z+ - z-)/2 (fields 0-2, 3-5):
//                   Eu(s) = 1/2 sum w |u|^2, Eb(s) = 1/2 sum w |b|^2,
//                   Hc(s) = 1/2 sum w Re(u . conj b).
// Bound by HBM reads at large boxes and by the latency of one wave's chunks
// at small ones.  Scanning once per orbit instead of once per row, with DPP
// moves instead of shuffles through LDS, took the MHD spectrum of a 512^3 FP32
// state (3.2 GB) from 2.14 to 0.78 ms (4.1 TB/s), the final sums over several
// workgroups from 0.126 to about 0.01 ms of it; NS 512^3 FP32 1.99 -> 0.42 ms,
// MHD 384^3 FP64 1.39 -> 0.66 ms, NS 32^3 FP64 18 -> 11 us.
// ---------------------------------------------------------------------------
constexpr int SPEC_ROWS = 8;     // waves per workgroup of k_spec_planes
constexpr int SPEC_WIN = 64;     // shells per window
constexpr int SPEC_MAXWIN = 16;  // windows at most (nshell <= 1024)
constexpr int SPEC_NF = 6;       // fields a spectrum reads at most

struct NSum {
  double s, c;
};
__device__ __forceinline__ void nadd(NSum& a, double x) {
  const double t = a.s + x;
  if (fabs(a.s) >= fabs(x))
    a.c += (a.s - t) + x;
  else
    a.c += (x - t) + a.s;
  a.s = t;
}
// another compensated sum
__device__ __forceinline__ void nadd(NSum& a, const NSum& b) {
  nadd(a, b.s);
  a.c += b.c;
}

template <typename T>
struct SpecArgs {
  const C2<T>* f;
  double* part;     // [nz/2 + 1][nshell][Q] per plane pair
  double* pmax;     // [nz/2 + 1][windows] max |k_d . f| (energy spectrum only)
  long fs, pitch;   // field stride, kx pitch
  int nx, ny, nz, nf, nshell;
  double sx, sy, sz;  // box factors 2 pi / L (enstrophy and divergence; shells stay on the index)
};

__host__ __device__ constexpr int spec_windows(int nshell) { return (nshell + SPEC_WIN - 1) / SPEC_WIN; }

// floor(sqrt(n)) and ceil(sqrt(n)) for 0 <= n < 2^24 (exact in float; the
// root's last place is settled in integers)
__device__ __forceinline__ int isqrt24(int n) {
  int r = (int)sqrtf((float)n);
  r -= r * r > n;
  r += (r + 1) * (r + 1) <= n;
  return r;
}
// shell of |k|^2 = k2 < 2^22: the smallest s with 4 k2 < (2 s + 1)^2
__device__ __forceinline__ int shell_of_k2(int k2) { return (isqrt24(4 * k2) + 1) >> 1; }

// x of the lane that DPP control C names, old where there is none
template <int C, int ROWS>
__device__ __forceinline__ int dpp_i(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, C, ROWS, 0xf, false);
}
template <int C, int ROWS>
__device__ __forceinline__ double dpp_d(double x) {
  const int2 v = __builtin_bit_cast(int2, x);
  const int2 r{dpp_i<C, ROWS>(0, v.x), dpp_i<C, ROWS>(0, v.y)};
  return __builtin_bit_cast(double, r);
}
// one step of the inclusive segmented scan: add the named lane's running sums
// where its segment (sh) is this lane's
template <int C, int ROWS, int Q>
__device__ __forceinline__ void seg_step(double (&v)[Q], int sh) {
  const bool same = dpp_i<C, ROWS>(-1, sh) == sh;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const double d = dpp_d<C, ROWS>(v[q]);
    v[q] += same ? d : 0.0;
  }
}
// inclusive segmented scan over a wave; equal sh are contiguous, sh >= 0
template <int Q>
__device__ __forceinline__ void seg_scan(double (&v)[Q], int sh) {
  seg_step<0x111, 0xf>(v, sh);  // row_shr:1, 2, 4, 8 inside rows of 16 lanes
  seg_step<0x112, 0xf>(v, sh);
  seg_step<0x114, 0xf>(v, sh);
  seg_step<0x118, 0xf>(v, sh);
  seg_step<0x142, 0xa>(v, sh);  // row_bcast:15 into rows 1 and 3
  seg_step<0x143, 0xc>(v, sh);  // row_bcast:31 into rows 2 and 3
}

// NF: fields read at most; FULL: a.nf == NF, so every load is unconditional.
// A chunk's time is a chain of memory latency, scan and LDS sums; with FP32
// fields the registers hold the next chunk's loads while this one is summed
// (FP64 chunks are twice as large, and a second one would cost occupancy).
template <typename T, bool MHD, int NF, bool FULL>
__global__ __launch_bounds__(SPEC_ROWS * 64, 4) void k_spec_planes(SpecArgs<T> a) {
  constexpr int Q = MHD ? 3 : 2;
  constexpr bool AHEAD = sizeof(T) == 4 && (MHD || NF == 3);  // six fields with divergences: no registers left
  const int NX = a.nx, NY = a.ny, NZ = a.nz, H = NX / 2 + 1;
  const int nwin = spec_windows(a.nshell);
  const int lane = threadIdx.x % 64, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int plane = blockIdx.x / nwin, win = blockIdx.x % nwin;  // plane pair kz = +-plane
  const bool two_z = plane > 0 && 2 * plane < NZ;
  const int z2 = plane * plane;
  const double qz2 = a.sz * a.sz * (double)z2;
  const double kzd = 2 * plane == NZ ? 0.0 : a.sz * plane;
  const int nf = FULL ? NF : a.nf;
  __shared__ NSum acc[SPEC_ROWS][SPEC_WIN][Q];
  __shared__ double red[SPEC_ROWS * 64];
  NSum(*sg)[Q] = acc[wv];
#pragma unroll
  for (int q = 0; q < Q; ++q) sg[lane][q] = NSum{0, 0};
  wave_lds_sync();
  double mx = 0;
  // shells s0 .. s1 of the window: 4|k|^2 in [lo2, hi2)
  const int s0 = SPEC_WIN * win, s1 = min(s0 + SPEC_WIN - 1, a.nshell - 1);
  const int lo2 = (2 * s0 - 1) * (2 * s0 - 1), hi2 = (2 * s1 + 1) * (2 * s1 + 1);
  const long zrow[2] = {(long)plane * NY, (long)(two_z ? NZ - plane : plane) * NY};
  // the wave's chunks in order: orbit iy (its kx range up to kx1, A = iy^2 +
  // plane^2), first kx base; uniform over the wave
  struct Cur {
    int iy, base, kx1, A;
  };
  auto advance = [&](Cur& c) -> bool {
    c.base += 64;
    while (c.base > c.kx1) {
      c.iy += SPEC_ROWS;
      if (2 * c.iy > NY) return false;
      c.A = c.iy * c.iy + z2;
      const int A4 = 4 * c.A;
      if (A4 >= hi2) return false;  // so for every larger iy
      // smallest kx with 4 kx^2 >= lo2 - A4, largest with 4 kx^2 < hi2 - A4
      c.base = s0 > 0 && lo2 - A4 > 0 ? __builtin_amdgcn_readfirstlane((isqrt24(lo2 - A4 - 1) + 2) / 2) : 0;
      c.kx1 = min(__builtin_amdgcn_readfirstlane(isqrt24(hi2 - A4 - 1) / 2), H - 1);
    }
    return true;
  };
  // all loads of a chunk; a row that is its own mirror image is read again
  // and its terms are left out of the sums
  auto load = [&](const Cur& c, C2<T>(&x)[4][NF]) {
    const int kxc = min(c.base + lane, c.kx1);
    const int ym = c.iy > 0 && 2 * c.iy < NY ? NY - c.iy : c.iy;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const C2<T>* row = a.f + (zrow[r >> 1] + ((r & 1) ? ym : c.iy)) * a.pitch + kxc;
#pragma unroll
      for (int ff = 0; ff < NF; ++ff) x[r][ff] = ff < nf ? row[ff * a.fs] : zero2<T>();
    }
  };
  auto sum = [&](const Cur& c, const C2<T>(&x)[4][NF]) {
    const int kx = c.base + lane;
    const bool live = kx <= c.kx1;
    const bool two_y = c.iy > 0 && 2 * c.iy < NY;
    const double kyd = 2 * c.iy == NY ? 0.0 : a.sy * c.iy;
    const int sh = live ? shell_of_k2(kx * kx + c.A) : s1 + 1;  // past the window: its own segment
    const double w = !live ? 0.0 : (kx == 0 || 2 * kx == NX) ? 0.5 : 1.0;  // (1/2) * weight
    double v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool on = ((r >> 1) == 0 || two_z) && ((r & 1) == 0 || two_y);
      if constexpr (MHD) {
        double eu = 0, eb = 0, hc = 0;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
          const C2<T> zp = x[r][f], zm = x[r][3 + f];
          const double ux = 0.5 * ((double)zp.x + (double)zm.x), uy = 0.5 * ((double)zp.y + (double)zm.y);
          const double bx = 0.5 * ((double)zp.x - (double)zm.x), by = 0.5 * ((double)zp.y - (double)zm.y);
          eu += ux * ux + uy * uy;
          eb += bx * bx + by * by;
          hc += ux * bx + uy * by;
        }
        v[0] += on ? eu : 0.0;
        v[1] += on ? eb : 0.0;
        v[2] += on ? hc : 0.0;
      } else {
        double e = 0;
#pragma unroll
        for (int ff = 0; ff < NF; ++ff)
          e += (double)x[r][ff].x * (double)x[r][ff].x + (double)x[r][ff].y * (double)x[r][ff].y;
        v[0] += on ? e : 0.0;
        const double kxd = 2 * kx == NX ? 0.0 : a.sx * kx;
        const double ky = (r & 1) ? -kyd : kyd, kz = (r >> 1) ? -kzd : kzd;
#pragma unroll
        for (int ff = 0; ff + 2 < NF; ff += 3) {
          const double dx = kxd * x[r][ff].x + ky * x[r][ff + 1].x + kz * x[r][ff + 2].x;
          const double dy = kxd * x[r][ff].y + ky * x[r][ff + 1].y + kz * x[r][ff + 2].y;
          const double d = dx * dx + dy * dy;
          const bool cnt = live && on && (FULL || ff + 2 < nf);
          mx = cnt && d > mx ? d : mx;  // the largest square; the root is taken once
        }
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = live ? w * v[q] : 0.0;
    if constexpr (!MHD)
      v[1] = (a.sx * a.sx * (double)(kx * kx) + a.sy * a.sy * (double)(c.iy * c.iy) + qz2) * v[0];
    seg_scan(v, sh);
    const int shn = __shfl_down(sh, 1, 64);
    if (live && (lane == 63 || shn != sh)) {  // last lane of its run
#pragma unroll
      for (int q = 0; q < Q; ++q) nadd(sg[sh - s0][q], v[q]);
    }
    wave_lds_sync();
  };
  Cur c{wv - SPEC_ROWS, 0, -1, 0};
  if constexpr (AHEAD) {
    C2<T> x[4][NF], y[4][NF];
    Cur n = c;
    bool have = advance(n);
    if (have) load(n, x);
    while (have) {
      c = n;
      have = advance(n);
      if (have) load(n, y);
      sum(c, x);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ff = 0; ff < NF; ++ff) x[r][ff] = y[r][ff];
    }
  } else {
    while (advance(c)) {
      C2<T> x[4][NF];
      load(c, x);
      sum(c, x);
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < SPEC_WIN * Q; t += SPEC_ROWS * 64) {
    const int l = t % SPEC_WIN, q = t / SPEC_WIN;
    if (s0 + l < a.nshell) {
      NSum sum{0, 0};
#pragma unroll
      for (int r = 0; r < SPEC_ROWS; ++r) nadd(sum, acc[r][l][q].s + acc[r][l][q].c);
      a.part[((long)plane * a.nshell + s0 + l) * Q + q] = sum.s + sum.c;
    }
  }
  if constexpr (!MHD) {
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int w = SPEC_ROWS * 32; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
      __syncthreads();
    }
    if (threadIdx.x == 0) a.pmax[blockIdx.x] = sqrt(red[0]);
  }
}

}  // namespace ps
