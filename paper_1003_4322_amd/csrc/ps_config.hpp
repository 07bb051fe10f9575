// ps_config.hpp -- compile-time launch configurations per transform length.
//
// For each supported length L: the radix schedule of the Stockham engine and
// the number of threads TQ that cooperate on one transform (about eight
// complex values per thread per stage).  For the strided passes, TX is the
// number of adjacent kx columns per workgroup: 16 (128-byte rows) in FP32 and
// 8 in FP64, fewer where the LDS tile L*TX would exceed 64 KB.
#pragma once

#include "ps_device.hpp"

namespace ps {

template <int L>
struct LenCfg;
#define PS_LEN(L_, TQ_, ...)                     \
  template <>                                    \
  struct LenCfg<L_> {                            \
    using RL = Radices<__VA_ARGS__>;             \
    static constexpr int TQ = TQ_;               \
  };
PS_LEN(4, 1, 4)
PS_LEN(6, 1, 3, 2)
PS_LEN(8, 1, 8)
PS_LEN(12, 3, 4, 3)
PS_LEN(16, 4, 4, 4)
PS_LEN(24, 3, 8, 3)
PS_LEN(32, 4, 8, 4)
PS_LEN(48, 6, 4, 4, 3)
PS_LEN(64, 8, 8, 8)
PS_LEN(96, 12, 8, 4, 3)
PS_LEN(128, 16, 8, 4, 4)
PS_LEN(192, 24, 8, 8, 3)
PS_LEN(256, 32, 8, 8, 4)
PS_LEN(384, 48, 8, 4, 4, 3)
PS_LEN(512, 64, 8, 8, 8)
PS_LEN(768, 96, 8, 8, 4, 3)
PS_LEN(1024, 128, 8, 8, 4, 4)

// Alternate schedules with radix-16 stages (fewer LDS exchanges, 16 values
// per thread), used by the kernel variants for N >= 256.
template <int L>
struct LenAlt : LenCfg<L> {};
#define PS_ALT(L_, TQ_, ...)                     \
  template <>                                    \
  struct LenAlt<L_> {                            \
    using RL = Radices<__VA_ARGS__>;             \
    static constexpr int TQ = TQ_;               \
  };
PS_ALT(128, 8, 16, 8)
PS_ALT(192, 12, 16, 4, 3)
PS_ALT(256, 16, 16, 16)
PS_ALT(384, 24, 16, 8, 3)
PS_ALT(512, 32, 16, 8, 4)
PS_ALT(768, 48, 16, 16, 3)
PS_ALT(1024, 64, 16, 8, 8)
#undef PS_ALT

// Wide schedules: a last radix of 4 over twice the threads (four values per
// thread at the end, whole waves for any number of rows at M = 256); product
// pass variants only.
template <int L>
struct LenWide : LenCfg<L> {};
#define PS_WIDE(L_, TQ_, ...)                    \
  template <>                                    \
  struct LenWide<L_> {                           \
    using RL = Radices<__VA_ARGS__>;             \
    static constexpr int TQ = TQ_;               \
  };
PS_WIDE(256, 64, 4, 4, 4, 4)
PS_WIDE(512, 128, 8, 4, 4, 4)
#undef PS_WIDE

#undef PS_LEN

// grid sizes with a compiled configuration
#define PS_FOR_EACH_N(X) \
  X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(384) X(512) X(768) X(1024)

// Tile width of a strided pass: 16 columns (FP32) or 8 (FP64), halved SH
// times, capped by 64 KB of LDS and 1024 threads.
template <typename T, int N, int TQ, int SH>
struct StridedTX {
  static constexpr int TX0 = (sizeof(T) == 4 ? 16 : 8) >> SH;
  static constexpr int TXL = (65536 / (N * 2 * (int)sizeof(T)));
  static constexpr int TX1 = TX0 < TXL ? TX0 : TXL;
  static constexpr int TX2 = (TX1 * TQ > 1024) ? 1024 / TQ : TX1;
  static constexpr int value = TX2 < 1 ? 1 : TX2;
};

constexpr bool has_variants(int N) { return N >= 256; }

// x passes: rows live in LDS with the padded layout (pad8, M + M/8 + 1 slots)
// or, in the fused pass's swizzled variants, LaySwz32 (32 (M/32 + 1) slots);
// the fused pass also stages twiddles (2M values).
template <typename T, int M, int TQ>
struct XCfg {
  // LDS slots per row: the larger of the padded and swizzled layouts
  static constexpr int SLOTS = (M + M / 8 + 1) > 32 * (M / 32 + 1) ? (M + M / 8 + 1) : 32 * (M / 32 + 1);
  // lim: LDS bytes per workgroup (64 KB; 80 KB for two workgroups per CU)
  static constexpr bool fits(int f, int rb, int lim = 65536) {
    return (f * rb * SLOTS + 2 * M) * 2 * (int)sizeof(T) <= lim && f * rb * TQ <= 1024;
  }
  static constexpr int rb(int f, int want, int lim = 65536) {
    int r = want < 1 ? 1 : want;
    while (r > 1 && !fits(f, r, lim)) r >>= 1;
    return r;
  }
  static constexpr bool MHD_OK = fits(12, 1, 65536);
  // launch limits alone: 1024 threads and the 160 KB of LDS a gfx950
  // workgroup may hold (rows that overflow 64 KB cost occupancy, not
  // correctness)
  static constexpr bool launchable(int f) {
    return (f * SLOTS + 2 * M) * 2 * (int)sizeof(T) <= 163840 && f * TQ <= 1024;
  }
};

// Packed x pass (k_x_prod_pk): W = max(ceil(FIN rb / 2), ceil(FOUT rb / 2))
// complex transforms of length N, TQ threads each; LDS of W rows of `slots`
// plus N staged twiddles.
// lp: LDS slots per transform.
template <typename T, int N, int TQ>
struct XPkCfg {
  static constexpr int w(int fin, int fout, int rb) {
    const int a = (fin * rb + 1) / 2, b = (fout * rb + 1) / 2;
    return a > b ? a : b;
  }
  static constexpr bool fits(int fin, int fout, int rb, int lp, int lim) {
    return (w(fin, fout, rb) * lp + N) * 2 * (int)sizeof(T) <= lim && w(fin, fout, rb) * TQ <= 1024;
  }
  // an even number of grid rows, so that every transform pairs one field on
  // two grid rows (two different fields, such as u and its curl, can differ
  // in size by |k|, and the smaller would carry the larger one's rounding)
  static constexpr int rb(int fin, int fout, int want, int lp, int lim) {
    int r = 2;
    while (2 * r <= want) r *= 2;  // a power of two, at least 2
    while (r > 2 && !fits(fin, fout, r, lp, lim)) r >>= 1;
    return r;
  }
};

// Kernel variant tables.  Strided-pass variants: tile shift, z_curl split and
// direct gather, minimum workgroups per CU asked of the register allocator,
// alternate (radix-16) schedule.  Product-pass variants: rows per workgroup,
// schedule.
struct ZV {
  int sh;       // tile width shift
  int split;    // z_curl: workgroups per tile sharing the output groups (1, 2 or 4; NS caps at 2);
                // z_epi: 2 = z+ and z- updated by two workgroups (Elsasser form only)
  int minb;     // workgroups per CU the register allocator must leave room for (1: no request)
  bool alt;     // radix-16 schedule
  bool direct;  // z_curl: gather inputs per output field instead of holding them in registers
  bool wide = false;  // wide schedule (LenWide: a last radix of 4 over twice the threads)
  bool tws = false;   // strided passes: twiddles staged in LDS beside the tile
  bool tile = false;  // z_epi: fields combined and in LDS side by side, in two groups (k_z_epi_tile)
};
struct XV {
  int rb_ns, rb_mhd;  // rows per workgroup (reduced while the LDS tile would not fit)
  int sched;          // 0 LenCfg, 1 radix-16 (LenAlt), 2 wide (LenWide)
  bool swz;           // rows in LDS swizzled (LaySwz32) instead of padded (LayPad8)
  bool big = false;   // up to 80 KB of LDS per workgroup (two per CU) instead of 64 KB
  bool pk = false;    // packed form (k_x_prod_pk): two real rows per complex transform of length N
  bool ex = false;    // packed form: per-exchange LDS layouts (LayEx) and rows in natural order
  bool pr = false;    // packed form on dealiased input (kx <= (N - 1) / 3): the slots of
                      // zeros and of unread outputs skipped (falls back when kmax is larger)
};
constexpr ZV ZCURL_V[] = {{1, 1, 1, false, false}, {1, 2, 1, false, false}, {1, 2, 2, false, false},
                          {1, 2, 1, true, false},  {1, 1, 1, false, true},  {0, 2, 1, true, false},
                          {0, 1, 1, true, false}};
constexpr ZV ZEPI_V[] = {{0, 1, 1, false}, {1, 1, 1, false}, {1, 1, 2, false}, {1, 1, 1, true},
                         {2, 1, 1, false}, {1, 2, 1, false}, {1, 2, 2, false}, {2, 2, 1, false},
                         {0, 1, 1, false, false, true}, {1, 1, 1, false, false, true},
                         {1, 1, 2, false, false, true}, {2, 1, 1, false, false, true},
                         {0, 1, 1, true, false, false, false, true}};
constexpr ZV STR_V[] = {{0, 1, 1, false}, {1, 1, 1, false}, {0, 1, 1, true}, {1, 1, 1, true},
                        {0, 1, 1, true, false, false, true}, {0, 1, 1, false, false, false, true}};
constexpr XV XPROD_V[] = {{2, 1, 0, false}, {4, 2, 0, false}, {4, 2, 1, false}, {2, 1, 1, false},
                          {2, 1, 0, true},  {4, 2, 0, true},  {1, 1, 2, true},  {1, 1, 2, false},
                          {8, 4, 0, true, true}, {8, 4, 0, false, true}, {4, 2, 2, true, true},
                          // packed form
                          {2, 2, 0, false, false, true, true}, {4, 4, 0, false, true, true, true},
                          {2, 2, 0, true, false, true}, {4, 4, 0, true, true, true},
                          {2, 2, 1, false, false, true, true}, {4, 4, 1, false, true, true, true},
                          {8, 8, 0, false, true, true, true},
                          // packed, dealiased input
                          {2, 2, 0, false, false, true, true, true}, {8, 8, 0, false, true, true, true, true},
                          {2, 2, 0, true, false, true, false, true}};
constexpr int NZCURL = sizeof(ZCURL_V) / sizeof(ZV);
// waves per SIMD that minb workgroups of `threads` threads occupy (4 SIMDs per CU)
constexpr int waves_per_simd(int minb, int threads) {
  const int w = minb * ((threads + 63) / 64) / 4;
  return w < 1 ? 1 : w;
}
constexpr int NZEPI = sizeof(ZEPI_V) / sizeof(ZV);
constexpr int NSTR = sizeof(STR_V) / sizeof(ZV);
constexpr int NXPROD = sizeof(XPROD_V) / sizeof(XV);

// The variant each pass runs with by default: where nothing else is compiled
// (lengths below 256) and on a plan that has been neither tuned nor set.
// Chosen by the length n of the axis the pass transforms, the type, the form and
// the size of the class of boxes (points: columns the z pass transforms times n;
// rows: grid rows), by timing the variants at every length from 24 to 512, and
// the candidates named below at 768 and 1024, on boxes of 10^3 to 10^8 points
// (launch times, us, former default -> this one; "pr": pruned).
//
// y and z: twiddles staged in LDS beside the tile, radix-8 schedule, except
// FP64 at 384, where radix 16 saves a whole exchange of a 98 KB tile (inverse +
// forward y, NS: FP32 192 108 -> 91, 256 247 -> 234, 384 1164 -> 889, 512 pr
// 1016 -> 953; FP64 192 172 -> 164, 384 1842 -> 1685).
constexpr int pick_strided(bool f32, int n) { return !f32 && n == 384 ? 4 : 5; }
// Products: the packed form wherever its transforms fill the workgroup (NS:
// FP32 192 97 -> 69, 256 229 -> 167, 512 1739 -> 1284; FP64 96 31 -> 25, 128 43
// -> 38, 192 211 -> 141, 256 430 -> 327); with the radix-16 schedule for FP64
// rows of 384 and more (NS 512 3878 -> 2733); the half-length form
// for short rows, MHD rotational FP32 at 384 (2237 -> 1570 with two rows; packed
// 1726) and FP64 at 192 (828, radix 16 packed 874) and 512 (6282; packed 7179), NS
// divergence form FP64 at 512 (4826; radix 16 packed 5431), and beyond 512 where
// the packed transforms of twelve fields would need more than 1024 threads.
// FP64 rows of 128 points by the fields: rotational NS packed radix 16 (128^3 84;
// radix 8 100, half-length 93), but half-length below 6144 rows; the NS
// divergence form half-length (81, packed 87) up to 98304 rows (six boxes 534,
// packed 476); rotational MHD half-length (168; packed 218 and, radix 16, 182), and
// packed radix 16 from 98304 rows on (six boxes 1025 against 1114); a few hundred
// rows packed radix 8 everywhere (NS 384 rows 19.5 against 23).
constexpr int pick_xprod(bool f32, int n, bool mhd, bool els, long rows) {
  const bool rot12 = mhd && !els;
  if (n < 64 || (n == 96 && f32 && els && !mhd)) return 0;
  if (f32) {
    if (n == 384 && mhd) return els ? 15 : 4;
    if (n > 512 && rot12) return 8;
    return 18;
  }
  if (n == 128 && !(els && mhd)) {
    if (rows < (mhd ? 1024 : 2048)) return 18;
    return rows < (mhd || els ? 98304 : 6144) ? 0 : els ? 18 : 15;
  }
  if (rot12) return n >= 512 ? 7 : n == 192 ? 0 : n == 256 ? 15 : 18;
  if (n == 512 && els) return mhd ? 18 : 7;
  return n >= 384 ? 15 : 18;
}
// whether some number of rows has variant i picked
constexpr bool xprod_picked(bool f32, int n, bool mhd, bool els, int i) {
  for (long rows : {0L, 4096L, 1L << 40})
    if (pick_xprod(f32, n, mhd, els, rows) == i) return true;
  return false;
}
// Inverse z + curl: full-width tiles (16 columns in FP32, 8 in FP64) with the
// radix-16 schedule, MHD in two workgroups per tile (NS FP64 256 471 -> 314, 512
// 3039 -> 2441; MHD FP64 192 458 -> 440, 512 7780 -> 6082; Elsasser FP32 256 73 ->
// 56, 512 521 -> 433).  At 128, and at 384 in FP32, that schedule leaves threads
// idle (NS FP64 128 32 against 40, MHD Elsasser FP32 384 208 against 237): there,
// at 48 and 64 in FP32, and for pruned FP64 NS at 96 and 192 (44 against 65) the
// radix-8 schedule, MHD rotational again in two workgroups (FP64 128 113 -> 81;
// FP32 256 461 -> 430, 512 4016 -> 3704).
// Few columns leave full-width tiles too few waves: NS boxes of fewer points run
// half-width tiles with the radix-8 schedule (FP64 256 points, 3456 columns 68 us
// against 91, at 12672 297 against 256; 512, 1600 columns FP32 40 against 57), in
// the divergence form, which loads half as much, below a million or so (FP64
// 384, 360 columns 30 against 33, 4312 88 against 79); below 96 points 32768
// columns are the line (512 x 384 x 8 MHD FP64, 98688 columns 896 against 313).
// FP64 columns of 768 fit in 64 KB five at a time, which splits every row's cache
// lines: four instead (NS 3824 -> 1775; MHD divergence form 4286 -> 2449), but two
// workgroups a tile while MHD columns are few (rotational 216: 141 -> 85, 1600:
// 367 -> 308).  MHD at 1024: two workgroups (FP32 rotational)
// and at 128 (FP64 divergence form) only while columns are few (1024: 216 152 ->
// 121, 24768 4650 -> 3903; 128: 1600 32 -> 27, 8320 132 -> 103).
constexpr int pick_zcurl(bool f32, int n, bool mhd, bool els, bool prune, long points) {
  const bool rot12 = mhd && !els;
  if (n < 96 && points / n <= 32768) return 0;
  const long few = !els ? (n == 384 ? 3200000 : 2450000) : f32 && n > 192 ? 1500000 : 1000000;
  if (n >= 96 && !mhd && points < few) return 0;
  if (n == 768 && !f32) return mhd && points < 1500000 ? 5 : 0;
  if (n == 1024 && f32 && rot12) return points < 1000000 ? 2 : 0;
  if (n == 128 && !f32 && mhd && els) return points < 640000 ? 1 : 0;
  if (f32) {
    if (n == 48 || n == 64 || n == 384 || n == 768) return 0;
    if (n == 128) return rot12 ? 1 : mhd ? 5 : 0;
    if (rot12) return n == 192 ? 0 : n >= 256 ? 2 : 5;
    return mhd ? 5 : 6;
  }
  if (n == 128) return mhd ? 1 : 0;
  if (!mhd && (n == 96 || (n == 192 && prune))) return 0;
  return mhd ? 5 : 6;
}
// whether some pruning and size have variant i picked
constexpr bool zcurl_picked(bool f32, int n, bool mhd, bool els, int i) {
  for (long points : {0L, 800000L, 1200000L, 2000000L, 3000000L, 1L << 40})
    if (pick_zcurl(f32, n, mhd, els, false, points) == i || pick_zcurl(f32, n, mhd, els, true, points) == i)
      return true;
  return false;
}
// Forward z + epilogue: full-width tiles with plain register use (NS FP32 256
// 209 -> 192, 384 pr 333 -> 251, FP64 512 3145 -> 2934); the wide schedule where
// the accumulators of the Elsasser form or twelve fields crowd the registers
// (MHD 512: Elsasser FP32 1123 -> 1036, FP64 2296 -> 1950; rotational FP64 7561 ->
// 7009); half-width tiles at 192 in FP32 (NS pr 41 -> 29) and for the NS
// divergence form at 256 and 512; z+ and z- in two workgroups for Elsasser
// fields at 192 in FP32 (71 -> 65); half-width tiles for
// MHD at 768 and 1024 (MHD 64 x 96 x 768 FP32, a step: 1262 against 1384 with the
// wide schedule; Elsasser with z+ and z- in two workgroups, 96 x 384 x 768 FP32
// pr 829 against 1789, 48 x 64 x 1024 118 against 217).
// The fields of a tile side by side (12) for MHD at 384 and, Elsasser, 512
// (k_z_epi_tile's comment has both sides), except where its tiles leave CUs idle
// (48 x 64 x 512 Elsasser FP32 102 against 156; 48 x 64 x 384 rotational 75
// against 107, at 16 x 24 columns 71 against 59 for the side-by-side tiles).
// Half-width tiles, two workgroups a CU, up to 512 where points are few (NS FP32
// 512 40 -> 46 us with full width, 384 pr up to 4 M points 71 -> 84; FP64 MHD
// rotational at 384 66 -> 104) and for large boxes of the NS divergence form in
// FP32 (512^3 pr, two launches, 995 against 1252 with the wide schedule).
constexpr int pick_zepi(bool f32, int n, bool mhd, bool els, bool prune, long points) {
  const bool mid = points >= 300000 && points < 1500000;
  if (n < 256) {
    if (mhd && els) return n == 192 ? 5 : 0;
    return f32 && n == 192 ? 1 : !f32 && mhd && n == 96 ? 1 : 0;
  }
  if (mhd && els) return n == 256 ? (f32 ? 9 : 8) : n >= 768 || (n == 512 && mid) ? 5 : 12;
  if (mhd && n == 384) return f32 ? (mid ? 5 : 12) : points < 3300000 ? 5 : 0;
  if (mhd) return n >= 768 ? 5 : n == 512 && !f32 ? 9 : 8;
  if (f32 && els && n != 384) return n > 512 ? 0 : points < 1000000 || (n == 256 && !prune) ? 9 : 2;
  return n <= 512 && points < (n != 384 ? 1200000 : !els ? 4000000 : f32 ? 700000 : 1200000) ? 2 : 0;
}

// Lengths below 256: k_z_epi_tile's groups (0: k_z_epi instead) and columns per
// tile, for the divergence forms where the columns are too many for
// k_z_epi_field (16 columns of 96 or 128 FP32 points in two groups still leave
// two workgroups per CU: 8 boxes of MHD 96^3 47 us against 52 with 8 columns).
struct EpiTilePick {
  int groups, tx;
};
constexpr EpiTilePick pick_epi_tile(bool f32, int n, bool mhd, bool els) {
  if (!els || n < 96 || n > 192 || (n == 192 && (!mhd || f32))) return {0, 0};
  if (n == 96 && !mhd) return {1, 8};
  return {2, f32 ? 16 : 8};
}

}  // namespace ps
