// The size classes of the wave engine (wave.h). A class NB holds axes of up to
// 32 NB points (n odd: 32 NB - 1, periodic: 32 NB - 1); FP64 classes of 5 to 8
// blocks those that fill all of them (wave_full). The library is built
// from one translation unit per class (wave_part.hip with SFRDE_PART) and the
// host code (SFRDE_IN_PARTS). sfrde.hip alone, without either, holds none of them:
// a build for checks of the host code, which refuses plans with engine axes (all
// classes in one unit take a quarter of an hour to compile).
#pragma once

#include "../../include/sfrde.h"
#include "wave.h"

namespace sfrde {

enum {
  WC_F32_2X, WC_F32_2E, WC_F32_2O, WC_F32_4X, WC_F32_4E, WC_F32_4O,
  WC_F32_8X, WC_F32_8E, WC_F32_8O, WC_F64_2X, WC_F64_2E, WC_F64_2O,
  WC_F64_4X, WC_F64_4E, WC_F64_4O, WC_F64_8X, WC_F64_8O, WC_F64_9E,
  WC_F32_6X, WC_F32_16E, WC_F32_16O, WC_F64_16E, WC_F64_16O,
  WC_F64_5E, WC_F64_6E, WC_F64_7E, WC_F64_8E, WC_F64_6O,
  WC_COUNT
};

// Size class of an axis, -1 if the engine has none.
inline int wave_class_of(int dtype, int bc, long long n, bool source) {
  // the one-point padding axis of a 1D plan has no transform (k_zpoint; as a
  // product with the identity it rounded FP32 values to two binary16 terms)
  if (n == 1) return -1;
  const bool per = bc == SFRDE_BC_PERIODIC, f32 = dtype == SFRDE_F32;
  const long long half = per ? n / 2 + 1 : (n + 1) / 2;  // positions of an even axis
  const bool odd = !per && n % 2 == 1;
  const int c2 = f32 ? WC_F32_2X : WC_F64_2X, c4 = f32 ? WC_F32_4X : WC_F64_4X;
  const int lay = odd ? 2 : 1;
  // exact classes, multiples of 64 points: no index of theirs is checked or clamped,
  // and the last axis has register order (they have no kernel for manufactured
  // sources). 192^3 FP32 in its own class / in the 8-block one: 604 / 835 us a step,
  // 192^2 65 / 74; FP64 192 points have the 6-block class without padding
  if (!per && !source && n == 64) return c2;
  if (!per && !source && n == 128) return c4;
  if (!per && !source && n == 192 && f32) return WC_F32_6X;
  if (!per && !source && n == 256) return f32 ? WC_F32_8X : WC_F64_8X;
  if (half <= 32) return c2 + lay;
  if (half <= 64) return c4 + lay;
  if (f32 && half <= 128) return WC_F32_8X + lay;
  // periodic axes of 256 points run as FFTs (as those of 512 and 1024, which have no
  // class): launches of 256^2 FP64, products / FFT: X 26.8 / 8.1, Z 25.2 / 8.5 us
  if (per && n == 256) return -1;
  if (!f32 && half <= (odd ? 128 : 144)) {  // the class whose blocks the axis fills
    if (odd) return (n - 1) / 2 / 2 + 1 <= 48 ? WC_F64_6O : WC_F64_8O;  // points of segment 0
    return half <= 80 ? WC_F64_5E : half <= 96 ? WC_F64_6E : half <= 112 ? WC_F64_7E
         : half <= 128 ? WC_F64_8E : WC_F64_9E;
  }
  // to 512 points on the group kernels (launches of the dense kernels / these: 300 x
  // 333 FP32 X 351 / 14.4, Z 289 / 16.2 us, 390 points FP64 Z 485 / 48, 512^2
  // Dirichlet FP32 X 630 / 19, Z 611 / 20); beyond, the matrix of an axis leaves the
  // caches
  if (half > 256) return -1;
  return (f32 ? WC_F32_16E : WC_F64_16E) + (odd ? 1 : 0);
}

// The engine's view of an axis: segments of pair positions (wave.h).
inline WaveAxis wave_axis(int bc, long long n) {
  WaveAxis x{};
  x.n = (int)n;
  x.periodic = bc == SFRDE_BC_PERIODIC;
  auto blocks = [](int c) { return (c + 15) / 16; };
  if (x.periodic) {
    const int half = (int)(n / 2) + 1;  // p = 0 .. n/2
    x.da = 1;
    x.s0 = WaveSeg{half, 1, (int)((n + 1) / 2), 0, (int)n, 0};
    if (n % 2 == 1) x.s0.ca = (int)((n + 1) / 2);
    x.nb = blocks(x.s0.ca);
  } else if (n % 2 == 0) {
    const int half = (int)(n / 2);
    x.da = 2;
    x.s0 = WaveSeg{half, 0, half, 0, (int)n - 1, half - 1};
    x.nb = blocks(half);
  } else {
    const int mid = (int)((n - 1) / 2);  // pairs; the middle index
    const int qe = (mid + 1) / 2, qo = mid / 2;
    x.da = 2;
    x.s0 = WaveSeg{qe + (mid % 2 == 0 ? 1 : 0), 0, qe, 0, (int)n - 1, mid};
    x.s1 = WaveSeg{qo + (mid % 2 == 1 ? 1 : 0), 0, qo, 1, (int)n - 2, mid - 1};
    x.nb = blocks(x.s0.ca);
    x.nb1 = blocks(x.s1.ca);
  }
  return x;
}

#if defined(SFRDE_PART) || defined(SFRDE_IN_PARTS)
template <int C>
WaveKernels wave_class();
#else
template <int C>
WaveKernels wave_class() {
  return WaveKernels{};
}
#endif

#define SFRDE_WAVE_CLASS(C, T, NB, LAY) \
  template <>                           \
  WaveKernels wave_class<C>() {         \
    return wave_kernels<T, NB, LAY>();  \
  }
#if defined(SFRDE_PART)
#define SFRDE_HAS(C) (SFRDE_PART == C)
#else
#define SFRDE_HAS(C) 0
#endif
#if SFRDE_HAS(0)
SFRDE_WAVE_CLASS(WC_F32_2X, float, 2, WL_EXACT)
#endif
#if SFRDE_HAS(1)
SFRDE_WAVE_CLASS(WC_F32_2E, float, 2, WL_EVEN)
#endif
#if SFRDE_HAS(2)
SFRDE_WAVE_CLASS(WC_F32_2O, float, 2, WL_ODD)
#endif
#if SFRDE_HAS(3)
SFRDE_WAVE_CLASS(WC_F32_4X, float, 4, WL_EXACT)
#endif
#if SFRDE_HAS(4)
SFRDE_WAVE_CLASS(WC_F32_4E, float, 4, WL_EVEN)
#endif
#if SFRDE_HAS(5)
SFRDE_WAVE_CLASS(WC_F32_4O, float, 4, WL_ODD)
#endif
#if SFRDE_HAS(6)
SFRDE_WAVE_CLASS(WC_F32_8X, float, 8, WL_EXACT)
#endif
#if SFRDE_HAS(7)
SFRDE_WAVE_CLASS(WC_F32_8E, float, 8, WL_EVEN)
#endif
#if SFRDE_HAS(8)
SFRDE_WAVE_CLASS(WC_F32_8O, float, 8, WL_ODD)
#endif
#if SFRDE_HAS(9)
SFRDE_WAVE_CLASS(WC_F64_2X, double, 2, WL_EXACT)
#endif
#if SFRDE_HAS(10)
SFRDE_WAVE_CLASS(WC_F64_2E, double, 2, WL_EVEN)
#endif
#if SFRDE_HAS(11)
SFRDE_WAVE_CLASS(WC_F64_2O, double, 2, WL_ODD)
#endif
#if SFRDE_HAS(12)
SFRDE_WAVE_CLASS(WC_F64_4X, double, 4, WL_EXACT)
#endif
#if SFRDE_HAS(13)
SFRDE_WAVE_CLASS(WC_F64_4E, double, 4, WL_EVEN)
#endif
#if SFRDE_HAS(14)
SFRDE_WAVE_CLASS(WC_F64_4O, double, 4, WL_ODD)
#endif
#if SFRDE_HAS(15)
SFRDE_WAVE_CLASS(WC_F64_8X, double, 8, WL_EXACT)
#endif
#if SFRDE_HAS(16)
SFRDE_WAVE_CLASS(WC_F64_8O, double, 8, WL_ODD)
#endif
#if SFRDE_HAS(17)
SFRDE_WAVE_CLASS(WC_F64_9E, double, 9, WL_EVEN)
#endif
#if SFRDE_HAS(18)
SFRDE_WAVE_CLASS(WC_F32_6X, float, 6, WL_EXACT)
#endif
#if SFRDE_HAS(19)
SFRDE_WAVE_CLASS(WC_F32_16E, float, 16, WL_EVEN)
#endif
#if SFRDE_HAS(20)
SFRDE_WAVE_CLASS(WC_F32_16O, float, 16, WL_ODD)
#endif
#if SFRDE_HAS(21)
SFRDE_WAVE_CLASS(WC_F64_16E, double, 16, WL_EVEN)
#endif
#if SFRDE_HAS(22)
SFRDE_WAVE_CLASS(WC_F64_16O, double, 16, WL_ODD)
#endif
#if SFRDE_HAS(23)
SFRDE_WAVE_CLASS(WC_F64_5E, double, 5, WL_EVEN)
#endif
#if SFRDE_HAS(24)
SFRDE_WAVE_CLASS(WC_F64_6E, double, 6, WL_EVEN)
#endif
#if SFRDE_HAS(25)
SFRDE_WAVE_CLASS(WC_F64_7E, double, 7, WL_EVEN)
#endif
#if SFRDE_HAS(26)
SFRDE_WAVE_CLASS(WC_F64_8E, double, 8, WL_EVEN)
#endif
#if SFRDE_HAS(27)
SFRDE_WAVE_CLASS(WC_F64_6O, double, 6, WL_ODD)
#endif
#undef SFRDE_HAS
#undef SFRDE_WAVE_CLASS

}  // namespace sfrde
