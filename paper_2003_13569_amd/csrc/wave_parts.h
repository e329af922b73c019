// The size classes of the wave engine (wave.h). A class NB holds axes of up to
// 32 NB points (n odd: 32 NB - 1, periodic: 32 NB - 1); FP64 classes of 5 to 8
// blocks those that fill all of them (wave_full). The library is built
// from one translation unit per class (wave_part.hip with SFRDE_PART) and the
// host code (SFRDE_IN_PARTS). sfrde.hip alone, without either, holds none of them:
// a build for checks of the host code, which refuses plans with engine axes (all
// classes in one unit take a quarter of an hour to compile).
#pragma once

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
