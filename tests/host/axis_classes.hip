// Every axis of the engine (2 to 512 points) in its size class, on the host: the
// row blocks of a stage combine hold each position, and none of them is padding alone (padding
// repeats the last position of its segment, which has to lie in the same block: a
// wave loads and stores a block at a time, and arrays that are read and written
// would otherwise get the position twice).
#include <hip/hip_runtime.h>

#include <cstdio>

#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))
#include "wave_parts.h"

using namespace sfrde;

int bad = 0, axes = 0;

template <typename T, int NB, int LAY>
void check(int bc, int n) {
  using XF = WaveXf<T, NB, LAY>;
  const WaveAxis x = wave_axis(bc, n);
  auto wrong = [&](const char* what) {
    ++bad;
    std::printf("%s: bc %d n %d, %d blocks, layout %d, FP%d\n", what, bc, n, NB, LAY,
                (int)sizeof(T) * 8);
  };
  ++axes;
  int seen[2] = {0, 0};
  const int ca[2] = {x.s0.ca, XF::ODD ? x.s1.ca : 0};
  for (int rb = 0; rb < NB; ++rb) {
    if (!XF::block_own(rb, x.nb, x.nb1)) continue;
    const int s = XF::seg(rb), first = 16 * XF::sb(rb);
    if (first >= ca[s]) wrong("a block of padding alone");
    if (first != seen[s]) wrong("blocks out of order");
    seen[s] = first + 16 < ca[s] ? first + 16 : ca[s];
  }
  for (int s = 0; s < 2; ++s)
    if (seen[s] != ca[s]) wrong("positions left out");
  if (XF::EXACT && n != 32 * NB) wrong("not an exact axis");
}

void check_class(int c, int bc, int n) {
  switch (c) {
    case WC_F32_2X: return check<float, 2, WL_EXACT>(bc, n);
    case WC_F32_2E: return check<float, 2, WL_EVEN>(bc, n);
    case WC_F32_2O: return check<float, 2, WL_ODD>(bc, n);
    case WC_F32_4X: return check<float, 4, WL_EXACT>(bc, n);
    case WC_F32_4E: return check<float, 4, WL_EVEN>(bc, n);
    case WC_F32_4O: return check<float, 4, WL_ODD>(bc, n);
    case WC_F32_6X: return check<float, 6, WL_EXACT>(bc, n);
    case WC_F32_8X: return check<float, 8, WL_EXACT>(bc, n);
    case WC_F32_8E: return check<float, 8, WL_EVEN>(bc, n);
    case WC_F32_8O: return check<float, 8, WL_ODD>(bc, n);
    case WC_F32_16E: return check<float, 16, WL_EVEN>(bc, n);
    case WC_F32_16O: return check<float, 16, WL_ODD>(bc, n);
    case WC_F64_2X: return check<double, 2, WL_EXACT>(bc, n);
    case WC_F64_2E: return check<double, 2, WL_EVEN>(bc, n);
    case WC_F64_2O: return check<double, 2, WL_ODD>(bc, n);
    case WC_F64_4X: return check<double, 4, WL_EXACT>(bc, n);
    case WC_F64_4E: return check<double, 4, WL_EVEN>(bc, n);
    case WC_F64_4O: return check<double, 4, WL_ODD>(bc, n);
    case WC_F64_5E: return check<double, 5, WL_EVEN>(bc, n);
    case WC_F64_6E: return check<double, 6, WL_EVEN>(bc, n);
    case WC_F64_6O: return check<double, 6, WL_ODD>(bc, n);
    case WC_F64_7E: return check<double, 7, WL_EVEN>(bc, n);
    case WC_F64_8X: return check<double, 8, WL_EXACT>(bc, n);
    case WC_F64_8E: return check<double, 8, WL_EVEN>(bc, n);
    case WC_F64_8O: return check<double, 8, WL_ODD>(bc, n);
    case WC_F64_9E: return check<double, 9, WL_EVEN>(bc, n);
    case WC_F64_16E: return check<double, 16, WL_EVEN>(bc, n);
    case WC_F64_16O: return check<double, 16, WL_ODD>(bc, n);
  }
  ++bad;
  std::printf("class %d is not checked\n", c);
}

int main() {
  for (int dtype : {SFRDE_F32, SFRDE_F64})
    for (int bc = 0; bc < 3; ++bc)
      for (int n = 2; n <= 1024; ++n)
        for (bool source : {false, true}) {
          const int c = wave_class_of(dtype, bc, n, source);
          if (c >= 0) check_class(c, bc, n);
        }
  std::printf("%d axes, %d wrong\n", axes, bad);
  return bad ? 1 : 0;
}
