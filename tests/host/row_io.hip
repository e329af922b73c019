// Where the engine's row accesses go (RowIO of wave.h, run on the host): values
// stored at the last rows of columns on both sides of a species boundary have to
// appear at their places in an array of FP64 values beside FP32 fields. The
// arrays are mapped without being backed: only the pages touched exist.
//   row_io ny nx nz : a last axis of nz points, inner extent ny nx, two species
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>

#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))
#include "wave.h"

using namespace sfrde;

// An odd axis of 16 blocks as a lane of group g sees it.
struct Axis {
  static constexpr int PG = 4, PR = 1, NBLK = 16, LAYOUT = WL_ODD;
  static constexpr bool EXACT = false;
  using Vals = float[NBLK][4];
  WaveAxis ax;
  int g;
  __host__ __device__ int da() const { return ax.da; }
  __host__ __device__ int n() const { return ax.n; }
  __host__ __device__ static constexpr int seg(int rb) { return 2 * rb >= NBLK ? 1 : 0; }
  __host__ __device__ static constexpr int sb(int rb) { return seg(rb) ? rb - NBLK / 2 : rb; }
  __host__ __device__ int q(int rb, int r) const { return 16 * sb(rb) + r + 4 * g; }
  __host__ __device__ bool vb(int rb, int r) const {
    const WaveSeg& s = seg(rb) ? ax.s1 : ax.s0;
    return q(rb, r) >= s.blo && q(rb, r) < s.bhi;
  }
};

template <typename U>
int check(const Axis& x0, const WaveTiles& tl, const char* what) {
  const long long n = x0.ax.n, total = n * tl.inner;
  const size_t bytes = (size_t)2 * total * sizeof(U);
  void* map = mmap(nullptr, bytes, PROT_READ | PROT_WRITE,
                   MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (map == MAP_FAILED) {
    std::printf("cannot map %zu bytes\n", bytes);
    return 2;
  }
  U* f = static_cast<U*>(map);
  int bad = 0;
  // the tile that holds the last columns of species 0 and the first of species 1
  const int tile = (int)(tl.inner / 16);
  for (int i = 0; i < 16; ++i)
    for (int g = 0; g < 4; ++g) {
      Axis x = x0;
      x.g = g;
      const StridedLane<float> ln(tl, (int)n, tile, i);
      const RowIO<float, Axis> io(x, tl, ln);
      const long long line = 16LL * tile + i;
      const long long col = (line / tl.inner) * total + line % tl.inner;
      for (int rb : {0, 8})
        for (int r = 0; r < 4; ++r) {
          const int q = x.q(rb, r);
          const WaveSeg& s = rb ? x.ax.s1 : x.ax.s0;
          if (q < s.blo || q >= s.bhi) continue;
          const auto of = io.offs(rb);
          U v[4] = {U(1), U(1), U(1), U(1)}, w[4];
          v[r] = U(7 + i);
          // the far end of the line: side b
          const long long at = col + (s.b0 - (long long)x.ax.da * q) * tl.inner;
          io.template store_rmw<1>(f, of.b, v, rb);
          bad += f[at] != U(7 + i);
          f[at] = U(9);
          io.load1(f, of.b, w);
          bad += w[r] != U(9);
          io.store1(f, of.b, v);
          bad += f[at] != U(7 + i);
        }
    }
  munmap(map, bytes);
  std::printf("%s: %d misplaced\n", what, bad);
  return bad ? 1 : 0;
}

int main(int argc, char** argv) {
  if (argc != 4) return 3;
  const long long ny = std::atoll(argv[1]), nx = std::atoll(argv[2]);
  const int n = std::atoi(argv[3]);
  Axis x{};
  const int mid = (n - 1) / 2, qe = (mid + 1) / 2, qo = mid / 2;
  x.ax.n = n;
  x.ax.da = 2;
  x.ax.s0 = WaveSeg{qe + (mid % 2 == 0 ? 1 : 0), 0, qe, 0, n - 1, mid};
  x.ax.s1 = WaveSeg{qo + (mid % 2 == 1 ? 1 : 0), 0, qo, 1, n - 2, mid - 1};
  WaveTiles tl{};
  tl.inner = ny * nx;
  tl.lines = 2 * tl.inner;
  tl.ntiles = (int)((tl.lines + 15) / 16);
  if (!wave_reach_ok(n, tl.inner, sizeof(float))) {
    std::printf("not an engine axis\n");
    return 4;
  }
  return check<float>(x, tl, "fields") | check<double>(x, tl, "FP64 beside FP32");
}
