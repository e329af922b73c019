// The tiles that the waves of a launch take (WaveRun of wave.h, run on the host):
// every tile once, and in each block as many barriers from every wave, those of its
// own rounds and those it drains together. The loop is that of the kernels.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))
#include "wave.h"

using namespace sfrde;

int main() {
  int bad = 0;
  long long launches = 0;
  auto check = [&](int ntiles, int sweep, int grid, int waves) {
    ++launches;
    std::vector<int> seen(ntiles, 0);
    for (int b = 0; b < grid; ++b) {
      int barriers = -1;
      for (int w = 0; w < waves; ++w) {
        WaveRun run(ntiles, sweep, b, grid, w, waves);
        const int r0 = run.rounds;
        int n = 0;
        for (int tile = run.t; tile < run.t1;) {
          if (run.rounds > 0) ++n;  // sync()
          if (tile < 0 || tile >= ntiles) ++bad;
          else ++seen[tile];
          tile += run.step();
          run.done();
        }
        if (r0 > 0 && run.rounds < 0) ++bad;  // more tiles than rounds
        if (run.rounds > 0) n += run.rounds;  // drain()
        if (barriers < 0) barriers = n;
        bad += n != barriers;
      }
    }
    for (int s : seen) bad += s != 1;
    if (bad) std::printf("ntiles %d sweep %d grid %d waves %d\n", ntiles, sweep, grid, waves);
  };
  for (int waves : {4, 8})
    for (int sweep : {0, 1})
      for (int grid : {1, 2, 3, 7, 16, 255, 256, 512})
        for (int k = 0; k < 40 && !bad; ++k) {
          const int all = grid * waves;
          const int n[] = {1 + k, all - 3 + k, 2 * all + 17 * k, 3 * all + all / 2 + k,
                           (int)((k + 1) * 2654435761u % 9973u) + 1};
          for (int v : n)
            if (v > 0) check(v, sweep, grid, waves);
        }
  std::printf("%lld launches, %d wrong\n", launches, bad);
  return bad ? 1 : 0;
}
