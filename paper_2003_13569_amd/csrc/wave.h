// Per-axis transforms in the registers of one wavefront (gfx950 MFMA).
//
// A wavefront takes 16 lines of one axis (16 columns of the product M x) and
// keeps all of their points in registers from the load to the store: loads,
// fold, products, the pointwise stage, the next fold and products, stores.
// The only data shared by the waves of a block is the axis matrix, which sits
// in LDS (read-only after one barrier), so the waves of a CU run independent
// of one another and hide each other's latencies.
//
// That works because the matrix cores' result layout can be read as the next
// product's operand. Lane l = 16 g + i holds column i; register r of row
// block rb holds position
//   FP32 (16x16x32 f16):  16 rb + 4 g + r,   FP64 (16x16x4 f64):  16 rb + 4 r + g,
// and the operand of the next product takes its k index from the same (rb,
// g, r): for FP64 k-step 4 rb + r is exactly register r of row block rb, for
// FP32 a k-step of 32 is two row blocks. The order of the k index is free as
// long as the matrix columns are laid out in it.
//
// Fold. With r(j) the mirrored index of the axis (DCT-I / DST-I: n - 1 - j,
// Hartley: N - j), M splits into two half-size matrices acting on
// s = x_a + x_b and d = x_a - x_b over the pairs (a, b = r(a)):
//   DCT-I / DST-I: y_2m = (E s)_m, y_2m+1 = (O d)_m;
//   Hartley: y_p = (E s)_p + (O d)_p, y_N-p = (E s)_p - (O d)_p.
// "Pair order" puts both members of a pair into one lane: two sides (a, b) of
// positions p with indices a_p, b_p. The fold is then lane-local, and a
// product writes its results in pair order too when its matrix rows are read
// in the right order:
//   n even:   a_p = 2p (row p of E), b_p = n - 1 - 2p (row n/2 - 1 - p of O);
//   n odd:    mirrored indices have the same parity. Segment 0 holds the even
//             pairs (a = 2q, b = n - 1 - 2q, both rows of E), segment 1 the odd
//             ones (a = 2q + 1, b = n - 2 - 2q, both rows of O); the middle
//             point has no partner;
//   periodic: a_p = p, b_p = N - p (both from rows p of E and O); 0 and N/2
//             have no partner.
// A point without a partner stands on both sides (its column of E holds half
// the entry, that of O zero), and padding positions repeat the last position
// of their segment (their columns are zero): every register holds a point of
// the field at all times, so no stage masks anything, and what repeated
// positions store is what the position itself stores. (Both sides of a row
// block are loaded before either is stored.)
//
// The last product of an x line is computed transposed (operands exchanged):
// the 16 lanes of a group then hold 16 consecutive output pairs 2m, 2m + 1 of
// one line, which are stored contiguously.
//
// FP32 fields: both operands split into two binary16 terms, v = v0 + v1 (v0
// the rounding of v, v1 of the rest) after a power-of-two scaling of every
// column to [2^14, 2^15); A1 X0 + A0 X1 + A0 X0 accumulated in FP32 (the
// dropped A1 X1 is below 2^-22 of the column scale), scaled back exactly.
// FP64 fields: the unsplit values.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace sfrde {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// vectors at element alignment (lines of odd length, fields at any element)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

// f(integral constant) for 0 .. N-1: loops whose register arrays need constant
// indices at any code size.
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// Computes x here: the terms of sums and the inputs of values that are used
// much later would otherwise stay in registers until then.
template <typename T>
__device__ __forceinline__ void keep(T& x) {
  asm volatile("" : "+v"(x));
}

// Threads per block: two waves per SIMD (256 registers per lane); FP64 axes
// past 128 points hold their points and operands in up to 512 registers, one
// wave per SIMD.
template <typename T, int NB>
constexpr int wave_threads() {
  return sizeof(T) == 8 && NB > 4 ? 256 : 512;
}
// A segment: positions q with a = a0 + da q for q < ca, b = b0 - da q for
// blo <= q < bhi (none: b0 = blo = bhi = 0); side b of a product: row rb - q,
// periodic: row q.
struct WaveSeg {
  int ca, blo, bhi, a0, b0, rb;
};

// One axis as the kernels see it (filled by the host).
struct WaveAxis {
  const void* A;       // the half matrices, device memory (layout: WaveXf)
  int n;
  int nb, nb1;         // row blocks per side in use, in segment 0 and 1
  WaveSeg s0, s1;
  int da;
  int periodic;
};

// Layouts: exact (n = 32 NB, DCT-I / DST-I: no padding, every index known),
// n even or periodic, n odd. Odd axes hold segment 0 in the first NB / 2 row
// blocks and segment 1 in the others.
enum { WL_EXACT = 0, WL_EVEN = 1, WL_ODD = 2 };

// Tiles of 16 lines. Strided axes: lines are counted over every outer block
// (species included), line = o inner + ib. x axis: 16 >> cpsh species columns
// of (1 << cpsh) lines, column = species (1 << cpsh) + line.
struct WaveTiles {
  long long lines;
  long long inner;
  int ntiles;
  int cpsh;
  // Register order (exact axes, every column in use): a tile is contiguous, row
  // block after row block, of each side a and side b, of each the lanes' four
  // values. x axis: stored stage values; last axis: the spectral arrays that live
  // within a step (private), all but u_hat.
  int priv;
  int sweep;  // WaveRun
};

// The tiles of a wave. Fields that the caches hold: a contiguous run of tiles per
// block, which its waves take in turn (the passes along x and y meet the same
// rows on the same XCD); with fewer tiles than waves the blocks (and so the CUs)
// fill first. Larger fields (sweep): the grid goes through the tiles front to
// back, so that what is in flight at a time is contiguous in memory, and the
// waves of a block start a tile together where a kernel asks for it by sync()
// (strided axes: together they touch 512 bytes to 1 KB of a row, each alone 64
// to 128).
struct WaveRun {
  int t, t1, rounds, stride;
  __device__ __forceinline__ explicit WaveRun(const WaveTiles& tl) : WaveRun(tl, tl.ntiles) {}
  __device__ __forceinline__ WaveRun(const WaveTiles& tl, int ntiles)
      : WaveRun(ntiles, tl.sweep, (int)blockIdx.x, (int)gridDim.x,
                __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), (int)(blockDim.x >> 6)) {}
  // wave w of `waves` in block `block` of `grid`
  __device__ __forceinline__ WaveRun(int ntiles, int sweep, int block, int grid, int w, int waves) {
    const int all = grid * waves;
    if (sweep && ntiles > all) {
      t = block * waves + w;
      t1 = ntiles;
      stride = all;
      rounds = (ntiles - block * waves + all - 1) / all;
    } else {
      t = (int)((long long)block * ntiles / grid) + w;
      t1 = (int)(((long long)block + 1) * ntiles / grid);
      stride = waves;
      rounds = 0;
    }
  }
  __device__ __forceinline__ int step() const { return stride; }
  __device__ __forceinline__ void sync() const {
    if (rounds > 0) __builtin_amdgcn_s_barrier();
  }
  // a round of N sync() calls done
  __device__ __forceinline__ void done() { --rounds; }
  // the barriers of the rounds that this wave has no tile in
  template <int N>
  __device__ __forceinline__ void drain() {
    for (; rounds > 0; --rounds)
      for (int k = 0; k < N; ++k) __builtin_amdgcn_s_barrier();
  }
};

// Maximum over the four lanes of a column (l, l ^ 16, l ^ 32, l ^ 48).
__device__ __forceinline__ float column_max(float m) {
  const unsigned u = __builtin_bit_cast(unsigned, m);
  auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  m = fmaxf(__builtin_bit_cast(float, (unsigned)h[0]), __builtin_bit_cast(float, (unsigned)h[1]));
  const unsigned v = __builtin_bit_cast(unsigned, m);
  auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)q[0]), __builtin_bit_cast(float, (unsigned)q[1]));
}

// The lane 8 columns away in the same group of 16 (the other species).
__device__ __forceinline__ float ror8(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xf, 0xf, false));
}
__device__ __forceinline__ double ror8(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x128, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x128, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// The half matrices in memory, RS = 16 NB rows and positions:
//   FP32: 16-byte units [half E|O][term][ks][g][row], binary16 entries e of
//         position 32 ks + (e < 4 ? 4 g + e : 12 + 4 g + e);
//   FP64: [half][ks][g][row], position 4 ks + g.
// LDSA: read from LDS (copied there by the constructor's caller), else from
// global memory (FP64 axes past 192 points: the matrix does not fit). 192^3 FP64
// in steps with the matrix of 6 blocks in LDS / from global memory: 2.09 / 2.36 ms.
template <typename T, int NB>
struct WaveTab;
template <int NB>
struct WaveTab<float, NB> {
  static constexpr int KS = NB / 2, RS = 16 * NB;
  static constexpr size_t bytes = (size_t)2 * 2 * KS * 4 * RS * 16;
};
template <int NB>
struct WaveTab<double, NB> {
  static constexpr int KS = 4 * NB, RS = 16 * NB;
  static constexpr size_t bytes = (size_t)2 * KS * 4 * RS * 8;
};

template <typename T, int NB>
constexpr bool wave_lds_a() {
  return WaveTab<T, NB>::bytes <= 144 * 1024;
}

// Classes whose row blocks are all in use (WaveXf).
template <typename T, int NB>
constexpr bool wave_full() {
  return sizeof(T) == 8 && NB > 4 && NB < 9;
}

template <typename T, int NB, int LAY>
struct WaveXf {
  static constexpr bool EX = LAY == WL_EXACT, ODD = LAY == WL_ODD;
  // FP64 axes of 129 to 256 points: a class for each number of row blocks, all of
  // them in use (with 9 of them the registers do not last: 100 spilled). A matrix
  // from global memory is read ahead, the next product's entries while this one
  // runs; with blocks left out at run time the compiler cannot count the loads in
  // flight and waits for all of them. Per launch, FP64, one class of 9 blocks / one
  // for each: 240^3 X 708 / 435 us, Y 298 / 230, Z 703 / 594; 150^3 X 149 / 77, Y 62 /
  // 48, Z 143 / 96 (8-wave phases 170, 109, 219).
  static constexpr bool FULL = wave_full<T, NB>();
  static_assert(!ODD || NB % 2 == 0, "two segments of NB / 2 row blocks");
  using Tab = WaveTab<T, NB>;
  static constexpr bool F32 = std::is_same<T, float>::value;
  static constexpr int PG = F32 ? 4 : 1, PR = F32 ? 1 : 4;
  static constexpr int KS = Tab::KS, RS = Tab::RS;
  static constexpr bool LDSA = wave_lds_a<T, NB>();
  static constexpr int NBLK = NB;
  static constexpr bool EXACT = EX;
  static constexpr int LAYOUT = LAY;
  using Vals = T[NB][4];

  const WaveAxis& ax;
  const char* tab;
  int i, g;
  unsigned lnat, lrev;  // byte offsets of this lane's rows (natural, reversed from the end)

  static constexpr int UB = F32 ? 16 : 8;  // bytes per (row, g) entry

  __device__ __forceinline__ WaveXf(const WaveAxis& ax_, const char* smem) : ax(ax_) {
    const int lane = threadIdx.x & 63;
    i = lane & 15;
    g = lane >> 4;
    lnat = (unsigned)(g * RS + i) * UB;
    lrev = (unsigned)(g * RS + 15 - i) * UB;
    tab = LDSA ? smem : reinterpret_cast<const char*>(ax.A);
  }
  // The block's copy of the matrix (a barrier must follow).
  __device__ __forceinline__ void copy_table(char* smem) const {
    if constexpr (LDSA) {
      const uint4* src = reinterpret_cast<const uint4*>(ax.A);
      uint4* dst = reinterpret_cast<uint4*>(smem);
      constexpr int NV = (int)(Tab::bytes / 16);
#pragma unroll 4
      for (int v = threadIdx.x; v < NV; v += (int)blockDim.x) dst[v] = src[v];
    }
  }
  static constexpr size_t lds_bytes() { return LDSA ? Tab::bytes : 0; }

  __device__ __forceinline__ int n() const { return EX ? 32 * NB : ax.n; }
  __device__ __forceinline__ int da() const { return EX ? 2 : ax.da; }
  // segment of row block rb, the block within it, and whether it is in use
  __device__ __forceinline__ static constexpr int seg(int rb) { return ODD && 2 * rb >= NB ? 1 : 0; }
  __device__ __forceinline__ static constexpr int sb(int rb) { return seg(rb) ? rb - NB / 2 : rb; }
  // Blocks that hold positions of their own. A block of padding alone (in full
  // classes the last of segment 1 may be one: 129 and 193 points) repeats the last
  // position of the block before, which is harmless where values are stored, but
  // arrays that are read and written would get it twice: the stage combines take
  // own() blocks only.
  __device__ __forceinline__ static constexpr bool block_own(int rb, int nb, int nb1) {
    return EX || (FULL && !(ODD && rb + 1 == NB)) || sb(rb) < (seg(rb) ? nb1 : nb);
  }
  __device__ __forceinline__ bool own(int rb) const { return block_own(rb, ax.nb, ax.nb1); }
  __device__ __forceinline__ bool used(int rb) const { return FULL || own(rb); }
  // A block that a stage combine leaves out, for the next product (its columns are
  // zero; blocks not in use hold zeros already).
  __device__ __forceinline__ static void clear(T (&va)[4], T (&vb)[4]) {
    if constexpr (FULL)
      for (int r = 0; r < 4; ++r) va[r] = vb[r] = T(0);
  }
  // position in the segment of register r of row block rb
  __device__ __forceinline__ int q(int rb, int r) const { return 16 * sb(rb) + PR * r + PG * g; }
  // whether it is a position of its own, side a / b (not padding; the points
  // without a partner count on side a)
  __device__ __forceinline__ bool va(int rb, int r) const {
    return EX || q(rb, r) < (seg(rb) ? ax.s1.ca : ax.s0.ca);
  }
  __device__ __forceinline__ bool vb(int rb, int r) const {
    return EX || (q(rb, r) >= (seg(rb) ? ax.s1.blo : ax.s0.blo) && q(rb, r) < (seg(rb) ? ax.s1.bhi : ax.s0.bhi));
  }
  // ---- operands and products
  // FP32: binary16 heads and tails of the scaled s and d; FP64: s and d.
  struct Ops32 {
    f16x8 s[KS][2], d[KS][2];
    float inv;
  };
  struct Ops64 {
    T s[NB][4], d[NB][4];
  };
  using Ops = typename std::conditional<F32, Ops32, Ops64>::type;

  __device__ __forceinline__ static void split2(float x0, float x1, float sc, f16x8& h, f16x8& t,
                                                int e) {
    const f32x2 x = {x0 * sc, x1 * sc};
    const f16x2 a = __builtin_convertvector(x, f16x2);
    const f32x2 rest = x - __builtin_convertvector(a, f32x2);
    const f16x2 b = __builtin_convertvector(rest, f16x2);
    h[e] = a[0];
    h[e + 1] = a[1];
    t[e] = b[0];
    t[e + 1] = b[1];
  }

  __device__ __forceinline__ void fold(const Vals& ya, const Vals& yb, Ops& o) const {
    if constexpr (F32) {
      float m = 0.f;
#pragma unroll
      for (int rb = 0; rb < NB; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          m = fmaxf(m, fabsf(ya[rb][r]) + fabsf(yb[rb][r]));
      // |a| + |b| = max(|s|, |d|)
      m = column_max(m);
      int k = 15 - __builtin_amdgcn_frexp_expf(m);
      k = k < -126 ? -126 : (k > 126 ? 126 : k);
      const float sc = __builtin_amdgcn_ldexpf(1.f, k);
      o.inv = __builtin_amdgcn_ldexpf(1.f, -k);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            const float a0 = ya[2 * ks + h][r], b0 = yb[2 * ks + h][r];
            const float a1 = ya[2 * ks + h][r + 1], b1 = yb[2 * ks + h][r + 1];
            split2(a0 + b0, a1 + b1, sc, o.s[ks][0], o.s[ks][1], 4 * h + r);
            split2(a0 - b0, a1 - b1, sc, o.d[ks][0], o.d[ks][1], 4 * h + r);
          }
    } else {
#pragma unroll
      for (int rb = 0; rb < NB; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          o.s[rb][r] = ya[rb][r] + yb[rb][r];
          o.d[rb][r] = ya[rb][r] - yb[rb][r];
        }
    }
  }

  // Rows at byte offset lo of half H times the folded columns (SWAP: the
  // transposed product).
  template <int H, bool SWAP>
  __device__ __forceinline__ void prod(unsigned lo, const Ops& o, T (&out)[4]) const {
    if constexpr (F32) {
      // the two small products in a sum of their own: two independent chains,
      // and the large one rounds a third as often
      f32x4 hi = {0.f, 0.f, 0.f, 0.f}, lo4 = {0.f, 0.f, 0.f, 0.f};
      const char* p = tab + lo;
      const auto& B = H ? o.d : o.s;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (!used(2 * ks) && !used(2 * ks + 1)) continue;
        const f16x8 a0 = *reinterpret_cast<const f16x8*>(p + (size_t)((H * 2 + 0) * KS + ks) * 4 * RS * UB);
        const f16x8 a1 = *reinterpret_cast<const f16x8*>(p + (size_t)((H * 2 + 1) * KS + ks) * 4 * RS * UB);
        if constexpr (SWAP) {
          hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(B[ks][0], a0, hi, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(B[ks][0], a1, lo4, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(B[ks][1], a0, lo4, 0, 0, 0);
        } else {
          hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, B[ks][0], hi, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, B[ks][0], lo4, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, B[ks][1], lo4, 0, 0, 0);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) out[r] = hi[r] + lo4[r];
    } else {
      T A[KS];
      fetch<H>(lo, A);
      mul<H, SWAP>(A, o, out);
    }
  }

  // FP32: one row block times two columns' operands.
  template <int H>
  __device__ __forceinline__ void prod2(unsigned lo, const Ops (&o)[2], T (&out)[2][4]) const {
    f32x4 hi[2] = {}, lo4[2] = {};
    const char* p = tab + lo;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (!used(2 * ks) && !used(2 * ks + 1)) continue;
      const f16x8 a0 = *reinterpret_cast<const f16x8*>(p + (size_t)((H * 2 + 0) * KS + ks) * 4 * RS * UB);
      const f16x8 a1 = *reinterpret_cast<const f16x8*>(p + (size_t)((H * 2 + 1) * KS + ks) * 4 * RS * UB);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const auto& B = H ? o[c].d : o[c].s;
        hi[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, B[ks][0], hi[c], 0, 0, 0);
        lo4[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, B[ks][0], lo4[c], 0, 0, 0);
        lo4[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, B[ks][1], lo4[c], 0, 0, 0);
      }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[c][r] = hi[c][r] + lo4[c][r];
  }

  // FP64: the matrix entries of one row block, and their product.
  template <int H>
  __device__ __forceinline__ void fetch(unsigned lo, T (&A)[KS]) const {
    const char* p = tab + lo;
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
      if (!used(rb)) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        A[4 * rb + r] = *reinterpret_cast<const T*>(p + (size_t)(H * KS + 4 * rb + r) * 4 * RS * UB);
    }
  }
  template <int H, bool SWAP>
  __device__ __forceinline__ void mul(const T (&A)[KS], const Ops& o, T (&out)[4]) const {
    f64x4 acc = {0.0, 0.0, 0.0, 0.0}, ac2 = {0.0, 0.0, 0.0, 0.0};
    const auto& B = H ? o.d : o.s;
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
      if (!used(rb)) continue;
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const T a0 = A[4 * rb + r], a1 = A[4 * rb + r + 1];
        if constexpr (SWAP) {
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(B[rb][r], a0, acc, 0, 0, 0);
          ac2 = __builtin_amdgcn_mfma_f64_16x16x4f64(B[rb][r + 1], a1, ac2, 0, 0, 0);
        } else {
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, B[rb][r], acc, 0, 0, 0);
          ac2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, B[rb][r + 1], ac2, 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = acc[r] + ac2[r];
  }

  // Byte offsets of row block rb's rows on both sides (pair order).
  __device__ __forceinline__ void rows(int rb, unsigned lnat, unsigned lrev, unsigned& la,
                                       unsigned& lb) const {
    if constexpr (EX) {
      la = lnat + rb * 16 * UB;
      lb = lrev + (NB - 1 - rb) * 16 * UB;
    } else {
      // padding repeats the segment's last position
      const WaveSeg& w = seg(rb) ? ax.s1 : ax.s0;
      const int s16 = 16 * sb(rb);
      const int qi = s16 + i < w.ca ? s16 + i : w.ca - 1;
      la = lnat + (unsigned)((qi - i) * UB);
      lb = !ODD && ax.periodic ? la : lnat + (unsigned)((w.rb - qi - i) * UB);
    }
  }
  __device__ __forceinline__ void finish(const Ops& o, T (&va)[4], T (&vb)[4]) const {
    if constexpr (LAY == WL_EVEN) {
      const bool per = ax.periodic;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const T e = va[r], d = vb[r];
        va[r] = per ? e + d : e;
        vb[r] = per ? e - d : d;
      }
    }
    if constexpr (F32) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        va[r] *= o.inv;
        vb[r] *= o.inv;
      }
    }
  }

  // Pair order to pair order: out(rb, va, vb) is called with the results of
  // every row block in use; between() after the fold, when ya and yb are free.
  template <class Between, class Out>
  __device__ __forceinline__ void pair_each(const Vals& ya, const Vals& yb, Between&& between,
                                            Out&& out) const {
    Ops o;
    fold(ya, yb, o);
    // opaque copies: the fragment reads stay inside the tile loop (hoisted out
    // of it, the whole matrix would be kept in registers and spilled)
    unsigned lnat = this->lnat, lrev = this->lrev;
    asm volatile("" : "+v"(lnat), "+v"(lrev));
    __builtin_amdgcn_sched_barrier(0);
    between();
    if constexpr (LDSA) {
      static_for<NB>([&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        if (!used(rb)) return;
        unsigned la, lb;
        rows(rb, lnat, lrev, la, lb);
        T va[4], vb[4];
        prod<seg(rb), false>(la, o, va);
        prod<ODD ? seg(rb) : 1, false>(lb, o, vb);
        finish(o, va, vb);
        out(rbc, va, vb);
      });
    } else {
      // the matrix comes from global memory: the entries of the next product
      // are loaded while this one runs
      T A[2][KS];
      unsigned la, lb;
      rows(0, lnat, lrev, la, lb);
      fetch<seg(0)>(la, A[0]);
      static_for<NB>([&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        if (!used(rb)) return;
        T va[4], vb[4];
        // (segment 1 of odd axes starts anew: the block before may be unused)
        constexpr bool first = ODD && 2 * rb == NB, last = rb + 1 == NB || (ODD && 2 * (rb + 1) == NB);
        if constexpr (first) {
          rows(rb, lnat, lrev, la, lb);
          fetch<seg(rb)>(la, A[0]);
        }
        fetch<ODD ? seg(rb) : 1>(lb, A[1]);
        __builtin_amdgcn_sched_barrier(0);
        mul<seg(rb), false>(A[0], o, va);
        if constexpr (!last) {
          rows(rb + 1, lnat, lrev, la, lb);
          fetch<seg(rb + 1)>(la, A[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
        mul<ODD ? seg(rb) : 1, false>(A[1], o, vb);
        finish(o, va, vb);
        out(rbc, va, vb);
      });
    }
  }

  // The same in place.
  __device__ __forceinline__ void pair(Vals& ya, Vals& yb) const {
    pair_each(ya, yb, [] {}, [&](auto rbc, const T (&va)[4], const T (&vb)[4]) {
      constexpr int rb = decltype(rbc)::value;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ya[rb][r] = va[r];
        yb[rb][r] = vb[r];
      }
    });
  }

  // Line (column) of register r after a transposed product.
  __device__ __forceinline__ int tcol(int r) const { return F32 ? 4 * g + r : 4 * r + g; }

  // Transposed products: f(rb, r, e, d) is called with the values of line
  // tcol(r) from rows 16 rb + i of E s and O d: outputs 2m and 2m + 1 with m =
  // 16 rb + i, or (periodic) p and N - p. between(): as in pair_each.
  template <class Between, class F>
  __device__ __forceinline__ void lines(const Vals& ya, const Vals& yb, Between&& between,
                                        F&& f) const {
    Ops o;
    fold(ya, yb, o);
    unsigned lnat = this->lnat;
    asm volatile("" : "+v"(lnat));
    __builtin_amdgcn_sched_barrier(0);
    between();
    T iv[4];
    if constexpr (F32) {
#pragma unroll
      for (int r = 0; r < 4; ++r) iv[r] = __shfl(o.inv, 4 * g + r, 64);
    }
    const bool per = LAY == WL_EVEN && ax.periodic;
    // rows of E (one more than O where n is odd) fill ceil(rows / 16) blocks
    const int rows_e = EX ? 16 * NB : (per ? ax.n / 2 + 1 : (ax.n + 1) / 2);
    T A[2][F32 ? 1 : KS];
    if constexpr (!LDSA) fetch<0>(lnat, A[0]);
    static_for<NB>([&](auto rbc) {
      constexpr int rb = decltype(rbc)::value;
      if (!EX && (!FULL || (ODD && rb + 1 == NB)) && 16 * rb >= rows_e) return;
      T e[4], d[4];
      const unsigned lo = lnat + rb * 16 * UB;
      if constexpr (LDSA) {
        prod<0, true>(lo, o, e);
        prod<1, true>(lo, o, d);
      } else {
        fetch<1>(lo, A[1]);
        __builtin_amdgcn_sched_barrier(0);
        mul<0, true>(A[0], o, e);
        if constexpr (rb + 1 < NB) fetch<0>(lo + 16 * UB, A[0]);
        __builtin_amdgcn_sched_barrier(0);
        mul<1, true>(A[1], o, d);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (F32) {
          e[r] *= iv[r];
          d[r] *= iv[r];
        }
        f(rb, r, per ? e[r] + d[r] : e[r], per ? e[r] - d[r] : d[r]);
      }
    });
  }
};

// ------------------------------------------------------------------ lines
// Whether the rows of 16 lines of a strided axis lie within 2^32 bytes of the
// first line, values of w bytes (a tile reaches into the next outer block where
// the inner extent is not a multiple of 16). Arrays of wider values beside them
// have their offsets scaled in 64 bits (RowIO).
inline bool wave_reach_ok(long long n, long long inner, long long w) {
  return (inner % 16 ? 2 : 1) * (n + 32) * inner * w < (1LL << 32);
}

// This lane's column of a strided tile: a uniform tile base and a 32-bit byte
// offset per lane (wave_reach_ok: the host gives the engine no other axis).
template <typename T>
struct StridedLane {
  long long base;   // element offset of the tile's first line (uniform)
  unsigned off;     // bytes from there to this lane's line
  int o;            // outer block (last axis: species)
  unsigned ib;      // index within the outer block
  bool ok;
  // (cpl: adjacent columns per lane, the first of them is described)
  __device__ __forceinline__ StridedLane(const WaveTiles& tl, int n, int tile, int i,
                                         unsigned cpl = 1u) {
    const unsigned l0 = (unsigned)tile * 16u * cpl;
    const unsigned last = (unsigned)tl.lines - cpl;
    unsigned line = l0 + i * cpl;
    ok = line <= last;
    line = ok ? line : last;
    const unsigned inner = (unsigned)tl.inner;
    const unsigned ou0 = l0 / inner;
    const unsigned ib0 = l0 - ou0 * inner;
    // the lane's outer block: a few steps from the tile's at most
    unsigned x = ib0 + (line - l0);
    unsigned ou = ou0;
    if (x >= inner) {
      const unsigned k = x / inner;
      ou += k;
      x -= k * inner;
    }
    o = (int)ou;
    ib = x;
    base = (long long)ou0 * n * tl.inner + ib0;
    off = (unsigned)(((long long)(ou - ou0) * n * tl.inner + (long long)x - (long long)ib0) *
                     (long long)sizeof(T));
  }
};

// Offsets of a lane's positions, in units of `unit` per index step (both sides;
// padding: those of the segment's last position).
template <class XF>
struct PosOff {
  const XF& xf;
  unsigned step;                 // units per position
  unsigned lane;                 // this lane's first position
  unsigned a0, b0, a1, b1;       // segment starts
  unsigned m0, m1;               // last distances
  __device__ __forceinline__ PosOff(const XF& xf_, unsigned unit, unsigned line) : xf(xf_) {
    step = (unsigned)xf.da() * unit;
    lane = (unsigned)(XF::PG * xf.g) * step;
    const WaveSeg &s0 = xf.ax.s0, &s1 = xf.ax.s1;
    a0 = line + (XF::EXACT ? 0u : (unsigned)s0.a0 * unit);
    b0 = line + (unsigned)(XF::EXACT ? 32 * XF::NBLK - 1 : s0.b0) * unit;
    a1 = line + (unsigned)s1.a0 * unit;
    b1 = line + (unsigned)s1.b0 * unit;
    m0 = (unsigned)(s0.ca - 1) * step;
    m1 = (unsigned)(s1.ca - 1) * step;
  }
  // The lane part through an opaque copy: offsets formed from one copy are used
  // there only (kept from use to use they would fill the register file).
  __device__ __forceinline__ unsigned opaque() const {
    unsigned l = lane;
    asm volatile("" : "+v"(l));
    return l;
  }
  __device__ __forceinline__ void at(unsigned l, int rb, int r, unsigned& a, unsigned& b) const {
    unsigned d = l + (unsigned)(16 * XF::sb(rb) + XF::PR * r) * step;
    const bool sg = XF::seg(rb) != 0;
    if (!XF::EXACT) {
      const unsigned m = sg ? m1 : m0;
      d = d < m ? d : m;
    }
    a = (sg ? a1 : a0) + d;
    b = (sg ? b1 : b0) - d;
    // periodic: position 0 is its own partner
    if (XF::LAYOUT == WL_EVEN && rb == 0 && r == 0 && xf.ax.periodic) b = d == 0u ? a : b;
  }
};

// Row access of a strided column: both sides of row block rb, va[r] and vb[r].
// A row's address is a scalar base and a 32-bit offset per lane. Exact axes: the
// row block is part of the scalar base, and a lane's eight offsets are the same
// in every row block and array (formed once per tile, no vector arithmetic per
// access); others form them per row block, clamped to the last position.
template <typename T, class XF>
struct RowIO {
  const XF& xf;
  long long base;
  PosOff<XF> po;
  struct Side {
    unsigned v[4];          // bytes, per lane
    unsigned long long rb;  // bytes of the row block (uniform)
  };
  struct Off {
    Side a, b;
  };
  unsigned la, lb;  // exact axes: row block 0 of side a, the last of side b
  bool priv;        // private arrays in register order
  long long pbase;  // element offset of the tile there (uniform)
  __device__ __forceinline__ RowIO(const XF& xf_, const WaveTiles& tl, const StridedLane<T>& ln,
                                   int tile = 0, bool priv_ = false)
      : xf(xf_), base(ln.base), po(xf_, (unsigned)tl.inner * (unsigned)sizeof(T), ln.off),
        priv(XF::EXACT && priv_), pbase((long long)tile * (16 * 32 * XF::NBLK)) {
    la = po.a0 + po.lane;
    lb = po.b0 - (unsigned)(16 * (XF::NBLK - 1)) * po.step - po.lane;
  }
  __device__ __forceinline__ Off offs(int rb) const {
    Off o;
    if constexpr (XF::EXACT) {
      // (opaque copies: offsets are formed where they are used; kept, they would
      // fill the register file)
      unsigned xa = la, xb = lb;
      asm volatile("" : "+v"(xa), "+v"(xb));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        o.a.v[r] = xa + (unsigned)(XF::PR * r) * po.step;
        o.b.v[r] = xb - (unsigned)(XF::PR * r) * po.step;
      }
      o.a.rb = (unsigned long long)(16 * rb) * po.step;
      o.b.rb = (unsigned long long)(16 * (XF::NBLK - 1 - rb)) * po.step;
    } else {
      const unsigned l = po.opaque();
#pragma unroll
      for (int r = 0; r < 4; ++r) po.at(l, rb, r, o.a.v[r], o.b.v[r]);
      o.a.rb = o.b.rb = 0;
    }
    return o;
  }
  template <typename U>
  __device__ __forceinline__ const char* at(const U* f, const Side& o) const {
    return reinterpret_cast<const char*>(f + base) + o.rb * (sizeof(U) / sizeof(T));
  }
  template <typename U>
  __device__ __forceinline__ char* at(U* f, const Side& o) const {
    return reinterpret_cast<char*>(f + base) + o.rb * (sizeof(U) / sizeof(T));
  }
  // A lane's byte offset in an array of U. Twice the 32-bit offset of an FP32 value
  // does not fit 32 bits (an FP64 array beside FP32 fields).
  template <typename U>
  __device__ __forceinline__ static auto bytes_of(unsigned v) {
    if constexpr (sizeof(U) == sizeof(T))
      return v;
    else
      return (unsigned long long)v * (sizeof(U) / sizeof(T));
  }
  template <typename U>
  __device__ __forceinline__ void load(const U* f, const Off& o, U (&va)[4], U (&vb)[4]) const {
    load1(f, o.a, va);
    load1(f, o.b, vb);
  }
  // (columns past the last line repeat it and store the same values again)
  template <typename U>
  __device__ __forceinline__ void store(U* f, const Off& o, const U (&va)[4], const U (&vb)[4]) const {
    store1(f, o.a, va);
    store1(f, o.b, vb);
  }
  template <typename U>
  __device__ __forceinline__ void load1(const U* f, const Side& o, U (&v)[4]) const {
    const char* p = at(f, o);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = *reinterpret_cast<const U*>(p + bytes_of<U>(o.v[r]));
  }
  template <typename U>
  __device__ __forceinline__ void store1(U* f, const Side& o, const U (&v)[4]) const {
    char* p = at(f, o);
#pragma unroll
    for (int r = 0; r < 4; ++r) *reinterpret_cast<U*>(p + bytes_of<U>(o.v[r])) = v[r];
  }
  // store of an array that this pass also read: side b of a row block is
  // loaded after side a is stored, so a point that stands on both sides is
  // written from side a only
  template <int SIDE, typename U>
  __device__ __forceinline__ void store_rmw(U* f, const Side& o, const U (&v)[4], int rb) const {
    if (XF::EXACT || SIDE == 0) {
      store1(f, o, v);
      return;
    }
    char* p = at(f, o);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (xf.vb(rb, r)) *reinterpret_cast<U*>(p + bytes_of<U>(o.v[r])) = v[r];
  }
  // ---- private arrays
  struct alignas(sizeof(T) * 2) Vec { T v[4]; };
  __device__ __forceinline__ long long at_priv(int rb, int side) const {
    return pbase + 512 * rb + 256 * side + 4 * (long long)(threadIdx.x & 63);
  }
  template <int SIDE>
  __device__ __forceinline__ void load_priv1(const T* f, int rb, const Side& o, T (&v)[4]) const {
    if (priv) {
      const Vec u = *reinterpret_cast<const Vec*>(f + at_priv(rb, SIDE));
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = u.v[r];
    } else {
      load1(f, o, v);
    }
  }
  template <int SIDE>
  __device__ __forceinline__ void store_priv1(T* f, int rb, const Side& o, const T (&v)[4]) const {
    if (priv)
      *reinterpret_cast<Vec*>(f + at_priv(rb, SIDE)) = Vec{{v[0], v[1], v[2], v[3]}};
    else
      store1(f, o, v);
  }
  template <int SIDE>
  __device__ __forceinline__ void store_priv_rmw(T* f, int rb, const Side& o, const T (&v)[4]) const {
    if (priv)
      store_priv1<SIDE>(f, rb, o, v);
    else
      store_rmw<SIDE>(f, o, v, rb);
  }
  __device__ __forceinline__ void load_priv(const T* f, int rb, const Off& o, T (&va)[4], T (&vb)[4]) const {
    load_priv1<0>(f, rb, o.a, va);
    load_priv1<1>(f, rb, o.b, vb);
  }
  __device__ __forceinline__ void store_priv(T* f, int rb, const Off& o, const T (&va)[4], const T (&vb)[4]) const {
    store_priv1<0>(f, rb, o.a, va);
    store_priv1<1>(f, rb, o.b, vb);
  }
  __device__ __forceinline__ void load_all(const T* f, typename XF::Vals& ya,
                                           typename XF::Vals& yb) const {
#pragma unroll
    for (int rb = 0; rb < XF::NBLK; ++rb) {
      T va[4] = {T(0), T(0), T(0), T(0)}, vb[4] = {T(0), T(0), T(0), T(0)};
      if (xf.used(rb)) load(f, offs(rb), va, vb);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ya[rb][r] = va[r];
        yb[rb][r] = vb[r];
      }
    }
  }
  __device__ __forceinline__ void store_all(T* f, const typename XF::Vals& ya,
                                            const typename XF::Vals& yb) const {
#pragma unroll
    for (int rb = 0; rb < XF::NBLK; ++rb) {
      if (!xf.used(rb)) continue;
      store(f, offs(rb), ya[rb], yb[rb]);
    }
  }
};

// This lane's column of an x tile: species sp, line `line` (clamped to the
// last ones where there is none: ok false).
template <typename T>
struct XLane {
  int sp;
  long long line;
  bool ok;
  __device__ __forceinline__ XLane(const WaveTiles& tl, int S, int tile, int i) {
    sp = i >> tl.cpsh;
    line = ((long long)tile << tl.cpsh) + (i & ((1 << tl.cpsh) - 1));
    ok = sp < S && line < tl.lines;
    sp = sp < S ? sp : S - 1;
    line = line < tl.lines ? line : tl.lines - 1;
  }
};

constexpr int LINE_CHUNK = 2;

// The points of one x line in pair order. Exact FP32 axes read a lane's four
// positions of a row block (every other element) from two overlapping 16-byte
// vectors at element alignment.
template <typename T, class XF>
__device__ __forceinline__ void load_line(const XF& xf, const T* p, typename XF::Vals& ya,
                                          typename XF::Vals& yb) {
  const PosOff<XF> po(xf, 1u, 0u);
#pragma unroll
  for (int rb = 0; rb < XF::NBLK; ++rb) {
    // the vectors of a few row blocks in flight at a time (all of them would
    // take twice the registers of the points)
    if (rb > 0 && rb % LINE_CHUNK == 0) __builtin_amdgcn_sched_barrier(0);
    if constexpr (XF::EXACT && XF::F32) {
      const float* q = p + 2 * xf.q(rb, 0);
      const f32x4u u = *reinterpret_cast<const f32x4u*>(q);
      const f32x4u v = *reinterpret_cast<const f32x4u*>(q + 3);
      ya[rb][0] = u[0];
      ya[rb][1] = u[2];
      ya[rb][2] = v[1];
      ya[rb][3] = v[3];
      q = p + (32 * XF::NBLK - 1 - 2 * xf.q(rb, 0));
      const f32x4u w = *reinterpret_cast<const f32x4u*>(q - 3);
      const f32x4u z = *reinterpret_cast<const f32x4u*>(q - 6);
      yb[rb][0] = w[3];
      yb[rb][1] = w[1];
      yb[rb][2] = z[2];
      yb[rb][3] = z[0];
    } else {
      T va[4] = {T(0), T(0), T(0), T(0)}, vb[4] = {T(0), T(0), T(0), T(0)};
      if (xf.used(rb)) {
        const unsigned l = po.opaque();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          unsigned ia, ib;
          po.at(l, rb, r, ia, ib);
          va[r] = p[ia];
          vb[r] = p[ib];
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ya[rb][r] = va[r];
        yb[rb][r] = vb[r];
      }
    }
  }
}

// Last product of an x tile and its store: line tcol(r) of the tile's
// columns, outputs 2m, 2m + 1 (periodic p, N - p) of 16 consecutive m per
// group of lanes (columns that repeat the last line or species store its
// values again). wt: Neumann point weights multiplied in.
template <typename T, class XF, class Between, class W>
__device__ __forceinline__ void store_lines(const XF& xf, const WaveTiles& tl, int S,
                                            long long total, int tile, T* dst,
                                            const typename XF::Vals& ya,
                                            const typename XF::Vals& yb, Between&& between, W&& wt) {
  const int n = xf.n();
  T* lp[4];
  long long ln[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = xf.tcol(r);
    int sp = c >> tl.cpsh;
    sp = sp < S ? sp : S - 1;
    ln[r] = ((long long)tile << tl.cpsh) + (c & ((1 << tl.cpsh) - 1));
    ln[r] = ln[r] < tl.lines ? ln[r] : tl.lines - 1;
    lp[r] = dst + (sp * total + ln[r] * n);
  }
  xf.lines(ya, yb, between, [&](int rb, int r, T e, T d) {
    const int m = 16 * rb + xf.i;
    if (XF::LAYOUT != WL_EVEN || !xf.ax.periodic) {
      e *= wt(ln[r], 2 * m, n);
      d *= wt(ln[r], 2 * m + 1, n);
      if (XF::EXACT || 2 * m + 1 < n) {
        if constexpr (XF::F32) {
          f32x2u v = {e, d};
          *reinterpret_cast<f32x2u*>(lp[r] + 2 * m) = v;
        } else {
          f64x2u v = {e, d};
          *reinterpret_cast<f64x2u*>(lp[r] + 2 * m) = v;
        }
      } else if (2 * m < n) {
        lp[r][2 * m] = e;
      }
    } else if (2 * m <= n) {
      lp[r][m] = e;
      if (m > 0 && 2 * m < n) lp[r][n - m] = d;
    }
  });
}

struct NoWeight {
  template <typename L>
  __device__ __forceinline__ int operator()(L, int, int) const { return 1; }
};

// Neumann weight of line `line` (y + n1 z): 1/2 per axis at an end.
__device__ __forceinline__ double line_weight(long long line, long long n1, long long n2) {
  double w = 1.0;
  const unsigned l = (unsigned)line, m1 = (unsigned)n1, m2 = (unsigned)n2;
  const unsigned z = l / m1, y = l - z * m1;
  if (n1 > 1 && (y == 0 || y == m1 - 1)) w *= 0.5;
  if (n2 > 1 && (z == 0 || z == m2 - 1)) w *= 0.5;
  return w;
}

// ------------------------------------------------------------------ reaction
// f of the stage values in ya, yb (in place). Two-species columns hold one
// species each, its partner 8 lanes away; every lane forms both components
// and keeps its own. Returns whether a value was not finite.
template <int KIND, typename T, class XF>
__device__ __forceinline__ void wave_react_rb(const XF& xf, const StageArgs<T>& a,
                                              const RxnT<T>& rx, const XLane<T>& ln,
                                              const PosOff<XF>& po, const MmsLine& ml, int rb,
                                              T (&va)[4], T (&vb)[4], T& chk) {
  const T lin = ln.sp == 0 ? rx.lin[0] : ln.sp == 1 ? rx.lin[1] : ln.sp == 2 ? rx.lin[2] : rx.lin[3];
#pragma unroll
  for (int side = 0; side < 2; ++side)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      T& cell = side ? vb[r] : va[r];
      const T own = cell;
      T f;
      if constexpr (KIND == RXN_LINEAR) {
        f = lin * own;
      } else if constexpr (KIND >= RXN_HUXLEY_MMS) {
        const T u[1] = {own};
        T o[1];
        rxn_eval_k<T, 1, KIND>(rx, u, o);
        unsigned ia, ib;
        po.at(po.lane, rb, r, ia, ib);
        f = o[0] + T(mms_source<KIND>(ml, (int)(side ? ib : ia)));
      } else {
        const T oth = ror8(own);
        const T u[2] = {ln.sp == 0 ? own : oth, ln.sp == 0 ? oth : own};
        T o[2];
        rxn_eval_k<T, 2, KIND>(rx, u, o);
        f = ln.sp == 0 ? o[0] : o[1];
      }
      chk = fma(own, T(0), chk);
      chk = fma(f, T(0), chk);
      cell = f;
      keep(cell);
    }
  keep(chk);
}

template <int KIND, typename T, class XF>
__device__ __forceinline__ bool wave_react_k(const XF& xf, const StageArgs<T>& a,
                                             const XLane<T>& ln, const MmsLine& ml,
                                             typename XF::Vals& ya, typename XF::Vals& yb) {
  const RxnT<T> rx(a.rxn);
  const PosOff<XF> po(xf, 1u, 0u);
  T chk = T(0);
  static_for<XF::NBLK>([&](auto rbc) {
    constexpr int rb = decltype(rbc)::value;
    if (!xf.used(rb)) return;
    __builtin_amdgcn_sched_barrier(0);
    wave_react_rb<KIND>(xf, a, rx, ln, po, ml, rb, ya[rb], yb[rb], chk);
  });
  return !(chk == T(0));
}

template <bool SRC, typename T, class XF>
__device__ __forceinline__ bool wave_react(const XF& xf, const StageArgs<T>& a,
                                           const XLane<T>& ln, const MmsLine& ml,
                                           typename XF::Vals& ya, typename XF::Vals& yb) {
  if constexpr (SRC) {
    if (a.rxn.kind == RXN_HUXLEY_MMS) return wave_react_k<RXN_HUXLEY_MMS>(xf, a, ln, ml, ya, yb);
    return wave_react_k<RXN_FISHER_MMS>(xf, a, ln, ml, ya, yb);
  }
  __builtin_amdgcn_sched_barrier(0);
  switch (a.rxn.kind) {  // uniform
    case RXN_LINEAR: return wave_react_k<RXN_LINEAR>(xf, a, ln, ml, ya, yb);
    case RXN_FHN: return wave_react_k<RXN_FHN>(xf, a, ln, ml, ya, yb);
    case RXN_GRAY_SCOTT: return wave_react_k<RXN_GRAY_SCOTT>(xf, a, ln, ml, ya, yb);
    case RXN_SCHNAKENBERG: return wave_react_k<RXN_SCHNAKENBERG>(xf, a, ln, ml, ya, yb);
    default: return wave_react_k<RXN_GM>(xf, a, ln, ml, ya, yb);
  }
}

// Stage values of an x tile to / from the segment store: in register order
// where every column of every tile is in use (tl.priv: 16 n values per tile),
// else at their natural places.
template <typename T, class XF>
__device__ __forceinline__ void store_stage(const XF& xf, const WaveTiles& tl, const XLane<T>& ln,
                                            int tile, long long total, T* st,
                                            const typename XF::Vals& ya,
                                            const typename XF::Vals& yb) {
  if (XF::EXACT && tl.priv) {
    T* p = st + (long long)tile * 16 * xf.n() + (threadIdx.x & 63) * 4;
#pragma unroll
    for (int rb = 0; rb < XF::NBLK; ++rb) {
      struct alignas(sizeof(T) * 2) V { T v[4]; };
      *reinterpret_cast<V*>(p + rb * 512) = V{{ya[rb][0], ya[rb][1], ya[rb][2], ya[rb][3]}};
      *reinterpret_cast<V*>(p + rb * 512 + 256) = V{{yb[rb][0], yb[rb][1], yb[rb][2], yb[rb][3]}};
    }
    return;
  }
  T* p = st + ln.sp * total + ln.line * xf.n();
  const PosOff<XF> po(xf, 1u, 0u);
#pragma unroll
  for (int rb = 0; rb < XF::NBLK; ++rb) {
    if (!xf.used(rb)) continue;
    const unsigned l = po.opaque();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      unsigned ia, ib;
      po.at(l, rb, r, ia, ib);
      p[ia] = ya[rb][r];
      p[ib] = yb[rb][r];
    }
  }
}

template <typename T, class XF>
struct StageIn {
  const T* p;
  PosOff<XF> po;
  bool priv;
  __device__ __forceinline__ StageIn(const XF& xf, const WaveTiles& tl, const XLane<T>& ln,
                                     int tile, long long total, const T* st)
      : po(xf, 1u, 0u), priv(XF::EXACT && tl.priv) {
    p = priv ? st + (long long)tile * 16 * xf.n() + (threadIdx.x & 63) * 4
             : st + ln.sp * total + ln.line * xf.n();
  }
  // both sides of row block rb
  __device__ __forceinline__ void load(int rb, T (&va)[4], T (&vb)[4]) const {
    if (priv) {
      struct alignas(sizeof(T) * 2) V { T v[4]; };
      const V u = *reinterpret_cast<const V*>(p + rb * 512);
      const V w = *reinterpret_cast<const V*>(p + rb * 512 + 256);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        va[r] = u.v[r];
        vb[r] = w.v[r];
      }
    } else {
      const unsigned l = po.opaque();
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        unsigned ia, ib;
        po.at(l, rb, r, ia, ib);
        va[r] = p[ia];
        vb[r] = p[ib];
      }
    }
  }
};

// ------------------------------------------------------------------ kernels
// Every kernel: the first tile's loads, the block's copy of the matrix, one
// barrier, then tile after tile without another. The next tile is loaded as
// soon as the fold of the last product has freed the registers of this one,
// and is in flight over that product and its stores.

// X: inverse-x, reaction, forward-x (in place on P). SRC: the reactions with a
// manufactured source (a kernel of their own: the source is a long function).
// Bound at 256^3 FP32 by its chain at two waves per SIMD (244 registers): 86 us
// (3.1 TB/s), 99 in the phases of an 8-wave block; 128^3 FP32 27 -> 15.5 us,
// FP64 71 -> 35.
template <typename T, int NB, int LAY, bool SRC>
__global__ __launch_bounds__((wave_threads<T, NB>())) void k_wx(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = WaveXf<T, NB, LAY>;
  const XF xf(ax, smem);
  const long long total = a.g.total;
  bool bad = false;
  WaveRun run(tl);
  typename XF::Vals ya, yb;
  auto load = [&](int tile) {
    const XLane<T> ln(tl, a.S, tile, xf.i);
    load_line<T>(xf, a.P + ln.sp * total + ln.line * xf.n(), ya, yb);
  };
  if (run.t < run.t1) load(run.t);
  xf.copy_table(smem);
  __syncthreads();
  for (int tile = run.t; tile < run.t1;) {
    const XLane<T> ln(tl, a.S, tile, xf.i);
    MmsLine ml{};
    if constexpr (SRC) ml = mms_line(a.rxn, a.t, ln.line % a.n1);
    xf.pair(ya, yb);
    if (a.st_phys)
      store_stage(xf, tl, ln, tile, total, a.st_phys + (long long)a.mode * a.S * total, ya, yb);
    bad |= wave_react<SRC>(xf, a, ln, ml, ya, yb);
    // (x lines are loaded after the stores: beside the operands their vectors
    // do not fit the registers)
    store_lines<T>(xf, tl, a.S, total, tile, a.P, ya, yb, [] {}, NoWeight{});
    tile += run.step();
    if (tile < run.t1) load(tile);
  }
  if (bad) a.flag[0] = 1;
}

// One transform along the x axis, src -> dst (may alias), with optional
// Neumann point weights before (divide) or after (multiply).
template <typename T, int NB, int LAY>
__global__ __launch_bounds__((wave_threads<T, NB>())) void k_wsx(SingleArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = WaveXf<T, NB, LAY>;
  const XF xf(ax, smem);
  const long long total = a.g.total;
  WaveRun run(tl);
  typename XF::Vals ya, yb;
  auto load = [&](int tile) {
    const XLane<T> ln(tl, a.S, tile, xf.i);
    load_line<T>(xf, a.src + ln.sp * total + ln.line * xf.n(), ya, yb);
    if (a.pre_divide_w) {
      const T wl = T(line_weight(ln.line, a.n1, a.n2));
#pragma unroll
      for (int rb = 0; rb < NB; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ya[rb][r] /= wl;
          yb[rb][r] /= wl;
        }
      // both ends of a line sit at position 0
      const T we = xf.g == 0 ? T(0.5) : T(1);
      ya[0][0] /= we;
      yb[0][0] /= we;
    }
  };
  if (run.t < run.t1) load(run.t);
  xf.copy_table(smem);
  __syncthreads();
  for (int tile = run.t; tile < run.t1;) {
    if (a.post_multiply_w)
      store_lines<T>(xf, tl, a.S, total, tile, a.dst, ya, yb, [] {},
                     [&](long long line, int e, int n) {
                       const T w = T(line_weight(line, a.n1, a.n2));
                       return e == 0 || e == n - 1 ? T(0.5) * w : w;
                     });
    else
      store_lines<T>(xf, tl, a.S, total, tile, a.dst, ya, yb, [] {}, NoWeight{});
    tile += run.step();
    if (tile < run.t1) load(tile);
  }
}

// One transform along a strided axis, src -> dst (may alias).
template <typename T, int NB, int LAY>
__global__ __launch_bounds__((wave_threads<T, NB>())) void k_wsy(SingleArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = WaveXf<T, NB, LAY>;
  const XF xf(ax, smem);
  WaveRun run(tl);
  typename XF::Vals ya, yb;
  auto load = [&](int tile) {
    const StridedLane<T> ln(tl, xf.n(), tile, xf.i);
    RowIO<T, XF>(xf, tl, ln).load_all(a.src, ya, yb);
  };
  if (run.t < run.t1) load(run.t);
  xf.copy_table(smem);
  __syncthreads();
  for (int tile = run.t; tile < run.t1;) {
    run.sync();
    const StridedLane<T> ln(tl, xf.n(), tile, xf.i);
    const RowIO<T, XF> io(xf, tl, ln);
    const int next = tile + run.step();
    xf.pair_each(
        ya, yb, [&] { if (next < run.t1) load(next); },
        [&](auto rbc, const T (&va)[4], const T (&vb)[4]) {
          io.store(a.dst, io.offs(decltype(rbc)::value), va, vb);
        });
    tile = next;
    run.done();
  }
  run.drain<1>();
}

// The same for FP32 with two columns per lane (32 lines per wave; inner even:
// both lie in one outer block): every matrix fragment read from LDS serves two
// products, and rows move in 128-byte pieces, 8 bytes per lane. One transform
// needs no registers beside the operands, so the second column fits. Memory
// bound: 256^3 54 us (4.9 TB/s; one column per lane 60), 128^3 18 -> 9.7 us.
template <int NB, int LAY>
__global__ __launch_bounds__(512) void k_wsy2(SingleArgs<float> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = WaveXf<float, NB, LAY>;
  const XF xf(ax, smem);
  WaveRun run(tl);
  xf.copy_table(smem);
  __syncthreads();
  for (int tile = run.t; tile < run.t1; tile += run.step()) {
    run.sync();
    const StridedLane<float> ln(tl, xf.n(), tile, xf.i, 2u);
    const RowIO<float, XF> io(xf, tl, ln);
    typename XF::Ops o[2];
    {
      typename XF::Vals ya[2], yb[2];
#pragma unroll
      for (int rb = 0; rb < NB; ++rb) {
        f32x2 va[4] = {}, vb[4] = {};
        if (xf.used(rb)) {
          const auto of = io.offs(rb);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            va[r] = *reinterpret_cast<const f32x2u*>(io.at(a.src, of.a) + of.a.v[r]);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            vb[r] = *reinterpret_cast<const f32x2u*>(io.at(a.src, of.b) + of.b.v[r]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            ya[c][rb][r] = va[r][c];
            yb[c][rb][r] = vb[r][c];
          }
      }
      __builtin_amdgcn_sched_barrier(0);
      xf.fold(ya[0], yb[0], o[0]);
      xf.fold(ya[1], yb[1], o[1]);
    }
    unsigned lnat = xf.lnat, lrev = xf.lrev;
    asm volatile("" : "+v"(lnat), "+v"(lrev));
    __builtin_amdgcn_sched_barrier(0);
    static_for<NB>([&](auto rbc) {
      constexpr int rb = decltype(rbc)::value;
      if (!xf.used(rb)) return;
      unsigned la, lb;
      xf.rows(rb, lnat, lrev, la, lb);
      float va[2][4], vb[2][4];
      xf.template prod2<XF::seg(rb)>(la, o, va);
      xf.template prod2<XF::LAYOUT == WL_ODD ? XF::seg(rb) : 1>(lb, o, vb);
      xf.finish(o[0], va[0], vb[0]);
      xf.finish(o[1], va[1], vb[1]);
      const auto of = io.offs(rb);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        *reinterpret_cast<f32x2u*>(io.at(a.dst, of.a) + of.a.v[r]) = f32x2u{va[0][r], va[1][r]};
        *reinterpret_cast<f32x2u*>(io.at(a.dst, of.b) + of.b.v[r]) = f32x2u{vb[0][r], vb[1][r]};
      }
    });
    run.done();
  }
  run.drain<1>();
}

// Last-axis eigenvalues in position order for L formed in the kernel:
// lam_lds[side][16 NB], then [n0] x and [n1] y (3D).
template <typename T, class XF>
__device__ __forceinline__ void fill_lam(const XF& xf, const StageArgs<T>& a, float* lam) {
  constexpr int NP = 16 * XF::NBLK;
  const double* lz = a.n2 > 1 ? a.lam[2] : a.lam[1];
  static_assert(XF::LAYOUT != WL_ODD, "one segment");
  const int ca = XF::EXACT ? NP : xf.ax.s0.ca;
  for (int t = threadIdx.x; t < 2 * NP; t += blockDim.x) {
    int p = t % NP;
    const int side = t / NP;
    p = p < ca ? p : ca - 1;
    int j = xf.da() * p;
    if (side) j = xf.n() - (XF::EXACT || !xf.ax.periodic ? 1 : 0) - j;
    if (j == xf.n()) j = 0;
    lam[t] = float(lz[j]);
  }
  const int nx = (int)a.n0, ny = a.n2 > 1 ? (int)a.n1 : 0;
  for (int t = threadIdx.x; t < nx + ny; t += blockDim.x)
    lam[2 * NP + t] = float(t < nx ? a.lam[0][t] : a.lam[1][t - nx]);
}

// Lambda's x and y part of a last-axis column.
template <typename T>
__device__ __forceinline__ float lam_xy(const StageArgs<T>& a, const float* tabs, unsigned ib,
                                        int& x, int& y) {
  const unsigned n0 = (unsigned)a.n0;
  y = a.n2 > 1 ? (int)(ib / n0) : 0;
  x = (int)(ib - (unsigned)y * n0);
  return a.n2 > 1 ? tabs[x] + tabs[n0 + y] : tabs[x];
}

// Four consecutive positions' eigenvalues of this lane.
template <class XF>
__device__ __forceinline__ void lam_z(const XF& xf, const float* lam, int side, int rb,
                                      float (&v)[4]) {
  int o = 4 * xf.g;
  asm volatile("" : "+v"(o));  // read here, not kept from tile to tile
  const float4 q = *reinterpret_cast<const float4*>(lam + side * 16 * XF::NBLK + 16 * rb + o);
  v[0] = q.x;
  v[1] = q.y;
  v[2] = q.z;
  v[3] = q.w;
}

// Where a Z kernel's coefficients come from: L formed in the kernel, the table of
// L, the tables of the coefficients. (At compile time: a choice at run time put
// the values read into scratch memory, 12 to 136 bytes per lane.)
enum { CO_FLY = 0, CO_LTAB = 1, CO_TABS = 2 };

// What the stage combine of a row block reads, both sides: the retained arrays
// x1 (stages 0, 1: u_hat; 2, 3: acc; loaded by the caller) and x2 (stage 1:
// acc; 2: c_tilde), L (in t0) or the coefficients.
template <typename T>
struct CombineIn {
  T x1[2][4], x2[2][4], t0[2][4], t1[2][4], t2[2][4], t3[2][4];
};
template <int MODE, int CO, typename T, class IO>
__device__ __forceinline__ void wave_combine_in(const IO& io, const StageArgs<T>& a, int rb,
                                                CombineIn<T>& in) {
  const long long cst = (long long)a.S * a.g.total;
  const auto of = io.offs(rb);
  if constexpr (CO == CO_LTAB) io.load(a.ltab, of, in.t0[0], in.t0[1]);
  if constexpr (CO == CO_TABS) {
    if (MODE <= 1) io.load(a.coef + C_Q * cst, of, in.t0[0], in.t0[1]);
    if (MODE <= 2) io.load(a.coef + C_PHI * cst, of, in.t1[0], in.t1[1]);
    io.load(a.coef + (MODE == 0 ? C_R : MODE == 3 ? C_PHI3 : C_PHI2) * cst, of, in.t2[0], in.t2[1]);
    if (MODE == 0) io.load(a.coef + C_PHI1 * cst, of, in.t3[0], in.t3[1]);
  }
  if (MODE == 1 || MODE == 2) io.load_priv(MODE == 1 ? a.acc : a.ctil, rb, of, in.x2[0], in.x2[1]);
}

// Stage combine (MODE 0..3) of a row block, both sides.
template <int MODE, int CO, typename T, class IO>
__device__ __forceinline__ void wave_combine_out(const IO& io, const StageArgs<T>& a, int rb,
                                                 float lxy, T kt, T ha, const float (&lz)[2][4],
                                                 const CombineIn<T>& in, T (&va)[4], T (&vb)[4]) {
  const long long cst = (long long)a.S * a.g.total;
  const auto of = io.offs(rb);
  T o0[2][4], o1[2][4], fh[2][4];
#pragma unroll
  for (int side = 0; side < 2; ++side) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      T c0 = T(0), c1 = T(0), c2 = T(0), c3 = T(0);
      if constexpr (CO == CO_FLY) {
        // Lambda is 0 or at least the smallest nonzero eigenvalue, far from
        // denormals: the hardware log2 / exp2 (about 1 ulp) suffice, and give
        // 0 at Lambda = 0 (log2 0 = -inf, alpha > 0) without a branch
        const float L =
            kt * __builtin_amdgcn_exp2f(ha * __builtin_amdgcn_logf(lxy + lz[side][r]));
        stage_coefs_L<T>(MODE, L, a.tau, c0, c1, c2, c3);
      } else if constexpr (CO == CO_LTAB) {
        stage_coefs_L<T>(MODE, in.t0[side][r], a.tau, c0, c1, c2, c3);
      } else {
        if (MODE <= 1) c0 = in.t0[side][r];
        if (MODE <= 2) c1 = in.t1[side][r];
        c2 = in.t2[side][r];
        if (MODE == 0) c3 = in.t3[side][r];
      }
      T& v = side ? vb[r] : va[r];
      const T x1 = in.x1[side][r];
      const T f = v;
      fh[side][r] = f;
      T out;
      if (MODE == 0) {
        const T av = dec_mul(c0, x1) + c1 * f;
        o0[side][r] = dec_mul(c0, av) - c1 * f;
        o1[side][r] = dec_mul(c2, x1) + c3 * f;
        out = av;
      } else if (MODE == 1) {
        out = dec_mul(c0, x1) + c1 * f;
        o1[side][r] = in.x2[side][r] + c2 * f;
      } else if (MODE == 2) {
        out = in.x2[side][r] + T(2) * c1 * f;
        o1[side][r] = x1 + c2 * f;
      } else {
        out = x1 + c2 * f;
        o0[side][r] = out;
      }
      v = a.cs * out;
    }
  }
  if (MODE == 0) io.store_priv(a.ctil, rb, of, o0[0], o0[1]);
  if (a.st_fhat) io.store_priv(a.st_fhat + MODE * cst, rb, of, fh[0], fh[1]);
  if (MODE <= 2) io.store_priv(a.acc, rb, of, o1[0], o1[1]);
  if (MODE == 3) io.store(a.uhat, of, o0[0], o0[1]);
}

// Z: forward transform along the last axis, stage combine, inverse transform
// (in place on P). MODE 0..3; MODE < 0: MODE_INIT or MODE_RESTORE (a.mode).
// CO: CO_FLY for FP32 P13 plans. Memory
// bound at 256^3 FP32, on 64-byte rows at 256 KB strides: 3.5 TB/s over five
// fields in stage 0 with every array in the fields' order; with c_tilde and acc
// in register order and the sweep a step went 1.43 -> 1.34 ms (1.43 in 8-wave
// blocks on the same GPU; the four stages 168 to 137 us there, 156 to 120 here). 128^3
// FP32 32-36 -> 17-20 us a stage, FP64 76-85 -> 43-54.
template <typename T, int NB, int LAY, int MODE, int CO>
__global__ __launch_bounds__((wave_threads<T, NB>())) void k_wz(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = WaveXf<T, NB, LAY>;
  const XF xf(ax, smem);
  WaveRun run(tl);
  typename XF::Vals ya, yb;
  const T* src = a.src ? a.src : a.P;
  auto load = [&](int tile) {
    const StridedLane<T> ln(tl, xf.n(), tile, xf.i);
    RowIO<T, XF>(xf, tl, ln).load_all(src, ya, yb);
  };
  if (run.t < run.t1) load(run.t);
  xf.copy_table(smem);
  float* lam = reinterpret_cast<float*>(smem + XF::lds_bytes());
  if constexpr (CO == CO_FLY) fill_lam(xf, a, lam);
  __syncthreads();
  for (int tile = run.t; tile < run.t1;) {
    run.sync();
    const StridedLane<T> ln(tl, xf.n(), tile, xf.i);
    const RowIO<T, XF> io(xf, tl, ln, tile, CO == CO_FLY || tl.priv);
    if constexpr (MODE >= 0) {
      // the first retained array, in flight over the transform (FP32)
      typename XF::Vals xa, xb;
      auto load_x1 = [&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        if (!xf.used(rb)) return;
        if (MODE <= 1)
          io.load(a.uhat, io.offs(rb), xa[rb], xb[rb]);
        else
          io.load_priv(a.acc, rb, io.offs(rb), xa[rb], xb[rb]);
      };
      if constexpr (XF::F32) static_for<NB>(load_x1);
      xf.pair(ya, yb);
      float lxy = 0.f;
      T kt = T(0), ha = T(0);
      if constexpr (CO == CO_FLY) {
        int x, y;
        lxy = lam_xy(a, lam + 32 * NB, ln.ib, x, y);
        kt = pick_species(a.kt, ln.o);
        ha = pick_species(a.ha, ln.o);
      }
      static_for<NB>([&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        if (!xf.own(rb)) return xf.clear(ya[rb], yb[rb]);
        if constexpr (!XF::F32) load_x1(rbc);
        float lz[2][4] = {};
        if constexpr (CO == CO_FLY) {
          lam_z(xf, lam, 0, rb, lz[0]);
          lam_z(xf, lam, 1, rb, lz[1]);
        }
        CombineIn<T> in;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          in.x1[0][r] = xa[rb][r];
          in.x1[1][r] = xb[rb][r];
        }
        wave_combine_in<MODE, CO>(io, a, rb, in);
        wave_combine_out<MODE, CO>(io, a, rb, lxy, kt, ha, lz, in, ya[rb], yb[rb]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          keep(ya[rb][r]);
          keep(yb[rb][r]);
        }
        // two row blocks' arrays in flight at a time
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {
      if (!a.src) xf.pair(ya, yb);
      if (a.mode == MODE_INIT) io.store_all(a.uhat, ya, yb);
#pragma unroll
      for (int rb = 0; rb < NB; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ya[rb][r] *= a.cs;
          yb[rb][r] *= a.cs;
          // rounded here as in the stage kernels (not contracted into the fold):
          // a state restored from u_hat continues bit for bit
          keep(ya[rb][r]);
          keep(yb[rb][r]);
        }
    }
    run.sync();
    const int next = tile + run.step();
    xf.pair_each(
        ya, yb, [&] { if (next < run.t1) load(next); },
        [&](auto rbc, const T (&va)[4], const T (&vb)[4]) {
          io.store(a.P, io.offs(decltype(rbc)::value), va, vb);
        });
    tile = next;
    run.done();
  }
  run.drain<2>();
}

// ------------------------------------------------------------------ adjoint
// Adjoint reaction: the cotangents of f become J^T of them at the stored stage
// values (wave engine: read two row blocks ahead); parameter partials (weighted
// by the point weights, each point once) are added to pacc.
template <int KIND, bool WP, typename T, class XF>
__device__ __forceinline__ void wave_adj_react_rb(const XF& xf, const StageArgs<T>& a,
                                                  const XLane<T>& ln, int rb, T (&va)[4],
                                                  T (&vb)[4], const T (&ua)[4], const T (&ub)[4],
                                                  double* pacc) {
  constexpr bool TWO = KIND >= RXN_FHN && KIND <= RXN_GM;
  double wl = 0.0;
  if constexpr (WP) {
    // two-species lanes see every point twice: species 0 counts it
    if (ln.ok && (!TWO || ln.sp == 0)) wl = a.neumann ? line_weight(ln.line, a.n1, a.n2) : 1.0;
  }
  const T lin = T(ln.sp == 0 ? a.rxn.p[0] : ln.sp == 1 ? a.rxn.p[1] : ln.sp == 2 ? a.rxn.p[2] : a.rxn.p[3]);
#pragma unroll
  for (int side = 0; side < 2; ++side)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      T& cell = side ? vb[r] : va[r];
      const T gown = cell, uown = side ? ub[r] : ua[r];
      double w = wl;
      if constexpr (WP) {
        if (!(side ? xf.vb(rb, r) : xf.va(rb, r))) w = 0.0;
        if (rb == 0 && r == 0 && a.neumann && xf.g == 0) w *= 0.5;  // the line's ends
      }
      if constexpr (KIND == RXN_LINEAR) {
        cell = lin * gown;
        if constexpr (WP) {
          const double c = w * double(gown * uown);
#pragma unroll
          for (int s = 0; s < MAX_SPECIES; ++s) pacc[s] += ln.sp == s ? c : 0.0;
        }
      } else if constexpr (TWO) {
        const T goth = ror8(gown), uoth = ror8(uown);
        const bool first = ln.sp == 0;
        const T u[2] = {first ? uown : uoth, first ? uoth : uown};
        const T g[2] = {first ? gown : goth, first ? goth : gown};
        T o[2];
        rxn_adjoint_k<T, 2, KIND>(a.rxn, u, g, o, w, pacc, WP);
        cell = first ? o[0] : o[1];
      } else {
        const T u[1] = {uown}, g[1] = {gown};
        T o[1];
        rxn_adjoint_k<T, 1, KIND>(a.rxn, u, g, o, w, pacc, false);
        cell = o[0];
      }
      keep(cell);
    }
  if constexpr (WP) {
#pragma unroll
    for (int k = 0; k < RXN_NP_MAX; ++k) keep(pacc[k]);
  }
}

template <int KIND, bool WP, typename T, class XF>
__device__ __forceinline__ void wave_adj_react_k(const XF& xf, const StageArgs<T>& a,
                                                 const XLane<T>& ln, typename XF::Vals& ya,
                                                 typename XF::Vals& yb, const StageIn<T, XF>& in,
                                                 double* pacc) {
  T ua[XF::NBLK][4] = {}, ub[XF::NBLK][4] = {};
  constexpr int AHEAD = 2;
  static_for<(AHEAD < XF::NBLK ? AHEAD : XF::NBLK)>([&](auto rbc) {
    constexpr int rb = decltype(rbc)::value;
    if (xf.used(rb)) in.load(rb, ua[rb], ub[rb]);
  });
  static_for<XF::NBLK>([&](auto rbc) {
    constexpr int rb = decltype(rbc)::value;
    if constexpr (rb + AHEAD < XF::NBLK) {
      if (xf.used(rb + AHEAD)) in.load(rb + AHEAD, ua[rb + AHEAD], ub[rb + AHEAD]);
    }
    if (!xf.used(rb)) return;
    __builtin_amdgcn_sched_barrier(0);
    wave_adj_react_rb<KIND, WP>(xf, a, ln, rb, ya[rb], yb[rb], ua[rb], ub[rb], pacc);
  });
}

template <bool WP, typename T, class XF>
__device__ __forceinline__ void wave_adj_react(const XF& xf, const StageArgs<T>& a,
                                               const XLane<T>& ln, typename XF::Vals& ya,
                                               typename XF::Vals& yb,
                                               const StageIn<T, XF>& in, double* pacc) {
  switch (a.rxn.kind) {  // uniform
    case RXN_LINEAR: wave_adj_react_k<RXN_LINEAR, WP>(xf, a, ln, ya, yb, in, pacc); break;
    case RXN_FHN: wave_adj_react_k<RXN_FHN, WP>(xf, a, ln, ya, yb, in, pacc); break;
    case RXN_GRAY_SCOTT: wave_adj_react_k<RXN_GRAY_SCOTT, WP>(xf, a, ln, ya, yb, in, pacc); break;
    case RXN_SCHNAKENBERG: wave_adj_react_k<RXN_SCHNAKENBERG, WP>(xf, a, ln, ya, yb, in, pacc); break;
    case RXN_GM: wave_adj_react_k<RXN_GM, WP>(xf, a, ln, ya, yb, in, pacc); break;
    case RXN_HUXLEY_MMS: wave_adj_react_k<RXN_HUXLEY_MMS, WP>(xf, a, ln, ya, yb, in, pacc); break;
    default: wave_adj_react_k<RXN_FISHER_MMS, WP>(xf, a, ln, ya, yb, in, pacc); break;
  }
}

// X, adjoint: inverse-x of the spectral cotangent of f(stage value), transposed
// reaction Jacobian at the stored stage value, forward-x. WP: with the
// reaction-parameter partials.
template <typename T, int NB, int LAY, bool WP>
__global__ __launch_bounds__((wave_threads<T, NB>())) void k_wxadj(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = WaveXf<T, NB, LAY>;
  const XF xf(ax, smem);
  const long long total = a.g.total;
  double pacc[RXN_NP_MAX];
#pragma unroll
  for (int k = 0; k < RXN_NP_MAX; ++k) pacc[k] = 0.0;
  const T* st = a.st_phys + (long long)a.mode * a.S * total;
  WaveRun run(tl);
  typename XF::Vals ya, yb;
  auto load = [&](int tile) {
    const XLane<T> ln(tl, a.S, tile, xf.i);
    load_line<T>(xf, a.P + ln.sp * total + ln.line * xf.n(), ya, yb);
  };
  if (run.t < run.t1) load(run.t);
  xf.copy_table(smem);
  __syncthreads();
  for (int tile = run.t; tile < run.t1;) {
    const XLane<T> ln(tl, a.S, tile, xf.i);
    xf.pair(ya, yb);
    const StageIn<T, XF> in(xf, tl, ln, tile, total, st);
    wave_adj_react<WP>(xf, a, ln, ya, yb, in, pacc);
    // (x lines are loaded after the stores: beside the operands their vectors
    // do not fit the registers)
    store_lines<T>(xf, tl, a.S, total, tile, a.P, ya, yb, [] {}, NoWeight{});
    tile += run.step();
    if (tile < run.t1) load(tile);
  }
  if constexpr (WP) block_add_partials(reinterpret_cast<double*>(smem), pacc, a.rxn.np, a.rp_acc);
}

// The six P13 coefficients of L (order C_R, C_Q, C_PHI, C_PHI1, C_PHI2,
// C_PHI3) and, for the parameter gradients, their derivatives in L from the
// quotient rule, g' = (num' - g den') / den, with D' = 18 + 12L + 3L^2 and
// Dh' = 72 + 24L + 3L^2 (Section 4's rational forms).
__device__ __forceinline__ void p13_all(float L, float tau, float* c) {
  const float D = 24.f + L * (18.f + L * (6.f + L));
  const float Dh = 192.f + L * (72.f + L * (12.f + L));
  const float iD = __builtin_amdgcn_rcpf(D), iDh = __builtin_amdgcn_rcpf(Dh);
  const bool small = L < 1.f;
  const float ph = 96.f + L * (12.f + L);
  const float rl = 1.f - L * (24.f + L * (6.f + L)) * iD, rh = (24.f - 6.f * L) * iD;
  const float ql = 1.f - L * ph * iDh, qh = 24.f * (8.f - L) * iDh;
  c[C_R] = small ? rl : rh;
  c[C_Q] = small ? ql : qh;
  c[C_PHI] = tau * ph * iDh;
  c[C_PHI1] = tau * (4.f - L) * iD;
  c[C_PHI2] = 2.f * tau * (4.f + L) * iD;
  c[C_PHI3] = tau * (4.f + L * (3.f + L)) * iD;
}
__device__ __forceinline__ void p13_dall(float L, float tau, const float* c, float* d) {
  const float D = 24.f + L * (18.f + L * (6.f + L));
  const float Dh = 192.f + L * (72.f + L * (12.f + L));
  const float iD = __builtin_amdgcn_rcpf(D), iDh = __builtin_amdgcn_rcpf(Dh);
  const float dD = 18.f + L * (12.f + 3.f * L), dDh = 72.f + L * (24.f + 3.f * L);
  d[C_R] = (-6.f - c[C_R] * dD) * iD;
  d[C_Q] = (-24.f - c[C_Q] * dDh) * iDh;
  d[C_PHI] = (tau * (12.f + 2.f * L) - c[C_PHI] * dDh) * iDh;
  d[C_PHI1] = (-tau - c[C_PHI1] * dD) * iD;
  d[C_PHI2] = (2.f * tau - c[C_PHI2] * dD) * iD;
  d[C_PHI3] = (tau * (3.f + 2.f * L) - c[C_PHI3] * dD) * iD;
}

// Lambda^ha (0 at Lambda = 0) and log2(Lambda) to about 2 ulp: the hardware
// log2's rounding of a value near 20 alone would be 10^-6 of the power, which
// the gradients of kappa and alpha see directly (L itself only through the
// decay rates). One Newton step on the logarithm, and the rounding of ha lg
// carried along.
__device__ __forceinline__ float lambda_power(float lam, float ha, float& lg) {
  const float l = fmaxf(lam, 1e-30f);
  const float h = __builtin_amdgcn_logf(l);
  const float corr = 1.44269504f * fmaf(l, __builtin_amdgcn_exp2f(-h), -1.f);
  lg = h + corr;
  const float p = ha * h;
  const float rest = fmaf(ha, h, -p) + ha * corr;
  const float pw = __builtin_amdgcn_exp2f(p) * fmaf(0.693147181f, rest, 1.f);
  return lam > 0.f ? pw : 0.f;
}

// Adjoint combine of one side of a row block with L formed in the kernel (same formulas as
// pw_adj_combine). TH: each coefficient application's y g'(L) x is turned into
// the kappa and alpha gradient contributions at once: times the spectral
// weight, then by dL/dkappa = tau Lambda^(alpha/2) and dL/dalpha =
// L ln(Lambda) / 2, summed per lane and row block in FP32 and beyond in FP64.
// wxy: cs times the x and y spectral weights of the column.
// in: what it reads, loaded ahead (wave_adj_fly_in).
struct AdjIn {
  float z[4], h[4], c4[4], u[4], f0[4], f1[4], f2[4], f3[4];
};
template <int MODE, bool TH, int SIDE, class XF>
__device__ __forceinline__ void wave_adj_fly_in(const RowIO<float, XF>& io,
                                                const StageArgs<float>& a, int rb, AdjIn& in) {
  const long long cst = (long long)a.S * a.g.total;
  const auto ofs = io.offs(rb);
  const auto& of = SIDE ? ofs.b : ofs.a;
  if (MODE <= 1) io.template load_priv1<SIDE>(a.zh, rb, of, in.z);
  if (MODE >= 1 && MODE <= 3) io.template load_priv1<SIDE>(a.aacc, rb, of, in.c4);
  if (MODE == 2) {
    io.template load_priv1<SIDE>(a.ahat, rb, of, in.h);
    io.template load_priv1<SIDE>(a.gu, rb, of, in.z);
  }
  if (TH && MODE <= 2) {
    io.load1(a.st_uhat, of, in.u);
    if (MODE == 0 || MODE == 2) io.template load_priv1<SIDE>(a.st_fhat, rb, of, in.f0);
    if (MODE == 0 || MODE == 1) io.template load_priv1<SIDE>(a.st_fhat + cst, rb, of, in.f1);
    if (MODE == 0) {
      io.template load_priv1<SIDE>(a.st_fhat + 2 * cst, rb, of, in.f2);
      io.template load_priv1<SIDE>(a.st_fhat + 3 * cst, rb, of, in.f3);
    }
  }
}
template <int MODE, bool TH, int SIDE, class XF>
__device__ __forceinline__ void wave_adj_fly(const XF& xf, const RowIO<float, XF>& io,
                                             const StageArgs<float>& a, int rb, float lxy,
                                             float wxy, float kt, float ha,
                                             const float (&lz)[4], const AdjIn& in, float (&v4)[4],
                                             double& sk, double& sa) {
  const auto ofs = io.offs(rb);
  const auto& of = SIDE ? ofs.b : ofs.a;
  const auto &z = in.z, &h = in.h, &c4 = in.c4, &u = in.u;
  const auto &f0 = in.f0, &f1 = in.f1, &f2 = in.f2, &f3 = in.f3;
  float o1[4], o2[4], o3[4];
  float ak = 0.f, aa = 0.f;
  {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float lg;
      const float pw = lambda_power(lxy + lz[r], ha, lg);
      const float L = kt * pw;
      float c[NCOEF];
      p13_all(L, a.tau, c);
      float d[NCOEF];
      if (TH && MODE <= 2) p13_dall(L, a.tau, c, d);
      float& v = v4[r];
      const float X = v;
      float out, gs = 0.f;
      if (MODE == 0) {
        const float zz = z[r];
        o1[r] = c[C_R] * zz;
        o2[r] = c[C_Q] * X;
        o3[r] = c[C_PHI1] * zz - c[C_PHI] * X;
        out = c[C_PHI2] * zz + 2.f * c[C_PHI] * X;
        if (TH) {
          const float uh = u[r], fu = f0[r], fa = f1[r];
          const float fb = f2[r], fc = f3[r];
          const float ah = c[C_Q] * uh + c[C_PHI] * fu;
          const float s1 = d[C_R] * uh + d[C_PHI1] * fu + d[C_PHI2] * (fa + fb) + d[C_PHI3] * fc;
          const float s2 = d[C_Q] * ah + d[C_PHI] * (2.f * fb - fu);
          gs = zz * s1 + X * s2;
        }
      } else if (MODE == 1) {
        o1[r] = c4[r] + c[C_Q] * X;
        out = c[C_PHI2] * z[r] + c[C_PHI] * X;
        if (TH) gs = X * (d[C_Q] * u[r] + d[C_PHI] * f1[r]);
      } else if (MODE == 2) {
        const float A = h[r] + X;
        o1[r] = c4[r] + c[C_Q] * A;
        out = z[r] + c[C_PHI] * A;
        if (TH) gs = A * (d[C_Q] * u[r] + d[C_PHI] * f0[r]);
      } else if (MODE == 3) {
        const float zn = c4[r] + X;
        o1[r] = zn;
        out = a.last ? zn : c[C_PHI3] * zn;
      } else {  // MODE_INIT
        o1[r] = X;
        out = c[C_PHI3] * X;
      }
      v = a.cs * out;
      if (TH && MODE <= 2) {
        float gw = wxy * gs;
        if (rb == 0 && r == 0 && a.neumann && xf.g == 0) gw *= 0.5f;  // the axis' ends
        if (!XF::EXACT && !(SIDE ? xf.vb(rb, r) : xf.va(rb, r))) gw = 0.f;
        ak += gw * (a.tau * pw);
        aa += gw * (0.34657359f * L * lg);  // L ln(Lambda) / 2 (0 where Lambda = 0)
      }
    }
  }
  if (MODE == 0) {
    io.template store_priv1<SIDE>(a.aacc, rb, of, o1);
    io.template store_priv1<SIDE>(a.ahat, rb, of, o2);
    io.template store_priv1<SIDE>(a.gu, rb, of, o3);
  } else if (MODE <= 2) {
    io.template store_priv_rmw<SIDE>(a.aacc, rb, of, o1);
  } else {
    io.template store_priv1<SIDE>(a.zh, rb, of, o1);
  }
  if (TH && MODE <= 2) {
    keep(ak);
    keep(aa);
    sk += double(ak);
    sa += double(aa);
    keep(sk);
    keep(sa);
  }
}

// The same from tables, any precision and scheme (formulas and terms of
// pw_adj_combine; the per-point accumulator G when the gradients of kappa and
// alpha are asked).
template <int SIDE, typename T, class IO>
__device__ __forceinline__ void wave_adj_tab(const IO& io, const StageArgs<T>& a, int rb,
                                             T (&v4)[4]) {
  const long long cst = (long long)a.S * a.g.total;
  const auto ofs = io.offs(rb);
  const auto& of = SIDE ? ofs.b : ofs.a;
  // FP64 P13 plans: the coefficients and their derivatives formed from L
  const bool from_l = std::is_same<T, double>::value && a.ltab != nullptr;
  const int mode = a.mode;
  T Lv[4];
  if (from_l) io.load1(a.ltab, of, Lv);
  auto coef = [&](int q, T (&c)[4]) { io.load1(a.coef + q * cst, of, c); };
  auto dcoef = [&](int q, T (&c)[4]) { io.load1(a.dcoef + q * cst, of, c); };
  auto each = [&](auto f) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double cl[NCOEF], dl[NCOEF];
      if (from_l) p13_table_derivs(double(Lv[r]), double(a.tau), cl, dl);
      v4[r] = a.cs * f(r, v4[r], cl, dl);
    }
  };
  if (mode == 0) {
    T z[4], R[4], Q[4], P[4], P1[4], P2[4];
    io.template load_priv1<SIDE>(a.zh, rb, of, z);
    if (!from_l) {
      coef(C_R, R);
      coef(C_Q, Q);
      coef(C_PHI, P);
      coef(C_PHI1, P1);
      coef(C_PHI2, P2);
    }
    T uh[4], fu[4], fa[4], fb[4], fc[4];
    T dR[4], dQ[4], dP[4], dP1[4], dP2[4], dP3[4];
    double G[4];
    if (a.G) {
      io.load1(a.st_uhat, of, uh);
      io.template load_priv1<SIDE>(a.st_fhat, rb, of, fu);
      io.template load_priv1<SIDE>(a.st_fhat + cst, rb, of, fa);
      io.template load_priv1<SIDE>(a.st_fhat + 2 * cst, rb, of, fb);
      io.template load_priv1<SIDE>(a.st_fhat + 3 * cst, rb, of, fc);
      io.load1(a.G, of, G);
      if (!from_l) {
        dcoef(C_R, dR);
        dcoef(C_Q, dQ);
        dcoef(C_PHI, dP);
        dcoef(C_PHI1, dP1);
        dcoef(C_PHI2, dP2);
        dcoef(C_PHI3, dP3);
      }
    }
    T o1[4], o2[4], o3[4];
    each([&](int r, T X, const double* cl, const double* dl) {
      const T cR = from_l ? T(cl[C_R]) : R[r], cQ = from_l ? T(cl[C_Q]) : Q[r];
      const T cP = from_l ? T(cl[C_PHI]) : P[r], cP1 = from_l ? T(cl[C_PHI1]) : P1[r];
      const T cP2 = from_l ? T(cl[C_PHI2]) : P2[r];
      const T zz = z[r];
      o1[r] = dec_mul(cR, zz);
      o2[r] = dec_mul(cQ, X);
      o3[r] = cP1 * zz - cP * X;
      if (a.G) {
        const T xR = from_l ? T(dl[C_R]) : dR[r], xQ = from_l ? T(dl[C_Q]) : dQ[r];
        const T xP = from_l ? T(dl[C_PHI]) : dP[r], xP1 = from_l ? T(dl[C_PHI1]) : dP1[r];
        const T xP2 = from_l ? T(dl[C_PHI2]) : dP2[r], xP3 = from_l ? T(dl[C_PHI3]) : dP3[r];
        const T ah = dec_mul(cQ, uh[r]) + cP * fu[r];
        const T s1 = xR * uh[r] + xP1 * fu[r] + xP2 * (fa[r] + fb[r]) + xP3 * fc[r];
        const T s2 = xQ * ah + xP * (T(2) * fb[r] - fu[r]);
        G[r] += double(zz) * double(s1) + double(X) * double(s2);
      }
      return cP2 * zz + T(2) * cP * X;
    });
    io.template store_priv1<SIDE>(a.aacc, rb, of, o1);
    io.template store_priv1<SIDE>(a.ahat, rb, of, o2);
    io.template store_priv1<SIDE>(a.gu, rb, of, o3);
    if (a.G) io.template store_rmw<SIDE>(a.G, of, G, rb);
  } else if (mode == 1 || mode == 2) {
    const bool b = mode == 1;
    // stage 1: z, aacc;  2: gu, aacc, ahat
    T z[4], c4[4], h[4], Q[4], P[4], P2[4];
    io.template load_priv1<SIDE>(b ? a.zh : a.gu, rb, of, z);
    io.template load_priv1<SIDE>(a.aacc, rb, of, c4);
    if (!b) io.template load_priv1<SIDE>(a.ahat, rb, of, h);
    if (!from_l) {
      coef(C_Q, Q);
      coef(C_PHI, P);
      if (b) coef(C_PHI2, P2);
    }
    T uh[4], f[4], dQ[4], dP[4];
    double G[4];
    if (a.G) {
      io.load1(a.st_uhat, of, uh);
      io.template load_priv1<SIDE>(a.st_fhat + (b ? cst : 0), rb, of, f);
      io.load1(a.G, of, G);
      if (!from_l) {
        dcoef(C_Q, dQ);
        dcoef(C_PHI, dP);
      }
    }
    T o1[4];
    each([&](int r, T X, const double* cl, const double* dl) {
      const T cQ = from_l ? T(cl[C_Q]) : Q[r], cP = from_l ? T(cl[C_PHI]) : P[r];
      const T A = b ? X : h[r] + X;
      o1[r] = c4[r] + dec_mul(cQ, A);
      if (a.G) {
        const T xQ = from_l ? T(dl[C_Q]) : dQ[r], xP = from_l ? T(dl[C_PHI]) : dP[r];
        G[r] += double(A) * double(xQ * uh[r] + xP * f[r]);
      }
      if (b) return (from_l ? T(cl[C_PHI2]) : P2[r]) * z[r] + cP * X;
      return z[r] + cP * A;
    });
    io.template store_priv_rmw<SIDE>(a.aacc, rb, of, o1);
    if (a.G) io.template store_rmw<SIDE>(a.G, of, G, rb);
  } else {
    // 3: z <- aacc + X;  MODE_INIT: X is the transformed cotangent of u(T)
    const bool init = mode != 3;
    T c4[4], P3[4], o1[4];
    if (!init) io.template load_priv1<SIDE>(a.aacc, rb, of, c4);
    if (!from_l) coef(C_PHI3, P3);
    each([&](int r, T X, const double* cl, const double*) {
      const T zn = init ? X : c4[r] + X;
      o1[r] = zn;
      return !init && a.last ? zn : (from_l ? T(cl[C_PHI3]) : P3[r]) * zn;
    });
    io.template store_priv1<SIDE>(a.zh, rb, of, o1);
  }
}

// Z, adjoint: forward-z, adjoint combine, inverse-z. MODE 0..MODE_INIT with L
// formed in the kernel (TH: with the kappa and alpha partials, a.thp); MODE <
// 0: from tables, a.mode at run time.
template <typename T, int NB, int LAY, int MODE, bool TH>
__global__ __launch_bounds__((wave_threads<T, NB>())) void k_wzadj(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = WaveXf<T, NB, LAY>;
  const XF xf(ax, smem);
  WaveRun run(tl);
  typename XF::Vals ya, yb;
  auto load = [&](int tile) {
    const StridedLane<T> ln(tl, xf.n(), tile, xf.i);
    RowIO<T, XF>(xf, tl, ln).load_all(a.P, ya, yb);
  };
  if (run.t < run.t1) load(run.t);
  xf.copy_table(smem);
  float* lam = reinterpret_cast<float*>(smem + XF::lds_bytes());
  if constexpr (MODE >= 0) fill_lam(xf, a, lam);
  __syncthreads();
  // kappa, alpha partials of (at most, host-checked) two species
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int tile = run.t; tile < run.t1;) {
    const StridedLane<T> ln(tl, xf.n(), tile, xf.i);
    const RowIO<T, XF> io(xf, tl, ln, tile, MODE >= 0 || tl.priv);
    AdjIn in[2];
    xf.pair(ya, yb);
    if constexpr (MODE >= 0) {
      int x, y;
      const float lxy = lam_xy(a, lam + 32 * NB, ln.ib, x, y);
      const float kt = pick_species(a.kt, ln.o), ha = pick_species(a.ha, ln.o);
      float wxy = ln.ok ? a.cs : 0.f;
      if (a.neumann) {
        if (x == 0 || x == (int)a.n0 - 1) wxy *= 0.5f;
        if (a.n2 > 1 && (y == 0 || y == (int)a.n1 - 1)) wxy *= 0.5f;
      }
      double sk = 0.0, sa = 0.0;
      static_for<NB>([&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        if (!xf.used(rb)) return;
        float lz[4];
        wave_adj_fly_in<MODE, TH, 0>(io, a, rb, in[0]);
        lam_z(xf, lam, 0, rb, lz);
        wave_adj_fly<MODE, TH, 0>(xf, io, a, rb, lxy, wxy, kt, ha, lz, in[0], ya[rb], sk, sa);
        wave_adj_fly_in<MODE, TH, 1>(io, a, rb, in[1]);
        lam_z(xf, lam, 1, rb, lz);
        wave_adj_fly<MODE, TH, 1>(xf, io, a, rb, lxy, wxy, kt, ha, lz, in[1], yb[rb], sk, sa);
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (TH && MODE <= 2) {
        acc[0] += ln.o == 0 ? sk : 0.0;
        acc[1] += ln.o == 0 ? sa : 0.0;
        acc[2] += ln.o == 0 ? 0.0 : sk;
        acc[3] += ln.o == 0 ? 0.0 : sa;
      }
    } else {
      static_for<NB>([&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        if (!xf.own(rb)) return xf.clear(ya[rb], yb[rb]);
        wave_adj_tab<0>(io, a, rb, ya[rb]);
        __builtin_amdgcn_sched_barrier(0);
        wave_adj_tab<1>(io, a, rb, yb[rb]);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    const int next = tile + run.step();
    xf.pair_each(
        ya, yb, [&] { if (next < run.t1) load(next); },
        [&](auto rbc, const T (&va)[4], const T (&vb)[4]) {
          io.store(a.P, io.offs(decltype(rbc)::value), va, vb);
        });
    tile = next;
  }
  if constexpr (TH && MODE >= 0 && MODE <= 2)
    block_sums(reinterpret_cast<double*>(smem), acc, 2 * a.S, a.thp, true);
}

// ------------------------------------------------------------------ groups
// One tile per block, one wave per row block (group kernels): the launch's
// tiles are too few to give every CU waves of their own, so what counts is the
// length of one tile's chain. Each wave holds its row block of both sides (8
// values per lane) and its rows of the matrix in registers, loaded beside the
// points; the folded columns are exchanged through LDS (one barrier per
// product, one more in FP32 for the column scale). Every product and sum is
// the wave engine's, in its order: the results are the same bit for bit. The
// code of a stage appears once, not once per row block, which a kernel of one
// pass (cold instruction cache) needs most. Bound by that chain: 64^2 FP64 X 16.8
// (8-wave block) -> 4.4 us, Z 12 -> 5; 256^2 FP32 X 15 -> 7.8, Z 13 -> 7.4.
template <typename T, int NB, int LAY>
struct GroupXf : WaveXf<T, NB, LAY> {
  using W = WaveXf<T, NB, LAY>;
  static constexpr bool F32 = W::F32;
  static constexpr int KS = W::KS, RS = W::RS, UB = W::UB;
  static constexpr int THREADS = 64 * NB;
  // operands in LDS: FP32 [half][ks][term][lane] of 16 bytes, FP64
  // [half][ks][lane] of 8; then (FP32) the waves' column maxima
  static constexpr size_t OPS = F32 ? (size_t)2 * KS * 2 * 1024 : (size_t)2 * KS * 512;
  static constexpr size_t BUF = OPS + (F32 ? NB * 64 : 0);
  static constexpr size_t lds_bytes() { return 2 * BUF; }  // a buffer per product
  // matrix rows of one side of this wave's row block
  struct Rows32 {
    f16x8 a[KS][2];
  };
  struct Rows64 {
    T a[KS];
  };
  // FP64 axes past 128 points, FP32 past 256: read during the product (the
  // rows of four sides do not fit; three or four waves per SIMD cover the reads)
  static constexpr bool STREAM = F32 ? NB > 8 : NB > 4;
  struct RowsAt {
    int half;
    unsigned lo;
  };
  using Rows = typename std::conditional<
      STREAM, RowsAt, typename std::conditional<F32, Rows32, Rows64>::type>::type;
  int rb;
  bool on;
  int lane;

  __device__ __forceinline__ GroupXf(const WaveAxis& ax_)
      : W(ax_, reinterpret_cast<const char*>(ax_.A)) {
    this->tab = reinterpret_cast<const char*>(ax_.A);  // read once, from global memory
    rb = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    on = W::own(rb);
    lane = threadIdx.x & 63;
  }
  __device__ __forceinline__ void rows_of(int half, unsigned lo, Rows& m) const {
    const char* p = this->tab + lo;
    if constexpr (STREAM) {
      m.half = half;
      m.lo = lo;
    } else if constexpr (F32) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          m.a[ks][t] = *reinterpret_cast<const f16x8*>(
              p + (size_t)((half * 2 + t) * KS + ks) * 4 * RS * UB);
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        m.a[ks] = *reinterpret_cast<const T*>(p + (size_t)(half * KS + ks) * 4 * RS * UB);
    }
  }
  // rows for a pair-order product (sides a, b) and for a transposed one (E, O)
  __device__ __forceinline__ int half_b() const { return W::ODD ? W::seg(rb) : 1; }
  __device__ __forceinline__ void pair_rows(Rows& ma, Rows& mb) const {
    if (!on) return;
    unsigned la, lb;
    this->rows(rb, this->lnat, this->lrev, la, lb);
    rows_of(W::seg(rb), la, ma);
    rows_of(half_b(), lb, mb);
  }
  __device__ __forceinline__ void nat_rows(Rows& me, Rows& mo) const {
    const unsigned lo = this->lnat + (unsigned)(rb * 16 * UB);
    rows_of(0, lo, me);
    rows_of(1, lo, mo);
  }

  // This wave's part of the folded columns to LDS buffer b; returns the inverse
  // column scale (FP32). Ends with a barrier. Waves without a row block
  // contribute zeros.
  __device__ __forceinline__ float share(char* smem, int b, const T (&va)[4],
                                         const T (&vb)[4]) const {
    char* buf = smem + b * BUF;
    if constexpr (F32) {
      float* mx = reinterpret_cast<float*>(buf + OPS);
      float m = 0.f;
      if (on) {
#pragma unroll
        for (int r = 0; r < 4; ++r) m = fmaxf(m, fabsf(va[r]) + fabsf(vb[r]));
        m = column_max(m);
      }
      if (this->g == 0) mx[rb * 16 + this->i] = m;
      __syncthreads();
      m = 0.f;
#pragma unroll
      for (int w = 0; w < NB; ++w) m = fmaxf(m, mx[w * 16 + this->i]);
      int k = 15 - __builtin_amdgcn_frexp_expf(m);
      k = k < -126 ? -126 : (k > 126 ? 126 : k);
      const float sc = __builtin_amdgcn_ldexpf(1.f, k);
      typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
      f16x4 q[2][2] = {};
      if (on) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          f16x8 hd = {}, tl = {};
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            const float x0 = h ? va[r] - vb[r] : va[r] + vb[r];
            const float x1 = h ? va[r + 1] - vb[r + 1] : va[r + 1] + vb[r + 1];
            W::split2(x0, x1, sc, hd, tl, r);
          }
          q[h][0] = f16x4{hd[0], hd[1], hd[2], hd[3]};
          q[h][1] = f16x4{tl[0], tl[1], tl[2], tl[3]};
        }
      }
      char* p = buf + (size_t)(rb >> 1) * 2048 + lane * 16 + (rb & 1) * 8;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          *reinterpret_cast<f16x4*>(p + (size_t)h * KS * 2048 + t * 1024) = q[h][t];
      __syncthreads();
      return __builtin_amdgcn_ldexpf(1.f, -k);
    } else {
      T* p = reinterpret_cast<T*>(buf) + (size_t)rb * 4 * 64 + lane;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[r * 64] = on ? va[r] + vb[r] : T(0);
        p[r * 64 + KS * 64] = on ? va[r] - vb[r] : T(0);
      }
      __syncthreads();
      return 1.f;
    }
  }
  __device__ __forceinline__ f16x8 row32(const Rows& m, int ks, int t) const {
    if constexpr (STREAM)
      return *reinterpret_cast<const f16x8*>(
          this->tab + m.lo + (size_t)((m.half * 2 + t) * KS + ks) * 4 * RS * UB);
    else
      return m.a[ks][t];
  }
  // One row block times the shared columns of half `half`.
  template <bool SWAP>
  __device__ __forceinline__ void mul_shared(const char* smem, int b, int half, const Rows& m,
                                             T (&out)[4]) const {
    const char* buf = smem + b * BUF;
    if constexpr (F32) {
      f32x4 hi = {0.f, 0.f, 0.f, 0.f}, lo4 = {0.f, 0.f, 0.f, 0.f};
      const char* p = buf + (size_t)half * KS * 2048 + lane * 16;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const f16x8 b0 = *reinterpret_cast<const f16x8*>(p + (size_t)ks * 2048);
        const f16x8 b1 = *reinterpret_cast<const f16x8*>(p + (size_t)ks * 2048 + 1024);
        const f16x8 a0 = row32(m, ks, 0), a1 = row32(m, ks, 1);
        if constexpr (SWAP) {
          hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a0, hi, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a1, lo4, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(b1, a0, lo4, 0, 0, 0);
        } else {
          hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, b0, hi, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, b0, lo4, 0, 0, 0);
          lo4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, b1, lo4, 0, 0, 0);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) out[r] = hi[r] + lo4[r];
    } else {
      f64x4 acc = {0.0, 0.0, 0.0, 0.0}, ac2 = {0.0, 0.0, 0.0, 0.0};
      const T* p = reinterpret_cast<const T*>(buf) + (size_t)half * KS * 64 + lane;
      auto row = [&](int ks) -> T {
        if constexpr (STREAM)
          return *reinterpret_cast<const T*>(this->tab + m.lo +
                                             (size_t)(m.half * KS + ks) * 4 * RS * UB);
        else
          return m.a[ks];
      };
#pragma unroll
      for (int ks = 0; ks < KS; ks += 2) {
        const T b0 = p[ks * 64], b1 = p[(ks + 1) * 64];
        const T a0 = row(ks), a1 = row(ks + 1);
        if constexpr (SWAP) {
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b0, a0, acc, 0, 0, 0);
          ac2 = __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a1, ac2, 0, 0, 0);
        } else {
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc, 0, 0, 0);
          ac2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, ac2, 0, 0, 0);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) out[r] = acc[r] + ac2[r];
    }
  }
  // Pair order to pair order (buffer b of LDS).
  __device__ __forceinline__ void pair_shared(char* smem, int b, const Rows& ma, const Rows& mb,
                                              T (&va)[4], T (&vb)[4]) const {
    typename W::Ops o;  // (only its scale is used)
    const float inv = share(smem, b, va, vb);
    if constexpr (F32) o.inv = inv;
    if (!on) return;
    mul_shared<false>(smem, b, W::seg(rb), ma, va);
    mul_shared<false>(smem, b, half_b(), mb, vb);
    this->finish(o, va, vb);
  }
};

// This wave's points of an x line.
template <typename T, class XF>
__device__ __forceinline__ void load_line_rb(const XF& xf, const T* p, T (&va)[4], T (&vb)[4]) {
  const PosOff<typename XF::W> po(xf, 1u, 0u);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    unsigned ia, ib;
    po.at(po.lane, xf.rb, r, ia, ib);
    va[r] = p[ia];
    vb[r] = p[ib];
  }
}

// Transposed product and store of this wave's output pairs.
template <typename T, class XF, class Wt>
__device__ __forceinline__ void store_lines_rb(const XF& xf, const WaveTiles& tl, int S,
                                               long long total, int tile, T* dst, char* smem, int b,
                                               const typename XF::Rows& me,
                                               const typename XF::Rows& mo, const T (&va)[4],
                                               const T (&vb)[4], Wt&& wt) {
  const float inv = xf.share(smem, b, va, vb);
  const int n = xf.n();
  const bool per = XF::LAYOUT == WL_EVEN && xf.ax.periodic;
  const int rows_e = per ? n / 2 + 1 : (n + 1) / 2;
  if (16 * xf.rb >= rows_e) return;
  T e[4], d[4];
  xf.template mul_shared<true>(smem, b, 0, me, e);
  xf.template mul_shared<true>(smem, b, 1, mo, d);
  const int m = 16 * xf.rb + xf.i;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = xf.tcol(r);
    int sp = c >> tl.cpsh;
    sp = sp < S ? sp : S - 1;
    long long ln = ((long long)tile << tl.cpsh) + (c & ((1 << tl.cpsh) - 1));
    ln = ln < tl.lines ? ln : tl.lines - 1;
    T* lp = dst + (sp * total + ln * n);
    if constexpr (XF::F32) {
      const float iv = __shfl(inv, 4 * xf.g + r, 64);
      e[r] *= iv;
      d[r] *= iv;
    }
    T x = per ? e[r] + d[r] : e[r], y = per ? e[r] - d[r] : d[r];
    if (!per) {
      x *= wt(ln, 2 * m, n);
      y *= wt(ln, 2 * m + 1, n);
      if (2 * m + 1 < n) {
        if constexpr (XF::F32)
          *reinterpret_cast<f32x2u*>(lp + 2 * m) = f32x2u{x, y};
        else
          *reinterpret_cast<f64x2u*>(lp + 2 * m) = f64x2u{x, y};
      } else if (2 * m < n) {
        lp[2 * m] = x;
      }
    } else if (2 * m <= n) {
      lp[m] = x;
      if (m > 0 && 2 * m < n) lp[n - m] = y;
    }
  }
}

// X of one tile (k_wx).
template <typename T, int NB, int LAY, bool SRC>
__global__ __launch_bounds__(64 * NB) void k_gx(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = GroupXf<T, NB, LAY>;
  using W = typename XF::W;
  const XF xf(ax);
  const long long total = a.g.total;
  const int tile = blockIdx.x;
  const XLane<T> ln(tl, a.S, tile, xf.i);
  T va[4] = {}, vb[4] = {};
  typename XF::Rows ma, mb, me, mo;
  if (xf.on) load_line_rb<T>(xf, a.P + ln.sp * total + ln.line * xf.n(), va, vb);
  xf.pair_rows(ma, mb);
  xf.nat_rows(me, mo);
  MmsLine ml{};
  if constexpr (SRC) ml = mms_line(a.rxn, a.t, ln.line % a.n1);
  xf.pair_shared(smem, 0, ma, mb, va, vb);
  if (xf.on) {
    const PosOff<W> po(xf, 1u, 0u);
    if (a.st_phys) {
      T* st = a.st_phys + (long long)a.mode * a.S * total;
      if (XF::EXACT && tl.priv) {
        struct alignas(sizeof(T) * 2) V { T v[4]; };
        T* p = st + (long long)tile * 16 * xf.n() + xf.rb * 512 + xf.lane * 4;
        *reinterpret_cast<V*>(p) = V{{va[0], va[1], va[2], va[3]}};
        *reinterpret_cast<V*>(p + 256) = V{{vb[0], vb[1], vb[2], vb[3]}};
      } else {
        T* p = st + ln.sp * total + ln.line * xf.n();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          unsigned ia, ib;
          po.at(po.lane, xf.rb, r, ia, ib);
          p[ia] = va[r];
          p[ib] = vb[r];
        }
      }
    }
    const RxnT<T> rx(a.rxn);
    T chk = T(0);
    const W& w = xf;
    if constexpr (SRC) {
      if (a.rxn.kind == RXN_HUXLEY_MMS)
        wave_react_rb<RXN_HUXLEY_MMS>(w, a, rx, ln, po, ml, xf.rb, va, vb, chk);
      else
        wave_react_rb<RXN_FISHER_MMS>(w, a, rx, ln, po, ml, xf.rb, va, vb, chk);
    } else {
      switch (a.rxn.kind) {  // uniform
        case RXN_LINEAR: wave_react_rb<RXN_LINEAR>(w, a, rx, ln, po, ml, xf.rb, va, vb, chk); break;
        case RXN_FHN: wave_react_rb<RXN_FHN>(w, a, rx, ln, po, ml, xf.rb, va, vb, chk); break;
        case RXN_GRAY_SCOTT: wave_react_rb<RXN_GRAY_SCOTT>(w, a, rx, ln, po, ml, xf.rb, va, vb, chk); break;
        case RXN_SCHNAKENBERG: wave_react_rb<RXN_SCHNAKENBERG>(w, a, rx, ln, po, ml, xf.rb, va, vb, chk); break;
        default: wave_react_rb<RXN_GM>(w, a, rx, ln, po, ml, xf.rb, va, vb, chk); break;
      }
    }
    if (!(chk == T(0))) a.flag[0] = 1;
  }
  store_lines_rb<T>(xf, tl, a.S, total, tile, a.P, smem, 1, me, mo, va, vb, NoWeight{});
}

// One transform of one x tile (k_wsx).
template <typename T, int NB, int LAY>
__global__ __launch_bounds__(64 * NB) void k_gsx(SingleArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = GroupXf<T, NB, LAY>;
  const XF xf(ax);
  const long long total = a.g.total;
  const int tile = blockIdx.x;
  const XLane<T> ln(tl, a.S, tile, xf.i);
  T va[4] = {}, vb[4] = {};
  typename XF::Rows me, mo;
  if (xf.on) load_line_rb<T>(xf, a.src + ln.sp * total + ln.line * xf.n(), va, vb);
  xf.nat_rows(me, mo);
  if (a.pre_divide_w) {
    const T wl = T(line_weight(ln.line, a.n1, a.n2));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      va[r] /= wl;
      vb[r] /= wl;
    }
    const T we = xf.g == 0 && xf.rb == 0 ? T(0.5) : T(1);
    va[0] /= we;
    vb[0] /= we;
  }
  if (a.post_multiply_w)
    store_lines_rb<T>(xf, tl, a.S, total, tile, a.dst, smem, 0, me, mo, va, vb,
                      [&](long long line, int e, int n) {
                        const T w = T(line_weight(line, a.n1, a.n2));
                        return e == 0 || e == n - 1 ? T(0.5) * w : w;
                      });
  else
    store_lines_rb<T>(xf, tl, a.S, total, tile, a.dst, smem, 0, me, mo, va, vb, NoWeight{});
}

// One transform of one strided tile (k_wsy).
template <typename T, int NB, int LAY>
__global__ __launch_bounds__(64 * NB) void k_gsy(SingleArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = GroupXf<T, NB, LAY>;
  using W = typename XF::W;
  const XF xf(ax);
  const W& w = xf;
  const StridedLane<T> ln(tl, xf.n(), blockIdx.x, xf.i);
  const RowIO<T, W> io(w, tl, ln);
  const auto of = io.offs(xf.rb);
  T va[4] = {}, vb[4] = {};
  typename XF::Rows ma, mb;
  if (xf.on) io.load(a.src, of, va, vb);
  xf.pair_rows(ma, mb);
  xf.pair_shared(smem, 0, ma, mb, va, vb);
  if (xf.on) io.store(a.dst, of, va, vb);
}

// Eigenvalues of this wave's positions and of the lane's column.
template <typename T, class XF>
__device__ __forceinline__ float group_lam(const XF& xf, const StageArgs<T>& a, unsigned ib,
                                           float (&lz)[2][4], int& x, int& y) {
  const PosOff<typename XF::W> po(xf, 1u, 0u);
  const double* lam = a.n2 > 1 ? a.lam[2] : a.lam[1];
  if (xf.on) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      unsigned ja, jb;
      po.at(po.lane, xf.rb, r, ja, jb);
      lz[0][r] = float(lam[ja]);
      lz[1][r] = float(lam[jb]);
    }
  }
  const unsigned n0 = (unsigned)a.n0;
  y = a.n2 > 1 ? (int)(ib / n0) : 0;
  x = (int)(ib - (unsigned)y * n0);
  const float lx = float(a.lam[0][x]);
  return a.n2 > 1 ? lx + float(a.lam[1][y]) : lx;
}

// Z of one tile (k_wz).
template <typename T, int NB, int LAY, int MODE, int CO>
__global__ __launch_bounds__(64 * NB) void k_gz(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = GroupXf<T, NB, LAY>;
  using W = typename XF::W;
  const XF xf(ax);
  const W& w = xf;
  const StridedLane<T> ln(tl, xf.n(), blockIdx.x, xf.i);
  const RowIO<T, W> io(w, tl, ln, blockIdx.x, CO == CO_FLY || tl.priv);
  const auto of = io.offs(xf.rb);
  T va[4] = {}, vb[4] = {};
  typename XF::Rows ma, mb;
  if (xf.on) io.load(a.src ? a.src : a.P, of, va, vb);
  CombineIn<T> in = {};
  if (MODE >= 0 && xf.on) {
    if (MODE <= 1)
      io.load(a.uhat, of, in.x1[0], in.x1[1]);
    else
      io.load_priv(a.acc, xf.rb, of, in.x1[0], in.x1[1]);
    wave_combine_in<MODE, CO>(io, a, xf.rb, in);
  }
  xf.pair_rows(ma, mb);
  float lz[2][4] = {}, lxy = 0.f;
  T kt = T(0), ha = T(0);
  if constexpr (CO == CO_FLY) {
    int x, y;
    lxy = group_lam(xf, a, ln.ib, lz, x, y);
    kt = pick_species(a.kt, ln.o);
    ha = pick_species(a.ha, ln.o);
  }
  if (MODE >= 0 || !a.src) xf.pair_shared(smem, 0, ma, mb, va, vb);
  if constexpr (MODE >= 0) {
    if (xf.on) wave_combine_out<MODE, CO>(io, a, xf.rb, lxy, kt, ha, lz, in, va, vb);
  } else {
    if (a.mode == MODE_INIT && xf.on) io.store(a.uhat, of, va, vb);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      va[r] *= a.cs;
      vb[r] *= a.cs;
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    keep(va[r]);
    keep(vb[r]);
  }
  xf.pair_shared(smem, 1, ma, mb, va, vb);
  if (xf.on) io.store(a.P, of, va, vb);
}

// X adjoint of one tile (k_wxadj).
template <typename T, int NB, int LAY, bool WP>
__global__ __launch_bounds__(64 * NB) void k_gxadj(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = GroupXf<T, NB, LAY>;
  using W = typename XF::W;
  const XF xf(ax);
  const W& w = xf;
  const long long total = a.g.total;
  const int tile = blockIdx.x;
  const XLane<T> ln(tl, a.S, tile, xf.i);
  T va[4] = {}, vb[4] = {}, ua[4] = {}, ub[4] = {};
  typename XF::Rows ma, mb, me, mo;
  if (xf.on) {
    load_line_rb<T>(xf, a.P + ln.sp * total + ln.line * xf.n(), va, vb);
    const StageIn<T, W> in(w, tl, ln, tile, total, a.st_phys + (long long)a.mode * a.S * total);
    in.load(xf.rb, ua, ub);
  }
  xf.pair_rows(ma, mb);
  xf.nat_rows(me, mo);
  double pacc[RXN_NP_MAX];
#pragma unroll
  for (int k = 0; k < RXN_NP_MAX; ++k) pacc[k] = 0.0;
  xf.pair_shared(smem, 0, ma, mb, va, vb);
  if (xf.on) {
    switch (a.rxn.kind) {  // uniform
      case RXN_LINEAR: wave_adj_react_rb<RXN_LINEAR, WP>(w, a, ln, xf.rb, va, vb, ua, ub, pacc); break;
      case RXN_FHN: wave_adj_react_rb<RXN_FHN, WP>(w, a, ln, xf.rb, va, vb, ua, ub, pacc); break;
      case RXN_GRAY_SCOTT: wave_adj_react_rb<RXN_GRAY_SCOTT, WP>(w, a, ln, xf.rb, va, vb, ua, ub, pacc); break;
      case RXN_SCHNAKENBERG: wave_adj_react_rb<RXN_SCHNAKENBERG, WP>(w, a, ln, xf.rb, va, vb, ua, ub, pacc); break;
      case RXN_GM: wave_adj_react_rb<RXN_GM, WP>(w, a, ln, xf.rb, va, vb, ua, ub, pacc); break;
      case RXN_HUXLEY_MMS: wave_adj_react_rb<RXN_HUXLEY_MMS, WP>(w, a, ln, xf.rb, va, vb, ua, ub, pacc); break;
      default: wave_adj_react_rb<RXN_FISHER_MMS, WP>(w, a, ln, xf.rb, va, vb, ua, ub, pacc); break;
    }
  }
  store_lines_rb<T>(xf, tl, a.S, total, tile, a.P, smem, 1, me, mo, va, vb, NoWeight{});
  // (buffer 0 was last read before the barrier inside the call above)
  if constexpr (WP) block_add_partials(reinterpret_cast<double*>(smem), pacc, a.rxn.np, a.rp_acc);
}

// Z adjoint of one tile (k_wzadj).
template <typename T, int NB, int LAY, int MODE, bool TH>
__global__ __launch_bounds__(64 * NB) void k_gzadj(StageArgs<T> a, WaveAxis ax, WaveTiles tl) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using XF = GroupXf<T, NB, LAY>;
  using W = typename XF::W;
  const XF xf(ax);
  const W& w = xf;
  const StridedLane<T> ln(tl, xf.n(), blockIdx.x, xf.i);
  const RowIO<T, W> io(w, tl, ln, blockIdx.x, MODE >= 0 || tl.priv);
  const auto of = io.offs(xf.rb);
  T va[4] = {}, vb[4] = {};
  typename XF::Rows ma, mb;
  if (xf.on) io.load(a.P, of, va, vb);
  AdjIn in[2] = {};
  if constexpr (MODE >= 0) {
    if (xf.on) {
      wave_adj_fly_in<MODE, TH, 0>(io, a, xf.rb, in[0]);
      wave_adj_fly_in<MODE, TH, 1>(io, a, xf.rb, in[1]);
    }
  }
  xf.pair_rows(ma, mb);
  float lz[2][4] = {}, lxy = 0.f;
  int x = 0, y = 0;
  if constexpr (MODE >= 0) lxy = group_lam(xf, a, ln.ib, lz, x, y);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  xf.pair_shared(smem, 0, ma, mb, va, vb);
  if (xf.on) {
    if constexpr (MODE >= 0) {
      const float kt = pick_species(a.kt, ln.o), ha = pick_species(a.ha, ln.o);
      float wxy = ln.ok ? a.cs : 0.f;
      if (a.neumann) {
        if (x == 0 || x == (int)a.n0 - 1) wxy *= 0.5f;
        if (a.n2 > 1 && (y == 0 || y == (int)a.n1 - 1)) wxy *= 0.5f;
      }
      double sk = 0.0, sa = 0.0;
      wave_adj_fly<MODE, TH, 0>(w, io, a, xf.rb, lxy, wxy, kt, ha, lz[0], in[0], va, sk, sa);
      wave_adj_fly<MODE, TH, 1>(w, io, a, xf.rb, lxy, wxy, kt, ha, lz[1], in[1], vb, sk, sa);
      if constexpr (TH && MODE <= 2) {
        acc[0] += ln.o == 0 ? sk : 0.0;
        acc[1] += ln.o == 0 ? sa : 0.0;
        acc[2] += ln.o == 0 ? 0.0 : sk;
        acc[3] += ln.o == 0 ? 0.0 : sa;
      }
    } else {
      wave_adj_tab<0>(io, a, xf.rb, va);
      wave_adj_tab<1>(io, a, xf.rb, vb);
    }
  }
  xf.pair_shared(smem, 1, ma, mb, va, vb);
  if (xf.on) io.store(a.P, of, va, vb);
  if constexpr (TH && MODE >= 0 && MODE <= 2)
    block_sums(reinterpret_cast<double*>(smem), acc, 2 * a.S, a.thp, true);
}

// ------------------------------------------------------------------ kernel table
// The kernels of one (type, size class, layout), for hipLaunchKernel.
enum {
  WK_X = 0,   // X
  WK_XSRC,    // X with a manufactured source (not in exact classes)
  WK_SX,      // one transform, x axis
  WK_SY,      // one transform, strided axis
  WK_SY2,     // the same with two columns per lane (FP32, even inner extent)
  WK_ZINIT,   // Z: MODE_INIT, MODE_RESTORE
  WK_Z,       // Z stages 0..3, the table of L
  WK_ZTABS = WK_Z + 4,    // Z stages, the tables of the coefficients
  WK_ZFLY = WK_ZTABS + 4,  // Z stages with L formed in the kernel (FP32, not odd axes)
  WK_XADJ = WK_ZFLY + 4,  // X adjoint, without / with parameter partials
  WK_ZADJ = WK_XADJ + 2,  // Z adjoint from tables
  WK_ZADJFLY,             // Z adjoint, L formed in the kernel: modes 0 .. MODE_INIT
  WK_ZADJTH = WK_ZADJFLY + 5,  // ... with kappa / alpha partials: modes 0 .. 2
  WK_COUNT = WK_ZADJTH + 3
};
struct WaveKernels {
  const void* fn[WK_COUNT];   // wave kernels
  const void* grp[WK_COUNT];  // group kernels (none for WK_SY2)
  int nb, layout, threads;
  size_t tab_bytes, lds_a;  // matrix table; its copy in LDS (0: read from global memory)
  size_t lds_g;             // LDS of the group kernels
};

template <typename T, int NB, int LAY, bool FN, int MODE = 3>
void wave_z_kernels(WaveKernels& k) {
  constexpr bool FLY = LAY != WL_ODD && sizeof(T) == 4 && FN;
  k.grp[WK_Z + MODE] = reinterpret_cast<const void*>(&k_gz<T, NB, LAY, MODE, CO_LTAB>);
  k.grp[WK_ZTABS + MODE] = reinterpret_cast<const void*>(&k_gz<T, NB, LAY, MODE, CO_TABS>);
  if constexpr (FLY) k.grp[WK_ZFLY + MODE] = reinterpret_cast<const void*>(&k_gz<T, NB, LAY, MODE, CO_FLY>);
  if constexpr (FN) {
    k.fn[WK_Z + MODE] = reinterpret_cast<const void*>(&k_wz<T, NB, LAY, MODE, CO_LTAB>);
    k.fn[WK_ZTABS + MODE] = reinterpret_cast<const void*>(&k_wz<T, NB, LAY, MODE, CO_TABS>);
  }
  if constexpr (FLY) k.fn[WK_ZFLY + MODE] = reinterpret_cast<const void*>(&k_wz<T, NB, LAY, MODE, CO_FLY>);
  if constexpr (MODE > 0) wave_z_kernels<T, NB, LAY, FN, MODE - 1>(k);
}

template <typename T, int NB, int LAY, int MODE = MODE_INIT>
void wave_zadj_kernels(WaveKernels& k) {
  k.fn[WK_ZADJFLY + MODE] = reinterpret_cast<const void*>(&k_wzadj<T, NB, LAY, MODE, false>);
  k.grp[WK_ZADJFLY + MODE] = reinterpret_cast<const void*>(&k_gzadj<T, NB, LAY, MODE, false>);
  if constexpr (MODE <= 2) {
    k.fn[WK_ZADJTH + MODE] = reinterpret_cast<const void*>(&k_wzadj<T, NB, LAY, MODE, true>);
    k.grp[WK_ZADJTH + MODE] = reinterpret_cast<const void*>(&k_gzadj<T, NB, LAY, MODE, true>);
  }
  if constexpr (MODE > 0) wave_zadj_kernels<T, NB, LAY, MODE - 1>(k);
}

// FN: with the wave kernels; classes past 288 points have the group kernels
// only (a wave cannot hold 16 of their lines).
template <typename T, int NB, int LAY, bool FN = (NB <= 9)>
WaveKernels wave_kernels() {
  WaveKernels k{};
  k.nb = NB;
  k.layout = LAY;
  k.threads = wave_threads<T, NB>();
  k.tab_bytes = WaveTab<T, NB>::bytes;
  k.lds_a = wave_lds_a<T, NB>() ? WaveTab<T, NB>::bytes : 0;
  k.lds_g = GroupXf<T, NB, LAY>::lds_bytes();
  k.grp[WK_X] = reinterpret_cast<const void*>(&k_gx<T, NB, LAY, false>);
  if constexpr (LAY != WL_EXACT)
    k.grp[WK_XSRC] = reinterpret_cast<const void*>(&k_gx<T, NB, LAY, true>);
  k.grp[WK_SX] = reinterpret_cast<const void*>(&k_gsx<T, NB, LAY>);
  k.grp[WK_SY] = reinterpret_cast<const void*>(&k_gsy<T, NB, LAY>);
  k.grp[WK_ZINIT] = reinterpret_cast<const void*>(&k_gz<T, NB, LAY, -1, CO_LTAB>);
  k.grp[WK_XADJ] = reinterpret_cast<const void*>(&k_gxadj<T, NB, LAY, false>);
  k.grp[WK_XADJ + 1] = reinterpret_cast<const void*>(&k_gxadj<T, NB, LAY, true>);
  k.grp[WK_ZADJ] = reinterpret_cast<const void*>(&k_gzadj<T, NB, LAY, -1, false>);
  wave_z_kernels<T, NB, LAY, FN>(k);
  if constexpr (FN) {
    k.fn[WK_X] = reinterpret_cast<const void*>(&k_wx<T, NB, LAY, false>);
    if constexpr (LAY != WL_EXACT)
      k.fn[WK_XSRC] = reinterpret_cast<const void*>(&k_wx<T, NB, LAY, true>);
    k.fn[WK_SX] = reinterpret_cast<const void*>(&k_wsx<T, NB, LAY>);
    k.fn[WK_SY] = reinterpret_cast<const void*>(&k_wsy<T, NB, LAY>);
    if constexpr (sizeof(T) == 4) k.fn[WK_SY2] = reinterpret_cast<const void*>(&k_wsy2<NB, LAY>);
    k.fn[WK_ZINIT] = reinterpret_cast<const void*>(&k_wz<T, NB, LAY, -1, CO_LTAB>);
    k.fn[WK_XADJ] = reinterpret_cast<const void*>(&k_wxadj<T, NB, LAY, false>);
    k.fn[WK_XADJ + 1] = reinterpret_cast<const void*>(&k_wxadj<T, NB, LAY, true>);
    k.fn[WK_ZADJ] = reinterpret_cast<const void*>(&k_wzadj<T, NB, LAY, -1, false>);
    if constexpr (LAY != WL_ODD && sizeof(T) == 4) wave_zadj_kernels<T, NB, LAY>(k);
  }
  return k;
}

}  // namespace sfrde
