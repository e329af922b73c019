// Hartley transforms of periodic axes of N = 256, 512 and 1024 points as
// radix-8/4 complex FFTs, one pair of lines per wavefront.
//
// The periodic operator's eigenvalues satisfy lambda_k = lambda_{N-k}
// (Section 3.1), so the real Hartley basis cas(2 pi jk/N) = cos + sin
// diagonalises it like the complex Fourier basis of Alg. 1's fftn. Two real
// lines a, b are transformed together as one complex sequence z = a + i b:
// with Z = DFT(z) and Z'_k = Z_{(N-k) mod N},
//   H(a)_k = (Re Z_k + Re Z'_k - Im Z_k + Im Z'_k) / 2
//   H(b)_k = (Re Z_k - Re Z'_k + Im Z_k + Im Z'_k) / 2
// (Re and Im of the DFT of a real line are its cosine sum and minus its sine
// sum; the halves separate a and b by the conjugate symmetry of a real
// line's DFT). The Hartley transform is its own inverse up to 1/N, which the
// stage combine applies, so one routine serves both directions.
//
// The complex DFT is a Stockham autosort FFT (no bit reversal): stage by
// stage, butterfly j of span Ns reads x[j + r N/R], r < R, multiplies input r
// by e^{-2 pi i r k / (Ns R)} with k = j mod Ns, takes the radix-R DFT, and
// writes x[(j - k) R + k + r Ns]. Lane l of the wavefront holds the points
// l + 64 e of its two lines in registers. That is exactly what its butterflies
// l, l + 64, ... of any stage read, so a stage is register work and one
// exchange through the wavefront's own LDS (written in the stage's output
// order, read back at l + 64 e). Nothing is shared between wavefronts: there
// is no barrier, and the launch can be cut into blocks of any size.
//
// The two lines of a pair are of one species: H(a) and H(b) are separated from
// sums of both, so each carries rounding errors of the size of the larger line
// (with the two species of a row as a pair, a species 10^-6 of the other came
// out 2 % off in FP32). On the x axis they are neighbouring rows, and the
// wavefronts of a row pair's two species sit side by side in one block and trade
// lines through LDS for the reaction; on strided axes
// they are neighbouring columns of one outer block. Twiddles (cos, sin of
// 2 pi m / N) come from a table built in FP64 on the host.
//
// A launch of 512^2 points is bound by the length of one wavefront's chain
// (512 wavefronts on 256 CUs). Gray-Scott steps against blocks of 256 threads
// with the tile in LDS, two of four wavefronts in the FFT and block barriers
// between stages: 512^2 155 -> 78 us (x launches 14.4 -> 6.5, the last axis' 22.4 ->
// 12.7; FP64 168 -> 96); 1024^2 363 -> 258 (FP64 416 -> 290); FHN 256^3 6.99 ->
// 4.00 ms (FP64 8.80 -> 4.95). Trading lines costs three barriers per x launch: with
// the two species of a row as a pair these steps took 76 (93), 255 (282) us and 4.03
// (4.85) ms. (Showing the other wavefront both lines, two barriers but every
// reaction twice: FP64 97 us, 512^2; adjoint of 1024^2 FP64 5.01 ms against 4.76.)
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"
#include "wave.h"

namespace sfrde {

// Radix-R DFT (e^{-2 pi i rk/R}) of v in place, R = 4 or 8.
template <typename T>
__device__ __forceinline__ void dft4(T& r0, T& i0, T& r1, T& i1, T& r2, T& i2, T& r3, T& i3) {
  const T t0r = r0 + r2, t0i = i0 + i2, t1r = r0 - r2, t1i = i0 - i2;
  const T t2r = r1 + r3, t2i = i1 + i3, t3r = r1 - r3, t3i = i1 - i3;
  r0 = t0r + t2r;
  i0 = t0i + t2i;
  r2 = t0r - t2r;
  i2 = t0i - t2i;
  // X1 = t1 - i t3, X3 = t1 + i t3
  r1 = t1r + t3i;
  i1 = t1i - t3r;
  r3 = t1r - t3i;
  i3 = t1i + t3r;
}

template <typename T, int R>
__device__ __forceinline__ void dft_r(T (&vr)[R], T (&vi)[R]) {
  if constexpr (R == 4) {
    dft4(vr[0], vi[0], vr[1], vi[1], vr[2], vi[2], vr[3], vi[3]);
  } else {
    static_assert(R == 8, "radix 4 or 8");
    // even and odd halves, then X_k = E_k + W8^k O_k, X_{k+4} = E_k - W8^k O_k
    T er[4] = {vr[0], vr[2], vr[4], vr[6]}, ei[4] = {vi[0], vi[2], vi[4], vi[6]};
    T orr[4] = {vr[1], vr[3], vr[5], vr[7]}, oi[4] = {vi[1], vi[3], vi[5], vi[7]};
    dft4(er[0], ei[0], er[1], ei[1], er[2], ei[2], er[3], ei[3]);
    dft4(orr[0], oi[0], orr[1], oi[1], orr[2], oi[2], orr[3], oi[3]);
    const T h = T(0.70710678118654752440);  // 1/sqrt(2)
    T wr[4], wi[4];
    wr[0] = orr[0];
    wi[0] = oi[0];
    wr[1] = (orr[1] + oi[1]) * h;  // (1 - i)/sqrt2
    wi[1] = (oi[1] - orr[1]) * h;
    wr[2] = oi[2];  // -i
    wi[2] = -orr[2];
    wr[3] = (oi[3] - orr[3]) * h;  // (-1 - i)/sqrt2
    wi[3] = -(orr[3] + oi[3]) * h;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      vr[k] = er[k] + wr[k];
      vi[k] = ei[k] + wi[k];
      vr[k + 4] = er[k] - wr[k];
      vi[k + 4] = ei[k] - wi[k];
    }
  }
}

// One pair of lines in registers: lane l holds points l + 64 e.
template <typename T, int N>
struct WaveFft {
  static constexpr int E = N / 64;
  using Vals = T[E];
  // LDS of one wavefront: real and imaginary parts, one spare word after every
  // eight (the strides of a stage's writes then spread over the banks)
  static constexpr int PART = N + N / 8;
  static constexpr size_t lds_bytes() { return (size_t)2 * PART * sizeof(T); }
  T *xr, *xi;
  int lane;
  // this lane's twiddles, read once for both transforms of a launch
  static constexpr int NTW = N == 256 ? 9 : N == 512 ? 14 : 22;
  T wc[NTW], ws[NTW];
  // tw: [N][2] cos, sin of 2 pi m / N
  __device__ __forceinline__ WaveFft(char* smem, const T* tw) {
    lane = threadIdx.x & 63;
    xr = reinterpret_cast<T*>(smem + (size_t)(threadIdx.x >> 6) * lds_bytes());
    xi = xr + PART;
    if constexpr (N == 256) {
      twiddles<4, 4, 0>(tw);
      twiddles<4, 16, 3>(tw);
      twiddles<4, 64, 6>(tw);
    } else if constexpr (N == 512) {
      twiddles<8, 8, 0>(tw);
      twiddles<8, 64, 7>(tw);
    } else {
      static_assert(N == 1024, "N = 256, 512 or 1024");
      twiddles<8, 8, 0>(tw);
      twiddles<4, 64, 7>(tw);
      twiddles<4, 256, 10>(tw);
    }
  }
  // Distinct twiddle sets of a lane's butterflies lane + 64 b in a stage of
  // span NS (k = butterfly mod NS).
  template <int NS>
  static constexpr int sets() { return NS > 64 ? NS / 64 : 1; }
  template <int R, int NS, int W0>
  __device__ __forceinline__ void twiddles(const T* tw) {
#pragma unroll
    for (int b = 0; b < sets<NS>(); ++b)
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const int m = r * ((lane + 64 * b) & (NS - 1)) * (N / (NS * R));  // < N
        wc[W0 + b * (R - 1) + r - 1] = tw[2 * m];
        ws[W0 + b * (R - 1) + r - 1] = tw[2 * m + 1];
      }
  }
  __device__ __forceinline__ static int at(int i) { return i + (i >> 3); }
  // The wavefront's LDS accesses complete in order; this keeps the compiler's
  // order, too.
  __device__ __forceinline__ static void sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  template <int R, int NS, int W0 = 0>
  __device__ __forceinline__ void stage(Vals& vr, Vals& vi) const {
    constexpr int NB = N / R, B = NB / 64;
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int j = lane + 64 * b, k = j & (NS - 1);
      T br[R], bi[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        br[r] = vr[b + B * r];
        bi[r] = vi[b + B * r];
      }
      if constexpr (NS > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const int w = W0 + (b % sets<NS>()) * (R - 1) + r - 1;
          const T c = wc[w], s = ws[w];
          const T ar = br[r], ai = bi[r];
          br[r] = ar * c + ai * s;  // times e^{-i theta}
          bi[r] = ai * c - ar * s;
        }
      }
      dft_r<T, R>(br, bi);
      const int base = (j - k) * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        xr[at(base + r * NS)] = br[r];
        xi[at(base + r * NS)] = bi[r];
      }
    }
    sync();
  }
  __device__ __forceinline__ void read(Vals& vr, Vals& vi) const {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      vr[e] = xr[at(lane + 64 * e)];
      vi[e] = xi[at(lane + 64 * e)];
    }
    sync();
  }
  // What this wavefront gives for what the wavefront of the other species gives, by
  // half `part` of the buffers (one barrier; one more before that half is written
  // again).
  __device__ __forceinline__ void trade(int part, const Vals& give, Vals& got) const {
    T* m = part ? xi : xr;
#pragma unroll
    for (int e = 0; e < E; ++e) m[at(lane + 64 * e)] = give[e];
    __syncthreads();
    const T* o = (threadIdx.x >> 6) & 1 ? m - 2 * PART : m + 2 * PART;
#pragma unroll
    for (int e = 0; e < E; ++e) got[e] = o[at(lane + 64 * e)];
  }
  // Hartley transforms of the lines in a and b, in place.
  __device__ __forceinline__ void hartley(Vals& a, Vals& b) const {
    if constexpr (N == 256) {
      stage<4, 1>(a, b);
      read(a, b);
      stage<4, 4>(a, b);
      read(a, b);
      stage<4, 16, 3>(a, b);
      read(a, b);
      stage<4, 64, 6>(a, b);
    } else if constexpr (N == 512) {
      stage<8, 1>(a, b);
      read(a, b);
      stage<8, 8>(a, b);
      read(a, b);
      stage<8, 64, 7>(a, b);
    } else {
      stage<8, 1>(a, b);
      read(a, b);
      stage<8, 8>(a, b);
      read(a, b);
      stage<4, 64, 7>(a, b);
      read(a, b);
      stage<4, 256, 10>(a, b);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int k = lane + 64 * e, kk = (N - k) & (N - 1);
      const T zr = xr[at(k)], zi = xi[at(k)], wr = xr[at(kk)], wi = xi[at(kk)];
      a[e] = T(0.5) * ((zr + wr) - (zi - wi));
      b[e] = T(0.5) * ((zr - wr) + (zi + wi));
    }
    sync();
  }
};

// Pairs of an axis. x axis: pair q holds lines 2k, 2k + 1 of species q mod S, k =
// q / S (the species of one k are neighbours). Strided: pair q holds columns 2k,
// 2k + 1 of outer block q / per, k = q mod per. A last line without a partner is
// repeated (and stored twice).
struct FftPairs {
  long long lines;   // x: per species
  long long inner;   // strided
  int npairs;
  int per;           // strided: pairs per outer block
};

// The wavefront's pair, -1 past the last. Blocks are dealt to the XCDs in turn;
// neighbouring pairs (which share cache lines on strided axes) go to one XCD.
__device__ __forceinline__ int fft_pair(int npairs) {
  const int nb = (int)gridDim.x, per = nb / 8;
  const int b = (int)blockIdx.x;
  const int g = b < 8 * per ? (b & 7) * per + (b >> 3) : b;
  const int q = g * (int)(blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return q < npairs ? q : -1;
}

struct FftXPair {
  long long la, lb;  // lines
  int sp;            // species
  __device__ __forceinline__ FftXPair(const FftPairs& fp, int S, int q) {
    const unsigned k = (unsigned)q / (unsigned)S;
    sp = (int)((unsigned)q - k * (unsigned)S);
    la = 2LL * k;
    lb = la + 1 < fp.lines ? la + 1 : la;
  }
};

// Barriers of a reaction that couples two species (fft_react, fft_adj_react).
constexpr int FFT_TRADE_BARRIERS = 3;
// Whether the reaction couples two species (their wavefronts exchange values).
__device__ __forceinline__ bool fft_coupled(int kind) {
  return kind >= RXN_FHN && kind <= RXN_GM;  // uniform
}

// Column pair of a strided axis, with the interface of RowIO (wave.h): "side"
// a / b are the two columns, row block rb the points lane + 64 (4 rb + r).
template <typename T>
struct FftCols {
  static constexpr bool EXACT = true;  // every point counts once
  long long oa, ob, step;              // elements; step: 64 rows
  bool adj;                            // b follows a in memory
  __device__ __forceinline__ FftCols(const FftPairs& fp, int n, int q, int lane) {
    const unsigned o = (unsigned)q / (unsigned)fp.per, c = 2u * ((unsigned)q - o * (unsigned)fp.per);
    adj = c + 1u < (unsigned)fp.inner;
    oa = ((long long)o * n + lane) * fp.inner + c;
    ob = oa + (adj ? 1 : 0);
    step = 64 * fp.inner;
  }
  struct Off {
    long long a[4], b[4];
    bool adj;
  };
  __device__ __forceinline__ Off offs(int rb) const {
    Off o;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      o.a[r] = oa + (4 * rb + r) * step;
      o.b[r] = ob + (4 * rb + r) * step;
    }
    o.adj = adj;
    return o;
  }
  template <typename U>
  struct alignas(sizeof(U)) Two {
    U x, y;
  };
  template <typename U>
  __device__ __forceinline__ void load(const U* f, const Off& o, U (&va)[4], U (&vb)[4]) const {
    if (o.adj) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const Two<U> t = *reinterpret_cast<const Two<U>*>(f + o.a[r]);
        va[r] = t.x;
        vb[r] = t.y;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        va[r] = f[o.a[r]];
        vb[r] = f[o.b[r]];
      }
    }
  }
  template <typename U>
  __device__ __forceinline__ void store(U* f, const Off& o, const U (&va)[4], const U (&vb)[4]) const {
    if (o.adj) {
#pragma unroll
      for (int r = 0; r < 4; ++r) *reinterpret_cast<Two<U>*>(f + o.a[r]) = Two<U>{va[r], vb[r]};
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        f[o.a[r]] = va[r];
        f[o.b[r]] = vb[r];
      }
    }
  }
  template <typename U>
  __device__ __forceinline__ void load1(const U* f, const long long (&o)[4], U (&v)[4]) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = f[o[r]];
  }
  template <typename U>
  __device__ __forceinline__ void store1(U* f, const long long (&o)[4], const U (&v)[4]) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) f[o[r]] = v[r];
  }
  // (private arrays of the stage combines have the fields' order here)
  template <typename U>
  __device__ __forceinline__ void load_priv(const U* f, int, const Off& o, U (&va)[4], U (&vb)[4]) const {
    load(f, o, va, vb);
  }
  template <typename U>
  __device__ __forceinline__ void store_priv(U* f, int, const Off& o, const U (&va)[4], const U (&vb)[4]) const {
    store(f, o, va, vb);
  }
  template <int SIDE, typename U>
  __device__ __forceinline__ void load_priv1(const U* f, int, const long long (&o)[4], U (&v)[4]) const {
    load1(f, o, v);
  }
  template <int SIDE, typename U>
  __device__ __forceinline__ void store_priv1(U* f, int, const long long (&o)[4], const U (&v)[4]) const {
    store1(f, o, v);
  }
  template <int SIDE, typename U>
  __device__ __forceinline__ void store_priv_rmw(U* f, int rb, const long long (&o)[4], const U (&v)[4]) const {
    store_rmw<SIDE>(f, o, v, rb);
  }
  // an array that this pass also read: a repeated last column (b on a) is
  // written from side a only
  template <int SIDE, typename U>
  __device__ __forceinline__ void store_rmw(U* f, const long long (&o)[4], const U (&v)[4], int) const {
    if (SIDE == 0 || ob != oa) store1(f, o, v);
  }
  template <int E>
  __device__ __forceinline__ void load_all(const T* f, T (&a)[E], T (&b)[E]) const {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      T va[4], vb[4];
      load(f, offs(q), va, vb);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        a[4 * q + r] = va[r];
        b[4 * q + r] = vb[r];
      }
    }
  }
  template <int E>
  __device__ __forceinline__ void store_all(T* f, const T (&a)[E], const T (&b)[E]) const {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      T va[4], vb[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        va[r] = a[4 * q + r];
        vb[r] = b[4 * q + r];
      }
      store(f, offs(q), va, vb);
    }
  }
};

template <int E, typename T>
__device__ __forceinline__ void fft_load_line(const T* p, int lane, T (&v)[E]) {
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = p[lane + 64 * e];
}
template <int E, typename T>
__device__ __forceinline__ void fft_store_line(T* p, int lane, const T (&v)[E]) {
#pragma unroll
  for (int e = 0; e < E; ++e) p[lane + 64 * e] = v[e];
}

// f of the pair's stage values; true if a value was not finite. Two coupled species:
// line a in the wavefront of species 0, line b in that of species 1; the wavefronts
// trade lines before and after.
template <int KIND, typename T, class FT>
__device__ __forceinline__ bool fft_react(const StageArgs<T>& a, const FftXPair& pr, const FT& ft,
                                          T (&va)[FT::E], T (&vb)[FT::E]) {
  const RxnT<T> rx(a.rxn);
  const int sp = pr.sp;  // uniform
  T chk = T(0);
  if constexpr (KIND >= RXN_FHN && KIND <= RXN_GM) {
    T give[FT::E], got[FT::E];
#pragma unroll
    for (int e = 0; e < FT::E; ++e) give[e] = sp == 0 ? vb[e] : va[e];
    ft.trade(0, give, got);
#pragma unroll
    for (int e = 0; e < FT::E; ++e) {
      const T own = sp == 0 ? va[e] : vb[e];
      const T u[2] = {sp == 0 ? own : got[e], sp == 0 ? got[e] : own};
      T f[2];
      rxn_eval_k<T, 2, KIND>(rx, u, f);
      chk = fma(u[0], T(0), chk);
      chk = fma(u[1], T(0), chk);
      chk = fma(f[0], T(0), chk);
      chk = fma(f[1], T(0), chk);
      va[e] = sp == 0 ? f[0] : f[1];
      give[e] = sp == 0 ? f[1] : f[0];
    }
    ft.trade(1, give, got);
#pragma unroll
    for (int e = 0; e < FT::E; ++e) {
      const T own = va[e];
      va[e] = sp == 0 ? own : got[e];
      vb[e] = sp == 0 ? got[e] : own;
    }
    __syncthreads();
  } else {
    const T lin = sp == 0 ? rx.lin[0] : sp == 1 ? rx.lin[1] : sp == 2 ? rx.lin[2] : rx.lin[3];
    MmsLine ml[2] = {};
    if constexpr (KIND >= RXN_HUXLEY_MMS) {
      ml[0] = mms_line(a.rxn, a.t, pr.la % a.n1);
      ml[1] = mms_line(a.rxn, a.t, pr.lb % a.n1);
    }
#pragma unroll
    for (int e = 0; e < FT::E; ++e) {
      const T u[2] = {va[e], vb[e]};
      T f[2];
      if constexpr (KIND == RXN_LINEAR) {
        f[0] = lin * u[0];
        f[1] = lin * u[1];
      } else {
        rxn_eval_k<T, 1, KIND>(rx, &u[0], &f[0]);
        rxn_eval_k<T, 1, KIND>(rx, &u[1], &f[1]);
        f[0] += T(mms_source<KIND>(ml[0], ft.lane + 64 * e));
        f[1] += T(mms_source<KIND>(ml[1], ft.lane + 64 * e));
      }
      chk = fma(u[0], T(0), chk);
      chk = fma(u[1], T(0), chk);
      chk = fma(f[0], T(0), chk);
      chk = fma(f[1], T(0), chk);
      va[e] = f[0];
      vb[e] = f[1];
    }
  }
  return !(chk == T(0));
}

// X: inverse-x, reaction, forward-x (in place on P). SRC: manufactured sources
// (a call, whose stack the other plans' kernel does without).
template <typename T, int N, bool SRC>
__global__ __launch_bounds__(256) void k_fx(StageArgs<T> a, FftPairs fp) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  const WaveFft<T, N> ft(smem, a.Mt);
  const int q = fft_pair(fp.npairs);
  if (q < 0) {
    if (!SRC && fft_coupled(a.rxn.kind))
      for (int k = 0; k < FFT_TRADE_BARRIERS; ++k) __syncthreads();
    return;
  }
  const FftXPair pr(fp, a.S, q);
  const long long oa = pr.sp * a.g.total + pr.la * N, ob = pr.sp * a.g.total + pr.lb * N;
  typename WaveFft<T, N>::Vals va, vb;
  fft_load_line(a.P + oa, ft.lane, va);
  fft_load_line(a.P + ob, ft.lane, vb);
  ft.hartley(va, vb);
  if (a.st_phys) {
    T* st = a.st_phys + (long long)a.mode * a.S * a.g.total;
    fft_store_line(st + oa, ft.lane, va);
    fft_store_line(st + ob, ft.lane, vb);
  }
  bool bad;
  if constexpr (SRC) {
    bad = a.rxn.kind == RXN_HUXLEY_MMS ? fft_react<RXN_HUXLEY_MMS>(a, pr, ft, va, vb)
                                       : fft_react<RXN_FISHER_MMS>(a, pr, ft, va, vb);
  } else {
    switch (a.rxn.kind) {  // uniform
      case RXN_LINEAR: bad = fft_react<RXN_LINEAR>(a, pr, ft, va, vb); break;
      case RXN_FHN: bad = fft_react<RXN_FHN>(a, pr, ft, va, vb); break;
      case RXN_GRAY_SCOTT: bad = fft_react<RXN_GRAY_SCOTT>(a, pr, ft, va, vb); break;
      case RXN_SCHNAKENBERG: bad = fft_react<RXN_SCHNAKENBERG>(a, pr, ft, va, vb); break;
      default: bad = fft_react<RXN_GM>(a, pr, ft, va, vb); break;
    }
  }
  if (bad) a.flag[0] = 1;
  ft.hartley(va, vb);
  fft_store_line(a.P + oa, ft.lane, va);
  fft_store_line(a.P + ob, ft.lane, vb);
}

// One transform along the x axis, src -> dst (may alias). (Neumann point
// weights never apply: the axis is periodic.)
template <typename T, int N>
__global__ __launch_bounds__(256) void k_fsx(SingleArgs<T> a, FftPairs fp) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  const WaveFft<T, N> ft(smem, a.Mt);
  const int q = fft_pair(fp.npairs);
  if (q < 0) return;
  const FftXPair pr(fp, a.S, q);
  const long long oa = pr.sp * a.g.total + pr.la * N, ob = pr.sp * a.g.total + pr.lb * N;
  typename WaveFft<T, N>::Vals va, vb;
  fft_load_line(a.src + oa, ft.lane, va);
  fft_load_line(a.src + ob, ft.lane, vb);
  ft.hartley(va, vb);
  fft_store_line(a.dst + oa, ft.lane, va);
  fft_store_line(a.dst + ob, ft.lane, vb);
}

// One transform along a strided axis, src -> dst (may alias).
template <typename T, int N>
__global__ __launch_bounds__(256) void k_fsy(SingleArgs<T> a, FftPairs fp) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  const WaveFft<T, N> ft(smem, a.Mt);
  const int q = fft_pair(fp.npairs);
  if (q < 0) return;
  const FftCols<T> io(fp, N, q, ft.lane);
  typename WaveFft<T, N>::Vals va, vb;
  io.load_all(a.src, va, vb);
  ft.hartley(va, vb);
  io.store_all(a.dst, va, vb);
}

// Z: forward transform along the last axis, stage combine, inverse transform
// (in place on P). MODE 0..3; MODE < 0: MODE_INIT or MODE_RESTORE (a.mode).
template <typename T, int N, int MODE>
__global__ __launch_bounds__(256) void k_fz(StageArgs<T> a, FftPairs fp) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using FT = WaveFft<T, N>;
  const FT ft(smem, a.Mt);
  const int q = fft_pair(fp.npairs);
  if (q < 0) return;
  const FftCols<T> io(fp, N, q, ft.lane);
  typename FT::Vals va, vb;
  io.load_all(a.src ? a.src : a.P, va, vb);
  if constexpr (MODE >= 0) {
    auto run = [&](auto co) {
      constexpr int CO = decltype(co)::value;
      // the retained arrays in flight over the transform, where they fit
      constexpr bool AHEAD = FT::E * sizeof(T) <= 64;
      CombineIn<T> in[FT::E / 4];
      auto read = [&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        io.load(MODE <= 1 ? a.uhat : a.acc, io.offs(rb), in[rb].x1[0], in[rb].x1[1]);
        wave_combine_in<MODE, CO>(io, a, rb, in[rb]);
      };
      if constexpr (AHEAD) static_for<FT::E / 4>(read);
      ft.hartley(va, vb);
      const float lz[2][4] = {};
      static_for<FT::E / 4>([&](auto rbc) {
        constexpr int rb = decltype(rbc)::value;
        if constexpr (!AHEAD) read(rbc);
        T ya[4], yb[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ya[r] = va[4 * rb + r];
          yb[r] = vb[4 * rb + r];
        }
        wave_combine_out<MODE, CO>(io, a, rb, 0.f, T(0), T(0), lz, in[rb], ya, yb);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          va[4 * rb + r] = ya[r];
          vb[4 * rb + r] = yb[r];
        }
      });
    };
    if (a.ltab)
      run(std::integral_constant<int, CO_LTAB>{});
    else
      run(std::integral_constant<int, CO_TABS>{});
  } else {
    if (!a.src) ft.hartley(va, vb);
    if (a.mode == MODE_INIT) io.store_all(a.uhat, va, vb);
#pragma unroll
    for (int e = 0; e < FT::E; ++e) {
      va[e] *= a.cs;
      vb[e] *= a.cs;
    }
  }
#pragma unroll
  for (int e = 0; e < FT::E; ++e) {
    keep(va[e]);
    keep(vb[e]);
  }
  ft.hartley(va, vb);
  io.store_all(a.P, va, vb);
}

// Adjoint reaction. Uncoupled species: of the pair's lines at their stage values ua,
// ub. Two coupled species: of line a in the wavefront of species 0 and of line b in
// that of species 1, ua and ub the two species' stage values of that line; the
// wavefronts trade lines before and after (three barriers with the one that lets
// the next transform write). So each point's Jacobian and parameter partials are
// formed once. Parameter partials: a repeated line does not count again.
template <int KIND, typename T, class FT>
__device__ __forceinline__ void fft_adj_react(const StageArgs<T>& a, const FftXPair& pr,
                                              const FT& ft, T (&ga)[FT::E], T (&gb)[FT::E],
                                              const T (&ua)[FT::E], const T (&ub)[FT::E],
                                              double* pacc) {
  const int sp = pr.sp;  // uniform
  const bool wp = a.rp_acc != nullptr;
  const double wb = pr.lb != pr.la ? 1.0 : 0.0;
  if constexpr (KIND >= RXN_FHN && KIND <= RXN_GM) {
    T give[FT::E], got[FT::E];
#pragma unroll
    for (int e = 0; e < FT::E; ++e) give[e] = sp == 0 ? gb[e] : ga[e];
    ft.trade(0, give, got);
#pragma unroll
    for (int e = 0; e < FT::E; ++e) {
      const T own = sp == 0 ? ga[e] : gb[e], u[2] = {ua[e], ub[e]};
      const T g[2] = {sp == 0 ? own : got[e], sp == 0 ? got[e] : own};
      T o[2];
      rxn_adjoint_k<T, 2, KIND>(a.rxn, u, g, o, sp == 0 ? 1.0 : wb, pacc, wp);
      ga[e] = sp == 0 ? o[0] : o[1];
      give[e] = sp == 0 ? o[1] : o[0];
    }
    ft.trade(1, give, got);
#pragma unroll
    for (int e = 0; e < FT::E; ++e) {
      const T own = ga[e];
      ga[e] = sp == 0 ? own : got[e];
      gb[e] = sp == 0 ? got[e] : own;
    }
    __syncthreads();
  } else {
    const T lin = T(sp == 0 ? a.rxn.p[0] : sp == 1 ? a.rxn.p[1] : sp == 2 ? a.rxn.p[2] : a.rxn.p[3]);
#pragma unroll
    for (int e = 0; e < FT::E; ++e) {
      const T g[2] = {ga[e], gb[e]}, u[2] = {ua[e], ub[e]};
      T o[2];
      if constexpr (KIND == RXN_LINEAR) {
        o[0] = lin * g[0];
        o[1] = lin * g[1];
        if (wp) {
          const double c = double(g[0] * u[0]) + wb * double(g[1] * u[1]);
#pragma unroll
          for (int s = 0; s < MAX_SPECIES; ++s) pacc[s] += sp == s ? c : 0.0;
        }
      } else {
        rxn_adjoint_k<T, 1, KIND>(a.rxn, &u[0], &g[0], &o[0], 1.0, pacc, false);
        rxn_adjoint_k<T, 1, KIND>(a.rxn, &u[1], &g[1], &o[1], 1.0, pacc, false);
      }
      ga[e] = o[0];
      gb[e] = o[1];
    }
  }
}

// X, adjoint. (Every wavefront of a block reaches the block sums.)
template <typename T, int N>
__global__ __launch_bounds__(256) void k_fxadj(StageArgs<T> a, FftPairs fp) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using FT = WaveFft<T, N>;
  const FT ft(smem, a.Mt);
  double pacc[RXN_NP_MAX];
#pragma unroll
  for (int k = 0; k < RXN_NP_MAX; ++k) pacc[k] = 0.0;
  const int q = fft_pair(fp.npairs);
  if (q >= 0) {
    const FftXPair pr(fp, a.S, q);
    const bool two = fft_coupled(a.rxn.kind);
    const long long oa = pr.sp * a.g.total + pr.la * N, ob = pr.sp * a.g.total + pr.lb * N;
    typename FT::Vals va, vb, ua, ub;
    fft_load_line(a.P + oa, ft.lane, va);
    fft_load_line(a.P + ob, ft.lane, vb);
    const T* st = a.st_phys + (long long)a.mode * a.S * a.g.total;
    const long long own = pr.sp == 0 ? pr.la * N : pr.lb * N;
    fft_load_line(st + (two ? own : oa), ft.lane, ua);
    fft_load_line(st + (two ? a.g.total + own : ob), ft.lane, ub);
    ft.hartley(va, vb);
    switch (a.rxn.kind) {  // uniform
      case RXN_LINEAR: fft_adj_react<RXN_LINEAR>(a, pr, ft, va, vb, ua, ub, pacc); break;
      case RXN_FHN: fft_adj_react<RXN_FHN>(a, pr, ft, va, vb, ua, ub, pacc); break;
      case RXN_GRAY_SCOTT: fft_adj_react<RXN_GRAY_SCOTT>(a, pr, ft, va, vb, ua, ub, pacc); break;
      case RXN_SCHNAKENBERG: fft_adj_react<RXN_SCHNAKENBERG>(a, pr, ft, va, vb, ua, ub, pacc); break;
      case RXN_GM: fft_adj_react<RXN_GM>(a, pr, ft, va, vb, ua, ub, pacc); break;
      case RXN_HUXLEY_MMS: fft_adj_react<RXN_HUXLEY_MMS>(a, pr, ft, va, vb, ua, ub, pacc); break;
      default: fft_adj_react<RXN_FISHER_MMS>(a, pr, ft, va, vb, ua, ub, pacc); break;
    }
    ft.hartley(va, vb);
    fft_store_line(a.P + oa, ft.lane, va);
    fft_store_line(a.P + ob, ft.lane, vb);
  } else if (fft_coupled(a.rxn.kind)) {
    for (int k = 0; k < FFT_TRADE_BARRIERS; ++k) __syncthreads();
  }
  if (a.rp_acc) block_add_partials(reinterpret_cast<double*>(smem), pacc, a.rxn.np, a.rp_acc);
}

// Z, adjoint (a.mode at run time).
template <typename T, int N>
__global__ __launch_bounds__(256) void k_fzadj(StageArgs<T> a, FftPairs fp) {
  to_member(a);
  extern __shared__ __align__(16) char smem[];
  using FT = WaveFft<T, N>;
  const FT ft(smem, a.Mt);
  const int q = fft_pair(fp.npairs);
  if (q < 0) return;
  const FftCols<T> io(fp, N, q, ft.lane);
  typename FT::Vals va, vb;
  io.load_all(a.P, va, vb);
  ft.hartley(va, vb);
  static_for<FT::E / 4>([&](auto rbc) {
    constexpr int rb = decltype(rbc)::value;
    T ya[4], yb[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      ya[r] = va[4 * rb + r];
      yb[r] = vb[4 * rb + r];
    }
    wave_adj_tab<0>(io, a, rb, ya);
    wave_adj_tab<1>(io, a, rb, yb);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      va[4 * rb + r] = ya[r];
      // (a repeated column: side b has read what side a wrote)
      vb[4 * rb + r] = io.ob != io.oa ? yb[r] : ya[r];
    }
  });
  ft.hartley(va, vb);
  io.store_all(a.P, va, vb);
}

// Kernels of one N, by the kernel numbers of the wave engine.
struct FftKernels {
  const void* fn[WK_COUNT];
  size_t lds;  // per wavefront
};
template <typename T, int N>
FftKernels fft_kernels() {
  FftKernels k{};
  k.fn[WK_X] = reinterpret_cast<const void*>(&k_fx<T, N, false>);
  k.fn[WK_XSRC] = reinterpret_cast<const void*>(&k_fx<T, N, true>);
  k.fn[WK_SX] = reinterpret_cast<const void*>(&k_fsx<T, N>);
  k.fn[WK_SY] = reinterpret_cast<const void*>(&k_fsy<T, N>);
  k.fn[WK_ZINIT] = reinterpret_cast<const void*>(&k_fz<T, N, -1>);
  k.fn[WK_Z] = reinterpret_cast<const void*>(&k_fz<T, N, 0>);
  k.fn[WK_Z + 1] = reinterpret_cast<const void*>(&k_fz<T, N, 1>);
  k.fn[WK_Z + 2] = reinterpret_cast<const void*>(&k_fz<T, N, 2>);
  k.fn[WK_Z + 3] = reinterpret_cast<const void*>(&k_fz<T, N, 3>);
  k.fn[WK_XADJ] = k.fn[WK_XADJ + 1] = reinterpret_cast<const void*>(&k_fxadj<T, N>);
  k.fn[WK_ZADJ] = reinterpret_cast<const void*>(&k_fzadj<T, N>);
  k.lds = WaveFft<T, N>::lds_bytes();
  return k;
}
template <typename T>
FftKernels fft_kernels(long long n) {
  return n == 256 ? fft_kernels<T, 256>() : n == 512 ? fft_kernels<T, 512>() : fft_kernels<T, 1024>();
}

}  // namespace sfrde
