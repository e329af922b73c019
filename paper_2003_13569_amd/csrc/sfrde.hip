// libsfrde: host plan, step drivers and the C ABI declared in include/sfrde.h.
//
// A plan holds, on the device: per-axis transform data (half matrices of
// the matrix-core engine, FFT twiddles or dense matrices, built in FP64 on the host from
// the closed forms of Section 3.1), per-axis FP64
// eigenvalue tables, the six coefficient tables of the Alg. 1 precompute
// (computed in FP64 on the device, stored in dtype), and the workspace of the
// step: one field buffer P that every kernel transforms in place, and the
// retained spectral arrays u_hat, c_til, acc. The backward pass adds the
// adjoint buffers, a segment store for recomputed stage data and the
// derivative tables.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cstdint>
#include <initializer_list>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/sfrde.h"
#include "coef.h"
#include "fft.h"
#include "kernels.h"
#include "stability.h"
#include "wave_parts.h"

using namespace sfrde;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIPCHECK(expr)                                                                  \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      return fail(e_ == hipErrorOutOfMemory ? SFRDE_ENOMEM : SFRDE_EDEVICE, "%s: %s (%s:%d)", \
                  #expr, hipGetErrorString(e_), __FILE__, __LINE__);                    \
  } while (0)

#define TRY(expr)              \
  do {                         \
    int rc_ = (expr);          \
    if (rc_ != SFRDE_OK) return rc_; \
  } while (0)

const long long CKPT_MAGIC = 0x5346524445434b31LL;  // "SFRDECK1"
constexpr int MAX_N = 1024;
constexpr int MAX_BATCH = 65535;  // ensemble members: the launch's grid y extent
// Reduction scratch of the backward pass: per-block partials first, then the
// results of each ensemble member (2 S kappa/alpha sums, then parameters).
constexpr long long RED_OUT = 2 * MAX_SPECIES * 1024 + 64;
constexpr long long RED_PER_MEMBER = 2 * MAX_SPECIES + MAX_PARAMS;

// Device memory of sfrde_backward_noalloc: one array per GPU the library
// runs on, held until the process ends. Host code never passes `scratch`
// itself (in host code the name is a stand-in, not a device address): it
// uses the address hipGetSymbolAddress returns on each device, looked up
// once per device at plan set-up.
// Behind it a part for the gradients' block partials, whose size follows the launch
// grids (0.2 MB at most on the engine's, but for ensembles of thousands): the
// fields alone decide whether a request fits.
constexpr size_t SCRATCH_BYTES = (size_t)SFRDE_NOALLOC_SCRATCH_BYTES;
constexpr size_t PARTIAL_BYTES = 1 << 20;
static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES + PARTIAL_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};

// Address of this device's scratch array (the device must be current).
int scratch_address(int dev, void** out) {
  if (dev < 0 || dev >= MAX_DEVICES) return fail(SFRDE_EDEVICE, "device %d out of range", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(SFRDE_EDEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                  hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return SFRDE_OK;
}

}  // namespace

struct sfrde_plan_s {
  int ndim = 0;
  long long n[3] = {1, 1, 1};
  int bc = 0;
  double h[3] = {1, 1, 1};
  int S = 0;
  double alpha[MAX_SPECIES] = {0};  // member 0
  double kappa[MAX_SPECIES] = {0};
  double dt = 0;
  Rxn rxn{};
  // ensembles: B members of this grid; per-member orders, coefficients and
  // reaction constants ([B][S], [B])
  int B = 1;
  std::vector<double> alpha_m, kappa_m;
  std::vector<Rxn> rxn_m;
  Rxn* rxm = nullptr;  // device copy of rxn_m
  int dtype = 0;
  int scheme = 0;
  hipStream_t stream = nullptr;
  long long total = 0;
  double cs = 1;  // product of per-axis inverse scales
  size_t w = 4;   // bytes per real
  Geom geom[3]{};
  size_t lds[3] = {0, 0, 0};
  // wave engine per axis (wave.h): size class (-1: not on it), tables, tiles
  int wcls[3] = {-1, -1, -1};
  WaveAxis wax[3]{};
  WaveTiles wtl[3]{};
  void* wA[3] = {nullptr, nullptr, nullptr};
  bool lfly = false;     // Z kernels of the wave engine form L from the eigenvalues
  // periodic axes of 256, 512 or 1024 points: FFT kernels (fft.h)
  bool use_f[3] = {false, false, false};
  FftPairs fft[3]{};
  unsigned wpb_f[3] = {0, 0, 0};  // wavefronts per block
  void* tw[3] = {nullptr, nullptr, nullptr};  // [N][2] cos, sin of 2 pi m / N
  int n_cu = 256;
  int device = 0;
  // the static scratch array of the plan's device (allocation-free backward)
  void* scratch = nullptr;
  bool noalloc = false;  // this backward call carves its buffers from scratch
  // device memory
  void* Mt[3] = {nullptr, nullptr, nullptr};
  double* lam[3] = {nullptr, nullptr, nullptr};
  void* coef = nullptr;
  void* dcoef = nullptr;
  void* ltab = nullptr;  // P13 plans: L per species and point
  double* thp = nullptr;  // adjoint kappa/alpha partials per Z block [4][blocks]
  bool thp_on = false;    // this backward call accumulates them (else G)
  void* P = nullptr;
  void* uhat = nullptr;
  void* ctil = nullptr;
  void* acc = nullptr;
  void* Pa = nullptr;
  void* zh = nullptr;
  void* aacc = nullptr;
  void* ahat = nullptr;
  void* gu = nullptr;
  double* G = nullptr;
  void* seg = nullptr;
  long long seg_steps = 0;   // steps the allocated segment store holds
  long long seg_cap = 0;     // its size in fields of [B][S][total]
  int seg_stride = 9;        // fields per step of the current backward (9, or 4 for u0 only)
  double* rp_acc = nullptr;
  double* red = nullptr;  // reduction scratch
  long long red_len = 0;
  int* flag = nullptr;
  int* h_flag = nullptr;  // pinned host mirror
  size_t bytes = 0;
  // measurement: optional HIP events around every kernel launch
  bool prof = false;
  std::vector<hipEvent_t> ev;    // start/stop pairs
  std::vector<int> ev_class;     // kernel class per pair
  size_t ev_used = 0;            // pairs recorded since the last reset
};

namespace {

// Elements and bytes of one field of every member: [B][S][total].
size_t field_elems(const sfrde_plan_s* p) { return (size_t)p->B * p->S * p->total; }
size_t field_bytes(const sfrde_plan_s* p) { return field_elems(p) * p->w; }

int dev_alloc(sfrde_plan_s* p, void** ptr, size_t bytes) {
  if (*ptr) return SFRDE_OK;
  hipError_t e = hipMalloc(ptr, bytes);
  if (e != hipSuccess) {
    *ptr = nullptr;
    return fail(e == hipErrorOutOfMemory ? SFRDE_ENOMEM : SFRDE_EDEVICE,
                "hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
  }
  p->bytes += bytes;
  return SFRDE_OK;
}

void dev_free(sfrde_plan_s* p, void** ptr, size_t bytes) {
  if (*ptr) {
    (void)hipFree(*ptr);
    p->bytes -= bytes;
    *ptr = nullptr;
  }
}

// Kernel classes for measurement (enum order of SFRDE_K_* in sfrde.h).
enum { KC_X = 0, KC_Y = 1, KC_Z = 2, KC_XADJ = 3, KC_ZADJ = 4, KC_OTHER = 5, KC_COUNT = 6 };

// Record the start event of a measured launch; returns the pair index or -1.
long long prof_start(sfrde_plan_s* p, int cls) {
  if (!p->prof) return -1;
  const size_t k = p->ev_used;
  while (p->ev.size() < 2 * (k + 1)) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return -1;
    p->ev.push_back(e);
  }
  if (p->ev_class.size() < k + 1) p->ev_class.resize(k + 1);
  p->ev_class[k] = cls;
  if (hipEventRecord(p->ev[2 * k], p->stream) != hipSuccess) return -1;
  p->ev_used = k + 1;
  return (long long)k;
}

void prof_stop(sfrde_plan_s* p, long long k) {
  if (k >= 0) (void)hipEventRecord(p->ev[2 * k + 1], p->stream);
}

int expected_nparams(int reaction, int S) {
  switch (reaction) {
    case RXN_LINEAR: return S;
    case RXN_FHN: return 5;
    case RXN_GRAY_SCOTT: return 2;
    case RXN_SCHNAKENBERG: return 3;
    case RXN_GM: return 5;
    case RXN_HUXLEY_MMS:
    case RXN_FISHER_MMS: return 0;
    default: return -1;
  }
}

// Transposed axis matrix Mt[j*n + k] = M[k][j] in FP64 (see kernels.h).
std::vector<double> axis_matrix_t(int bc, long long n) {
  const double pi = 3.14159265358979323846;
  std::vector<double> Mt((size_t)n * n);
  for (long long k = 0; k < n; ++k) {
    for (long long j = 0; j < n; ++j) {
      double v;
      if (bc == SFRDE_BC_PERIODIC) {
        const long long N = n;
        const long long m = (k * j) % N;
        const double th = 2.0 * pi * double(m) / double(N);
        v = cos(th) + sin(th);
      } else if (bc == SFRDE_BC_DIRICHLET) {
        const long long N = n + 1;
        const long long m = ((k + 1) * (j + 1)) % (2 * N);
        v = sin(pi * double(m) / double(N));
      } else {
        const long long N = n - 1;
        const long long m = (k * j) % (2 * N);
        v = cos(pi * double(m) / double(N));
        if (j == 0 || j == n - 1) v *= 0.5;
      }
      Mt[(size_t)j * n + k] = v;
    }
  }
  return Mt;
}

double axis_inverse_scale(int bc, long long n) {
  if (n == 1) return 1.0;  // padding axis of a 1D plan
  if (bc == SFRDE_BC_PERIODIC) return 1.0 / double(n);
  if (bc == SFRDE_BC_DIRICHLET) return 2.0 / double(n + 1);
  return 2.0 / double(n - 1);
}

// log2(x) for a power of two x >= 1, else -1.
int pow2_shift(long long x) {
  if (x < 1 || (x & (x - 1)) != 0) return -1;
  int k = 0;
  while ((1LL << k) < x) ++k;
  return k;
}

long long pow2_floor(long long x) {
  long long p = 1;
  while (p * 2 <= x) p *= 2;
  return p;
}

void make_geom(sfrde_plan_s* p, int axis, long long min_tiles = 0) {
  Geom& g = p->geom[axis];
  const long long n = p->n[axis];
  long long inner = 1;
  for (int a = 0; a < axis; ++a) inner *= p->n[a];
  g.n = (int)n;
  g.spt = p->S;
  g.inner = inner;
  g.total = p->total;
  // Tile width: a power of two with n*W <= KMAX*NTHREADS, the tile of all
  // species within 64 KB of LDS, and no wider than the lines available.
  long long W = std::min<long long>(64, pow2_floor(std::max<long long>(1, (KMAX * NTHREADS) / n)));
  while (W > 1 && (size_t)p->S * n * (W + 1) * p->w > 65536) W /= 2;
  if (inner > 1) W = std::min<long long>(W, pow2_floor(inner) * (pow2_floor(inner) < inner ? 2 : 1));
  // Narrower tiles where there are too few lines to fill the device (small
  // grids, e.g. 2D): the dense kernels run one tile per block.
  auto tiles_for = [&](long long w) {
    const long long lines = p->total / n;
    return inner == 1 ? (lines + w - 1) / w : (p->total / (n * inner)) * ((inner + w - 1) / w);
  };
  while (W > 1 && tiles_for(W) < min_tiles) W /= 2;
  g.W = (int)W;
  g.pitch = (int)(W + 1);
  g.wshift = 0;
  while ((1 << g.wshift) < g.W) ++g.wshift;
  g.inv_n = 1.0f / (float)n;
  if (inner == 1) {
    g.outer = p->total / n;
    g.tpo = 1;
    g.tposh = 0;
    g.ntiles = (g.outer + W - 1) / W;
  } else {
    g.outer = p->total / (n * inner);
    g.tpo = (inner + W - 1) / W;
    g.tposh = pow2_shift(g.tpo);
    g.ntiles = g.outer * g.tpo;
  }
  size_t tile = (size_t)p->S * n * g.pitch * p->w;
  p->lds[axis] = std::max<size_t>(tile, NTHREADS * sizeof(double));
}

// ------------------------------------------------------------------ wave engine
// binary16 bits of x rounded to nearest even (subnormals included; |x| is
// far below the binary16 maximum here).
unsigned short host_f16(double x) {
  uint64_t b;
  std::memcpy(&b, &x, sizeof(b));
  const unsigned short sign = (unsigned short)((b >> 48) & 0x8000u);
  b &= ~(1ull << 63);
  const double a = std::fabs(x);
  if (a < std::ldexp(1.0, -14))  // subnormal (or rounds up to the smallest normal)
    return (unsigned short)(sign | (unsigned)std::nearbyint(a * 16777216.0));
  b += (1ull << 41) - 1 + ((b >> 42) & 1);  // to nearest even at 10 fraction bits
  const unsigned e = (unsigned)(b >> 52) - 1023 + 15, m = (unsigned)(b >> 42) & 1023u;
  return (unsigned short)(sign | (e << 10) | m);
}
double host_f16_value(unsigned short h) {
  const int ex = (h >> 10) & 31, man = h & 1023;
  const double v = ex == 0 ? std::ldexp((double)man, -24) : std::ldexp((double)(man + 1024), ex - 25);
  return (h & 0x8000) ? -v : v;
}

// Kernels of a size class with what their launches need: the blocks of each
// kernel that fit a CU (registers, LDS).
struct WaveClass {
  WaveKernels k{};
  int regs[WK_COUNT] = {0};
};

template <int C = WC_COUNT - 1>
void fill_wave_classes(WaveClass* out) {
  out[C].k = wave_class<C>();
  if constexpr (C > 0) fill_wave_classes<C - 1>(out);
}

// The class table (filled on first use) and, per class on first use by a
// plan, its kernels' register counts.
int wave_class_info(int c, const WaveClass** out) {
  static std::mutex mu;
  static WaveClass tab[WC_COUNT];
  static bool filled = false, known[WC_COUNT] = {false};
  std::lock_guard<std::mutex> lock(mu);
  if (!filled) {
    fill_wave_classes(tab);
    filled = true;
  }
  if (!tab[c].k.nb) return fail(SFRDE_EDEVICE, "this build holds no matrix-core kernels");
  if (!known[c]) {
    for (int i = 0; i < WK_COUNT; ++i) {
      if (!tab[c].k.fn[i]) continue;
      hipFuncAttributes at{};
      HIPCHECK(hipFuncGetAttributes(&at, tab[c].k.fn[i]));
      tab[c].regs[i] = at.numRegs;
    }
    known[c] = true;
  }
  *out = &tab[c];
  return SFRDE_OK;
}

// The half matrices E and O [row][position] in FP64. A point without a partner
// stands on both sides: half the entry in E, none in O.
struct WaveMatrix {
  const WaveAxis& x;
  int bc, seg_at;
  std::vector<double> trig;  // cos / sin of the axis' angles
  std::vector<double> trig2;
  WaveMatrix(int bc_, const WaveAxis& x_, int layout, int nb)
      : x(x_), bc(bc_), seg_at(layout == WL_ODD ? 16 * (nb / 2) : 16 * nb) {
    const double pi = 3.14159265358979323846;
    const long long n = x.n;
    if (bc == SFRDE_BC_PERIODIC) {
      trig.resize(n);
      trig2.resize(n);
      for (long long m = 0; m < n; ++m) {
        trig[m] = cos(2.0 * pi * double(m) / double(n));
        trig2[m] = 2 * m == n ? 0.0 : sin(2.0 * pi * double(m) / double(n));
      }
    } else if (bc == SFRDE_BC_DIRICHLET) {
      trig.resize(2 * (n + 1));
      for (long long m = 0; m < 2 * (n + 1); ++m) trig[m] = sin(pi * double(m) / double(n + 1));
    } else {
      trig.resize(2 * (n - 1));
      for (long long m = 0; m < 2 * (n - 1); ++m) trig[m] = cos(pi * double(m) / double(n - 1));
    }
  }
  double operator()(int half, int row, int pos) const {
    const long long n = x.n;
    const WaveSeg& g = pos < seg_at ? x.s0 : x.s1;
    const int q = pos < seg_at ? pos : pos - seg_at;
    const int rows = x.periodic ? (int)(n / 2) + 1 : (int)(half ? n / 2 : (n + 1) / 2);
    if (q >= g.ca || row >= rows) return 0.0;
    const bool fixed = !(q >= g.blo && q < g.bhi);
    if (half && fixed) return 0.0;
    const double f = fixed ? 0.5 : 1.0;
    const long long a = g.a0 + (long long)x.da * q;
    if (x.periodic) return half ? trig2[(row * a) % n] : f * trig[(row * a) % n];
    const long long k = 2LL * row + half;
    if (bc == SFRDE_BC_DIRICHLET) return f * trig[((k + 1) * (a + 1)) % (2 * (n + 1))];
    return f * (a == 0 || a == n - 1 ? 0.5 : 1.0) * trig[(k * a) % (2 * (n - 1))];
  }
};

int setup_wave_axis(sfrde_plan_s* p, int axis) {
  const long long n = p->n[axis];
  const int c = wave_class_of(p->dtype, p->bc, n, p->rxn.kind >= RXN_HUXLEY_MMS);
  if (c < 0) return SFRDE_OK;
  long long inner = 1;
  for (int a = 0; a < axis; ++a) inner *= p->n[a];
  // 32-bit lane offsets within a tile of a strided axis, 32-bit line numbers
  const long long lines = axis == 0 ? p->total / n : (long long)p->S * (p->total / n);
  if (axis > 0 && !wave_reach_ok(n, inner, (long long)p->w)) return SFRDE_OK;
  if (lines >= (1LL << 31) - 64) return SFRDE_OK;
  const WaveClass* wc = nullptr;
  TRY(wave_class_info(c, &wc));
  const int nb = wc->k.nb, layout = wc->k.layout;
  WaveAxis& x = p->wax[axis];
  x = wave_axis(p->bc, n);
  WaveTiles& t = p->wtl[axis];
  t.lines = lines;
  t.inner = inner;
  t.cpsh = p->S == 1 ? 4 : p->S == 2 ? 3 : 2;
  const long long per = axis == 0 ? 1LL << t.cpsh : 16;
  t.ntiles = (int)((lines + per - 1) / per);
  // (x tiles of three species have a column to spare)
  t.priv = layout == WL_EXACT && (axis > 0 || p->S != 3) && lines % per == 0;
  // FP32 fields past 96 MB (the caches keep nothing from pass to pass): a step of
  // 256^3 1.31 ms by the sweep, 1.40 by runs; 256 x 256 x 128 (67 MB) 683 / 678 us,
  // 192^3 (57 MB) 671 / 587; FP64 rows are twice as long, 256^3 7.23 / 7.12 ms
  t.sweep = p->dtype == SFRDE_F32 &&
            (long long)p->S * p->total * p->B * (long long)sizeof(float) > (96LL << 20);
  const int RS = 16 * nb;
  // axes of one length share a table
  for (int b = 0; b < axis && !x.A; ++b)
    if (p->wcls[b] >= 0 && p->n[b] == n) x.A = p->wax[b].A;
  const WaveMatrix mat(p->bc, x, layout, nb);
  if (x.A) {
  } else if (p->dtype == SFRDE_F32) {
    const int KS = nb / 2;
    std::vector<unsigned short> tab(wc->k.tab_bytes / 2, 0);
    for (int h = 0; h < 2; ++h)
      for (int ks = 0; ks < KS; ++ks)
        for (int g = 0; g < 4; ++g)
          for (int row = 0; row < RS; ++row)
            for (int e = 0; e < 8; ++e) {
              const int pos = 32 * ks + 4 * g + (e < 4 ? e : 12 + e);
              const double v = mat(h, row, pos);
              const unsigned short h0 = host_f16(v);
              const unsigned short h1 = host_f16(v - host_f16_value(h0));
              const size_t u = ((size_t)((h * 2 * KS + ks) * 4 + g) * RS + row) * 8 + e;
              tab[u] = h0;
              tab[u + (size_t)KS * 4 * RS * 8] = h1;
            }
    TRY(dev_alloc(p, &p->wA[axis], wc->k.tab_bytes));
    HIPCHECK(hipMemcpy(p->wA[axis], tab.data(), wc->k.tab_bytes, hipMemcpyHostToDevice));
  } else {
    const int KS = 4 * nb;
    std::vector<double> tab(wc->k.tab_bytes / 8, 0.0);
    for (int h = 0; h < 2; ++h)
      for (int ks = 0; ks < KS; ++ks)
        for (int g = 0; g < 4; ++g)
          for (int row = 0; row < RS; ++row)
            tab[((size_t)(h * KS + ks) * 4 + g) * RS + row] =
                mat(h, row, 4 * ks + g);
    TRY(dev_alloc(p, &p->wA[axis], wc->k.tab_bytes));
    HIPCHECK(hipMemcpy(p->wA[axis], tab.data(), wc->k.tab_bytes, hipMemcpyHostToDevice));
  }
  if (!x.A) x.A = p->wA[axis];
  // more LDS than the default limit where the table needs it
  for (int i = 0; i < WK_COUNT; ++i)
    for (const void* f : {wc->k.fn[i], wc->k.grp[i]})
      if (f)
        HIPCHECK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
  p->wcls[axis] = c;
  return SFRDE_OK;
}

// Launch of a wave kernel over an axis. Blocks: one tile per block while the
// tiles do not outnumber the CUs (every CU gets work; the other waves help to
// load the matrix), one tile per wave up to a full device, then runs of tiles.
int wave_grid(const sfrde_plan_s* p, int axis, int kernel, size_t lds, const WaveClass** out,
              unsigned* blocks) {
  const WaveClass* wc = nullptr;
  TRY(wave_class_info(p->wcls[axis], &wc));
  const int waves = wc->k.threads / 64;
  int regs = wc->regs[kernel];
  // the kernels that add to one set of partials run on one grid
  if (kernel >= WK_ZADJTH)
    regs = std::max({wc->regs[WK_ZADJTH], wc->regs[WK_ZADJTH + 1], wc->regs[WK_ZADJTH + 2]});
  const int per_simd = 512 / std::max(1, (regs + 7) / 8 * 8);
  long long fit = std::max(1, std::min(per_simd * 4, 32) / waves);
  if (lds > 0) fit = std::min<long long>(fit, std::max<long long>(1, (160 * 1024) / (long long)lds));
  const long long tiles =
      kernel == WK_SY2 ? (p->wtl[axis].lines + 31) / 32 : (long long)p->wtl[axis].ntiles;
  const long long cus = std::max<long long>(1, (p->n_cu + p->B - 1) / p->B);
  const long long most = std::max<long long>(1, ((long long)p->n_cu * fit + p->B - 1) / p->B);
  long long g = tiles;
  if (tiles > cus) g = std::min(most, std::max(cus, (tiles + waves - 1) / waves));
  *out = wc;
  *blocks = (unsigned)g;
  return SFRDE_OK;
}

// LDS of a launch: the class' matrix copy, the eigenvalue tables of the
// kernels that form L, the scratch of the block sums.
size_t wave_lds(const sfrde_plan_s* p, int axis, int kernel, const WaveKernels& k) {
  size_t lds = k.lds_a;
  if ((kernel >= WK_ZFLY && kernel < WK_ZFLY + 4) || kernel >= WK_ZADJFLY)
    lds += (size_t)(32 * k.nb + p->n[0] + (p->ndim == 3 ? p->n[1] : 0)) * sizeof(float);
  if (kernel == WK_XADJ + 1 || kernel >= WK_ZADJTH)
    lds = std::max<size_t>(lds, (size_t)RXN_NP_MAX * 16 * sizeof(double));
  return lds;
}

// Whether an axis runs the group kernels (one tile per block, a wave per row
// block): at most GROUP_WAVES waves per CU in all, or no wave kernels. A group
// kernel spends nb waves on the chain of one, and moves its operands through LDS:
// it wins while the device is not full of chains. Step times, wave kernels /
// groups up to 8 waves per CU: 64^2 FP64, 16 members 127 / 46 us, 64 157 / 70;
// 256^2 FP64 257 / 134; 64^3 FP32 149 / 98. Limits of 4 / 8 / 16 waves: 256
// members of 64^2 FP64 127 / 127 / 143, FP32 70 / 70 / 96; 48 x 80 FP32, 64
// members 69 / 62 / 62; periodic 64^3 FP32 128 / 108 / 108.
constexpr long long GROUP_WAVES = 8;
bool use_group(const sfrde_plan_s* p, int axis, const WaveKernels& k) {
  return !k.fn[WK_X] ||
         (long long)p->wtl[axis].ntiles * p->B * k.nb <= GROUP_WAVES * p->n_cu;
}

// Blocks of a kernel's launch over an axis.
int wave_blocks(const sfrde_plan_s* p, int axis, int kernel, unsigned* blocks) {
  const WaveClass* wc = nullptr;
  TRY(wave_class_info(p->wcls[axis], &wc));
  if (use_group(p, axis, wc->k)) {
    *blocks = (unsigned)p->wtl[axis].ntiles;
    return SFRDE_OK;
  }
  return wave_grid(p, axis, kernel, wave_lds(p, axis, kernel, wc->k), &wc, blocks);
}

template <class Args>
int launch_wave(sfrde_plan_s* p, int axis, int kernel, Args& a) {
  const WaveClass* wc = nullptr;
  TRY(wave_class_info(p->wcls[axis], &wc));
  if (kernel != WK_SY2 && use_group(p, axis, wc->k)) {
    void* args[] = {&a, &p->wax[axis], &p->wtl[axis]};
    HIPCHECK(hipLaunchKernel(wc->k.grp[kernel],
                             dim3((unsigned)p->wtl[axis].ntiles, (unsigned)p->B),
                             dim3((unsigned)(64 * wc->k.nb)), args, wc->k.lds_g, p->stream));
    return SFRDE_OK;
  }
  const size_t lds = wave_lds(p, axis, kernel, wc->k);
  unsigned g = 1;
  TRY(wave_grid(p, axis, kernel, lds, &wc, &g));
  WaveTiles tl = p->wtl[axis];
  if (kernel == WK_SY2) tl.ntiles = (int)((tl.lines + 31) / 32);
  void* args[] = {&a, &p->wax[axis], &tl};
  HIPCHECK(hipLaunchKernel(wc->k.fn[kernel], dim3(g, (unsigned)p->B), dim3((unsigned)wc->k.threads), args, lds, p->stream));
  return SFRDE_OK;
}

// Periodic axes of N = 256, 512 or 1024 points run the FFT kernels (fft.h): a
// wavefront per pair of lines, every CU its share of the wavefronts before a
// block gets a second one (wavefronts of a block share the cache lines of
// strided axes).
constexpr unsigned FFT_WAVES = 4;  // wavefronts per block at most
template <typename T>
int setup_fft_axis(sfrde_plan_s* p, int axis) {
  const long long n = p->n[axis];
  if (p->wcls[axis] >= 0 || p->bc != SFRDE_BC_PERIODIC ||
      !(n == 256 || n == 512 || n == 1024))
    return SFRDE_OK;
  FftPairs& f = p->fft[axis];
  f.inner = 1;
  for (int a = 0; a < axis; ++a) f.inner *= p->n[a];
  f.lines = p->total / n;  // per species
  const long long per = axis == 0 ? (f.lines + 1) / 2 : (f.inner + 1) / 2;
  const long long pairs = per * p->S * (axis == 0 ? 1 : f.lines / f.inner);
  // 32-bit pair and column numbers
  if (pairs >= (1LL << 31) - 64) return SFRDE_OK;
  f.per = (int)per;
  f.npairs = (int)pairs;
  p->wpb_f[axis] =
      pairs * p->B >= 4LL * p->n_cu ? FFT_WAVES : pairs * p->B >= 2LL * p->n_cu ? 2 : 1;
  // (two species of a row pair share a block)
  if (axis == 0 && p->S == 2) p->wpb_f[axis] = std::max(2u, p->wpb_f[axis]);
  const double pi = 3.14159265358979323846;
  std::vector<T> tw((size_t)2 * n);
  for (long long m = 0; m < n; ++m) {
    tw[2 * m] = T(cos(2.0 * pi * double(m) / double(n)));
    tw[2 * m + 1] = T(sin(2.0 * pi * double(m) / double(n)));
  }
  TRY(dev_alloc(p, &p->tw[axis], tw.size() * sizeof(T)));
  HIPCHECK(hipMemcpy(p->tw[axis], tw.data(), tw.size() * sizeof(T), hipMemcpyHostToDevice));
  // (the limit belongs to the kernels, not to the plan: what any plan launches)
  const FftKernels k = fft_kernels<T>(n);
  for (const void* fn : k.fn)
    if (fn)
      HIPCHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)(FFT_WAVES * k.lds)));
  p->use_f[axis] = true;
  return SFRDE_OK;
}

// Blocks of an FFT launch over an axis.
unsigned fft_blocks(const sfrde_plan_s* p, int axis) {
  return (unsigned)((p->fft[axis].npairs + p->wpb_f[axis] - 1) / p->wpb_f[axis]);
}

template <typename T, class Args>
int launch_fft(sfrde_plan_s* p, int axis, int kernel, Args& a) {
  const FftKernels k = fft_kernels<T>(p->n[axis]);
  void* args[] = {&a, &p->fft[axis]};
  HIPCHECK(hipLaunchKernel(k.fn[kernel], dim3(fft_blocks(p, axis), (unsigned)p->B),
                           dim3(64 * p->wpb_f[axis]), args, p->wpb_f[axis] * k.lds, p->stream));
  return SFRDE_OK;
}

// --------------------------------------------------------------------------
template <typename T>
StageArgs<T> stage_args(sfrde_plan_s* p, int axis, void* P) {
  StageArgs<T> a{};
  a.g = p->geom[axis];
  a.Mt = (const T*)(p->use_f[axis] ? p->tw[axis] : p->Mt[axis]);
  a.P = (T*)P;
  a.coef = (const T*)p->coef;
  a.ltab = (const T*)p->ltab;
  a.dcoef = (const T*)p->dcoef;
  a.tau = T(p->dt);
  for (int k = 0; k < 3; ++k) a.lam[k] = p->lam[k];
  for (int s = 0; s < p->S; ++s) {
    a.kt[s] = T(p->kappa[s] * p->dt);
    a.ha[s] = T(0.5 * p->alpha[s]);
  }
  a.uhat = (T*)p->uhat;
  a.ctil = (T*)p->ctil;
  a.acc = (T*)p->acc;
  a.zh = (T*)p->zh;
  a.aacc = (T*)p->aacc;
  a.ahat = (T*)p->ahat;
  a.gu = (T*)p->gu;
  a.flag = p->flag;
  a.rxn = p->rxn;
  a.nmem = p->B;
  a.fsz = (long long)p->S * p->total;
  a.rxm = p->rxm;
  a.cs = T(p->cs);
  a.S = p->S;
  a.neumann = p->bc == SFRDE_BC_NEUMANN;
  a.n0 = p->n[0];
  a.n1 = p->n[1];
  a.n2 = p->n[2];
  return a;
}

template <typename T>
int launch_single(sfrde_plan_s* p, int axis, const void* src, void* dst, int pre_div, int post_mul) {
  SingleArgs<T> a{};
  a.g = p->geom[axis];
  a.Mt = (const T*)(p->use_f[axis] ? p->tw[axis] : p->Mt[axis]);
  a.src = (const T*)src;
  a.dst = (T*)dst;
  a.S = p->S;
  a.pre_divide_w = pre_div && p->bc == SFRDE_BC_NEUMANN;
  a.post_multiply_w = post_mul && p->bc == SFRDE_BC_NEUMANN;
  a.nmem = p->B;
  a.fsz = (long long)p->S * p->total;
  a.n0 = p->n[0];
  a.n1 = p->n[1];
  a.n2 = p->n[2];
  const long long pk = prof_start(p, KC_Y);
  if (p->wcls[axis] >= 0) {
    // two columns per lane where the tiles still give every CU four waves or
    // more (below that the shorter chain of one column wins)
    const bool two = p->dtype == SFRDE_F32 && p->wtl[axis].inner % 2 == 0 &&
                     p->wtl[axis].lines / 32 * p->B >= 4LL * p->n_cu &&
                     p->n[axis] <= 256;
    TRY(launch_wave(p, axis, axis == 0 ? WK_SX : two ? WK_SY2 : WK_SY, a));
  } else if (p->use_f[axis]) {
    TRY(launch_fft<T>(p, axis, axis == 0 ? WK_SX : WK_SY, a));
  } else
    hipLaunchKernelGGL(k_single<T>, dim3((unsigned)a.g.ntiles, p->B), dim3(NTHREADS),
                       p->lds[axis], p->stream, a);
  prof_stop(p, pk);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

// Stored data of one step inside the segment store.
template <typename T>
struct StepStore {
  T* phys;  // [B][4][S][total]
  T* uhat;  // [B][S][total]
  T* fhat;  // [B][4][S][total]
};

template <typename T>
StepStore<T> step_store(sfrde_plan_s* p, long long slot) {
  StepStore<T> s{nullptr, nullptr, nullptr};
  if (!p->seg) return s;
  const size_t f = field_elems(p);
  T* base = (T*)p->seg + (size_t)slot * p->seg_stride * f;
  s.phys = base;
  if (p->seg_stride == 9) {  // u_hat and the four f_hat: the kappa/alpha terms
    s.uhat = base + 4 * f;
    s.fhat = base + 5 * f;
  }
  return s;
}

template <typename T>
int launch_x(sfrde_plan_s* p, int stage, double t, T* st_phys) {
  StageArgs<T> a = stage_args<T>(p, 0, p->P);
  a.mode = stage;
  a.t = t;
  a.st_phys = st_phys;
  const long long pk = prof_start(p, KC_X);
  if (p->wcls[0] >= 0) {
    TRY(launch_wave(p, 0, p->rxn.kind >= RXN_HUXLEY_MMS ? WK_XSRC : WK_X, a));
  } else if (p->use_f[0]) {
    TRY(launch_fft<T>(p, 0, p->rxn.kind >= RXN_HUXLEY_MMS ? WK_XSRC : WK_X, a));
  } else
    hipLaunchKernelGGL(k_xstage<T>, dim3((unsigned)a.g.ntiles, p->B), dim3(NTHREADS),
                       p->lds[0], p->stream, a);
  prof_stop(p, pk);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

// Grid of the last-axis kernels of an axis of one point.
dim3 point_grid(const sfrde_plan_s* p) {
  return dim3((unsigned)((p->S * p->total + POINT_THREADS - 1) / POINT_THREADS), (unsigned)p->B);
}

// uhat: the spectral state this stage reads (stages 0, 1) or writes (stage
// 3); NULL: the plan's own.
template <typename T>
int launch_z(sfrde_plan_s* p, int mode, const void* src, T* st_fhat, T* uhat = nullptr) {
  const int ax = p->ndim - 1;
  StageArgs<T> a = stage_args<T>(p, ax, p->P);
  a.mode = mode;
  a.src = (const T*)src;
  a.st_fhat = st_fhat;
  if (uhat) a.uhat = uhat;
  const long long pk = prof_start(p, KC_Z);
  if (p->wcls[ax] >= 0) {
    const int k = p->lfly ? WK_ZFLY : p->ltab ? WK_Z : WK_ZTABS;
    TRY(launch_wave(p, ax, mode > 3 ? WK_ZINIT : k + mode, a));
  } else if (p->use_f[ax]) {
    TRY(launch_fft<T>(p, ax, mode > 3 ? WK_ZINIT : WK_Z + mode, a));
  } else if (p->n[ax] == 1)
    hipLaunchKernelGGL(k_zpoint<T>, point_grid(p), dim3(POINT_THREADS), 0, p->stream, a);
  else
    hipLaunchKernelGGL(k_zstage<T>, dim3((unsigned)a.g.ntiles, p->B), dim3(NTHREADS),
                       p->lds[ax], p->stream, a);
  prof_stop(p, pk);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

// The middle axis of a 3D field (y), in place on buffer B.
template <typename T>
int ypass(sfrde_plan_s* p, void* B) {
  if (p->ndim == 3) return launch_single<T>(p, 1, B, B, 0, 0);
  return SFRDE_OK;
}

// u_hat = F u and P = the partial inverse of cs*u_hat that the first X
// kernel expects (everything but the x axis).
template <typename T>
int prologue_physical(sfrde_plan_s* p, const void* state) {
  TRY(launch_single<T>(p, 0, state, p->P, 0, 0));
  TRY(ypass<T>(p, p->P));
  TRY(launch_z<T>(p, MODE_INIT, nullptr, nullptr));
  return ypass<T>(p, p->P);
}

// P from a stored spectral state (a checkpoint slot), read in place; the
// plan's u_hat is set from it when `set_uhat` (a forward continuation).
template <typename T>
int prologue_spectral(sfrde_plan_s* p, const void* spec, bool set_uhat = true) {
  if (set_uhat)
    HIPCHECK(hipMemcpyAsync(p->uhat, spec, field_bytes(p), hipMemcpyDeviceToDevice, p->stream));
  TRY(launch_z<T>(p, MODE_RESTORE, set_uhat ? p->uhat : spec, nullptr));
  return ypass<T>(p, p->P);
}

// One step of eq. ETDRK4P13 from t (four stages); stores stage data if asked.
// uh_in / uh_out: where the step reads u_hat and writes the next one (NULL:
// the plan's u_hat); the recompute of a segment reads and writes the
// segment store's slots, so that u_hat of every step is stored without a
// copy.
template <typename T>
int run_step(sfrde_plan_s* p, double t, const StepStore<T>* st, T* uh_in = nullptr,
             T* uh_out = nullptr) {
  const double off[4] = {0.0, 0.5 * p->dt, 0.5 * p->dt, p->dt};
  for (int j = 0; j < 4; ++j) {
    TRY(launch_x<T>(p, j, t + off[j], st ? st->phys : nullptr));
    TRY(ypass<T>(p, p->P));
    TRY(launch_z<T>(p, j, nullptr, st ? st->fhat : nullptr, j == 3 ? uh_out : uh_in));
    TRY(ypass<T>(p, p->P));
  }
  return SFRDE_OK;
}

template <typename T>
int fill(sfrde_plan_s* p, T* ptr, long long n, T v) {
  if (n <= 0) return SFRDE_OK;
  long long blocks = std::min<long long>((n + NTHREADS - 1) / NTHREADS, 65536);
  hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(NTHREADS), 0, p->stream, ptr, n, v);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

// Checkpoint header words: magic, nsteps, K, S, total, dtype, ndim, bc, B,
// then the unknowns per axis n[0..2] (a transposed shape or another
// boundary condition has another spectral basis and must not be resumed).
CkptHeader header_words(const sfrde_plan_s* p, long long nsteps, long long K) {
  CkptHeader h{};
  const long long w[CKPT_WORDS] = {CKPT_MAGIC, nsteps, K, (long long)p->S, p->total,
                                   (long long)p->dtype, (long long)p->ndim, (long long)p->bc,
                                   (long long)p->B, p->n[0], p->n[1], p->n[2]};
  for (int i = 0; i < CKPT_WORDS; ++i) h.w[i] = w[i];
  return h;
}

int write_header(sfrde_plan_s* p, void* ckpt, long long nsteps, long long K) {
  hipLaunchKernelGGL(k_header, dim3(1), dim3(64), 0, p->stream, (long long*)ckpt,
                     header_words(p, nsteps, K));
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

// Reads the header of ckpt into h and checks that this plan wrote it (every
// word but nsteps and K).
int read_header(sfrde_plan_s* p, const void* ckpt, long long (&h)[CKPT_WORDS]) {
  HIPCHECK(hipMemcpyAsync(h, ckpt, sizeof(h), hipMemcpyDeviceToHost, p->stream));
  HIPCHECK(hipStreamSynchronize(p->stream));
  if (h[0] != CKPT_MAGIC) return fail(SFRDE_ESTATE, "checkpoint has no valid header");
  const CkptHeader mine = header_words(p, 0, 0);
  static const char* const what[CKPT_WORDS] = {"", "", "", "species count", "point count",
                                               "dtype", "dimension", "boundary condition",
                                               "ensemble size", "x size", "y size", "z size"};
  for (int i = 3; i < CKPT_WORDS; ++i)
    if (h[i] != mine.w[i])
      return fail(SFRDE_ESTATE, "checkpoint was written by a plan of another %s (%lld != %lld)",
                  what[i], h[i], mine.w[i]);
  if (h[2] < 1 || h[1] < 1) return fail(SFRDE_ESTATE, "checkpoint header has no steps");
  return SFRDE_OK;
}

int check_header(sfrde_plan_s* p, const void* ckpt, long long nsteps, long long K) {
  long long h[CKPT_WORDS];
  TRY(read_header(p, ckpt, h));
  if (h[2] != K) return fail(SFRDE_ESTATE, "checkpoint spacing %lld != %lld", h[2], K);
  if (h[1] < nsteps) return fail(SFRDE_ESTATE, "checkpoint covers %lld < %lld steps", h[1], nsteps);
  return SFRDE_OK;
}

char* ckpt_slot(sfrde_plan_s* p, void* ckpt, long long slot) {
  return (char*)ckpt + SFRDE_CKPT_HEADER_BYTES + (size_t)slot * field_bytes(p);
}

template <typename T>
int finish_forward(sfrde_plan_s* p, void* state) {
  TRY(launch_single<T>(p, 0, p->P, state, 0, 0));
  HIPCHECK(hipMemcpyAsync(p->h_flag, p->flag, sizeof(int), hipMemcpyDeviceToHost, p->stream));
  HIPCHECK(hipStreamSynchronize(p->stream));
  if (*p->h_flag) return fail(SFRDE_ENONFINITE, "a stage value or reaction became non-finite");
  return SFRDE_OK;
}

template <typename T>
int run_steps(sfrde_plan_s* p, long long k0, long long nsteps, double t0, long long K, void* ckpt) {
  for (long long k = 0; k < nsteps; ++k) {
    if (ckpt && K > 0 && k % K == 0)
      HIPCHECK(hipMemcpyAsync(ckpt_slot(p, ckpt, k / K), p->uhat, field_bytes(p),
                              hipMemcpyDeviceToDevice, p->stream));
    TRY(run_step<T>(p, t0 + double(k0 + k) * p->dt, (const StepStore<T>*)nullptr));
  }
  return SFRDE_OK;
}

template <typename T>
int integrate_t(sfrde_plan_s* p, void* state, long long nsteps, double t0, long long K, void* ckpt) {
  TRY(fill<int>(p, p->flag, 1, 0));
  if (ckpt && K > 0) TRY(write_header(p, ckpt, nsteps, K));
  TRY(prologue_physical<T>(p, state));
  TRY(run_steps<T>(p, 0, nsteps, t0, K, ckpt));
  return finish_forward<T>(p, state);
}

template <typename T>
int resume_t(sfrde_plan_s* p, const void* ckpt, long long slot, void* state, long long nsteps,
             double t0, long long K, void* ckpt_out) {
  TRY(fill<int>(p, p->flag, 1, 0));
  if (ckpt_out && K > 0) TRY(write_header(p, ckpt_out, nsteps, K));
  TRY(prologue_spectral<T>(p, ckpt_slot(p, (void*)ckpt, slot)));
  TRY(run_steps<T>(p, 0, nsteps, t0, K, ckpt_out));
  return finish_forward<T>(p, state);
}

// --------------------------------------------------------------------------
template <typename T>
int launch_xadj(sfrde_plan_s* p, int stage, const StepStore<T>& st) {
  StageArgs<T> a = stage_args<T>(p, 0, p->Pa);
  a.mode = stage;
  a.st_phys = st.phys;
  a.rp_acc = p->rp_acc;
  const long long pk = prof_start(p, KC_XADJ);
  if (p->wcls[0] >= 0) {
    TRY(launch_wave(p, 0, a.rp_acc ? WK_XADJ + 1 : WK_XADJ, a));
  } else if (p->use_f[0]) {
    TRY(launch_fft<T>(p, 0, WK_XADJ, a));
  } else
    hipLaunchKernelGGL(k_xadj<T>, dim3((unsigned)a.g.ntiles, p->B), dim3(NTHREADS),
                       p->lds[0], p->stream, a);
  prof_stop(p, pk);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

template <typename T>
int launch_zadj(sfrde_plan_s* p, int mode, const StepStore<T>* st, int last) {
  const int ax = p->ndim - 1;
  StageArgs<T> a = stage_args<T>(p, ax, p->Pa);
  a.mode = mode;
  a.last = last;
  a.G = p->G;
  a.thp = p->thp_on ? p->thp : nullptr;
  if (st) {
    a.st_uhat = st->uhat;
    a.st_fhat = st->fhat;
  }
  if (!p->G) a.dcoef = nullptr;
  const long long pk = prof_start(p, KC_ZADJ);
  if (p->wcls[ax] >= 0) {
    // L formed in the kernel (no per-point accumulator), else from tables
    const bool fly = p->lfly && (p->thp_on || !p->G);
    const int k = !fly ? WK_ZADJ : (p->thp_on && mode <= 2 ? WK_ZADJTH : WK_ZADJFLY) + mode;
    TRY(launch_wave(p, ax, k, a));
  } else if (p->use_f[ax]) {
    TRY(launch_fft<T>(p, ax, WK_ZADJ, a));
  } else if (p->n[ax] == 1)
    hipLaunchKernelGGL(k_zadjpoint<T>, point_grid(p), dim3(POINT_THREADS), 0, p->stream, a);
  else
    hipLaunchKernelGGL(k_zadj<T>, dim3((unsigned)a.g.ntiles, p->B), dim3(NTHREADS),
                       p->lds[ax], p->stream, a);
  prof_stop(p, pk);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

// Reverse sweep over one step whose stage data sit in `st`.
template <typename T>
int adjoint_step(sfrde_plan_s* p, const StepStore<T>& st, int last) {
  // adjoint stage m visits the forward stage value 3 - m (c, b, a, u)
  for (int m = 0; m < 4; ++m) {
    TRY(launch_xadj<T>(p, 3 - m, st));
    TRY(ypass<T>(p, p->Pa));
    TRY(launch_zadj<T>(p, m, &st, last));
    TRY(ypass<T>(p, p->Pa));
  }
  return SFRDE_OK;
}

// Coefficient arguments of member b (eigenvalue tables, kappa, alpha).
CoefArgs coef_args(const sfrde_plan_s* p, int b, int deriv) {
  CoefArgs c{};
  c.lam0 = p->lam[0];
  c.lam1 = p->lam[1];
  c.lam2 = p->lam[2] ? p->lam[2] : p->lam[1];
  c.n0 = p->n[0];
  c.n1 = p->n[1];
  c.n2 = p->n[2];
  c.total = p->total;
  c.S = p->S;
  c.scheme = p->scheme;
  c.deriv = deriv;
  c.tau = p->dt;
  for (int s = 0; s < p->S; ++s) {
    c.alpha[s] = p->alpha_m[(size_t)b * p->S + s];
    c.kappa[s] = p->kappa_m[(size_t)b * p->S + s];
  }
  return c;
}

// Per-point tables of every member, [B][k][S][total]: deriv 0 the six
// coefficients (k = 6), 1 their d/dL (k = 6), 2 L itself (k = 1).
int coef_tables(sfrde_plan_s* p, int deriv, void* out) {
  const size_t per = (size_t)(deriv == 2 ? 1 : NCOEF) * p->S * p->total;
  const long long blocks = std::min<long long>((p->total + NTHREADS - 1) / NTHREADS, 8192);
  for (int b = 0; b < p->B; ++b) {
    const CoefArgs c = coef_args(p, b, deriv);
    if (p->dtype == SFRDE_F32)
      hipLaunchKernelGGL(k_coefs<float>, dim3((unsigned)blocks), dim3(NTHREADS), 0, p->stream, c,
                         (float*)out + b * per);
    else
      hipLaunchKernelGGL(k_coefs<double>, dim3((unsigned)blocks), dim3(NTHREADS), 0, p->stream,
                         c, (double*)out + b * per);
    HIPCHECK(hipGetLastError());
  }
  return SFRDE_OK;
}

// Blocks of the adjoint X kernel (each owns one accumulator per parameter).
long long rp_blocks(const sfrde_plan_s* p) {
  if (p->wcls[0] < 0) return p->use_f[0] ? (long long)fft_blocks(p, 0) : p->geom[0].ntiles;
  unsigned g = 1;
  (void)wave_blocks(p, 0, WK_XADJ + 1, &g);  // (the class is known since the plan was made)
  return g;
}

// Row length of the kappa/alpha partials (the blocks of the adjoint Z kernels
// that add to them).
long long thp_blocks(const sfrde_plan_s* p) {
  unsigned g = 1;
  (void)wave_blocks(p, p->ndim - 1, WK_ZADJTH, &g);
  return g;
}

// Bytes of the backward buffers (what ensure_backward_buffers allocates),
// each rounded up to 256 bytes as carve_backward_buffers lays them out.
size_t round256(size_t b) { return (b + 255) / 256 * 256; }

// The backward buffers laid out in the static scratch array (no allocation;
// the plan's own pointers are saved and restored by the caller). Fails with
// EINVAL, before any device work, if they do not fit.
int carve_backward_buffers(sfrde_plan_s* p, long long seg_steps, bool want_theta, bool want_p) {
  const size_t f = field_bytes(p);
  char* base = static_cast<char*>(p->scratch);
  size_t off = 0;
  auto take = [&](void** ptr, size_t bytes) {
    *ptr = base + off;
    off += round256(bytes);
  };
  size_t poff = 0;
  auto take_partials = [&](double** ptr, size_t bytes) {
    if (poff + bytes > PARTIAL_BYTES) return take((void**)ptr, bytes);
    *ptr = (double*)(base + SCRATCH_BYTES + poff);
    poff += round256(bytes);
  };
  take(&p->Pa, f);
  take(&p->zh, f);
  take(&p->aacc, f);
  take(&p->ahat, f);
  take(&p->gu, f);
  take(&p->seg, (size_t)seg_steps * p->seg_stride * f);
  p->seg_steps = seg_steps;
  p->seg_cap = seg_steps * p->seg_stride;
  p->thp = nullptr;
  p->G = nullptr;
  p->dcoef = nullptr;
  p->rp_acc = nullptr;
  bool fill_dcoef = false;
  if (want_theta && p->thp_on) {
    take_partials(&p->thp, (size_t)4 * thp_blocks(p) * sizeof(double));
  } else if (want_theta) {
    take((void**)&p->G, field_elems(p) * sizeof(double));
    // FP64 P13 plans form the coefficient derivatives from L in the combine
    if (!(p->ltab && p->dtype == SFRDE_F64)) {
      take(&p->dcoef, NCOEF * f);
      fill_dcoef = true;
    }
  }
  if (want_p)
    take_partials(&p->rp_acc, (size_t)p->B * MAX_PARAMS * rp_blocks(p) * sizeof(double));
  const long long need = RED_OUT + (long long)p->B * RED_PER_MEMBER;
  take((void**)&p->red, (size_t)need * sizeof(double));
  p->red_len = need;
  if (off > SCRATCH_BYTES)
    return fail(SFRDE_EINVAL,
                "this backward needs %zu bytes of workspace; the allocation-free entry point "
                "holds %zu (use sfrde_backward, or a smaller ckpt_every or grid)",
                off, SCRATCH_BYTES);
  if (fill_dcoef) TRY(coef_tables(p, 1, p->dcoef));
  return SFRDE_OK;
}

int ensure_backward_buffers(sfrde_plan_s* p, long long seg_steps, bool want_theta, bool want_p) {
  if (p->noalloc) return carve_backward_buffers(p, seg_steps, want_theta, want_p);
  const size_t f = field_bytes(p);
  TRY(dev_alloc(p, &p->Pa, f));
  TRY(dev_alloc(p, &p->zh, f));
  TRY(dev_alloc(p, &p->aacc, f));
  TRY(dev_alloc(p, &p->ahat, f));
  TRY(dev_alloc(p, &p->gu, f));
  const long long seg_need = seg_steps * p->seg_stride;
  if (p->seg && p->seg_cap < seg_need) {
    dev_free(p, &p->seg, (size_t)p->seg_cap * f);
    p->seg_cap = 0;
  }
  if (!p->seg) {
    TRY(dev_alloc(p, &p->seg, (size_t)seg_need * f));
    p->seg_cap = seg_need;
  }
  p->seg_steps = seg_steps;
  if (want_theta && p->thp_on) {
    TRY(dev_alloc(p, (void**)&p->thp, (size_t)4 * thp_blocks(p) * sizeof(double)));
  } else if (want_theta) {
    TRY(dev_alloc(p, (void**)&p->G, field_elems(p) * sizeof(double)));
    // FP64 P13 plans form the coefficient derivatives from L in the combine
    if (!p->dcoef && !(p->ltab && p->dtype == SFRDE_F64)) {
      TRY(dev_alloc(p, &p->dcoef, NCOEF * f));
      TRY(coef_tables(p, 1, p->dcoef));
    }
  }
  if (want_p) {
    TRY(dev_alloc(p, (void**)&p->rp_acc,
                  (size_t)p->B * MAX_PARAMS * rp_blocks(p) * sizeof(double)));
  }
  const long long need = RED_OUT + (long long)p->B * RED_PER_MEMBER;
  if (p->red && p->red_len < need) dev_free(p, (void**)&p->red, p->red_len * sizeof(double));
  if (!p->red) {
    TRY(dev_alloc(p, (void**)&p->red, need * sizeof(double)));
    p->red_len = need;
  }
  return SFRDE_OK;
}

template <typename T>
int backward_t(sfrde_plan_s* p, const void* ckpt, long long nsteps, long long K, double t0,
               const void* grad_uT, void* grad_u0, double* gk, double* ga, double* gp) {
  const bool want_theta = gk || ga;
  const bool want_p = gp != nullptr && p->rxn.np > 0;
  const long long seg_steps = std::min(K, nsteps);
  // the recompute stores the stage values; u_hat and the four f_hat only for
  // the kappa/alpha terms
  p->seg_stride = want_theta ? 9 : 4;
  // kappa/alpha gradients formed inside the vector adjoint Z kernels (L
  // formed there too), else through the per-point accumulator G
  p->thp_on = want_theta && p->lfly && p->S <= 2;
  {
    const int rc0 = ensure_backward_buffers(p, seg_steps, want_theta, want_p);
    if (rc0 != SFRDE_OK) {
      p->thp_on = false;
      return rc0;
    }
  }
  // Buffers from an earlier call stay allocated; accumulate only what is asked.
  double* G_saved = p->G;
  if (!want_theta || p->thp_on) p->G = nullptr;
  if (p->G) TRY(fill<double>(p, p->G, (long long)field_elems(p), 0.0));
  const long long zgrid = p->thp_on ? thp_blocks(p) : 0;
  if (p->thp_on) TRY(fill<double>(p, p->thp, 4 * zgrid, 0.0));
  double* rp_saved = p->rp_acc;
  if (!want_p) p->rp_acc = nullptr;
  if (p->rp_acc)
    TRY(fill<double>(p, p->rp_acc, (long long)p->B * MAX_PARAMS * rp_blocks(p), 0.0));

  int rc = SFRDE_OK;
  do {
    // cotangent of u(T) into the adjoint variables, then its first stage input
    if ((rc = launch_single<T>(p, 0, grad_uT, p->Pa, 1, 0))) break;
    if ((rc = ypass<T>(p, p->Pa))) break;
    if ((rc = launch_zadj<T>(p, MODE_INIT, nullptr, 0))) break;
    if ((rc = ypass<T>(p, p->Pa))) break;
    const long long nseg = (nsteps + K - 1) / K;
    for (long long sgi = nseg - 1; sgi >= 0 && rc == SFRDE_OK; --sgi) {
      const long long k0 = sgi * K, k1 = std::min(nsteps, k0 + K);
      // the segment's u_hat of step k sits in store slot k - k0, that of its
      // first step in the checkpoint itself (read in place)
      // (without the kappa/alpha terms u_hat is not stored: the recompute
      // runs on the plan's own)
      T* ck = reinterpret_cast<T*>(ckpt_slot(p, (void*)ckpt, sgi));
      const bool keep_uhat = p->seg_stride == 9;
      auto store_at = [&](long long k) {
        StepStore<T> st = step_store<T>(p, k - k0);
        if (k == k0 && keep_uhat) st.uhat = ck;
        return st;
      };
      if ((rc = prologue_spectral<T>(p, ck, !keep_uhat))) break;
      for (long long k = k0; k < k1 && rc == SFRDE_OK; ++k) {
        StepStore<T> st = store_at(k);
        T* out = k + 1 < k1 ? store_at(k + 1).uhat : (T*)p->uhat;
        rc = run_step<T>(p, t0 + double(k) * p->dt, &st, st.uhat, keep_uhat ? out : nullptr);
      }
      for (long long k = k1 - 1; k >= k0 && rc == SFRDE_OK; --k) {
        StepStore<T> st = store_at(k);
        rc = adjoint_step<T>(p, st, k == 0);
      }
    }
    if (rc) break;
    if (grad_u0 && (rc = launch_single<T>(p, 0, p->Pa, grad_u0, 0, 1))) break;
    const int nb = 1024;
    double* rout = p->red + RED_OUT;
    for (int m = 0; m < p->B && rc == SFRDE_OK; ++m) {
      double* ro = rout + (size_t)m * RED_PER_MEMBER;
      if (want_theta && p->thp_on) {  // one member only (L formed in the kernels)
        hipLaunchKernelGGL(k_rowsum, dim3(2 * p->S), dim3(NTHREADS), 0, p->stream, p->thp, zgrid,
                           ro);
        if (hipGetLastError() != hipSuccess) { rc = fail(SFRDE_EDEVICE, "k_rowsum launch"); break; }
      } else if (want_theta) {
        const CoefArgs c = coef_args(p, m, 0);
        hipLaunchKernelGGL(k_greduce, dim3(nb), dim3(NTHREADS), 0, p->stream, c,
                           p->G + (size_t)m * p->S * p->total, p->cs,
                           (int)(p->bc == SFRDE_BC_NEUMANN), p->red);
        if (hipGetLastError() != hipSuccess) { rc = fail(SFRDE_EDEVICE, "k_greduce launch"); break; }
        hipLaunchKernelGGL(k_rowsum, dim3(2 * p->S), dim3(NTHREADS), 0, p->stream, p->red,
                           (long long)nb, ro);
        if (hipGetLastError() != hipSuccess) { rc = fail(SFRDE_EDEVICE, "k_rowsum launch"); break; }
      }
      if (want_p) {
        hipLaunchKernelGGL(k_rowsum, dim3(p->rxn.np), dim3(NTHREADS), 0, p->stream,
                           p->rp_acc + (size_t)m * MAX_PARAMS * rp_blocks(p), rp_blocks(p),
                           ro + 2 * MAX_SPECIES);
        if (hipGetLastError() != hipSuccess) { rc = fail(SFRDE_EDEVICE, "k_rowsum launch"); break; }
      }
    }
    if (rc) break;
    if (hipStreamSynchronize(p->stream) != hipSuccess) {
      rc = fail(SFRDE_EDEVICE, "stream synchronize");
      break;
    }
    // the members' sums, copied in chunks through a buffer on the stack
    constexpr int CHUNK = 64;
    double host[CHUNK * RED_PER_MEMBER];
    for (int m0 = 0; m0 < p->B && (want_theta || want_p); m0 += CHUNK) {
      const int nm = std::min(CHUNK, p->B - m0);
      if (hipMemcpyAsync(host, rout + (size_t)m0 * RED_PER_MEMBER,
                         (size_t)nm * RED_PER_MEMBER * sizeof(double), hipMemcpyDeviceToHost,
                         p->stream) != hipSuccess ||
          hipStreamSynchronize(p->stream) != hipSuccess) {
        rc = fail(SFRDE_EDEVICE, "copy of gradient partials");
        break;
      }
      for (int i = 0; i < nm; ++i) {
        const int m = m0 + i;
        const double* hm = host + (size_t)i * RED_PER_MEMBER;
        for (int s = 0; s < p->S; ++s) {
          if (gk) gk[m * p->S + s] = hm[2 * s];
          if (ga) ga[m * p->S + s] = hm[2 * s + 1];
        }
        if (want_p)
          for (int k = 0; k < p->rxn.np; ++k) gp[m * p->rxn.np + k] = hm[2 * MAX_SPECIES + k];
      }
    }
  } while (0);
  p->G = G_saved;
  p->rp_acc = rp_saved;
  p->thp_on = false;
  return rc;
}

void destroy_plan(sfrde_plan_s* p) {
  if (!p) return;
  (void)hipStreamSynchronize(p->stream);
  void** ptrs[] = {&p->Mt[0], &p->Mt[1], &p->Mt[2], (void**)&p->lam[0], (void**)&p->lam[1],
                   (void**)&p->lam[2], &p->coef, &p->dcoef, &p->ltab, &p->P, &p->uhat, &p->ctil, &p->acc,
                   &p->Pa, &p->zh, &p->aacc, &p->ahat, &p->gu, (void**)&p->G, &p->seg,
                   (void**)&p->rp_acc, (void**)&p->thp, (void**)&p->red, (void**)&p->flag, (void**)&p->rxm, &p->tw[0], &p->tw[1], &p->tw[2],
                   &p->wA[0], &p->wA[1], &p->wA[2]};
  for (void** q : ptrs) {
    if (*q) (void)hipFree(*q);
    *q = nullptr;
  }
  if (p->h_flag) (void)hipHostFree(p->h_flag);
  for (hipEvent_t e : p->ev) (void)hipEventDestroy(e);
  delete p;
}

int validate(int32_t ndim, const int64_t* n, int32_t bc, const double* h, int32_t S,
             const double* alpha, const double* kappa, double dt, int32_t reaction,
             int32_t nparams, const double* params, int32_t dtype, int32_t scheme) {
  if (ndim < 1 || ndim > 3) return fail(SFRDE_EINVAL, "ndim must be 1, 2 or 3 (got %d)", ndim);
  if (!n || !h) return fail(SFRDE_EINVAL, "n and h must not be NULL");
  for (int a = 0; a < ndim; ++a) {
    if (n[a] < 2 || n[a] > MAX_N)
      return fail(SFRDE_EINVAL, "n[%d] = %lld outside [2, %d]", a, (long long)n[a], MAX_N);
    if (!(h[a] > 0.0) || !std::isfinite(h[a]))
      return fail(SFRDE_EINVAL, "h[%d] must be finite and > 0", a);
  }
  if (bc < 0 || bc > 2) return fail(SFRDE_EINVAL, "unknown boundary condition %d", bc);
  if (S < 1 || S > MAX_SPECIES) return fail(SFRDE_EINVAL, "nspecies %d outside [1, 4]", S);
  if (!alpha || !kappa) return fail(SFRDE_EINVAL, "alpha and kappa must not be NULL");
  for (int s = 0; s < S; ++s) {
    if (!(alpha[s] > 0.0 && alpha[s] <= 2.0))
      return fail(SFRDE_EINVAL, "alpha[%d] = %g outside (0, 2]", s, alpha[s]);
    if (!(kappa[s] >= 0.0) || !std::isfinite(kappa[s]))
      return fail(SFRDE_EINVAL, "kappa[%d] must be finite and >= 0", s);
  }
  if (!(dt > 0.0) || !std::isfinite(dt)) return fail(SFRDE_EINVAL, "dt must be finite and > 0");
  if (reaction < 0 || reaction > RXN_FISHER_MMS)
    return fail(SFRDE_EINVAL, "unknown reaction %d", reaction);
  if (reaction >= RXN_HUXLEY_MMS) {
    if (S != 1) return fail(SFRDE_EINVAL, "reaction %d needs exactly 1 species", reaction);
    if (reaction == RXN_HUXLEY_MMS && (ndim != 2 || bc == SFRDE_BC_DIRICHLET))
      return fail(SFRDE_EINVAL, "the Example 2 source is for 2D periodic or Neumann grids");
    if (reaction == RXN_FISHER_MMS && (ndim != 1 || bc != SFRDE_BC_DIRICHLET))
      return fail(SFRDE_EINVAL, "the Example 1 source is for 1D Dirichlet grids");
  } else if (reaction != RXN_LINEAR && S != 2) {
    return fail(SFRDE_EINVAL, "reaction %d needs exactly 2 species", reaction);
  }
  if (nparams != expected_nparams(reaction, S))
    return fail(SFRDE_EINVAL, "reaction %d takes %d parameters (got %d)", reaction,
                expected_nparams(reaction, S), nparams);
  if (nparams > 0 && !params) return fail(SFRDE_EINVAL, "params must not be NULL");
  for (int k = 0; k < nparams; ++k)
    if (!std::isfinite(params[k])) return fail(SFRDE_EINVAL, "params[%d] is not finite", k);
  if (dtype != SFRDE_F32 && dtype != SFRDE_F64) return fail(SFRDE_EINVAL, "unknown dtype %d", dtype);
  if (scheme != SFRDE_SCHEME_P13 && scheme != SFRDE_SCHEME_EXP)
    return fail(SFRDE_EINVAL, "unknown scheme %d", scheme);
  return SFRDE_OK;
}

template <typename T>
int upload_matrix(sfrde_plan_s* p, int axis) {
  const long long n = p->n[axis];
  std::vector<double> Mt = axis_matrix_t(p->bc, n);
  std::vector<T> conv(Mt.size());
  for (size_t i = 0; i < Mt.size(); ++i) conv[i] = T(Mt[i]);
  TRY(dev_alloc(p, &p->Mt[axis], conv.size() * sizeof(T)));
  HIPCHECK(hipMemcpy(p->Mt[axis], conv.data(), conv.size() * sizeof(T), hipMemcpyHostToDevice));
  return SFRDE_OK;
}

int build_plan(sfrde_plan_s* p) {
  int dev = 0;
  HIPCHECK(hipGetDevice(&dev));
  HIPCHECK(hipDeviceGetAttribute(&p->n_cu, hipDeviceAttributeMultiprocessorCount, dev));
  p->device = dev;
  TRY(scratch_address(dev, &p->scratch));
  for (int a = 0; a < p->ndim; ++a) {
    std::vector<double> lam(p->n[a]);
    for (long long k = 0; k < p->n[a]; ++k)
      lam[k] = p->n[a] == 1 ? 0.0 : axis_eigenvalue(p->bc, p->n[a], p->h[a], k);
    TRY(dev_alloc(p, (void**)&p->lam[a], lam.size() * sizeof(double)));
    HIPCHECK(hipMemcpy(p->lam[a], lam.data(), lam.size() * sizeof(double), hipMemcpyHostToDevice));
  }
  // dense tiles narrowed until the launch (all members) fills the device
  for (int a = 0; a < p->ndim; ++a)
    make_geom(p, a, std::max<long long>(1, (2LL * p->n_cu + p->B - 1) / p->B));
  for (int a = 0; a < p->ndim; ++a) TRY(setup_wave_axis(p, a));
  // Periodic axes of 256, 512 or 1024 points: FFT kernels. Any other axis the
  // matrix-core engine does not take (past 512 points) runs the dense LDS
  // kernels with the axis matrix.
  for (int a = 0; a < p->ndim; ++a) {
    if (p->dtype == SFRDE_F32)
      TRY(setup_fft_axis<float>(p, a));
    else
      TRY(setup_fft_axis<double>(p, a));
    if (p->wcls[a] < 0 && !p->use_f[a] && p->n[a] > 1) {
      if (p->dtype == SFRDE_F32)
        TRY(upload_matrix<float>(p, a));
      else
        TRY(upload_matrix<double>(p, a));
    }
  }
  {
    // FP32 P13 plans form L in the Z kernels from the eigenvalue tables
    // instead of reading an L table where the last axis has 64, 128, 192 or
    // 256 points and its columns come in whole tiles of 32; other grids read
    // the table (rounded from FP64 L, and no slower on the sizes they have).
    const int za = p->ndim - 1;
    const long long inner = za == 2 ? p->n[0] * p->n[1] : p->n[0];
    p->lfly = p->dtype == SFRDE_F32 && p->scheme == SFRDE_SCHEME_P13 && p->B == 1 &&
              p->wcls[za] >= 0 && p->n[za] % 64 == 0 && p->n[za] <= 256 && inner % 32 == 0 && p->n[0] % 4 == 0;
  }
  const size_t f = field_bytes(p);
  TRY(dev_alloc(p, &p->coef, NCOEF * f));
  TRY(dev_alloc(p, &p->P, f));
  TRY(dev_alloc(p, &p->uhat, f));
  TRY(dev_alloc(p, &p->ctil, f));
  TRY(dev_alloc(p, &p->acc, f));
  TRY(dev_alloc(p, (void**)&p->flag, 64));
  HIPCHECK(hipHostMalloc((void**)&p->h_flag, sizeof(int), hipHostMallocDefault));
  *p->h_flag = 0;
  if (p->B > 1) {
    TRY(dev_alloc(p, (void**)&p->rxm, p->rxn_m.size() * sizeof(Rxn)));
    HIPCHECK(hipMemcpy(p->rxm, p->rxn_m.data(), p->rxn_m.size() * sizeof(Rxn),
                       hipMemcpyHostToDevice));
  }
  TRY(coef_tables(p, 0, p->coef));
  if (p->scheme == SFRDE_SCHEME_P13) {
    // The forward combine forms the P13 coefficients from L: one table read
    // per species and stage instead of up to four. The six tables stay for
    // the adjoint.
    TRY(dev_alloc(p, &p->ltab, f));
    TRY(coef_tables(p, 2, p->ltab));
  }
  TRY(fill<int>(p, p->flag, 16, 0));
  HIPCHECK(hipStreamSynchronize(p->stream));
  return SFRDE_OK;
}

}  // namespace

// ==========================================================================
extern "C" {

const char* sfrde_last_error(void) { return g_err.c_str(); }

int sfrde_plan_batch(sfrde_plan_t* out, int32_t batch, int32_t ndim, const int64_t* n,
                     int32_t bc, const double* h, int32_t nspecies, const double* alpha,
                     const double* kappa, double dt, int32_t reaction, int32_t nparams,
                     const double* params, int32_t dtype, int32_t scheme, void* hip_stream) {
  g_err.clear();
  if (!out) return fail(SFRDE_EINVAL, "out must not be NULL");
  *out = nullptr;
  if (batch < 1 || batch > MAX_BATCH)
    return fail(SFRDE_EINVAL, "batch %d outside [1, %d]", batch, MAX_BATCH);
  if (!alpha || !kappa) return fail(SFRDE_EINVAL, "alpha and kappa must not be NULL");
  if (nparams > 0 && !params) return fail(SFRDE_EINVAL, "params must not be NULL");
  for (int b = 0; b < batch; ++b) {
    const int rc = validate(ndim, n, bc, h, nspecies, alpha + (size_t)b * nspecies,
                            kappa + (size_t)b * nspecies, dt, reaction, nparams,
                            params ? params + (size_t)b * nparams : nullptr, dtype, scheme);
    if (rc != SFRDE_OK) {
      if (batch > 1) g_err += " (ensemble member " + std::to_string(b) + ")";
      return rc;
    }
  }
  sfrde_plan_s* p = new (std::nothrow) sfrde_plan_s();
  if (!p) return fail(SFRDE_ENOMEM, "host allocation of the plan failed");
  // A 1D plan runs as a 2D one whose second axis has one point (eigenvalue
  // 0, identity transform, weight 1): the field layout is the same.
  p->ndim = ndim == 1 ? 2 : ndim;
  p->n[1] = 1;
  p->h[1] = 1.0;
  for (int a = 0; a < ndim; ++a) {
    p->n[a] = n[a];
    p->h[a] = h[a];
  }
  p->total = 1;
  for (int a = 0; a < p->ndim; ++a) {
    p->total *= p->n[a];
    p->cs *= axis_inverse_scale(bc, p->n[a]);
  }
  p->bc = bc;
  p->S = nspecies;
  p->B = batch;
  p->alpha_m.assign(alpha, alpha + (size_t)batch * nspecies);
  p->kappa_m.assign(kappa, kappa + (size_t)batch * nspecies);
  for (int s = 0; s < nspecies; ++s) {
    p->alpha[s] = alpha[s];
    p->kappa[s] = kappa[s];
  }
  p->dt = dt;
  p->rxn_m.resize(batch);
  for (int b = 0; b < batch; ++b) {
    Rxn& r = p->rxn_m[b];
    r = Rxn{};
    r.kind = reaction;
    r.S = nspecies;
    r.np = nparams;
    for (int k = 0; k < nparams; ++k) r.p[k] = params[(size_t)b * nparams + k];
    if (reaction >= RXN_HUXLEY_MMS) {
      // source constants of Examples 1 and 2 (Section 5.1), see mms_line()
      const double pi = 3.14159265358979323846, a = alpha[(size_t)b * nspecies],
                   k = kappa[(size_t)b * nspecies];
      double* c = r.p + MMS_P0;
      c[0] = a;
      if (reaction == RXN_HUXLEY_MMS) {
        c[1] = k / 16.0 * 9.0 * pow(8.0 * pi * pi, 0.5 * a);
        c[2] = k / 16.0 * 3.0 * pow(40.0 * pi * pi, 0.5 * a);
        c[3] = k / 16.0 * pow(72.0 * pi * pi, 0.5 * a);
      } else {
        c[1] = k / 4.0 * 3.0 * pow(2.0 * pi, a);
        c[2] = 0.0;
        c[3] = k / 4.0 * pow(6.0 * pi, a);
      }
      c[4] = h[0];
      c[5] = ndim > 1 ? h[1] : 0.0;
    }
  }
  p->rxn = p->rxn_m[0];
  p->dtype = dtype;
  p->scheme = scheme;
  p->stream = (hipStream_t)hip_stream;
  p->w = dtype == SFRDE_F32 ? 4 : 8;
  for (int a = 0; a < p->ndim; ++a) make_geom(p, a);
  int rc = build_plan(p);
  if (rc != SFRDE_OK) {
    std::string msg = g_err;
    destroy_plan(p);
    g_err = msg;
    return rc;
  }
  *out = p;
  return SFRDE_OK;
}

int sfrde_plan(sfrde_plan_t* out, int32_t ndim, const int64_t* n, int32_t bc, const double* h,
               int32_t nspecies, const double* alpha, const double* kappa, double dt,
               int32_t reaction, int32_t nparams, const double* params, int32_t dtype,
               int32_t scheme, void* hip_stream) {
  return sfrde_plan_batch(out, 1, ndim, n, bc, h, nspecies, alpha, kappa, dt, reaction, nparams,
                          params, dtype, scheme, hip_stream);
}

int sfrde_destroy(sfrde_plan_t plan) {
  g_err.clear();
  if (!plan) return fail(SFRDE_EINVAL, "plan is NULL");
  destroy_plan(plan);
  return SFRDE_OK;
}

int sfrde_integrate(sfrde_plan_t p, void* state, int64_t nsteps, double t0, int64_t ckpt_every,
                    void* ckpt) {
  g_err.clear();
  if (!p) return fail(SFRDE_EINVAL, "plan is NULL");
  if (!state) return fail(SFRDE_EINVAL, "state must not be NULL");
  if (nsteps < 0) return fail(SFRDE_EINVAL, "nsteps must be >= 0");
  if (ckpt_every < 0) return fail(SFRDE_EINVAL, "ckpt_every must be >= 0");
  if (!std::isfinite(t0)) return fail(SFRDE_EINVAL, "t0 must be finite");
  if (nsteps == 0) return SFRDE_OK;
  if (p->dtype == SFRDE_F32) return integrate_t<float>(p, state, nsteps, t0, ckpt_every, ckpt);
  return integrate_t<double>(p, state, nsteps, t0, ckpt_every, ckpt);
}

int sfrde_step(sfrde_plan_t p, void* state, double t) {
  return sfrde_integrate(p, state, 1, t, 0, nullptr);
}

int64_t sfrde_ckpt_bytes(sfrde_plan_t p, int64_t nsteps, int64_t ckpt_every) {
  g_err.clear();
  if (!p) return fail(SFRDE_EINVAL, "plan is NULL");
  if (nsteps < 1 || ckpt_every < 1)
    return fail(SFRDE_EINVAL, "nsteps and ckpt_every must be >= 1");
  const int64_t nslots = (nsteps + ckpt_every - 1) / ckpt_every;
  return SFRDE_CKPT_HEADER_BYTES + nslots * (int64_t)field_bytes(p);
}

int sfrde_resume(sfrde_plan_t p, const void* ckpt, int64_t slot, void* state, int64_t nsteps,
                 double t0, int64_t ckpt_every, void* ckpt_out) {
  g_err.clear();
  if (!p) return fail(SFRDE_EINVAL, "plan is NULL");
  if (!ckpt || !state) return fail(SFRDE_EINVAL, "ckpt and state must not be NULL");
  if (slot < 0 || nsteps < 0 || ckpt_every < 0) return fail(SFRDE_EINVAL, "negative argument");
  long long h[CKPT_WORDS];
  TRY(read_header(p, ckpt, h));
  const long long nslots = (h[1] + h[2] - 1) / h[2];
  if (slot >= nslots) return fail(SFRDE_ESTATE, "slot %lld >= %lld slots", (long long)slot, nslots);
  if (nsteps == 0) return SFRDE_OK;
  if (p->dtype == SFRDE_F32)
    return resume_t<float>(p, ckpt, slot, state, nsteps, t0, ckpt_every, ckpt_out);
  return resume_t<double>(p, ckpt, slot, state, nsteps, t0, ckpt_every, ckpt_out);
}

int sfrde_backward(sfrde_plan_t p, const void* ckpt, int64_t nsteps, int64_t ckpt_every,
                   double t0, const void* grad_uT, void* grad_u0, double* grad_kappa,
                   double* grad_alpha, double* grad_params) {
  g_err.clear();
  if (!p) return fail(SFRDE_EINVAL, "plan is NULL");
  if (!ckpt || !grad_uT) return fail(SFRDE_EINVAL, "ckpt and grad_uT must not be NULL");
  if (nsteps < 1 || ckpt_every < 1) return fail(SFRDE_EINVAL, "nsteps, ckpt_every must be >= 1");
  TRY(check_header(p, ckpt, nsteps, ckpt_every));
  if (p->rxn.kind >= RXN_HUXLEY_MMS && (grad_kappa || grad_alpha))
    return fail(SFRDE_EUNSUPPORTED,
                "kappa and alpha gradients of the manufactured sources are not implemented");
  if (p->dtype == SFRDE_F32)
    return backward_t<float>(p, ckpt, nsteps, ckpt_every, t0, grad_uT, grad_u0, grad_kappa,
                             grad_alpha, grad_params);
  return backward_t<double>(p, ckpt, nsteps, ckpt_every, t0, grad_uT, grad_u0, grad_kappa,
                            grad_alpha, grad_params);
}

int sfrde_backward_noalloc(sfrde_plan_t p, const void* ckpt, int64_t nsteps,
                           int64_t ckpt_every, double t0, const void* grad_uT, void* grad_u0,
                           double* grad_kappa, double* grad_alpha, double* grad_params) {
  g_err.clear();
  if (!p) return fail(SFRDE_EINVAL, "plan is NULL");
  if (!ckpt || !grad_uT) return fail(SFRDE_EINVAL, "ckpt and grad_uT must not be NULL");
  if (nsteps < 1 || ckpt_every < 1) return fail(SFRDE_EINVAL, "nsteps, ckpt_every must be >= 1");
  if (!p->scratch) return fail(SFRDE_EDEVICE, "the plan has no scratch address");
  TRY(check_header(p, ckpt, nsteps, ckpt_every));
  if (p->rxn.kind >= RXN_HUXLEY_MMS && (grad_kappa || grad_alpha))
    return fail(SFRDE_EUNSUPPORTED,
                "kappa and alpha gradients of the manufactured sources are not implemented");
  // the plan's own backward buffers are set aside for this call
  void* saved[] = {p->Pa, p->zh, p->aacc, p->ahat, p->gu, p->seg, p->G, p->dcoef, p->rp_acc,
                   p->thp, p->red};
  const long long saved_seg = p->seg_steps, saved_red = p->red_len, saved_cap = p->seg_cap;
  p->noalloc = true;
  int rc;
  if (p->dtype == SFRDE_F32)
    rc = backward_t<float>(p, ckpt, nsteps, ckpt_every, t0, grad_uT, grad_u0, grad_kappa,
                           grad_alpha, grad_params);
  else
    rc = backward_t<double>(p, ckpt, nsteps, ckpt_every, t0, grad_uT, grad_u0, grad_kappa,
                            grad_alpha, grad_params);
  p->noalloc = false;
  p->Pa = saved[0];
  p->zh = saved[1];
  p->aacc = saved[2];
  p->ahat = saved[3];
  p->gu = saved[4];
  p->seg = saved[5];
  p->G = (double*)saved[6];
  p->dcoef = saved[7];
  p->rp_acc = (double*)saved[8];
  p->thp = (double*)saved[9];
  p->red = (double*)saved[10];
  p->seg_steps = saved_seg;
  p->seg_cap = saved_cap;
  p->red_len = saved_red;
  return rc;
}

int64_t sfrde_workspace_bytes(sfrde_plan_t p) {
  if (!p) return fail(SFRDE_EINVAL, "plan is NULL");
  return (int64_t)p->bytes;
}

int sfrde_profile(sfrde_plan_t p, int32_t enable) {
  g_err.clear();
  if (!p) return fail(SFRDE_EINVAL, "plan is NULL");
  if (enable) {
    HIPCHECK(hipStreamSynchronize(p->stream));
    p->ev_used = 0;
    // Pre-create events for `enable` launches so that recording does not
    // create them inside a measured region.
    while (p->ev.size() < 2 * (size_t)enable) {
      hipEvent_t e;
      HIPCHECK(hipEventCreate(&e));
      p->ev.push_back(e);
    }
  }
  p->prof = enable != 0;
  return SFRDE_OK;
}

int sfrde_profile_read(sfrde_plan_t p, double* ms, int64_t* launches) {
  g_err.clear();
  if (!p || !ms || !launches) return fail(SFRDE_EINVAL, "NULL argument");
  HIPCHECK(hipStreamSynchronize(p->stream));
  for (int c = 0; c < KC_COUNT; ++c) {
    ms[c] = 0.0;
    launches[c] = 0;
  }
  for (size_t k = 0; k < p->ev_used; ++k) {
    float t = 0.f;
    HIPCHECK(hipEventElapsedTime(&t, p->ev[2 * k], p->ev[2 * k + 1]));
    ms[p->ev_class[k]] += double(t);
    launches[p->ev_class[k]] += 1;
  }
  return SFRDE_OK;
}

int sfrde_axis_eigenvalues(int32_t bc, int64_t n, double h, double* out) {
  g_err.clear();
  if (bc < 0 || bc > 2 || n < 2 || !(h > 0) || !out) return fail(SFRDE_EINVAL, "bad argument");
  for (int64_t k = 0; k < n; ++k) out[k] = axis_eigenvalue(bc, n, h, k);
  return SFRDE_OK;
}

int sfrde_eval_coefficients(int32_t scheme, double L, double dt, int32_t deriv, double* out6) {
  g_err.clear();
  if ((scheme != 0 && scheme != 1) || !(L >= 0) || !(dt > 0) || !out6)
    return fail(SFRDE_EINVAL, "bad argument");
  if (deriv)
    coef_derivs(scheme, L, dt, out6);
  else
    coef_values(scheme, L, dt, out6);
  return SFRDE_OK;
}

int sfrde_amplification(int32_t scheme, int64_t count, const double* x, const double* y,
                        double* r, void* hip_stream) {
  g_err.clear();
  if (scheme != SFRDE_SCHEME_P13 && scheme != SFRDE_SCHEME_EXP)
    return fail(SFRDE_EINVAL, "unknown scheme %d", scheme);
  if (count < 0 || count > (int64_t)1 << 36) return fail(SFRDE_EINVAL, "count out of range");
  if (count == 0) return SFRDE_OK;
  if (!x || !y || !r) return fail(SFRDE_EINVAL, "x, y and r must not be NULL");
  const unsigned blocks = (unsigned)((count + 255) / 256);
  hipLaunchKernelGGL(k_amplification, dim3(blocks), dim3(256), 0, (hipStream_t)hip_stream,
                     (int)scheme, (long long)count, x, y, r);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

int sfrde_stability_boundary(int32_t scheme, int64_t ny, const double* y, int64_t ntheta,
                             double* roots, double* poly, void* hip_stream) {
  g_err.clear();
  if (scheme != SFRDE_SCHEME_P13 && scheme != SFRDE_SCHEME_EXP)
    return fail(SFRDE_EINVAL, "unknown scheme %d", scheme);
  if (ny < 0 || ntheta < 1 || ny > ((int64_t)1 << 30) || ntheta > ((int64_t)1 << 30) ||
      ny * ntheta > ((int64_t)1 << 34))
    return fail(SFRDE_EINVAL, "ny, ntheta out of range");
  if (ny == 0) return SFRDE_OK;
  if (!y || !roots) return fail(SFRDE_EINVAL, "y and roots must not be NULL");
  const long long total = (long long)ny * ntheta;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  hipLaunchKernelGGL(k_stability_boundary, dim3(blocks), dim3(256), 0, (hipStream_t)hip_stream,
                     (int)scheme, (long long)ny, y, (long long)ntheta, roots, poly);
  HIPCHECK(hipGetLastError());
  return SFRDE_OK;
}

}  // extern "C"
