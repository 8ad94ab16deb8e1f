// mhd_gravity.hip -- self-gravity source of the step (the paper's Poisson
// equation Lap Psi = 4 pi G rho, section 2.1, "FFT-based" solver), on a
// periodic box, where only rho - <rho> can source the potential.
//
// Per stage, five FFT passes over the half spectrum of the real density,
// a complex array [nz][ny][nx/2 + 1]: x-lines, two rows of the density at a
// time as the real and imaginary part of one complex line; y-lines; z-lines
// forward, each mode divided by the eigenvalue of the 7-point Laplacian
// (times 4 pi G / N, the mean mode set to zero) and back, in one pass; y
// back; x back, which writes Psi into its padded array.  Then the central
// gradient of Psi (periodic wrap), which the update reads for
// S = (0, -rho grad Psi, -rho v.grad Psi, 0).  Extents are powers of two up
// to 1024.
//
// FFT lines: a block takes a tile of lines of one axis into LDS, splits
// each line's n = R1 R2 points into R2 DFTs of R1 points and R1 DFTs of R2
// points done in registers (two LDS passes), and writes the result out.
// x-lines are contiguous; y- and z-lines are tiled over consecutive x, so
// each element row of a tile is one contiguous run in HBM.
//
// The passes are bound by memory and launch latency, so the steps that only
// re-read the array are folded away: a full complex array with passes of
// its own for the load and the division (nine launches) took 132 us a solve
// at 128^3 FP32 and 620 us at 256^3; this form takes 68 and 251 us (256^3:
// about 0.9 GB, 3.6 TB/s; 128^3: six launches of 6 to 14 us; 65 and 232 us with
// all its arithmetic in FP32, see Fine).  The in-register
// DFTs' factors are literals and the other twiddles are loaded ahead of the
// values (with both read from the table where used: 96 and 374 us).  y- and
// z-lines come from memory in the order their first half takes them, without
// a pass through LDS, on blocks ordered by XCD (76 and 313 -> 66 and 277 us), and
// the x-lines' LDS slots are spread over the banks (-> 65 and 232 us).
#include <math.h>

#include <type_traits>

#include "mhd_kernels.hpp"

namespace mhd {

template <class T>
struct Cplx {
  T re, im;
};

// Arithmetic of the z-lines and of the y- and x-lines on the way back: FP32 ones
// are transformed in FP64 registers (what they read, keep in LDS and write is
// FP32).  Half spectra and paired rows round each value once where a full complex
// array rounded it and its mirror image apart: all in FP32, the error of grad Psi
// was 3.0 to 3.7 times that of rounding Psi itself (32^3 to 256^3; a full array
// 3.0 to 3.4), and 1.7 to 2.3 so.  A step with two solves 467 -> 474 us at 128^3,
// 2972 -> 3010 at 256^3 (the x-lines forward too: no smaller error, 477 and
// 3018).
using Fine = double;

template <class A, class T>
__device__ __forceinline__ Cplx<A> cast(Cplx<T> v) {
  return Cplx<A>{(A)v.re, (A)v.im};
}
template <class A, class T>
__device__ __forceinline__ Cplx<A> cmul(Cplx<A> a, Cplx<T> w) {
  const Cplx<A> b = cast<A>(w);
  return Cplx<A>{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}

// Row l = j + ny k of the box: the padded index of its first cell (ny is a
// power of two).
__device__ __forceinline__ int row_start(const Geo& g, int l) {
  const int k = l >> (31 - __builtin_clz((unsigned)g.n[1])), j = l & (g.n[1] - 1);
  return NG + g.sy * (j + NG) + g.sz * (k + NG);
}

// The source density of a run with particles, which the deposit adds to:
// the stage's gas density, or zero for a gas that is decoupled from gravity.
template <class T>
__global__ void __launch_bounds__(256) k_grav_load(Geo g, const T* __restrict__ rho, T* dst,
                                                   int with_gas) {
  const int l = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (l >= g.n[1] * g.n[2]) return;
  const int p0 = row_start(g, l);
  for (int i = threadIdx.x & 63; i < g.n[0]; i += 64) dst[p0 + i] = with_gas ? rho[p0 + i] : T(0);
}

// cos(pi j / 16), 0 <= j <= 8.
__device__ constexpr double kCos16[9] = {1.0,
                                         0.98078528040323044913,
                                         0.92387953251128675613,
                                         0.83146961230254523708,
                                         0.70710678118654752440,
                                         0.55557023301960222474,
                                         0.38268343236508977173,
                                         0.19509032201612826785,
                                         0.0};

template <int R>
__device__ constexpr int bitrev(int i) {
  int r = 0;
  for (int b = 1; b < R; b <<= 1) r = (r << 1) | ((i & b) ? 1 : 0);
  return r;
}

// v exp(-+ 2 pi i q / 32), 0 <= q < 16 (SIGN -1: forward); q is a constant
// after unrolling, so the factors are literals.
template <class T, int SIGN>
__device__ __forceinline__ Cplx<T> rotate(Cplx<T> v, int q) {
  if (q == 0) return v;
  if (q == 8) return SIGN < 0 ? Cplx<T>{v.im, -v.re} : Cplx<T>{-v.im, v.re};
  const T c = (T)(q < 8 ? kCos16[q] : -kCos16[16 - q]);
  const T s = (T)(SIGN * (q < 8 ? kCos16[8 - q] : kCos16[q - 8]));
  return Cplx<T>{v.re * c - v.im * s, v.re * s + v.im * c};
}

// In-register DFT of R points (R a power of two up to 32): the radix-2
// decimation-in-time butterflies, fully unrolled.  SIGN -1 forward, +1
// inverse (unnormalised).
template <class T, int R, int SIGN>
__device__ __forceinline__ void dft_reg(Cplx<T> a[R]) {
  Cplx<T> b[R];
#pragma unroll
  for (int i = 0; i < R; ++i) b[bitrev<R>(i)] = a[i];
#pragma unroll
  for (int m = 1; m < R; m <<= 1) {
#pragma unroll
    for (int j = 0; j < m; ++j) {
#pragma unroll
      for (int k = j; k < R; k += 2 * m) {
        const Cplx<T> u = b[k], v = rotate<T, SIGN>(b[k + m], j * (16 / m));
        b[k] = Cplx<T>{u.re + v.re, u.im + v.im};
        b[k + m] = Cplx<T>{u.re - v.re, u.im - v.im};
      }
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i) a[i] = b[i];
}

// exp(SIGN 2 pi i q / N) for 0 <= q < N, from the N/2 values exp(-2 pi i q / N)
// of tw.
template <class T, int N, int SIGN>
__device__ __forceinline__ Cplx<T> twiddle(const Cplx<T>* __restrict__ tw, int q) {
  Cplx<T> w = tw[q & (N / 2 - 1)];
  if (q >= N / 2) w = Cplx<T>{-w.re, -w.im};
  if (SIGN > 0) w.im = -w.im;
  return w;
}

// The two halves of a line's DFT of N = R1 R2 points in LDS (L).
// Both in arithmetic of type A, on values of type T.
// first: for one n2 < R2 the R1-point DFT over x[R2 n1 + n2] (a[n1]), times
// W_N^(n2 k1) (w, loaded before the values), to the slots R2 k1 + n2.
// second: for one k1 < R1 the R2-point DFT over the R2 contiguous values, left
// in a[k2] = X[k1 + R1 k2].
template <class T, int R1, int R2, int SIGN>
__device__ __forceinline__ void load_twiddles(Cplx<T> w[R1], int n2,
                                              const Cplx<T>* __restrict__ tw) {
  constexpr int N = R1 * R2;
#pragma unroll
  for (int k1 = 1; k1 < R1; ++k1) w[k1] = twiddle<T, N, SIGN>(tw, (n2 * k1) & (N - 1));
}
template <class A, class T, int R1, int R2, int SIGN, int S = R2>
__device__ __forceinline__ void dft_first(Cplx<T>* L, int n2, Cplx<A> a[R1],
                                          const Cplx<T> w[R1]) {
  dft_reg<A, R1, SIGN>(a);
  L[n2] = cast<T>(a[0]);
#pragma unroll
  for (int k1 = 1; k1 < R1; ++k1) L[S * k1 + n2] = cast<T>(cmul(a[k1], w[k1]));
}
// x-lines: from the line in LDS, in place.
template <class A, class T, int R1, int R2, int SIGN, int S>
__device__ __forceinline__ void dft_first_lds(Cplx<T>* L, int n2, const Cplx<T> w[R1]) {
  Cplx<A> a[R1];
#pragma unroll
  for (int n1 = 0; n1 < R1; ++n1) a[n1] = cast<A>(L[S * n1 + n2]);
  dft_first<A, T, R1, R2, SIGN, S>(L, n2, a, w);
}
template <class A, class T, int R1, int R2, int SIGN, int S = R2>
__device__ __forceinline__ void dft_second(const Cplx<T>* L, int k1, Cplx<A> a[R2]) {
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) a[n2] = cast<A>(L[S * k1 + n2]);
  dft_reg<A, R2, SIGN>(a);
}

// x-lines.  A line pair holds rows 2m and 2m + 1 (of ny nz rows) as real and
// imaginary part, so one complex DFT serves two rows (the last row of an odd
// count is paired with zeros).  A block takes 2048 / N pairs (at most 64).
template <int R1, int R2>
constexpr int pairs_per_block() {
  return 2048 / (R1 * R2) < 64 ? 2048 / (R1 * R2) : 64;
}
constexpr int kFftXThreads = 128;
// Where the R1 runs of R2 values of a line pair begin: R2 + 1 apart, and lines
// 8 values mod 32 apart, so that a wave's 8-byte accesses -- the same place in
// several runs, or in several lines -- spread over the 64 LDS banks (with runs
// 8 or 16 values apart they fell on a few: a solve at 256^3 FP32 277 us, 232
// with this).
template <int R1, int R2>
constexpr int line_slots() {
  return R1 * (R2 + 1) + (40 - R1 * (R2 + 1) % 32) % 32;
}
// Slots of the line's element e before its DFT, and of X[e] after both halves
// (X[k1 + R1 k2] at place k2 of run k1).
template <int R1, int R2>
__device__ __forceinline__ int slot_in(int e) {
  return e + e / R2;
}
template <int R1, int R2>
__device__ __forceinline__ int slot_out(int e) {
  return (R2 + 1) * (e % R1) + e / R1;
}

// Forward: rho (padded; null: zero) -> half spectra c[row][N/2 + 1].
template <class T, int R1, int R2>
__global__ void __launch_bounds__(kFftXThreads) k_fft_x(Geo g, const T* __restrict__ rho,
                                                        Cplx<T>* __restrict__ c,
                                                        const Cplx<T>* __restrict__ tw) {
  constexpr int N = R1 * R2, H = N / 2 + 1, LS = line_slots<R1, R2>();
  constexpr int TP = pairs_per_block<R1, R2>();
  __shared__ Cplx<T> buf[TP * LS];
  const int rows = g.n[1] * g.n[2];
  const int m0 = blockIdx.x * TP;
  const int np = min(TP, (rows + 1) / 2 - m0);
  const int n2 = threadIdx.x % R2;
  Cplx<T> w[R1];
  load_twiddles<T, R1, R2, -1>(w, n2, tw);
  constexpr int U = (TP * N + kFftXThreads - 1) / kFftXThreads;
  Cplx<T> v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = threadIdx.x + u * kFftXThreads, m = t / N, e = t % N, l = 2 * (m0 + m);
    v[u] = Cplx<T>{T(0), T(0)};
    if (rho && m < np) {
      v[u].re = rho[row_start(g, l) + e];
      if (l + 1 < rows) v[u].im = rho[row_start(g, l + 1) + e];
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = threadIdx.x + u * kFftXThreads;
    if (t < TP * N) buf[(t / N) * LS + slot_in<R1, R2>(t % N)] = v[u];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < np * R2; t += kFftXThreads)  // one n2: R2 divides the step
    dft_first_lds<T, T, R1, R2, -1, R2 + 1>(buf + (t / R2) * LS, n2, w);
  __syncthreads();
  for (int t = threadIdx.x; t < np * R1; t += kFftXThreads) {
    Cplx<T>* L = buf + (t / R1) * LS;
    const int k1 = t % R1;
    Cplx<T> a[R2];
    dft_second<T, T, R1, R2, -1, R2 + 1>(L, k1, a);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) L[(R2 + 1) * k1 + k2] = a[k2];
  }
  __syncthreads();
  // the rows' own spectra: (Z_e + conj Z_-e) / 2 and (Z_e - conj Z_-e) / 2i
  for (int t = threadIdx.x; t < np * 2 * H; t += kFftXThreads) {
    const int row = t / H, e = t - row * H, l = 2 * m0 + row;
    if (l >= rows) continue;
    const Cplx<T>* L = buf + (row >> 1) * LS;
    const Cplx<T> A = L[slot_out<R1, R2>(e)], B = L[slot_out<R1, R2>((N - e) & (N - 1))];
    c[(size_t)l * H + e] =
        (row & 1) ? Cplx<T>{T(0.5) * (A.im + B.im), T(0.5) * (B.re - A.re)}
                  : Cplx<T>{T(0.5) * (A.re + B.re), T(0.5) * (A.im - B.im)};
  }
}

// Back: half spectra -> real rows of the padded array psi.  The imaginary
// parts of the modes 0 and N/2 vanish (the spectrum is a real array's).
template <class T, int R1, int R2>
__global__ void __launch_bounds__(kFftXThreads) k_fft_x_back(Geo g, const Cplx<T>* __restrict__ c,
                                                             T* __restrict__ psi,
                                                             const Cplx<T>* __restrict__ tw) {
  constexpr int N = R1 * R2, H = N / 2 + 1, LS = line_slots<R1, R2>();
  constexpr int TP = pairs_per_block<R1, R2>();
  __shared__ Cplx<T> buf[TP * LS];
  const int rows = g.n[1] * g.n[2];
  const int m0 = blockIdx.x * TP;
  const int np = min(TP, (rows + 1) / 2 - m0);
  const int n2 = threadIdx.x % R2;
  Cplx<T> w[R1];
  load_twiddles<T, R1, R2, +1>(w, n2, tw);
  constexpr int U = (TP * H + kFftXThreads - 1) / kFftXThreads;
  Cplx<T> va[U], vb[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = threadIdx.x + u * kFftXThreads, m = t / H, e = t - m * H, l = 2 * (m0 + m);
    va[u] = vb[u] = Cplx<T>{T(0), T(0)};
    if (m < np) {
      va[u] = c[(size_t)l * H + e];
      if (l + 1 < rows) vb[u] = c[(size_t)(l + 1) * H + e];
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = threadIdx.x + u * kFftXThreads, m = t / H, e = t - m * H;
    if (m >= np) continue;
    Cplx<T> A = va[u], B = vb[u];
    if (e == 0 || 2 * e == N) A.im = B.im = T(0);
    Cplx<T>* L = buf + m * LS;
    L[slot_in<R1, R2>(e)] = Cplx<T>{A.re - B.im, A.im + B.re};
    if (e > 0 && 2 * e < N)
      L[slot_in<R1, R2>(N - e)] = Cplx<T>{A.re + B.im, B.re - A.im};
  }
  __syncthreads();
  for (int t = threadIdx.x; t < np * R2; t += kFftXThreads)  // one n2: R2 divides the step
    dft_first_lds<Fine, T, R1, R2, +1, R2 + 1>(buf + (t / R2) * LS, n2, w);
  __syncthreads();
  for (int t = threadIdx.x; t < np * R1; t += kFftXThreads) {
    Cplx<T>* L = buf + (t / R1) * LS;
    const int k1 = t % R1;
    Cplx<Fine> a[R2];
    dft_second<Fine, T, R1, R2, +1, R2 + 1>(L, k1, a);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) L[(R2 + 1) * k1 + k2] = cast<T>(a[k2]);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < np * 2 * N; t += kFftXThreads) {
    const int row = t / N, e = t % N, l = 2 * m0 + row;
    if (l >= rows) continue;
    const Cplx<T> v = buf[(row >> 1) * LS + slot_out<R1, R2>(e)];
    psi[row_start(g, l) + e] = (row & 1) ? v.im : v.re;
  }
}

// y- and z-lines of the half spectrum: a block takes TL lines of consecutive
// x (y-lines wrap into the next plane), a thread one line and every
// (threads / TL)-th element of it, so a wave's accesses are runs of TL
// values.  TL: 16 lines, fewer from 512 points up (the tile stays within 4096
// values of LDS).
template <int R1, int R2>
constexpr int lines_per_block() {
  return R1 * R2 <= 256 ? 16 : 4096 / (R1 * R2);
}
// This block's place in an order that gives each XCD (blocks are dealt out
// round-robin, block b to XCD b mod 8) a contiguous range: neighbouring tiles of
// y- or z-lines share the memory lines their runs end in, which then meet in
// one L2 (a y-pass at 128^3 FP32: 13 -> 7 us).
__device__ __forceinline__ int xcd_block() {
  const unsigned n = gridDim.x, b = blockIdx.x, q = n >> 3, r = n & 7u, x = b & 7u;
  return (int)(x * q + (x < r ? x : r) + (b >> 3));
}
template <int R1, int R2>
constexpr int line_threads() {
  constexpr int t = lines_per_block<R1, R2>() * R2;
  return t < 64 ? 64 : (t > 256 ? 256 : t);
}

// The first half of a line at base (element stride st) straight from memory:
// thread e0 < R2 of the line's G takes n2 = e0, whose elements are the ones it
// would stage for the others anyway.
template <class A, class T, int R1, int R2, int SIGN>
__device__ __forceinline__ void first_from(Cplx<T>* L, const Cplx<T>* base, int st, int e0,
                                           const Cplx<T>* __restrict__ tw) {
  Cplx<T> v[R1], w[R1];
  load_twiddles<T, R1, R2, SIGN>(w, e0, tw);
#pragma unroll
  for (int n1 = 0; n1 < R1; ++n1) v[n1] = base[(size_t)(R2 * n1 + e0) * st];
  Cplx<A> a[R1];
#pragma unroll
  for (int n1 = 0; n1 < R1; ++n1) a[n1] = cast<A>(v[n1]);
  dft_first<A, T, R1, R2, SIGN>(L, e0, a, w);
}

template <class T, int R1, int R2, int SIGN>
__global__ void __launch_bounds__((line_threads<R1, R2>()))
    k_fft_y(Geo g, Cplx<T>* c, const Cplx<T>* __restrict__ tw) {
  constexpr int N = R1 * R2, LS = N + 1, TL = lines_per_block<R1, R2>();
  constexpr int NT = line_threads<R1, R2>(), G = NT / TL;
  static_assert(G >= R2, "a thread a first-half DFT");
  __shared__ Cplx<T> buf[TL * LS];
  using A = std::conditional_t<(SIGN < 0), T, Fine>;
  const int H = g.n[0] / 2 + 1;
  const int line = threadIdx.x % TL, e0 = threadIdx.x / TL;
  const int l = xcd_block() * TL + line;  // x + H k
  const bool on = l < H * g.n[2];
  const int k = l / H;
  Cplx<T>* base = c + (size_t)k * H * N + (l - k * H);
  Cplx<T>* L = buf + line * LS;
  if (on && e0 < R2) first_from<A, T, R1, R2, SIGN>(L, base, H, e0, tw);
  __syncthreads();
  if (on)
    for (int k1 = e0; k1 < R1; k1 += G) {
      Cplx<A> a[R2];
      dft_second<A, T, R1, R2, SIGN>(L, k1, a);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) base[(size_t)(k1 + R1 * k2) * H] = cast<T>(a[k2]);
    }
}

// z-lines: forward, the division, and back.  After the forward DFT a thread
// holds the modes k1 + R1 k2 of one k1; mode (i, j, k) is multiplied by
// fac / (lx[i] + ly[j] + lz[k]) (4 pi G / N over the Laplacian's eigenvalue),
// the mean mode by zero.  The way back splits the other way round -- the
// R2-point DFT over k2 first, times W_N^(-k1 m2), then the R1-point DFT over
// k1 -- so it starts from the values in hand.
template <class T, int R1, int R2>
__global__ void __launch_bounds__((line_threads<R1, R2>())) k_fft_z_solve(
    Geo g, Cplx<T>* c, const Cplx<T>* __restrict__ tw, const T* __restrict__ lx,
    const T* __restrict__ ly, const T* __restrict__ lz, double fac) {
  constexpr int N = R1 * R2, LS = N + 1, TL = lines_per_block<R1, R2>();
  constexpr int NT = line_threads<R1, R2>(), G = NT / TL;
  __shared__ Cplx<T> buf[TL * LS];
  const int H = g.n[0] / 2 + 1;
  const int line = threadIdx.x % TL, e0 = threadIdx.x / TL;
  const int l = xcd_block() * TL + line;  // x + H j
  const int plane = H * g.n[1];
  const bool on = l < plane;
  const int j = on ? l / H : 0, i = on ? l - j * H : 0;
  Cplx<T>* base = c + l;
  Cplx<T>* L = buf + line * LS;
  // the modes a thread divides (k1 = e0 + G u), their factors and the way
  // back's twiddles: formed while the line is on its way
  constexpr int U = (R1 + G - 1) / G;
  T s[U][R2];
  Cplx<T> wb[U][R2];
  if (on) {
    const double lxy = (double)lx[i] + (double)ly[j];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k1 = min(e0 + G * u, R1 - 1);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) {
        const int k = k1 + R1 * k2;
        s[u][k2] = (l | k) == 0 ? T(0) : (T)(fac / (lxy + (double)lz[k]));
        if (k2 > 0) wb[u][k2] = twiddle<T, N, +1>(tw, (k1 * k2) & (N - 1));
      }
    }
    if (e0 < R2) first_from<Fine, T, R1, R2, -1>(L, base, plane, e0, tw);
  }
  __syncthreads();
  if (on) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k1 = e0 + G * u;
      if (k1 >= R1) break;
      Cplx<Fine> a[R2];
      dft_second<Fine, T, R1, R2, -1>(L, k1, a);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
        a[k2] = Cplx<Fine>{a[k2].re * s[u][k2], a[k2].im * s[u][k2]};
      dft_reg<Fine, R2, +1>(a);
      L[R2 * k1] = cast<T>(a[0]);
#pragma unroll
      for (int m2 = 1; m2 < R2; ++m2) L[R2 * k1 + m2] = cast<T>(cmul(a[m2], wb[u][m2]));
    }
  }
  __syncthreads();
  if (on)
    for (int m2 = e0; m2 < R2; m2 += G) {
      Cplx<Fine> a[R1];
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) a[k1] = cast<Fine>(L[R2 * k1 + m2]);
      dft_reg<Fine, R1, +1>(a);
#pragma unroll
      for (int m1 = 0; m1 < R1; ++m1) base[(size_t)(m2 + R2 * m1) * plane] = cast<T>(a[m1]);
    }
}

// Central gradient of Psi, periodic wrap; a wave takes a row.
template <class T>
__global__ void __launch_bounds__(256) k_grav_grad(Geo g, Grav<T> gr) {
  const int l = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (l >= g.n[1] * g.n[2]) return;
  const int k = l / g.n[1], j = l - k * g.n[1];
  const int wx = g.n[0] - 1, wy = (g.n[1] - 1) * g.sy, wz = (g.n[2] - 1) * g.sz;
  const int yu = j + 1 < g.n[1] ? g.sy : -wy, yd = j > 0 ? -g.sy : wy;
  const int zu = k + 1 < g.n[2] ? g.sz : -wz, zd = k > 0 ? -g.sz : wz;
  const T hx = (T)(0.5 / g.d[0]), hy = (T)(0.5 / g.d[1]), hz = (T)(0.5 / g.d[2]);
  const T* __restrict__ psi = gr.psi;
  T* __restrict__ gx = gr.g[0];
  T* __restrict__ gy = gr.g[1];
  T* __restrict__ gz = gr.g[2];
  const int p0 = row_start(g, l);
  for (int i = threadIdx.x & 63; i <= wx; i += 64) {
    const int p = p0 + i;
    gx[p] = (psi[i < wx ? p + 1 : p - wx] - psi[i > 0 ? p - 1 : p + wx]) * hx;
    gy[p] = (psi[p + yu] - psi[p + yd]) * hy;
    gz[p] = (psi[p + zu] - psi[p + zd]) * hz;
  }
}

// f<R1, R2>() for a line of n = R1 R2 points.
template <class F>
static void with_factors(int n, F f) {
  switch (n) {
    case 1: f.template operator()<1, 1>(); break;
    case 2: f.template operator()<2, 1>(); break;
    case 4: f.template operator()<2, 2>(); break;
    case 8: f.template operator()<4, 2>(); break;
    case 16: f.template operator()<4, 4>(); break;
    case 32: f.template operator()<8, 4>(); break;
    case 64: f.template operator()<8, 8>(); break;
    case 128: f.template operator()<16, 8>(); break;
    case 256: f.template operator()<16, 16>(); break;
    case 512: f.template operator()<32, 16>(); break;
    default: f.template operator()<32, 32>(); break;  // 1024
  }
}

template <class T>
struct FftX {
  const Geo& g;
  const T* rho;  // forward; null with back
  Cplx<T>* c;
  T* psi;
  const Cplx<T>* tw;
  bool back;
  hipStream_t st;
  template <int R1, int R2>
  void operator()() const {
    const int pairs = (g.n[1] * g.n[2] + 1) / 2, tp = pairs_per_block<R1, R2>();
    const dim3 gr((unsigned)((pairs + tp - 1) / tp)), bl(kFftXThreads);
    if (back)
      hipLaunchKernelGGL((k_fft_x_back<T, R1, R2>), gr, bl, 0, st, g, c, psi, tw);
    else
      hipLaunchKernelGGL((k_fft_x<T, R1, R2>), gr, bl, 0, st, g, rho, c, tw);
  }
};

template <class T>
struct FftY {
  const Geo& g;
  Cplx<T>* c;
  const Cplx<T>* tw;
  bool back;
  hipStream_t st;
  template <int R1, int R2>
  void operator()() const {
    const int lines = (g.n[0] / 2 + 1) * g.n[2], tl = lines_per_block<R1, R2>();
    const dim3 gr((unsigned)((lines + tl - 1) / tl)), bl(line_threads<R1, R2>());
    if (back)
      hipLaunchKernelGGL((k_fft_y<T, R1, R2, +1>), gr, bl, 0, st, g, c, tw);
    else
      hipLaunchKernelGGL((k_fft_y<T, R1, R2, -1>), gr, bl, 0, st, g, c, tw);
  }
};

template <class T>
struct FftZ {
  const Geo& g;
  Cplx<T>* c;
  const Cplx<T>* tw;
  const T *lx, *ly, *lz;
  double fac;
  hipStream_t st;
  template <int R1, int R2>
  void operator()() const {
    const int lines = (g.n[0] / 2 + 1) * g.n[1], tl = lines_per_block<R1, R2>();
    hipLaunchKernelGGL((k_fft_z_solve<T, R1, R2>), dim3((unsigned)((lines + tl - 1) / tl)),
                       dim3(line_threads<R1, R2>()), 0, st, g, c, tw, lx, ly, lz, fac);
  }
};

template <class T>
void launch_self_gravity(const Geo& g, const Physics& ph, const T* rho, GravFFT<T> f, Grav<T> gr,
                         Parts<T> pp, DtRef h, hipStream_t st) {
  const double N = (double)g.n[0] * g.n[1] * g.n[2];
  const dim3 rows((unsigned)((g.n[1] * g.n[2] + 3) / 4));
  Cplx<T>* c = (Cplx<T>*)f.c;
  const Cplx<T>* tw[3] = {(const Cplx<T>*)f.tw[0], (const Cplx<T>*)f.tw[1],
                          (const Cplx<T>*)f.tw[2]};
  const bool with_gas = ph.src[1] != 1.0;
  const T* src = with_gas ? rho : nullptr;
  if (pp.n > 0) {  // gathered in Psi's array, which the solve writes last
    hipLaunchKernelGGL(k_grav_load<T>, rows, dim3(256), 0, st, g, rho, gr.psi, with_gas ? 1 : 0);
    launch_deposit<T>(g, pp, h, gr.psi, st);
    src = gr.psi;
  }
  const double fac = 4.0 * 3.14159265358979323846 * ph.src[0] / N;
  with_factors(g.n[0], FftX<T>{g, src, c, nullptr, tw[0], false, st});
  if (g.n[1] > 1) with_factors(g.n[1], FftY<T>{g, c, tw[1], false, st});
  with_factors(g.n[2], FftZ<T>{g, c, tw[2], f.lam[0], f.lam[1], f.lam[2], fac, st});
  if (g.n[1] > 1) with_factors(g.n[1], FftY<T>{g, c, tw[1], true, st});
  with_factors(g.n[0], FftX<T>{g, nullptr, c, gr.psi, tw[0], true, st});
  hipLaunchKernelGGL(k_grav_grad<T>, rows, dim3(256), 0, st, g, gr);
}

template void launch_self_gravity<double>(const Geo&, const Physics&, const double*,
                                          GravFFT<double>, Grav<double>, Parts<double>, DtRef,
                                          hipStream_t);
template void launch_self_gravity<float>(const Geo&, const Physics&, const float*, GravFFT<float>,
                                         Grav<float>, Parts<float>, DtRef, hipStream_t);

}  // namespace mhd
