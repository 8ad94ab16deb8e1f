// mhd_nbody.hip -- N-body particles of the step (section 2.1 of the paper:
// particle-in-cell dynamics with the "flip-flop" integrator, a
// mass-conserving second-order mass assignment), sharing the periodic
// potential of the self-gravity solve.
//
// Cloud in cell: a particle is a cube of one cell's size; along each axis,
// in cell-centre units s = (x - x0)/d - 1/2, it overlaps cells floor(s)
// and floor(s) + 1 (periodic) with fractions 1 - f and f, f = s - floor(s).
// The deposit adds m w_x w_y w_z / dV to each of the 8 cells; the force is
// minus the cell-centred central gradient of Psi interpolated with the same
// weights, which keeps the total momentum.
//
// The particles are kept sorted by tile (kTile^3 cells): every step starts
// with a counting sort by the tile of each particle's cell (counts gathered
// per block in LDS, one global atomic per distinct tile and block), and
// each tile's particles are cut into chunks of at most kChunk.  One block per chunk then works in LDS: the deposit
// adds into a private copy of the cells the tile's particles can reach (the
// tile and 2 cells around it: a particle moves at most half a cell between
// the sort and the half-step deposit under the CFL limit) and flushes it
// with one atomic per touched cell; the kick stages the potential gradient
// of the same cells.  A target outside that window (a step larger than the
// CFL limit) goes to HBM directly.  The device-scope atomics of the first
// version -- 8 per particle, piled onto the few cells of a dense core -- took
// most of the step.
#include <limits.h>
#include <math.h>

#include "mhd_span.hpp"

namespace mhd {

constexpr int kPartThreads = 256;
constexpr int kWin = kTile + 5;  // LDS window per axis: tile cells -2 .. kTile + 2
constexpr int kWin3 = kWin * kWin * kWin;
constexpr int kStageMin = 256;   // particles per tile from which the kick stages in LDS

static unsigned part_blocks(long long n) {
  const long long b = (n + kPartThreads - 1) / kPartThreads;
  return (unsigned)(b < 65536 ? (b > 0 ? b : 1) : 65536);
}

// A position inside the box (nearly all) stands as it is: the floor is 0.
template <class T>
__device__ __forceinline__ T wrap_coord(T x, double lo, double L) {
  const double r = (double)x - lo;
  if (r >= 0.0 && r < L) return x;
  return (T)((double)x - L * floor(r / L));
}

// Weights of one axis: cells c[0], c[1] (interior indices), fractions w.  x
// is wrapped, so its lower cell lies in -1 .. n; the clamp keeps the indices
// of a position that is no number in range.
template <class T>
__device__ __forceinline__ void cic_axis(const Geo& g, int a, T x, int c[2], T w[2]) {
  const T s = (x - (T)g.x0[a]) / (T)g.d[a] - T(0.5);
  const T fl = floor(s);
  const int n = g.n[a];
  int c0 = (int)fl;
  c0 = c0 < 0 ? c0 + n : (c0 >= n ? c0 - n : c0);
  c0 = min(max(c0, 0), n - 1);
  c[0] = c0;
  c[1] = c0 + 1 < n ? c0 + 1 : 0;
  w[1] = s - fl;
  w[0] = T(1) - w[1];
}

// Cell of a (wrapped) position along axis a, for the choice of its tile (a
// position on a cell's side may go to either one: both windows hold it).
template <class T>
__device__ __forceinline__ int cell_of(const Geo& g, int a, T x) {
  const int c = (int)floor(((double)x - g.x0[a]) * g.id[a]);
  return min(max(c, 0), g.n[a] - 1);
}

template <class T>
__device__ __forceinline__ int tile_of(const Geo& g, const Parts<T>& pp, long long q) {
  const long long n = pp.n;
  const int tx = cell_of(g, 0, pp.x[q]) / kTile;
  const int ty = cell_of(g, 1, pp.x[n + q]) / kTile;
  const int tz = cell_of(g, 2, pp.x[2 * n + q]) / kTile;
  return (tz * pp.nt[1] + ty) * pp.nt[0] + tx;
}

// Window index of global cell c along an axis whose window starts at cell
// o - 2 (periodic extent n), or -1 outside the window.
__device__ __forceinline__ int win_index(int c, int o, int n) {
  int d = c - (o - 2);
  if (d < 0) d += n;
  if (d >= n) d -= n;
  return d < kWin ? d : -1;
}
// Its inverse: the box's cell of window cell w along an axis of extent n whose
// window starts at cell o - 2 (o < n).  From kWin cells up one step of n
// brings it into the box, without a remainder an axis and cell.
__device__ __forceinline__ int win_cell(int w, int o, int n) {
  int c = o - 2 + w;
  if (n >= kWin) return c < 0 ? c + n : (c >= n ? c - n : c);
  c %= n;
  return c < 0 ? c + n : c;
}
// Window index of the lower of a particle's two cells, the upper one's being the
// next, or -1 if they do not both lie in the window.  A box narrower than the
// window has its cells there more than once (win_cell), so this holds at its
// sides too: looked up by itself, the upper cell's first index is not the next
// one there, and such particles, 1 in n an axis, went past the window (2^20
// particles on 8^3 cells: 3449 us a step, 312 with this).
__device__ __forceinline__ int win_pair(int c, int o, int n) {
  const int d = win_index(c, o, n);
  return d + 1 < kWin ? d : -1;
}

__device__ __forceinline__ void atomic_add_t(double* p, double v) { atomicAdd(p, v); }
__device__ __forceinline__ void atomic_add_t(float* p, float v) { atomicAdd(p, v); }

// ---------------------------------------------------------------------------
// Sort by tile
// ---------------------------------------------------------------------------

// Block-level aggregation of the sort's counters: a block takes kSortChunk
// consecutive particles -- in the order of the last sort, so a few tiles
// and their neighbours -- and gathers their per-tile counts in an LDS hash
// table (kSortSlots slots, linear probing) before one global atomic per
// distinct tile.  A key the table cannot place within kSortProbes probes
// goes to HBM directly (the first sort of particles in arbitrary order).
// (Per-wave aggregation alone still piled ~2000 atomics per step onto the
// counter of a dense core tile.)
constexpr int kSortChunk = 4096;
constexpr int kSortSlots = 512;
constexpr int kSortProbes = 32;  // a key not placed within this many probes goes to HBM

struct SortTable {
  int key[kSortSlots];
  int cnt[kSortSlots];
  int base[kSortSlots];
};

__device__ __forceinline__ void table_clear(SortTable& tb) {
  for (int i = threadIdx.x; i < kSortSlots; i += kPartThreads) {
    tb.key[i] = -1;
    tb.cnt[i] = 0;
  }
}

// Slot of key in the table (inserted if absent), or -1 if it finds no place
// within kSortProbes probes.
__device__ __forceinline__ int table_find(SortTable& tb, int key) {
  int h = (int)(((unsigned)key * 2654435761u) >> 20) & (kSortSlots - 1);
  for (int probe = 0; probe < kSortProbes; ++probe) {
    const int k = __atomic_load_n(&tb.key[h], __ATOMIC_RELAXED);
    if (k == key) return h;
    if (k == -1) {
      const int old = atomicCAS(&tb.key[h], -1, key);
      if (old == -1 || old == key) return h;
    }
    h = (h + 1) & (kSortSlots - 1);
  }
  return -1;
}

static unsigned sort_blocks(long long n) {
  return (unsigned)((n + kSortChunk - 1) / kSortChunk);
}

template <class T>
__global__ void __launch_bounds__(kPartThreads) k_tile_count(Geo g, Parts<T> pp, int* cnt) {
  __shared__ SortTable tb;
  table_clear(tb);
  __syncthreads();
  const long long n = pp.n;
  const long long q0 = (long long)blockIdx.x * kSortChunk;
  const long long q1 = q0 + kSortChunk < n ? q0 + kSortChunk : n;
  for (long long q = q0 + threadIdx.x; q < q1; q += kPartThreads) {
    const int key = tile_of(g, pp, q);
    const int h = table_find(tb, key);
    if (h >= 0)
      atomicAdd(&tb.cnt[h], 1);
    else
      atomicAdd(cnt + key, 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kSortSlots; i += kPartThreads)
    if (tb.cnt[i] > 0) atomicAdd(cnt + tb.key[i], tb.cnt[i]);
}

// One block, each thread a contiguous share of the tiles: the exclusive scan
// of cnt into the scatter's cursors, cnt back to zero for the next sort, and the
// list of chunks of at most kChunk particles within each tile (count, then tile, first, end of each).  (As seven
// launches -- clear, count, scan, scatter, chunk counts, their scan, the list
// -- the small ones took 25 us a sort.)
__global__ void __launch_bounds__(1024) k_tile_scan(int* cnt, int* cur, int* chunk, int ntiles) {
  __shared__ int part[1024], cpart[1024];
  const int share = (ntiles + 1023) / 1024;
  const int lo = min(ntiles, (int)threadIdx.x * share), hi = min(ntiles, lo + share);
  int s = 0, nc = 0;
  for (int t = lo; t < hi; ++t) {
    s += cnt[t];
    nc += chunk_count(cnt[t]);
  }
  part[threadIdx.x] = s;
  cpart[threadIdx.x] = nc;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {  // inclusive Hillis-Steele scans of the shares
    const int v = threadIdx.x >= (unsigned)d ? part[threadIdx.x - d] : 0;
    const int w = threadIdx.x >= (unsigned)d ? cpart[threadIdx.x - d] : 0;
    __syncthreads();
    part[threadIdx.x] += v;
    cpart[threadIdx.x] += w;
    __syncthreads();
  }
  int base = part[threadIdx.x] - s, k = cpart[threadIdx.x] - nc;
  for (int t = lo; t < hi; ++t) {
    const int c = cnt[t];
    cur[t] = base;
    cnt[t] = 0;
    k = list_chunks(chunk, k, t, base, c);
    base += c;
  }
  if (threadIdx.x == 1023) chunk[0] = cpart[1023];
}

// Same blocks and table as the count: each distinct tile reserves its
// block's range of slots with one global atomic on its cursor; a particle's
// place in that range is its rank in the table's counter (the order within a
// tile's range is not deterministic).  A thread keeps the table slots and
// ranks of its particles between the two passes.
template <class T>
__global__ void __launch_bounds__(kPartThreads) k_tile_scatter(Geo g, Parts<T> pp, PartSort<T> s) {
  constexpr int U = kSortChunk / kPartThreads;
  __shared__ SortTable tb;
  table_clear(tb);
  __syncthreads();
  const long long n = pp.n;
  const long long q0 = (long long)blockIdx.x * kSortChunk + threadIdx.x;
  int slot[U], rank[U];  // slot -1 - tile: not in the table
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const long long q = q0 + u * kPartThreads;
    slot[u] = rank[u] = 0;
    if (q < n) {
      const int key = tile_of(g, pp, q), h = table_find(tb, key);
      slot[u] = h >= 0 ? h : -1 - key;
      if (h >= 0) rank[u] = atomicAdd(&tb.cnt[h], 1);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kSortSlots; i += kPartThreads)
    if (tb.cnt[i] > 0) tb.base[i] = atomicAdd(s.cur + tb.key[i], tb.cnt[i]);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const long long q = q0 + u * kPartThreads;
    if (q >= n) continue;
    const int to = slot[u] >= 0 ? tb.base[slot[u]] + rank[u] : atomicAdd(s.cur + (-1 - slot[u]), 1);
    T x[3], v[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      x[a] = pp.x[a * n + q];
      v[a] = pp.v[a * n + q];
    }
    const T m = pp.m[q];
    const int id = pp.id[q];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      s.x[a * n + to] = x[a];
      s.v[a * n + to] = v[a];
    }
    s.m[to] = m;
    s.id[to] = id;
  }
}

template <class T>
void launch_particle_sort(const Geo& g, Parts<T> pp, PartSort<T> s, hipStream_t st) {
  if (pp.n <= 0) return;
  hipLaunchKernelGGL(k_tile_count<T>, dim3(sort_blocks(pp.n)), dim3(kPartThreads), 0, st, g, pp,
                     s.cnt);
  hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(1024), 0, st, s.cnt, s.cur, s.chunk, pp.ntiles);
  hipLaunchKernelGGL(k_tile_scatter<T>, dim3(sort_blocks(pp.n)), dim3(kPartThreads), 0, st, g,
                     pp, s);
}

// ---------------------------------------------------------------------------
// Deposit, kick-drift
// ---------------------------------------------------------------------------

// The deposit's window in LDS.  FP32: 64-bit fixed point.  An LDS add of
// floats occupies the LDS 111 cycles a wave whatever its addresses (74 % of a
// 219 us launch for 2^22 particles), an integer add 8.5.  The unit is 2^-50 of a bound on one particle's density, so the sum
// of a chunk's particles (at most kChunk = 2^11) stays below 2^62 and is exact
// to that unit; a chunk whose masses differ by more than 2^20 (the unit would
// no longer be far below the smallest one's rounding), or are not finite,
// takes float adds in the window (2^20 particles in a clump, masses over nine
// decades: 295 us a step; with adds to the array 35500).  A particle
// whose position is no number adds to the array.  In fixed point a launch took
// 75 us, its waves waiting for a particle's values and for the array's atomics at
// the end; 56 with the values loaded a turn ahead (waiting 51 % of the time).
// FP64 keeps floating adds.
template <class T>
struct DepositCell {
  typedef T type;
};
template <>
struct DepositCell<float> {
  typedef unsigned long long type;
};
static_assert(kChunk <= 2048, "fixed-point headroom of the deposit");

__device__ __forceinline__ void window_add(double* a, double v, double) { atomicAdd(a, v); }
__device__ __forceinline__ void window_add(unsigned long long* a, float v, double scale) {
  if (scale == 0.0) {
    atomicAdd((float*)a, v);
    return;
  }
  // |v scale| < 2^51: adding 1.5 2^52 leaves the nearest integer in the
  // low bits of the sum
  const double m = 0x1.8p52;
  atomicAdd(a, (unsigned long long)(__double_as_longlong(fma((double)v, scale, m)) -
                                    __double_as_longlong(m)));
}
__device__ __forceinline__ double window_value(const double* a, double) { return *a; }
// scale, unit 0: the cell holds a float
__device__ __forceinline__ float window_value(const unsigned long long* a, double unit) {
  return unit != 0.0 ? (float)((double)(long long)*a * unit) : *(const float*)a;
}

// Exponent e with |m| idv < 2^e for every mass m of the nq particles at m,
// or INT_MIN if the chunk cannot use fixed point.
__device__ __forceinline__ int chunk_exponent(const float* __restrict__ m, int nq, float idv) {
  __shared__ float hi[kPartThreads / 64], lo[kPartThreads / 64];
  float a = 0.f, b = INFINITY;
  for (int u = (int)threadIdx.x; u < nq; u += kPartThreads) {
    const float v = fabsf(m[u]) * idv;
    a = v <= a || a != a ? a : v;  // a NaN stays
    if (v > 0.f) b = fminf(b, v);
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float v = __shfl_xor(a, o, 64);
    a = v <= a ? a : (a == a ? v : a);
    b = fminf(b, __shfl_xor(b, o, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    hi[threadIdx.x >> 6] = a;
    lo[threadIdx.x >> 6] = b;
  }
  __syncthreads();
  bool bad = false;
  a = 0.f, b = INFINITY;
  for (int w = 0; w < kPartThreads / 64; ++w) {
    bad = bad || !(hi[w] < INFINITY);
    a = fmaxf(a, hi[w]);
    b = fminf(b, lo[w]);
  }
  if (bad || !(b * 0x1p20f >= a)) return INT_MIN;
  int e = 0;
  (void)frexpf(a, &e);
  return e;
}

// One block per chunk: the cloud-in-cell density of the tile's particles at
// x + h v (h = dt x factor), added to the padded array c.
template <class T>
__global__ void __launch_bounds__(kPartThreads) k_deposit(Geo g, Parts<T> pp, DtRef hr, T* c) {
  __shared__ typename DepositCell<T>::type acc[kWin3];
  if ((int)blockIdx.x >= pp.chunk[0]) return;
  const int t = pp.chunk[1 + 3 * blockIdx.x];
  // its particles q0 .. q0 + nq - 1, counted from q0: the end may be the largest int
  const int q0 = pp.chunk[2 + 3 * blockIdx.x], nq = pp.chunk[3 + 3 * blockIdx.x] - q0;
  const int tx = t % pp.nt[0], ty = (t / pp.nt[0]) % pp.nt[1], tz = t / (pp.nt[0] * pp.nt[1]);
  const int o[3] = {tx * kTile, ty * kTile, tz * kTile};
  for (int i = threadIdx.x; i < kWin3; i += kPartThreads) acc[i] = 0;
  const double h = (hr.ptr ? *hr.ptr : hr.value) * hr.factor;
  const T idv = (T)(1.0 / (g.d[0] * g.d[1] * g.d[2]));
  const long long n = pp.n;
  double scale = 1.0, unit = 1.0;
  if constexpr (sizeof(T) == 4) {
    const int e = __builtin_amdgcn_readfirstlane(chunk_exponent(pp.m + q0, nq, idv));
    scale = e != INT_MIN ? ldexp(1.0, 50 - e) : 0.0;
    unit = e != INT_MIN ? ldexp(1.0, e - 50) : 0.0;
  }
  // a particle's values are loaded a turn ahead
  T px[3], pv[3], pm = T(0);
  const auto fetch = [&](int u) {
    if (u >= nq) return;
    const int q = q0 + u;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      px[a] = pp.x[a * n + q];
      pv[a] = h != 0.0 ? pp.v[a * n + q] : T(0);
    }
    pm = pp.m[q];
  };
  fetch((int)threadIdx.x);
  __syncthreads();
  for (int u = (int)threadIdx.x; u < nq; u += kPartThreads) {
    int ci[3][2], wi[3];
    T w[3][2];
    bool in = true;
    const T cx[3] = {px[0], px[1], px[2]}, cv[3] = {pv[0], pv[1], pv[2]}, m = pm;
    fetch(u + kPartThreads);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T x = cx[a];
      if (h != 0.0) x = wrap_coord<T>(x + (T)h * cv[a], g.x0[a], g.n[a] * g.d[a]);
      cic_axis<T>(g, a, x, ci[a], w[a]);
      wi[a] = win_pair(ci[a][0], o[a], g.n[a]);
      in = in && wi[a] >= 0 && w[a][1] >= T(0) && w[a][1] <= T(1);
    }
    const int wb = (wi[2] * kWin + wi[1]) * kWin + wi[0];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const T val = m * w[0][a] * w[1][b] * w[2][e] * idv;
          if (in)
            window_add(&acc[wb + (e * kWin + b) * kWin + a], val, scale);
          else
            atomic_add_t(c + pidx(g, ci[0][a], ci[1][b], ci[2][e]), val);
        }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kWin3; i += kPartThreads) {
    const T v = window_value(&acc[i], unit);
    if (v == T(0)) continue;
    const int a0 = i % kWin, a1 = (i / kWin) % kWin, a2 = i / (kWin * kWin);
    int gc[3];
    const int ai[3] = {a0, a1, a2};
#pragma unroll
    for (int a = 0; a < 3; ++a) gc[a] = win_cell(ai[a], o[a], g.n[a]);
    atomic_add_t(c + pidx(g, gc[0], gc[1], gc[2]), v);
  }
}

template <class T>
__device__ __forceinline__ T grad_at(const Geo& g, const Grav<T>& gr, int a, int i, int j, int k) {
  return gr.g[a][(i + NG) + g.sy * (j + NG) + g.sz * (k + NG)];
}

// One block per tile: x_h = x + dt/2 v, v -= dt grad Psi(x_h) (cloud in
// cell), x = x_h + dt/2 v; tiles with many particles stage the gradient of
// their window in LDS first.  Bound by the latency of its loads: 82 us for 2^22
// particles (FP32, 128^3) with a particle's values loaded where used, 67 a turn
// ahead.
template <class T>
__global__ void __launch_bounds__(kPartThreads) k_kick_drift(Geo g, Parts<T> pp, Grav<T> gr,
                                                             DtRef dtr) {
  __shared__ T gl[3][kWin3];
  if ((int)blockIdx.x >= pp.chunk[0]) return;
  const int t = pp.chunk[1 + 3 * blockIdx.x];
  // its particles q0 .. q0 + nq - 1, counted from q0: the end may be the largest int
  const int q0 = pp.chunk[2 + 3 * blockIdx.x], nq = pp.chunk[3 + 3 * blockIdx.x] - q0;
  const int tx = t % pp.nt[0], ty = (t / pp.nt[0]) % pp.nt[1], tz = t / (pp.nt[0] * pp.nt[1]);
  const int o[3] = {tx * kTile, ty * kTile, tz * kTile};
  const bool staged = nq >= kStageMin;
  const long long n = pp.n;
  // a particle's values are loaded a turn ahead, the first beside the window's
  T px[3], pv[3];
  const auto fetch = [&](int u) {
    if (u >= nq) return;
    const int q = q0 + u;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      px[a] = pp.x[a * n + q];
      pv[a] = pp.v[a * n + q];
    }
  };
  fetch((int)threadIdx.x);
  if (staged) {
    for (int i = threadIdx.x; i < kWin3; i += kPartThreads) {
      const int ai[3] = {i % kWin, (i / kWin) % kWin, i / (kWin * kWin)};
      int gc[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) gc[a] = win_cell(ai[a], o[a], g.n[a]);
#pragma unroll
      for (int a = 0; a < 3; ++a) gl[a][i] = grad_at(g, gr, a, gc[0], gc[1], gc[2]);
    }
  }
  __syncthreads();
  const double dt = (dtr.ptr ? *dtr.ptr : dtr.value) * dtr.factor;
  const T hdt = (T)(0.5 * dt), Tdt = (T)dt;
  for (int u = (int)threadIdx.x; u < nq; u += kPartThreads) {
    const int q = q0 + u;
    T xh[3], vh[3], w[3][2], acc[3] = {T(0), T(0), T(0)};
    int ci[3][2], wi[3];
    bool in = staged;
    const T cx[3] = {px[0], px[1], px[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) vh[a] = pv[a];
    fetch(u + kPartThreads);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      xh[a] = wrap_coord<T>(cx[a] + hdt * vh[a], g.x0[a], g.n[a] * g.d[a]);
      cic_axis<T>(g, a, xh[a], ci[a], w[a]);
      wi[a] = win_pair(ci[a][0], o[a], g.n[a]);
      in = in && wi[a] >= 0;
    }
    const int wb = (wi[2] * kWin + wi[1]) * kWin + wi[0];
    // one branch a particle (a choice per value between the window and the
    // array took as many instructions as the interpolation)
    if (in) {
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const T wt = w[0][i] * w[1][b] * w[2][e];
#pragma unroll
            for (int a = 0; a < 3; ++a) acc[a] += wt * gl[a][wb + (e * kWin + b) * kWin + i];
          }
    } else {
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const T wt = w[0][i] * w[1][b] * w[2][e];
#pragma unroll
            for (int a = 0; a < 3; ++a)
              acc[a] += wt * grad_at(g, gr, a, ci[0][i], ci[1][b], ci[2][e]);
          }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const T v = vh[a] - Tdt * acc[a];
      pp.v[a * n + q] = v;
      pp.x[a * n + q] = wrap_coord<T>(xh[a] + hdt * v, g.x0[a], g.n[a] * g.d[a]);
    }
  }
}

template <class T>
__global__ void __launch_bounds__(kPartThreads) k_particles_init(Geo g, Parts<T> pp) {
  const long long n = pp.n;
  for (long long q = (long long)blockIdx.x * kPartThreads + threadIdx.x; q < n;
       q += (long long)gridDim.x * kPartThreads) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
      pp.x[a * n + q] = wrap_coord<T>(pp.x[a * n + q], g.x0[a], g.n[a] * g.d[a]);
    pp.id[q] = (int)q;
  }
}

// Particles in the caller's order, each value straight to its place.
template <class T>
__global__ void __launch_bounds__(kPartThreads) k_particles_place(Parts<T> pp, T* xo, T* vo) {
  const long long n = pp.n;
  for (long long q = (long long)blockIdx.x * kPartThreads + threadIdx.x; q < n;
       q += (long long)gridDim.x * kPartThreads) {
    const long long u = pp.id[q];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (xo) xo[a * n + u] = pp.x[a * n + q];
      if (vo) vo[a * n + u] = pp.v[a * n + q];
    }
  }
}

// The same by way of records: first each particle's six values as one record
// at its place in rec (the other particle buffer), then the records turned
// into rows.  Six separate rows written in the particles' random order touch
// six lines a particle.
template <class T>
__global__ void __launch_bounds__(kPartThreads) k_particles_record(Parts<T> pp, T* rec) {
  const long long n = pp.n;
  for (long long q = (long long)blockIdx.x * kPartThreads + threadIdx.x; q < n;
       q += (long long)gridDim.x * kPartThreads) {
    T* r = rec + 6 * (long long)pp.id[q];
    T v[6];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] = pp.x[a * n + q];
      v[3 + a] = pp.v[a * n + q];
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) r[a] = v[a];
  }
}

template <class T>
__global__ void __launch_bounds__(kPartThreads) k_particles_out(long long n,
                                                                const T* __restrict__ rec, T* xo,
                                                                T* vo) {
  for (long long u = (long long)blockIdx.x * kPartThreads + threadIdx.x; u < n;
       u += (long long)gridDim.x * kPartThreads) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (xo) xo[a * n + u] = rec[6 * u + a];
      if (vo) vo[a * n + u] = rec[6 * u + 3 + a];
    }
  }
}

// Block minimum of d_a / |v_a| over the particles into part[blockIdx.x]
// (kPartCflBlocks blocks, grid-stride).
template <class T>
__global__ void __launch_bounds__(kPartThreads) k_particle_cfl(Geo g, Parts<T> pp, double* part) {
  __shared__ double red[kPartThreads / 64];
  const long long n = pp.n;
  // the smallest quotient is the one of the largest speed: one division an
  // axis and thread
  T top[3] = {T(0), T(0), T(0)};
  for (long long q = (long long)blockIdx.x * kPartThreads + threadIdx.x; q < n;
       q += (long long)gridDim.x * kPartThreads)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const T v = fabs(pp.v[a * n + q]);
      top[a] = v > top[a] ? v : top[a];
    }
  double r = INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if (top[a] > T(0)) r = fmin(r, g.d[a] / (double)top[a]);
  for (int off = 32; off > 0; off >>= 1) r = fmin(r, __shfl_xor(r, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = r;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = red[0];
    for (int wv = 1; wv < kPartThreads / 64; ++wv) m = fmin(m, red[wv]);
    part[blockIdx.x] = m;
  }
}

template <class T>
void launch_particle_cfl(const Geo& g, Parts<T> pp, double* part, hipStream_t st) {
  hipLaunchKernelGGL(k_particle_cfl<T>, dim3(kPartCflBlocks), dim3(kPartThreads), 0, st, g, pp,
                     part);
}

template <class T>
void launch_deposit(const Geo& g, Parts<T> pp, DtRef h, T* c, hipStream_t st) {
  if (pp.n <= 0) return;
  hipLaunchKernelGGL(k_deposit<T>, dim3((unsigned)pp.max_chunks), dim3(kPartThreads), 0, st, g, pp,
                     h, c);
}

template <class T>
void launch_kick_drift(const Geo& g, Parts<T> pp, Grav<T> gr, DtRef dt, hipStream_t st) {
  if (pp.n <= 0) return;
  hipLaunchKernelGGL(k_kick_drift<T>, dim3((unsigned)pp.max_chunks), dim3(kPartThreads), 0, st, g,
                     pp, gr, dt);
}

template <class T>
void launch_particles_init(const Geo& g, Parts<T> pp, hipStream_t st) {
  if (pp.n <= 0) return;
  hipLaunchKernelGGL(k_particles_init<T>, dim3(part_blocks(pp.n)), dim3(kPartThreads), 0, st, g,
                     pp);
}

template <class T>
void launch_particles_out(Parts<T> pp, T* rec, T* x_out, T* v_out, hipStream_t st) {
  if (pp.n <= 0) return;
  // Records pay from where the rows' lines no longer meet in the caches before
  // they are written back, if many tiles scatter the order: us a call on 64^3
  // cells straight / by records, FP32 10^5 particles 23.8 / 23.7, 3 10^5 34.7 /
  // 29.2, 4 10^6 300 / 211 (FP64 25.0 / 25.6, 39.4 / 35.7, 667 / 277), 10^3
  // 19.5 / 21.7; 4 10^6 in 1, 2 and 8 tiles 48 / 89, 106 / 132 and 178 / 179.
  if (pp.n <= (1 << 17) || pp.ntiles < 8) {
    hipLaunchKernelGGL(k_particles_place<T>, dim3(part_blocks(pp.n)), dim3(kPartThreads), 0, st,
                       pp, x_out, v_out);
    return;
  }
  hipLaunchKernelGGL(k_particles_record<T>, dim3(part_blocks(pp.n)), dim3(kPartThreads), 0, st,
                     pp, rec);
  hipLaunchKernelGGL(k_particles_out<T>, dim3(part_blocks(pp.n)), dim3(kPartThreads), 0, st, pp.n,
                     rec, x_out, v_out);
}

#define MHD_NBODY_INST(T)                                                                        \
  template void launch_particle_cfl<T>(const Geo&, Parts<T>, double*, hipStream_t);             \
  template void launch_deposit<T>(const Geo&, Parts<T>, DtRef, T*, hipStream_t);                \
  template void launch_kick_drift<T>(const Geo&, Parts<T>, Grav<T>, DtRef, hipStream_t);        \
  template void launch_particles_init<T>(const Geo&, Parts<T>, hipStream_t);                    \
  template void launch_particle_sort<T>(const Geo&, Parts<T>, PartSort<T>, hipStream_t);        \
  template void launch_particles_out<T>(Parts<T>, T*, T*, T*, hipStream_t);

MHD_NBODY_INST(double)
MHD_NBODY_INST(float)

}  // namespace mhd
