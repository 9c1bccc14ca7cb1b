// ILU(0) sweeps by tiles: x = U^{-1} L^{-1} b for one right-hand side.
//
// What bounds a triangular sweep in natural order is its dependency chain
// (for a 3D grid about nx + ny + nz rows, plus the fractures'), not its
// bytes.  A sweep that hands every level over through global memory pays a
// memory round trip per level; here a level costs a few LDS accesses:
//
//  * Rows are cut into tiles whose dependencies run from lower to higher
//    tile numbers: boxes of tx x ty x tz cells where the matrix rows form a
//    grid in natural order (ty * tz = 64 grid lines, so that a level of a
//    box, the cells with equal x + y + z, is at most one row per lane), and
//    runs of consecutive rows elsewhere.  A workgroup owns a tile and walks
//    it level by level; values of its own rows pass through LDS.
//  * Positions: rows sorted by (tile, level).  Levels are increasing along
//    every coupling in either direction, so the upper sweep walks the same
//    positions backwards, and vectors, factor values and column codes are
//    read contiguously, by slices (<= 64 rows of one level).
//  * Rows of other tiles are read from global memory, published value by
//    value (ready.hpp); only rows that another tile depends on are published.
//    The dependency chain crosses about nx/tx + ny/ty + nz/tz tiles, each a
//    memory round trip.
//  * The two media are two phases, one launch each: every coupling between
//    a matrix row and a fracture row (or well) is subtracted in between by a
//    parallel pass (k_pre_lower, k_pre_upper), off the chain.
//
// Measured per application (lower + upper, all launches), against one launch
// a sweep over ranges of 8192 rows with a barrier per level: 104 against 376
// us on the 100x100 grid with 20 fractures (199 levels), 354 against 1122 us
// on 100x100x50 with 100 plates (FP64, 619k rows, 311 levels), 1.0 against
// 3.3 ms on 256x256x128 with 2000 plates (FP32, 9.4M rows).  Eight
// wavefronts a workgroup with two slices each, and sixteen with one where a
// row has eight places, were the best of {4, 8, 16} x {1, 2, 4, 8}; boxes of
// 64 cells along x instead of 128 cost 20%, runs of 1024 rows instead of
// 4096 60% more time in the fracture phase.
//
// A row's terms are subtracted in ascending column order in the lower sweep
// and in descending order in the upper one (the order in which they become
// available), each with one fused multiply-add; the result does not depend
// on the tiles.
#include <algorithm>
#include <climits>
#include <type_traits>
#include <vector>

#include "internal.hpp"
#include "ready.hpp"

namespace fams {
namespace {

// Looks at the turn together with the dependencies (k_tile_sweep).  The turn
// comes by itself: the wavefronts ahead wait for nothing but earlier turns and
// other tiles, by the clock (2 s, and no longer once an error is flagged).  The
// count is a guard beyond that, over 4 s at an LDS round trip each.  (Both sweeps
// of 10k FP64 rows take 110 us so, 114 with the clock in this loop and 115 with
// the error word too.  2^27, whose constant is 4 bytes shorter, took 111: the loop
// is sensitive to where its instructions lie.)
constexpr int kTurnSpins = 120000000;
constexpr int kT = 256;
constexpr int kRunRows = 4096;     // rows of a tile of consecutive rows
constexpr int kBoxX = 128;         // cells of a box along x
constexpr int kBoxLines = 64;      // grid lines of a box

enum : int { M_PUB_LO = 1, M_PUB_UP = 2, M_OVF_LO = 4, M_OVF_UP = 8 };

// ---- the schedule ---------------------------------------------------------------
struct GridShape {
  int sy, sz;   // strides of y and z (sz = nm for a 2D grid)
  int ok;
};

// The grid behind the first nm rows, from the forward couplings of row 0 (a
// corner of the grid): offsets 1, sy and (3D) sz.
__global__ void k_grid_guess(int nm, const int* rp, const int* ci, GridShape* g) {
  int off[4], k = 0;
  for (int p = rp[0]; p < rp[1] && k < 4; ++p)
    if (ci[p] > 0 && ci[p] < nm) off[k++] = ci[p];
  GridShape s{0, 0, 0};
  if ((k == 2 || k == 3) && off[0] == 1) {
    s.sy = off[1];
    s.sz = k == 3 ? off[2] : nm;
    s.ok = s.sy > 1 && s.sz > s.sy && s.sz % s.sy == 0 && nm % s.sz == 0;
  }
  *g = s;
}

// Boxes are a valid order only if every coupling inside the first nm rows is
// componentwise: j < i needs x, y and z of j no larger than i's, j > i no
// smaller.
__global__ void k_grid_check(int nm, const int* rp, const int* ci, GridShape* g) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nm) return;
  const int sy = g->sy, sz = g->sz;
  if (sy < 2 || sz < sy) return;
  const int xi = i % sy, yi = i % sz / sy, zi = i / sz;
  bool bad = false;
  for (int p = rp[i]; p < rp[i + 1]; ++p) {
    const int j = ci[p];
    if (j == i || j >= nm) continue;
    const int dx = j % sy - xi, dy = j % sz / sy - yi, dz = j / sz - zi;
    bad |= j < i ? (dx > 0 || dy > 0 || dz > 0) : (dx < 0 || dy < 0 || dz < 0);
  }
  if (bad) g->ok = 0;
}

struct Boxes {
  int sy, sz, tx, ty, tz, ntx, nty;
};

__global__ void k_box_keys(int nm, Boxes b, int lb, int* key, int* row) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nm) return;
  const int x = i % b.sy, y = i % b.sz / b.sy, z = i / b.sz;
  const int tile = (z / b.tz * b.nty + y / b.ty) * b.ntx + x / b.tx;
  key[i] = tile << lb | (x % b.tx + y % b.ty + z % b.tz);
  row[i] = i;
}

// Levels of the rows [row0, n) by their couplings with each other (longest
// path over lower columns): a wavefront's rows wait for the levels of the
// rows they depend on, whose chunks were drawn earlier (value as ready flag:
// -1 = not known yet).  Every pass finishes a row or leaves it for the next
// one; bounded by the wall clock.
__global__ void __launch_bounds__(256)
k_run_levels(int row0, int n, const int* rp, const int* ci, int* lev, int* ticket, int* err,
             unsigned long long limit) {
  __shared__ int s_c;
  const int nchunks = (n - row0 + 255) / 256;
  while (true) {
    if (threadIdx.x == 0) s_c = atomicAdd(ticket, 1);
    __syncthreads();
    const int c = s_c;
    __syncthreads();
    if (c >= nchunks) break;
    const int i = row0 + c * 256 + static_cast<int>(threadIdx.x);
    bool done = i >= n;
    int p = done ? 0 : rp[i], L = 0;
    const unsigned long long t0 = wall_clock64();
    while (__any(!done)) {  // a vote, so that a finished lane publishes at once
      if (!done) {
        int j = ci[p];
        while (j < row0) j = ci[++p];
        while (j < i) {
          const int v = __hip_atomic_load(lev + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (v < 0) break;
          L = max(L, v + 1);
          j = ci[++p];
        }
        if (j >= i) {
          __hip_atomic_store(lev + i, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          done = true;
        } else if (wall_clock64() - t0 > limit ||
                   __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
          atomicOr(err, 2);
          done = true;
        }
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
}

// keys of rows in tiles of S consecutive rows.  A level that does not fit its
// bits, or an upper column without its mirror whose level is not higher (a
// pattern that is not symmetric), sets *bad: no schedule for both sweeps.  The
// tile of such a key stays right (level 0), as everything up to the host's
// look at *bad indexes by it; run_keys_on_host finds another order then.
__global__ void k_run_keys(int row0, int n, int S, int tile0, int lb, const int* rp, const int* ci,
                           const int* lev, int* key, int* row, int* bad) {
  const int i = row0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int L = lev[i];
  bool no = L < 0 || L >> lb != 0;
  for (int p = rp[i + 1] - 1; p >= rp[i] && ci[p] > i; --p) no |= lev[ci[p]] <= L;
  if (no) *bad = 1;
  key[i] = (tile0 + (i - row0) / S) << lb | (no ? 0 : L);
  row[i] = i;
}

// most dependencies of a row inside its phase (rows [row0, row1)), either sweep
__global__ void k_most_deps(int row0, int row1, const int* rp, const int* ci, int* most) {
  const int i = row0 + blockIdx.x * blockDim.x + threadIdx.x;
  int lo = 0, up = 0;
  if (i < row1)
    for (int p = rp[i]; p < rp[i + 1]; ++p) {
      const int j = ci[p];
      lo += j >= row0 && j < i;
      up += j > i && j < row1;
    }
  int m = max(lo, up);
  for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
  if (threadIdx.x % 64 == 0) atomicMax(most, m);
}

__global__ void k_tile_starts(int n, int ntiles, int lb, const int* key, const int* row, int* pos,
                              int* tstart) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int k = key[t] >> lb;
  if (t == 0 || key[t - 1] >> lb != k) tstart[k] = t;
  if (t == n - 1) tstart[ntiles] = n;
  pos[row[t]] = t;
}

// slices of a tile: runs of at most 64 positions of one level.  Counts
// (slice == null) or starts; one wavefront a tile.
__global__ void __launch_bounds__(64)
k_tile_slices(const int* tstart, const int* key, int* tslice, int* slice, int* maxs) {
  const int K = blockIdx.x, t0 = tstart[K], t1 = tstart[K + 1], lane = threadIdx.x;
  const unsigned long long upto = lane == 63 ? ~0ull : (2ull << lane) - 1;
  int base = slice ? tslice[K] : 0, carry = t0;
  for (int b = t0; b < t1; b += 256) {
    int k0[4], k1[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = min(b + 64 * u + lane, t1 - 1);
      k1[u] = key[t];
      k0[u] = key[max(t - 1, 0)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = b + 64 * u + lane;
      const unsigned long long m = __ballot(t < t1 && (t == t0 || k0[u] != k1[u]));
      const unsigned long long mine = m & upto;
      const int start = mine ? b + 64 * u + 63 - __builtin_clzll(mine) : carry;
      const bool first = t < t1 && (t - start) % 64 == 0;
      const unsigned long long f = __ballot(first);
      if (first && slice) slice[base + __popcll(f & upto) - 1] = t;
      base += __popcll(f);
      if (m) carry = b + 64 * u + 63 - __builtin_clzll(m);
    }
  }
  if (lane == 0 && !slice) {
    tslice[K] = base;
    atomicMax(maxs, base);
  }
}

// A position's dependencies inside its phase (rows [row0, row1)): the first C
// of the row's terms (at W places) as codes -- a row of the same tile as its index in the
// tile (the workgroup's LDS), a row of another tile as ~position, `pad` past
// the end -- and the flags of the row and of the rows it reads.
__global__ void k_tile_codes(int t0, int t1, int row0, int row1, int C, int W, int pad, int lb,
                             const int* key, const int* row, const int* pos, const int* tstart,
                             const int* rp, const int* ci, const int* diag, int* lcol, int* ucol,
                             int* meta, int* pre_list, int* pre_count) {
  const int t = t0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= t1) return;
  const int i = row[t], tile = key[t] >> lb, a = tstart[tile], b = tstart[tile + 1];
  const int d = diag[i], e = rp[i + 1];
  auto code = [&](int j, int mark) {
    const int q = pos[j];
    if (q >= a && q < b) return q - a;
    atomicOr(meta + q, mark);
    return ~q;
  };
  int* lc = lcol + static_cast<int64_t>(t - t0) * W;
  int* uc = ucol + static_cast<int64_t>(t - t0) * W;
  int k = 0, m = 0;
  for (int p = rp[i]; p < d; ++p) {
    if (ci[p] < row0) continue;
    const int c = code(ci[p], M_PUB_LO);
    if (k < C) lc[k++] = c;
    else m |= M_OVF_LO;
  }
  for (; k < W; ++k) lc[k] = pad;
  k = 0;
  bool pre = false;
  for (int p = e - 1; p > d; --p) {
    if (ci[p] >= row1) {
      pre = true;
      continue;
    }
    const int c = code(ci[p], M_PUB_UP);
    if (k < C) uc[k++] = c;
    else m |= M_OVF_UP;
  }
  for (; k < W; ++k) uc[k] = pad;
  if (m) atomicOr(meta + t, m);
  if (pre) pre_list[atomicAdd(pre_count, 1)] = i;
}

template <class T>
__global__ void k_tile_vals(int t0, int t1, int row0, int row1, int C, int W, const int* row,
                            const int* rp, const int* ci, const int* diag, const T* lu, T* lval,
                            T* uval, T* udiag) {
  const int t = t0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= t1) return;
  const int i = row[t], d = diag[i], e = rp[i + 1];
  T* lv = lval + static_cast<int64_t>(t - t0) * W;
  T* uv = uval + static_cast<int64_t>(t - t0) * W;
  int k = 0;
  for (int p = rp[i]; p < d && k < C; ++p)
    if (ci[p] >= row0) lv[k++] = lu[p];
  for (; k < W; ++k) lv[k] = T(0);
  k = 0;
  for (int p = e - 1; p > d && k < C; --p)
    if (ci[p] < row1) uv[k++] = lu[p];
  for (; k < W; ++k) uv[k] = T(0);
  udiag[t] = lu[d];
}

template <class T>
__global__ void k_arm(int64_t n, T* a, T* b) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  using U = typename Sentinel<T>::U;
  if (i < n) {
    reinterpret_cast<U*>(a)[i] = Sentinel<T>::bits;
    reinterpret_cast<U*>(b)[i] = Sentinel<T>::bits;
  }
}

// ---- the sweeps -----------------------------------------------------------------
template <class T>
__global__ void k_to_positions(int n, const int* pos, const T* b, T* X) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) X[pos[i]] = b[i];
}

template <class T>
__global__ void k_natural(int n, const int* pos, const T* X, T* x) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = X[pos[i]];
}

template <class T>
__global__ void k_sum_natural(int n, const int* pos, const T* X, const T* add, double* sum) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) sum[i] = static_cast<double>(add[i]) + static_cast<double>(X[pos[i]]);
}

// lower sweep, between the phases: the second phase's rows take their terms
// of the first phase's rows (ascending; the entries of a row come first)
template <class T>
__global__ void k_pre_lower(int t0, int t1, int row0, const int* row, const int* pos,
                            const int* rp, const int* ci, const T* lu, T* X) {
  const int t = t0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= t1) return;
  const int i = row[t];
  int p = rp[i];
  T s = X[t];
  for (int j; (j = ci[p]) < row0; ++p) s = fmadd(-lu[p], X[pos[j]], s);
  X[t] = s;
}

// upper sweep, between the phases: the first phase's rows with couplings to
// the second (listed) take those terms, descending
template <class T>
__global__ void k_pre_upper(int m, const int* list, int row1, const int* pos, const int* rp,
                            const int* ci, const T* lu, T* X) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  const int i = list[k], t = pos[i];
  int p = rp[i + 1] - 1;
  T s = X[t];
  for (int j; (j = ci[p]) >= row1; --p) s = fmadd(-lu[p], X[pos[j]], s);
  X[t] = s;
}

// a row in flight: its first C dependencies, held at W = 4 or 8 places
template <class T, int C>
struct Entry {
  static constexpr int W = C <= 4 ? 4 : 8;
  int t, meta;  // t < 0: no row
  int c[W];
  T v[W], in, dg;
  typename Sentinel<T>::U raw[C];
};

template <class T, int C>
__device__ __forceinline__ void load_row(const int* col, const T* val, Entry<T, C>& e) {
  constexpr int W = Entry<T, C>::W;
#pragma unroll
  for (int k = 0; k < W; k += 4) {
    const int4 c = reinterpret_cast<const int4*>(col)[k / 4];
    e.c[k] = c.x;
    e.c[k + 1] = c.y;
    e.c[k + 2] = c.z;
    e.c[k + 3] = c.w;
  }
  constexpr int Q = 16 / sizeof(T);
#pragma unroll
  for (int k = 0; k < W; k += Q) {
    const int4 u = reinterpret_cast<const int4*>(val)[k / Q];
    __builtin_memcpy(&e.v[k], &u, 16);
  }
}

// what a launch of one phase reads and writes
template <class T>
struct TileArgs {
  int tile0, ntiles, t0, t1, row0, row1, cap, n;
  const int *tslice, *slice, *col, *meta, *row, *pos, *rp, *ci, *diag;
  const T *val, *udiag, *lu;
  T *X, *H, *arm;
  int *ticket, *ticket_clear;
  int* err;
  unsigned long long limit;
};

// Terms beyond the C a position holds, from the CSR in the same order.
template <class T, int C, bool kUpper>
__device__ __forceinline__ T tile_overflow(const TileArgs<T>& a, const T* loc, int i, int tb, int te,
                                        T s) {
  int k = 0;
  const int d = a.diag[i], p0 = kUpper ? a.rp[i + 1] - 1 : a.rp[i];
  for (int p = p0; p != d; p += kUpper ? -1 : 1) {
    const int j = a.ci[p];
    if (kUpper ? j >= a.row1 : j < a.row0) continue;
    if (k++ < C) continue;
    const int q = a.pos[j];
    const T x = q >= tb && q < te ? loc[q - tb]
                                  : wait_ready<T, kLongTileWait>(a.H + q, load_raw<T>(a.H + q),
                                                                 a.err, a.limit);
    s = fmadd(-a.lu[p], x, s);
  }
  return s;
}

// A workgroup takes tiles by ticket in dependency order (the lowest
// unfinished tile always belongs to a running workgroup, so the waits end).
// Its wavefronts take groups of G of the tile's slices in turn: while a
// wavefront waits for its turn it has already read its slices' codes, factors
// and rows of other tiles, so a level's chain is the LDS reads of its
// dependencies, the multiply-adds and the LDS write; the turn word is read
// together with the first slice's dependencies (one round trip), and the
// global stores follow off the chain.  Dynamic LDS: the tile's values (cap +
// 2: a zero for the padding code and a spare), then its slice starts.
template <int C>
constexpr int kWaves = C <= 4 ? 8 : 16;
template <int C>
constexpr int kGroup = C <= 4 ? 2 : 1;

// keeps a value computed where it stands (the compiler would sink address
// arithmetic into the chain)
template <class V>
__device__ __forceinline__ void pin(V& v) {
  asm volatile("" : "+v"(v));
}

template <class T, int C, bool kUpper>
__global__ void __launch_bounds__(64 * kWaves<C>)
k_tile_sweep(TileArgs<T> a) {
  using U = typename Sentinel<T>::U;
  using E = Entry<T, C>;
  constexpr int W = E::W, G = kGroup<C>, NW = kWaves<C>;
  extern __shared__ double lds_raw[];
  __shared__ int s_tile, s_turn;
  T* loc = reinterpret_cast<T*>(lds_raw);
  int* sl = reinterpret_cast<int*>(loc + (a.cap + 3) / 2 * 2);
  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  if (blockIdx.x == 0 && threadIdx.x < 2) a.ticket_clear[threadIdx.x * kTicketStride] = 0;
  constexpr int kPub = kUpper ? M_PUB_UP : M_PUB_LO, kArm = kUpper ? M_PUB_LO : M_PUB_UP,
                kOvf = kUpper ? M_OVF_UP : M_OVF_LO;
  while (true) {
    if (threadIdx.x == 0) {
      s_tile = atomicAdd(a.ticket, 1);
      s_turn = 0;
      loc[a.cap] = T(0);
    }
    __syncthreads();
    const int c0 = __builtin_amdgcn_readfirstlane(s_tile);
    if (c0 >= a.ntiles) break;
    const int tile = a.tile0 + (kUpper ? a.ntiles - 1 - c0 : c0);
    const int s0 = a.tslice[tile], ns = a.tslice[tile + 1] - s0;
    for (int k = threadIdx.x; k <= ns; k += blockDim.x) sl[k] = a.slice[s0 + k];
    __syncthreads();
    const int tb = __builtin_amdgcn_readfirstlane(sl[0]);
    const int te = __builtin_amdgcn_readfirstlane(sl[ns]);
    auto fetch = [&](E& e, int k) {  // slice k of the walk (past the end: no row)
      const int q = kUpper ? max(ns - 1 - k, 0) : min(k, ns - 1);
      const int t = sl[q] + lane;
      e.t = k < ns && t < sl[q + 1] ? t : -1;
      const int u = min(t, a.t1 - 1);
      const int64_t o = static_cast<int64_t>(u - a.t0) * W;
      load_row<T, C>(a.col + o, a.val + o, e);
      e.in = a.X[u];
      e.meta = a.meta[u];
      if constexpr (kUpper) e.dg = a.udiag[u];
    };
    constexpr int S = sizeof(T);
    const auto outside = buffer_of(a.H, static_cast<int64_t>(a.n) * S);
    const auto own_h = buffer_of(a.H + tb, static_cast<int64_t>(te - tb) * S);
    const auto own_x = buffer_of(a.X + tb, static_cast<int64_t>(te - tb) * S);
    const auto own_arm = buffer_of(a.arm + tb, static_cast<int64_t>(te - tb) * S);
    // first read of a slice's rows of other tiles
    auto fetch_outside = [&](E& e) {
#pragma unroll
      for (int q = 0; q < C; ++q)
        e.raw[q] = buffer_get<U, kCoherent>(
            outside, e.c[q] < 0 ? static_cast<int>(static_cast<unsigned>(~e.c[q]) * S) : kNowhere);
    };
    E e[G], nx[G];
    const int ng = (ns + G - 1) / G;
#pragma unroll
    for (int g = 0; g < G; ++g) fetch(e[g], wave * G + g);
#pragma unroll
    for (int g = 0; g < G; ++g) fetch_outside(e[g]);
    for (int j = wave; j < ng; j += NW) {
#pragma unroll
      for (int g = 0; g < G; ++g) fetch(nx[g], (j + NW) * G + g);
      // LDS indices of the dependencies (rows of other tiles: the zero) and
      // of the row itself (no row: the spare)
      Quotient<T> quot[G];
      int idx[G][C], self[G];
      bool plain = false, over = false;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const bool on = e[g].t >= 0;
        if constexpr (kUpper) {
          quot[g].of(e[g].dg);
          plain |= on && quot[g].plain(e[g].in);
        }
        over |= on && (e[g].meta & kOvf);
#pragma unroll
        for (int q = 0; q < C; ++q) {
          idx[g][q] = on && e[g].c[q] >= 0 ? e[g].c[q] : a.cap;
          pin(idx[g][q]);
        }
        self[g] = on ? e[g].t - tb : a.cap + 1;
        pin(self[g]);
      }
      const bool any_plain = __any(plain), any_over = __any(over);
      auto missing = [&]() {
        bool m = false;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int q = 0; q < C; ++q)
            m |= e[g].t >= 0 && e[g].c[q] < 0 && e[g].raw[q] == Sentinel<T>::bits;
        return m;
      };
      // rows of other tiles that were not published yet at the first read
      if (__any(missing())) {
        const unsigned long long w0 = wall_clock64();
        bool gave_up = false;
        do {
#pragma unroll
          for (int g = 0; g < G; ++g)
#pragma unroll
            for (int q = 0; q < C; ++q)
              if (e[g].t >= 0 && e[g].c[q] < 0 && e[g].raw[q] == Sentinel<T>::bits)
                e[g].raw[q] = gave_up ? U(0) : load_raw<T>(a.H + ~e[g].c[q]);
          if (wall_clock64() - w0 > a.limit ||
              __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            gave_up = true;
            if (lane == 0) atomicOr(a.err, 2);
          }
        } while (__any(missing()));
        if (!gave_up && lane == 0 && wall_clock64() - w0 > (a.limit >> kLongTileWait))
          atomicAdd(a.err + 1, 1);
      }
      // the turn: groups 0 .. j - 1 done.  LDS accesses of a wavefront are in
      // order, so dependencies read after a turn word of j are final.
      wait_turn<true>(&s_turn, j - 1, a.err, a.limit);
      T lv[C], x[G];
      for (int spin = 1;; ++spin) {
        const int f = __hip_atomic_load(&s_turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < C; ++q) lv[q] = loc[idx[0][q]];
        asm volatile("" ::: "memory");
        if (__builtin_amdgcn_readfirstlane(f) >= j) break;
        if (spin == kTurnSpins) {  // a guard: that turn always comes
          atomicOr(a.err, 2);
          break;
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g > 0)
#pragma unroll
          for (int q = 0; q < C; ++q) lv[q] = loc[idx[g][q]];
        T s = e[g].in;
#pragma unroll
        for (int q = 0; q < C; ++q) {
          // one of the two is zero: LDS for rows of other tiles, the buffer
          // read for the tile's own
          U u;
          __builtin_memcpy(&u, &lv[q], S);
          u |= e[g].raw[q];
          __builtin_memcpy(&lv[q], &u, S);
          s = fmadd(-e[g].v[q], lv[q], s);
        }
        if (any_over && e[g].t >= 0 && (e[g].meta & kOvf))
          s = tile_overflow<T, C, kUpper>(a, loc, a.row[e[g].t], tb, te, s);
        if constexpr (kUpper) {
          T qv = quot[g](s, e[g].dg);
          if (any_plain) {
            asm volatile("" : "+v"(s));  // (a branch: not both and a select)
            qv = s / e[g].dg;
          }
          s = qv;
        }
        loc[self[g]] = s;
        x[g] = s;
        asm volatile("" ::: "memory");
      }
      __hip_atomic_store(&s_turn, j + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int g = 0; g < G; ++g) fetch_outside(nx[g]);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const bool on = e[g].t >= 0;
        const int own = (e[g].t - tb) * S;
        U u;
        __builtin_memcpy(&u, &x[g], S);
        if (u == Sentinel<T>::bits) u ^= 1;  // never publish the sentinel itself
        buffer_put<U, kCoherent>(own_h, on && (e[g].meta & kPub) ? own : kNowhere, u);
        buffer_put<T, 0>(own_x, on ? own : kNowhere, x[g]);
        buffer_put<U, 0>(own_arm, on && (e[g].meta & kArm) ? own : kNowhere, Sentinel<T>::bits);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) e[g] = nx[g];
    }
    __syncthreads();
  }
}

// Dependency levels of a whole triangle in the schedule's order, for their
// number (the longest chain).  A workgroup takes a tile by ticket and its
// wavefronts take slices in turn, each row waiting for its own dependencies:
// a level costs one published value's way through memory, and all tiles that
// the chain allows are under way.  (Workgroups that take rows in storage order
// hold eight planes of a 256 x 256 x 128 grid at a time, each as long as the
// whole chain: 24 ms a triangle, this form
// 3.2 ms.  Two wavefronts: eight poll so much that it takes 11 ms.)
constexpr int kLevelWaves = 2;

template <bool kUpper>
__global__ void __launch_bounds__(64 * kLevelWaves)
k_tile_levels(int ntiles, const int* slice, const int* tslice, const int* row, const int* rp,
              const int* ci, const int* diag, int* lev, int* top, int* ticket, int* err,
              unsigned long long limit) {
  constexpr int D = 8;  // dependencies read together
  __shared__ int s_c;
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  int most = 0;
  while (true) {
    if (threadIdx.x == 0) s_c = atomicAdd(ticket, 1);
    __syncthreads();
    const int c = s_c;
    __syncthreads();
    if (c >= ntiles) break;
    const int tile = kUpper ? ntiles - 1 - c : c;
    const int s0 = tslice[tile], ns = tslice[tile + 1] - s0;
    for (int k = wave; k < ns; k += kLevelWaves) {
      const int s = s0 + (kUpper ? ns - 1 - k : k);
      const int t = slice[s] + lane;
      const bool on = t < slice[s + 1];
      const int i = on ? row[t] : 0;
      const int p1 = on ? (kUpper ? rp[i + 1] : diag[i]) : 0;
      int p = on ? (kUpper ? diag[i] + 1 : rp[i]) : 0, L = 0;
      const unsigned long long t0 = wall_clock64();
      // D at a time; a wavefront vote ends the wait, so that no lane waits on
      // another one's way out of the loop
      while (__any(p < p1)) {
        int dep[D], v[D];
#pragma unroll
        for (int q = 0; q < D; ++q) {
          dep[q] = p + q < p1 ? ci[p + q] : -1;
          v[q] = dep[q] < 0 ? 0 : -1;
        }
        bool wait = true;
        while (__any(wait)) {
          wait = false;
#pragma unroll
          for (int q = 0; q < D; ++q)
            if (v[q] < 0)
              v[q] = __hip_atomic_load(lev + dep[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int q = 0; q < D; ++q) wait |= v[q] < 0;
          if (wait && (wall_clock64() - t0 > limit ||
                       __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
            atomicOr(err, 2);
            wait = false;
          }
          __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int q = 0; q < D; ++q)
          if (dep[q] >= 0) L = max(L, v[q] + 1);
        p += D;
      }
      if (on) __hip_atomic_store(lev + i, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      most = max(most, L);
    }
  }
  for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
  if (lane == 0) atomicMax(top, most);
}

// The keys of k_run_keys for any pattern, on the host: the longest path over
// the couplings of either triangle, in either direction, which increases along
// every coupling by itself; inside a tile its rank among the tile's levels, so
// that it fits where the level would not.  One pass over the rows' columns:
// lower ones are final when a row is reached, upper ones are pushed ahead.
// false: more ranks than the key has bits for.
bool run_keys_on_host(Handle* h, int row0, int S, int tile0, int lb, int* key) {
  const int m = h->n - row0;
  std::vector<int> rp(m + 1);
  HIPX(hipMemcpyAsync(rp.data(), h->rp.get() + row0, rp.size() * sizeof(int),
                      hipMemcpyDeviceToHost, h->stream));
  HIPX(hipStreamSynchronize(h->stream));
  const int p0 = rp[0];
  std::vector<int> ci(rp[m] - p0), lev(m, 0), out(m), ranks;
  HIPX(hipMemcpyAsync(ci.data(), h->ci.get() + p0, ci.size() * sizeof(int),
                      hipMemcpyDeviceToHost, h->stream));
  HIPX(hipStreamSynchronize(h->stream));
  for (int i = 0; i < m; ++i) {
    const int* c = ci.data() + (rp[i] - p0);
    const int* e = ci.data() + (rp[i + 1] - p0);
    int L = lev[i];
    for (const int* p = c; p < e; ++p)
      if (*p >= row0 && *p - row0 < i) L = std::max(L, lev[*p - row0] + 1);
    lev[i] = L;
    for (const int* p = c; p < e; ++p)
      if (*p - row0 > i) lev[*p - row0] = std::max(lev[*p - row0], L + 1);
  }
  for (int a = 0; a < m; a += S) {
    const int b = std::min(m, a + S);
    ranks.assign(lev.begin() + a, lev.begin() + b);
    std::sort(ranks.begin(), ranks.end());
    ranks.erase(std::unique(ranks.begin(), ranks.end()), ranks.end());
    if (ranks.size() > size_t(1) << lb) return false;
    for (int i = a; i < b; ++i)
      out[i] = (tile0 + a / S) << lb |
               static_cast<int>(std::lower_bound(ranks.begin(), ranks.end(), lev[i]) -
                                ranks.begin());
  }
  HIPX(hipMemcpyAsync(key + row0, out.data(), out.size() * sizeof(int), hipMemcpyHostToDevice,
                      h->stream));
  HIPX(hipStreamSynchronize(h->stream));
  return true;
}

}  // namespace

// Schedule of the sweeps (pattern only; kept by fams_update_values).  `cap`:
// most rows of a tile.
void build_tiles(Handle* h, int cap) {
  Allocator* A = &h->alloc;
  TileSched& S = h->tiles;
  const int n = h->n, nm = h->nm;
  S.clear();
  const double vec = n * (h->precision == FAMS_PREC_MIXED ? 4.0 : 8.0);
  if (vec >= 4294967296.0 - 512) return;  // buffer offsets of 32 bits: level-chunk sweeps
  // the grid behind the matrix rows
  GridShape g{0, 0, 0};
  if (nm >= 4) {
    DBuf<GridShape> d(A, 1);
    LAUNCH(h, "tiles", k_grid_guess, 1, 1, 0, nm, h->rp.get(), h->ci.get(), d.get());
    LAUNCH(h, "tiles", k_grid_check, blocks_for(nm, kT), kT, 0, nm, h->rp.get(), h->ci.get(),
           d.get());
    HIPX(hipMemcpyAsync(&g, d.get(), sizeof(g), hipMemcpyDeviceToHost, h->stream));
    HIPX(hipStreamSynchronize(h->stream));
  }
  Boxes b{};
  int nt = 0;
  if (g.ok) {
    const int nx = g.sy, ny = g.sz / g.sy, nz = nm / g.sz;
    // kBoxLines lines a box, near square; a shorter side gives its share away
    b.sy = g.sy;
    b.sz = g.sz;
    const int lines = std::max(1, std::min(kBoxLines, cap));
    int sq = 1;
    while ((sq + 1) * (sq + 1) <= lines) ++sq;
    b.tz = std::min(nz, ny < sq ? lines / ny : sq);
    b.ty = std::min(ny, lines / b.tz);
    const int most = std::max(1, std::min(kBoxX, cap / (b.ty * b.tz)));
    const int parts = (nx + most - 1) / most;
    b.tx = (nx + parts - 1) / parts;
    b.ntx = (nx + b.tx - 1) / b.tx;
    b.nty = (ny + b.ty - 1) / b.ty;
    nt = b.ntx * b.nty * ((nz + b.tz - 1) / b.tz);
    TilePhase p;
    p.row1 = nm;
    p.ntiles = nt;
    p.boxes = true;
    p.cap = b.tx * b.ty * b.tz;
    S.ph.push_back(p);
  }
  const int run = std::max(1, std::min(kRunRows, cap));
  if (!g.ok || nm < n) {
    TilePhase p;
    p.row0 = g.ok ? nm : 0;
    p.row1 = n;
    p.tile0 = nt;
    p.ntiles = (n - p.row0 + run - 1) / run;
    p.cap = std::min(run, n - p.row0);
    S.ph.push_back(p);
    nt += p.ntiles;
  }
  int tb = 1;
  while ((1 << tb) < nt) ++tb;
  const int lb = 31 - tb;  // level bits of a key
  S.row.reset(A, n);
  S.pos.reset(A, n);
  S.meta.reset(A, n);
  S.tslice.reset(A, nt + 1);
  DBuf<int> key(A, n), rows(A, n), keys(A, n), tstart(A, nt + 1), cnt(A, nt + 1), small(A, 8);
  HIPX(hipMemsetAsync(small, 0, 8 * sizeof(int), h->stream));
  int total = 0, hs[8] = {};
  for (TilePhase& p : S.ph) {
    if (p.boxes) {
      LAUNCH(h, "tiles", k_box_keys, blocks_for(nm, kT), kT, 0, nm, b, lb, key.get(), rows.get());
      continue;
    }
    const int m = p.row1 - p.row0;
    // levels into `keys` (sorted into later): -1 = not known yet
    HIPX(hipMemsetAsync(keys, 0xFF, n * sizeof(int), h->stream));
    LAUNCH(h, "tiles", k_run_levels, std::min((m + 255) / 256, 1024), 256, 0, p.row0, n,
           h->rp.get(), h->ci.get(), keys.get(), small.get() + 4, small.get() + 5, wait_limit(h));
    LAUNCH(h, "tiles", k_run_keys, blocks_for(m, kT), kT, 0, p.row0, n, run, p.tile0, lb,
           h->rp.get(), h->ci.get(), keys.get(), key.get(), rows.get(), small.get() + 6);
  }
  auto order = [&]() {  // positions, tiles and slices of the keys
    sort_pairs_i32(h, key, keys, rows, S.row, n, 31);
    LAUNCH(h, "tiles", k_tile_starts, blocks_for(n, kT), kT, 0, n, nt, lb, keys.get(), S.row.get(),
           S.pos.get(), tstart.get());
    // slices: counts per tile, then starts; maxima per phase
    HIPX(hipMemsetAsync(cnt, 0, (nt + 1) * sizeof(int), h->stream));
    for (size_t k = 0; k < S.ph.size(); ++k) {
      TilePhase& p = S.ph[k];
      LAUNCH(h, "tiles", k_tile_slices, p.ntiles, 64, 0, tstart.get() + p.tile0, keys.get(),
             cnt.get() + p.tile0, static_cast<int*>(nullptr), small.get() + k);
      LAUNCH(h, "tiles", k_most_deps, blocks_for(p.row1 - p.row0, kT), kT, 0, p.row0, p.row1,
             h->rp.get(), h->ci.get(), small.get() + 2 + k);
    }
    exclusive_scan_i32(h, cnt, S.tslice, nt + 1);
    HIPX(hipMemcpyAsync(&total, S.tslice.get() + nt, sizeof(int), hipMemcpyDeviceToHost,
                        h->stream));
    HIPX(hipMemcpyAsync(hs, small.get(), sizeof(hs), hipMemcpyDeviceToHost, h->stream));
    HIPX(hipStreamSynchronize(h->stream));
  };
  order();
  FAMS_REQUIRE(hs[5] == 0, FAMS_ERR_DEVICE, "ILU level computation did not complete");
  if (hs[6]) {
    // The device's levels are no order for both sweeps.  (60 x 50 x 30 cells
    // and 30 plates in FP64, 7% more couplings stored on one side: a two-stage step
    // takes 2000 us by level chunks and 377 us by the tiles of this order; the
    // setup, with its LU local solves, 136.5 and 140.1 ms.)
    const TilePhase& p = S.ph.back();
    if (!run_keys_on_host(h, p.row0, run, p.tile0, lb, key.get())) {
      S.clear();
      return;
    }
    HIPX(hipMemsetAsync(small, 0, 8 * sizeof(int), h->stream));
    order();
  }
  S.slices = total;
  S.slice.reset(A, total + 1);
  HIPX(hipMemcpyAsync(S.slice.get() + total, tstart.get() + nt, sizeof(int),
                      hipMemcpyDeviceToDevice, h->stream));
  DBuf<int> list(A, n);
  size_t codes = 0;
  for (size_t k = 0; k < S.ph.size(); ++k) {
    TilePhase& p = S.ph[k];
    p.max_slices = hs[k];
    LAUNCH(h, "tiles", k_tile_slices, p.ntiles, 64, 0, tstart.get() + p.tile0, keys.get(),
           S.tslice.get() + p.tile0, S.slice.get(), static_cast<int*>(nullptr));
    // a grid row has three dependencies, a fracture row rarely more than four;
    // beyond eight they come from the CSR, a memory round trip each
    p.C = hs[2 + k] <= 3 ? 3 : hs[2 + k] <= 4 ? 4 : 8;
    p.W = p.C <= 4 ? 4 : 8;
    p.over = hs[2 + k] > p.C;
    p.code0 = codes;
    codes += static_cast<size_t>(p.row1 - p.row0) * p.W;
  }
  S.lcol.reset(A, codes);
  S.ucol.reset(A, codes);
  HIPX(hipMemsetAsync(S.meta, 0, n * sizeof(int), h->stream));
  for (const TilePhase& p : S.ph)
    LAUNCH(h, "tiles", k_tile_codes, blocks_for(p.row1 - p.row0, kT), kT, 0, p.row0, p.row1,
           p.row0, p.row1, p.C, p.W, p.cap, lb, keys.get(), S.row.get(), S.pos.get(), tstart.get(),
           h->rp.get(), h->ci.get(), h->diag.get(), S.lcol.get() + p.code0,
           S.ucol.get() + p.code0, S.meta.get(), list.get(), small.get() + 7);
  HIPX(hipMemcpyAsync(&S.npre, small.get() + 7, sizeof(int), hipMemcpyDeviceToHost, h->stream));
  HIPX(hipStreamSynchronize(h->stream));
  if (S.npre) {
    S.pre.reset(A, S.npre);
    HIPX(hipMemcpyAsync(S.pre, list.get(), S.npre * sizeof(int), hipMemcpyDeviceToDevice,
                        h->stream));
  }
  S.ticket.reset(A, 4 * kTicketStride);
  // what the sweeps keep between launches, allocated now so that applying the
  // smoother allocates nothing
  auto state = [&](TileState& v, size_t s) {
    v.lval.reset(A, codes * s);
    v.uval.reset(A, codes * s);
    v.udiag.reset(A, n * s);
    v.x.reset(A, n * s);
    v.hl.reset(A, n * s);
    v.hu.reset(A, n * s);
  };
  state(S.st, h->precision == FAMS_PREC_MIXED ? sizeof(float) : sizeof(double));
  S.armed = false;
  HIPX(hipStreamSynchronize(h->stream));
}

// levels of the lower and the upper triangle
void tile_level_counts(Handle* h, int out[2]) {
  const TileSched& S = h->tiles;
  const int n = h->n;
  int nt = 0;
  for (const TilePhase& p : S.ph) nt += p.ntiles;
  DBuf<int> lev(&h->alloc, 2 * static_cast<size_t>(n)), small(&h->alloc, 6);
  HIPX(hipMemsetAsync(lev, 0xFF, 2 * static_cast<size_t>(n) * sizeof(int), h->stream));
  HIPX(hipMemsetAsync(small, 0, 6 * sizeof(int), h->stream));  // a triangle: top, ticket, error
  {
    Fork fork(h);
    hipStream_t s0 = fork.next(), s1 = fork.next();
    LAUNCH_ON(h, s0, "ilu_levels", k_tile_levels<false>, std::min(nt, 1024), 64 * kLevelWaves, 0, nt,
              S.slice.get(), S.tslice.get(), S.row.get(), h->rp.get(), h->ci.get(), h->diag.get(),
              lev.get(), small.get(), small.get() + 1, small.get() + 2, wait_limit(h));
    LAUNCH_ON(h, s1, "ilu_levels", k_tile_levels<true>, std::min(nt, 1024), 64 * kLevelWaves, 0, nt,
              S.slice.get(), S.tslice.get(), S.row.get(), h->rp.get(), h->ci.get(), h->diag.get(),
              lev.get() + n, small.get() + 3, small.get() + 4, small.get() + 5, wait_limit(h));
    fork.join();
  }
  int hs[6] = {};
  HIPX(hipMemcpyAsync(hs, small.get(), sizeof(hs), hipMemcpyDeviceToHost, h->stream));
  HIPX(hipStreamSynchronize(h->stream));
  FAMS_REQUIRE(hs[2] == 0 && hs[5] == 0, FAMS_ERR_DEVICE, "ILU level computation did not complete");
  out[0] = hs[0] + 1;
  out[1] = hs[3] + 1;
}

// the factors in the schedule's order
template <class T>
void tile_values(Handle* h, const T* lu) {
  TileSched& S = h->tiles;
  for (const TilePhase& p : S.ph)
    LAUNCH(h, "tiles", k_tile_vals<T>, blocks_for(p.row1 - p.row0, kT), kT, 0, p.row0, p.row1,
           p.row0, p.row1, p.C, p.W, S.row.get(), h->rp.get(), h->ci.get(), h->diag.get(), lu,
           S.st.lval.as<T>() + p.code0, S.st.uval.as<T>() + p.code0, S.st.udiag.as<T>());
}

// x = U^{-1} L^{-1} b in natural order (b null: already in the schedule's
// order in tiles.st.x); or with `sum` only sum = add + x in FP64
template <class T>
void tile_apply(Handle* h, const T* lu, const T* b, T* x, const T* add, double* sum) {
  TileSched& S = h->tiles;
  const int n = h->n;
  T* X = S.st.x.as<T>();
  T* HL = S.st.hl.as<T>();
  T* HU = S.st.hu.as<T>();
  if (!S.armed) {  // first use, or an application that did not come to its end
    LAUNCH(h, "ilu_arm", k_arm<T>, blocks_for(n, kT), kT, 0, (int64_t)n, HL, HU);
    HIPX(hipMemsetAsync(S.ticket, 0, 4 * kTicketStride * sizeof(int), h->stream));
  }
  S.armed = false;  // until every launch is queued: the sweeps arm for each other
  if (b) LAUNCH(h, "ilu_gather", k_to_positions<T>, blocks_for(n, kT), kT, 0, n, S.pos.get(), b, X);
  const unsigned long long limit = wait_limit(h);
  const bool two = S.ph.size() == 2;
  auto sweep = [&](int k, bool upper) {
    const TilePhase& p = S.ph[k];
    TileArgs<T> a{};
    a.tile0 = p.tile0;
    a.ntiles = p.ntiles;
    a.t0 = a.row0 = p.row0;
    a.t1 = a.row1 = p.row1;
    a.cap = p.cap;
    a.n = n;
    a.tslice = S.tslice.get();
    a.slice = S.slice.get();
    a.col = (upper ? S.ucol : S.lcol).get() + p.code0;
    a.val = (upper ? S.st.uval : S.st.lval).as<T>() + p.code0;
    a.udiag = S.st.udiag.as<T>();
    a.lu = lu;
    a.meta = S.meta.get();
    a.row = S.row.get();
    a.pos = S.pos.get();
    a.rp = h->rp.get();
    a.ci = h->ci.get();
    a.diag = h->diag.get();
    a.X = X;
    a.H = upper ? HU : HL;
    a.arm = upper ? HL : HU;
    a.ticket = S.ticket.get() + (upper ? 2 + k : k) * kTicketStride;
    a.ticket_clear = S.ticket.get() + (upper ? 0 : 2) * kTicketStride;
    a.err = h->sweep_err.get();
    a.limit = limit;
    const size_t lds = static_cast<size_t>((p.cap + 3) / 2 * 2) * sizeof(T) +
                       static_cast<size_t>(p.max_slices + 1) * sizeof(int);
    FAMS_REQUIRE(lds <= static_cast<size_t>(lds_hw_budget(h)), FAMS_ERR_CAPACITY,
                 "ILU tile does not fit in LDS");
    const int groups = std::min(p.ntiles, 2048);
#define FAMS_TILE(C)                                                                     \
  do {                                                                                   \
    if (upper) {                                                                         \
      allow_lds(reinterpret_cast<const void*>(&k_tile_sweep<T, C, true>), lds);          \
      LAUNCH(h, "ilu_upper", (k_tile_sweep<T, C, true>), groups, 64 * kWaves<C>, lds, a); \
    } else {                                                                             \
      allow_lds(reinterpret_cast<const void*>(&k_tile_sweep<T, C, false>), lds);         \
      LAUNCH(h, "ilu_lower", (k_tile_sweep<T, C, false>), groups, 64 * kWaves<C>, lds, a); \
    }                                                                                    \
  } while (0)
    switch (p.C) {
      case 3: FAMS_TILE(3); break;
      case 4: FAMS_TILE(4); break;
      default: FAMS_TILE(8); break;
    }
#undef FAMS_TILE
  };
  sweep(0, false);
  if (two) {
    const TilePhase& p = S.ph[1];
    LAUNCH(h, "ilu_pre", k_pre_lower<T>, blocks_for(p.row1 - p.row0, kT), kT, 0, p.row0, p.row1,
           p.row0, S.row.get(), S.pos.get(), h->rp.get(), h->ci.get(), lu, X);
    sweep(1, false);
    sweep(1, true);
    if (S.npre)
      LAUNCH(h, "ilu_pre", k_pre_upper<T>, blocks_for(S.npre, kT), kT, 0, S.npre, S.pre.get(),
             S.ph[0].row1, S.pos.get(), h->rp.get(), h->ci.get(), lu, X);
  }
  sweep(0, true);
  S.armed = true;
  // back to natural order in a pass of its own: the sweep's rows of a level
  // lie on as many cache lines, and its scattered stores cost more than this
  // pass (upper sweep of the 9.4M-row FP32 system: 567 against 334 us)
  if (sum)
    LAUNCH(h, "ilu_sum", k_sum_natural<T>, blocks_for(n, kT), kT, 0, n, S.pos.get(), X, add, sum);
  else
    LAUNCH(h, "ilu_sum", k_natural<T>, blocks_for(n, kT), kT, 0, n, S.pos.get(), X, x);
}

template void tile_values<double>(Handle*, const double*);
template void tile_values<float>(Handle*, const float*);
template void tile_apply<double>(Handle*, const double*, const double*, double*, const double*,
                                 double*);
template void tile_apply<float>(Handle*, const float*, const float*, float*, const float*, double*);

}  // namespace fams
