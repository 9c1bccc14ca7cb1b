// ILU(0) sweeps by tiles for K right-hand sides in lock-step (x[i K + r]):
// the tiles, levels and phases of tiles.hip.
//
// What bounds these sweeps is again the chain of levels, with the memory
// transactions behind it: a row's K values are one contiguous stretch, and a
// lane takes 16 bytes of it, so a wavefront's accesses cover whole stretches
// (a lane per row holding several right-hand sides ran the grid rows of the
// wide groups at half this rate).  A slice (<= 64 rows of one level) is shared
// by a team of wavefronts; teams take a tile's slices in turn as in tiles.hip,
// and a level's chain is one LDS round trip, the multiply-adds and the LDS
// write.  LDS holds the values of the last kRing slices; a row's dependencies
// are read from there, and from a compact array of published values when they
// lie in another tile or further back.  Only published rows (about a quarter)
// are armed and published, and the upper sweep of the first phase writes the
// two-stage sum in place of x.
//
// One application (both sweeps, all phases), this form against the dataflow
// over level chunks: 50.7k grid rows K = 4 FP32 82 against 515 us; 2.1M grid rows
// and their fracture rows K = 16 FP64 1390 against 2610 us, K = 32 FP32 1900
// against 2840 us.  The grid rows then move 0.9 to 2.0 GB at 1.0 to 1.4 TB/s;
// a workgroup with a barrier a slice instead of turns took 1305 for 1077 us.
#include <algorithm>
#include <cstdlib>
#include <type_traits>
#include <vector>

#include "internal.hpp"
#include "ready.hpp"

namespace fams {
namespace {

constexpr int kT = 256;
constexpr int kRing = 8;     // slices whose values LDS holds
constexpr int kZeroRow = kRing * 64;  // a row of zeros after them: the padding code

// A row's record: W codes, W factors, the row (and kMore: terms beyond the
// record's), the slots it publishes to in the lower and the upper sweep (-1:
// none) and the diagonal of U.
constexpr int kMore = 1 << 30;
template <class T, int W> struct Rec;
template <> struct Rec<float, 4> {
  int c[4];
  float v[4];
  int row, lo, up;
  float dg;
};
template <> struct Rec<float, 8> {
  int c[8];
  float v[8];
  int row, lo, up;
  float dg;
};
template <> struct Rec<double, 4> {
  int c[4];
  double v[4];
  int row, lo, up, pad;
  double dg, pad2;
};
template <> struct Rec<double, 8> {
  int c[8];
  double v[8];
  int row, lo, up, pad;
  double dg, pad2;
};
static_assert(sizeof(Rec<float, 4>) == 48 && sizeof(Rec<double, 4>) == 80 &&
              sizeof(Rec<float, 8>) == 80 && sizeof(Rec<double, 8>) == 128, "record sizes");

// ---- the schedule ---------------------------------------------------------------
// number (inside its tile) of the slice of every position; one wavefront a tile
__global__ void __launch_bounds__(64)
k_slice_numbers(const int* tslice, const int* slice, int* sno, int* tile_of) {
  const int K = blockIdx.x, s0 = tslice[K], s1 = tslice[K + 1];
  for (int s = s0; s < s1; ++s) {
    const int t = slice[s] + threadIdx.x;
    if (t < slice[s + 1]) {
      sno[t] = s - s0;
      tile_of[t] = K;
    }
  }
}

// The k-th dependency of position t's row inside its phase, from position q:
// held in LDS when it is one of the first C, of the same tile and at most
// kRing - 1 slices away; else its row is published (mark[q] = 1).
struct Near {
  const int *sno, *tile_of;
  __device__ bool operator()(int t, int q, int k, int C) const {
    return k < C && tile_of[t] == tile_of[q] && abs(sno[t] - sno[q]) < kRing;
  }
};

__global__ void k_bmarks(int t0, int t1, int row0, int row1, int C, const int* row, const int* pos,
                         const int* rp, const int* ci, const int* diag, Near near, int* lo,
                         int* up) {
  const int t = t0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= t1) return;
  const int i = row[t], d = diag[i], e = rp[i + 1];
  int k = 0;
  for (int p = rp[i]; p < d; ++p)
    if (ci[p] >= row0) {
      const int q = pos[ci[p]];
      if (!near(t, q, k++, C)) lo[q] = 1;
    }
  k = 0;
  for (int p = e - 1; p > d; --p)
    if (ci[p] < row1) {
      const int q = pos[ci[p]];
      if (!near(t, q, k++, C)) up[q] = 1;
    }
}

// slots: the marks' running count where marked, else -1
__global__ void k_bslots(int n, const int* mark, const int* scan, int* slot) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) slot[t] = mark[t] ? scan[t] : -1;
}

template <class T, int W>
__global__ void k_brecords(int t0, int t1, int row0, int row1, int C, const int* row,
                           const int* pos, const int* rp, const int* ci, const int* diag,
                           const int* slice, const int* tslice, Near near, const int* lo,
                           const int* up, const T* lu, Rec<T, W>* RL, Rec<T, W>* RU) {
  const int t = t0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= t1) return;
  const int i = row[t], d = diag[i], e = rp[i + 1];
  auto code = [&](int q, int k, const int* slot) {
    if (!near(t, q, k, C)) return ~slot[q];
    const int s = near.sno[q];
    return (s % kRing) * 64 + q - slice[tslice[near.tile_of[q]] + s];
  };
  Rec<T, W> r{};
  r.row = i;
  r.lo = lo[t];
  r.up = up[t];
  r.dg = lu[d];
  auto pad = [&](int k) {
    for (; k < W; ++k) {
      r.c[k] = kZeroRow;
      r.v[k] = T(0);
    }
  };
  int k = 0;
  for (int p = rp[i]; p < d; ++p)
    if (ci[p] >= row0) {
      if (k == C) {
        r.row |= kMore;
        break;
      }
      r.c[k] = code(pos[ci[p]], k, lo);
      r.v[k++] = lu[p];
    }
  pad(k);
  RL[t - t0] = r;
  r.row = i;
  k = 0;
  for (int p = e - 1; p > d; --p)
    if (ci[p] < row1) {
      if (k == C) {
        r.row |= kMore;
        break;
      }
      r.c[k] = code(pos[ci[p]], k, up);
      r.v[k++] = lu[p];
    }
  pad(k);
  RU[t - t0] = r;
}

template <class T>
__global__ void k_barm(int64_t n, T* a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  using U = typename Sentinel<T>::U;
  if (i < n) reinterpret_cast<U*>(a)[i] = Sentinel<T>::bits;
}

// ---- between the phases (see tiles.hip) -------------------------------------------
// (the second phase's lower sweep then works in y in place)
template <class T, int K>
__global__ void k_bpre_lower(int row0, int n, const int* rp, const int* ci, const T* lu,
                             const T* b, T* y) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t i = row0 + e / K;
  if (i >= n) return;
  const int r = static_cast<int>(e % K);
  int p = rp[i];
  T s = b[i * K + r];
  for (int j; (j = ci[p]) < row0; ++p) s = fmadd(-lu[p], y[static_cast<int64_t>(j) * K + r], s);
  y[i * K + r] = s;
}

template <class T, int K>
__global__ void k_bpre_upper(int m, const int* list, int row1, const int* rp, const int* ci,
                             const T* lu, const T* x, T* y) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= static_cast<int64_t>(m) * K) return;
  const int64_t i = list[e / K];
  const int r = static_cast<int>(e % K);
  int p = rp[i + 1] - 1;
  T s = y[i * K + r];
  for (int j; (j = ci[p]) >= row1; --p) s = fmadd(-lu[p], x[static_cast<int64_t>(j) * K + r], s);
  y[i * K + r] = s;
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// ---- the sweeps -----------------------------------------------------------------
template <class T>
struct BTileArgs {
  int tile0, ntiles, t0, t1, row0, row1, n, K;  // K: stride of the published rows
  int C;                     // dependencies in a record
  const int *tslice, *slice, *pos, *rp, *ci, *diag, *slot;
  const void* rec;           // the phase's records
  const T* lu;
  const T* in;
  T* out;                    // null: not written
  const T* add;              // upper: with sum, sum = add + x
  double* sum;
  T *H, *arm;                // published values of this sweep and of the other one
  int64_t hbytes, abytes;
  int *ticket, *ticket_clear;
  int* err;
  unsigned long long limit;
};

// A workgroup works on KG of the K right-hand sides, a lane on 16 bytes of a
// row's.  Pieces of 64 bytes a row for boxes of a grid and of 32 bytes where
// rows have more dependencies (phases of few rows, bound by the chain: four
// wavefronts a slice leave few slices read ahead).  Lower and upper sweep of
// 2.07M grid rows, K = 16 FP64, with pieces of 32 / 64 / 128 bytes: 1540 / 1077
// / 1064 us; K = 32 FP32: 1940 / 1478 / 1526 us; of the same systems' fracture
// rows with pieces of 16 / 32 / 64 bytes: 362 / 301 / 386 us, 551 / 421 / 543 us.
// Vectors beyond the last-level cache (256 MB) take pieces twice as wide (kWide):
// half a line would be read again from memory by another workgroup.  Both sweeps,
// all phases, with 64 and 32 / 128 and 32 / 128 and 64 bytes: 9.4M rows FP64 K =
// 16 (1.2 GB a vector) 6096 / 5398 / 5266 us, K = 32 10507 / 9304 / 8909 (level
// chunks 5181 and 8740); FP32 K = 32 (1.2 GB) 5785 / 5504 / 5479; 2.1M rows FP64
// K = 32 (0.54 GB) 3166 / 2964 / 3122 (chunks 3053), FP32 K = 32 (0.27 GB) 1990 /
// 2088 / 2206: from 0.5 GB on for boxes, from 1 GB for runs.
template <class T, int K, int C, bool kWide>
struct Lanes {
  static constexpr int KG =
      std::min(K, (C > 3 ? 32 : 64) * (kWide ? 2 : 1) / static_cast<int>(sizeof(T)));
  static constexpr int N = std::min(K, 16 / static_cast<int>(sizeof(T)));  // values a lane
  static constexpr int per_row = KG / N;
  static constexpr int rows = 64 / per_row;  // of one access
};
template <class T, int K>
constexpr bool kCanWiden = K * sizeof(T) >= 128;
constexpr int kWaves = 16;

// N values at a byte offset of a buffer (past the end: zero, dropped)
template <class T, int N, int kPolicy>
__device__ __forceinline__ void vec_get(__amdgpu_buffer_rsrc_t r, int off, T (&v)[N]) {
  constexpr int B = N * sizeof(T);
  if constexpr (B == 8) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kPolicy);
    __builtin_memcpy(v, &w, 8);
  } else {
    static_assert(B == 16, "a lane's values");
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kPolicy);
    __builtin_memcpy(v, &w, 16);
  }
}

template <class T, int N, int kPolicy>
__device__ __forceinline__ void vec_put(__amdgpu_buffer_rsrc_t r, int off, const T (&v)[N]) {
  constexpr int B = N * sizeof(T);
  if constexpr (B == 8) {
    u32x2 w;
    __builtin_memcpy(&w, v, 8);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, off, 0, kPolicy);
  } else {
#pragma unroll
    for (int b = 0; b < B; b += 16) {
      u32x4 w;
      __builtin_memcpy(&w, reinterpret_cast<const char*>(v) + b, 16);
      __builtin_amdgcn_raw_buffer_store_b128(w, r, off + b, 0, kPolicy);
    }
  }
}

// terms beyond the record's, from the CSR in the same order (published rows);
// r: the first of the lane's right-hand sides
template <class T, int N, bool kUpper>
__device__ __forceinline__ void btile_overflow(const BTileArgs<T>& a, int i, int r, T (&s)[N]) {
  int k = 0;
  const int d = a.diag[i], p0 = kUpper ? a.rp[i + 1] - 1 : a.rp[i];
  for (int p = p0; p != d; p += kUpper ? -1 : 1) {
    const int j = a.ci[p];
    if (kUpper ? j >= a.row1 : j < a.row0) continue;
    if (k++ < a.C) continue;
    const T* h = a.H + static_cast<int64_t>(a.slot[a.pos[j]]) * a.K + r;
#pragma unroll
    for (int v = 0; v < N; ++v)
      s[v] = fmadd(-a.lu[p],
                   wait_ready<T, kLongTileWait>(h + v, load_raw<T>(h + v), a.err, a.limit), s[v]);
  }
}

// A workgroup takes tiles by ticket in dependency order.
template <class T, int K, int C, bool kUpper, bool kOver, bool kWide>
__global__ void __launch_bounds__(64 * kWaves)
k_btile_sweep(BTileArgs<T> a) {
  using U = typename Sentinel<T>::U;
  using L = Lanes<T, K, C, kWide>;
  constexpr int W = C <= 4 ? 4 : 8, S = sizeof(T), N = L::N, KG = L::KG, kGroups = K / KG;
  constexpr int kTeam = 64 / L::rows, kTeams = kWaves / kTeam;
  using R = Rec<T, W>;
  extern __shared__ __align__(16) char lds_raw[];
  __shared__ int s_tile, s_turn;
  T* val = reinterpret_cast<T*>(lds_raw);  // rows of KG: the ring, zeros
  int* sl = reinterpret_cast<int*>(val + (kZeroRow + 1) * KG);
  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int team = wave / kTeam;
  const int rl = lane % L::per_row * N;  // first right-hand side of the group's
  int r = rl;
  const int p = wave % kTeam * L::rows + lane / L::per_row;  // row of the slice
  if (blockIdx.x == 0 && threadIdx.x < 2) a.ticket_clear[threadIdx.x * kTicketStride] = 0;
  const int64_t vbytes = static_cast<int64_t>(a.n) * K * S;
  const auto b_in = buffer_of(a.in, vbytes);
  const auto b_out = buffer_of(a.out, a.out ? vbytes : 0);
  const auto b_add = buffer_of(a.add, a.sum ? vbytes : 0);
  const auto b_sum = buffer_of(a.sum, a.sum ? static_cast<int64_t>(a.n) * K * 8 : 0);
  const auto b_h = buffer_of(a.H, a.hbytes);
  const auto b_arm = buffer_of(a.arm, a.abytes);
  auto at = [&r](int i, int size) {  // byte offset of (row or slot i, r)
    return static_cast<int>((static_cast<unsigned>(i) * K + r) * size);
  };
  if (threadIdx.x < KG) val[kZeroRow * KG + threadIdx.x] = T(0);
  while (true) {
    if (threadIdx.x == 0) {
      s_tile = atomicAdd(a.ticket, 1);
      s_turn = 0;
    }
    __syncthreads();
    const int c1 = __builtin_amdgcn_readfirstlane(s_tile), c0 = c1 / kGroups;
    if (c0 >= a.ntiles) break;
    r = rl + c1 % kGroups * KG;
    const int tile = a.tile0 + (kUpper ? a.ntiles - 1 - c0 : c0);
    const int s0 = a.tslice[tile], ns = a.tslice[tile + 1] - s0;
    for (int k = threadIdx.x; k <= ns; k += blockDim.x) sl[k] = a.slice[s0 + k];
    __syncthreads();
    struct X {  // a row's record
      int c[C], row, lo, up;
      T v[C], dg;
      bool on;
    };
    auto rec_load = [&](X& x, int k) {  // slice k of the walk (past the end: no row)
      const int q = kUpper ? max(ns - 1 - k, 0) : min(k, ns - 1);
      const int t = sl[q] + p;
      x.on = (t < sl[q + 1]) & (k < ns);
      const R& y = reinterpret_cast<const R*>(a.rec)[min(t, a.t1 - 1) - a.t0];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        x.c[j] = y.c[j];
        x.v[j] = y.v[j];
      }
      x.row = y.row;
      x.lo = y.lo;
      x.up = y.up;
      if constexpr (kUpper) x.dg = y.dg;
    };
    struct E {
      T in[N], add[N];
      T raw[C][N];
    };
    auto read_published = [&](E& e, const X& x, bool on) {
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const int off = at(~x.c[j], S);
        vec_get<T, N, kCoherent>(b_h, (on & (x.c[j] < 0)) ? off : kNowhere, e.raw[j]);
      }
    };
    auto vec_load = [&](E& e, const X& x) {
      read_published(e, x, x.on);
      const int off = at(x.row & (kMore - 1), S);
      vec_get<T, N, 0>(b_in, x.on ? off : kNowhere, e.in);
      if constexpr (kUpper) vec_get<T, N, 0>(b_add, x.on ? off : kNowhere, e.add);
    };
    X x, nx;
    E e;
    rec_load(x, team);
    vec_load(e, x);
    for (int k = team; k < ns; k += kTeams) {
      rec_load(nx, k + kTeams);
      const int slot = kUpper ? ns - 1 - k : k;
      int idx[C], self = (slot % kRing * 64 + p) * KG + rl;
      asm volatile("" : "+v"(self));
#pragma unroll
      for (int j = 0; j < C; ++j) {
        idx[j] = (x.c[j] < 0 ? kZeroRow : x.c[j]) * KG + rl;
        asm volatile("" : "+v"(idx[j]));
      }
      Quotient<T> quot;
      if constexpr (kUpper) quot.of(x.dg);
      bool plain = false;
      if constexpr (kUpper)
#pragma unroll
        for (int g = 0; g < N; ++g) plain |= x.on && quot.plain(e.in[g]);
      const bool any_plain = kUpper && __any(plain);
      const bool any_more = kOver && __any(x.on && (x.row & kMore));
      // published values that were not there at the first read (zero where
      // nothing was read)
      auto missing = [&]() {
        bool m = false;
#pragma unroll
        for (int j = 0; j < C; ++j)
#pragma unroll
          for (int g = 0; g < N; ++g) {
            U u;
            __builtin_memcpy(&u, &e.raw[j][g], S);
            m |= u == Sentinel<T>::bits;
          }
        return m;
      };
      if (__any(missing())) {
        const unsigned long long t0 = wall_clock64();
        bool gave_up = false;
        do {
          read_published(e, x, x.on & !gave_up);
          asm volatile("" ::: "memory");  // the next pass reads again
          if (wall_clock64() - t0 > a.limit ||
              __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            gave_up = true;
            if (lane == 0) atomicOr(a.err, 2);
          }
        } while (__any(missing()));
        if (!gave_up && lane == 0 && wall_clock64() - t0 > (a.limit >> kLongTileWait))
          atomicAdd(a.err + 1, 1);
      }
      // the turn: the teams' wavefronts have done slices 0 .. k - 1 (LDS
      // accesses of a wavefront are in order, so dependencies read after that
      // turn word are final)
      wait_turn<true>(&s_turn, (k - 1) * kTeam, a.err, a.limit);
      wait_turn<false>(&s_turn, k * kTeam, a.err, a.limit);
      asm volatile("" ::: "memory");
      T lv[C][N], s[N];
#pragma unroll
      for (int j = 0; j < C; ++j)
        __builtin_memcpy(lv[j], __builtin_assume_aligned(val + idx[j], N * S), N * S);
#pragma unroll
      for (int g = 0; g < N; ++g) s[g] = e.in[g];
#pragma unroll
      for (int j = 0; j < C; ++j)
#pragma unroll
        for (int g = 0; g < N; ++g) {
          // one of the two is zero: LDS for published rows, the buffer read
          // for the tile's own
          U u, w;
          __builtin_memcpy(&u, &lv[j][g], S);
          __builtin_memcpy(&w, &e.raw[j][g], S);
          u |= w;
          T o;
          __builtin_memcpy(&o, &u, S);
          s[g] = fmadd(-x.v[j], o, s[g]);
        }
      if (any_more && x.on && (x.row & kMore))
        btile_overflow<T, N, kUpper>(a, x.row & (kMore - 1), r, s);
      if constexpr (kUpper) {
#pragma unroll
        for (int g = 0; g < N; ++g) {
          T w = quot(s[g], x.dg);
          if (any_plain) {
            asm volatile("" : "+v"(s[g]));  // (a branch: not both and a select)
            w = s[g] / x.dg;
          }
          s[g] = w;
        }
      }
      __builtin_memcpy(__builtin_assume_aligned(val + self, N * S), s, N * S);
      asm volatile("" ::: "memory");
      if (lane == 0)
        __hip_atomic_fetch_add(&s_turn, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      asm volatile("" ::: "memory");
      // publish, then read ahead, then the other stores
      T h[N];
#pragma unroll
      for (int g = 0; g < N; ++g) {
        U u;
        __builtin_memcpy(&u, &s[g], S);
        if (u == Sentinel<T>::bits) u ^= 1;  // never publish the sentinel itself
        __builtin_memcpy(&h[g], &u, S);
      }
      const int pub = kUpper ? x.up : x.lo, arm = kUpper ? x.lo : x.up;
      int off = at(pub, S);
      vec_put<T, N, kCoherent>(b_h, (x.on & (pub >= 0)) ? off : kNowhere, h);
      double z[N];
      if constexpr (kUpper)
#pragma unroll
        for (int g = 0; g < N; ++g)
          z[g] = static_cast<double>(e.add[g]) + static_cast<double>(s[g]);
      vec_load(e, nx);
      const int row = x.row & (kMore - 1);
      if constexpr (kUpper) {
        off = at(row, 8);
        vec_put<double, N, 0>(b_sum, x.on ? off : kNowhere, z);
      }
      off = at(row, S);
      vec_put<T, N, 0>(b_out, x.on ? off : kNowhere, s);
      const U bits = Sentinel<T>::bits;
#pragma unroll
      for (int g = 0; g < N; ++g) __builtin_memcpy(&h[g], &bits, S);
      off = at(arm, S);
      vec_put<T, N, 0>(b_arm, (x.on & (arm >= 0)) ? off : kNowhere, h);
      x = nx;
    }
    __syncthreads();
  }
}

template <class T, int W>
void records(Handle* h, const TilePhase& p, const T* lu, Bytes& lrec, Bytes& urec, size_t off) {
  TileSched& S = h->tiles;
  BlockTiles& B = h->btiles;
  LAUNCH(h, "btiles", (k_brecords<T, W>), blocks_for(p.row1 - p.row0, kT), kT, 0, p.row0, p.row1,
         p.row0, p.row1, p.C, S.row.get(), S.pos.get(), h->rp.get(), h->ci.get(), h->diag.get(),
         S.slice.get(), S.tslice.get(), Near{B.sno.get(), B.tile_of.get()}, B.lo.get(), B.up.get(),
         lu, reinterpret_cast<Rec<T, W>*>(lrec.get() + off),
         reinterpret_cast<Rec<T, W>*>(urec.get() + off));
}

template <class T>
size_t rec_bytes(const TilePhase& p) {
  return p.W == 4 ? sizeof(Rec<T, 4>) : sizeof(Rec<T, 8>);
}

}  // namespace

static size_t record_bytes(Handle* h) {  // of one direction
  size_t b = 0;
  for (const TilePhase& p : h->tiles.ph)
    b += (h->precision == FAMS_PREC_MIXED ? rec_bytes<float>(p) : rec_bytes<double>(p)) *
         (p.row1 - p.row0);
  return b;
}

// Whether the tiles are the faster form for groups of K.  With boxes of a grid
// they are.  Where every row is in a run of consecutive rows, tiles have many
// narrow levels: a task (a tile and 32 bytes of each row's values) holds a
// workgroup for some time a slice, and the device runs some 256 at a time, so
// that a sweep takes time by the number of tasks; the level chunks take theirs by
// the levels and rows, whatever the width.  Both sweeps, tiles / chunks in us, of
// grids with one coupling out of place:
//   0.62M rows  FP64 K = 8 1048 / 1666, 16 1478 / 1543, 32 2225 / 1566
//   2.29M rows  FP64 K = 4 1861 / 3168, 8 2990 / 2922, 16 5471 / 2795, 32 9449 / 3053
//               FP32 K = 16 1852 / 2856, 32 3342 / 2853
//   9.4M rows   FP64 K = 2 4605 / 7753, 4 6182 / 5828, 8 11994 / 5122, 32 42405 / 8745
//               FP32 K = 8 3229 / 5164, 16 6614 / 4667, 32 13513 / 5863
// and of 2.29M rows in random order (82 slices a tile instead of 239) FP64 K = 8
// 1882 / 2033, 16 3138 / 2113, FP32 K = 16 1367 / 1882, 32 2307 / 2185.  Few wide
// levels (random order: 46 rows a slice instead of 17 to 31) leave the chunks the
// better form of wide rows at any size: 0.12M rows FP64 K = 16 872 / 714.
static bool tiles_faster(Handle* h, int K) {
  const TileSched& S = h->tiles;
  if (S.ph[0].boxes) return true;
  const bool mixed = h->precision == FAMS_PREC_MIXED;
  const int ntiles = S.ph[0].ntiles, row = K * (mixed ? 4 : 8);
  const double per_tile = static_cast<double>(S.slices) / ntiles;
  if (row >= 128 && h->n >= 40.0 * S.slices) return false;
  const double task = (mixed ? 0.8 + 0.003 * per_tile : 1.0 + 0.0065 * per_tile) *
                      (row < 32 ? 0.75 : 1.0);
  const double levels = static_cast<double>(h->info.ilu_levels_lower + h->info.ilu_levels_upper);
  const double chunks = (2.5 * levels + 0.2e-3 * h->n) * (K == 2 ? 1.5 : K == 4 ? 1.05 : 1.0);
  return ntiles * std::max(1, row / 32) * task <= chunks;
}

static bool served(Handle* h, int K) {
  return !h->tiles.ph.empty() && static_cast<double>(h->n) * K * 8 < 4294967296.0 - 512 &&
         tiles_faster(h, K);
}

// What block_tiles_prepare still has to allocate for groups of K (the published
// values of another K, which it gives back, not deducted; before the schedule
// is there, every row may have to be published in both directions).
size_t block_tiles_bytes(Handle* h, int K) {
  const BlockTiles& B = h->btiles;
  if (!served(h, K) || B.K == K) return 0;
  const size_t n = h->n, s = h->precision == FAMS_PREC_MIXED ? sizeof(float) : sizeof(double);
  size_t b = B.urec.get() ? 0 : 2 * record_bytes(h);
  if (!B.built) b += 4 * n * sizeof(int);
  return b + (B.built ? static_cast<size_t>(B.nlo) + B.nup : 2 * n) * K * s;
}

// The schedule's part for lock-step sweeps and the published values of
// groups of K, on first use; false: these sizes are not served.  A refused
// allocation leaves what is there in use, and the rest to the next call.
bool block_tiles_prepare(Handle* h, int K) {
  TileSched& S = h->tiles;
  BlockTiles& B = h->btiles;
  Allocator* A = &h->alloc;
  const bool mixed = h->precision == FAMS_PREC_MIXED;
  const size_t s = mixed ? sizeof(float) : sizeof(double);
  const int n = h->n;
  if (!served(h, K)) {
    B.K = 0;
    return false;
  }
  if (!B.built) {
    int nt = 0;
    for (const TilePhase& p : S.ph) nt += p.ntiles;
    BlockTiles N;
    N.sno.reset(A, n);
    N.tile_of.reset(A, n);
    N.lo.reset(A, n);
    N.up.reset(A, n);
    N.ticket.reset(A, 4 * kTicketStride);
    LAUNCH(h, "btiles", k_slice_numbers, nt, 64, 0, S.tslice.get(), S.slice.get(), N.sno.get(),
           N.tile_of.get());
    DBuf<int> ml(A, n + 1), mu(A, n + 1), sc(A, n + 1);
    HIPX(hipMemsetAsync(ml, 0, (n + 1) * sizeof(int), h->stream));
    HIPX(hipMemsetAsync(mu, 0, (n + 1) * sizeof(int), h->stream));
    for (const TilePhase& p : S.ph)
      LAUNCH(h, "btiles", k_bmarks, blocks_for(p.row1 - p.row0, kT), kT, 0, p.row0, p.row1, p.row0,
             p.row1, p.C, S.row.get(), S.pos.get(), h->rp.get(), h->ci.get(), h->diag.get(),
             Near{N.sno.get(), N.tile_of.get()}, ml.get(), mu.get());
    int cnt[2];
    for (int u = 0; u < 2; ++u) {
      DBuf<int>& m = u ? mu : ml;
      exclusive_scan_i32(h, m, sc, n + 1);
      LAUNCH(h, "btiles", k_bslots, blocks_for(n, kT), kT, 0, n, m.get(), sc.get(),
             (u ? N.up : N.lo).get());
      HIPX(hipMemcpyAsync(&cnt[u], sc.get() + n, sizeof(int), hipMemcpyDeviceToHost, h->stream));
    }
    HIPX(hipStreamSynchronize(h->stream));
    N.nlo = cnt[0];
    N.nup = cnt[1];
    if (const char* e = std::getenv("FAMS_SWEEP_WIDE")) N.wide_from = std::atof(e);
    N.built = true;
    B = std::move(N);
  }
  if (!B.values) {
    if (!B.urec.get()) {
      Bytes l, u;
      l.reset(A, record_bytes(h));
      u.reset(A, record_bytes(h));
      B.lrec = std::move(l);
      B.urec = std::move(u);
    }
    size_t off = 0;
    for (const TilePhase& p : S.ph) {
      if (mixed) {
        if (p.W == 4) records<float, 4>(h, p, h->ilu32.get(), B.lrec, B.urec, off);
        else records<float, 8>(h, p, h->ilu32.get(), B.lrec, B.urec, off);
      } else {
        if (p.W == 4) records<double, 4>(h, p, h->ilu.get(), B.lrec, B.urec, off);
        else records<double, 8>(h, p, h->ilu.get(), B.lrec, B.urec, off);
      }
      off += (mixed ? rec_bytes<float>(p) : rec_bytes<double>(p)) * (p.row1 - p.row0);
    }
    B.values = true;
  }
  if (B.K != K) {
    B.K = 0;
    B.hl.reset(A, std::max<size_t>(1, B.nlo) * K * s);
    B.hu.reset(A, std::max<size_t>(1, B.nup) * K * s);
    B.K = K;
    B.armed = false;
  }
  return true;
}

// x = U^{-1} L^{-1} b for K right-hand sides; y is scratch.
// With `sum`, sum = add + x in FP64 and x holds the second phase's rows only.
template <class T, int K>
void block_tiles_apply(Handle* h, const T* lu, const T* b, T* x, T* y, const T* add, double* sum) {
  TileSched& S = h->tiles;
  BlockTiles& B = h->btiles;
  const int n = h->n;
  T* HL = B.hl.as<T>();
  T* HU = B.hu.as<T>();
  if (!B.armed) {
    for (int u = 0; u < 2; ++u) {
      const int64_t m = static_cast<int64_t>(u ? B.nup : B.nlo) * K;
      LAUNCH(h, "bilu_arm", k_barm<T>, blocks_for(m, kT), kT, 0, m, u ? HU : HL);
    }
    HIPX(hipMemsetAsync(B.ticket, 0, 4 * kTicketStride * sizeof(int), h->stream));
  }
  B.armed = false;  // until every launch is queued (see tiles.hip)
  const unsigned long long limit = wait_limit(h);
  auto sweep = [&](int k, bool upper) {
    const TilePhase& p = S.ph[k];
    size_t off = 0;
    for (int q = 0; q < k; ++q) off += rec_bytes<T>(S.ph[q]) * (S.ph[q].row1 - S.ph[q].row0);
    BTileArgs<T> a{};
    a.tile0 = p.tile0;
    a.ntiles = p.ntiles;
    a.t0 = a.row0 = p.row0;
    a.t1 = a.row1 = p.row1;
    a.n = n;
    a.K = K;
    a.C = p.C;
    a.tslice = S.tslice.get();
    a.slice = S.slice.get();
    a.pos = S.pos.get();
    a.rp = h->rp.get();
    a.ci = h->ci.get();
    a.diag = h->diag.get();
    a.slot = (upper ? B.up : B.lo).get();
    a.rec = (upper ? B.urec : B.lrec).get() + off;
    a.lu = lu;
    a.in = upper || k == 1 ? y : b;
    a.out = !upper ? y : (sum && k == 0 ? nullptr : x);
    a.add = add;
    a.sum = upper ? sum : nullptr;
    a.H = upper ? HU : HL;
    a.arm = upper ? HL : HU;
    const int64_t hb = static_cast<int64_t>(B.nlo) * K * sizeof(T);
    const int64_t ub = static_cast<int64_t>(B.nup) * K * sizeof(T);
    a.hbytes = upper ? ub : hb;
    a.abytes = upper ? hb : ub;
    a.ticket = B.ticket.get() + (upper ? 2 + k : k) * kTicketStride;
    a.ticket_clear = B.ticket.get() + (upper ? 0 : 2) * kTicketStride;
    a.err = h->sweep_err.get();
    a.limit = limit;
    const double bytes = static_cast<double>(n) * K * sizeof(T);
    const bool wide = kCanWiden<T, K> && bytes >= (B.wide_from >= 0 ? B.wide_from
                                                   : p.C > 3 ? 1e9 : 0.5e9);
    const int KG = std::min(K, (p.C > 3 ? 32 : 64) * (wide ? 2 : 1) / static_cast<int>(sizeof(T)));
    const size_t lds = static_cast<size_t>(kZeroRow + 1) * KG * sizeof(T) +
                       (p.max_slices + 1) * sizeof(int);
    FAMS_REQUIRE(lds <= static_cast<size_t>(lds_hw_budget(h)), FAMS_ERR_CAPACITY,
                 "ILU tile does not fit in LDS");
#define FAMS_BTILE(C, UP, OVER, WIDE)                                                       \
  do {                                                                                      \
    allow_lds(reinterpret_cast<const void*>(&k_btile_sweep<T, K, C, UP, OVER, WIDE>), lds); \
    LAUNCH(h, UP ? "bilu_upper" : "bilu_lower", (k_btile_sweep<T, K, C, UP, OVER, WIDE>),   \
           std::min(p.ntiles * (K / KG), 2048), 64 * kWaves, lds, a);                       \
  } while (0)
#define FAMS_BTILE_W(C, UP, OVER)                                        \
  do {                                                                   \
    if (wide) FAMS_BTILE(C, UP, OVER, (kCanWiden<T, K>));                \
    else FAMS_BTILE(C, UP, OVER, false);                                 \
  } while (0)
#define FAMS_BTILES(C, OVER)                \
  do {                                      \
    if (upper) FAMS_BTILE_W(C, true, OVER); \
    else FAMS_BTILE_W(C, false, OVER);      \
  } while (0)
    switch (p.C) {
      case 3: FAMS_BTILES(3, false); break;
      case 4: FAMS_BTILES(4, false); break;
      default:
        if (p.over) FAMS_BTILES(8, true);
        else FAMS_BTILES(8, false);
        break;
    }
#undef FAMS_BTILES
#undef FAMS_BTILE_W
#undef FAMS_BTILE
  };
  sweep(0, false);
  if (S.ph.size() == 2) {
    const TilePhase& p = S.ph[1];
    const int64_t m = static_cast<int64_t>(p.row1 - p.row0) * K;
    LAUNCH(h, "bilu_pre", (k_bpre_lower<T, K>), blocks_for(m, kT), kT, 0, p.row0, n, h->rp.get(),
           h->ci.get(), lu, b, y);
    sweep(1, false);
    sweep(1, true);
    if (S.npre)
      LAUNCH(h, "bilu_pre", (k_bpre_upper<T, K>),
             blocks_for(static_cast<int64_t>(S.npre) * K, kT), kT, 0, S.npre, S.pre.get(),
             S.ph[0].row1, h->rp.get(), h->ci.get(), lu, x, y);
  }
  sweep(0, true);
  B.armed = true;
}

#define FAMS_BLOCK_TILES(K)                                                                     \
  template void block_tiles_apply<double, K>(Handle*, const double*, const double*, double*, double*, \
                                             const double*, double*);                           \
  template void block_tiles_apply<float, K>(Handle*, const float*, const float*, float*, float*, \
                                            const float*, double*);
FAMS_BLOCK_TILES(2)
FAMS_BLOCK_TILES(4)
FAMS_BLOCK_TILES(8)
FAMS_BLOCK_TILES(16)
FAMS_BLOCK_TILES(32)
#undef FAMS_BLOCK_TILES

}  // namespace fams
