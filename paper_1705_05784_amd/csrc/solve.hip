// The F-AMS iteration (Table 1) on the GPU, as a Richardson loop or as the
// right preconditioner of restarted GMRES (Sec. 4.6).
//
// Stage (Table 1 steps 5-7) applied to a residual r:
//   r_c = R r;  x_c = A_c^{-1} r_c;  dp1 = P x_c;       (multiscale stage)
//   r_half = r - A dp1;  dp2 = U^{-1} L^{-1} r_half;    (ILU(0) smoothing)
//   z = dp1 + dp2.
// Precision form: the stage runs on FP32 copies of A, P, R and the ILU(0)
// factors with FP32 vectors; the coarse solve, the outer residual q - A p,
// the Krylov basis and the solution update stay FP64.  Because the FP32
// stage is not exactly linear, GMRES keeps the preconditioned vectors
// (flexible GMRES); with an FP64 stage this is the same iteration as
// right-preconditioned GMRES.
//
// Reductions are two-stage with a fixed block count and fixed order, so a
// solve is bitwise reproducible.
#include <chrono>
#include <cmath>
#include <type_traits>
#include <vector>

#include "internal.hpp"

namespace fams {
namespace {

constexpr int kT = 256;
constexpr int kRedBlocks = 512;

// y = b - A x (b may be null: y = -A x; pos: row i's result goes to
// y[pos[i]], the order of the ILU(0) sweeps); 8 lanes per row, so a wavefront
// reads 8 consecutive rows' entries as one contiguous stretch; fixed-order
// shuffle reduction (deterministic).
constexpr int kSub = 8;
template <class TV, class TX, class TB, class TY>
__global__ void __launch_bounds__(256)
k_resid(int n, const int* rp, const int* ci, const TV* val, const TX* x, const TB* b, TY* y,
        const int* pos) {
  const int i = blockIdx.x * (blockDim.x / kSub) + threadIdx.x / kSub;
  const int l = threadIdx.x % kSub;
  double s = 0.0;
  if (i < n)
    for (int p = rp[i] + l; p < rp[i + 1]; p += kSub)
      s += static_cast<double>(val[p]) * static_cast<double>(x[ci[p]]);
  for (int o = kSub / 2; o > 0; o >>= 1) s += __shfl_down(s, o, kSub);
  if (i < n && l == 0)
    y[pos ? pos[i] : i] = static_cast<TY>((b ? static_cast<double>(b[i]) : 0.0) - s);
}

// y = M x with 8 lanes per row (see k_resid)
template <class TV, class TX, class TY>
__global__ void __launch_bounds__(256)
k_spmv8(int n, const int* rp, const int* ci, const TV* val, const TX* x, TY* y) {
  const int i = blockIdx.x * (blockDim.x / kSub) + threadIdx.x / kSub;
  const int l = threadIdx.x % kSub;
  double s = 0.0;
  if (i < n)
    for (int p = rp[i] + l; p < rp[i + 1]; p += kSub)
      s += static_cast<double>(val[p]) * static_cast<double>(x[ci[p]]);
  for (int o = kSub / 2; o > 0; o >>= 1) s += __shfl_down(s, o, kSub);
  if (i < n && l == 0) y[i] = static_cast<TY>(s);
}

__device__ double block_sum(double v) {
  __shared__ double s[kT / 64];
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  int w = threadIdx.x / 64, l = threadIdx.x % 64;
  __syncthreads();
  if (l == 0) s[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < (int)(blockDim.x / 64); ++k) r += s[k];
  return r;
}

// y[r] = sum_k M[r,k] x[k] for the fat rows of R = P^T (some N / n_c entries):
// a workgroup per row, four entries of a thread in flight, fixed-order sums --
// deterministic.  Bound by the latency of index and gather: a wavefront per
// row with one entry a lane at a time took 101 us for 0.5M unknowns in FP64
// and 60 us in FP32, this form 18 us and 19 us (10k unknowns: 4.8 and 2.9 us).
template <class TV, class TX>
__global__ void __launch_bounds__(kT)
k_restrict(int nrows, const int* rp, const int* ci, const TV* val, const TX* x, double* y) {
  constexpr int U = 4;
  const int row = blockIdx.x;
  if (row >= nrows) return;
  const int p1 = rp[row + 1];
  double s = 0.0;
  for (int pb = rp[row] + threadIdx.x; pb < p1; pb += U * kT) {
    int c[U];
    TV v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int p = min(pb + k * kT, p1 - 1);
      c[k] = ci[p];
      v[k] = val[p];
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (pb + k * kT < p1) s += static_cast<double>(v[k]) * static_cast<double>(x[c[k]]);
  }
  s = block_sum(s);
  if (threadIdx.x == 0) y[row] = s;
}

__global__ void k_dot_part(int64_t n, const double* a, const double* b, double* part) {
  double s = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    s += a[i] * b[i];
  s = block_sum(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// out[k] (+)= sum over blocks of part[b * stride + k]: one workgroup per k,
// strided partial sums then a fixed tree -- deterministic
__global__ void __launch_bounds__(256)
k_reduce(int nblk, int nv, int stride, const double* part, double* out, int accumulate) {
  const int k = blockIdx.x;
  double s = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) s += part[static_cast<int64_t>(b) * stride + k];
  s = block_sum(s);
  if (threadIdx.x == 0) out[k] = accumulate ? out[k] + s : s;
}

// One pass of the CGS2 orthogonalisation of w against V_0 .. V_{nv-1}:
//   kUpdate  w -= sum_k c_k V_k, c_k = the sum of cpart[k * kGsBlocks + b] over
//            b < nb, which every workgroup forms for itself in the same order;
//            the first one keeps it: coef[k] (+)= c_k,
//   kDots    part[k * kGsBlocks + b] = this workgroup's V_k . w (the new w),
//   kNorm    npart[b] = this workgroup's w . w (the new w).
// Bound by HBM: a pass reads V once, and a thread holds its row of V in
// registers, so an update and the next dot products share one pass (three
// reads of V where separate kernels took four, and no kernel between them).
// The dot products of a wavefront are summed by halves: each step exchanges
// half of the remaining values, NV exchanges in all instead of six for each.
// NV: nv rounded up to a power of two (the padding re-reads V_{nv-1}).
// Measured per step of a restart of 30 (orthogonalisation and rotation, kernel
// time), before and after: 8.6M rows 1490 and 720 us (V then read at 3.9 to
// 4.5 TB/s), 0.54M rows 131 and 65 us, 10k rows 47 and 29 us in 4 launches
// instead of 11.
constexpr int kGsT = 512, kGsBlocks = 256;
constexpr int kGsMax = 32;  // vectors of one pass

template <int NV, bool kUpdate, bool kDots, bool kNorm>
__global__ void __launch_bounds__(kGsT)
k_gs(int64_t n, int nv, const double* V, int64_t ldv, double* w, const double* cpart, double* coef,
     bool add, double* part, double* npart) {
  constexpr int kWaves = kGsT / 64;
  __shared__ double c[NV], red[kWaves][NV];
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, nb = gridDim.x;
  if constexpr (kUpdate) {
    for (int k = wave; k < NV; k += kWaves) {
      double s = 0.0;
      if (k < nv)
        for (int b = lane; b < nb; b += 64) s += cpart[k * kGsBlocks + b];
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (lane == 0) {
        c[k] = s;
        if (k < nv && blockIdx.x == 0) coef[k] = add ? coef[k] + s : s;
      }
    }
    __syncthreads();
  }
  double acc[NV], nrm = 0.0;
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kGsT + threadIdx.x; i < n;
       i += static_cast<int64_t>(nb) * kGsT) {
    double v[NV], x = w[i];
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = V[min(k, nv - 1) * ldv + i];
    if constexpr (kUpdate) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < NV; ++k)
        if (k < nv) s += c[k] * v[k];
      x -= s;
      w[i] = x;
    }
    if constexpr (kDots)
#pragma unroll
      for (int k = 0; k < NV; ++k) acc[k] += v[k] * x;
    if constexpr (kNorm) nrm += x * x;
  }
  if constexpr (kDots) {
    int own = 0;  // the value that this lane ends up with
#pragma unroll
    for (int h = NV / 2, o = 32; o > 0; h /= 2, o >>= 1) {
      if (h > 0) {
        const bool hi = lane & o;
        own += hi ? h : 0;
#pragma unroll
        for (int k = 0; k < h; ++k) {
          const double send = hi ? acc[k] : acc[k + h], keep = hi ? acc[k + h] : acc[k];
          acc[k] = keep + __shfl_xor(send, o, 64);
        }
      } else {
        acc[0] += __shfl_xor(acc[0], o, 64);
      }
    }
    if (lane % (64 / NV) == 0) red[wave][own] = acc[0];
    __syncthreads();
    if (threadIdx.x < nv) {
      double s = 0.0;
      for (int q = 0; q < kWaves; ++q) s += red[q][threadIdx.x];
      part[threadIdx.x * kGsBlocks + blockIdx.x] = s;
    }
  }
  if constexpr (kNorm) {
    for (int o = 32; o > 0; o >>= 1) nrm += __shfl_xor(nrm, o, 64);
    if (lane == 0) red[wave][0] = nrm;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int q = 0; q < kWaves; ++q) s += red[q][0];
      npart[blockIdx.x] = s;
    }
  }
}

// w -= sum_k coef[k] V_k   (or x += sum_k coef[k] V_k with sign = +1)
__global__ void k_maxpy(int64_t n, int nv, const double* V, int64_t ldv, const double* coef,
                        double sign, double* w) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int k = 0; k < nv; ++k) s += coef[k] * V[k * ldv + i];
  w[i] += sign * s;
}

__global__ void k_scale_by(int64_t n, const double* x, const double* den, double* y) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] = x[i] / *den;
}

__global__ void k_axpy(int64_t n, double a, const double* x, double* y) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] += a * x[i];
}

template <class TA, class TB, class TY>
__global__ void k_add(int64_t n, const TA* a, const TB* b, TY* y) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] = static_cast<TY>(static_cast<double>(a[i]) + static_cast<double>(b[i]));
}

template <class TA, class TY>
__global__ void k_cast(int64_t n, const TA* a, TY* y) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] = static_cast<TY>(a[i]);
}

__global__ void k_fill(int64_t n, double v, double* y) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) y[i] = v;
}

__global__ void k_sqrt_into(const double* src, double* dst) { *dst = sqrt(*src); }

// GMRES small dense part (one thread): Hessenberg column j from hcol,
// previous rotations, the new rotation and the residual estimate
struct GmresState {
  double* H;    // (m+1) x m, column-major
  double* cs;   // m
  double* sn;   // m
  double* g;    // m+1
  double* y;    // m
  double* hcol; // m+2
  double* out;  // 2: scratch scalars
};

__global__ void k_gmres_init(GmresState s, int m, const double* beta) {
  for (int k = 0; k <= m; ++k) s.g[k] = 0.0;
  s.g[0] = *beta;
}

// One wavefront: h_{j+1,j} = sqrt(sum of npart), then the rotations, from LDS
// (a serial chain: in global memory each rotation took a round trip).
constexpr int kGivensLds = 64;  // columns of the longest restart (fams_solve: 60)
__global__ void __launch_bounds__(64)
k_givens(GmresState s, int m, int j, int nb, const double* npart, double* host) {
  __shared__ double lds[3 * (kGivensLds + 2)];
  double sum = 0.0;
  for (int b = threadIdx.x; b < nb; b += 64) sum += npart[b];
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  const double hn = sqrt(sum);
  double *col = lds, *cs = lds + kGivensLds + 2, *sn = cs + kGivensLds + 2;
  for (int i = threadIdx.x; i <= j; i += 64) {
    col[i] = s.hcol[i];
    cs[i] = s.cs[i];
    sn[i] = s.sn[i];
  }
  if (threadIdx.x == 0) s.hcol[j + 1] = col[j + 1] = hn;
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = col[0];
    for (int i = 0; i < j; ++i) {
      const double b = col[i + 1];
      col[i] = cs[i] * a + sn[i] * b;
      a = -sn[i] * a + cs[i] * b;
    }
    const double den = hypot(a, hn);
    const double c = den == 0.0 ? 1.0 : a / den;
    const double sg = den == 0.0 ? 0.0 : hn / den;
    s.cs[j] = c;
    s.sn[j] = sg;
    col[j] = c * a + sg * hn;
    col[j + 1] = 0.0;
    const double g = s.g[j];
    s.g[j + 1] = -sg * g;
    s.g[j] = c * g;
    host[0] = fabs(sg * g);
    host[1] = hn;
  }
  __syncthreads();
  double* H = s.H + static_cast<int64_t>(j) * (m + 1);
  for (int i = threadIdx.x; i <= j + 1; i += 64) H[i] = col[i];
}

__global__ void k_backsolve(GmresState s, int m, int k) {
  for (int i = k - 1; i >= 0; --i) {
    double t = s.g[i];
    for (int c = i + 1; c < k; ++c) t -= s.H[static_cast<int64_t>(c) * (m + 1) + i] * s.y[c];
    s.y[i] = t / s.H[static_cast<int64_t>(i) * (m + 1) + i];
  }
}

// ---- helpers ------------------------------------------------------------------
struct Work {
  double *r, *w, *d1, *z, *rc, *xc, *part, *V, *Z;
  double* gpart;  // partial sums of the coarse matrix-vector product
  double *gs_part[2], *gs_npart;  // partial sums of the CGS2 passes
  float *r32, *d1_32, *rh32, *x32, *y32;
  double *rh, *x, *y;
  GmresState gs;
  int m;
};

Work work_of(Handle* h) {
  Work k{};
  int64_t n = h->n;
  int m = static_cast<int>((h->wk_vectors - 7) / 2);
  double* b = h->wk.get();
  k.m = m;
  k.r = b;
  k.w = b + n;
  k.d1 = b + 2 * n;
  k.z = b + 3 * n;
  k.rh = b + 4 * n;
  k.x = b + 5 * n;
  k.y = b + 6 * n;
  k.V = b + 7 * n;
  k.Z = k.V + static_cast<int64_t>(m + 1) * n;
  double* s = h->red.get();
  k.part = s;
  k.gs_part[0] = s;
  k.gs_part[1] = s + static_cast<int64_t>(kGsBlocks) * m;
  k.gs_npart = s + static_cast<int64_t>(kGsBlocks) * 2 * m;
  k.gpart = h->gpart.get();
  double* hs = h->hred.get();
  k.rc = hs;
  k.xc = hs + h->nc;
  double* q = hs + 2 * h->nc;
  k.gs.H = q;
  q += static_cast<int64_t>(m + 1) * m;
  k.gs.cs = q;
  q += m;
  k.gs.sn = q;
  q += m;
  k.gs.g = q;
  q += m + 1;
  k.gs.y = q;
  q += m;
  k.gs.hcol = q;
  q += m + 2;
  k.gs.out = q;
  if (h->precision == FAMS_PREC_MIXED) {
    float* f = h->wk32.get();
    k.r32 = f;
    k.d1_32 = f + n;
    k.rh32 = f + 2 * n;
    k.x32 = f + 3 * n;
    k.y32 = f + 4 * n;
  }
  return k;
}

// ||a||^2 or a.b into dst (device)
void dot_into(Handle* h, const double* a, const double* b, int64_t n, double* part, double* dst) {
  int nb = std::min<int64_t>(kRedBlocks, blocks_for(n, kT));
  LAUNCH(h, "dot", k_dot_part, nb, kT, 0, n, a, b, part);
  LAUNCH(h, "reduce", k_reduce, 1, 256, 0, nb, 1, 1, part, dst, 0);
}

double read_d(Handle* h, const double* d) {
  double v = 0.0;
  HIPX(hipMemcpyAsync(&v, d, sizeof(double), hipMemcpyDeviceToHost, h->stream));
  HIPX(hipStreamSynchronize(h->stream));
  return v;
}

double norm_host(Handle* h, const double* a, int64_t n, double* part, double* scratch) {
  dot_into(h, a, a, n, part, scratch);
  return std::sqrt(read_d(h, scratch));
}

int gs_blocks(int64_t n) { return static_cast<int>(std::min<int64_t>(kGsBlocks, blocks_for(n, kGsT))); }

template <bool kUpdate, bool kDots, bool kNorm>
void gs_pass(Handle* h, int64_t n, int nv, const double* V, double* w, const double* cpart,
             double* coef, bool add, double* part, double* npart) {
  const int nb = gs_blocks(n);
#define FAMS_GS(NV)                                                                             \
  LAUNCH(h, "gs_pass", (k_gs<NV, kUpdate, kDots, kNorm>), nb, kGsT, 0, n, nv, V, n, w, cpart, coef, \
         add, part, npart)
  if (nv <= 4) FAMS_GS(4);
  else if (nv <= 8) FAMS_GS(8);
  else if (nv <= 16) FAMS_GS(16);
  else FAMS_GS(32);
#undef FAMS_GS
}

// w orthogonal to V_0 .. V_{nv-1} by CGS2 (h = V^T w, w -= V h; c = V^T w,
// w -= V c; hcol = h + c), and the partial sums of ||w||^2.  Up to kGsMax
// vectors take the three passes of k_gs; with more, every product is finished
// over all vectors before the next update.
void orthogonalise(Handle* h, const Work& k, int64_t n, int nv) {
  double *p0 = k.gs_part[0], *p1 = k.gs_part[1], *hc = k.gs.hcol;
  if (nv <= kGsMax) {
    gs_pass<false, true, false>(h, n, nv, k.V, k.w, nullptr, nullptr, false, p0, nullptr);
    gs_pass<true, true, false>(h, n, nv, k.V, k.w, p0, hc, false, p1, nullptr);
    gs_pass<true, false, true>(h, n, nv, k.V, k.w, p1, hc, true, nullptr, k.gs_npart);
    return;
  }
  for (int pass = 0; pass < 2; ++pass) {
    auto each = [&](auto&& f) {
      for (int k0 = 0; k0 < nv; k0 += kGsMax) f(k0, std::min(kGsMax, nv - k0), k.V + k0 * n);
    };
    each([&](int k0, int c, const double* V) {
      gs_pass<false, true, false>(h, n, c, V, k.w, nullptr, nullptr, false, p0 + k0 * kGsBlocks,
                                  nullptr);
    });
    each([&](int k0, int c, const double* V) {
      gs_pass<true, false, true>(h, n, c, V, k.w, p0 + k0 * kGsBlocks, hc + k0, pass == 1, nullptr,
                                 k.gs_npart);
    });
  }
}

template <class TV, class TX, class TB, class TY>
void resid(Handle* h, const TV* val, const TX* x, const TB* b, TY* y, const int* pos = nullptr) {
  LAUNCH(h, "spmv_resid", (k_resid<TV, TX, TB, TY>), blocks_for(h->n, kT / kSub), kT, 0, h->n,
         h->rp.get(), h->ci.get(), val, x, b, y, pos);
}

// Table 1 steps 5-7 on a residual r (FP64 in, FP64 out); T = stage type.  The
// coarse half (d1 = P A_c^{-1} R r) depends on r alone and touches only scratch
// vectors, so the outer loops queue it before they wait for r's norm: the
// device works through the host's wait and the next launches (10k unknowns:
// 214 -> 179 us a GMRES step; the last step's share is wasted, 0.2% to 0.7% of
// a solve).
template <class T>
void stage_coarse(Handle* h, const Work& k, const double* r) {
  const int n = h->n, nc = h->nc;
  const T *pv, *rv, *rT;
  T* d1;
  if constexpr (std::is_same<T, double>::value) {
    pv = h->p_val.get();
    rv = h->r_val.get();
    rT = r;
    d1 = k.d1;
  } else {
    pv = h->p_val32.get();
    rv = h->r_val32.get();
    LAUNCH(h, "cast_d2f", (k_cast<double, float>), blocks_for(n, kT), kT, 0, (int64_t)n, r,
           k.r32);
    rT = k.r32;
    d1 = k.d1_32;
  }
  LAUNCH(h, "restrict", (k_restrict<T, T>), nc, kT, 0, nc, h->r_rp.get(), h->r_ci.get(), rv, rT,
         k.rc);
  coarse_apply(h, h->Ainv.get(), nc, k.rc, k.xc, k.gpart);
  LAUNCH(h, "prolong", (k_spmv8<T, double, T>), blocks_for(n, kT / kSub), kT, 0, n,
         h->p_rp.get(), h->p_ci.get(), pv, k.xc, d1);
}

// the rest: smoothing after stage_coarse on the same r
template <class T>
void stage_smooth(Handle* h, const Work& k, const double* r, double* z) {
  const int n = h->n;
  const T *av, *lu, *rT;
  T *d1, *rh, *x, *ysc;
  if constexpr (std::is_same<T, double>::value) {
    av = h->val.get();
    lu = h->ilu.get();
    rT = r;
    d1 = k.d1;
    rh = k.rh;
    x = k.x;
    ysc = k.y;
  } else {
    av = h->val32.get();
    lu = h->ilu32.get();
    rT = k.r32;
    d1 = k.d1_32;
    rh = k.rh32;
    x = k.x32;
    ysc = k.y32;
  }
  if (h->smoother && !h->blk) {  // z = d1 + x is written by the upper sweep
    if (!h->tiles.ph.empty()) {
      resid<T, T, T, T>(h, av, d1, rT, h->tiles.st.x.as<T>(), h->tiles.pos.get());
      ilu_apply<T>(h, lu, nullptr, nullptr, ysc, d1, z);
    } else {
      resid<T, T, T, T>(h, av, d1, rT, rh);
      ilu_apply<T>(h, lu, rh, x, ysc, d1, z);
    }
  } else if (h->smoother) {
    resid<T, T, T, T>(h, av, d1, rT, rh);
    ilu_apply<T>(h, lu, rh, x, ysc);
    {  // per-medium stage: r <- r - A x (row by row, in place), x += M_B^{-1} r
      Handle* b = h->blk.get();
      T* xb;
      const T* blu;
      if constexpr (std::is_same<T, double>::value) {
        xb = h->blk_x.get();
        blu = b->ilu.get();
      } else {
        xb = h->blk_x32.get();
        blu = b->ilu32.get();
      }
      resid<T, T, T, T>(h, av, x, rh, rh);
      ilu_apply<T>(b, blu, rh, xb, ysc);
      LAUNCH(h, "add", (k_add<T, T, T>), blocks_for(n, kT), kT, 0, (int64_t)n, x, xb, x);
    }
    LAUNCH(h, "add", (k_add<T, T, double>), blocks_for(n, kT), kT, 0, (int64_t)n, d1, x, z);
  } else {
    LAUNCH(h, "cast", (k_cast<T, double>), blocks_for(n, kT), kT, 0, (int64_t)n, d1, z);
  }
}

void coarse_any(Handle* h, const Work& k, const double* r) {
  if (h->precision == FAMS_PREC_MIXED) stage_coarse<float>(h, k, r);
  else stage_coarse<double>(h, k, r);
}

void smooth_any(Handle* h, const Work& k, const double* r, double* z) {
  if (h->precision == FAMS_PREC_MIXED) stage_smooth<float>(h, k, r, z);
  else stage_smooth<double>(h, k, r, z);
}

void stage_any(Handle* h, const Work& k, const double* r, double* z) {
  coarse_any(h, k, r);
  smooth_any(h, k, r, z);
}

fams_status_t richardson(Handle* h, const Work& k, const double* q, double* p,
                         const fams_solve_opts_t* o, fams_info_t* info) {
  const int n = h->n;
  double* scratch = k.gs.out;
  resid<double, double, double, double>(h, h->val.get(), p, q, k.r);
  double r0 = norm_host(h, k.r, n, k.part, scratch);
  int it = 0;
  fams_status_t st = FAMS_NOT_CONVERGED;
  double nr = r0;
  if (r0 == 0.0) st = FAMS_OK;
  HostOut& host = h->host_out;
  host.ensure();
  if (st != FAMS_OK && it < o->max_iter) coarse_any(h, k, k.r);
  while (st != FAMS_OK && it < o->max_iter) {
    smooth_any(h, k, k.r, k.z);
    LAUNCH(h, "axpy", k_axpy, blocks_for(n, kT), kT, 0, (int64_t)n, 1.0, k.z, p);
    resid<double, double, double, double>(h, h->val.get(), p, q, k.r);
    ++it;
    dot_into(h, k.r, k.r, n, k.part, host.p);
    HIPX(hipEventRecord(host.ev, h->stream));
    if (it < o->max_iter) coarse_any(h, k, k.r);  // the next iteration's, unless this is the last
    HIPX(hipEventSynchronize(host.ev));
    nr = std::sqrt(host.p[0]);
    if (!std::isfinite(nr) || nr > 1e8 * r0) {
      st = FAMS_DIVERGED;
      break;
    }
    if (nr <= o->rtol * r0) st = FAMS_OK;
  }
  info->iterations = it;
  info->rel_residual = r0 > 0 ? nr / r0 : 0.0;
  return st;
}

fams_status_t gmres(Handle* h, const Work& k, const double* q, double* p,
                    const fams_solve_opts_t* o, fams_info_t* info) {
  const int64_t n = h->n;
  const int m = std::min(o->restart, k.m);
  FAMS_REQUIRE(m <= kGivensLds, FAMS_ERR_CAPACITY, "GMRES restart too long");
  double* scratch = k.gs.out;
  resid<double, double, double, double>(h, h->val.get(), p, q, k.r);
  double r0 = norm_host(h, k.r, n, k.part, scratch);
  double tol = o->rtol * r0;
  int it = 0;
  fams_status_t st = FAMS_NOT_CONVERGED;
  double beta = r0;
  HostOut& host = h->host_out;
  host.ensure();
  while (true) {
    if (beta <= tol) {
      st = FAMS_OK;
      break;
    }
    if (!std::isfinite(beta) || beta > 1e8 * r0) {
      st = FAMS_DIVERGED;
      break;
    }
    if (it >= o->max_iter) break;
    // V_0 = r / beta
    dot_into(h, k.r, k.r, n, k.part, k.gs.hcol + m + 1);
    LAUNCH(h, "sqrt", k_sqrt_into, 1, 1, 0, k.gs.hcol + m + 1, k.gs.hcol + m + 1);
    LAUNCH(h, "scale", k_scale_by, blocks_for(n, kT), kT, 0, n, k.r, k.gs.hcol + m + 1, k.V);
    LAUNCH(h, "gmres_init", k_gmres_init, 1, 1, 0, k.gs, m, k.gs.hcol + m + 1);
    int kk = 0;
    coarse_any(h, k, k.V);
    for (int j = 0; j < m; ++j) {
      double* vj = k.V + j * n;
      double* zj = k.Z + j * n;
      smooth_any(h, k, vj, zj);
      LAUNCH(h, "spmv", (k_spmv8<double, double, double>), blocks_for(n, kT / kSub), kT, 0,
             (int)n, h->rp.get(), h->ci.get(), h->val.get(), zj, k.w);
      orthogonalise(h, k, n, j + 1);
      LAUNCH(h, "givens", k_givens, 1, 64, 0, k.gs, m, j, gs_blocks(n), k.gs_npart,
             host.p);
      HIPX(hipEventRecord(host.ev, h->stream));
      if (j + 1 < m && it + 1 < o->max_iter) {  // the next step's start, unless this is the last
        LAUNCH(h, "scale", k_scale_by, blocks_for(n, kT), kT, 0, n, k.w, k.gs.hcol + j + 1,
               vj + n);
        coarse_any(h, k, vj + n);
      }
      HIPX(hipEventSynchronize(host.ev));
      ++it;
      kk = j + 1;
      if (host.p[0] <= tol || it >= o->max_iter || !(host.p[1] > 0.0) || !std::isfinite(host.p[0]))
        break;
    }
    LAUNCH(h, "backsolve", k_backsolve, 1, 1, 0, k.gs, m, kk);
    LAUNCH(h, "maxpy", k_maxpy, blocks_for(n, kT), kT, 0, n, kk, k.Z, n, k.gs.y, 1.0, p);
    resid<double, double, double, double>(h, h->val.get(), p, q, k.r);
    beta = norm_host(h, k.r, n, k.part, scratch);
  }
  info->iterations = it;
  info->rel_residual = r0 > 0 ? beta / r0 : 0.0;
  return st;
}

}  // namespace

// A bounded wait that gave up means the sweep's dependency order was broken.
// The per-medium stage sweeps on a handle of its own, with words of its own.
// Words that were set are cleared, and the published values of that handle
// armed again, so that the next call starts anew.
void check_sweeps(Handle* h) {
  Handle* gs[2] = {h, h->blk.get()};
  int e[2][2] = {};
  for (int k = 0; k < 2; ++k)
    if (gs[k] && gs[k]->sweep_err.get())
      HIPX(hipMemcpyAsync(e[k], gs[k]->sweep_err.get(), sizeof(e[k]), hipMemcpyDeviceToHost,
                          h->stream));
  HIPX(hipStreamSynchronize(h->stream));
  for (int k = 0; k < 2; ++k) {
    if (e[k][0] || e[k][1])
      HIPX(hipMemsetAsync(gs[k]->sweep_err, 0, sizeof(e[k]), h->stream));
    if (e[k][0]) gs[k]->tiles.armed = gs[k]->btiles.armed = false;
    h->info.long_waits += e[k][1];
  }
  FAMS_REQUIRE(!e[0][0] && !e[1][0], FAMS_ERR_DEVICE,
               "ILU(0) sweep: a dependency wait exceeded its bound");
}

void ensure_workspace(Handle* h, int restart) {
  int m = std::max(restart, 1);
  size_t need = static_cast<size_t>(7 + 2 * m + 1);
  if (h->wk_vectors >= need) return;
  h->wk_vectors = 0;  // none until every buffer is there
  h->wk.reset(&h->alloc, need * static_cast<size_t>(h->n));
  h->red.reset(&h->alloc, static_cast<size_t>(kRedBlocks) * (m + 2) + 16);
  h->hred.reset(&h->alloc, 2 * static_cast<size_t>(h->nc) + static_cast<size_t>(m + 1) * m +
                               6 * static_cast<size_t>(m) + 16);
  if (h->precision == FAMS_PREC_MIXED) h->wk32.reset(&h->alloc, 5 * static_cast<size_t>(h->n));
  const size_t nch = (static_cast<size_t>(h->nc) + 63) / 64;   // coarse GEMV column chunks
  if (!h->gpart.get()) h->gpart.reset(&h->alloc, nch * h->nc);
  h->wk_vectors = need;
}

fams_status_t solve_one(Handle* h, const double* q, double* p, const fams_solve_opts_t* o,
                        fams_info_t* info) {
  ensure_workspace(h, o->outer == FAMS_GMRES ? o->restart : 1);
  Work k = work_of(h);
  for (Handle* g : {h, h->blk.get()})
    if (g && g->sweep_err.get()) HIPX(hipMemsetAsync(g->sweep_err, 0, sizeof(int), h->stream));
  if (!o->use_initial_guess) HIPX(hipMemsetAsync(p, 0, sizeof(double) * h->n, h->stream));
  auto t0 = std::chrono::steady_clock::now();
  fams_status_t st = o->outer == FAMS_GMRES ? gmres(h, k, q, p, o, info)
                                            : richardson(h, k, q, p, o, info);
  HIPX(hipStreamSynchronize(h->stream));
  check_sweeps(h);
  info->ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0)
                 .count();
  info->status = st;
  return st;
}

void apply_stage_fp64(Handle* h, const double* r, double* z) {
  ensure_workspace(h, 1);
  Work k = work_of(h);
  stage_any(h, k, r, z);
  HIPX(hipStreamSynchronize(h->stream));
  check_sweeps(h);
}

// The stage's scratch inside one caller-provided region of device memory:
// [rc | xc | gpart | d1 rh x y] (FP64 handles) or [rc | xc | gpart | r32 d1
// rh x y] in float (precision form), each part 256-byte aligned.  Returns
// the bytes needed; with `base` != null, also fills `k`.
static size_t stage_scratch_layout(Handle* h, void* base, Work* k) {
  const size_t n = h->n, nc = h->nc, nch = (nc + 63) / 64;
  auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t o_xc = up(nc * sizeof(double));
  const size_t o_gp = o_xc + up(nc * sizeof(double));
  const size_t o_v = o_gp + up(nch * nc * sizeof(double));
  const bool mixed = h->precision == FAMS_PREC_MIXED;
  const size_t vb = up(n * (mixed ? sizeof(float) : sizeof(double)));
  const size_t total = o_v + (mixed ? 5 : 4) * vb;
  if (base && k) {
    char* b = static_cast<char*>(base);
    *k = Work{};
    k->rc = reinterpret_cast<double*>(b);
    k->xc = reinterpret_cast<double*>(b + o_xc);
    k->gpart = reinterpret_cast<double*>(b + o_gp);
    if (mixed) {
      float* f[5];
      for (int i = 0; i < 5; ++i) f[i] = reinterpret_cast<float*>(b + o_v + i * vb);
      k->r32 = f[0];
      k->d1_32 = f[1];
      k->rh32 = f[2];
      k->x32 = f[3];
      k->y32 = f[4];
    } else {
      double* d[4];
      for (int i = 0; i < 4; ++i) d[i] = reinterpret_cast<double*>(b + o_v + i * vb);
      k->d1 = d[0];
      k->rh = d[1];
      k->x = d[2];
      k->y = d[3];
    }
  }
  return total;
}

size_t stage_scratch_bytes(Handle* h) { return stage_scratch_layout(h, nullptr, nullptr); }

// the stage with its scratch in `base` (stage_scratch_bytes bytes); the
// handle's own structures were all allocated by the setup
void apply_stage_in(Handle* h, void* base, const double* r, double* z) {
  Work k;
  stage_scratch_layout(h, base, &k);
  stage_any(h, k, r, z);
  HIPX(hipStreamSynchronize(h->stream));
  check_sweeps(h);
}

double dev_dot(Handle* h, const double* a, const double* b, int64_t n) {
  ensure_workspace(h, 1);
  Work k = work_of(h);
  dot_into(h, a, b, n, k.part, k.gs.out);
  return read_d(h, k.gs.out);
}

void dev_copy_d(Handle* h, double* dst, const double* src, int64_t n) {
  HIPX(hipMemcpyAsync(dst, src, n * sizeof(double), hipMemcpyDeviceToDevice, h->stream));
}

}  // namespace fams
