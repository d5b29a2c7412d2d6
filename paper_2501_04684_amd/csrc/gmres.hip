// Restarted GMRES kernels for (sigma I + Z^F) x = b, with nrhs independent
// right-hand sides sharing each far-zone product launch.
//
// Krylov vectors are complex64 (the product's input format); every inner
// product, norm, Gram-Schmidt update and the Hessenberg / Givens / least-
// squares state are FP64. Reductions are two-level with a fixed block count
// and a fixed summation order, so results repeat bit for bit.
#include <hip/hip_runtime.h>

#include <type_traits>

#include <cstdint>

#include "gmres.hpp"

namespace ubf {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kColTile = 4;    // Krylov columns per pass over w
constexpr int kElems = 2;      // elements of a slice per thread and batch of loads (dots)

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) * b
__device__ inline double2 cmulc(double2 a, double2 b) {
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__device__ inline double2 f2d(float2 v) { return make_double2(v.x, v.y); }

// Sum over the 64 lanes, in every lane.
__device__ inline double2 wave_sum(double2 v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    v.x += __shfl_xor(v.x, o, 64);
    v.y += __shfl_xor(v.y, o, 64);
  }
  return v;
}

// The sums of the Arnoldi step are two-level with a fixed block count and
// order: each block of a kernel leaves the partial sums of its slice, and
// every block of the next kernel adds them up for itself (a wavefront per
// column, a lane per block), so no reduction kernel stands in between. That
// kernel ran one thread per column over all blocks' partials, a chain of 256
// dependent additions with exposed loads: 55 us each on the 762-box sphere
// (one vector), 74 us on a 5,288-box mask (four), three times per step.
// The block count depends on n alone (gmres_blocks), so that a right-hand
// side's sums do not depend on its neighbours. partial: [R][ldp][blocks].
__device__ inline double2* partial_of(double2* partial, int r, int ldp, int c) {
  return partial + ((int64_t)r * ldp + c) * gridDim.x;
}

// hs[c] = sum over the blocks of column c's partials, c < ncol (ends with a
// barrier).
__device__ __forceinline__ void gather_partials(const double2* __restrict__ partial, int r, int ldp, int ncol,
                                double2* hs) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nblk = gridDim.x;
  for (int c = wave; c < ncol; c += kWaves) {
    const double2* p = partial + ((int64_t)r * ldp + c) * nblk;
    double2 s = make_double2(0.0, 0.0);
    for (int b = lane; b < nblk; b += 64) {
      s.x += p[b].x;
      s.y += p[b].y;
    }
    s = wave_sum(s);
    if (lane == 0) hs[c] = s;
  }
  __syncthreads();
}

// The block's slice [lo, hi) of a vector of n elements.
__device__ inline void slice_of(int64_t n, int64_t& lo, int64_t& hi) {
  const int64_t len = (n + gridDim.x - 1) / gridDim.x;
  lo = (int64_t)blockIdx.x * len;
  hi = min(lo + len, n);
}

// Calls f(integral_constant<NC>) for a tile of nc = 1..kColTile columns, so
// that a tile's loads are one batch. Behind a test per column each load was
// waited for before the next was issued, and the routine, not inlined, held
// its kernels at one block per CU: at 428,328 elements and four vectors
// orth_first took 44 us and orth_second 47 us a step (1 to 5 columns), now 24
// and 27. Tiles of eight columns and four elements need 214 registers: 50, 53.
template <class F>
__device__ inline void with_columns(int nc, F f) {
  static_assert(kColTile == 4, "cases");
  switch (nc) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    default: f(std::integral_constant<int, 4>()); break;
  }
}

// This block's partial sums of conj(V_c[i]) w[i] over its slice, columns
// c < ncol; V and w at the right-hand side's first element.
__device__ __forceinline__ void slice_dots(const float2* __restrict__ V, int64_t vstride, int ncol,
                           const float2* w, int64_t lo, int64_t hi, double2* partial, int r,
                           int ldp, double2 (*sh)[kColTile]) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int c0 = 0; c0 < ncol; c0 += kColTile) {
    double2 acc[kColTile];
#pragma unroll
    for (int t = 0; t < kColTile; ++t) acc[t] = make_double2(0.0, 0.0);
    with_columns(min(ncol - c0, kColTile), [&](auto tag) {
      constexpr int NC = decltype(tag)::value;
      for (int64_t i = lo + threadIdx.x; i < hi; i += kElems * kThreads) {
        float2 v[NC][kElems], wv[kElems];
#pragma unroll
        for (int e = 0; e < kElems; ++e) {  // clamped to the slice, left out below
          const int64_t k = min(i + e * kThreads, hi - 1);
          wv[e] = w[k];
#pragma unroll
          for (int t = 0; t < NC; ++t) v[t][e] = V[(int64_t)(c0 + t) * vstride + k];
        }
#pragma unroll
        for (int e = 0; e < kElems; ++e)
          if (i + e * kThreads < hi) {
#pragma unroll
            for (int t = 0; t < NC; ++t) {
              const double2 p = cmulc(f2d(v[t][e]), f2d(wv[e]));
              acc[t].x += p.x;
              acc[t].y += p.y;
            }
          }
      }
    });
#pragma unroll
    for (int t = 0; t < kColTile; ++t)
      if (c0 + t < ncol) {  // uniform
        const double2 s = wave_sum(acc[t]);
        if (lane == 0) sh[wave][t] = s;
      }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < kColTile && c0 + t < ncol) {
      double2 s = make_double2(0.0, 0.0);
      for (int v = 0; v < kWaves; ++v) {
        s.x += sh[v][t].x;
        s.y += sh[v][t].y;
      }
      partial_of(partial, r, ldp, c0 + t)[blockIdx.x] = s;
    }
    __syncthreads();  // sh is written again
  }
}

// This block's partial of sum |w_i|^2 from each thread's own sum.
__device__ void slice_norm(double v, double2* partial, int r, double2 (*sh)[kColTile]) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double2 s = wave_sum(make_double2(v, 0.0));
  if (lane == 0) sh[wave][0] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w) t += sh[w][0].x;
    partial_of(partial, r, 1, 0)[blockIdx.x] = make_double2(t, 0.0);
  }
}

__device__ inline double norm2(float2 v) {
  return (double)v.x * v.x + (double)v.y * v.y;
}

// An Arnoldi step after the product w = Z v_j is four kernels over slices
// of the vectors, bound by memory for long vectors (V is read twice per
// Gram-Schmidt pass) and by the launches for short ones:
//   orth_first:  w += sigma v_j; partials of h1 = V^H w
//   orth_second: w -= V h1; partials of h2 = V^H w (second pass)
//   orth_last:   w -= V h2; partials of ||w||^2
//   next_column: v_{j+1} = w / ||w||; the rotations, the residual estimate
//                and the status row of the step (one block per right-hand side)
// w is rounded to FP32 between the passes. Before, the same work took eleven
// kernels and a copy (207 us of 320 us per step on the 762-box sphere).
__global__ __launch_bounds__(kThreads, 4) void orth_first_kernel(
    const float2* __restrict__ V, int64_t vstride, int j, float2* __restrict__ w, double sr,
    double si, int64_t n, int R, double2* __restrict__ partial, int ldp) {
  __shared__ double2 sh[kWaves][kColTile];
  const int r = blockIdx.y;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  float2* wr = w + (int64_t)r * n;
  const float2* Vr = V + (int64_t)r * n;
  const float2* vj = Vr + (int64_t)j * vstride;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) {
    const double2 a = f2d(wr[i]), b = f2d(vj[i]);
    wr[i] = make_float2((float)(a.x + sr * b.x - si * b.y), (float)(a.y + sr * b.y + si * b.x));
  }
  slice_dots(Vr, vstride, j + 1, wr, lo, hi, partial, r, ldp, sh);
}

// w -= V h over the slice (FP64 sum, one rounding to FP32); the thread's sum
// of |w|^2 afterwards.
__device__ __forceinline__ double slice_update(const float2* __restrict__ V, int64_t vstride, int ncol,
                               const double2* hs, float2* w, int64_t lo, int64_t hi) {
  double nn = 0.0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) {
    double2 s = f2d(w[i]);
    for (int c0 = 0; c0 < ncol; c0 += kColTile)
      with_columns(min(ncol - c0, kColTile), [&](auto tag) {
        constexpr int NC = decltype(tag)::value;
        float2 v[NC];
#pragma unroll
        for (int t = 0; t < NC; ++t) v[t] = V[(int64_t)(c0 + t) * vstride + i];
#pragma unroll
        for (int t = 0; t < NC; ++t) {
          const double2 p = cmul(f2d(v[t]), hs[c0 + t]);
          s.x -= p.x;
          s.y -= p.y;
        }
      });
    const float2 o = make_float2((float)s.x, (float)s.y);
    w[i] = o;
    nn += norm2(o);
  }
  return nn;
}

__global__ __launch_bounds__(kThreads, 4) void orth_second_kernel(
    const float2* __restrict__ V, int64_t vstride, int ncol, float2* __restrict__ w, int64_t n,
    int R, const double2* __restrict__ partial1, double2* __restrict__ partial2, int ldp,
    double2* __restrict__ h1, int ldh) {
  __shared__ double2 sh[kWaves][kColTile];
  __shared__ double2 hs[kMaxRestart + 1];
  const int r = blockIdx.y;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  gather_partials(partial1, r, ldp, ncol, hs);
  if (blockIdx.x == 0)
    for (int c = threadIdx.x; c < ncol; c += kThreads) h1[(int64_t)r * ldh + c] = hs[c];
  float2* wr = w + (int64_t)r * n;
  const float2* Vr = V + (int64_t)r * n;
  slice_update(Vr, vstride, ncol, hs, wr, lo, hi);
  slice_dots(Vr, vstride, ncol, wr, lo, hi, partial2, r, ldp, sh);
}

__global__ __launch_bounds__(kThreads, 4) void orth_last_kernel(
    const float2* __restrict__ V, int64_t vstride, int ncol, float2* __restrict__ w, int64_t n,
    int R, const double2* __restrict__ partial2, int ldp, double2* __restrict__ norm_partial,
    double2* __restrict__ h2, int ldh) {
  __shared__ double2 sh[kWaves][kColTile];
  __shared__ double2 hs[kMaxRestart + 1];
  const int r = blockIdx.y;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  gather_partials(partial2, r, ldp, ncol, hs);
  if (blockIdx.x == 0)
    for (int c = threadIdx.x; c < ncol; c += kThreads) h2[(int64_t)r * ldh + c] = hs[c];
  const double nn = slice_update(V + (int64_t)r * n, vstride, ncol, hs, w + (int64_t)r * n, lo, hi);
  slice_norm(nn, norm_partial, r, sh);
}

// dst = src * f over the slice.
__device__ void slice_scale(float2* dst, const float2* src, double f, int64_t lo,
                            int64_t hi) {
  for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) {
    const float2 v = src[i];
    dst[i] = make_float2((float)(v.x * f), (float)(v.y * f));
  }
}

__device__ inline void put_status(GmresStatusRow* row, double res, int active, int iters) {
  row->res = res;
  row->active = active;
  row->iters = iters;
}

// The rotations of Arnoldi column j (one thread; H column, rotations and g
// in LDS): h = h1 + h2 (two Gram-Schmidt passes), h_{j+1,j} = hn; apply the
// earlier Givens rotations, make the new one, update the least-squares
// right-hand side g and the residual estimate |g_{j+1}|.
__device__ void rotate_column(const GmresState& st, int r, int j, double hn, double tol,
                              bool broke, double2* Hc, const double* cs, const double2* sn,
                              int32_t* active_out, GmresStatusRow* row) {
  const int m = st.m, ld = m + 1;
  // earlier rotations: [x; y] <- [c x + s y; -conj(s) x + c y]
  for (int i = 0; i < j; ++i) {
    const double c = cs[i];
    const double2 s = sn[i];
    const double2 x = Hc[i], y = Hc[i + 1];
    const double2 sy = cmul(s, y), sx = cmulc(s, x);
    Hc[i] = make_double2(c * x.x + sy.x, c * x.y + sy.y);
    Hc[i + 1] = make_double2(-sx.x + c * y.x, -sx.y + c * y.y);
  }
  // new rotation zeroing hn below a = Hc[j]
  const double2 a = Hc[j];
  const double aa = sqrt(a.x * a.x + a.y * a.y);
  const double t = sqrt(aa * aa + hn * hn);
  double c;
  double2 s;
  if (hn == 0.0) {
    c = 1.0;
    s = make_double2(0.0, 0.0);
  } else if (aa == 0.0) {
    c = 0.0;
    s = make_double2(1.0, 0.0);
  } else {
    c = aa / t;
    s = make_double2(a.x / aa * hn / t, a.y / aa * hn / t);
  }
  st.cs[r * m + j] = c;
  st.sn[r * m + j] = s;
  Hc[j] = aa == 0.0 ? make_double2(hn, 0.0) : make_double2(a.x / aa * t, a.y / aa * t);
  Hc[j + 1] = make_double2(0.0, 0.0);
  const double2 gj = st.g[r * ld + j];
  const double2 sg = cmulc(s, gj);
  const double2 gn = make_double2(-sg.x, -sg.y);
  st.g[r * ld + j] = make_double2(c * gj.x, c * gj.y);
  st.g[r * ld + j + 1] = gn;
  st.k[r] = j + 1;
  const int32_t iters = st.iters[r] + 1;
  st.iters[r] = iters;
  const double rel = sqrt(gn.x * gn.x + gn.y * gn.y) / st.bnorm[r];
  st.res[r] = rel;
  // lucky breakdown (the Krylov space is invariant) or convergence
  const int32_t on = (rel <= tol || broke) ? 0 : 1;
  active_out[r] = on;
  put_status(row, rel, on, iters);
}

// v_{j+1} = w / ||w||, and in block 0 of each right-hand side the step's
// rotations and status row. Every block needs the flag of the step before,
// so block 0 writes the new one to another array (the host swaps them).
__global__ __launch_bounds__(kThreads) void next_column_kernel(
    GmresState st, int j, double tol, const double2* __restrict__ norm_partial,
    const int32_t* __restrict__ active_in, int32_t* __restrict__ active_out,
    const float2* __restrict__ w, float2* __restrict__ vnext, int64_t n, int R,
    GmresStatusRow* __restrict__ status) {
  __shared__ double2 nrm[1];
  __shared__ double2 Hc[kMaxRestart + 2];
  __shared__ double cs[kMaxRestart];
  __shared__ double2 sn[kMaxRestart];
  __shared__ double colnorm2;
  const int r = blockIdx.y, m = st.m, ld = m + 1, t = threadIdx.x;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  float2* dst = vnext + (int64_t)r * n;
  const float2* src = w + (int64_t)r * n;
  if (!active_in[r]) {  // uniform per right-hand side
    slice_scale(dst, src, 0.0, lo, hi);
    if (blockIdx.x == 0 && t == 0) {
      active_out[r] = 0;
      put_status(&status[r], st.res[r], 0, st.iters[r]);
    }
    return;
  }
  for (int i = t; i <= j; i += kThreads) {
    const double2 a = st.h1[(int64_t)r * ld + i], b = st.h2[(int64_t)r * ld + i];
    Hc[i] = make_double2(a.x + b.x, a.y + b.y);
    if (i < j) {
      cs[i] = st.cs[r * m + i];
      sn[i] = st.sn[r * m + i];
    }
  }
  gather_partials(norm_partial, r, 1, 1, nrm);
  if (t < 64) {
    double2 q = make_double2(0.0, 0.0);
    for (int i = t; i <= j; i += 64) q.x += Hc[i].x * Hc[i].x + Hc[i].y * Hc[i].y;
    q = wave_sum(q);
    if (t == 0) colnorm2 = q.x;
  }
  __syncthreads();
  const double hn = sqrt(nrm[0].x);
  const bool broke = hn <= 1e-14 * sqrt(colnorm2 + hn * hn);
  slice_scale(dst, src, (broke || hn == 0.0) ? 0.0 : 1.0 / hn, lo, hi);
  if (blockIdx.x != 0) return;
  if (t == 0) rotate_column(st, r, j, hn, tol, broke, Hc, cs, sn, active_out, &status[r]);
  __syncthreads();
  double2* H = st.H + ((int64_t)r * m + j) * ld;  // column j of this right-hand side
  for (int i = t; i <= j + 1; i += kThreads) H[i] = Hc[i];
}

// Start of a solve: x = 0, V_0 = b and the partials of ||b||^2.
__global__ __launch_bounds__(kThreads) void begin_kernel(const float2* __restrict__ b,
                                                         float2* __restrict__ x,
                                                         float2* __restrict__ v0, int64_t n,
                                                         int R, double2* __restrict__ partial) {
  __shared__ double2 sh[kWaves][kColTile];
  const int r = blockIdx.y;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  double nn = 0.0;
  for (int64_t i = (int64_t)r * n + lo + threadIdx.x; i < (int64_t)r * n + hi; i += kThreads) {
    const float2 v = b[i];
    x[i] = make_float2(0.f, 0.f);
    v0[i] = v;
    nn += norm2(v);
  }
  slice_norm(nn, partial, r, sh);
}

// V_0 = b - sigma x - ax (residual of the shifted system) and the partials
// of its norm.
__global__ __launch_bounds__(kThreads) void residual_kernel(
    float2* __restrict__ v0, const float2* __restrict__ b, const float2* __restrict__ x,
    const float2* __restrict__ ax, double sr, double si, int64_t n, int R,
    double2* __restrict__ partial) {
  __shared__ double2 sh[kWaves][kColTile];
  const int r = blockIdx.y;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  double nn = 0.0;
  for (int64_t i = (int64_t)r * n + lo + threadIdx.x; i < (int64_t)r * n + hi; i += kThreads) {
    const double2 bv = f2d(b[i]), xv = f2d(x[i]), av = f2d(ax[i]);
    const float2 o = make_float2((float)(bv.x - (sr * xv.x - si * xv.y) - av.x),
                                 (float)(bv.y - (sr * xv.y + si * xv.x) - av.y));
    v0[i] = o;
    nn += norm2(o);
  }
  slice_norm(nn, partial, r, sh);
}

// Start of a cycle: beta = ||r||. For the first cycle the norm is also
// ||b||. Sets g = (beta, 0, ...), scales V_0 by 1/beta, deactivates
// right-hand sides already within tolerance and writes the status rows.
__global__ __launch_bounds__(kThreads) void cycle_start_kernel(
    GmresState st, int first, double tol, const double2* __restrict__ norm_partial,
    const int32_t* __restrict__ active_in, int32_t* __restrict__ active_out,
    float2* __restrict__ v0, int64_t n, int R, GmresStatusRow* __restrict__ status) {
  __shared__ double2 nrm[1];
  const int r = blockIdx.y;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  gather_partials(norm_partial, r, 1, 1, nrm);
  const double beta = sqrt(nrm[0].x);
  const double bn = first ? beta : st.bnorm[r];
  const double rel = bn > 0.0 ? beta / bn : 0.0;
  const int32_t was = first ? 1 : active_in[r];
  const int32_t on = (was && (beta == 0.0 || rel <= tol)) ? 0 : was;
  float2* v = v0 + (int64_t)r * n;
  slice_scale(v, v, on ? 1.0 / beta : 0.0, lo, hi);
  if (blockIdx.x != 0) return;
  double2* g = st.g + (int64_t)r * (st.m + 1);
  for (int i = threadIdx.x; i <= st.m; i += kThreads)
    g[i] = make_double2(i == 0 && on ? beta : 0.0, 0.0);
  if (threadIdx.x == 0) {
    const double res = was ? rel : st.res[r];
    const int32_t iters = first ? 0 : st.iters[r];
    st.bnorm[r] = bn;
    st.res[r] = res;
    st.iters[r] = iters;
    st.k[r] = 0;
    active_out[r] = on;
    put_status(&status[r], res, on, iters);
  }
}

// Solve H[0:k, 0:k] y = g[0:k] (upper triangular), one block per right-hand
// side: column by column from the last, a thread per row.
__global__ __launch_bounds__(kMaxRestart) void backsolve_kernel(GmresState st) {
  __shared__ double2 yi;
  const int r = blockIdx.x, c = threadIdx.x;
  const int m = st.m, ld = m + 1, k = st.k[r];
  const double2* H = st.H + (int64_t)r * m * ld;
  double2 s = c < k ? st.g[r * ld + c] : make_double2(0.0, 0.0);
  for (int i = k - 1; i >= 0; --i) {
    const double2 h = c <= i ? H[(int64_t)i * ld + c] : make_double2(0.0, 0.0);
    if (c == i) {
      const double dd = h.x * h.x + h.y * h.y;
      const double2 y = make_double2((s.x * h.x + s.y * h.y) / dd, (s.y * h.x - s.x * h.y) / dd);
      st.y[r * m + i] = y;
      yi = y;
    }
    __syncthreads();
    if (c < i) {
      const double2 p = cmul(h, yi);
      s.x -= p.x;
      s.y -= p.y;
    }
    __syncthreads();  // yi is written again
  }
}

// x[r][i] += sum_{c < k[r]} V_c[r][i] y[r][c]  (FP64 sum)
__global__ __launch_bounds__(kThreads) void combine_kernel(const float2* __restrict__ V,
                                                           int64_t vstride, GmresState st,
                                                           float2* __restrict__ x, int64_t n,
                                                           int R) {
  __shared__ double2 ys[kMaxRestart];
  const int r = blockIdx.y;
  const int k = st.k[r];
  for (int c = threadIdx.x; c < k; c += kThreads) ys[c] = st.y[r * st.m + c];
  __syncthreads();
  if (k == 0) return;
  int64_t lo, hi;
  slice_of(n, lo, hi);
  for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) {
    double2 s = f2d(x[(int64_t)r * n + i]);
#pragma unroll 8
    for (int c = 0; c < k; ++c) {
      const double2 p = cmul(f2d(V[(int64_t)c * vstride + (int64_t)r * n + i]), ys[c]);
      s.x += p.x;
      s.y += p.y;
    }
    x[(int64_t)r * n + i] = make_float2((float)s.x, (float)s.y);
  }
}

// conj(a)^T b of one pair of vectors: the slice's partial, then the sum.
__global__ __launch_bounds__(kThreads) void dot_kernel(const float2* __restrict__ a,
                                                       const float2* __restrict__ b, int64_t n,
                                                       double2* __restrict__ partial) {
  __shared__ double2 sh[kWaves][kColTile];
  int64_t lo, hi;
  slice_of(n, lo, hi);
  slice_dots(a, 0, 1, b, lo, hi, partial, 0, 1, sh);
}
__global__ __launch_bounds__(64) void dot_sum_kernel(const double2* __restrict__ partial,
                                                     int nblk, double2* __restrict__ out) {
  double2 s = make_double2(0.0, 0.0);
  for (int b = threadIdx.x; b < nblk; b += 64) {
    s.x += partial[b].x;
    s.y += partial[b].y;
  }
  s = wave_sum(s);
  if (threadIdx.x == 0) *out = s;
}

// dst = src * s[0]
__global__ __launch_bounds__(kThreads) void scale_kernel(float2* dst, const float2* src,
                                                         const double* __restrict__ s,
                                                         int64_t n) {
  int64_t lo, hi;
  slice_of(n, lo, hi);
  slice_scale(dst, src, s[0], lo, hi);
}

// v[i] = (u(2i), u(2i+1)), u uniform in [-1, 1) from a 64-bit counter hash
// (the finaliser of SplitMix64) of (seed, index): a reproducible start
// vector with no host transfer.
__device__ inline double hash_uniform(uint64_t seed, uint64_t i) {
  uint64_t z = seed + 0x9E3779B97F4A7C15ull * (i + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

__global__ __launch_bounds__(kThreads) void rand_fill_kernel(float2* __restrict__ v, int64_t n,
                                                             uint64_t seed) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads)
    v[i] = make_float2((float)hash_uniform(seed, 2 * i), (float)hash_uniform(seed, 2 * i + 1));
}

// dst = conj(src)
__global__ __launch_bounds__(kThreads) void conj_kernel(float2* __restrict__ dst,
                                                        const float2* __restrict__ src,
                                                        int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    const float2 v = src[i];
    dst[i] = make_float2(v.x, -v.y);
  }
}

// scale[0] = 1 / sqrt(nrm[0].x)  (0 for a zero vector)
__global__ void inv_norm_kernel(const double2* __restrict__ nrm, double* __restrict__ scale) {
  if (threadIdx.x == 0) {
    const double n2 = nrm[0].x;
    scale[0] = n2 > 0.0 ? 1.0 / sqrt(n2) : 0.0;
  }
}

unsigned slices(int64_t n) { return (unsigned)gmres_blocks(n); }

}  // namespace

int launch_gmres_step(const GmresState& st, const float2* V, int64_t vstride, int j, float2* w,
                      float2* vnext, double sr, double si, double tol, int64_t n, int R,
                      double2* partial, double2* partial2, const int32_t* active_in,
                      int32_t* active_out, GmresStatusRow* status, hipStream_t s) {
  const dim3 grid(slices(n), R), block(kThreads);
  const int ld = st.m + 1;  // of h1, h2 and the partials
  hipLaunchKernelGGL(orth_first_kernel, grid, block, 0, s, V, vstride, j, w, sr, si, n, R,
                     partial, ld);
  hipLaunchKernelGGL(orth_second_kernel, grid, block, 0, s, V, vstride, j + 1, w, n, R, partial,
                     partial2, ld, st.h1, ld);
  hipLaunchKernelGGL(orth_last_kernel, grid, block, 0, s, V, vstride, j + 1, w, n, R, partial2,
                     ld, partial, st.h2, ld);
  hipLaunchKernelGGL(next_column_kernel, grid, block, 0, s, st, j, tol, partial, active_in,
                     active_out, w, vnext, n, R, status);
  return (int)hipGetLastError();
}

int launch_gmres_begin(const float2* b, float2* x, float2* v0, int64_t n, int R,
                       double2* partial, hipStream_t s) {
  hipLaunchKernelGGL(begin_kernel, dim3(slices(n), R), dim3(kThreads), 0, s, b, x, v0, n, R,
                     partial);
  return (int)hipGetLastError();
}

int launch_gmres_residual(float2* v0, const float2* b, const float2* x, const float2* ax,
                          double sr, double si, int64_t n, int R, double2* partial,
                          hipStream_t s) {
  hipLaunchKernelGGL(residual_kernel, dim3(slices(n), R), dim3(kThreads), 0, s, v0, b, x, ax, sr,
                     si, n, R, partial);
  return (int)hipGetLastError();
}

int launch_gmres_cycle_start(const GmresState& st, int first, double tol, float2* v0, int64_t n,
                             int R, const double2* partial, const int32_t* active_in,
                             int32_t* active_out, GmresStatusRow* status, hipStream_t s) {
  hipLaunchKernelGGL(cycle_start_kernel, dim3(slices(n), R), dim3(kThreads), 0, s, st, first,
                     tol, partial, active_in, active_out, v0, n, R, status);
  return (int)hipGetLastError();
}

int launch_gmres_combine(const float2* V, int64_t vstride, const GmresState& st, float2* x,
                         int64_t n, int R, hipStream_t s) {
  hipLaunchKernelGGL(backsolve_kernel, dim3(R), dim3(kMaxRestart), 0, s, st);
  hipLaunchKernelGGL(combine_kernel, dim3(slices(n), R), dim3(kThreads), 0, s, V, vstride, st, x,
                     n, R);
  return (int)hipGetLastError();
}

int launch_gmres_dot(const float2* a, const float2* b, int64_t n, double2* partial, double2* out,
                     hipStream_t s) {
  const unsigned nb = slices(n);
  hipLaunchKernelGGL(dot_kernel, dim3(nb), dim3(kThreads), 0, s, a, b, n, partial);
  hipLaunchKernelGGL(dot_sum_kernel, dim3(1), dim3(64), 0, s, partial, (int)nb, out);
  return (int)hipGetLastError();
}

int launch_gmres_scale(float2* dst, const float2* src, const double* sc, int64_t n,
                       hipStream_t s) {
  hipLaunchKernelGGL(scale_kernel, dim3(slices(n)), dim3(kThreads), 0, s, dst, src, sc, n);
  return (int)hipGetLastError();
}

int launch_gmres_rand(float2* v, int64_t n, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(rand_fill_kernel, dim3(slices(n)), dim3(kThreads), 0, s, v, n, seed);
  return (int)hipGetLastError();
}

int launch_gmres_conj(float2* dst, const float2* src, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(conj_kernel, dim3(slices(n)), dim3(kThreads), 0, s, dst, src, n);
  return (int)hipGetLastError();
}

int launch_gmres_inv_norm(const double2* nrm, double* scale, hipStream_t s) {
  hipLaunchKernelGGL(inv_norm_kernel, dim3(1), dim3(64), 0, s, nrm, scale);
  return (int)hipGetLastError();
}

}  // namespace ubf
