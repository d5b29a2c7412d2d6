// FULL far sets as a discrete convolution over the lattices of the sites
// (FftGrid in plan.hpp), in FP64. Two kernels per product look at the box
// vectors, then five kernels each transform lines of the zero-padded lattices
// in LDS, for a group of scatterers and right-hand sides at a time (FftGroup):
//   fft_z:    box vectors -> [x][y][kz][component]          (x, y < sites)
//   fft_y:    -> [x][ky][kz][component]                     (x < sites)
//   fft_x:    transform along x, product with the spectrum of D (a symmetric
//             3 x 3 matrix per frequency), transform back, in place
//   ifft_y:   -> [x][y][kz][component]
//   ifft_z:   -> the first partial row of every box
// Only lines that can hold a value are touched, so the zero padding of an
// axis is never in memory before that axis is transformed.
//
// A transform's rounding errors are relative to the whole scatterer's field,
// those of a pair's own product to what reaches the test box, which may be
// far less. So everything here is FP64, and the boxes that even so would see
// mostly rounding errors are summed pair by pair: those that no strong box
// is far from (strong: at least 2^-24 of the scatterer's largest coefficient;
// Reach). The strong boxes are then within one of them on every axis, so
// there are at most 27. One box 10^4 times stronger than the others left its
// neighbours, which it does not reach, wrong by 5e-5 with FP32 transforms.
//
// The transforms are bound by memory (z, y) and by their own arithmetic and
// LDS traffic (x). On the 3,338-box shell (105^3 sites, transforms of 216;
// arrays of 114 and 235 MB, four passes each, and a spectrum of 124 MB): 42 +
// 59 + 211 + 63 + 45 us, 14 us to look at the box vectors, and the whole
// product 530 us against 6,290 pair by pair; 398 with FP32 transforms.
// Small lattices are bound by the launches, which a group shares: 8 shells of
// 762 boxes at n_d = 1 take 54 us (234 with five launches for each, 174 pair
// by pair), 16 masks of 200 at n_d = 3 in FP32 264 (613, 575).
#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>

#include "fft.hpp"

namespace ubf {
namespace {

constexpr int kThreads = 256;       // spectrum kernels
__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
// a * b + c
__device__ inline double2 cfma(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// a * (-i) forward, a * i backward
template <bool INV>
__device__ inline double2 mul_mi(double2 a) {
  return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// Discrete Fourier transform of R values in registers (in place, natural
// order): exp(-2 pi i jk / R), conjugated when INV.
template <int R, bool INV>
struct Butterfly;
template <bool INV>
struct Butterfly<2, INV> {
  static __device__ inline void run(double2 (&v)[2]) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};
template <bool INV>
struct Butterfly<3, INV> {
  static __device__ inline void run(double2 (&v)[3]) {
    const double s = 0.866025403784438647;
    const double2 t = cadd(v[1], v[2]), d = mul_mi<INV>(csub(v[1], v[2]));
    const double2 m = make_double2(fma(-0.5, t.x, v[0].x), fma(-0.5, t.y, v[0].y));
    v[0] = cadd(v[0], t);
    v[1] = make_double2(fma(s, d.x, m.x), fma(s, d.y, m.y));
    v[2] = make_double2(fma(-s, d.x, m.x), fma(-s, d.y, m.y));
  }
};
template <bool INV>
struct Butterfly<4, INV> {
  static __device__ inline void run(double2 (&v)[4]) {
    const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
    const double2 c = cadd(v[1], v[3]), d = mul_mi<INV>(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[1] = cadd(b, d);
    v[2] = csub(a, c);
    v[3] = csub(b, d);
  }
};
template <bool INV>
struct Butterfly<5, INV> {
  static __device__ inline void run(double2 (&v)[5]) {
    // cos and sin of 2 pi / 5 and 4 pi / 5
    const double c1 = 0.309016994374947424, c2 = -0.809016994374947424;
    const double s1 = 0.951056516295153572, s2 = 0.587785252292473129;
    const double2 a = cadd(v[1], v[4]), b = cadd(v[2], v[3]);
    const double2 d = mul_mi<INV>(csub(v[1], v[4])), e = mul_mi<INV>(csub(v[2], v[3]));
    const double2 p = make_double2(fma(c1, a.x, fma(c2, b.x, v[0].x)),
                                 fma(c1, a.y, fma(c2, b.y, v[0].y)));
    const double2 q = make_double2(fma(c2, a.x, fma(c1, b.x, v[0].x)),
                                 fma(c2, a.y, fma(c1, b.y, v[0].y)));
    const double2 r = make_double2(fma(s1, d.x, s2 * e.x), fma(s1, d.y, s2 * e.y));
    const double2 t = make_double2(fma(s2, d.x, -s1 * e.x), fma(s2, d.y, -s1 * e.y));
    v[0] = cadd(v[0], cadd(a, b));
    v[1] = cadd(p, r);
    v[4] = csub(p, r);
    v[2] = cadd(q, t);
    v[3] = csub(q, t);
  }
};
template <bool INV>
struct Butterfly<6, INV> {  // two of three, combined by twos
  static __device__ inline void run(double2 (&v)[6]) {
    double2 e[3] = {v[0], v[2], v[4]}, o[3] = {v[1], v[3], v[5]};
    Butterfly<3, INV>::run(e);
    Butterfly<3, INV>::run(o);
    const double s = 0.866025403784438647, sg = INV ? 1.0 : -1.0;
    o[1] = cmul(o[1], make_double2(0.5, sg * s));
    o[2] = cmul(o[2], make_double2(-0.5, sg * s));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      v[k] = cadd(e[k], o[k]);
      v[k + 3] = csub(e[k], o[k]);
    }
  }
};
template <bool INV>
struct Butterfly<8, INV> {
  static __device__ inline void run(double2 (&v)[8]) {
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    Butterfly<4, INV>::run(e);
    Butterfly<4, INV>::run(o);
    const double h = 0.707106781186547524, sg = INV ? 1.0 : -1.0;
    o[1] = cmul(o[1], make_double2(h, sg * h));
    o[2] = mul_mi<INV>(o[2]);
    o[3] = cmul(o[3], make_double2(-h, sg * h));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = cadd(e[k], o[k]);
      v[k + 4] = csub(e[k], o[k]);
    }
  }
};

// q = i / d for 0 <= i < 2^20 and inv = 1 / d: the quotient's rounding error
// stays below half a unit of i.
__device__ inline int fdiv(int i, float inv) { return (int)(((float)i + 0.5f) * inv); }

// A workgroup transforms `w` neighbouring lines of three components, taken as
// 3 w lines of one: value (position, line) is at position * w3 + line in LDS,
// line = 3 (line of sites) + component. Thread i has butterfly j = i / w3 of
// line i mod w3 in every stage, so what depends on the line is computed once,
// and neighbouring threads hold neighbouring values. (With the three
// components in one thread the indices and twiddle factors are shared, but
// the registers and the LDS leave two wavefronts to a SIMD: on 105^3 sites
// 385 + 118 + 118 us along x, y and back.)
struct Lane {
  int j, line, w3;
  __device__ Lane(int w) : w3(3 * w) {
    j = fdiv(threadIdx.x, 1.f / (float)w3);
    line = (int)threadIdx.x - j * w3;
  }
};

// One Stockham stage of radix R: butterfly j reads positions j + r L / R,
// applies the twiddle factors of k = j mod Ns and writes positions
// (j / Ns) Ns R + k + r Ns. load(position) and store(position, value) go to
// LDS or, for a transform's first and last stage, straight to memory; between
// the two every thread waits, so that one buffer serves both.
// A line of s sites is transformed at L >= 2 s - 1 positions: with an even
// radix (L even, s <= L / 2) the upper R / 2 inputs of the forward
// transform's first stage are the zero padding (HALF_IN), and the upper
// R / 2 outputs of the backward transform's last stage are not wanted
// (HALF_OUT).
template <int R, bool INV, bool TW, bool HALF_IN, bool HALF_OUT, class Load, class Store>
__device__ inline void stage(int L, int j, const double2* tw, int Ns, Load load, Store store) {
  constexpr int RI = HALF_IN && R % 2 == 0 ? R / 2 : R;
  constexpr int RO = HALF_OUT && R % 2 == 0 ? R / 2 : R;
  const int m = L / R;
  const bool on = j < m;
  double2 v[R];
  if (on) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = r < RI ? load(j + r * m) : make_double2(0.0, 0.0);
  }
  __syncthreads();
  if (on) {
    int o = j * R;
    if (TW) {
      const int q = fdiv(j, 1.f / (float)Ns), k = j - q * Ns;
      const int step = k * (m / Ns);
      o = q * Ns * R + k;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        double2 t = tw[r * step];
        if (INV) t.y = -t.y;
        v[r] = cmul(v[r], t);
      }
    }
    Butterfly<R, INV>::run(v);
#pragma unroll
    for (int r = 0; r < RO; ++r) store(o + r * Ns, v[r]);
  }
  __syncthreads();
}

template <bool INV, bool TW, bool HALF_IN, bool HALF_OUT, class Load, class Store>
__device__ inline void stage_of(int R, int L, int j, const double2* tw, int Ns, Load load,
                                Store store) {
  switch (R) {  // uniform
    case 2: stage<2, INV, TW, HALF_IN, HALF_OUT>(L, j, tw, Ns, load, store); break;
    case 3: stage<3, INV, TW, HALF_IN, HALF_OUT>(L, j, tw, Ns, load, store); break;
    case 4: stage<4, INV, TW, HALF_IN, HALF_OUT>(L, j, tw, Ns, load, store); break;
    case 5: stage<5, INV, TW, HALF_IN, HALF_OUT>(L, j, tw, Ns, load, store); break;
    case 6: stage<6, INV, TW, HALF_IN, HALF_OUT>(L, j, tw, Ns, load, store); break;
    default: stage<8, INV, TW, HALF_IN, HALF_OUT>(L, j, tw, Ns, load, store); break;
  }
}

// A whole transform in the buffer `a`: the first stage takes its values from
// load, the last one gives them to store (either may be the buffer). The
// twiddle factors and the buffer may have been written just before; ends with
// a barrier. An axis of length 1 passes its values through.
template <bool INV, class Load, class Store>
__device__ inline void transform(const FftAxis& ax, const Lane& t, const double2* tw, double2* a,
                                 Load load, Store store) {
  const int L = ax.L, n = ax.stages;
  double2* mine = a + t.line;
  const int w3 = t.w3;
  auto get = [mine, w3](int pos) { return mine[pos * w3]; };
  auto put = [mine, w3](int pos, double2 v) { mine[pos * w3] = v; };
  __syncthreads();
  if (n == 0) {
    double2 v = make_double2(0.0, 0.0);
    if (t.j == 0) v = load(0);
    __syncthreads();
    if (t.j == 0) store(0, v);
    __syncthreads();
    return;
  }
  if (n == 1) {
    stage_of<INV, false, !INV, INV>(ax.radix[0], L, t.j, tw, 1, load, store);
    return;
  }
  stage_of<INV, false, !INV, false>(ax.radix[0], L, t.j, tw, 1, load, put);
  int Ns = ax.radix[0];
  for (int s = 1; s + 1 < n; ++s) {
    stage_of<INV, true, false, false>(ax.radix[s], L, t.j, tw, Ns, get, put);
    Ns *= ax.radix[s];
  }
  stage_of<INV, true, false, INV>(ax.radix[n - 1], L, t.j, tw, Ns, get, store);
}

__device__ inline void load_twiddles(double2* tw, const double2* __restrict__ all, const FftAxis& ax) {
  for (int i = threadIdx.x; i < ax.L; i += blockDim.x) tw[i] = all[ax.tw + i];
}

// Box vectors of one right-hand side, in the form stage 1 wrote them.
struct Source {
  const float* P;
  const float* box_scale;  // FP16 form
  int mode, kh, khb, nd;   // mode 0 FP32, 1 BF16 parts, 2 FP16 parts
  int64_t stride;          // floats from one right-hand side to the next
  int64_t n_box;
  __device__ inline void select(int rhs) {
    P += rhs * stride;
    if (mode == 2) box_scale += rhs * n_box;
  }
  __device__ inline double2 at(int box, int u) const {
    if (mode == 0) {
      const float* b = P + (int64_t)box * 2 * kh;
      return make_double2(b[u], b[kh + u]);
    }
    const int at = khb == 192 ? (u % 3) * 64 + u / 3 : u;  // pos16 of stage 1
    const unsigned short* q = reinterpret_cast<const unsigned short*>(P + (int64_t)box * 2 * khb) +
                              32 * (at >> 3) + (at & 7);
    if (mode == 1) {
      auto f = [](unsigned short b) { return (double)__uint_as_float((unsigned)b << 16); };
      return make_double2(f(q[0]) + f(q[16]), f(q[8]) + f(q[24]));
    }
    auto f = [](unsigned short b) { return (double)__half2float(__ushort_as_half(b)); };
    const double sc = box_scale[box];  // a power of two
    return make_double2((f(q[0]) + f(q[16])) * sc, (f(q[8]) + f(q[24])) * sc);
  }
};

extern __shared__ double2 lds[];

// Workgroups are dealt round robin to the 8 XCDs: give each XCD a contiguous
// range, so that workgroups sharing memory lines share an L2. The grid is a
// multiple of 8; positions past the work are the caller's to skip.
__device__ inline int xcd_block() {
  return (int)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

// The task whose part of launch `kind` holds workgroup `block`, of n.
__device__ inline const FftTask& task_of(const FftTask* __restrict__ tasks, int n, int kind,
                                         int block) {
  int lo = 0;
  while (n > 1) {  // uniform
    const int half = n / 2;
    if (tasks[lo + half].first[kind] <= block) lo += half;
    n -= half;
  }
  return tasks[lo];
}

// ---------------------------------------------------- what reaches a box

// D(R), R = step (dx, dy, dz), in FP64: xx, yy, zz, xy, xz, yz.
__device__ void green(int dx, int dy, int dz, double step, double k, double eta,
                      double2 (&D)[6]) {
  const double R[3] = {step * dx, step * dy, step * dz};
  const double r2 = R[0] * R[0] + R[1] * R[1] + R[2] * R[2];
  const double r = sqrt(r2), kr = k * r, ik = 1.0 / kr;
  double sn, cs;
  sincos(kr, &sn, &cs);
  // psi = -j k eta e^{-j kr} / (4 pi r)
  const double f = k * eta / (4.0 * 3.14159265358979323846 * r);
  const double pr = -f * sn, pi = -f * cs;
  const int pa[6] = {0, 1, 2, 0, 0, 1}, pb[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    const double rr = R[pa[e]] * R[pb[e]] / r2, iso = e < 3 ? 1.0 : 0.0;
    const double tr = iso * (1.0 - ik * ik) - rr * (1.0 - 3.0 * ik * ik);
    const double ti = -iso * ik + rr * 3.0 * ik;
    D[e] = make_double2(pr * tr - pi * ti, pr * ti + pi * tr);
  }
}

// Largest real or imaginary part of every box vector of a lattice, infinity
// where one is not finite; a wavefront per box.
__global__ __launch_bounds__(kThreads) void norm_kernel(Source src, const int4* __restrict__ cells,
                                                        int nu, float* __restrict__ norm) {
  src.select(blockIdx.y);
  const int64_t box = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (box >= src.n_box || cells[box].w < 0) return;
  const int lane = threadIdx.x & 63;
  double m = 0.0;
  bool finite = true;
  for (int u = lane; u < nu; u += 64) {
    const double2 v = src.at((int)box, u);
    finite = finite && isfinite(v.x) && isfinite(v.y);
    m = fmax(m, fmax(fabs(v.x), fabs(v.y)));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  finite = __all(finite);
  if (lane == 0)
    norm[blockIdx.y * src.n_box + box] =
        finite ? (float)fmin(m, (double)FLT_MAX) : __builtin_inff();
}

// Bounding grid of some boxes.
struct Bounds {
  int lo[3], hi[3];
  __device__ inline void clear() {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = 0x7fffffff;
      hi[d] = -1;
    }
  }
  __device__ inline void add(int x, int y, int z) {
    lo[0] = min(lo[0], x);
    lo[1] = min(lo[1], y);
    lo[2] = min(lo[2], z);
    hi[0] = max(hi[0], x);
    hi[1] = max(hi[1], y);
    hi[2] = max(hi[2], z);
  }
  __device__ inline bool empty() const { return lo[0] > hi[0]; }
  // None of them is far from (x, y, z): all are within one of it on every
  // axis (true where there are none).
  __device__ inline bool near(int x, int y, int z) const {
    return lo[0] >= x - 1 && hi[0] <= x + 1 && lo[1] >= y - 1 && hi[1] <= y + 1 &&
           lo[2] >= z - 1 && hi[2] <= z + 1;
  }
};

// The strong boxes of one lattice and right-hand side, and those whose
// coefficients are not all finite. The latter are left out of the transforms,
// and the boxes that one of them is far from get NaN, as from its pairs.
// Without weak ones the boxes that no strong box is far from get zero.
struct Reach {
  Bounds strong, bad;
  int weak;  // whether any box is neither strong nor zero (nor bad)
  // The box (x, y, z), which no strong box is far from, among the at most 27
  // such boxes.
  __device__ inline int slot(int x, int y, int z) const {
    return ((x - strong.hi[0] + 1) * 3 + (y - strong.hi[1] + 1)) * 3 + (z - strong.hi[2] + 1);
  }
};

static_assert(sizeof(Reach) == kReachBytes && alignof(Reach) <= 4, "fft_scratch_bytes");

// Per lattice and right-hand side 27 x `splits` workgroups. Each finds the
// strong boxes (the first one also leaves them for ifft_z). Where weak ones
// are left, workgroup (slot, split) takes a box that no strong box is far from
// and sums, for every kReachParts-th source box, the site pairs that the
// convolution stands for: a few source boxes at a time, D once per lattice
// difference of the box pair, then a thread per output coefficient and share
// of the source sites. ifft_z adds the parts, in order whatever `splits` is.
// Reads 4 bytes per box in the ordinary case (8 us, latency). With one of
// 3,338 boxes 10^9 times the others the product takes 0.73 ms (11.7 with D for
// each site pair and one workgroup per box; pair by pair 6.5), of 314 111 us
// (1,232; 133).
constexpr int kReachThreads = 512;
__global__ __launch_bounds__(kReachThreads) void reach_kernel(
    Source src, const int2* __restrict__ map, const int4* __restrict__ cells,
    const int4* __restrict__ grids, const float* __restrict__ norm, double step, double k,
    double eta, int nu, Reach* __restrict__ reach, double2* __restrict__ parts, int splits) {
  constexpr int kSources = 3 * kReachThreads;  // most coefficients of the boxes at a time
  __shared__ float wave_max[kReachThreads / 64];
  __shared__ Reach all;
  __shared__ double2 D[kReachThreads][6];  // [box][difference]; then the threads' sums
  __shared__ double2 P[kSources];          // [box][coefficient]
  __shared__ int at_site[kReachThreads];   // (box, source site) q: its part of the place in D
  const int rhs = blockIdx.z, t = threadIdx.x;
  src.select(rhs);
  norm += rhs * src.n_box;
  const int4 ga = grids[2 * blockIdx.y], gb = grids[2 * blockIdx.y + 1];
  const int first = ga.x, count = ga.y;           // its boxes
  const int nx = gb.x, ny = gb.y, nz = gb.z;
  const int64_t cell0 = ((int64_t)ga.w << 32) | (unsigned)ga.z;
  float m = 0.f;
#pragma unroll 8
  for (int i = t; i < count; i += kReachThreads) {
    const float v = norm[first + i];
    if (v <= FLT_MAX) m = fmaxf(m, v);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((t & 63) == 0) wave_max[t >> 6] = m;
  if (t == 0) {
    all.strong.clear();
    all.bad.clear();
    all.weak = 0;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kReachThreads / 64; ++w) m = fmaxf(m, wave_max[w]);
  const float bar = m * 0x1p-24f;
  Reach mine;
  mine.strong.clear();
  mine.bad.clear();
  bool weak = false;
#pragma unroll 4
  for (int i = t; i < count; i += kReachThreads) {
    const float v = norm[first + i];
    const int4 c = cells[first + i];
    if (!(v <= FLT_MAX))
      mine.bad.add(c.x, c.y, c.z);
    else if (v > 0.f && v >= bar)
      mine.strong.add(c.x, c.y, c.z);
    else
      weak = weak || v > 0.f;
  }
  if (weak) all.weak = 1;  // every writer writes the same
  auto join = [t](Bounds& to, Bounds& b) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        b.lo[d] = min(b.lo[d], __shfl_xor(b.lo[d], o, 64));
        b.hi[d] = max(b.hi[d], __shfl_xor(b.hi[d], o, 64));
      }
      if ((t & 63) == 0) {
        atomicMin(&to.lo[d], b.lo[d]);
        atomicMax(&to.hi[d], b.hi[d]);
      }
    }
  };
  join(all.strong, mine.strong);
  if (__any(!mine.bad.empty())) join(all.bad, mine.bad);
  __syncthreads();
  if (blockIdx.x == 0 && t == 0) reach[rhs * gridDim.y + blockIdx.y] = all;
  const Bounds strong = all.strong;
  if (strong.empty() || !all.weak) return;
  const int slot = blockIdx.x / splits;
  const int x = strong.hi[0] - 1 + slot / 9, y = strong.hi[1] - 1 + slot / 3 % 3,
            z = strong.hi[2] - 1 + slot % 3;
  if (x < 0 || y < 0 || z < 0 || x >= nx || y >= ny || z >= nz || !strong.near(x, y, z) ||
      !all.bad.near(x, y, z) || map[cell0 + ((int64_t)x * ny + y) * nz + z].y < 0)
    return;
  const int nd = src.nd, nd2 = nd * nd, nd3 = nd2 * nd, span = 2 * nd - 1, span3 = span * span * span;
  const int boxes = kReachThreads / span3;  // source boxes at a time: 512, 18, 4, 1
  // this thread's difference of a source box, and output coefficient u with
  // its share of the source sites
  const int db = t / span3, dd = t - db * span3;
  const int ox = dd / (span * span) - (nd - 1), oy = dd / span % span - (nd - 1),
            oz = dd % span - (nd - 1);
  const int shares = kReachThreads / nu, share = t / nu, u = t - share * nu;
  const int l = u / 3, al = u - 3 * l;
  const int e0 = al == 0 ? 0 : 2 + al, e1 = al == 0 ? 3 : (al == 1 ? 1 : 5),
            e2 = al == 2 ? 2 : 4 + al;  // (al, x), (al, y), (al, z)
  // difference l - s of the sites: (3 digits of l) - (of s) + nd - 1 each, base span
  auto digits = [=](int i) { return (i / nd2 * span + i / nd % nd) * span + i % nd; };
  if (t < boxes * nd3) at_site[t] = t / nd3 * span3 - digits(t % nd3);
  const int at_l = digits(l) + ((nd - 1) * span + nd - 1) * span + nd - 1;
  parts += (((int64_t)rhs * gridDim.y + blockIdx.y) * 27 + slot) * kReachParts * nu;
  for (int part = blockIdx.x - slot * splits; part < kReachParts; part += splits) {
    double2 E = make_double2(0.0, 0.0);
    for (int base = part; base < count; base += kReachParts * boxes) {
      __syncthreads();  // every thread is done with the last boxes
      for (int e = t; e < boxes * nu; e += kReachThreads) {
        const int b = e / nu, i = base + kReachParts * b;
        const bool on = i < count && norm[first + min(i, count - 1)] <= FLT_MAX;
        P[e] = on ? src.at(first + i, e - b * nu) : make_double2(0.0, 0.0);
      }
      if (db < boxes) {
        const int i = min(base + kReachParts * db, count - 1);
        const int4 c = cells[first + i];
        const int dx = nd * (x - c.x) + ox, dy = nd * (y - c.y) + oy, dz = nd * (z - c.z) + oz;
        double2 v[6];
        const bool on = norm[first + i] > 0.f && max(abs(dx), max(abs(dy), abs(dz))) >= 2 * nd;
        if (on) green(dx, dy, dz, step, k, eta, v);
#pragma unroll
        for (int e = 0; e < 6; ++e) D[t][e] = on ? v[e] : make_double2(0.0, 0.0);
      }
      __syncthreads();
      if (share < shares)
        for (int q = share; q < boxes * nd3; q += shares) {
          const double2* d = D[at_l + at_site[q]];
          const double2* p = P + 3 * q;
          E = cfma(d[e0], p[0], cfma(d[e1], p[1], cfma(d[e2], p[2], E)));
        }
    }
    __syncthreads();
    double2* sums = D[0];
    sums[t] = E;
    __syncthreads();
    for (int left = shares; left > 1;) {
      const int half = (left + 1) / 2;
      if (share < left - half) sums[t] = cadd(sums[t], sums[t + half * nu]);
      __syncthreads();
      left = half;
    }
    if (t < nu) parts[part * nu + t] = sums[t];
  }
}

// A workgroup of the z transforms: w of the n_d lines (site rows my) of a
// column of boxes (x, y) and a site plane mx of it.
struct ZBlock {
  int w, bx, by, mx, my0, X;  // X: sites along x
  __device__ ZBlock(const FftTask& t, int nd) : w(t.lines[0]) {
    const int groups = nd / w, row = t.g.n[0] * nd * groups;
    const int b = (int)blockIdx.x - t.first[0];
    by = b / row;
    X = (b - by * row) / groups;
    my0 = (b - by * row - X * groups) * w;
    bx = X / nd;
    mx = X - bx * nd;
  }
};

__global__ __launch_bounds__(kMaxFftThreads) void fft_z_kernel(
    Source src, const int2* __restrict__ maps, const FftTask* __restrict__ tasks, int n_tasks,
    const double2* __restrict__ twiddles, double2* __restrict__ scratch, int64_t scratch_rhs,
    const float* __restrict__ norm) {
  src.select(blockIdx.y);
  norm += blockIdx.y * src.n_box;
  const FftTask& task = task_of(tasks, n_tasks, 0, blockIdx.x);
  const FftGrid& g = task.g;
  const ZBlock blk(task, src.nd);
  double2* out = scratch + blockIdx.y * scratch_rhs + task.z;
  const int nd = src.nd, w = blk.w, L = g.ax[2].L, row = 3 * nd * nd;
  double2 *a = lds, *tw = a + 3 * L * w;
  const int by = blk.by, X = blk.X, my0 = blk.my0, bx = blk.bx, mx = blk.mx;
  const int2* col = maps + g.map + ((int64_t)bx * g.n[1] + by) * g.n[2];
  load_twiddles(tw, twiddles, g.ax[2]);
  const int part = 3 * nd * w;  // a box's values here
  const float inv_part = 1.f / part, inv_line = 1.f / (3 * nd);
  bool any = false;
  for (int i = threadIdx.x; i < g.n[2] * part; i += blockDim.x) {
    const int bz = fdiv(i, inv_part), v = i - bz * part;   // v = (line nd + mz) 3 + alpha
    const int line = fdiv(v, inv_line), t = v - line * 3 * nd;  // t = 3 mz + alpha
    const int mz = t / 3, al = t - 3 * mz;
    const int box = col[bz].x;
    double2 z = make_double2(0.0, 0.0);
    if (box >= 0) {
      if (norm[box] <= FLT_MAX) z = src.at(box, mx * row + my0 * 3 * nd + v);
      any = true;
    }
    a[((bz * nd + mz) * w + line) * 3 + al] = z;
  }
  const int s = g.s[2];
  double2* o = out + ((int64_t)X * g.s[1] + by * nd + my0) * L * 3;
  if (!__syncthreads_or(any)) {  // a column without boxes transforms to zeros
    for (int i = threadIdx.x; i < 3 * L * w; i += blockDim.x) o[i] = make_double2(0.0, 0.0);
    return;
  }
  const Lane t(w);
  const int line = t.line / 3, al = t.line - 3 * line;
  o += 3 * line * L + al;
  transform<false>(
      g.ax[2], t, tw, a,
      [&](int pos) { return pos < s ? a[pos * t.w3 + t.line] : make_double2(0.0, 0.0); },
      [&](int pos, double2 v) { o[3 * pos] = v; });
}

// y transforms of w neighbouring lines (x, kz with kz fastest); forward from
// s to L positions, backward from L to s.
template <bool INV>
__global__ __launch_bounds__(kMaxFftThreads) void fft_y_kernel(
    const FftTask* __restrict__ tasks, int n_tasks, int blocks,
    const double2* __restrict__ twiddles, double2* __restrict__ scratch, int64_t scratch_rhs) {
  const int block = xcd_block();
  if (block >= blocks) return;
  const FftTask& task = task_of(tasks, n_tasks, 1, block);
  const FftGrid& g = task.g;
  scratch += blockIdx.y * scratch_rhs;
  const int w = task.lines[1], L = g.ax[1].L, s = g.s[1], Lz = g.ax[2].L;
  const int nin = INV ? L : s, nout = INV ? s : L;
  double2 *a = lds, *tw = a + 3 * L * w;
  const int all = g.s[0] * Lz, l0 = (block - task.first[1]) * w;
  load_twiddles(tw, twiddles, g.ax[1]);
  const Lane t(w);
  const int l = l0 + t.line / 3;
  const bool live = l < all;  // line l = (x, kz)
  const int x = l / Lz, kz = l - x * Lz, at = 3 * kz + t.line % 3;
  const double2* p = scratch + (INV ? task.yz : task.z) + (int64_t)x * nin * Lz * 3 + at;
  double2* o = scratch + (INV ? task.z : task.yz) + (int64_t)x * nout * Lz * 3 + at;
  transform<INV>(
      g.ax[1], t, tw, a,
      [&](int pos) { return live && pos < nin ? p[3 * pos * Lz] : make_double2(0.0, 0.0); },
      [&](int pos, double2 v) {
        if (live && pos < nout) o[3 * pos * Lz] = v;
      });
}

// Along x: transform, product with the spectrum, transform back, for w (a
// power of two) neighbouring lines (ky, kz). The spectrum is stored for
// frequencies 0 .. L/2 per axis; D is even along its two equal axes and odd
// along each of two different ones, so a frequency mirrored along some axes
// (s = -1) has component (alpha, beta) times s_alpha s_beta. For the product a
// thread takes the three components of every (blockDim / w)-th position of a
// line.
__global__ __launch_bounds__(kMaxFftThreads) void fft_x_kernel(
    const FftTask* __restrict__ tasks, int n_tasks, int blocks,
    const double2* __restrict__ twiddles, const double2* __restrict__ spectra,
    double2* __restrict__ scratch, int64_t scratch_rhs) {
  const int block = xcd_block();
  if (block >= blocks) return;
  const FftTask& task = task_of(tasks, n_tasks, 2, block);
  const FftGrid& g = task.g;
  const FftAxis& ax = g.ax[0];
  double2* data = scratch + blockIdx.y * scratch_rhs + task.yz;
  const double2* spec = spectra + g.spec;
  const int w = task.lines[2], L = ax.L, s = g.s[0], Ly = g.ax[1].L, Lz = g.ax[2].L;
  double2 *a = lds, *tw = a + 3 * L * w;
  const int plane = Ly * Lz, l0 = (block - task.first[2]) * w;
  load_twiddles(tw, twiddles, ax);
  const Lane t(w);
  const bool live = l0 + t.line / 3 < plane;
  double2* p = data + (int64_t)l0 * 3 + t.line;
  const int64_t step = 3LL * plane;
  transform<false>(
      ax, t, tw, a,
      [&](int pos) { return live && pos < s ? p[pos * step] : make_double2(0.0, 0.0); },
      [&](int pos, double2 v) { a[pos * t.w3 + t.line] = v; });
  {
    const int line = threadIdx.x & (w - 1);
    const int l = min(l0 + line, plane - 1), ky = l / Lz, kz = l - ky * Lz;
    const int hy = Ly / 2 + 1, hz = Lz / 2 + 1;
    const bool my = 2 * ky > Ly, mz = 2 * kz > Lz;
    const double2* kyz = spec + 6 * ((int64_t)(my ? Ly - ky : ky) * hz + (mz ? Lz - kz : kz));
    const int64_t kstep = 6LL * hy * hz;
    const double syz = my == mz ? 1.0 : -1.0;
    for (int pos = threadIdx.x / w; pos < L; pos += blockDim.x / w) {
      const bool mx = 2 * pos > L;
      const double2* k = kyz + (mx ? L - pos : pos) * kstep;
      const double sxy = mx == my ? 1.0 : -1.0, sxz = mx == mz ? 1.0 : -1.0;
      const double2 xx = k[0], yy = k[1], zz = k[2];
      const double2 xy = make_double2(k[3].x * sxy, k[3].y * sxy);
      const double2 xz = make_double2(k[4].x * sxz, k[4].y * sxz);
      const double2 yz = make_double2(k[5].x * syz, k[5].y * syz);
      double2* f = a + 3 * (pos * w + line);
      const double2 u = f[0], v = f[1], z = f[2];
      f[0] = cfma(xx, u, cfma(xy, v, cmul(xz, z)));
      f[1] = cfma(xy, u, cfma(yy, v, cmul(yz, z)));
      f[2] = cfma(xz, u, cfma(yz, v, cmul(zz, z)));
    }
  }
  transform<true>(
      ax, t, tw, a, [&](int pos) { return a[pos * t.w3 + t.line]; },
      [&](int pos, double2 v) {
        if (live && pos < s) p[pos * step] = v;
      });
}

// Backward z transforms into the boxes' rows: the lines of fft_z_kernel. The
// rows of boxes that no strong box is far from are the sum of reach_kernel's
// parts, or zero without weak boxes; those that a box without finite
// coefficients is far from are NaN.
__global__ __launch_bounds__(kMaxFftThreads) void ifft_z_kernel(
    const int2* __restrict__ maps, const FftTask* __restrict__ tasks, int n_tasks,
    const double2* __restrict__ twiddles, const double2* __restrict__ scratch,
    int64_t scratch_rhs, float* __restrict__ part, int nd, int kh, int64_t part_rhs,
    const Reach* __restrict__ reach, const double2* __restrict__ parts, int n_grid) {
  const FftTask& task = task_of(tasks, n_tasks, 0, blockIdx.x);
  const FftGrid& g = task.g;
  const ZBlock blk(task, nd);
  const double2* in = scratch + blockIdx.y * scratch_rhs + task.z;
  part += blockIdx.y * part_rhs;
  const Reach of = reach[blockIdx.y * n_grid + task.index];
  const int L = g.ax[2].L, w = blk.w, row = 3 * nd * nd, nu = row * nd, s = g.s[2];
  double2 *a = lds, *tw = a + 3 * L * w;
  const int by = blk.by, X = blk.X, my0 = blk.my0, bx = blk.bx, mx = blk.mx;
  const int2* col = maps + g.map + ((int64_t)bx * g.n[1] + by) * g.n[2];
  bool any = false;
  for (int i = threadIdx.x; i < g.n[2]; i += blockDim.x) any = any || col[i].y >= 0;
  if (!__syncthreads_or(any)) return;  // a column without rows
  load_twiddles(tw, twiddles, g.ax[2]);
  const Lane t(w);
  const int line = t.line / 3;
  const double2* p =
      in + ((int64_t)X * g.s[1] + by * nd + my0 + line) * L * 3 + (t.line - 3 * line);
  transform<true>(
      g.ax[2], t, tw, a, [&](int pos) { return p[3 * pos]; },
      [&](int pos, double2 v) {
        if (pos < s) a[pos * t.w3 + t.line] = v;
      });
  const int values = 3 * nd * w;  // a box's values here
  const float inv_values = 1.f / values, inv_line = 1.f / (3 * nd);
  for (int i = threadIdx.x; i < g.n[2] * values; i += blockDim.x) {
    const int bz = fdiv(i, inv_values), v = i - bz * values;
    const int ln = fdiv(v, inv_line), q = v - ln * 3 * nd;
    const int mz = q / 3, al = q - 3 * mz;
    const int at = col[bz].y, u = mx * row + my0 * 3 * nd + v;
    if (at < 0) continue;
    double2 z = a[((bz * nd + mz) * w + ln) * 3 + al];
    if (!of.bad.near(bx, by, bz)) {
      z.x = z.y = __builtin_nan("");
    } else if (of.strong.near(bx, by, bz)) {
      z = make_double2(0.0, 0.0);
      if (!of.strong.empty() && of.weak) {
        const double2* q = parts + (((int64_t)blockIdx.y * n_grid + task.index) * 27 +
                                    of.slot(bx, by, bz)) * kReachParts * nu + u;
        for (int k = 0; k < kReachParts; ++k) z = cadd(z, q[k * nu]);
      }
    }
    float* e = part + (int64_t)at * 2 * kh + u;  // [Er | Ei]
    e[0] = (float)z.x;
    e[nu] = (float)z.y;
  }
}

// ---------------------------------------------------------------- spectrum

// Weight of the value at distance d for frequency kf of one axis of a real
// even (cosine) or odd (sine) sequence of period L.
__device__ inline double axis_weight(bool odd, int d, int kf, int L) {
  if (d == 0) return odd ? 0.0 : 1.0;
  const double a = 2.0 * (double)((int64_t)d * kf % L) / L;
  return 2.0 * (odd ? sinpi(a) : cospi(a));
}
__device__ inline bool odd_axis(int e, int axis) {
  return e >= 3 && axis != 5 - e;  // xy is even along z, xz along y, yz along x
}

// Along z: T[x][y][kz] = sum_z weight D, one workgroup per (x, y).
__global__ __launch_bounds__(kThreads) void spectrum_z_kernel(FftGrid g, int e, double step,
                                                              double k, double eta, int nd,
                                                              double2* __restrict__ T) {
  __shared__ double2 D[kMaxFftLength];
  const int x = blockIdx.x, y = blockIdx.y, L = g.ax[2].L, h = L / 2 + 1;
  for (int z = threadIdx.x; z < g.s[2]; z += kThreads)
  {
    double2 v[6];
    const bool kept = max(x, max(y, z)) >= 2 * nd;  // the rest: masked operators
    if (kept) green(x, y, z, step, k, eta, v);
    D[z] = kept ? v[e] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int kz = threadIdx.x; kz < h; kz += kThreads) {
    double2 s = make_double2(0.0, 0.0);
    for (int z = 0; z < g.s[2]; ++z) {
      const double w = axis_weight(odd_axis(e, 2), z, kz, L);
      s.x = fma(w, D[z].x, s.x);
      s.y = fma(w, D[z].y, s.y);
    }
    T[((int64_t)x * g.s[1] + y) * h + kz] = s;
  }
}

// Along y: U[x][ky][kz] from T[x][y][kz]; workgroups over (x, ky).
__global__ __launch_bounds__(kThreads) void spectrum_y_kernel(FftGrid g, int e,
                                                              const double2* __restrict__ T,
                                                              double2* __restrict__ U) {
  __shared__ double w[kMaxFftLength];
  const int x = blockIdx.x, ky = blockIdx.y, L = g.ax[1].L, hy = L / 2 + 1;
  const int hz = g.ax[2].L / 2 + 1;
  for (int y = threadIdx.x; y < g.s[1]; y += kThreads) w[y] = axis_weight(odd_axis(e, 1), y, ky, L);
  __syncthreads();
  for (int kz = threadIdx.x; kz < hz; kz += kThreads) {
    double2 s = make_double2(0.0, 0.0);
    for (int y = 0; y < g.s[1]; ++y) {
      const double2 t = T[((int64_t)x * g.s[1] + y) * hz + kz];
      s.x = fma(w[y], t.x, s.x);
      s.y = fma(w[y], t.y, s.y);
    }
    U[((int64_t)x * hy + ky) * hz + kz] = s;
  }
}

// Along x into the spectrum, with the 1 / (Lx Ly Lz) of the backward
// transforms; a pair of odd axes carries (-j)^2 = -1.
__global__ __launch_bounds__(kThreads) void spectrum_x_kernel(FftGrid g, int e,
                                                              const double2* __restrict__ U,
                                                              double2* __restrict__ spec) {
  __shared__ double w[kMaxFftLength];
  const int kx = blockIdx.x, ky = blockIdx.y, L = g.ax[0].L;
  const int hy = g.ax[1].L / 2 + 1, hz = g.ax[2].L / 2 + 1;
  for (int x = threadIdx.x; x < g.s[0]; x += kThreads) w[x] = axis_weight(odd_axis(e, 0), x, kx, L);
  __syncthreads();
  const double f = (e >= 3 ? -1.0 : 1.0) / ((double)L * g.ax[1].L * g.ax[2].L);
  for (int kz = threadIdx.x; kz < hz; kz += kThreads) {
    double2 s = make_double2(0.0, 0.0);
    for (int x = 0; x < g.s[0]; ++x) {
      const double2 t = U[((int64_t)x * hy + ky) * hz + kz];
      s.x = fma(w[x], t.x, s.x);
      s.y = fma(w[x], t.y, s.y);
    }
    // six components side by side: xx, yy, zz, xy, xz, yz
    spec[6 * (((int64_t)kx * hy + ky) * hz + kz) + e] = make_double2(s.x * f, s.y * f);
  }
}

// Kernel launch with optional events at its start and end.
template <typename... Args>
void launch(void (*kernel)(Args...), dim3 grid, dim3 block, size_t shared, hipStream_t s,
            hipEvent_t start, hipEvent_t stop, Args... args) {
  if (start || stop)
    hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)shared, s, start, stop, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, (uint32_t)shared, s, args...);
}

}  // namespace

int launch_fft_spectra(const Plan& p, hipStream_t s) {
  const double step = p.a / p.n_d;
  for (size_t i = 0; i < p.fft.size(); ++i) {
    const FftGrid& g = p.fft[i];
    bool done = false;
    for (size_t o = 0; o < i; ++o) done = done || p.fft[o].spec == g.spec;
    if (done) continue;
    double2* T = reinterpret_cast<double2*>(p.d_fft);
    const int hx = g.ax[0].L / 2 + 1, hy = g.ax[1].L / 2 + 1, hz = g.ax[2].L / 2 + 1;
    double2* U = T + (int64_t)g.s[0] * g.s[1] * hz;
    double2* spec = reinterpret_cast<double2*>(p.d_fft_spec) + g.spec;
    for (int e = 0; e < 6; ++e) {
      hipLaunchKernelGGL(spectrum_z_kernel, dim3(g.s[0], g.s[1]), dim3(kThreads), 0, s, g, e,
                         step, p.k, p.eta, p.n_d, T);
      hipLaunchKernelGGL(spectrum_y_kernel, dim3(g.s[0], hy), dim3(kThreads), 0, s, g, e, T, U);
      hipLaunchKernelGGL(spectrum_x_kernel, dim3(hx, hy), dim3(kThreads), 0, s, g, e, U, spec);
    }
  }
  return (int)hipGetLastError();
}

int launch_fft(const Plan& p, const float* P, float* part, int nrhs, hipStream_t s,
               hipEvent_t start, hipEvent_t stop) {
  const double2* tw = reinterpret_cast<const double2*>(p.d_fft_tw);
  const double2* spectra = reinterpret_cast<const double2*>(p.d_fft_spec);
  const int64_t part_rhs = p.rest->n_pairs() * p.pstride();
  const int n_grid = (int)p.fft.size();
  double2* lattices = reinterpret_cast<double2*>(p.d_fft);
  double2* parts = lattices + fft_scratch_len(p, p.max_nrhs);
  const int64_t parts_rhs = 27LL * n_grid * kReachParts * p.nu;
  float* norm = reinterpret_cast<float*>(parts + p.max_nrhs * parts_rhs);
  Reach* reach = reinterpret_cast<Reach*>(norm + p.n_box * p.max_nrhs);
  const int2* maps = reinterpret_cast<const int2*>(p.d_fft_map);
  const int4* cells = reinterpret_cast<const int4*>(p.d_fft_cells);
  const Source all{P,
                   p.d_box_scale,
                   p.fp16() ? 2 : (p.split() ? 1 : 0),
                   p.kh,
                   p.khb,
                   p.n_d,
                   p.n_box * p.vstride(),
                   p.n_box};
  launch(norm_kernel, dim3((unsigned)((p.n_box + kThreads / 64 - 1) / (kThreads / 64)), nrhs),
         dim3(kThreads), 0, s, start, nullptr, all, cells, p.nu, norm);
  int splits = kReachParts;  // all resident at once (two per compute unit) or one each
  while (splits > 1 && 27 * splits * n_grid * nrhs > 512) splits /= 2;
  launch(reach_kernel, dim3(27 * splits, n_grid, nrhs), dim3(kReachThreads), 0, s, nullptr, nullptr,
         all, maps, cells, cells + p.n_box, (const float*)norm, p.a / p.n_d, p.k, p.eta, p.nu,
         reach, parts, splits);
  for (const FftGroup& g : p.fft_groups) {
    const FftTask* tasks = p.d_fft_tasks + g.first;
    const int n = g.count, block = (int)fft_block(g, p.max_nrhs);
    const unsigned zb = (unsigned)g.blocks[0], yb = (unsigned)(g.blocks[1] + 7) / 8 * 8,
                   xb = (unsigned)(g.blocks[2] + 7) / 8 * 8;  // multiples of 8: xcd_block
    for (int r0 = 0; r0 < nrhs; r0 += block) {
      const unsigned nr = (unsigned)std::min(block, nrhs - r0);
      const bool last = &g == &p.fft_groups.back() && r0 + block >= nrhs;
      Source src = all;
      src.P += (int64_t)r0 * p.n_box * p.vstride();
      src.box_scale += (int64_t)r0 * p.n_box;
      launch(fft_z_kernel, dim3(zb, nr), dim3(g.threads[0]), g.lds[0], s, nullptr, nullptr, src,
             maps, tasks, n, tw, lattices, g.len, (const float*)(norm + (int64_t)r0 * p.n_box));
      launch(fft_y_kernel<false>, dim3(yb, nr), dim3(g.threads[1]), g.lds[1], s, nullptr, nullptr,
             tasks, n, g.blocks[1], tw, lattices, g.len);
      launch(fft_x_kernel, dim3(xb, nr), dim3(g.threads[2]), g.lds[2], s, nullptr, nullptr, tasks,
             n, g.blocks[2], tw, spectra, lattices, g.len);
      launch(fft_y_kernel<true>, dim3(yb, nr), dim3(g.threads[1]), g.lds[1], s, nullptr, nullptr,
             tasks, n, g.blocks[1], tw, lattices, g.len);
      launch(ifft_z_kernel, dim3(zb, nr), dim3(g.threads[0]), g.lds[0], s, nullptr,
             last ? stop : nullptr, maps, tasks, n, tw, (const double2*)lattices, g.len,
             part + r0 * part_rhs, p.n_d, p.kh, part_rhs,
             (const Reach*)(reach + (int64_t)r0 * n_grid),
             (const double2*)(parts + r0 * parts_rhs), n_grid);
    }
  }
  return (int)hipGetLastError();
}

}  // namespace ubf
