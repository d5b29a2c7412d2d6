// FULL far sets as a discrete convolution over the lattice of the sites
// (FftGrid in plan.hpp). Per scatterer and right-hand side five kernels, each
// transforming lines of the zero-padded lattice in LDS:
//   fft_z:    box vectors -> [x][y][kz][component]          (x, y < sites)
//   fft_y:    -> [x][ky][kz][component]                     (x < sites)
//   fft_x:    transform along x, product with the spectrum of D (a symmetric
//             3 x 3 matrix per frequency), transform back, in place
//   ifft_y:   -> [x][y][kz][component]
//   ifft_z:   -> the first partial row of every box
// Only lines that can hold a value are touched, so the zero padding of an
// axis is never in memory before that axis is transformed. All are bound by
// memory and by the transforms' own arithmetic: on the 3,338-box shell (105^3
// sites, transforms of 216) 57 MB and 118 MB arrays, about 590 MB in all,
// against 15 GB of partial rows that 11.1 million pairs write and read one
// by one. Measured there: 27 + 50 + 131 + 55 + 22 us, and the whole product
// 407 us against 6,335 with every pair's operator evaluated and applied.
#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fft.hpp"

namespace ubf {
namespace {

constexpr int kThreads = 256;       // spectrum kernels
constexpr int kMaxThreads = kMaxFftThreads;  // transform kernels: one butterfly per thread
// LDS of one workgroup's lines: three workgroups share a compute unit (160 KB).
constexpr size_t kLineBytes = 50 << 10;

__device__ inline float2 cmul(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}
// a * b + c
__device__ inline float2 cfma(float2 a, float2 b, float2 c) {
  return make_float2(fmaf(a.x, b.x, fmaf(-a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(a.y, b.x, c.y)));
}
__device__ inline float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ inline float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// a * (-i) forward, a * i backward
template <bool INV>
__device__ inline float2 mul_mi(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// Discrete Fourier transform of R values in registers (in place, natural
// order): exp(-2 pi i jk / R), conjugated when INV.
template <int R, bool INV>
struct Butterfly;
template <bool INV>
struct Butterfly<2, INV> {
  static __device__ inline void run(float2 (&v)[2]) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};
template <bool INV>
struct Butterfly<3, INV> {
  static __device__ inline void run(float2 (&v)[3]) {
    const float s = 0.866025403784438647f;
    const float2 t = cadd(v[1], v[2]), d = mul_mi<INV>(csub(v[1], v[2]));
    const float2 m = make_float2(fmaf(-0.5f, t.x, v[0].x), fmaf(-0.5f, t.y, v[0].y));
    v[0] = cadd(v[0], t);
    v[1] = make_float2(fmaf(s, d.x, m.x), fmaf(s, d.y, m.y));
    v[2] = make_float2(fmaf(-s, d.x, m.x), fmaf(-s, d.y, m.y));
  }
};
template <bool INV>
struct Butterfly<4, INV> {
  static __device__ inline void run(float2 (&v)[4]) {
    const float2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
    const float2 c = cadd(v[1], v[3]), d = mul_mi<INV>(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[1] = cadd(b, d);
    v[2] = csub(a, c);
    v[3] = csub(b, d);
  }
};
template <bool INV>
struct Butterfly<5, INV> {
  static __device__ inline void run(float2 (&v)[5]) {
    // cos and sin of 2 pi / 5 and 4 pi / 5
    const float c1 = 0.309016994374947424f, c2 = -0.809016994374947424f;
    const float s1 = 0.951056516295153572f, s2 = 0.587785252292473129f;
    const float2 a = cadd(v[1], v[4]), b = cadd(v[2], v[3]);
    const float2 d = mul_mi<INV>(csub(v[1], v[4])), e = mul_mi<INV>(csub(v[2], v[3]));
    const float2 p = make_float2(fmaf(c1, a.x, fmaf(c2, b.x, v[0].x)),
                                 fmaf(c1, a.y, fmaf(c2, b.y, v[0].y)));
    const float2 q = make_float2(fmaf(c2, a.x, fmaf(c1, b.x, v[0].x)),
                                 fmaf(c2, a.y, fmaf(c1, b.y, v[0].y)));
    const float2 r = make_float2(fmaf(s1, d.x, s2 * e.x), fmaf(s1, d.y, s2 * e.y));
    const float2 t = make_float2(fmaf(s2, d.x, -s1 * e.x), fmaf(s2, d.y, -s1 * e.y));
    v[0] = cadd(v[0], cadd(a, b));
    v[1] = cadd(p, r);
    v[4] = csub(p, r);
    v[2] = cadd(q, t);
    v[3] = csub(q, t);
  }
};
template <bool INV>
struct Butterfly<6, INV> {  // two of three, combined by twos
  static __device__ inline void run(float2 (&v)[6]) {
    float2 e[3] = {v[0], v[2], v[4]}, o[3] = {v[1], v[3], v[5]};
    Butterfly<3, INV>::run(e);
    Butterfly<3, INV>::run(o);
    const float s = 0.866025403784438647f, sg = INV ? 1.f : -1.f;
    o[1] = cmul(o[1], make_float2(0.5f, sg * s));
    o[2] = cmul(o[2], make_float2(-0.5f, sg * s));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      v[k] = cadd(e[k], o[k]);
      v[k + 3] = csub(e[k], o[k]);
    }
  }
};
template <bool INV>
struct Butterfly<8, INV> {
  static __device__ inline void run(float2 (&v)[8]) {
    float2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    Butterfly<4, INV>::run(e);
    Butterfly<4, INV>::run(o);
    const float h = 0.707106781186547524f, sg = INV ? 1.f : -1.f;
    o[1] = cmul(o[1], make_float2(h, sg * h));
    o[2] = mul_mi<INV>(o[2]);
    o[3] = cmul(o[3], make_float2(-h, sg * h));
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

// `w` neighbouring lines of length L in LDS, three components each: value
// (position, line, component) at (position * w + line) * 3 + component. The
// index of (position, line) times three is what load and store below take.
//
// One Stockham stage of radix R, one butterfly (of all three components) per
// thread: butterfly j of a line reads positions j + r L / R, applies the
// twiddle factors of k = j mod Ns and writes positions (j / Ns) Ns R + k +
// r Ns. The components share the index arithmetic and the twiddle factors.
// load(position, line, v) and store(position, line, v) go to LDS or, for a
// transform's first and last stage, straight to memory; between the two every
// thread waits, so that one buffer serves both.
// A line of s sites is transformed at L >= 2 s - 1 positions: with an even
// radix (L even, s <= L / 2) the upper R / 2 inputs of the forward
// transform's first stage are the zero padding (HALF_IN), and the upper
// R / 2 outputs of the backward transform's last stage are not wanted
// (HALF_OUT).
template <int R, bool INV, bool TW, bool HALF_IN, bool HALF_OUT, class Load, class Store>
__device__ inline void stage(int L, int w, float inv_w, const float2* tw, int Ns, Load load,
                             Store store) {
  constexpr int RI = HALF_IN && R % 2 == 0 ? R / 2 : R;
  constexpr int RO = HALF_OUT && R % 2 == 0 ? R / 2 : R;
  const int m = L / R, i = threadIdx.x;
  const int j = fdiv(i, inv_w), line = i - j * w;
  const bool on = i < m * w;
  float2 v[R][3];
  if (on) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r < RI)
        load(j + r * m, line, v[r]);
      else
        v[r][0] = v[r][1] = v[r][2] = make_float2(0.f, 0.f);
    }
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
        float2 t = tw[r * step];
        if (INV) t.y = -t.y;
#pragma unroll
        for (int al = 0; al < 3; ++al) v[r][al] = cmul(v[r][al], t);
      }
    }
#pragma unroll
    for (int al = 0; al < 3; ++al) {
      float2 x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = v[r][al];
      Butterfly<R, INV>::run(x);
#pragma unroll
      for (int r = 0; r < R; ++r) v[r][al] = x[r];
    }
#pragma unroll
    for (int r = 0; r < RO; ++r) store(o + r * Ns, line, v[r]);
  }
  __syncthreads();
}

template <bool INV, bool TW, bool HALF_IN, bool HALF_OUT, class Load, class Store>
__device__ inline void stage_of(int R, int L, int w, float inv_w, const float2* tw, int Ns,
                                Load load, Store store) {
  switch (R) {  // uniform
    case 2: stage<2, INV, TW, HALF_IN, HALF_OUT>(L, w, inv_w, tw, Ns, load, store); break;
    case 3: stage<3, INV, TW, HALF_IN, HALF_OUT>(L, w, inv_w, tw, Ns, load, store); break;
    case 4: stage<4, INV, TW, HALF_IN, HALF_OUT>(L, w, inv_w, tw, Ns, load, store); break;
    case 5: stage<5, INV, TW, HALF_IN, HALF_OUT>(L, w, inv_w, tw, Ns, load, store); break;
    case 6: stage<6, INV, TW, HALF_IN, HALF_OUT>(L, w, inv_w, tw, Ns, load, store); break;
    default: stage<8, INV, TW, HALF_IN, HALF_OUT>(L, w, inv_w, tw, Ns, load, store); break;
  }
}

// Lines in LDS, as load and store of a stage.
struct Buffer {
  float2* b;
  int w;
  __device__ inline void operator()(int pos, int line, float2 (&v)[3]) const {  // load
    const float2* p = b + 3 * (pos * w + line);
#pragma unroll
    for (int al = 0; al < 3; ++al) v[al] = p[al];
  }
};
struct BufferStore {
  float2* b;
  int w;
  __device__ inline void operator()(int pos, int line, const float2 (&v)[3]) const {
    float2* p = b + 3 * (pos * w + line);
#pragma unroll
    for (int al = 0; al < 3; ++al) p[al] = v[al];
  }
};

// A whole transform in the buffer `a`: the first stage takes its values from
// load, the last one gives them to store (either may be the buffer). The
// twiddle factors and the buffer may have been written just before; ends with
// a barrier. An axis of length 1 passes its values through.
template <bool INV, class Load, class Store>
__device__ inline void transform(const FftAxis& ax, int w, const float2* tw, float2* a, Load load,
                                 Store store) {
  const int L = ax.L, n = ax.stages;
  const float inv_w = 1.f / (float)w;
  const Buffer get{a, w};
  const BufferStore put{a, w};
  __syncthreads();
  if (n == 0) {
    if ((int)threadIdx.x < w) {
      float2 v[3];
      load(0, threadIdx.x, v);
      store(0, threadIdx.x, v);
    }
    __syncthreads();
    return;
  }
  if (n == 1) {
    stage_of<INV, false, !INV, INV>(ax.radix[0], L, w, inv_w, tw, 1, load, store);
    return;
  }
  stage_of<INV, false, !INV, false>(ax.radix[0], L, w, inv_w, tw, 1, load, put);
  int Ns = ax.radix[0];
  for (int s = 1; s + 1 < n; ++s) {
    stage_of<INV, true, false, false>(ax.radix[s], L, w, inv_w, tw, Ns, get, put);
    Ns *= ax.radix[s];
  }
  stage_of<INV, true, false, INV>(ax.radix[n - 1], L, w, inv_w, tw, Ns, get, store);
}

__device__ inline void load_twiddles(float2* tw, const float2* __restrict__ all, const FftAxis& ax) {
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
  __device__ inline float2 at(int box, int u) const {
    if (mode == 0) {
      const float* b = P + (int64_t)box * 2 * kh;
      return make_float2(b[u], b[kh + u]);
    }
    const int at = khb == 192 ? (u % 3) * 64 + u / 3 : u;  // pos16 of stage 1
    const unsigned short* q = reinterpret_cast<const unsigned short*>(P + (int64_t)box * 2 * khb) +
                              32 * (at >> 3) + (at & 7);
    if (mode == 1) {
      auto f = [](unsigned short b) { return __uint_as_float((unsigned)b << 16); };
      return make_float2(f(q[0]) + f(q[16]), f(q[8]) + f(q[24]));
    }
    auto f = [](unsigned short b) { return __half2float(__ushort_as_half(b)); };
    const float sc = box_scale[box];  // a power of two
    return make_float2((f(q[0]) + f(q[16])) * sc, (f(q[8]) + f(q[24])) * sc);
  }
};

extern __shared__ float2 lds[];

// Workgroups are dealt round robin to the 8 XCDs: give each XCD a contiguous
// range, so that workgroups sharing memory lines share an L2. The grid is a
// multiple of 8; positions past the work are the caller's to skip.
__device__ inline int xcd_block() {
  return (int)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

// z transforms: one workgroup per column of boxes (x, y) and site plane mx
// of it, n_d lines (site rows my).
__global__ __launch_bounds__(kMaxThreads) void fft_z_kernel(
    Source src, const int2* __restrict__ map, FftGrid g, const float2* __restrict__ twiddles,
    float2* __restrict__ out, int64_t out_rhs) {
  src.select(blockIdx.z);
  out += blockIdx.z * out_rhs;
  const int nd = src.nd, L = g.ax[2].L, row = 3 * nd * nd;
  float2 *a = lds, *tw = a + 3 * L * nd;
  const int by = blockIdx.y, bx = blockIdx.x / nd, mx = blockIdx.x - bx * nd;
  const int2* col = map + ((int64_t)bx * g.n[1] + by) * g.n[2];
  load_twiddles(tw, twiddles, g.ax[2]);
  const float inv_row = 1.f / row, inv_line = 1.f / (3 * nd);
  bool any = false;
  for (int i = threadIdx.x; i < g.n[2] * row; i += blockDim.x) {
    const int bz = fdiv(i, inv_row), v = i - bz * row;     // v = (my nd + mz) 3 + alpha
    const int my = fdiv(v, inv_line), t = v - my * 3 * nd;  // t = 3 mz + alpha
    const int mz = t / 3, al = t - 3 * mz;
    const int box = col[bz].x;
    float2 z = make_float2(0.f, 0.f);
    if (box >= 0) {
      z = src.at(box, mx * row + v);
      any = true;
    }
    a[((bz * nd + mz) * nd + my) * 3 + al] = z;
  }
  const int X = bx * nd + mx, s = g.s[2];
  float2* o = out + ((int64_t)X * g.s[1] + by * nd) * L * 3;
  if (!__syncthreads_or(any)) {  // a column without boxes transforms to zeros
    for (int i = threadIdx.x; i < 3 * L * nd; i += blockDim.x) o[i] = make_float2(0.f, 0.f);
    return;
  }
  transform<false>(
      g.ax[2], nd, tw, a,
      [&](int pos, int line, float2 (&v)[3]) {
#pragma unroll
        for (int al = 0; al < 3; ++al)
          v[al] = pos < s ? a[(pos * nd + line) * 3 + al] : make_float2(0.f, 0.f);
      },
      [&](int pos, int line, const float2 (&v)[3]) {
        float2* q = o + 3 * (line * L + pos);
#pragma unroll
        for (int al = 0; al < 3; ++al) q[al] = v[al];
      });
}

// y transforms of w neighbouring lines (x, kz with kz fastest); forward from
// s to L positions, backward from L to s.
template <bool INV>
__global__ __launch_bounds__(kMaxThreads) void fft_y_kernel(
    const float2* __restrict__ in, FftGrid g, const float2* __restrict__ twiddles,
    float2* __restrict__ out, int w, int64_t in_rhs, int64_t out_rhs) {
  in += blockIdx.y * in_rhs;
  out += blockIdx.y * out_rhs;
  const int L = g.ax[1].L, s = g.s[1], Lz = g.ax[2].L;
  const int nin = INV ? L : s, nout = INV ? s : L;
  float2 *a = lds, *tw = a + 3 * L * w;
  const int all = g.s[0] * Lz, l0 = xcd_block() * w;
  if (l0 >= all) return;
  load_twiddles(tw, twiddles, g.ax[1]);
  const float inv_lz = 1.f / Lz;
  // line l = (x, kz): its first value in an array of n positions along y
  auto first = [&](int l, int n) {
    const int x = l / Lz;
    return ((int64_t)x * n * Lz + (l - x * Lz)) * 3;
  };
  transform<INV>(
      g.ax[1], w, tw, a,
      [&](int pos, int line, float2 (&v)[3]) {
        const int l = l0 + line;
        const float2* p = in + first(l, nin) + 3 * pos * Lz;
#pragma unroll
        for (int al = 0; al < 3; ++al)
          v[al] = pos < nin && l < all ? p[al] : make_float2(0.f, 0.f);
      },
      [&](int pos, int line, const float2 (&v)[3]) {
        const int l = l0 + line;
        float2* p = out + first(l, nout) + 3 * pos * Lz;
        if (pos < nout && l < all) {
#pragma unroll
          for (int al = 0; al < 3; ++al) p[al] = v[al];
        }
      });
}

// The last forward stage along x, the product with the spectrum and the
// first backward stage: butterfly j ends with the frequencies j + r L / R in
// registers, which is what the backward transform's first butterfly of the
// same radix starts from.
template <int R, bool TW, class Load, class Store, class Spec>
__device__ inline void middle_stage(int L, int w, float inv_w, const float2* tw, Load load,
                                    Store store, Spec spectrum) {
  const int m = L / R, i = threadIdx.x;
  const int j = fdiv(i, inv_w), line = i - j * w;
  const bool on = i < m * w;
  float2 v[R][3];
  if (on) {
#pragma unroll
    for (int r = 0; r < R; ++r) load(j + r * m, line, v[r]);
    if (TW) {
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const float2 t = tw[r * j];  // Ns = m: k = j
#pragma unroll
        for (int al = 0; al < 3; ++al) v[r][al] = cmul(v[r][al], t);
      }
    }
#pragma unroll
    for (int al = 0; al < 3; ++al) {
      float2 x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = v[r][al];
      Butterfly<R, false>::run(x);
#pragma unroll
      for (int r = 0; r < R; ++r) v[r][al] = x[r];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) spectrum(j + r * m, line, v[r]);
#pragma unroll
    for (int al = 0; al < 3; ++al) {
      float2 x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = v[r][al];
      Butterfly<R, true>::run(x);
#pragma unroll
      for (int r = 0; r < R; ++r) v[r][al] = x[r];
    }
  }
  __syncthreads();
  if (on) {
#pragma unroll
    for (int r = 0; r < R; ++r) store(j * R + r, line, v[r]);
  }
  __syncthreads();
}

// Along x: transform, product with the spectrum, transform back, for w
// neighbouring lines (ky, kz). The spectrum is stored for frequencies
// 0 .. L/2 per axis; D is even along its two equal axes and odd along each
// of two different ones, so a mirrored frequency changes the sign of the
// components odd along that axis. The backward transform takes the radices
// in the opposite order, so that the two stages around the product share
// their butterflies.
__global__ __launch_bounds__(kMaxThreads) void fft_x_kernel(
    float2* __restrict__ data, FftGrid g, const float2* __restrict__ twiddles,
    const float4* __restrict__ spec, int w, int64_t rhs) {
  data += blockIdx.y * rhs;
  const int L = g.ax[0].L, s = g.s[0], Ly = g.ax[1].L, Lz = g.ax[2].L;
  const int hy = Ly / 2 + 1, hz = Lz / 2 + 1;
  float2 *a = lds, *tw = a + 3 * L * w;
  const int plane = Ly * Lz, l0 = xcd_block() * w;
  if (l0 >= plane) return;
  load_twiddles(tw, twiddles, g.ax[0]);
  const float inv_w = 1.f / (float)w;
  auto load = [&](int pos, int line, float2 (&v)[3]) {
    const int l = l0 + line;
    const float2* p = data + ((int64_t)pos * plane + l) * 3;
#pragma unroll
    for (int al = 0; al < 3; ++al) v[al] = pos < s && l < plane ? p[al] : make_float2(0.f, 0.f);
  };
  auto store = [&](int pos, int line, const float2 (&v)[3]) {
    const int l = l0 + line;
    float2* p = data + ((int64_t)pos * plane + l) * 3;
    if (pos < s && l < plane) {
#pragma unroll
      for (int al = 0; al < 3; ++al) p[al] = v[al];
    }
  };
  auto spectrum = [&](int kx, int line, float2 (&f)[3]) {
    const int l = min(l0 + line, plane - 1);
    const int ky = l / Lz, kz = l - ky * Lz;
    const bool mx = 2 * kx > L, my = 2 * ky > Ly, mz = 2 * kz > Lz;
    const float4* k = spec + 3 * (((int64_t)(mx ? L - kx : kx) * hy + (my ? Ly - ky : ky)) * hz +
                                  (mz ? Lz - kz : kz));
    const float4 k0 = k[0], k1 = k[1], k2 = k[2];  // xx, yy | zz, xy | xz, yz
    const float sxy = mx == my ? 1.f : -1.f, sxz = mx == mz ? 1.f : -1.f,
                syz = my == mz ? 1.f : -1.f;
    const float2 xx = make_float2(k0.x, k0.y), yy = make_float2(k0.z, k0.w);
    const float2 zz = make_float2(k1.x, k1.y), xy = make_float2(k1.z * sxy, k1.w * sxy);
    const float2 xz = make_float2(k2.x * sxz, k2.y * sxz), yz = make_float2(k2.z * syz, k2.w * syz);
    const float2 u = f[0], v = f[1], z = f[2];
    f[0] = cfma(xx, u, cfma(xy, v, cmul(xz, z)));
    f[1] = cfma(xy, u, cfma(yy, v, cmul(yz, z)));
    f[2] = cfma(xz, u, cfma(yz, v, cmul(zz, z)));
  };
  const Buffer get{a, w};
  const BufferStore put{a, w};
  const FftAxis& ax = g.ax[0];
  const int n = ax.stages;
  __syncthreads();
  if (n == 0) {
    if ((int)threadIdx.x < w) {
      float2 v[3];
      load(0, threadIdx.x, v);
      spectrum(0, threadIdx.x, v);
      store(0, threadIdx.x, v);
    }
    return;
  }
  if (n == 1) {
    switch (L) {  // uniform
      case 2: middle_stage<2, false>(L, w, inv_w, tw, load, store, spectrum); break;
      case 3: middle_stage<3, false>(L, w, inv_w, tw, load, store, spectrum); break;
      case 4: middle_stage<4, false>(L, w, inv_w, tw, load, store, spectrum); break;
      case 5: middle_stage<5, false>(L, w, inv_w, tw, load, store, spectrum); break;
      default: middle_stage<6, false>(L, w, inv_w, tw, load, store, spectrum); break;
    }
    return;
  }
  stage_of<false, false, true, false>(ax.radix[0], L, w, inv_w, tw, 1, load, put);
  int Ns = ax.radix[0];
  for (int st = 1; st + 1 < n; ++st) {
    stage_of<false, true, false, false>(ax.radix[st], L, w, inv_w, tw, Ns, get, put);
    Ns *= ax.radix[st];
  }
  switch (ax.radix[n - 1]) {  // uniform; at most 6 (fft_axis)
    case 2: middle_stage<2, true>(L, w, inv_w, tw, get, put, spectrum); break;
    case 3: middle_stage<3, true>(L, w, inv_w, tw, get, put, spectrum); break;
    case 4: middle_stage<4, true>(L, w, inv_w, tw, get, put, spectrum); break;
    case 5: middle_stage<5, true>(L, w, inv_w, tw, get, put, spectrum); break;
    default: middle_stage<6, true>(L, w, inv_w, tw, get, put, spectrum); break;
  }
  Ns = ax.radix[n - 1];
  for (int st = n - 2; st > 0; --st) {
    stage_of<true, true, false, false>(ax.radix[st], L, w, inv_w, tw, Ns, get, put);
    Ns *= ax.radix[st];
  }
  stage_of<true, true, false, true>(ax.radix[0], L, w, inv_w, tw, Ns, get, store);
}

// Backward z transforms into the boxes' rows: the lines of fft_z_kernel.
__global__ __launch_bounds__(kMaxThreads) void ifft_z_kernel(
    const float2* __restrict__ in, const int2* __restrict__ map, FftGrid g,
    const float2* __restrict__ twiddles, float* __restrict__ part, int nd, int kh,
    int64_t in_rhs, int64_t part_rhs) {
  in += blockIdx.z * in_rhs;
  part += blockIdx.z * part_rhs;
  const int L = g.ax[2].L, row = 3 * nd * nd, nu = row * nd, s = g.s[2];
  float2 *a = lds, *tw = a + 3 * L * nd;
  const int by = blockIdx.y, bx = blockIdx.x / nd, mx = blockIdx.x - bx * nd;
  const int2* col = map + ((int64_t)bx * g.n[1] + by) * g.n[2];
  bool any = false;
  for (int i = threadIdx.x; i < g.n[2]; i += blockDim.x) any = any || col[i].y >= 0;
  if (!__syncthreads_or(any)) return;  // a column without rows
  load_twiddles(tw, twiddles, g.ax[2]);
  const int X = bx * nd + mx;
  const float2* p = in + ((int64_t)X * g.s[1] + by * nd) * L * 3;
  transform<true>(
      g.ax[2], nd, tw, a,
      [&](int pos, int line, float2 (&v)[3]) {
        const float2* q = p + 3 * (line * L + pos);
#pragma unroll
        for (int al = 0; al < 3; ++al) v[al] = q[al];
      },
      [&](int pos, int line, const float2 (&v)[3]) {
        if (pos < s) {
#pragma unroll
          for (int al = 0; al < 3; ++al) a[(pos * nd + line) * 3 + al] = v[al];
        }
      });
  const float inv_row = 1.f / row, inv_line = 1.f / (3 * nd);
  for (int i = threadIdx.x; i < g.n[2] * row; i += blockDim.x) {
    const int bz = fdiv(i, inv_row), v = i - bz * row;
    const int my = fdiv(v, inv_line), t = v - my * 3 * nd;
    const int mz = t / 3, al = t - 3 * mz;
    const int at = col[bz].y;
    if (at < 0) continue;
    const float2 z = a[((bz * nd + mz) * nd + my) * 3 + al];
    float* q = part + (int64_t)at * 2 * kh + mx * row + v;  // [Er | Ei] of N_u each
    q[0] = z.x;
    q[nu] = z.y;
  }
}

// ---------------------------------------------------------------- spectrum

// Component e (xx, yy, zz, xy, xz, yz) of D(R) in FP64, zero where the
// convolution leaves the pair to the masked operators.
__device__ double2 green_component(int e, int dx, int dy, int dz, double step, double k,
                                   double eta, int nd) {
  if (max(dx, max(dy, dz)) < 2 * nd) return make_double2(0.0, 0.0);
  const int pa[6] = {0, 1, 2, 0, 0, 1}, pb[6] = {0, 1, 2, 1, 2, 2};
  const double R[3] = {step * dx, step * dy, step * dz};
  const double r2 = R[0] * R[0] + R[1] * R[1] + R[2] * R[2];
  const double r = sqrt(r2), kr = k * r, ik = 1.0 / kr;
  double sn, cs;
  sincos(kr, &sn, &cs);
  // psi = -j k eta e^{-j kr} / (4 pi r)
  const double f = k * eta / (4.0 * 3.14159265358979323846 * r);
  const double pr = -f * sn, pi = -f * cs;
  const double rr = R[pa[e]] * R[pb[e]] / r2, iso = pa[e] == pb[e] ? 1.0 : 0.0;
  const double tr = iso * (1.0 - ik * ik) - rr * (1.0 - 3.0 * ik * ik);
  const double ti = -iso * ik + rr * 3.0 * ik;
  return make_double2(pr * tr - pi * ti, pr * ti + pi * tr);
}

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
    D[z] = green_component(e, x, y, z, step, k, eta, nd);
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
                                                              float2* __restrict__ spec) {
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
    spec[6 * (((int64_t)kx * hy + ky) * hz + kz) + e] =
        make_float2((float)(s.x * f), (float)(s.y * f));
  }
}

// Lines of a workgroup, of `all`: as many as the LDS budget and about 320
// threads take, but no fewer than 1,024 workgroups (four per compute unit)
// while a workgroup keeps a wavefront busy.
int fit_lines(const FftAxis& ax, int all) {
  int w = 64;
  while (w > 1 && (3 * (size_t)ax.L * w * sizeof(float2) > kLineBytes ||
                   ax.butterflies() * w > 320 ||
                   (all < 1024 * w && ax.butterflies() * w >= 128)))
    w /= 2;
  return w;
}
size_t line_bytes(const FftAxis& ax, int w) { return (3 * (size_t)ax.L * w + ax.L) * sizeof(float2); }
dim3 line_threads(const FftAxis& ax, int w) { return dim3((ax.butterflies() * w + 63) / 64 * 64); }

// Workgroups of `lines` lines each, a multiple of 8 (xcd_block).
unsigned blocks_of(int all, int lines) {
  return (unsigned)((all + lines - 1) / lines + 7) / 8 * 8;
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
    float2* spec = reinterpret_cast<float2*>(p.d_fft_spec) + g.spec;
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
  const float2* tw = reinterpret_cast<const float2*>(p.d_fft_tw);
  const int64_t part_rhs = p.rest->n_pairs() * p.pstride();
  int64_t zmax = 0, ymax = 0;
  for (const FftGrid& g : p.fft) {
    zmax = std::max(zmax, g.zlen());
    ymax = std::max(ymax, g.yzlen());
  }
  // right-hand sides go through the scratch in blocks (fft_block)
  const int block = (int)fft_block(p, p.max_nrhs);
  float2* bz = reinterpret_cast<float2*>(p.d_fft);
  float2* by = bz + block * zmax;
  for (size_t i = 0; i < p.fft.size(); ++i) {
    const FftGrid& g = p.fft[i];
    const int2* map = reinterpret_cast<const int2*>(p.d_fft_map) + g.map;
    const float4* spec = reinterpret_cast<const float4*>(p.d_fft_spec) + g.spec / 2;
    const int ny = g.s[0] * g.ax[2].L, nx = g.ax[1].L * g.ax[2].L;
    const int yw = fit_lines(g.ax[1], ny), xw = fit_lines(g.ax[0], nx);
    const dim3 zblock = line_threads(g.ax[2], p.n_d), yblock = line_threads(g.ax[1], yw),
               xblock = line_threads(g.ax[0], xw);
    const size_t zb = line_bytes(g.ax[2], p.n_d), yb = line_bytes(g.ax[1], yw),
                 xb = line_bytes(g.ax[0], xw);
    for (int r0 = 0; r0 < nrhs; r0 += block) {
      const int nr = std::min(block, nrhs - r0);
      const bool first = i == 0 && r0 == 0, last = i + 1 == p.fft.size() && r0 + nr == nrhs;
      const dim3 zgrid(g.n[0] * p.n_d, g.n[1], nr), ygrid(blocks_of(ny, yw), nr),
          xgrid(blocks_of(nx, xw), nr);
      const Source src{P + (int64_t)r0 * p.n_box * p.vstride(),
                       p.d_box_scale + (int64_t)r0 * p.n_box,
                       p.fp16() ? 2 : (p.split() ? 1 : 0),
                       p.kh,
                       p.khb,
                       p.n_d,
                       p.n_box * p.vstride(),
                       p.n_box};
      launch(fft_z_kernel, zgrid, zblock, zb, s, first ? start : nullptr, nullptr, src, map, g, tw,
             bz, zmax);
      launch(fft_y_kernel<false>, ygrid, yblock, yb, s, nullptr, nullptr, (const float2*)bz, g, tw,
             by, yw, zmax, ymax);
      launch(fft_x_kernel, xgrid, xblock, xb, s, nullptr, nullptr, by, g, tw, spec, xw, ymax);
      launch(fft_y_kernel<true>, ygrid, yblock, yb, s, nullptr, nullptr, (const float2*)by, g, tw,
             bz, yw, ymax, zmax);
      launch(ifft_z_kernel, zgrid, zblock, zb, s, nullptr, last ? stop : nullptr,
             (const float2*)bz, map, g, tw, part + r0 * part_rhs, p.n_d, p.kh, zmax, part_rhs);
    }
  }
  return (int)hipGetLastError();
}

}  // namespace ubf
