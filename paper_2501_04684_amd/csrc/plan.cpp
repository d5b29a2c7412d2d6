// Host plan builder: validation, far set (Algorithm 2), offset grouping,
// symmetry orbits (Sec. 2.2) and the FP32 operator table (Eq. 5-6, 13).
#include "plan.hpp"

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <limits>
#include <mutex>
#include <thread>
#include <numeric>
#include <unordered_map>

namespace ubf {

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr double kEta0 = 376.730313668;
// Dense box-index grids above this many cells use a hash map instead.
constexpr int64_t kDenseCells = int64_t(1) << 24;
// Largest operator table accepted (bytes).
constexpr double kMaxTableBytes = 16.0 * (1ull << 30);

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Lookup of a box index from integer coordinates. Small bounding grids use
// a dense array; larger ones a hash map keyed on the exact coordinate
// triple (any int32 >= 0 per axis), so distinct boxes never share a key.
struct BoxIndex {
  struct Key {
    int32_t x, y, z;
    bool operator==(const Key& o) const { return x == o.x && y == o.y && z == o.z; }
  };
  struct KeyHash {
    size_t operator()(const Key& k) const {
      uint64_t h = (uint32_t)k.x;
      h = h * 0x9E3779B97F4A7C15ull ^ (uint32_t)k.y;
      h = h * 0x9E3779B97F4A7C15ull ^ (uint32_t)k.z;
      return (size_t)(h ^ (h >> 31));
    }
  };
  int64_t nx = 0, ny = 0, nz = 0;
  std::vector<int32_t> dense;
  std::unordered_map<Key, int32_t, KeyHash> sparse;
  bool use_dense = true;

  // Index boxes b[0..n) (3 coordinates each, all >= 0); false on a duplicate.
  bool build(const int32_t* b, int64_t n) {
    int64_t mx = 0, my = 0, mz = 0;
    for (int64_t i = 0; i < n; ++i) {
      mx = std::max<int64_t>(mx, b[3 * i]);
      my = std::max<int64_t>(my, b[3 * i + 1]);
      mz = std::max<int64_t>(mz, b[3 * i + 2]);
    }
    nx = mx + 1;
    ny = my + 1;
    nz = mz + 1;
    // the product of three extents up to 2^31 overflows int64: test stepwise
    use_dense = nx <= kDenseCells && ny <= kDenseCells && nz <= kDenseCells &&
                nx * ny <= kDenseCells && nx * ny * nz <= kDenseCells;
    dense.clear();
    sparse.clear();
    if (use_dense) {
      dense.assign((size_t)(nx * ny * nz), -1);
      for (int64_t i = 0; i < n; ++i) {
        int32_t& slot = dense[((size_t)b[3 * i] * ny + b[3 * i + 1]) * nz + b[3 * i + 2]];
        if (slot >= 0) return false;
        slot = (int32_t)i;
      }
    } else {
      sparse.reserve((size_t)n * 2);
      for (int64_t i = 0; i < n; ++i)
        if (!sparse.emplace(Key{b[3 * i], b[3 * i + 1], b[3 * i + 2]}, (int32_t)i).second)
          return false;
    }
    return true;
  }
  int32_t find(int64_t x, int64_t y, int64_t z) const {
    if (x < 0 || y < 0 || z < 0 || x >= nx || y >= ny || z >= nz) return -1;
    if (use_dense) return dense[((size_t)x * ny + y) * nz + z];
    auto it = sparse.find(Key{(int32_t)x, (int32_t)y, (int32_t)z});
    return it == sparse.end() ? -1 : it->second;
  }
};

int32_t cheb(int64_t x, int64_t y, int64_t z) {
  return (int32_t)std::max({std::llabs(x), std::llabs(y), std::llabs(z)});
}

int64_t floordiv2(int64_t c) { return c >= 0 ? c / 2 : -((-c + 1) / 2); }

// The site pairs of an operator that a convolution leaves (FftGrid): those
// whose lattice difference n_d w + m_l - m_s stays below 2 n_d on every axis.
void mask_operator(const int32_t* w, int n_d, std::vector<std::complex<double>>& G) {
  const int nd3 = n_d * n_d * n_d, nu = 3 * nd3;
  auto axis = [n_d](int s, int d) { return d == 0 ? s / (n_d * n_d) : d == 1 ? (s / n_d) % n_d : s % n_d; };
  for (int l = 0; l < nd3; ++l)
    for (int s = 0; s < nd3; ++s) {
      bool keep = true;
      for (int d = 0; d < 3; ++d)
        keep = keep && std::abs(n_d * w[d] + axis(l, d) - axis(s, d)) < 2 * n_d;
      if (keep) continue;
      for (int al = 0; al < 3; ++al)
        for (int be = 0; be < 3; ++be) G[(size_t)(3 * l + al) * nu + 3 * s + be] = 0.0;
    }
}

// The 16-bit image of 192-coefficient boxes by lattice difference
// (Plan::kLatticeHalves): value sz of run (be, part, plane, al, dx, dy, lz)
// is that of a site pair with l - s = (dx - 3, dy - 3, lz - sz). Each
// operator value v (divided by the offset's power-of-two scale in the FP16
// forms) is hi = round16(v), lo = round16(v - hi).
void staged_split_image(const Plan& P, const std::vector<std::complex<double>>& G, double inv,
                        uint16_t* out) {
  const int np = P.precision == 3 ? 1 : 2;
  std::fill(out, out + P.staged_split_halves(), (uint16_t)0);
  for (int be = 0; be < 3; ++be)
    for (int c = 0; c < 2; ++c)
      for (int al = 0; al < 3; ++al)
        for (int dx = -3; dx <= 3; ++dx)
          for (int dy = -3; dy <= 3; ++dy)
            for (int lz = 0; lz < 4; ++lz)
              for (int sz = 0; sz < 4; ++sz) {
                // any site pair with this difference
                const int l = (std::max(dx, 0) * 4 + std::max(dy, 0)) * 4 + lz;
                const int s = (std::max(-dx, 0) * 4 + std::max(-dy, 0)) * 4 + sz;
                const std::complex<double> g = G[(size_t)(3 * l + al) * P.nu + 3 * s + be];
                const float f = (float)((c ? g.imag() : g.real()) * inv);
                const size_t run = (size_t)be * np * Plan::kLatticePart +
                                   c * Plan::kLatticePlane + al * Plan::kLatticeAl +
                                   ((dx + 3) * 7 + dy + 3) * 4 + lz;
                const uint16_t hi = P.fp16() ? fp16_bits(f) : bf16_bits(f);
                out[run * 4 + sz] = hi;
                if (np == 2)
                  out[(run + Plan::kLatticePart) * 4 + sz] =
                      P.fp16() ? fp16_bits(f - fp16_value(hi)) : bf16_bits(f - bf16_value(hi));
              }
}

// One offset's operator image in the table layout. FP32: planes re, im of
// nu rows of kh floats. Split: G is rounded to FP32 first (as in the FP32
// path), then hi = bf16(G), lo = bf16(G - hi); planes re.hi, im.hi, re.lo,
// im.lo of nu rows of khb values. Padding columns are zero.
void offset_image(const Plan& P, const int32_t* w, bool masked,
                  std::vector<std::complex<double>>& G, char* dst, float* scale) {
  operator_fp64(w, P.a, P.k, P.eta, P.n_d, G);
  if (masked) mask_operator(w, P.n_d, G);
  *scale = 1.0f;
  if (P.staged_split()) {
    double inv = 1.0;
    if (P.fp16()) {  // power of two bringing the largest |Re|, |Im| to [2^14, 2^15)
      double mx = 0.0;
      for (const auto& g : G) mx = std::max({mx, std::abs(g.real()), std::abs(g.imag())});
      const int e = mx > 0.0 ? std::ilogb(mx) - 14 : 0;
      *scale = (float)std::ldexp(1.0, e);
      inv = std::ldexp(1.0, -e);  // exact power of two
    }
    staged_split_image(P, G, inv, (uint16_t*)dst);
    return;
  }
  if (P.fp16()) {
    // power of two bringing the largest |Re|, |Im| to [2^14, 2^15)
    double mx = 0.0;
    for (const auto& g : G) mx = std::max({mx, std::abs(g.real()), std::abs(g.imag())});
    const int e = mx > 0.0 ? std::ilogb(mx) - 14 : 0;
    *scale = (float)std::ldexp(1.0, e);
    const double inv = std::ldexp(1.0, -e);  // exact power of two
    const uint16_t zero = 0;
    const size_t plane = (size_t)P.nu * P.khb;
    uint16_t* base = (uint16_t*)dst;
    std::fill(base, base + 4 * plane, zero);
    for (int u = 0; u < P.nu; ++u)
      for (int v = 0; v < P.nu; ++v) {
        const std::complex<double> g = G[(size_t)u * P.nu + v];
        const float parts[2] = {(float)(g.real() * inv), (float)(g.imag() * inv)};
        for (int c = 0; c < 2; ++c) {
          const uint16_t hi = fp16_bits(parts[c]);
          const uint16_t lo = fp16_bits(parts[c] - fp16_value(hi));
          base[c * plane + (size_t)u * P.khb + v] = hi;
          base[(2 + c) * plane + (size_t)u * P.khb + v] = lo;
        }
      }
    return;
  }
  if (P.staged()) {
    // block b, group g, lane l (row r = l % 32 of the block, K half h = l / 32:
    // the real inputs for h = 0, the imaginary ones for h = 1), k-steps
    // 4g..4g+3: Er rows take (Gr, -Gi), Ei rows (Gi, Gr); rows past 2 N_u and
    // columns past N_u are zero
    const int g4 = P.kh / 4, nb = (2 * P.nu + 31) / 32;
    float* f = (float*)dst;
    for (int b = 0; b < nb; ++b)
      for (int g = 0; g < g4; ++g)
        for (int l = 0; l < 64; ++l)
          for (int j = 0; j < 4; ++j) {
            const int row = 32 * b + (l & 31), h = l >> 5, k = 4 * g + j;
            double v = 0.0;
            if (row < 2 * P.nu && k < P.nu) {
              const bool ei = row >= P.nu;
              const std::complex<double> c = G[(size_t)(ei ? row - P.nu : row) * P.nu + k];
              v = !ei ? (h == 0 ? c.real() : -c.imag()) : (h == 0 ? c.imag() : c.real());
            }
            f[(((size_t)b * g4 + g) * 64 + l) * 4 + j] = (float)v;
          }
    return;
  }
  if (!P.split()) {
    const size_t plane = P.plane_floats();
    float* re = (float*)dst;
    float* im = re + plane;
    std::fill(re, re + 2 * plane, 0.0f);
    for (int u = 0; u < P.nu; ++u)
      for (int v = 0; v < P.nu; ++v) {
        re[(size_t)u * P.kh + v] = (float)G[(size_t)u * P.nu + v].real();
        im[(size_t)u * P.kh + v] = (float)G[(size_t)u * P.nu + v].imag();
      }
  } else {
    const size_t plane = (size_t)P.nu * P.khb;
    uint16_t* base = (uint16_t*)dst;
    std::fill(base, base + 4 * plane, (uint16_t)0);
    for (int u = 0; u < P.nu; ++u)
      for (int v = 0; v < P.nu; ++v) {
        const std::complex<double> g = G[(size_t)u * P.nu + v];
        const float parts[2] = {(float)g.real(), (float)g.imag()};
        for (int c = 0; c < 2; ++c) {
          const uint16_t hi = bf16_bits(parts[c]);
          const uint16_t lo = bf16_bits(parts[c] - bf16_value(hi));
          base[c * plane + (size_t)u * P.khb + v] = hi;
          base[(2 + c) * plane + (size_t)u * P.khb + v] = lo;
        }
      }
  }
}

// Process-wide cache of operator images for offsets within +-3 (every
// ILIST offset), keyed by the exact parameters; bounded in bytes. Plans of
// repeated problems (serving) then skip the FP64 Green's evaluations.
struct ImageKey {
  double a, k, eta;
  int32_t n_d, precision, w0, w1, w2, masked;
  bool operator==(const ImageKey& o) const {
    return a == o.a && k == o.k && eta == o.eta && n_d == o.n_d && masked == o.masked &&
           precision == o.precision && w0 == o.w0 && w1 == o.w1 && w2 == o.w2;
  }
};
struct ImageKeyHash {
  size_t operator()(const ImageKey& x) const {
    uint64_t h = 0;
    auto mix = [&h](uint64_t v) { h = (h ^ v) * 0x100000001B3ull + 0x9E3779B97F4A7C15ull; };
    uint64_t bits;
    std::memcpy(&bits, &x.a, 8); mix(bits);
    std::memcpy(&bits, &x.k, 8); mix(bits);
    std::memcpy(&bits, &x.eta, 8); mix(bits);
    mix((uint32_t)x.n_d); mix((uint32_t)x.precision);
    mix((uint32_t)x.w0); mix((uint32_t)x.w1); mix((uint32_t)x.w2); mix((uint32_t)x.masked);
    return (size_t)h;
  }
};
constexpr size_t kImageCacheBytes = size_t(256) << 20;
std::mutex g_image_mu;
std::unordered_map<ImageKey, std::vector<char>, ImageKeyHash> g_images;
size_t g_image_bytes = 0;

bool cacheable(const int32_t* w) {
  return std::abs(w[0]) <= 3 && std::abs(w[1]) <= 3 && std::abs(w[2]) <= 3;
}
ImageKey image_key(const Plan& P, const int32_t* w, bool masked) {
  return ImageKey{P.a, P.k, P.eta, P.n_d, P.precision, w[0], w[1], w[2], masked ? 1 : 0};
}
// An entry holds the image followed by its float scale.
bool image_cache_get(const Plan& P, const int32_t* w, bool masked, char* dst, size_t bytes,
                     float* scale) {
  if (!cacheable(w)) return false;
  std::lock_guard<std::mutex> lock(g_image_mu);
  auto it = g_images.find(image_key(P, w, masked));
  if (it == g_images.end() || it->second.size() != bytes + sizeof(float)) return false;
  std::memcpy(dst, it->second.data(), bytes);
  std::memcpy(scale, it->second.data() + bytes, sizeof(float));
  return true;
}
void image_cache_put(const Plan& P, const int32_t* w, bool masked, const char* src,
                     size_t bytes, float scale) {
  if (!cacheable(w)) return;
  std::lock_guard<std::mutex> lock(g_image_mu);
  if (g_image_bytes + bytes > kImageCacheBytes) return;
  std::vector<char> entry(src, src + bytes);
  entry.resize(bytes + sizeof(float));
  std::memcpy(entry.data() + bytes, &scale, sizeof(float));
  auto ins = g_images.emplace(image_key(P, w, masked), std::move(entry));
  if (ins.second) g_image_bytes += bytes;
}

}  // namespace

void dyadic_green(const double R[3], double k, double eta,
                  std::complex<double> D[3][3]) {
  const double r = std::sqrt(R[0] * R[0] + R[1] * R[1] + R[2] * R[2]);
  const double rh[3] = {R[0] / r, R[1] / r, R[2] / r};
  const double kr = k * r;
  const std::complex<double> j(0.0, 1.0);
  const std::complex<double> psi =
      -j * k * eta * std::exp(-j * kr) / (4.0 * kPi * r);
  const std::complex<double> c_iso = 1.0 - j / kr - 1.0 / (kr * kr);
  const std::complex<double> c_rr = 1.0 - 3.0 * j / kr - 3.0 / (kr * kr);
  for (int p = 0; p < 3; ++p)
    for (int q = 0; q < 3; ++q)
      D[p][q] = psi * ((p == q ? c_iso : 0.0) - rh[p] * rh[q] * c_rr);
}

std::vector<double> site_offsets(double a, int n_d) {
  std::vector<double> r;
  r.reserve(3 * n_d * n_d * n_d);
  for (int mx = 0; mx < n_d; ++mx)
    for (int my = 0; my < n_d; ++my)
      for (int mz = 0; mz < n_d; ++mz) {
        r.push_back(a * ((mx + 0.5) / n_d - 0.5));
        r.push_back(a * ((my + 0.5) / n_d - 0.5));
        r.push_back(a * ((mz + 0.5) / n_d - 0.5));
      }
  return r;
}

void operator_fp64(const int32_t w[3], double a, double k, double eta, int n_d,
                   std::vector<std::complex<double>>& G) {
  // The sites form one uniform lattice of step a / n_d, so r_l - r_s depends
  // only on the lattice difference d = m_l - m_s in [-(n_d-1), n_d-1]^3:
  // evaluate D once per difference, then fill the site-pair blocks.
  const int nd3 = n_d * n_d * n_d, nu = 3 * nd3;
  const int span = 2 * n_d - 1;
  const double step = a / n_d;
  std::vector<std::complex<double>> Dd((size_t)span * span * span * 9);
  for (int dx = 0; dx < span; ++dx)
    for (int dy = 0; dy < span; ++dy)
      for (int dz = 0; dz < span; ++dz) {
        const double R[3] = {a * w[0] + step * (dx - (n_d - 1)),
                             a * w[1] + step * (dy - (n_d - 1)),
                             a * w[2] + step * (dz - (n_d - 1))};
        std::complex<double> D[3][3];
        dyadic_green(R, k, eta, D);
        std::complex<double>* out = &Dd[(((size_t)dx * span + dy) * span + dz) * 9];
        for (int al = 0; al < 3; ++al)
          for (int be = 0; be < 3; ++be) out[3 * al + be] = D[al][be];
      }
  G.assign((size_t)nu * nu, 0.0);
  for (int l = 0; l < nd3; ++l) {
    const int lx = l / (n_d * n_d), ly = (l / n_d) % n_d, lz = l % n_d;
    for (int s = 0; s < nd3; ++s) {
      const int sx = s / (n_d * n_d), sy = (s / n_d) % n_d, sz = s % n_d;
      const std::complex<double>* D =
          &Dd[((((size_t)(lx - sx + n_d - 1)) * span + (ly - sy + n_d - 1)) * span +
               (lz - sz + n_d - 1)) * 9];
      for (int al = 0; al < 3; ++al)
        for (int be = 0; be < 3; ++be)
          G[(size_t)(3 * l + al) * nu + 3 * s + be] = D[3 * al + be];
    }
  }
}

// The four wavefronts of a group work on one chunk at a time, so a group's
// time is its number of chunks whatever their fill: ranges are balanced by
// chunk count. Trailing groups may get empty ranges.
void partition_groups(Plan& P, int64_t groups) {
  const int64_t nch = P.n_chunks();
  groups = std::min<int64_t>(groups, std::max<int64_t>(P.grid_units(), 1));
  groups = std::min<int64_t>((groups + 7) / 8 * 8, kMaxTranslateGroups);
  P.wg_ptr.assign(groups + 1, (int32_t)nch);
  P.wg_ptr[0] = 0;
  for (int64_t g = 1; g < groups; ++g) P.wg_ptr[g] = (int32_t)((nch * g + groups - 1) / groups);
}

void build_rounds(Plan& P, int64_t groups) {
  const int64_t ni = P.n_items();
  groups = std::min<int64_t>(groups, std::max<int64_t>(ni, 1));
  groups = std::min<int64_t>((groups + 7) / 8 * 8, kMaxTranslateGroups);
  P.rounds.clear();
  P.wg_round_ptr.assign(groups + 1, 0);
  const int32_t* it = P.items.data();
  for (int64_t g = 0; g < groups; ++g) {
    const int64_t ib = ni * g / groups, ie = ni * (g + 1) / groups;
    for (int64_t i = ib; i < ie;) {
      const int32_t o = it[4 * i];
      int64_t j = i;
      while (j < ie && it[4 * j] == o) ++j;
      const int32_t next = j < ie ? it[4 * j] + 1 : 0;  // next segment's offset + 1
      for (int64_t r = i; r < j; r += 4)
        for (int w = 0; w < 4; ++w) {
          const int64_t q = r + w;
          P.rounds.push_back(o);
          P.rounds.push_back(q < j ? it[4 * q + 1] : 0);
          P.rounds.push_back(q < j ? it[4 * q + 2] : 0);
          P.rounds.push_back(r == i ? (1 | (next << 1)) : 0);
        }
      i = j;
    }
    P.wg_round_ptr[g + 1] = (int32_t)(P.rounds.size() / 16);
  }
}

int64_t max_rounds(const Plan& p) {
  // ceil(items / 4) rounds, plus at most one partial round per segment;
  // segments are runs of one offset cut at most once per workgroup
  return p.n_items() / 4 + p.n_off() + kMaxTranslateGroups + 1;
}

namespace {

// Places allocations one after another, 256-byte aligned.
struct Taker {
  size_t at = 0;
  size_t operator()(size_t bytes) {
    const size_t here = at;
    at = align256(at + bytes);
    return here;
  }
};

size_t row_bytes(const Plan& p, int32_t nrhs) {
  // one spare row at the end receives the stores of idle matrix-core lanes
  return ((size_t)nrhs * p.n_pairs() + 1) * p.pstride() * sizeof(float);
}

}  // namespace

int64_t fft_block(const FftGroup& g, int32_t nrhs) {
  return std::max<int64_t>(1, std::min<int64_t>(nrhs, kFftScratch / std::max<int64_t>(g.len, 1)));
}

int64_t fft_scratch_len(const Plan& p, int32_t nrhs) {
  int64_t len = 0;
  for (const FftGroup& g : p.fft_groups) len = std::max(len, fft_block(g, nrhs) * g.len);
  return len;
}

size_t fft_scratch_bytes(const Plan& p, int32_t nrhs) {
  const size_t parts = 27 * kReachParts * (size_t)p.nu * 16;
  return (size_t)fft_scratch_len(p, nrhs) * 16 +
         (size_t)nrhs * (p.n_box * sizeof(float) + p.fft.size() * (kReachBytes + parts));
}

Layout workspace_layout(const Plan& p, int32_t max_nrhs) {
  Layout L{};
  Taker take;
  auto pairs = [&take](const Plan& q) {
    Layout::Pairs a{};
    a.table = take(q.table_bytes());
    a.chunks = take(q.chunks.size() * sizeof(int32_t));
    a.items = take(q.items.size() * sizeof(int32_t));
    a.wg_ptr = take((size_t)(kMaxTranslateGroups + 1) * sizeof(int32_t));
    a.rounds = take((size_t)max_rounds(q) * 16 * sizeof(int32_t));
    a.wg_round_ptr = take((size_t)(kMaxTranslateGroups + 1) * sizeof(int32_t));
    a.pair_src = take(q.pair_src.size() * sizeof(int32_t));
    a.pair_dst = take(q.pair_dst.size() * sizeof(int32_t));
    a.test_ptr = take(q.test_ptr.size() * sizeof(int32_t));
    a.off_scale = take((size_t)std::max<int32_t>(q.n_off(), 1) * sizeof(float));
    a.offsets = take((size_t)q.n_off() * 4 * sizeof(int32_t));
    return a;
  };
  if (holds_own_pairs(p)) L.own = pairs(p);
  if (p.rest) L.rest = pairs(*p.rest);
  L.nb_ptr = take((size_t)(p.n_box + 1) * sizeof(int64_t));
  L.P = take((size_t)max_nrhs * p.n_box * p.vstride() * sizeof(float));
  size_t rows = 0;
  if (holds_own_pairs(p)) rows = row_bytes(p, max_nrhs);
  if (p.rest) rows = std::max(rows, row_bytes(*p.rest, max_nrhs));
  L.part = take(rows);
  L.box_scale = take((size_t)max_nrhs * p.n_box * sizeof(float));
  if (p.rest) {
    L.fft = take(fft_scratch_bytes(p, max_nrhs));
    L.fft_spec = take((size_t)p.fft_spec_len * 16);
    L.fft_tw = take(p.fft_twiddles.size() * sizeof(double));
    L.fft_map = take(p.fft_map.size() * sizeof(int32_t));
    L.fft_cells = take(p.fft_cells.size() * sizeof(int32_t));
    L.fft_tasks = take(p.fft_tasks.size() * sizeof(FftTask));
  }
  L.total = take.at;
  return L;
}

ScratchLayout scratch_layout(const Plan& p, int32_t nrhs) {
  ScratchLayout L{};
  auto lay = [&](bool direct) {
    Taker take;
    L.P = take((size_t)nrhs * p.n_box * p.vstride() * sizeof(float));
    L.part = take(row_bytes(direct ? p : p.pairs_plan(), nrhs));
    L.box_scale = take((size_t)nrhs * p.n_box * sizeof(float));
    L.fft = take(direct ? 0 : fft_scratch_bytes(p, nrhs));
    return take.at;
  };
  L.direct = lay(true);
  // networks take the rows of every far pair
  L.total = p.rest && p.hidden == 0 ? lay(false) : L.direct;
  return L;
}

namespace {

// Work units of a plan's pairs: chunks of up to kChunk and items of up to 32
// consecutive pairs of one offset, and their default partitions.
void build_units(Plan& P) {
  P.chunks.clear();
  P.items.clear();
  auto cut = [&P](std::vector<int32_t>& out, int64_t size) {
    for (int32_t o = 0; o < P.n_off(); ++o)
      for (int64_t s = P.off_ptr[o]; s < P.off_ptr[o + 1]; s += size) {
        out.push_back(o);
        out.push_back((int32_t)s);
        out.push_back((int32_t)std::min<int64_t>(size, P.off_ptr[o + 1] - s));
        out.push_back(0);
      }
  };
  cut(P.chunks, kChunk);
  cut(P.items, 32);
  partition_groups(P, kTranslateGroups);
  build_rounds(P, kRoundGroups);
}

// Bytes of one offset's image in the table layout of the plan's form.
size_t image_bytes(const Plan& P) {
  return P.staged_split() ? P.staged_split_halves() * sizeof(uint16_t)
         : P.split()      ? (size_t)4 * P.nu * P.khb * sizeof(uint16_t)
         : P.staged()     ? P.staged_op_floats() * sizeof(float)
                          : (size_t)2 * P.nu * P.kh * sizeof(float);
}

// Operator table image, one offset at a time (cached across plans). Large
// tables (FULL far sets have one operator per distinct offset, ~10^5 on a
// few-thousand-box scatterer) are built on several host threads, each over a
// contiguous range of offsets.
void build_table(Plan& P) {
  const int64_t n_off = P.n_off();
  const size_t img_bytes = image_bytes(P);
  P.off_scale.assign(n_off, 1.0f);
  if (P.gen_ops) return;  // evaluated by the translation kernel
  if (P.split())
    P.table_bf16.assign((size_t)n_off * img_bytes / sizeof(uint16_t), 0);
  else
    P.table.assign((size_t)n_off * img_bytes / sizeof(float), 0.0f);
  char* table = P.split() ? (char*)P.table_bf16.data() : (char*)P.table.data();
  auto build_range = [&](int64_t lo, int64_t hi) {
    std::vector<std::complex<double>> G;
    for (int64_t o = lo; o < hi; ++o) {
      char* dst = table + (size_t)o * img_bytes;
      const int32_t* w = &P.offsets[3 * o];
      const bool m = P.masked((int32_t)o);
      if (!image_cache_get(P, w, m, dst, img_bytes, &P.off_scale[o])) {
        offset_image(P, w, m, G, dst, &P.off_scale[o]);
        image_cache_put(P, w, m, dst, img_bytes, P.off_scale[o]);
      }
    }
  };
  const int64_t kPerThread = 1024;
  const int hw = (int)std::max(1u, std::thread::hardware_concurrency());
  const int64_t nthr = std::min<int64_t>(std::min(hw, 16), (n_off + kPerThread - 1) / kPerThread);
  if (nthr <= 1) {
    build_range(0, n_off);
  } else {
    std::vector<std::thread> pool;
    for (int64_t t = 0; t < nthr; ++t)
      pool.emplace_back(build_range, n_off * t / nthr, n_off * (t + 1) / nthr);
    for (auto& th : pool) th.join();
  }
}

// Smallest 5-smooth length >= n, split into radices of 2..8, the largest
// first: as few as possible, and among those the split whose smallest radix
// is largest (L / radix butterflies run side by side: at most 256 up to
// kMaxFftLength, so the 3 components of a line fit a workgroup).
// False above kMaxFftLength.
bool fft_axis(int64_t n, FftAxis& ax) {
  for (int64_t L = std::max<int64_t>(n, 1); L <= kMaxFftLength; ++L) {
    int64_t m = L;
    for (int f : {2, 3, 5})
      while (m % f == 0) m /= f;
    if (m != 1) continue;
    std::vector<std::vector<int>> level = {{}};
    for (int depth = 0; depth <= kMaxFftStages; ++depth) {
      const std::vector<int>* best = nullptr;
      std::vector<std::vector<int>> next;
      for (const auto& f : level) {
        int64_t q = L;
        for (int r : f) q /= r;
        if (q == 1) {
          if (!best || (!f.empty() && f.back() > best->back())) best = &f;
        }
        for (int r : {8, 6, 5, 4, 3, 2})
          if (q % r == 0 && (f.empty() || r <= f.back())) {
            next.push_back(f);
            next.back().push_back(r);
          }
      }
      if (best) {
        ax.L = (int32_t)L;
        ax.stages = (int32_t)best->size();
        for (size_t i = 0; i < best->size(); ++i) ax.radix[i] = (*best)[i];
        return true;
      }
      level.swap(next);
    }
  }
  return false;
}

// LDS of one workgroup's lines: three workgroups share a compute unit (160 KB).
constexpr size_t kLineBytes = 50 << 10;

// Lines of a workgroup, of `all`: as many as the LDS budget and 512 threads
// take, but no fewer than 1,024 workgroups (four per compute unit) while a
// workgroup keeps a wavefront busy.
int fit_lines(const FftAxis& ax, int64_t all) {
  int w = 64;
  while (w > 1 && (48 * (size_t)ax.L * w > kLineBytes || 3 * ax.butterflies() * w > 512 ||
                   (all < 1024 * w && 3 * ax.butterflies() * w >= 128)))
    w /= 2;
  return w;
}
// Workgroups that share the n_d z lines of a plane of boxes.
int z_groups(const FftAxis& ax, int nd) {
  int groups = 1;
  while (groups < nd && (nd % groups || 3 * ax.butterflies() * (nd / groups) > 512)) ++groups;
  return groups;
}

// Tasks and groups of the plan's lattices: consecutive ones share launches
// while a right-hand side of them fits the scratch.
void build_fft_tasks(Plan& P) {
  for (size_t i = 0; i < P.fft.size(); ++i) {
    FftTask t{};
    t.g = P.fft[i];
    const FftGrid& g = t.g;
    t.index = (int32_t)i;
    const int64_t ny = (int64_t)g.s[0] * g.ax[2].L, nx = (int64_t)g.ax[1].L * g.ax[2].L;
    const int zg = z_groups(g.ax[2], P.n_d), yw = fit_lines(g.ax[1], ny),
              xw = fit_lines(g.ax[0], nx);
    const int32_t lines[3] = {P.n_d / zg, yw, xw};
    const int64_t blocks[3] = {(int64_t)g.n[0] * P.n_d * zg * g.n[1], (ny + yw - 1) / yw,
                               (nx + xw - 1) / xw};
    const int64_t len = g.zlen() + g.yzlen();
    if (P.fft_groups.empty() || P.fft_groups.back().len + len > kFftScratch) {
      P.fft_groups.emplace_back();
      P.fft_groups.back().first = (int32_t)i;
      P.fft_groups.back().count = 0;
    }
    FftGroup& G = P.fft_groups.back();
    t.z = G.len;
    t.yz = G.len + g.zlen();
    G.len += len;
    G.count += 1;
    for (int k = 0; k < 3; ++k) {
      const FftAxis& ax = g.ax[2 - k];
      t.lines[k] = lines[k];
      t.blocks[k] = (int32_t)blocks[k];
      t.first[k] = G.blocks[k];
      G.blocks[k] += t.blocks[k];
      G.threads[k] = std::max(G.threads[k], (3 * ax.butterflies() * lines[k] + 63) / 64 * 64);
      G.lds[k] = std::max(G.lds[k], (size_t)(3 * lines[k] + 1) * ax.L * 16);
    }
    P.fft_tasks.push_back(t);
  }
}

// Whether a scatterer's FULL product runs as a convolution: by estimates of
// both ways' microseconds for stages 2 and 3, fitted to both measured side by
// side on 90 plans: cubes, plates, lines, shells, hollow cubes and masks of 64
// to 2,000 boxes, n_d 1..4, FP32 and 16-bit forms (rms errors 15% and 7%).
// Measured, pairs against convolution: 4^3 boxes, n_d = 3 FP32 31 and 44,
// n_d = 4 59 and 75; 6^3, n_d = 3 16-bit 50 and 53, FP32 100 and 62; shells of
// 314 boxes, n_d = 1 17 and 37, n_d = 3 16-bit 119 and 76, of 762, n_d = 1 45
// and 38; a 40 x 23 plate, n_d = 1 39 and 38.
bool convolution_pays(const Plan& P, const FftGrid& g, double n_box, double n_pairs,
                      double n_rest, double n_off) {
  const double row = 4.0 * P.pstride();
  // the scratch has to fit where the rows of the pairs would be (a caller
  // without allocation has room for those)
  if (16.0 * (g.zlen() + g.yzlen() + 27.0 * kReachParts * P.nu) + row * (n_rest + 2.0 * n_box) >
      0.9 * row * n_pairs)
    return false;
  // of the pair kernels: per chunk (N_u = 192: item) of pairs of one offset,
  // and with few of them
  const double fp32[] = {0.56e-3, 2.3e-3, 30e-3, 51e-3}, half[] = {1.1e-3, 2.3e-3, 8.2e-3, 27e-3};
  const double unit = (P.split() ? half : fp32)[P.n_d - 1];
  const double start = P.split() || P.n_d < 3 ? 0.0 : (P.n_d == 3 ? 10.0 : 25.0);
  const double per_unit = P.nu == 192 ? 32 : kChunk;
  const double direct = 8.5 + start + unit * (n_off + n_pairs / per_unit) +
                        n_off * image_bytes(P) / 13e6 + 2.0 * row * n_pairs / 4.3e6;
  // the lattices, each transform in and out, and the spectrum; the pairs left
  const double lattices = 16.0 * (4.0 * g.zlen() + 4.0 * g.yzlen() + g.spec_len());
  const double conv = 30.0 + lattices / 2.35e6 +
                      (n_rest > 0 ? 10.6 + start + unit * n_rest / per_unit +
                                        2.0 * row * n_rest / 4.3e6
                                  : 0.0);
  return conv < direct;
}

// Lattices of the scatterers whose FULL product runs as a convolution, and
// the plan of the pairs left (FftGrid). P's far set is complete and grouped.
void build_convolution(Plan& P) {
  // not for the single FP16 product: its result would differ from the one
  // that form gives by the form's own error (2^-11 a term)
  if (P.far_mode != 1 || P.precision == 3) return;
  const int64_t np = P.n_pairs();
  const int32_t n_scat = P.n_scat();
  auto scat_of = [&P](int32_t box) {
    return (int32_t)(std::upper_bound(P.scat_ptr.begin(), P.scat_ptr.end(), (int64_t)box) -
                     P.scat_ptr.begin()) - 1;
  };
  std::vector<uint8_t> two(P.n_off());  // offsets a masked operator exists for
  for (int32_t o = 0; o < P.n_off(); ++o) {
    const int32_t* w = &P.offsets[3 * o];
    two[o] = P.n_d > 1 && cheb(w[0], w[1], w[2]) == 2;
  }
  // per scatterer: pairs, those of two, and offsets (pairs are grouped by
  // offset: a new one where it differs from the scatterer's last)
  std::vector<int64_t> n_pairs(n_scat, 0), n_rest(n_scat, 0), n_off(n_scat, 0);
  std::vector<int32_t> last(n_scat, -1);
  std::vector<int32_t> scat(n_scat > 1 ? np : 0);
  for (int64_t q = 0; q < np; ++q) {
    const int32_t s = n_scat > 1 ? (scat[q] = scat_of(P.pair_test[q])) : 0;
    n_pairs[s] += 1;
    n_rest[s] += two[P.pair_off[q]];
    n_off[s] += last[s] != P.pair_off[q];
    last[s] = P.pair_off[q];
  }
  std::vector<int32_t> grid_of(n_scat, -1);
  for (int32_t s = 0; s < n_scat; ++s) {
    FftGrid g{};
    int64_t lo[3], hi[3];
    for (int d = 0; d < 3; ++d) {
      lo[d] = std::numeric_limits<int32_t>::max();
      hi[d] = 0;
      for (int64_t i = P.scat_ptr[s]; i < P.scat_ptr[s + 1]; ++i) {
        lo[d] = std::min<int64_t>(lo[d], P.boxes[3 * i + d]);
        hi[d] = std::max<int64_t>(hi[d], P.boxes[3 * i + d]);
      }
    }
    bool fits = true;
    for (int d = 0; d < 3 && fits; ++d) {
      const int64_t n = hi[d] - lo[d] + 1;
      fits = n * P.n_d <= kMaxFftLength && fft_axis(2 * n * P.n_d - 1, g.ax[d]);
      g.n[d] = (int32_t)std::min<int64_t>(n, kMaxFftLength);
      g.s[d] = g.n[d] * P.n_d;
    }
    if (!fits || !convolution_pays(P, g, (double)(P.scat_ptr[s + 1] - P.scat_ptr[s]),
                                   (double)n_pairs[s], (double)n_rest[s], (double)n_off[s]))
      continue;
    grid_of[s] = (int32_t)P.fft.size();
    g.box = P.scat_ptr[s];
    g.count = P.scat_ptr[s + 1] - g.box;
    g.map = (int64_t)P.fft_map.size() / 2;
    P.fft_cells.resize(4 * (size_t)P.n_box, -1);
    P.fft_map.resize(P.fft_map.size() + 2 * (size_t)g.n[0] * g.n[1] * g.n[2], -1);
    for (int64_t i = P.scat_ptr[s]; i < P.scat_ptr[s + 1]; ++i) {
      const int32_t* c = &P.boxes[3 * i];
      const int64_t cell =
          g.map + ((c[0] - lo[0]) * g.n[1] + (c[1] - lo[1])) * g.n[2] + (c[2] - lo[2]);
      P.fft_map[2 * cell] = (int32_t)i;
      for (int d = 0; d < 3; ++d) P.fft_cells[4 * i + d] = (int32_t)(c[d] - lo[d]);
      P.fft_cells[4 * i + 3] = grid_of[s];
    }
    // a spectrum depends on the lattice alone: equal lattices share one
    g.spec = -1;
    for (const FftGrid& o : P.fft)
      if (std::equal(o.s, o.s + 3, g.s)) g.spec = o.spec;
    if (g.spec < 0) {
      g.spec = P.fft_spec_len;
      P.fft_spec_len += g.spec_len();
    }
    P.fft.push_back(g);
  }
  if (P.fft.empty()) return;
  for (const FftGrid& g : P.fft)
    P.fft_cells.insert(P.fft_cells.end(),
                       {(int32_t)g.box, (int32_t)g.count, (int32_t)(g.map & 0xffffffff),
                        (int32_t)(g.map >> 32), g.n[0], g.n[1], g.n[2], 0});
  for (FftGrid& g : P.fft)
    for (FftAxis& ax : g.ax) {
      ax.tw = (int32_t)P.fft_twiddles.size() / 2;
      for (const FftGrid& o : P.fft)
        for (const FftAxis& b : o.ax)
          if (&b < &ax && b.L == ax.L) ax.tw = b.tw;
      if (ax.tw < (int32_t)P.fft_twiddles.size() / 2) continue;
      for (int32_t k = 0; k < ax.L; ++k) {
        P.fft_twiddles.push_back(std::cos(2.0 * kPi * k / ax.L));
        P.fft_twiddles.push_back(-std::sin(2.0 * kPi * k / ax.L));
      }
    }

  build_fft_tasks(P);

  // The pairs left: all of a scatterer without a lattice, the masked ones of
  // the others; grouped by (offset, masked), in P's order within a group.
  auto R = std::make_unique<Plan>();
  R->n_box = P.n_box;
  R->scat_ptr = P.scat_ptr;
  R->a = P.a;
  R->k = P.k;
  R->eta = P.eta;
  R->n_d = P.n_d;
  R->nu = P.nu;
  R->kh = P.kh;
  R->khb = P.khb;
  R->far_mode = P.far_mode;
  R->precision = P.precision;
  R->gen_ops = P.gen_ops;
  R->off_ptr.push_back(0);
  for (int32_t o = 0; o < P.n_off(); ++o)
    for (int m = 0; m < 2; ++m) {
      if (m && !two[o]) continue;
      for (int64_t q = P.off_ptr[o]; q < P.off_ptr[o + 1]; ++q)
        if ((grid_of[n_scat > 1 ? scat[q] : 0] >= 0) == (m == 1)) {
          R->pair_test.push_back(P.pair_test[q]);
          R->pair_src.push_back(P.pair_src[q]);
        }
      if ((int64_t)R->pair_src.size() == R->off_ptr.back()) continue;
      R->off_ptr.push_back((int64_t)R->pair_src.size());
      R->offsets.insert(R->offsets.end(), &P.offsets[3 * o], &P.offsets[3 * o] + 3);
      R->op_masked.push_back((uint8_t)m);
    }
  // Rows: the convolution's (boxes of a lattice with a far pair; the others
  // get none, so that a box without far pairs stays exactly zero), then the
  // pairs' in grouped order.
  const int64_t nr = (int64_t)R->pair_src.size();
  std::vector<int32_t> conv(P.n_box, 0);
  for (int64_t j = 0; j < P.n_box; ++j)
    conv[j] = P.test_ptr[j + 1] > P.test_ptr[j] && grid_of[scat_of((int32_t)j)] >= 0;
  R->test_ptr.assign(P.n_box + 1, 0);
  for (int64_t q = 0; q < nr; ++q) R->test_ptr[R->pair_test[q] + 1]++;
  for (int64_t j = 0; j < P.n_box; ++j) R->test_ptr[j + 1] += R->test_ptr[j] + conv[j];
  std::vector<int32_t> fill(R->test_ptr.begin(), R->test_ptr.end() - 1);
  for (size_t c = 0; c < P.fft_map.size(); c += 2) {
    const int32_t box = P.fft_map[c];
    if (box >= 0 && conv[box]) P.fft_map[c + 1] = fill[box]++;
  }
  const int64_t n_rows = R->test_ptr.back();
  R->pair_dst.resize(nr);
  for (int64_t q = 0; q < nr; ++q) R->pair_dst[q] = fill[R->pair_test[q]]++;
  R->count_rows();
  build_units(*R);
  R->pair_src.resize(n_rows, 0);
  R->pair_dst.resize(n_rows, 0);
  build_table(*R);
  P.rest = std::move(R);
}

}  // namespace

std::string build_plan(const int32_t* box_ijk, int64_t n_box, double a,
                       double k, double eta, int n_d, int far_mode,
                       int precision, int operators, const int64_t* scat_ptr,
                       int64_t n_scat, Plan& P) {
  if (!box_ijk) return "box_ijk is NULL";
  if (n_box < 1) return "n_boxes must be >= 1";
  if (n_box > std::numeric_limits<int32_t>::max() / 2) return "n_boxes too large";
  if (!(a > 0.0) || !std::isfinite(a)) return "box side a must be > 0";
  if (!(k > 0.0) || !std::isfinite(k)) return "wavenumber k must be > 0";
  if (!(eta >= 0.0) || !std::isfinite(eta)) return "eta must be >= 0 (0 = free space)";
  if (n_d < 1 || n_d > 4) return "n_d must be in 1..4";
  if (far_mode != 0 && far_mode != 1) return "unknown far_mode";
  if (precision < 0 || precision > 3) return "unknown precision";
  if (operators != 0 && operators != 1) return "unknown operator source";
  if (operators == 1 && (precision == 0 || n_d > 3))
    return "generated operators need a 16-bit form (precision 1..3) and n_d 1..3";

  P.n_box = n_box;
  P.boxes.assign(box_ijk, box_ijk + 3 * n_box);
  for (int64_t i = 0; i < 3 * n_box; ++i)
    if (P.boxes[i] < 0) return "box coordinates must be >= 0";
  P.a = a;
  P.k = k;
  P.eta = eta == 0.0 ? kEta0 : eta;
  P.n_d = n_d;
  P.nu = 3 * n_d * n_d * n_d;
  P.kh = half_len(P.nu);
  P.khb = half_len_bf16(P.nu);
  P.far_mode = far_mode;
  P.precision = precision;
  P.gen_ops = operators == 1;

  if (scat_ptr) {
    if (n_scat < 1) return "n_scatterers must be >= 1";
    if (scat_ptr[0] != 0) return "scatterer_ptr[0] must be 0";
    for (int64_t s = 0; s < n_scat; ++s)
      if (scat_ptr[s + 1] <= scat_ptr[s]) return "every scatterer needs at least one box";
    if (scat_ptr[n_scat] != n_box) return "scatterer_ptr[n_scatterers] must equal n_boxes";
    P.scat_ptr.assign(scat_ptr, scat_ptr + n_scat + 1);
  } else {
    P.scat_ptr = {0, n_box};
  }
  const int32_t* b = P.boxes.data();

  // Far set: (test j, source i, offset w = c_j - c_i), test-major, built
  // within each scatterer (global box indices).
  std::vector<int32_t> pj, pi;
  std::vector<std::array<int32_t, 3>> pw;
  const int64_t kMaxPairs = std::numeric_limits<int32_t>::max();
  BoxIndex index;
  for (int64_t sc = 0; sc + 1 < (int64_t)P.scat_ptr.size(); ++sc) {
    const int64_t lo = P.scat_ptr[sc], hi = P.scat_ptr[sc + 1];
    if (!index.build(b + 3 * lo, hi - lo)) return "duplicate box coordinates";
    if (far_mode == 0) {
      for (int64_t j = lo; j < hi; ++j) {
        const int64_t cx = b[3 * j], cy = b[3 * j + 1], cz = b[3 * j + 2];
        for (int wx = -3; wx <= 3; ++wx)
          for (int wy = -3; wy <= 3; ++wy)
            for (int wz = -3; wz <= 3; ++wz) {
              if (cheb(wx, wy, wz) < 2) continue;
              const int64_t sx = cx - wx, sy = cy - wy, sz = cz - wz;
              const int32_t il = index.find(sx, sy, sz);
              if (il < 0) continue;
              if (cheb(floordiv2(cx) - floordiv2(sx), floordiv2(cy) - floordiv2(sy),
                       floordiv2(cz) - floordiv2(sz)) > 1)
                continue;
              if ((int64_t)pj.size() >= kMaxPairs) return "far set exceeds 2^31-1 pairs";
              pj.push_back((int32_t)j);
              pi.push_back((int32_t)(lo + il));
              pw.push_back({wx, wy, wz});
            }
      }
    } else {
      for (int64_t j = lo; j < hi; ++j)
        for (int64_t i = lo; i < hi; ++i) {
          const int64_t wx = (int64_t)b[3 * j] - b[3 * i];
          const int64_t wy = (int64_t)b[3 * j + 1] - b[3 * i + 1];
          const int64_t wz = (int64_t)b[3 * j + 2] - b[3 * i + 2];
          if (cheb(wx, wy, wz) < 2) continue;
          if ((int64_t)pj.size() >= kMaxPairs) return "far set exceeds 2^31-1 pairs";
          pj.push_back((int32_t)j);
          pi.push_back((int32_t)i);
          pw.push_back({(int32_t)wx, (int32_t)wy, (int32_t)wz});
        }
    }
  }
  if ((int64_t)pj.size() > kMaxPairs) return "far set exceeds 2^31-1 pairs";

  // Distinct offsets, lexicographic: collect them through a hash of the
  // pairs' offsets (far fewer than pairs), sort only those, then map.
  const int64_t np = (int64_t)pj.size();
  std::vector<int32_t> oid(np);
  std::vector<std::array<int32_t, 3>> uniq;
  {
    struct Hash {
      size_t operator()(const std::array<int32_t, 3>& w) const {
        uint64_t h = (uint32_t)w[0];
        h = h * 0x9E3779B97F4A7C15ull ^ (uint32_t)w[1];
        h = h * 0x9E3779B97F4A7C15ull ^ (uint32_t)w[2];
        return (size_t)(h ^ (h >> 29));
      }
    };
    std::unordered_map<std::array<int32_t, 3>, int32_t, Hash> seen;
    for (int64_t p = 0; p < np; ++p) {
      auto it = seen.find(pw[p]);
      if (it == seen.end()) {
        it = seen.emplace(pw[p], (int32_t)uniq.size()).first;
        uniq.push_back(pw[p]);
      }
      oid[p] = it->second;
    }
    std::vector<int32_t> order(uniq.size());
    std::iota(order.begin(), order.end(), 0);
    std::sort(order.begin(), order.end(),
              [&](int32_t x, int32_t y) { return uniq[x] < uniq[y]; });
    std::vector<int32_t> rank(uniq.size());
    std::vector<std::array<int32_t, 3>> sorted(uniq.size());
    for (size_t r = 0; r < order.size(); ++r) {
      rank[order[r]] = (int32_t)r;
      sorted[r] = uniq[order[r]];
    }
    uniq.swap(sorted);
    for (int64_t p = 0; p < np; ++p) oid[p] = rank[oid[p]];
  }
  const int64_t n_off = (int64_t)uniq.size();
  const size_t img_bytes = image_bytes(P);
  if (!P.gen_ops && (double)n_off * (double)img_bytes > kMaxTableBytes)
    return "operator table would exceed 16 GiB";
  P.offsets.resize(3 * n_off);
  for (int64_t o = 0; o < n_off; ++o)
    for (int d = 0; d < 3; ++d) P.offsets[3 * o + d] = uniq[o][d];

  // Stable counting sort of the pairs by offset.
  P.off_ptr.assign(n_off + 1, 0);
  for (int64_t p = 0; p < np; ++p) P.off_ptr[oid[p] + 1]++;
  for (int64_t o = 0; o < n_off; ++o) P.off_ptr[o + 1] += P.off_ptr[o];
  std::vector<int64_t> fill(P.off_ptr.begin(), P.off_ptr.end() - 1);
  P.pair_test.resize(np);
  P.pair_src.resize(np);
  P.pair_off.resize(np);
  for (int64_t p = 0; p < np; ++p) {
    const int64_t at = fill[oid[p]]++;
    P.pair_test[at] = pj[p];
    P.pair_src[at] = pi[p];
    P.pair_off[at] = oid[p];
  }

  // Test box -> positions of its pairs in the grouped order.
  P.test_ptr.assign(n_box + 1, 0);
  for (int64_t p = 0; p < np; ++p) P.test_ptr[P.pair_test[p] + 1]++;
  for (int64_t j = 0; j < n_box; ++j) P.test_ptr[j + 1] += P.test_ptr[j];
  std::vector<int32_t> tfill(P.test_ptr.begin(), P.test_ptr.end() - 1);
  P.test_pos.resize(np);
  for (int64_t p = 0; p < np; ++p) P.test_pos[tfill[P.pair_test[p]]++] = (int32_t)p;
  // Partial products are written at their test-major position, so the
  // pairs of one test box occupy consecutive rows.
  P.pair_dst.resize(np);
  for (int64_t q = 0; q < np; ++q) P.pair_dst[P.test_pos[q]] = (int32_t)q;

  P.count_rows();
  build_units(P);

  // Orbits under the 48 signed permutations: key = sorted |w|.
  std::vector<std::array<int32_t, 3>> keys(n_off);
  for (int64_t o = 0; o < n_off; ++o) {
    std::array<int32_t, 3> kk = {std::abs(uniq[o][0]), std::abs(uniq[o][1]),
                                 std::abs(uniq[o][2])};
    std::sort(kk.begin(), kk.end());
    keys[o] = kk;
  }
  std::sort(keys.begin(), keys.end());
  P.n_orbits = (int32_t)(std::unique(keys.begin(), keys.end()) - keys.begin());

  P.off_scale.assign(n_off, 1.0f);
  build_convolution(P);
  if (!P.rest) build_table(P);
  return std::string();
}

}  // namespace ubf
