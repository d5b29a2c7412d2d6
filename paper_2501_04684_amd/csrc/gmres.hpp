// Restarted GMRES for (sigma I + Z^F) x = b on one plan: device state and
// the kernel launchers (gmres.hip). All sums, norms and the Hessenberg /
// Givens / least-squares state are FP64; Krylov vectors are complex64.
#pragma once

#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>

#include <cstdint>

namespace ubf {

constexpr int kMaxRestart = 128;  // Krylov columns per cycle (restart length)
constexpr int kMaxGmresRhs = 64;  // right-hand sides per solver
constexpr int kDotBlocks = 256;   // most blocks of the two-level sums
constexpr int kSlice = 2048;      // elements of a block's slice (more once kDotBlocks are out)

// Blocks per right-hand side of the vector kernels.
inline int gmres_blocks(int64_t n) {
  const int64_t b = (n + kSlice - 1) / kSlice;
  return (int)(b < 1 ? 1 : (b > kDotBlocks ? kDotBlocks : b));
}

// Per-RHS row copied to the host after each step.
struct GmresStatusRow {
  double res;     // relative residual estimate |g_{k}| / ||b||
  int32_t active; // 1 while the right-hand side is still iterating
  int32_t iters;  // Arnoldi steps taken
};

// Device pointers into the solver workspace (passed to kernels by value).
struct GmresState {
  int m;            // restart length
  double2* H;       // [R][m][m+1]: column j of rhs r at (r*m + j)*(m+1)
  double2* h1;      // [R][m+1] first Gram-Schmidt pass
  double2* h2;      // [R][m+1] second pass
  double2* nrm;     // [1] norm estimate: sum |w|^2 (real part)
  double* cs;       // [R][m] Givens cosines
  double2* sn;      // [R][m] Givens sines
  double2* g;       // [R][m+1] rotated least-squares right-hand side
  double2* y;       // [R][m] cycle coefficients
  double* scale;    // [1] scale of the norm estimate's vector
  double* bnorm;    // [R] ||b||
  double* res;      // [R] relative residual estimate
  int32_t* k;       // [R] columns of the current cycle
  int32_t* iters;   // [R]
};

// One Arnoldi step after w = Z v_j (four launches): w += sigma v_j, two
// classical Gram-Schmidt passes, v_{j+1}, the rotations and the status rows
// (written by the kernel; the caller's pinned host memory). partial and
// partial2 hold [R][m + 1][gmres_blocks(n)] each; partial2 may lie in vnext,
// which is written last. active_in/active_out: the flags before and after the
// step (different arrays).
int launch_gmres_step(const GmresState& st, const float2* V, int64_t vstride, int j, float2* w,
                      float2* vnext, double sr, double si, double tol, int64_t n, int R,
                      double2* partial, double2* partial2, const int32_t* active_in,
                      int32_t* active_out, GmresStatusRow* status, hipStream_t s);
// x = 0, v0 = b, and v0 = b - sigma x - ax: each leaves the partials of
// ||v0||^2, which launch_gmres_cycle_start (next on the stream) adds up.
int launch_gmres_begin(const float2* b, float2* x, float2* v0, int64_t n, int R,
                       double2* partial, hipStream_t s);
int launch_gmres_residual(float2* v0, const float2* b, const float2* x, const float2* ax,
                          double sr, double si, int64_t n, int R, double2* partial,
                          hipStream_t s);
int launch_gmres_cycle_start(const GmresState& st, int first, double tol, float2* v0, int64_t n,
                             int R, const double2* partial, const int32_t* active_in,
                             int32_t* active_out, GmresStatusRow* status, hipStream_t s);
// x += V y with y from the triangular system of the cycle.
int launch_gmres_combine(const float2* V, int64_t vstride, const GmresState& st, float2* x,
                         int64_t n, int R, hipStream_t s);
// conj(a)^T b of one pair of vectors into *out.
int launch_gmres_dot(const float2* a, const float2* b, int64_t n, double2* partial, double2* out,
                     hipStream_t s);
int launch_gmres_scale(float2* dst, const float2* src, const double* sc, int64_t n,
                       hipStream_t s);
int launch_gmres_rand(float2* v, int64_t n, uint64_t seed, hipStream_t s);
int launch_gmres_conj(float2* dst, const float2* src, int64_t n, hipStream_t s);
int launch_gmres_inv_norm(const double2* nrm, double* scale, hipStream_t s);

}  // namespace ubf
