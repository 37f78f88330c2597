// FP64 vector kernels of the device GMRES (Saad-Schultz, restarted, right
// preconditioned with the 2x2 panel blocks of the singular entries).  All
// reductions are two-pass with a fixed order, so results are reproducible.
#include <algorithm>

#include "kernels.hpp"

namespace pbmp {

namespace {

constexpr int kB = 256;

typedef double d2 __attribute__((ext_vector_type(2)));

// sum over the block (fixed order), for thread 0
__device__ __forceinline__ double block_sum(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = red[0];
  for (int w = 1; w < kB / 64; ++w) t += red[w];
  return t;
}

// Block (b, k): the part of v_k . w in elements [b per, (b + 1) per), per even,
// vectors 16-byte aligned.  HBM bound on large surfaces; on small ones the
// latency of its loads and of the reduction, which takes lane shuffles and one
// barrier.
__global__ __launch_bounds__(kB) void k_mdot_partial(int n, const double *__restrict__ V,
                                                     size_t ld,
                                                     const double *__restrict__ w,
                                                     int per_block,
                                                     double *__restrict__ partial) {
  __shared__ double red[kB / 64];
  const int k = blockIdx.y;
  const int b = blockIdx.x;
  const int i0 = b * per_block, i1 = min(n, i0 + per_block);
  const double *v = V + (size_t)k * ld;
  const d2 *v2 = reinterpret_cast<const d2 *>(v + i0);
  const d2 *w2 = reinterpret_cast<const d2 *>(w + i0);
  const int np = max(0, i1 - i0) / 2;
  double a0 = 0.0, a1 = 0.0;
#pragma unroll 4
  for (int p = threadIdx.x; p < np; p += kB) {
    const d2 x = v2[p], y = w2[p];
    a0 += x.x * y.x;
    a1 += x.y * y.y;
  }
  const double t = block_sum(a0 + a1, red);
  if (threadIdx.x == 0) partial[(size_t)k * gridDim.x + b] = t;
}

__global__ void k_mdot_final(int nv, int nblk, const double *__restrict__ partial,
                             double *__restrict__ h) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nv) return;
  double s = 0.0;
  for (int b = 0; b < nblk; ++b) s += partial[(size_t)k * nblk + b];
  h[k] = s;
}

__global__ void k_gemv_sub(int n, int nv, const double *__restrict__ V, size_t ld,
                           const double *__restrict__ h, double *__restrict__ w) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int k = 0; k < nv; ++k) s += V[(size_t)k * ld + i] * h[k];
  w[i] -= s;
}

// The Arnoldi step's reductions without separate final passes: every
// block of the consuming kernel adds the k_mdot_partial block sums itself
// (nv * nblk values, four lanes to a vector, the same order in every block, so
// all blocks hold the same totals) and block 0 also stores them for the host.
constexpr int kMaxNV = 256;

__device__ inline void sum_partials(int nv, int nblk, const double *__restrict__ partial,
                                    double *h, double *__restrict__ hout) {
  for (int t = threadIdx.x; t < 4 * nv; t += kB) {
    const double *pk = partial + (size_t)(t / 4) * nblk;
    double s = 0.0;
    for (int b = t % 4; b < nblk; b += 4) s += pk[b];
    s += __shfl_xor(s, 1, 4);
    s += __shfl_xor(s, 2, 4);
    if (t % 4 == 0) {
      h[t / 4] = s;
      if (blockIdx.x == 0) hout[t / 4] = s;
    }
  }
  __syncthreads();
}

// w -= V h with h summed from the partials (stored to hout by block 0); NORM:
// also the block's share of |w|^2, so that the step's norm needs no pass of its
// own
template <bool NORM>
__global__ __launch_bounds__(kB) void k_gemv_sub_p(int n, int nv, const double *__restrict__ V,
                                                   size_t ld, int nblk,
                                                   const double *__restrict__ partial,
                                                   double *__restrict__ hout,
                                                   double *__restrict__ w,
                                                   double *__restrict__ norm) {
  __shared__ double h[kMaxNV];
  __shared__ double red[kB / 64];
  sum_partials(nv, nblk, partial, h, hout);
  const int i = blockIdx.x * kB + threadIdx.x;
  double r = 0.0;
  if (i < n) {
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < nv; ++k) s += V[(size_t)k * ld + i] * h[k];
    r = w[i] - s;
    w[i] = r;
  }
  if (NORM) {
    const double t = block_sum(r * r, red);
    if (threadIdx.x == 0) norm[blockIdx.x] = t;
  }
}

// block [[1/2, -a], [1/2, e b]]^{-1} = 1/det [[e b, a], [-1/2, 1/2]],
// det = (e b + a) / 2, and its transpose
__device__ inline void block_solve(double a, double b, double e, double u1,
                                   double u2, double &z1, double &z2) {
  const double det = 0.5 * (e * b + a);
  z1 = (e * b * u1 + a * u2) / det;
  z2 = (-0.5 * u1 + 0.5 * u2) / det;
}

__device__ inline void block_solve_T(double a, double b, double e, double u1, double u2,
                                     double &z1, double &z2) {
  const double det = 0.5 * (e * b + a);
  z1 = (e * b * u1 - 0.5 * u2) / det;
  z2 = (a * u1 + 0.5 * u2) / det;
}

// strengths of the panel's record (as k_pack_strengths)
__device__ inline void pack_record(int i, int nf, double area, double e, double z1, double z2,
                                   double *__restrict__ src64, float *__restrict__ src32) {
  const double wA = area * 0.07957747154594767 / nf;  // A / (4 pi nf)
  const double sv = wA * z2, sk = wA * z1;
  src64[16 * (size_t)i + 13] = sv;
  src64[16 * (size_t)i + 14] = sk;
  src64[16 * (size_t)i + 15] = e * sv;
  src32[16 * (size_t)i + 13] = (float)sv;
  src32[16 * (size_t)i + 14] = (float)sk;
  src32[16 * (size_t)i + 15] = (float)(e * sv);
}

// v = w / |w| with |w|^2 summed from the nb block shares (stored to hout by
// block 0; a zero vector, Arnoldi breakdown, stays zero), and the next step's
// product input in the same launch.  MODE 0: v alone (any n); 1: also z =
// M^{-1} v with the strengths of z packed into the source records; 2: z =
// M^{-T} v (1 and 2: n = 2N, one thread per panel).
template <int MODE>
__global__ __launch_bounds__(kB) void k_next_vector(
    int n, int nb, const double *__restrict__ norm, double *__restrict__ hout,
    const double *__restrict__ w, double *__restrict__ v, int nf,
    const double *__restrict__ diag, double e, const double *__restrict__ geo,
    double *__restrict__ z, double *__restrict__ src64, float *__restrict__ src32) {
  __shared__ double red[kB / 64];
  double q = 0.0;
  for (int b = threadIdx.x; b < nb; b += kB) q += norm[b];
  q = block_sum(q, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) *hout = q;
  const int i = blockIdx.x * kB + threadIdx.x;
  const double root = sqrt(q);
  if (MODE == 0) {
    if (i < n) v[i] = q > 0.0 ? w[i] / root : 0.0;
    return;
  }
  const int N = n / 2;
  if (i >= N) return;
  const double u1 = q > 0.0 ? w[i] / root : 0.0, u2 = q > 0.0 ? w[N + i] / root : 0.0;
  v[i] = u1;
  v[N + i] = u2;
  double z1, z2;
  if (MODE == 1) block_solve(diag[i], diag[N + i], e, u1, u2, z1, z2);
  else block_solve_T(diag[i], diag[N + i], e, u1, u2, z1, z2);
  z[i] = z1;
  z[N + i] = z2;
  if (MODE == 1) pack_record(i, nf, geo[6 * (size_t)N + i], e, z1, z2, src64, src32);
}

__global__ void k_axpy(int n, double a, const double *__restrict__ x,
                       double *__restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] += a * x[i];
}

__global__ void k_scale(int n, double a, const double *__restrict__ x,
                        double *__restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = a * x[i];
}

__global__ void k_xmy(int n, const double *__restrict__ b,
                      const double *__restrict__ ax, double *__restrict__ r) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r[i] = b[i] - ax[i];
}

__global__ void k_precond(int N, const double *__restrict__ diag, double e,
                          const double *__restrict__ u, double *__restrict__ z) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  double z1, z2;
  block_solve(diag[i], diag[N + i], e, u[i], u[N + i], z1, z2);
  z[i] = z1;
  z[N + i] = z2;
}

// z = M^{-1} u (as k_precond) and the far-field strengths of z packed into
// the source records (as k_pack_strengths): the Arnoldi step's product
// input in one launch
__global__ void k_precond_pack(int N, int nf, const double *__restrict__ diag, double e,
                               const double *__restrict__ geo, const double *__restrict__ u,
                               double *__restrict__ z, double *__restrict__ src64,
                               float *__restrict__ src32) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  double z1, z2;
  block_solve(diag[i], diag[N + i], e, u[i], u[N + i], z1, z2);
  z[i] = z1;
  z[N + i] = z2;
  pack_record(i, nf, geo[6 * (size_t)N + i], e, z1, z2, src64, src32);
}

__global__ void k_precond_T(int N, const double *__restrict__ diag, double e,
                            const double *__restrict__ u, double *__restrict__ z) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  double z1, z2;
  block_solve_T(diag[i], diag[N + i], e, u[i], u[N + i], z1, z2);
  z[i] = z1;
  z[N + i] = z2;
}

__global__ void k_update_solution(int N, int nv, const double *__restrict__ V,
                                  size_t ld, const double *__restrict__ y,
                                  const double *__restrict__ diag, double e,
                                  double *__restrict__ x) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  double u1 = 0.0, u2 = 0.0;
  for (int k = 0; k < nv; ++k) {
    u1 += V[(size_t)k * ld + i] * y[k];
    u2 += V[(size_t)k * ld + N + i] * y[k];
  }
  double z1, z2;
  block_solve(diag[i], diag[N + i], e, u1, u2, z1, z2);
  x[i] += z1;
  x[N + i] += z2;
}

__global__ void k_permute(int n, int blocks, const int *__restrict__ perm,
                          const double *__restrict__ in, double *__restrict__ out,
                          int gather) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * blocks) return;
  const int b = t / n, i = t % n;
  const size_t o = (size_t)b * n;
  if (gather)
    out[o + i] = in[o + perm[i]];
  else
    out[o + perm[i]] = in[o + i];
}

inline dim3 g1(int n) { return dim3((n + kB - 1) / kB); }

}  // namespace

namespace {
// Blocks per vector of the dot products: about 2048 blocks in all, between 8
// and 64 per vector of at least 1024 elements (every consumer block adds all
// of them).
inline int mdot_blocks(int n, int nv) {
  const int most = (n + 1023) / 1024;
  return std::max(1, std::min(most, std::max(8, std::min(64, 2048 / nv))));
}
inline int mdot_per(int n, int nblk) { return ((n + nblk - 1) / nblk + 1) / 2 * 2; }
}  // namespace

size_t krylov_partials(int n, int m) {
  // the largest nv * mdot_blocks for nv <= m + 1
  size_t most = 0;
  for (int nv = 1; nv <= m + 1; ++nv) most = std::max(most, (size_t)nv * mdot_blocks(n, nv));
  return most;
}

void launch_mdot(hipStream_t s, int n, int nv, const double *V, size_t ld,
                 const double *w, double *partial, double *h) {
  const int nblk = launch_mdot_partial(s, n, nv, V, ld, w, partial);
  hipLaunchKernelGGL(k_mdot_final, dim3((nv + 63) / 64), dim3(64), 0, s, nv,
                     nblk, partial, h);
  PBMP_HIP(hipGetLastError());
}

int launch_mdot_partial(hipStream_t s, int n, int nv, const double *V, size_t ld,
                        const double *w, double *partial) {
  if (n % 2 || ld % 2) throw Error(PBMP_EARG, "odd Krylov vector length");
  const int nblk = mdot_blocks(n, nv);
  hipLaunchKernelGGL(k_mdot_partial, dim3(nblk, nv), dim3(kB), 0, s, n, V, ld, w,
                     mdot_per(n, nblk), partial);
  PBMP_HIP(hipGetLastError());
  return nblk;
}

int launch_gemv_sub_p(hipStream_t s, int n, int nv, const double *V, size_t ld, int nblk,
                      const double *partial, double *hout, double *w, double *norm) {
  if (nv > kMaxNV) throw Error(PBMP_EARG, "too many Krylov vectors");
  const dim3 g = g1(n);
  if (norm)
    hipLaunchKernelGGL(k_gemv_sub_p<true>, g, dim3(kB), 0, s, n, nv, V, ld, nblk, partial, hout,
                       w, norm);
  else
    hipLaunchKernelGGL(k_gemv_sub_p<false>, g, dim3(kB), 0, s, n, nv, V, ld, nblk, partial,
                       hout, w, norm);
  PBMP_HIP(hipGetLastError());
  return (int)g.x;
}

void launch_next_vector(hipStream_t s, int mode, int n, int nb, const double *norm, double *hout,
                        const double *w, double *v, int nf, const double *diag, double eps_ratio,
                        const double *geo, double *z, double *src64, float *src32) {
#define PBMP_NV(M)                                                                           \
  hipLaunchKernelGGL(k_next_vector<M>, g1(M ? n / 2 : n), dim3(kB), 0, s, n, nb, norm, hout, \
                     w, v, nf, diag, eps_ratio, geo, z, src64, src32)
  if (mode == 1) PBMP_NV(1);
  else if (mode == 2) PBMP_NV(2);
  else PBMP_NV(0);
#undef PBMP_NV
  PBMP_HIP(hipGetLastError());
}

void launch_precond_T(hipStream_t s, int N, const double *diag, double eps_ratio,
                      const double *u, double *z) {
  hipLaunchKernelGGL(k_precond_T, g1(N), dim3(kB), 0, s, N, diag, eps_ratio, u, z);
  PBMP_HIP(hipGetLastError());
}

void launch_gemv_sub(hipStream_t s, int n, int nv, const double *V, size_t ld,
                     const double *h, double *w) {
  hipLaunchKernelGGL(k_gemv_sub, g1(n), dim3(kB), 0, s, n, nv, V, ld, h, w);
  PBMP_HIP(hipGetLastError());
}

void launch_axpy(hipStream_t s, int n, double a, const double *x, double *y) {
  hipLaunchKernelGGL(k_axpy, g1(n), dim3(kB), 0, s, n, a, x, y);
  PBMP_HIP(hipGetLastError());
}

void launch_scale(hipStream_t s, int n, double a, const double *x, double *y) {
  hipLaunchKernelGGL(k_scale, g1(n), dim3(kB), 0, s, n, a, x, y);
  PBMP_HIP(hipGetLastError());
}

void launch_xmy(hipStream_t s, int n, const double *b, const double *ax,
                double *r) {
  hipLaunchKernelGGL(k_xmy, g1(n), dim3(kB), 0, s, n, b, ax, r);
  PBMP_HIP(hipGetLastError());
}

void launch_precond(hipStream_t s, int N, const double *diag, double eps_ratio,
                    const double *u, double *z) {
  hipLaunchKernelGGL(k_precond, g1(N), dim3(kB), 0, s, N, diag, eps_ratio, u, z);
  PBMP_HIP(hipGetLastError());
}

void launch_precond_pack(hipStream_t s, int N, int nf, const double *diag, double eps_ratio,
                         const double *geo, const double *u, double *z, double *src64,
                         float *src32) {
  hipLaunchKernelGGL(k_precond_pack, g1(N), dim3(kB), 0, s, N, nf, diag, eps_ratio, geo, u, z,
                     src64, src32);
  PBMP_HIP(hipGetLastError());
}

void launch_update_solution(hipStream_t s, int N, int nv, const double *V,
                            size_t ld, const double *y, const double *diag,
                            double eps_ratio, double *x) {
  hipLaunchKernelGGL(k_update_solution, g1(N), dim3(kB), 0, s, N, nv, V, ld, y,
                     diag, eps_ratio, x);
  PBMP_HIP(hipGetLastError());
}

void launch_permute(hipStream_t s, int n, int blocks, const int *perm,
                    const double *in, double *out, bool gather) {
  hipLaunchKernelGGL(k_permute, g1(n * blocks), dim3(kB), 0, s, n, blocks, perm,
                     in, out, gather ? 1 : 0);
  PBMP_HIP(hipGetLastError());
}

namespace {
__global__ void k_add_strided(int n, double sign, const double *__restrict__ p, int stride,
                              double *__restrict__ y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] += sign * p[(size_t)stride * i];
}
}  // namespace

// y[i] += sign * p[stride * i]
void launch_add_strided(hipStream_t s, int n, double sign, const double *p, int stride,
                        double *y) {
  hipLaunchKernelGGL(k_add_strided, dim3((n + 255) / 256), dim3(256), 0, s, n, sign, p, stride,
                     y);
  PBMP_HIP(hipGetLastError());
}

}  // namespace pbmp
