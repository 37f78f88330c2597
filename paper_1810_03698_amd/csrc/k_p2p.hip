// Far-field source-target (P2P) sums of the boundary-integral operator
// (section "The treecode algorithm": the product is an N-body problem with
// the Gauss nodes as sources and the collocation points as targets), and the
// step that adds the partial rows and the near/self correction to y = A x
// (eq. integral_eq).
//
// Layout: one target per lane, source panels staged through LDS in tiles;
// the lanes of a wave read the same panel record (LDS broadcast).  A panel
// record is 16 words: three far-field nodes, the unit normal, the plane
// offset n.y (the site readout's) and the strengths s_V, s_K, eps s_V.
// The nodes of a flat panel share its plane, so n.R for R = x - y_q is the same
// for all q; the products take it from the first node's difference vector.
//
// Per (target, node) pair one reciprocal square root and one exponential give
// both rows of y = A x, the layers combined per node (pair.hpp):
//   (s_K n.R / r^2 - s_V) / r   and   (eps s_V - s_K n.R (1/r + k) / r) e^{-kr} / r.
// FP32 variant: per-tile FP32 sums folded into FP64 accumulators.
#include <algorithm>
#include <cmath>

#include "kernels.hpp"
#include "pair.hpp"

namespace pbmp {

namespace {

constexpr double kInv4Pi = 0.07957747154594767;
constexpr int kBlock = 256;
constexpr int kTile = 128;  // panels per LDS tile

// x = the caller's vector gathered into the internal panel order, and its
// strengths packed (as k_pack_strengths): a product's input in one launch
__global__ void k_gather_pack(int N, int nf, double eps_ratio, const int *__restrict__ perm,
                              const double *__restrict__ geo, const double *__restrict__ user,
                              double *__restrict__ x, double *__restrict__ src64,
                              float *__restrict__ src32) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const double ph = user[perm[j]], dp = user[N + perm[j]];
  x[j] = ph;
  x[N + j] = dp;
  const double wA = geo[6 * (size_t)N + j] * kInv4Pi / nf;  // equal-weight rules
  const double sv = wA * dp, sk = wA * ph;
  src64[16 * (size_t)j + 13] = sv;
  src64[16 * (size_t)j + 14] = sk;
  src64[16 * (size_t)j + 15] = eps_ratio * sv;
  src32[16 * (size_t)j + 13] = (float)sv;
  src32[16 * (size_t)j + 14] = (float)sk;
  src32[16 * (size_t)j + 15] = (float)(eps_ratio * sv);
}

__global__ void k_pack_strengths(int N, int nf, double eps_ratio,
                                 const double *__restrict__ geo,
                                 const double *__restrict__ x,
                                 double *__restrict__ src64,
                                 float *__restrict__ src32) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const double wA = geo[6 * N + j] * kInv4Pi / nf;  // equal-weight rules
  const double sv = wA * x[N + j];
  const double sk = wA * x[j];
  src64[16 * (size_t)j + 13] = sv;
  src64[16 * (size_t)j + 14] = sk;
  src64[16 * (size_t)j + 15] = eps_ratio * sv;
  src32[16 * (size_t)j + 13] = (float)sv;
  src32[16 * (size_t)j + 14] = (float)sk;
  src32[16 * (size_t)j + 15] = (float)(eps_ratio * sv);
}

// Direct product.  A block takes 64 targets, one per lane, and one source chunk:
// its four waves stage the chunk's records tile by tile and each takes every
// fourth panel; the waves' sums are added through LDS in wave order.  VALU issue
// bound.  One target per lane and eight blocks per CU measured fastest: 19220
// panels in FP32 took 507 us, with two, three and four targets per lane 519,
// 590 and 606 us; 8000 panels 88, 91, 101 and 105 us (256 targets to a block,
// two per lane, all waves on the same panels, as before: 640 and 105 us).
template <class T, int NF, bool FLOOR>
__global__ __launch_bounds__(kBlock) void k_p2p(const T *__restrict__ src, int N,
                                                const T *__restrict__ tgt, int Nt, int chunk,
                                                T kappa, double *__restrict__ part) {
  constexpr int kWaves = kBlock / 64;
  constexpr int kTileR = sizeof(T) == 4 ? kTile : kTile / 2;  // records per tile (8 KB)
  constexpr int PER = (int)sizeof(T);                         // 16-byte units per record
  typedef T v2 __attribute__((ext_vector_type(16 / sizeof(T))));
  __shared__ __align__(16) T sh[kTileR * 16];
  __shared__ double red[kWaves - 1][2][64];
  __shared__ double etab[sizeof(T) == 8 ? 64 : 1];
  const Screen<T> sc = make_screen(kappa, etab);
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int j0 = blockIdx.y * chunk;
  const int j1 = min(N, j0 + chunk);
  const int ti = blockIdx.x * 64 + lane, tl = min(ti, Nt - 1);
  const T px = tgt[tl], py = tgt[Nt + tl], pz = tgt[2 * (size_t)Nt + tl];
  double S[2] = {0.0, 0.0};
  for (int jt = j0; jt < j1; jt += kTileR) {
    const int nj = min(kTileR, j1 - jt);
    __syncthreads();
    const v2 *g = reinterpret_cast<const v2 *>(src + (size_t)jt * 16);
    for (int e = threadIdx.x; e < nj * PER; e += kBlock) reinterpret_cast<v2 *>(sh)[e] = g[e];
    __syncthreads();
    T a[2][kAcc<T, NF>];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      for (int q = 0; q < kAcc<T, NF>; ++q) a[c][q] = T(0);
    for (int jj = wave; jj < nj; jj += kWaves)
      panel_rows<NF, FLOOR>(sh + 16 * jj, px, py, pz, sc, a);
#pragma unroll
    for (int c = 0; c < 2; ++c)
      for (int q = 0; q < kAcc<T, NF>; ++q) S[c] += (double)a[c][q];
  }
  if (wave > 0)
    for (int c = 0; c < 2; ++c) red[wave - 1][c][lane] = S[c];
  __syncthreads();
  if (wave == 0 && ti < Nt)
    for (int c = 0; c < 2; ++c) {
      double v = S[c];
      for (int w = 0; w < kWaves - 1; ++w) v += red[w][c][lane];
      part[((size_t)blockIdx.y * 2 + c) * Nt + ti] = v;
    }
}

// y = A x from the far partials and the near/self correction.  Eight lanes
// per row: lane u takes the row's chunks u, u + 8, ... and its correction
// entries u, u + 8, ...; one lane per row walked both lists serially, about
// 100 dependent scattered loads (30 us on 8000 rows).
constexpr int kFinLanes = 8;

__global__ __launch_bounds__(kBlock) void k_finish(
    int N, int nchunk, const double *__restrict__ part, const int *__restrict__ rowptr,
    const int *__restrict__ col, const double *__restrict__ val, const double *__restrict__ x,
    double eps_ratio, const int *__restrict__ perm, double *__restrict__ y) {
  const int t = blockIdx.x * kBlock + (int)threadIdx.x;
  const int i = t / kFinLanes, u = t % kFinLanes;
  const int il = min(i, N - 1);
  double S[2] = {0.0, 0.0};
  for (int c = u; c < nchunk; c += kFinLanes)
    for (int k = 0; k < 2; ++k) S[k] += part[((size_t)c * 2 + k) * N + il];
  const int e1 = rowptr[il + 1];
  for (int e = rowptr[il] + u; e < e1; e += kFinLanes) {
    const int j = col[e];
    const double ph = x[j], dp = x[N + j];
    const double *v = val + 4 * (size_t)e;
    S[0] += v[1] * ph - v[0] * dp;
    S[1] += eps_ratio * v[2] * dp - v[3] * ph;
  }
  for (int w = 1; w < kFinLanes; w <<= 1)
    for (int k = 0; k < 2; ++k) S[k] += __shfl_xor(S[k], w, kFinLanes);
  if (i >= N || u != 0) return;
  const double ph = x[i];
  const int o = perm ? perm[i] : i;
  y[o] = 0.5 * ph + S[0];
  y[N + o] = 0.5 * ph + S[1];
}

// Transposed far-field sums: targets are the far-field nodes of panel j
// (normal n_j), sources the collocation points c_i with weights z1_i, z2_i:
//   T_VL_j = sum_q w A_j/(4 pi) sum_i z1_i / r,   T_KL_j = ... z1_i n_j.(c_i - y)/r^3
//   T_VY_j = ... z2_i e^{-kr}/r,                   T_KY_j = ... z2_i n_j.(c_i-y)(1+kr)e^{-kr}/r^3
// Blocks as in k_p2p with the roles exchanged: 64 panels on the lanes, the
// chunk's collocation points staged through LDS, every fourth one to a wave.
template <class T, int NF, bool FLOOR>
__global__ __launch_bounds__(kBlock) void k_p2p_transpose(
    int N, const T *__restrict__ src, const T *__restrict__ tgt, const double *__restrict__ geo,
    const double *__restrict__ z, int chunk, T kappa, double eps_ratio,
    double *__restrict__ part) {
  constexpr int kWaves = kBlock / 64;
  constexpr int kRec = 8;  // x y z z1 z2 eps z2
  __shared__ __align__(16) T sh[kTile * kRec];
  __shared__ double red[kWaves - 1][2][64];
  __shared__ double etab[sizeof(T) == 8 ? 64 : 1];
  const Screen<T> sc = make_screen(kappa, etab);
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int sj = blockIdx.x * 64 + lane, jl = min(sj, N - 1);
  T rec[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) rec[c] = src[16 * (size_t)jl + c];
  const int i0 = blockIdx.y * chunk, i1 = min(N, i0 + chunk);
  double S[2] = {0.0, 0.0};
  for (int it = i0; it < i1; it += kTile) {
    const int ni = min(kTile, i1 - it);
    __syncthreads();
    for (int e = threadIdx.x; e < ni; e += kBlock) {
      const int i = it + e;
      T *r = sh + kRec * e;
      r[0] = tgt[i];
      r[1] = tgt[N + i];
      r[2] = tgt[2 * (size_t)N + i];
      r[3] = (T)z[i];
      r[4] = (T)z[N + i];
      r[5] = (T)(eps_ratio * z[N + i]);
    }
    __syncthreads();
    T a[2][kAcc<T, NF>];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      for (int q = 0; q < kAcc<T, NF>; ++q) a[c][q] = T(0);
    for (int e = wave; e < ni; e += kWaves) {
      const T *r = sh + kRec * e;
      panel_columns<NF, FLOOR>(rec, r[0], r[1], r[2], r[3], r[4], r[5], sc, a);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
      for (int q = 0; q < kAcc<T, NF>; ++q) S[c] += (double)a[c][q];
  }
  if (wave > 0)
    for (int c = 0; c < 2; ++c) red[wave - 1][c][lane] = S[c];
  __syncthreads();
  if (wave == 0 && sj < N) {
    const double wA = geo[6 * (size_t)N + sj] * kInv4Pi / NF;
    for (int c = 0; c < 2; ++c) {
      double v = S[c];
      for (int w = 0; w < kWaves - 1; ++w) v += red[w][c][lane];
      part[((size_t)blockIdx.y * 2 + c) * N + sj] = wA * v;
    }
  }
}

// (A^T z) from the transposed far partials, the transposed near/self
// correction (entries of column j) and the identity terms; lanes per row as
// in k_finish.
__global__ __launch_bounds__(kBlock) void k_finish_transpose(
    int N, int nchunk, const double *__restrict__ part, const int *__restrict__ trow,
    const int *__restrict__ tcol, const int *__restrict__ tent, const double *__restrict__ val,
    const double *__restrict__ z, double eps_ratio, const int *__restrict__ perm,
    double *__restrict__ y) {
  const int t = blockIdx.x * kBlock + (int)threadIdx.x;
  const int j = t / kFinLanes, u = t % kFinLanes;
  const int jl = min(j, N - 1);
  double S[2] = {0.0, 0.0};
  for (int c = u; c < nchunk; c += kFinLanes)
    for (int k = 0; k < 2; ++k) S[k] += part[((size_t)c * 2 + k) * N + jl];
  const int e1 = trow[jl + 1];
  for (int e = trow[jl] + u; e < e1; e += kFinLanes) {
    const int i = tcol[e];
    const double *v = val + 4 * (size_t)tent[e];
    const double z1 = z[i], z2 = z[N + i];
    S[0] += v[1] * z1 - v[3] * z2;
    S[1] += eps_ratio * v[2] * z2 - v[0] * z1;
  }
  for (int w = 1; w < kFinLanes; w <<= 1)
    for (int k = 0; k < 2; ++k) S[k] += __shfl_xor(S[k], w, kFinLanes);
  if (j >= N || u != 0) return;
  const int o = perm ? perm[j] : j;
  y[o] = 0.5 * z[j] + 0.5 * z[N + j] + S[0];
  y[N + o] = S[1];
}

}  // namespace

void launch_gather_pack(hipStream_t s, int N, int nf, double eps_ratio, const int *perm,
                        const double *geo, const double *user, double *x, double *src64,
                        float *src32) {
  hipLaunchKernelGGL(k_gather_pack, dim3((N + 255) / 256), dim3(256), 0, s, N, nf, eps_ratio,
                     perm, geo, user, x, src64, src32);
  PBMP_HIP(hipGetLastError());
}

void launch_pack_strengths(hipStream_t s, int N, int nf, double eps_ratio,
                           const double *geo, const double *x, double *src64,
                           float *src32) {
  hipLaunchKernelGGL(k_pack_strengths, dim3((N + 255) / 256), dim3(256), 0, s,
                     N, nf, eps_ratio, geo, x, src64, src32);
  PBMP_HIP(hipGetLastError());
}

int direct_chunks(int N) {
  // about 8192 blocks of four waves (4096, 8192, 12288: 527, 507, 511 us on
  // 19220 panels, 97, 94, 97 us on 8000 with the finish kernel), each wave at
  // least eight panels
  const int bx = (N + 63) / 64;
  return std::max(1, std::min((8192 + bx - 1) / bx, (N + 31) / 32));
}

#define PBMP_P2P_RULE(T, CALL)                \
  do {                                        \
    if (nf == 3 && floor_r2) CALL(T, 3, true); \
    else if (nf == 3) CALL(T, 3, false);      \
    else if (floor_r2) CALL(T, 1, true);      \
    else CALL(T, 1, false);                   \
  } while (0)

void launch_p2p_direct(hipStream_t s, bool fp64, int nf, int N, int Nt,
                       const double *src64, const float *src32,
                       const double *geo, const float *tgt32, double kappa,
                       int nchunk, double *part, bool floor_r2) {
  const int chunk = (N + nchunk - 1) / nchunk;
  const dim3 grid((Nt + 63) / 64, nchunk);
#define PBMP_P2P(T, NFV, FL)                                                                  \
  hipLaunchKernelGGL((k_p2p<T, NFV, FL>), grid, dim3(kBlock), 0, s, src, N, tgt, Nt, chunk,    \
                     kap, part)
  if (fp64) {
    const double *src = src64, *tgt = geo, kap = kappa;
    PBMP_P2P_RULE(double, PBMP_P2P);
  } else {
    const float *src = src32, *tgt = tgt32, kap = kappa32(kappa);
    PBMP_P2P_RULE(float, PBMP_P2P);
  }
#undef PBMP_P2P
  PBMP_HIP(hipGetLastError());
}

void launch_finish(hipStream_t s, int N, int nchunk, const double *part,
                   const int *rowptr, const int *col, const double *val,
                   const double *x, double eps_ratio, const int *perm, double *y) {
  const int rows = kBlock / kFinLanes;
  hipLaunchKernelGGL(k_finish, dim3((N + rows - 1) / rows), dim3(kBlock), 0, s, N,
                     nchunk, part, rowptr, col, val, x, eps_ratio, perm, y);
  PBMP_HIP(hipGetLastError());
}

void launch_transpose(hipStream_t s, bool fp64, int nf, int N,
                      const double *src64, const float *src32,
                      const double *geo, const float *tgt32, const double *z,
                      double kappa, int nchunk, double *part,
                      const int *trow, const int *tcol, const int *tent,
                      const double *val, double eps_ratio, const int *perm, double *y,
                      bool floor_r2) {
  const int chunk = (N + nchunk - 1) / nchunk;
  const dim3 grid((N + 63) / 64, nchunk);
#define PBMP_P2PT(T, NFV, FL)                                                                 \
  hipLaunchKernelGGL((k_p2p_transpose<T, NFV, FL>), grid, dim3(kBlock), 0, s, N, src, tgt,    \
                     geo, z, chunk, kap, eps_ratio, part)
  if (fp64) {
    const double *src = src64, *tgt = geo, kap = kappa;
    PBMP_P2P_RULE(double, PBMP_P2PT);
  } else {
    const float *src = src32, *tgt = tgt32, kap = kappa32(kappa);
    PBMP_P2P_RULE(float, PBMP_P2PT);
  }
#undef PBMP_P2PT
#undef PBMP_P2P_RULE
  PBMP_HIP(hipGetLastError());
  const int rows = kBlock / kFinLanes;
  hipLaunchKernelGGL(k_finish_transpose, dim3((N + rows - 1) / rows), dim3(kBlock), 0, s,
                     N, nchunk, part, trow, tcol, tent, val, z, eps_ratio, perm, y);
  PBMP_HIP(hipGetLastError());
}

}  // namespace pbmp
