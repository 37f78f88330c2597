// Far-field source-target (P2P) sums of the boundary-integral operator
// (section "The treecode algorithm": the product is an N-body problem with
// the Gauss nodes as sources and the collocation points as targets), and the
// step that turns the four operator sums into y = A x (eq. integral_eq).
//
// Layout: TPT targets per lane, source panels staged through LDS in tiles;
// the lanes of a wave read the same panel record (LDS broadcast).  A panel
// record is 16 words: three far-field nodes, the unit normal, the plane
// offset n.y and the strengths s_V, s_K, eps s_V.  Because the
// nodes of a flat panel share its plane, n.(x - y_q) = n.x - n.y0 for all q.
//
// Per (target, node) pair the four kernels need one reciprocal square root
// and one exponential:  V_L += 1/r, V_Y += e^{-kr}/r, K_L += 1/r^3,
// K_Y += (1 + kr) e^{-kr}/r^3; the panel's sums are then weighted by s_V and
// s_K n.R.  FP32 variant: per-tile FP32 sums folded into FP64 accumulators.
#include <algorithm>
#include <cmath>

#include "kernels.hpp"
#include "pair.hpp"

namespace pbmp {

namespace {

constexpr double kInv4Pi = 0.07957747154594767;
constexpr int kBlock = 256;
constexpr int kTile = 128;  // panels per LDS tile

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

// Direct product.  A block takes 64 TPT targets (lane l: targets l, l + 64,
// ...) and one source chunk: its four waves stage the chunk's records tile by
// tile and each takes every fourth panel, so a launch holds four times the
// waves of a block of 256 targets for the same partial sums (the waves' sums
// are added through LDS in wave order); on the 1280-panel sphere the 256
// lanes of a block otherwise cover the surface in five blocks.
template <class T, int NF, int TPT, bool FLOOR>
__global__ __launch_bounds__(kBlock) void k_p2p(const T *__restrict__ src, int N,
                                                const T *__restrict__ tgt, int Nt, int chunk,
                                                T kappa, double *__restrict__ part) {
  constexpr int kWaves = kBlock / 64;
  constexpr int kTileR = sizeof(T) == 4 ? kTile : kTile / 2;  // records per tile (8 KB)
  typedef T v2 __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int PER = 16 * sizeof(T) / 16;  // 16-byte units per record
  __shared__ __align__(16) T sh[kTileR * 16];
  __shared__ double red[kWaves - 1][TPT][2][64];
  __shared__ double etab[sizeof(T) == 8 ? 64 : 1];
  const Screen<T> sc = make_screen(kappa, etab);
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int j0 = blockIdx.y * chunk;
  const int j1 = min(N, j0 + chunk);
  T px[TPT], py[TPT], pz[TPT];
  int ti[TPT];
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    ti[k] = blockIdx.x * (64 * TPT) + k * 64 + lane;
    const int tl = min(ti[k], Nt - 1);
    px[k] = tgt[tl];
    py[k] = tgt[Nt + tl];
    pz[k] = tgt[2 * Nt + tl];
  }
  double S[TPT][2];
#pragma unroll
  for (int k = 0; k < TPT; ++k) S[k][0] = S[k][1] = 0.0;
  for (int jt = j0; jt < j1; jt += kTileR) {
    const int nj = min(kTileR, j1 - jt);
    __syncthreads();
    const v2 *g = reinterpret_cast<const v2 *>(src + (size_t)jt * 16);
    for (int e = threadIdx.x; e < nj * PER; e += kBlock) reinterpret_cast<v2 *>(sh)[e] = g[e];
    __syncthreads();
    T a[TPT][2][kAcc<T, NF>];
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      for (int c = 0; c < 2; ++c)
        for (int q = 0; q < kAcc<T, NF>; ++q) a[k][c][q] = T(0);
    for (int jj = wave; jj < nj; jj += kWaves) {
      const T *r = sh + 16 * jj;
#pragma unroll
      for (int k = 0; k < TPT; ++k)
        panel_rows<NF, FLOOR>(r, px[k], py[k], pz[k], sc, a[k]);
    }
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      for (int c = 0; c < 2; ++c)
        for (int q = 0; q < kAcc<T, NF>; ++q) S[k][c] += (double)a[k][c][q];
  }
  if (wave > 0)
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      for (int c = 0; c < 2; ++c) red[wave - 1][k][c][lane] = S[k][c];
  __syncthreads();
  if (wave == 0)
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      for (int c = 0; c < 2; ++c) {
        double v = S[k][c];
        for (int w = 0; w < kWaves - 1; ++w) v += red[w][k][c][lane];
        if (ti[k] < Nt) part[((size_t)blockIdx.y * 2 + c) * Nt + ti[k]] = v;
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
    double eps_ratio, double *__restrict__ y) {
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
  y[i] = 0.5 * ph + S[0];
  y[N + i] = 0.5 * ph + S[1];
}

// Transposed far-field sums: targets are the far-field nodes of panel j
// (normal n_j), sources the collocation points c_i with weights z1_i, z2_i:
//   T_VL_j = sum_q w A_j/(4 pi) sum_i z1_i / r,   T_KL_j = ... z1_i n_j.(c_i - y)/r^3
//   T_VY_j = ... z2_i e^{-kr}/r,                   T_KY_j = ... z2_i n_j.(c_i-y)(1+kr)e^{-kr}/r^3
// Blocks as in k_p2p with the roles exchanged: 64 TPT panels on the lanes, the
// chunk's collocation points staged through LDS, every fourth one to a wave.
template <class T, int NF, int TPT, bool FLOOR>
__global__ __launch_bounds__(kBlock) void k_p2p_transpose(
    int N, const T *__restrict__ src, const T *__restrict__ tgt, const double *__restrict__ geo,
    const double *__restrict__ z, int chunk, T kappa, double eps_ratio,
    double *__restrict__ part) {
  constexpr int kWaves = kBlock / 64;
  constexpr int kRec = 8;  // x y z z1 z2 eps z2
  __shared__ __align__(16) T sh[kTile * kRec];
  __shared__ double red[kWaves - 1][TPT][2][64];
  __shared__ double etab[sizeof(T) == 8 ? 64 : 1];
  const Screen<T> sc = make_screen(kappa, etab);
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  T rec[TPT][12];
  int sj[TPT];
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    sj[k] = blockIdx.x * (64 * TPT) + k * 64 + lane;
    const int jl = min(sj[k], N - 1);
#pragma unroll
    for (int c = 0; c < 12; ++c) rec[k][c] = src[16 * (size_t)jl + c];
  }
  const int i0 = blockIdx.y * chunk, i1 = min(N, i0 + chunk);
  double S[TPT][2];
#pragma unroll
  for (int k = 0; k < TPT; ++k) S[k][0] = S[k][1] = 0.0;
  for (int it = i0; it < i1; it += kTile) {
    const int ni = min(kTile, i1 - it);
    __syncthreads();
    for (int e = threadIdx.x; e < ni; e += kBlock) {
      const int i = it + e;
      T *r = sh + kRec * e;
      r[0] = tgt[i];
      r[1] = tgt[N + i];
      r[2] = tgt[2 * N + i];
      r[3] = (T)z[i];
      r[4] = (T)z[N + i];
      r[5] = (T)(eps_ratio * z[N + i]);
    }
    __syncthreads();
    T a[TPT][2][kAcc<T, NF>];
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      for (int c = 0; c < 2; ++c)
        for (int q = 0; q < kAcc<T, NF>; ++q) a[k][c][q] = T(0);
    for (int e = wave; e < ni; e += kWaves) {
      const T *r = sh + kRec * e;
#pragma unroll
      for (int k = 0; k < TPT; ++k)
        panel_columns<NF, FLOOR>(rec[k], r[0], r[1], r[2], r[3], r[4], r[5], sc, a[k]);
    }
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      for (int c = 0; c < 2; ++c)
        for (int q = 0; q < kAcc<T, NF>; ++q) S[k][c] += (double)a[k][c][q];
  }
  if (wave > 0)
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      for (int c = 0; c < 2; ++c) red[wave - 1][k][c][lane] = S[k][c];
  __syncthreads();
  if (wave == 0)
#pragma unroll
    for (int k = 0; k < TPT; ++k)
      if (sj[k] < N) {
        const double wA = geo[6 * N + sj[k]] * kInv4Pi / NF;
        for (int c = 0; c < 2; ++c) {
          double v = S[k][c];
          for (int w = 0; w < kWaves - 1; ++w) v += red[w][k][c][lane];
          part[((size_t)blockIdx.y * 2 + c) * N + sj[k]] = wA * v;
        }
      }
}

// (A^T z) from the transposed far partials, the transposed near/self
// correction (entries of column j) and the identity terms; lanes per row as
// in k_finish.
__global__ __launch_bounds__(kBlock) void k_finish_transpose(
    int N, int nchunk, const double *__restrict__ part, const int *__restrict__ trow,
    const int *__restrict__ tcol, const int *__restrict__ tent, const double *__restrict__ val,
    const double *__restrict__ z, double eps_ratio, double *__restrict__ y) {
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
  y[j] = 0.5 * z[j] + 0.5 * z[N + j] + S[0];
  y[N + j] = S[1];
}

}  // namespace

void launch_pack_strengths(hipStream_t s, int N, int nf, double eps_ratio,
                           const double *geo, const double *x, double *src64,
                           float *src32) {
  hipLaunchKernelGGL(k_pack_strengths, dim3((N + 255) / 256), dim3(256), 0, s,
                     N, nf, eps_ratio, geo, x, src64, src32);
  PBMP_HIP(hipGetLastError());
}

namespace {
// Targets per lane of the direct product: two share every record read where
// there are targets enough to fill the device, one below.
inline int direct_tpt(bool fp64, int Nt) { return !fp64 && Nt > 6144 ? 2 : 1; }
}  // namespace

int direct_chunks(bool fp64, int N) {
  // about 4096 blocks (four waves each), each wave at least eight panels
  const int bx = (N + 64 * direct_tpt(fp64, N) - 1) / (64 * direct_tpt(fp64, N));
  return std::max(1, std::min((4096 + bx - 1) / bx, (N + 31) / 32));
}

void launch_p2p_direct(hipStream_t s, bool fp64, int nf, int N, int Nt,
                       const double *src64, const float *src32,
                       const double *geo, const float *tgt32, double kappa,
                       int nchunk, double *part, bool floor_r2) {
  const int chunk = (N + nchunk - 1) / nchunk;
  const int tpt = direct_tpt(fp64, Nt);
  const dim3 grid((Nt + 64 * tpt - 1) / (64 * tpt), nchunk);
#define PBMP_P2P(TT, NFV, TPT, FL, SRC, TGT)                                             \
  hipLaunchKernelGGL((k_p2p<TT, NFV, TPT, FL>), grid, dim3(kBlock), 0, s, SRC, N, TGT, Nt, \
                     chunk, (TT)kappa, part)
#define PBMP_P2P_RULE(CALL)                \
  if (nf == 3 && floor_r2) CALL(3, true);  \
  else if (nf == 3) CALL(3, false);        \
  else if (floor_r2) CALL(1, true);        \
  else CALL(1, false)
#define PBMP_P2P64(NFV, FL) PBMP_P2P(double, NFV, 1, FL, src64, geo)
#define PBMP_P2P32(NFV, FL)                                  \
  if (tpt == 2) PBMP_P2P(float, NFV, 2, FL, src32, tgt32);   \
  else PBMP_P2P(float, NFV, 1, FL, src32, tgt32)
  if (fp64) {
    PBMP_P2P_RULE(PBMP_P2P64);
  } else {
    PBMP_P2P_RULE(PBMP_P2P32);
  }
#undef PBMP_P2P64
#undef PBMP_P2P32
#undef PBMP_P2P
  PBMP_HIP(hipGetLastError());
}

void launch_finish(hipStream_t s, int N, int nchunk, const double *part,
                   const int *rowptr, const int *col, const double *val,
                   const double *x, double eps_ratio, double *y) {
  const int rows = kBlock / kFinLanes;
  hipLaunchKernelGGL(k_finish, dim3((N + rows - 1) / rows), dim3(kBlock), 0, s, N,
                     nchunk, part, rowptr, col, val, x, eps_ratio, y);
  PBMP_HIP(hipGetLastError());
}

void launch_transpose(hipStream_t s, bool fp64, int nf, int N,
                      const double *src64, const float *src32,
                      const double *geo, const float *tgt32, const double *z,
                      double kappa, int nchunk, double *part,
                      const int *trow, const int *tcol, const int *tent,
                      const double *val, double eps_ratio, double *y, bool floor_r2) {
  const int chunk = (N + nchunk - 1) / nchunk;
  const int tpt = direct_tpt(fp64, N);
  const dim3 grid((N + 64 * tpt - 1) / (64 * tpt), nchunk);
#define PBMP_P2PT(TT, NFV, TPT, FL, SRC, TGT)                                              \
  hipLaunchKernelGGL((k_p2p_transpose<TT, NFV, TPT, FL>), grid, dim3(kBlock), 0, s, N, SRC, \
                     TGT, geo, z, chunk, (TT)kappa, eps_ratio, part)
#define PBMP_P2PT64(NFV, FL) PBMP_P2PT(double, NFV, 1, FL, src64, geo)
#define PBMP_P2PT32(NFV, FL)                                  \
  if (tpt == 2) PBMP_P2PT(float, NFV, 2, FL, src32, tgt32);   \
  else PBMP_P2PT(float, NFV, 1, FL, src32, tgt32)
  if (fp64) {
    PBMP_P2P_RULE(PBMP_P2PT64);
  } else {
    PBMP_P2P_RULE(PBMP_P2PT32);
  }
#undef PBMP_P2PT64
#undef PBMP_P2PT32
#undef PBMP_P2PT
#undef PBMP_P2P_RULE
  PBMP_HIP(hipGetLastError());
  const int rows = kBlock / kFinLanes;
  hipLaunchKernelGGL(k_finish_transpose, dim3((N + rows - 1) / rows), dim3(kBlock), 0, s,
                     N, nchunk, part, trow, tcol, tent, val, z, eps_ratio, y);
  PBMP_HIP(hipGetLastError());
}

}  // namespace pbmp
