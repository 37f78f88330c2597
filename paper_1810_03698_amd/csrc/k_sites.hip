// Kernels at the point-multipole sites: right-hand side (eq. rhs_multipole),
// reaction-potential readout (eq. pot_solvent, Efield_solv, ddphi),
// multipole Coulomb fields (eq. Efield_mult, appendix derivatives) with the
// group masking and Thole damping of the section "Calculation of the
// electric field", the relaxed induced-dipole update and the energy sum of
// eq. energy_multipole_polarizable.
#include <cmath>

#include "kernels.hpp"
#include "pair.hpp"

namespace pbmp {

namespace {

constexpr double kInv4Pi = 0.07957747154594767;
constexpr double kFourPi = 12.566370614359172;

// ------------------------------------------------------------------ RHS
// Blocks of 64 TPT panels: lane l holds panels l, l + 64, ...; the block's
// four waves take every fourth site of the staged tiles, and their sums are
// added through LDS in wave order (a panel per thread left a 30k-panel surface
// with fewer waves than SIMDs).  The multipoles are staged in T, once per
// block instead of once per pair; the differences are formed in FP64 and the
// sums kept there.  Bound by VALU issue, the FP64 differences and sums about
// 40 % of it: 1376 -> 595 us on 144500 panels and 5000 sites, 202 -> 37 us on
// 28880 and 1000 (mixed precision).
constexpr int kSiteTile = 128;
constexpr int kRhsVal = 12;  // q px py pz Qxx Qxy Qxz Qyy Qyz Qzz per site

template <class T, int TPT>
__global__ __launch_bounds__(256) void k_rhs(int N, int M, const double *__restrict__ geo,
                                             const double *__restrict__ xyz,
                                             const double *__restrict__ q,
                                             const double *__restrict__ p,
                                             const double *__restrict__ Q9, double scale,
                                             double *__restrict__ f) {
  __shared__ __align__(16) double spos[kSiteTile * 4];
  __shared__ __align__(16) T sval[kSiteTile * kRhsVal];
  __shared__ double red[3][TPT][64];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  double c[TPT][3], acc[TPT];
  int ti[TPT];
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    ti[k] = blockIdx.x * (64 * TPT) + 64 * k + lane;
    const int il = min(ti[k], N - 1);
    for (int d = 0; d < 3; ++d) c[k][d] = geo[(size_t)d * N + il];
    acc[k] = 0.0;
  }
  for (int k0 = 0; k0 < M; k0 += kSiteTile) {
    const int nk = min(kSiteTile, M - k0);
    __syncthreads();
    for (int e = threadIdx.x; e < nk; e += 256) {
      const int m = k0 + e;
      for (int d = 0; d < 3; ++d) spos[4 * e + d] = xyz[3 * m + d];
      T *r = sval + kRhsVal * e;
      r[0] = (T)q[m];
      for (int d = 0; d < 3; ++d) r[1 + d] = (T)p[3 * m + d];
      const double *Q = Q9 + 9 * (size_t)m;
      r[4] = (T)Q[0];
      r[5] = (T)Q[1];
      r[6] = (T)Q[2];
      r[7] = (T)Q[4];
      r[8] = (T)Q[5];
      r[9] = (T)Q[8];
    }
    __syncthreads();
    for (int e = wave; e < nk; e += 4) {
      const double *s = spos + 4 * e;
      const T *r = sval + kRhsVal * e;
#pragma unroll
      for (int k = 0; k < TPT; ++k) {
        const T X = (T)(c[k][0] - s[0]), Y = (T)(c[k][1] - s[1]), Z = (T)(c[k][2] - s[2]);
        T rr, ri;
        if constexpr (sizeof(T) == 4) {
          rr = fmaf(X, X, fmaf(Y, Y, Z * Z));
          ri = __builtin_amdgcn_rsqf(rr);
        } else {
          rr = X * X + Y * Y + Z * Z;
          ri = rsqrt_fp64(rr);
        }
        const T ri2 = ri * ri;
        const T pR = r[1] * X + r[2] * Y + r[3] * Z;
        const T QRR = r[4] * X * X + r[7] * Y * Y + r[9] * Z * Z +
                      T(2) * (r[5] * X * Y + r[6] * X * Z + r[8] * Y * Z);
        acc[k] += (double)(ri * (r[0] + ri2 * (pR + T(0.5) * QRR * ri2)));
      }
    }
  }
  if (wave > 0)
    for (int k = 0; k < TPT; ++k) red[wave - 1][k][lane] = acc[k];
  __syncthreads();
  if (wave == 0)
    for (int k = 0; k < TPT; ++k)
      if (ti[k] < N)
        f[ti[k]] = (acc[k] + red[0][k][lane] + red[1][k][lane] + red[2][k][lane]) * scale;
}

// ------------------------------------------------------------- readout
// Kernel values of one source node at a target, for the single layer
// (G = 1/r) and double layer (H = n.R/r^3) with their first and second
// derivatives in the target point: out[0..9] = G data, out[10..19] = H data
// (order: value, d/dx, d/dy, d/dz, xx, xy, xz, yy, yz, zz).
template <class T, bool FULL>
__device__ inline void node_kernels(T X, T Y, T Z, T nx, T ny, T nz, T nR,
                                    T *g, T *h) {
  const T rr = X * X + Y * Y + Z * Z;
  T i1;
  if constexpr (sizeof(T) == 4)
    i1 = __builtin_amdgcn_rsqf(rr);
  else
    i1 = T(1) / sqrt(rr);
  const T i2 = i1 * i1;
  const T i3 = i1 * i2;
  const T i5 = i3 * i2;
  const T R[3] = {X, Y, Z};
  const T n[3] = {nx, ny, nz};
  g[0] += i1;
  h[0] += nR * i3;
  for (int a = 0; a < 3; ++a) {
    g[1 + a] -= R[a] * i3;
    h[1 + a] += n[a] * i3 - T(3) * nR * R[a] * i5;
  }
  if constexpr (FULL) {
    const T i7 = i5 * i2;
    int o = 4;
    for (int a = 0; a < 3; ++a)
      for (int b = a; b < 3; ++b) {
        const T del = (a == b) ? T(1) : T(0);
        g[o] += T(3) * R[a] * R[b] * i5 - del * i3;
        h[o] += T(-3) * (n[a] * R[b] + n[b] * R[a] + nR * del) * i5 +
                T(15) * nR * R[a] * R[b] * i7;
        ++o;
      }
  }
}

// Far-field readout.  A block takes 64 sites (or the next power of two of
// fewer) and one source chunk, its panels staged through LDS in tiles of
// kRoTile records (16-byte loads, all issued before the first store); its four
// waves take every fourth panel, and with L < 64 site lanes the 64 / L groups
// of a wave share those.  Per-chunk partial sums part[chunk][site][k].  (Blocks
// of one wave with the same tiles were bound to 3.5 waves per SIMD by their
// LDS: 3.65 ms against 3.15 ms on 144500 panels and 5000 sites.)
//
// Node differences and n.R are formed in FP64, the kernels in T, and each
// panel's sums are added in FP64.  With s_V, s_K the strengths and R the
// difference, one node adds to the potential and its derivatives
//   value  s_V/r - s_K n.R/r^3,   gradient  a R + b n,
//   second derivatives  c R R^T + d (n R^T + R n^T) + a I,
//   a = 3 s_K n.R/r^5 - s_V/r^3,  b = -s_K/r^3,
//   c = 3 s_V/r^5 - 15 s_K n.R/r^7,  d = 3 s_K/r^5,
// so the nodes' sums of a R, a, b, c R R^T and d R suffice and the normal enters
// once per panel: 33 FP32 operations per node where single and double layer
// accumulated apart took about 90.  VALU issue bound; the FP64 differences,
// conversions and per-panel additions are half of it.  All ten values on
// 144500 panels and 5000 sites 7.90 -> 3.15 ms, the field alone on 28880 and
// 1000 127 -> 67 us, on 1280 and 8 in FP64 39 -> 4.5 us.
constexpr int kRoTile = 64;
constexpr int kRoRec = 18;  // padded FP64 record: lane groups read different ones

template <class T, bool FULL, int NF>
__global__ __launch_bounds__(256) void k_readout_far(
    int N, int M, const double *__restrict__ src64, const double *__restrict__ xyz,
    int chunk, int L, double *__restrict__ part) {
  constexpr int NO = FULL ? 10 : 4;
  typedef double d2 __attribute__((ext_vector_type(2)));
  __shared__ __align__(16) double s64[kRoTile * kRoRec];
  __shared__ __align__(16) T sval[kRoTile * 8];  // n, s_V, s_K in T
  __shared__ double red[3][64];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int G = 64 / L, gi = lane / L, li = lane - gi * L;
  const int j0 = blockIdx.y * chunk, j1 = min(N, j0 + chunk);
  const int l = blockIdx.x * L + li, lc = min(l, M - 1);
  const double P[3] = {xyz[3 * lc], xyz[3 * lc + 1], xyz[3 * lc + 2]};
  double acc[NO];
  for (int c = 0; c < NO; ++c) acc[c] = 0.0;
  for (int jt = j0; jt < j1; jt += kRoTile) {
    const int nj = min(kRoTile, j1 - jt);
    __syncthreads();
    {
      const d2 *g = reinterpret_cast<const d2 *>(src64 + 16 * (size_t)jt);
      const int n = nj * 8;
      d2 v[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int e = (int)threadIdx.x + 256 * u;
        if (e < n) v[u] = g[e];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int e = (int)threadIdx.x + 256 * u;
        if (e < n) *reinterpret_cast<d2 *>(s64 + kRoRec * (e >> 3) + 2 * (e & 7)) = v[u];
      }
    }
    __syncthreads();
    if ((int)threadIdx.x < nj) {
      const double *r = s64 + kRoRec * threadIdx.x;
      T *t = sval + 8 * threadIdx.x;
      for (int d = 0; d < 3; ++d) t[d] = (T)r[9 + d];
      t[3] = (T)r[13];
      t[4] = (T)r[14];
    }
    __syncthreads();
    for (int jj = wave + 4 * gi; jj < nj; jj += 4 * G) {
      const double *r = s64 + kRoRec * jj;
      const T n[3] = {sval[8 * jj], sval[8 * jj + 1], sval[8 * jj + 2]};
      const T sv = sval[8 * jj + 3], sk = sval[8 * jj + 4];
      const T nR = (T)(r[9] * P[0] + r[10] * P[1] + r[11] * P[2] - r[12]);
      const T skn = sk * nR;
      T val = T(0), sa = T(0), sb = T(0), aR[3] = {T(0), T(0), T(0)};
      T dR[3] = {T(0), T(0), T(0)}, rr6[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        const T R[3] = {(T)(P[0] - r[3 * q]), (T)(P[1] - r[3 * q + 1]), (T)(P[2] - r[3 * q + 2])};
        const T rr = R[0] * R[0] + R[1] * R[1] + R[2] * R[2];
        T i1;
        if constexpr (sizeof(T) == 4) i1 = __builtin_amdgcn_rsqf(rr);
        else i1 = rsqrt_fp64(rr);
        const T i2 = i1 * i1, i3 = i1 * i2, i5 = i3 * i2;
        const T a = T(3) * skn * i5 - sv * i3;
        val += sv * i1 - skn * i3;
        sb -= sk * i3;
        for (int d = 0; d < 3; ++d) aR[d] += a * R[d];
        if constexpr (FULL) {
          const T i7 = i5 * i2;
          const T c = T(3) * sv * i5 - T(15) * skn * i7;
          const T d = T(3) * sk * i5;
          sa += a;
          for (int e = 0; e < 3; ++e) dR[e] += d * R[e];
          const T cx = c * R[0], cy = c * R[1], cz = c * R[2];
          rr6[0] += cx * R[0];
          rr6[1] += cx * R[1];
          rr6[2] += cx * R[2];
          rr6[3] += cy * R[1];
          rr6[4] += cy * R[2];
          rr6[5] += cz * R[2];
        }
      }
      acc[0] += (double)val;
      for (int d = 0; d < 3; ++d) acc[1 + d] += (double)(aR[d] + sb * n[d]);
      if constexpr (FULL) {
        acc[4] += (double)(rr6[0] + (T(2) * n[0] * dR[0] + sa));
        acc[5] += (double)(rr6[1] + (n[0] * dR[1] + n[1] * dR[0]));
        acc[6] += (double)(rr6[2] + (n[0] * dR[2] + n[2] * dR[0]));
        acc[7] += (double)(rr6[3] + (T(2) * n[1] * dR[1] + sa));
        acc[8] += (double)(rr6[4] + (n[1] * dR[2] + n[2] * dR[1]));
        acc[9] += (double)(rr6[5] + (T(2) * n[2] * dR[2] + sa));
      }
    }
  }
  // groups, then waves, in a fixed order (L is a power of two)
  for (int c = 0; c < NO; ++c) {
    for (int o = L; o < 64; o <<= 1) acc[c] += __shfl_xor(acc[c], o, 64);
    __syncthreads();
    if (wave > 0) red[wave - 1][lane] = acc[c];
    __syncthreads();
    if (wave == 0 && gi == 0 && l < M)
      part[((size_t)blockIdx.y * M + l) * NO + c] =
          acc[c] + red[0][lane] + red[1][lane] + red[2][lane];
  }
}

// Near-singular correction at the sites (19-node rule instead of the far
// rule for panels with |r_l - c_j| < eta sqrt(A_j)), chunk sum, and the
// 4 pi factor to physical units.  One 64-lane block per site.
template <bool FULL>
__global__ __launch_bounds__(64) void k_readout_near(
    int N, int M, int nchunk, const double *__restrict__ part,
    const double *__restrict__ verts, const int *__restrict__ tri,
    const double *__restrict__ geo, RuleArgs ru, const double *__restrict__ x,
    const double *__restrict__ xyz, const int *__restrict__ srow,
    const int *__restrict__ scol, double *__restrict__ out) {
  constexpr int NO = FULL ? 10 : 4;
  __shared__ double red[64];
  const int l = blockIdx.x;
  const double P[3] = {xyz[3 * l], xyz[3 * l + 1], xyz[3 * l + 2]};
  double acc[NO];
  for (int k = 0; k < NO; ++k) acc[k] = 0.0;
  for (int e = srow[l] + threadIdx.x; e < srow[l + 1]; e += blockDim.x) {
    const int j = scol[e];
    double v[3][3];
    for (int a = 0; a < 3; ++a)
      for (int d = 0; d < 3; ++d) v[a][d] = verts[3 * tri[3 * j + a] + d];
    const double n[3] = {geo[3 * N + j], geo[4 * N + j], geo[5 * N + j]};
    const double A = geo[6 * N + j];
    const double ph = x[j], dp = x[N + j];
    for (int pass = 0; pass < 2; ++pass) {
      const int nq = pass ? ru.nf : ru.nn;
      const double sign = pass ? -1.0 : 1.0;
      for (int qn = 0; qn < nq; ++qn) {
        const double *b = pass ? ru.fb[qn] : ru.nb[qn];
        const double w = pass ? ru.fw[qn] : ru.nw[qn];
        double y[3];
        for (int d = 0; d < 3; ++d) y[d] = b[0] * v[0][d] + b[1] * v[1][d] + b[2] * v[2][d];
        const double X = P[0] - y[0], Y = P[1] - y[1], Z = P[2] - y[2];
        const double nR = n[0] * X + n[1] * Y + n[2] * Z;
        double g[NO], h[NO];
        for (int k = 0; k < NO; ++k) g[k] = h[k] = 0.0;
        node_kernels<double, FULL>(X, Y, Z, n[0], n[1], n[2], nR, g, h);
        const double sa = sign * w * A * dp * kInv4Pi;
        const double sb = sign * w * A * ph * kInv4Pi;
        for (int k = 0; k < NO; ++k) acc[k] += sa * g[k] - sb * h[k];
      }
    }
  }
  // the far chunks' partial sums join the lanes' near sums (chunk c on lane
  // c mod 64), then a fixed-order tree over the lanes
  for (int k = 0; k < NO; ++k) {
    double v = acc[k];
    for (int c = threadIdx.x; c < nchunk; c += blockDim.x) v += part[((size_t)c * M + l) * NO + k];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 32; w > 0; w >>= 1) {
      if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[(size_t)l * NO + k] = kFourPi * red[0];
    __syncthreads();
  }
}

// ------------------------------------------------------------- Coulomb
// Sum over the 64 lanes of a wave (every lane receives the total).
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The site-pair kernels below take one wave per site l, lanes over the
// sources m (strided), and reduce over the wave at the end.
__global__ __launch_bounds__(64) void k_perm_field(int M, const double *__restrict__ xyz,
                                                   const double *__restrict__ q,
                                                   const double *__restrict__ d,
                                                   const double *__restrict__ Q9,
                                                   const int *__restrict__ group,
                                                   double inv_eps, double *__restrict__ E) {
  const int l = blockIdx.x;
  const int lane = (int)threadIdx.x;
  const double P[3] = {xyz[3 * l], xyz[3 * l + 1], xyz[3 * l + 2]};
  const int gl = group[l];
  double g[3] = {0.0, 0.0, 0.0};
  for (int m = lane; m < M; m += 64) {
    if (group[m] == gl) continue;  // includes m == l
    const double R[3] = {P[0] - xyz[3 * m], P[1] - xyz[3 * m + 1],
                         P[2] - xyz[3 * m + 2]};
    const double rr = R[0] * R[0] + R[1] * R[1] + R[2] * R[2];
    const double ri = 1.0 / sqrt(rr);
    const double ri2 = ri * ri, ri3 = ri * ri2, ri5 = ri3 * ri2, ri7 = ri5 * ri2;
    const double *pm = d + 3 * m;
    const double *Qm = Q9 + 9 * m;
    double QR[3];
    for (int a = 0; a < 3; ++a)
      QR[a] = Qm[3 * a] * R[0] + Qm[3 * a + 1] * R[1] + Qm[3 * a + 2] * R[2];
    const double S = QR[0] * R[0] + QR[1] * R[1] + QR[2] * R[2];
    const double pR = pm[0] * R[0] + pm[1] * R[1] + pm[2] * R[2];
    for (int a = 0; a < 3; ++a)
      g[a] += -q[m] * R[a] * ri3 + pm[a] * ri3 - 3.0 * pR * R[a] * ri5 +
              QR[a] * ri5 - 2.5 * S * R[a] * ri7;
  }
  for (int a = 0; a < 3; ++a) g[a] = wave_sum(g[a]);
  if (lane == 0)
    for (int a = 0; a < 3; ++a) E[3 * l + a] = -g[a] * inv_eps;
}

template <bool FULL>
__global__ __launch_bounds__(64) void k_induced(int M, const double *__restrict__ xyz,
                                                const double *__restrict__ mu,
                                                const double *__restrict__ alpha, double ta,
                                                double inv_eps, double *__restrict__ out) {
  const int l = blockIdx.x;
  const int lane = (int)threadIdx.x;
  const double P[3] = {xyz[3 * l], xyz[3 * l + 1], xyz[3 * l + 2]};
  const double al = alpha[l];
  double acc[10];
  for (int k = 0; k < 10; ++k) acc[k] = 0.0;
  for (int m = lane; m < M; m += 64) {
    if (m == l) continue;
    const double R[3] = {P[0] - xyz[3 * m], P[1] - xyz[3 * m + 1],
                         P[2] - xyz[3 * m + 2]};
    const double rr = R[0] * R[0] + R[1] * R[1] + R[2] * R[2];
    const double rad = sqrt(rr);
    const double ri = 1.0 / rad;
    const double ri2 = ri * ri, ri3 = ri * ri2, ri5 = ri3 * ri2, ri7 = ri5 * ri2;
    double l3 = 1.0, l5 = 1.0, l7 = 1.0;
    const double ap = al * alpha[m];
    if (ap > 0.0) {
      const double sd = ta * rr * rad / sqrt(ap);
      const double es = exp(-sd);
      l3 = 1.0 - es;
      l5 = 1.0 - (1.0 + sd) * es;
      l7 = 1.0 - (1.0 + sd + 0.6 * sd * sd) * es;
    }
    const double *u = mu + 3 * m;
    const double uR = u[0] * R[0] + u[1] * R[1] + u[2] * R[2];
    acc[0] += l3 * uR * ri3;
    for (int a = 0; a < 3; ++a) acc[1 + a] += l3 * u[a] * ri3 - 3.0 * l5 * uR * R[a] * ri5;
    if (FULL) {
      int o = 4;
      for (int a = 0; a < 3; ++a)
        for (int b = a; b < 3; ++b) {
          const double del = (a == b) ? 1.0 : 0.0;
          acc[o++] += -3.0 * l5 * (u[a] * R[b] + u[b] * R[a] + uR * del) * ri5 +
                      15.0 * l7 * uR * R[a] * R[b] * ri7;
        }
    }
  }
  if (FULL) {
    for (int k = 0; k < 10; ++k) acc[k] = wave_sum(acc[k]);
    if (lane == 0)
      for (int k = 0; k < 10; ++k) out[10 * l + k] = acc[k] * inv_eps;
  } else {
    for (int a = 0; a < 3; ++a) acc[1 + a] = wave_sum(acc[1 + a]);
    if (lane == 0)
      for (int a = 0; a < 3; ++a) out[3 * l + a] = -acc[1 + a] * inv_eps;
  }
}

__global__ void k_scf_update(int M, const double *__restrict__ alpha,
                             const double *__restrict__ Eperm,
                             const double *__restrict__ Eind,
                             const double *__restrict__ solv, int stride,
                             double omega, double *__restrict__ mu,
                             double *__restrict__ dmu2) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int l = threadIdx.x; l < M; l += blockDim.x) {
    for (int a = 0; a < 3; ++a) {
      double E = Eperm[3 * l + a] + Eind[3 * l + a];
      if (solv) E -= solv[(size_t)stride * l + 1 + a];
      const double old = mu[3 * l + a];
      const double nw = (1.0 - omega) * old + omega * alpha[l] * E;
      mu[3 * l + a] = nw;
      acc += (nw - old) * (nw - old);
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *dmu2 = red[0];
}

__device__ inline double apply_D(const double *q, const double *d,
                                 const double *Q, int l, const double *v) {
  // q phi + d.grad phi + (1/6) sum_ab Q_ab H_ab, H from its upper triangle
  const double H[3][3] = {{v[4], v[5], v[6]}, {v[5], v[7], v[8]}, {v[6], v[8], v[9]}};
  double qh = 0.0;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) qh += Q[9 * l + 3 * a + b] * H[a][b];
  return q[l] * v[0] + d[3 * l] * v[1] + d[3 * l + 1] * v[2] + d[3 * l + 2] * v[3] +
         qh / 6.0;
}

__global__ void k_energy(int M, const double *__restrict__ q,
                         const double *__restrict__ d,
                         const double *__restrict__ Q9,
                         const double *__restrict__ reac,
                         const double *__restrict__ ind, double *__restrict__ e) {
  __shared__ double r1[256], r2[256];
  double a1 = 0.0, a2 = 0.0;
  for (int l = threadIdx.x; l < M; l += blockDim.x) {
    a1 += apply_D(q, d, Q9, l, reac + 10 * (size_t)l);
    a2 += apply_D(q, d, Q9, l, ind + 10 * (size_t)l);
  }
  r1[threadIdx.x] = a1;
  r2[threadIdx.x] = a2;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      r1[threadIdx.x] += r1[threadIdx.x + w];
      r2[threadIdx.x] += r2[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    e[0] = 0.5 * r1[0];
    e[1] = 0.5 * r2[0];
  }
}

// Total dipole of the molecule for the vacuum and dissolved dipoles:
// sum_l q_l (r_l - o) + d_l + mu_l with o the mean site position, e*A.
__global__ void k_total_dipole(int M, const double *__restrict__ xyz,
                               const double *__restrict__ q,
                               const double *__restrict__ d,
                               const double *__restrict__ mu_v,
                               const double *__restrict__ mu_d,
                               double *__restrict__ out) {
  constexpr int K = 13;  // sum q, sum q r, sum r, sum (d + mu_v), sum mu_d - mu_v
  __shared__ double red[K][256];
  double a[K];
  for (int k = 0; k < K; ++k) a[k] = 0.0;
  for (int l = threadIdx.x; l < M; l += blockDim.x) {
    const double ql = q[l];
    a[0] += ql;
    for (int c = 0; c < 3; ++c) {
      const double r = xyz[3 * l + c];
      a[1 + c] += ql * r;
      a[4 + c] += r;
      a[7 + c] += d[3 * l + c] + mu_v[3 * l + c];
      a[10 + c] += mu_d[3 * l + c] - mu_v[3 * l + c];
    }
  }
  for (int k = 0; k < K; ++k) red[k][threadIdx.x] = a[k];
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < K; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 3) {
    const int c = threadIdx.x;
    const double pv = red[1 + c][0] - red[0][0] * red[4 + c][0] / M + red[7 + c][0];
    out[c] = pv;
    out[3 + c] = pv + red[10 + c][0];
  }
}

}  // namespace

void launch_total_dipole(hipStream_t s, int M, const double *xyz, const double *q,
                         const double *d, const double *mu_v, const double *mu_d,
                         double *out) {
  hipLaunchKernelGGL(k_total_dipole, dim3(1), dim3(256), 0, s, M, xyz, q, d, mu_v,
                     mu_d, out);
  PBMP_HIP(hipGetLastError());
}

void launch_rhs(hipStream_t s, bool fp64, int N, int M, const double *geo,
                const double *xyz, const double *q, const double *p,
                const double *Q9, double eps_in, double *f) {
  const double scale = kInv4Pi / eps_in;
  // Two panels per lane share the reads of a site but halve the blocks: worth it
  // from some four blocks per CU of FP64 pairs, which issue for longer, and only
  // beyond sixteen in FP32 (one against two panels per lane, sites at the density
  // of an inside; FP64: 40500 panels 154 and 172 us, 50000 255 and 241, 60500 350
  // and 322, 144500 2.61 and 2.61 ms, 288000 15.7 and 14.2; FP32: 60500 236 and 246
  // us, 144500 1.62 and 1.79 ms, 233280 5.78 and 6.00, 255380 7.11 and 6.77).
  const int tpt = N > (fp64 ? 45000 : 245000) ? 2 : 1;
  const dim3 grid((N + 64 * tpt - 1) / (64 * tpt));
#define PBMP_RHS(T, TPT)                                                                      \
  hipLaunchKernelGGL((k_rhs<T, TPT>), grid, dim3(256), 0, s, N, M, geo, xyz, q, p, Q9, scale, f)
  if (fp64 && tpt == 2) PBMP_RHS(double, 2);
  else if (fp64) PBMP_RHS(double, 1);
  else if (tpt == 2) PBMP_RHS(float, 2);
  else PBMP_RHS(float, 1);
#undef PBMP_RHS
  PBMP_HIP(hipGetLastError());
}

int readout_chunks(int N, int M) {
  // about 2048 blocks of four waves, each chunk at least one tile of panels
  const int tiles = (std::max(M, 1) + 63) / 64;
  const int c = (2048 + tiles - 1) / tiles;
  return std::max(1, std::min(c, N / kRoTile));
}

void launch_readout(hipStream_t s, bool fp64, bool full, int N, int M,
                    const double *src64, const double *geo,
                    const double *verts, const int *tri, const RuleArgs &ru,
                    const double *x, const double *xyz, const int *srow,
                    const int *scol, int nchunk, double *part, double *out) {
  if (M <= 0) return;
  const int chunk = (N + nchunk - 1) / nchunk;
  int L = 64;
  while (L / 2 >= M) L /= 2;
  const dim3 grid((M + L - 1) / L, nchunk);
#define PBMP_RO(T, FULL)                                                                       \
  do {                                                                                         \
    if (ru.nf == 3)                                                                            \
      hipLaunchKernelGGL((k_readout_far<T, FULL, 3>), grid, dim3(256), 0, s, N, M, src64, xyz, \
                         chunk, L, part);                                                      \
    else                                                                                       \
      hipLaunchKernelGGL((k_readout_far<T, FULL, 1>), grid, dim3(256), 0, s, N, M, src64, xyz, \
                         chunk, L, part);                                                      \
  } while (0)
  if (fp64 && full) PBMP_RO(double, true);
  else if (fp64) PBMP_RO(double, false);
  else if (full) PBMP_RO(float, true);
  else PBMP_RO(float, false);
#undef PBMP_RO
  PBMP_HIP(hipGetLastError());
  if (full)
    hipLaunchKernelGGL(k_readout_near<true>, dim3(M), dim3(64), 0, s, N, M,
                       nchunk, part, verts, tri, geo, ru, x, xyz, srow, scol, out);
  else
    hipLaunchKernelGGL(k_readout_near<false>, dim3(M), dim3(64), 0, s, N, M,
                       nchunk, part, verts, tri, geo, ru, x, xyz, srow, scol, out);
  PBMP_HIP(hipGetLastError());
}

void launch_perm_field(hipStream_t s, int M, const double *xyz,
                       const double *q, const double *d, const double *Q9,
                       const int *group, double eps_in, double *E) {
  if (M <= 0) return;
  hipLaunchKernelGGL(k_perm_field, dim3(M), dim3(64), 0, s, M,
                     xyz, q, d, Q9, group, 1.0 / eps_in, E);
  PBMP_HIP(hipGetLastError());
}

void launch_induced(hipStream_t s, bool full, int M, const double *xyz,
                    const double *mu, const double *alpha, double thole_a,
                    double eps_in, double *out) {
  if (M <= 0) return;
  if (full)
    hipLaunchKernelGGL(k_induced<true>, dim3(M), dim3(64), 0, s,
                       M, xyz, mu, alpha, thole_a, 1.0 / eps_in, out);
  else
    hipLaunchKernelGGL(k_induced<false>, dim3(M), dim3(64), 0, s,
                       M, xyz, mu, alpha, thole_a, 1.0 / eps_in, out);
  PBMP_HIP(hipGetLastError());
}

void launch_scf_update(hipStream_t s, int M, const double *alpha,
                       const double *Eperm, const double *Eind,
                       const double *solv10, int solv_stride, double omega,
                       double *mu, double *dmu2) {
  hipLaunchKernelGGL(k_scf_update, dim3(1), dim3(256), 0, s, M, alpha, Eperm,
                     Eind, solv10, solv_stride, omega, mu, dmu2);
  PBMP_HIP(hipGetLastError());
}

void launch_energy(hipStream_t s, int M, const double *q, const double *d,
                   const double *Q9, const double *reac10, const double *ind10,
                   double *e) {
  hipLaunchKernelGGL(k_energy, dim3(1), dim3(256), 0, s, M, q, d, Q9, reac10,
                     ind10, e);
  PBMP_HIP(hipGetLastError());
}

}  // namespace pbmp
