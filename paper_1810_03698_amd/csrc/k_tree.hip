// Treecode product (section "The treecode algorithm"): Cartesian Taylor
// expansion of the kernels about box centres.
//
//   G(x, y_c + h) = sum_{|k|<=P} a_k(x) h^k,   a_k = (1/k!) D_y^k G(x, y_c)
//
// With D = x - y_c the coefficients follow the recurrences of Lindsay-Krasny
// (Laplace, G = 1/r) and Li-Johnston-Krasny (Yukawa, G = e^{-kr}/r, with
// auxiliary coefficients b_k of e^{-kr}); n = |k|:
//   n |D|^2 a_k = (2n-1) sum_i D_i a_{k-e_i} - (n-1) sum_i a_{k-2e_i}
//                 + kappa (sum_i D_i b_{k-e_i} - sum_i b_{k-2e_i}),
//   n b_k       = kappa (sum_i D_i a_{k-e_i} - sum_i a_{k-2e_i}),
// a_0 = e^{-k|D|}/|D|, b_0 = e^{-k|D|} (kappa = 0: Laplace).  Box moments
//   single layer  m_k  = sum_nodes s_V h^k,
//   double layer  mK_k = sum_nodes s_K sum_i k_i n_i h^{k-e_i}
// (the double-layer kernel is n.grad_y G) give V = sum_{|k|<=P} a_k m_k and
// K = sum_{|k|<=P+1} a_k mK_k: the double-layer moment of degree |k| holds
// h^(|k|-1), so its series is carried one degree further and both layers
// are truncated at degree P in h.  Moments are formed in FP64: those of the
// leaves from their nodes, those of the accepted boxes above the leaves
// from the leaf moments by exact binomial shifts.  The products evaluate the
// two series regrouped by solid harmonics (harmonic.hpp), from words made of
// a box's finished moments; the recurrences serve the vertex gradient.
#include <algorithm>
#include <cmath>

#include <type_traits>

#include "harmonic.hpp"
#include "kernels.hpp"
#include "pair.hpp"
#include "runtime.hpp"

namespace pbmp {

namespace {

// Multi-indices |k| <= P ordered by degree, then x exponent descending,
// then y exponent descending; m1/m2: positions of k - e_i and k - 2 e_i.
template <int P> struct Multi {
  static constexpr int n = (P + 1) * (P + 2) * (P + 3) / 6;
  int e[n][3];
  int m1[n][3];
  int m2[n][3];
  int p1[n][3];  // position of k + e_i (-1 beyond degree P)
  int deg[n];
  static constexpr int index(int i, int j, int l) {
    const int s = i + j + l;
    return s * (s + 1) * (s + 2) / 6 + (s - i) * (s - i + 1) / 2 + (s - i - j);
  }
  constexpr Multi() : e(), m1(), m2(), p1(), deg() {
    int k = 0;
    for (int s = 0; s <= P; ++s)
      for (int i = s; i >= 0; --i)
        for (int j = s - i; j >= 0; --j) {
          const int l = s - i - j;
          e[k][0] = i;
          e[k][1] = j;
          e[k][2] = l;
          deg[k] = s;
          const int ex[3] = {i, j, l};
          for (int d = 0; d < 3; ++d) {
            int a[3] = {ex[0], ex[1], ex[2]};
            a[d] -= 1;
            m1[k][d] = (a[d] >= 0) ? index(a[0], a[1], a[2]) : -1;
            a[d] -= 1;
            m2[k][d] = (a[d] >= 0) ? index(a[0], a[1], a[2]) : -1;
            a[d] += 3;
            p1[k][d] = (s < P) ? index(a[0], a[1], a[2]) : -1;
          }
          ++k;
        }
  }
};

constexpr double kInv4PiT = 0.07957747154594767;

inline int ncoef_of(int P) { return (P + 1) * (P + 2) * (P + 3) / 6; }

// coefficient counts of order P: NV single-layer terms (|k| <= P), NK
// double-layer terms (|k| <= P + 1); a box's moments are [NV | NK]
template <int P> struct Orders {
  static constexpr int NV = Multi<P>::n;
  static constexpr int NK = Multi<P + 1>::n;
  static constexpr int NM = NV + NK;
  static constexpr int L = P + 1;       // degree of the harmonic form
  static constexpr int NS = Harm<L>::S; // its words per box
};

// blockIdx -> task: consecutive tasks (neighbouring target leaves, similar
// source lists) land on the same XCD so they share its L2.
__device__ inline int xcd_task(int ntasks) {
  const int per = (gridDim.x + 7) / 8;
  const int t = (blockIdx.x % 8) * per + blockIdx.x / 8;
  return t < ntasks ? t : -1;
}

// ------------------------------------------------------------- harmonics
// The harmonic words of a box (harmonic.hpp) from its Cartesian moments m
// [NV | NK] in LDS, merged into the two rows of the product: Laplace mK - mV,
// Yukawa eps mV - mK.  A lane per harmonic (at most 64), its terms (k, C for
// Laplace, C for Yukawa) from a table.  Called by the first wave of whichever
// block holds a box's final moments, so that the map costs no launch of its
// own; to words64 or, rounded, to words32 (the other is null).
struct HarmOut {
  const int *off, *k, *pos;
  const double *c;
  double eps_ratio;
  double *words64;
  float *words32;
};

template <int P>
__device__ __forceinline__ void harmonic_words(int box, const double *m, const HarmOut &h) {
  constexpr int NC = Orders<P>::NV, NS = Orders<P>::NS, NH = Harm<P + 1>::NH;
  static_assert(NH <= 64, "a lane per harmonic");
  const int lane = (int)threadIdx.x;
  if (lane >= NH) return;
  double a = 0.0, b = 0.0;
  for (int t = h.off[lane]; t < h.off[lane + 1]; ++t) {
    const int k = h.k[t];
    const double mv = k < NC ? m[k] : 0.0, mk = m[NC + k];
    a += h.c[2 * t] * (mk - mv);
    b += h.c[2 * t + 1] * (h.eps_ratio * mv - mk);
  }
  const size_t o = (size_t)box * NS + h.pos[lane];
  if (h.words64) {
    h.words64[o] = a;
    h.words64[o + 1] = b;
  } else {
    h.words32[o] = (float)a;
    h.words32[o + 1] = (float)b;
  }
}

// ---------------------------------------------------------------- P2M
// Moments of every leaf straight from its nodes (every box is a contiguous
// panel range), one block per task, a task being a leaf's panels [s0, s1) or a
// slice of at most kMomChunkPanels of them.  With h the node offsets,
//   mV_k = sum s_V h^k,   mK_k = sum_d k_d sum s_K n_d h^(k - e_d),
// so the four weighted sums of h^k with weights s_V, s_K n_x, s_K n_y, s_K n_z
// over |k| <= P suffice: one per wave, lanes over the nodes, all monomials built
// incrementally (each from its parent multi-index).  The panel records pass
// through LDS in tiles, padded to 17 doubles against bank conflicts.
// k_mom_reduce adds a leaf's slices in a fixed order.  Latency bound (a few
// hundred to a thousand leaves); one wave per leaf with both moment sets of
// 140 coefficients at P 5 left one wave per SIMD.
constexpr int kP2MTile = 64;  // panels per LDS tile

// direct: every leaf is one task, so the task's sums are the leaf's moments
// and go straight to mom64 and the harmonic words instead of part
template <int P>
__global__ __launch_bounds__(256) void k_p2m_tasks(int nf, const int *__restrict__ tasks,
                                                   const double *__restrict__ center,
                                                   const double *__restrict__ src,
                                                   const int *__restrict__ monos,
                                                   double *__restrict__ part, int direct,
                                                   double *__restrict__ mom64, HarmOut ho) {
  constexpr Multi<P> mi{};
  constexpr int NC = Orders<P>::NV, NM = Orders<P>::NM, NA = (NC + 3) / 4 * 4;
  __shared__ double sh[kP2MTile * 17];
  __shared__ double col[4][NC];
  __shared__ double fin[NM];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int B = tasks[3 * blockIdx.x];
  const int s0 = tasks[3 * blockIdx.x + 1], s1 = tasks[3 * blockIdx.x + 2];
  const double c[3] = {center[3 * B], center[3 * B + 1], center[3 * B + 2]};
  double acc[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) acc[k] = 0.0;
  for (int jt = s0; jt < s1; jt += kP2MTile) {
    const int nj = min(kP2MTile, s1 - jt);
    __syncthreads();
    {
      typedef double d2 __attribute__((ext_vector_type(2)));
      const d2 *s2 = reinterpret_cast<const d2 *>(src + (size_t)jt * 16);
      d2 buf[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int e = (int)threadIdx.x + 256 * u;
        if (e < nj * 8) buf[u] = s2[e];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int e = (int)threadIdx.x + 256 * u;
        if (e < nj * 8) {
          double *d = sh + 17 * (e >> 3) + 2 * (e & 7);
          d[0] = buf[u].x;
          d[1] = buf[u].y;
        }
      }
    }
    __syncthreads();
    for (int g = lane; g < nj * nf; g += 64) {
      const int q = g % nf;
      const double *r = sh + 17 * (g / nf);
      const double h[3] = {r[3 * q] - c[0], r[3 * q + 1] - c[1], r[3 * q + 2] - c[2]};
      const double w = wave == 0 ? r[13] : r[14] * r[8 + wave];
      double mono[NC];
      mono[0] = w;
      acc[0] += w;
#pragma unroll
      for (int k = 1; k < NC; ++k) {
        const int d = mi.e[k][0] ? 0 : (mi.e[k][1] ? 1 : 2);
        mono[k] = mono[mi.m1[k][d]] * h[d];
        acc[k] += mono[k];
      }
    }
  }
  wave_sums(acc, [&](int k, double v) {
    if (k < NC) col[wave][k] = v;
  });
  __syncthreads();
  for (int e = threadIdx.x; e < NM; e += 256) {
    double v;
    if (e < NC) {
      v = col[0][e];
    } else {
      const int *x = monos + 3 * (e - NC);
      v = 0.0;
      if (x[0]) v += x[0] * col[1][Multi<P>::index(x[0] - 1, x[1], x[2])];
      if (x[1]) v += x[1] * col[2][Multi<P>::index(x[0], x[1] - 1, x[2])];
      if (x[2]) v += x[2] * col[3][Multi<P>::index(x[0], x[1], x[2] - 1)];
    }
    if (direct) {
      fin[e] = v;
      mom64[(size_t)B * NM + e] = v;
    } else {
      part[(size_t)blockIdx.x * NM + e] = v;
    }
  }
  if (direct) {
    __syncthreads();
    harmonic_words<P>(B, fin, ho);
  }
}

// mom[B] = sum of the partial moments of B's slices, in slice order, and the
// box's harmonic words (boxes with fewer than min_tasks tasks are skipped: not
// this pass's, or written by their single task)
template <int P>
__global__ __launch_bounds__(128) void k_mom_reduce(const int *__restrict__ first,
                                                    const int *__restrict__ count,
                                                    const double *__restrict__ part,
                                                    double *__restrict__ mom, int min_tasks,
                                                    HarmOut ho) {
  constexpr int NM = Orders<P>::NM;
  __shared__ double fin[NM];
  const int B = blockIdx.x, t0 = first[B], nt = count[B];
  if (nt == 0 || nt < min_tasks) return;
  for (int k = threadIdx.x; k < NM; k += 128) {
    double v = 0.0;
    for (int t = t0; t < t0 + nt; ++t) v += part[(size_t)t * NM + k];
    fin[k] = v;
    mom[(size_t)B * NM + k] = v;
  }
  __syncthreads();
  harmonic_words<P>(B, fin, ho);
}

// Moments of the accepted boxes with children from the leaf moments: with
// d = c_L - c_B, (h + d)^k = sum_{j <= k} C(k, j) d^(k-j) h^j, and the
// double-layer moments (n . grad_h) h^k shift with the same coefficients,
// so m_k(B) = sum over the leaves L under B of sum_{j <= k} C(k, j)
// d^(k-j) m_j(L), for both moment sets.  One block of eight waves per task (a
// run of at most kShiftLeaves of a box's leaves, two to a wave): the moments of
// the leaves, the monomials of their d and the
// term table (j, k - j, C(k, j) in one word) are staged in LDS, then each lane
// owns coefficients k and walks its terms.  LDS bound (24 bytes per lane, term
// and leaf, 2.6 us per block at P 5) and latency bound below some 500 tasks;
// one wave with sixteen leaves and the table in global memory took 76 us on
// 144500 panels at P 5 and 40 us on 28880 at P 4, this 18 and 9.
constexpr int kShiftWaves = 8;

template <int P>
__global__ __launch_bounds__(64 * kShiftWaves) void k_shift_tasks(
    const int *__restrict__ tasks, const int *__restrict__ leaves,
    const double *__restrict__ center, const int *__restrict__ monos,
    const int *__restrict__ toff, const unsigned *__restrict__ terms,
    double *__restrict__ mom, const int *__restrict__ count, double *__restrict__ part,
    HarmOut ho) {
  // single-layer moments k < NC, double-layer k < NK (the terms of a
  // coefficient reach only coefficients of lower or equal degree, so one
  // table of degree P + 1 serves both)
  constexpr int NC = Orders<P>::NV, NK = Orders<P>::NK, NM = Orders<P>::NM;
  constexpr int R = (NK + 63) / 64, TH = 64 * kShiftWaves, LW = kShiftLeaves / kShiftWaves;
  constexpr int NT = (P + 2) * (P + 3) * (P + 4) * (P + 5) * (P + 6) * (P + 7) / 720;
  __shared__ __align__(16) double sm[kShiftLeaves][NK][2];  // (mV, mK); mV 0 beyond NC
  __shared__ double sd[kShiftLeaves][NK];
  __shared__ double pw[kShiftLeaves][3][P + 2];
  __shared__ unsigned st[NT];
  __shared__ int sL[kShiftLeaves];
  static_assert(sizeof(sm) >= sizeof(double) * kShiftWaves * NM, "the reduction reuses sm");
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int B = tasks[3 * blockIdx.x];
  const int l0 = tasks[3 * blockIdx.x + 1], l1 = tasks[3 * blockIdx.x + 2];
  for (int e = threadIdx.x; e < NT; e += TH) st[e] = terms[e];
  double aV[R], aK[R];
#pragma unroll
  for (int r = 0; r < R; ++r) aV[r] = aK[r] = 0.0;
  const int nl = l1 - l0;
  if ((int)threadIdx.x < nl) sL[threadIdx.x] = leaves[l0 + threadIdx.x];
  __syncthreads();
  for (int e = threadIdx.x; e < nl * NK; e += TH) {
    const int l = e / NK, k = e % NK;
    const double *m = mom + (size_t)sL[l] * NM;
    sm[l][k][0] = k < NC ? m[k] : 0.0;
    sm[l][k][1] = m[NC + k];
  }
  if ((int)threadIdx.x < nl * 3) {
    const int l = threadIdx.x / 3, d = threadIdx.x % 3;
    const double x = center[3 * sL[l] + d] - center[3 * B + d];
    double v = 1.0;
    for (int u = 0; u < P + 2; ++u) {
      pw[l][d][u] = v;
      v *= x;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < nl * NK; e += TH) {
    const int l = e / NK, k = e % NK;
    sd[l][k] = pw[l][0][monos[3 * k]] * pw[l][1][monos[3 * k + 1]] * pw[l][2][monos[3 * k + 2]];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = lane + 64 * r;
    if (k >= NK) continue;
    const int t0 = toff[k], t1 = toff[k + 1];
    for (int t = t0; t < t1; ++t) {
      const unsigned w = st[t];
      const int j = w & 255, q = (w >> 8) & 255;
      const double ct = (double)(w >> 16);
#pragma unroll
      for (int u = 0; u < LW; ++u) {
        const int l = LW * wave + u;
        if (l < nl) {
          const double c = ct * sd[l][q];
          aV[r] += c * sm[l][j][0];
          aK[r] += c * sm[l][j][1];
        }
      }
    }
  }
  __syncthreads();
  double *red = &sm[0][0][0];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = lane + 64 * r;
    if (k >= NK) continue;
    if (k < NC) red[wave * NM + k] = aV[r];
    red[wave * NM + NC + k] = aK[r];
  }
  __syncthreads();
  const bool last = count[B] == 1;  // the box's only task: its moments
  for (int k = threadIdx.x; k < NM; k += TH) {
    double v = red[k];
    for (int w = 1; w < kShiftWaves; ++w) v += red[w * NM + k];
    red[k] = v;
    if (last) mom[(size_t)B * NM + k] = v;
    else part[(size_t)blockIdx.x * NM + k] = v;
  }
  if (last) {
    __syncthreads();
    harmonic_words<P>(B, red, ho);
  }
}


// ------------------------------------------------------------ P2P tasks
// One 64-lane block per task: targets [t0, t1) of a leaf, sources = the
// task's panel sub-ranges, streamed through LDS.  Leaves are often much
// smaller than a wave, so the lanes are split into G groups of L = 64 / G:
// every group holds all targets (TPT per lane) and takes every G-th source
// panel of a tile; group 0 adds the other groups' FP64 sums through lane
// shuffles in a fixed order.  G and TPT are chosen per task to use the most
// lanes.  Tile, TPT bound and the use of groups are compile-time settings
// (the defaults were the fastest measured; M2P runs without groups).
constexpr int kTileT = PBMP_P2P_TILE;
constexpr int kMaxTPT = PBMP_P2P_MAXTPT;

// Copies nj (<= MAXREC) records of 16 T from global memory to LDS in
// 16-byte accesses, every load of the lane issued before the first store
// (a plain copy loop waits for each load before its store).
template <class T, int MAXREC>
__device__ __forceinline__ void stage_records(const T *__restrict__ src, T *sh, int nj,
                                              int lane) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef double d2 __attribute__((ext_vector_type(2)));
  using V = typename std::conditional<sizeof(T) == 4, f4, d2>::type;
  constexpr int PER = 16 * (int)sizeof(T) / 16;  // 16-byte units per record
  constexpr int U = (MAXREC * PER + 63) / 64;
  const V *s = reinterpret_cast<const V *>(src);
  V *d = reinterpret_cast<V *>(sh);
  constexpr int B = 2;  // loads in flight per round (registers of the caller stay free)
  const int n = nj * PER;
#pragma unroll
  for (int u0 = 0; u0 < U; u0 += B) {
    V buf[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int e = lane + 64 * (u0 + u);
      if (u0 + u < U && e < n) buf[u] = s[e];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int e = lane + 64 * (u0 + u);
      if (u0 + u < U && e < n) d[e] = buf[u];
    }
  }
}

template <class T, int NF, int TPT, bool FLOOR>
__device__ void p2p_task_body(const T *__restrict__ src, const T *__restrict__ tgt,
                              int N, int t0, int t1, const int *__restrict__ ranges,
                              int lb, int le, const Screen<T> &sc, int slot,
                              double *__restrict__ part, T *sh, int G, int L) {
  const int lane = (int)threadIdx.x;
  const int gi = lane / L, li = lane - gi * L;
  const bool active = gi < G;
  for (int tb = t0; tb < t1; tb += L * TPT) {
    T px[TPT], py[TPT], pz[TPT];
    int ti[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      ti[k] = tb + k * L + li;
      const int tl = min(ti[k], t1 - 1);
      px[k] = tgt[tl];
      py[k] = tgt[N + tl];
      pz[k] = tgt[2 * N + tl];
    }
    double S[TPT][2];
#pragma unroll
    for (int k = 0; k < TPT; ++k) S[k][0] = S[k][1] = 0.0;
    for (int l = lb; l < le; ++l) {
      const int s0 = ranges[2 * l], s1 = ranges[2 * l + 1];
      for (int jt = s0; jt < s1; jt += kTileT) {
        const int nj = min(kTileT, s1 - jt);
        __syncthreads();
        stage_records<T, kTileT>(src + (size_t)jt * 16, sh, nj, lane);
        __syncthreads();
        T a[TPT][2][kAcc<T, NF>];
#pragma unroll
        for (int k = 0; k < TPT; ++k)
          for (int c = 0; c < 2; ++c)
            for (int q = 0; q < kAcc<T, NF>; ++q) a[k][c][q] = T(0);
        for (int jj = active ? gi : nj; jj < nj; jj += G) {
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
    }
    if (G > 1) {
      // group 0 adds the other groups' sums (lane li of group g is lane
      // li + g L); every lane takes part in the shuffles
#pragma unroll
      for (int k = 0; k < TPT; ++k)
        for (int c = 0; c < 2; ++c) {
          const double v = S[k][c];
          double acc = v;
          for (int g = 1; g < G; ++g) acc += __shfl(v, li + g * L, 64);
          S[k][c] = acc;
        }
    }
    if (gi == 0)
#pragma unroll
      for (int k = 0; k < TPT; ++k)
        if (ti[k] < t1)
          for (int c = 0; c < 2; ++c) part[((size_t)slot * 2 + c) * N + ti[k]] = S[k][c];
  }
}

template <class T, int NF, bool FLOOR>
__global__ __launch_bounds__(64) void k_p2p_tasks(int ntask, const int *__restrict__ tasks,
                                                  const int *__restrict__ slots,
                                                  const int *__restrict__ ranges,
                                                  const T *__restrict__ src,
                                                  const T *__restrict__ tgt, int N,
                                                  T kappa, double *__restrict__ part) {
  __shared__ __align__(16) T sh[kTileT * 16];
  __shared__ double etab[sizeof(T) == 8 ? 64 : 1];
  const Screen<T> sc = make_screen(kappa, etab);
  const int task = xcd_task(ntask);
  if (task < 0) return;
  const int t0 = tasks[4 * task], t1 = tasks[4 * task + 1];
  const int lb = tasks[4 * task + 2], le = tasks[4 * task + 3];
  const int slot = slots[task];
  const LaneSplit ls = lane_split(t1 - t0, kMaxTPT);
  switch (ls.tpt) {
#define PBMP_BODY(K)                                                                        \
  p2p_task_body<T, NF, K, FLOOR>(src, tgt, N, t0, t1, ranges, lb, le, sc, slot, part, sh, ls.G, \
                                 ls.L)
    case 1: PBMP_BODY(1); break;
    case 2: PBMP_BODY(2); break;
#if PBMP_P2P_MAXTPT >= 4
    case 3: PBMP_BODY(3); break;
    case 4: PBMP_BODY(4); break;
    default: PBMP_BODY(kMaxTPT); break;
#else
    default: PBMP_BODY(3); break;
#endif
#undef PBMP_BODY
  }
}

// ------------------------------------------------------------ M2P tasks

template <class T> __device__ inline T rsqrt_t(T x);
template <> __device__ inline float rsqrt_t<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <> __device__ inline double rsqrt_t<double>(double x) { return rsqrt_fp64(x); }
template <class T> __device__ inline T expneg_t(T nk, T kappa, T r);
template <> __device__ inline float expneg_t<float>(float nk, float, float r) {
  return __builtin_amdgcn_exp2f(nk * r);
}
template <> __device__ inline double expneg_t<double>(double, double kappa, double r) {
  return exp_fp64(-kappa * r);
}

// M2P.  A task is a target leaf against a run of its accepted boxes, one wave,
// TPT targets per lane (the fewest passes): the words of up to kStage boxes
// pass through LDS and every read serves TPT targets.  VALU issue bound: 220
// instructions per (target, box) pair at P 5 where the Cartesian recurrences
// (three families of 84 coefficients) took about 2000: 814 -> 149 us in FP32
// and 1829 -> 326 us in FP64 on 144500 panels at P 5, 120 -> 44 us in FP32 on
// 28880 at P 4.  FP32 sums span the boxes of one stage and are added in FP64.
template <class T, int P> constexpr int m2p_stage() {
  constexpr int n = kM2PStageBytes / (Orders<P>::NS * (int)sizeof(T));
  return n < kM2PChunkBoxes ? n : kM2PChunkBoxes;
}

template <class T, int P, int TPT>
__device__ void m2p_body(int t0, int t1, int lb, int le, const int *__restrict__ boxes,
                         const double *__restrict__ center, const T *__restrict__ words,
                         const T *__restrict__ tgt, int N, T kappa, T nk, int slot,
                         double *__restrict__ part, T *sh, T *scen, int *sbox) {
  constexpr int NS = Orders<P>::NS;
  constexpr int kStage = m2p_stage<T, P>();
  typedef T v2 __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int UN = NS * (int)sizeof(T) / 16;  // 16-byte units per box
  const int lane = (int)threadIdx.x;
  for (int tb = t0; tb < t1; tb += 64 * TPT) {
    T p[TPT][3];
    double S[TPT][2];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      const int tl = min(tb + 64 * k + lane, t1 - 1);
      for (int d = 0; d < 3; ++d) p[k][d] = tgt[(size_t)d * N + tl];
      S[k][0] = S[k][1] = 0.0;
    }
    for (int cb = lb; cb < le; cb += kStage) {
      const int nb = min(kStage, le - cb);
      if (tb == t0 || le - lb > kStage) {
        __syncthreads();
        if (lane < nb) sbox[lane] = boxes[cb + lane];
        __syncthreads();
        const v2 *g = reinterpret_cast<const v2 *>(words);
        v2 *d = reinterpret_cast<v2 *>(sh);
        for (int e0 = lane; e0 < nb * UN; e0 += 4 * 64) {
          v2 v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = e0 + 64 * u;
            if (e < nb * UN) v[u] = g[(size_t)sbox[e / UN] * UN + e % UN];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = e0 + 64 * u;
            if (e < nb * UN) d[e] = v[u];
          }
        }
        for (int e = lane; e < nb * 3; e += 64) scen[e] = (T)center[3 * sbox[e / 3] + e % 3];
        __syncthreads();
      }
      T acc[TPT][2];
#pragma unroll
      for (int k = 0; k < TPT; ++k) acc[k][0] = acc[k][1] = T(0);
      for (int b = 0; b < nb; ++b) {
        T D[TPT][3], ri[TPT], ek[TPT];
#pragma unroll
        for (int k = 0; k < TPT; ++k) {
          for (int d = 0; d < 3; ++d) D[k][d] = p[k][d] - scen[3 * b + d];
          const T R2 = D[k][0] * D[k][0] + D[k][1] * D[k][1] + D[k][2] * D[k][2];
          ri[k] = rsqrt_t<T>(R2);
          ek[k] = expneg_t<T>(nk, kappa, R2 * ri[k]);
        }
        harmonic_m2p<T, P + 1, TPT>(sh + b * NS, D, ri, ek, kappa, acc);
      }
#pragma unroll
      for (int k = 0; k < TPT; ++k)
        for (int c = 0; c < 2; ++c) S[k][c] += (double)acc[k][c];
    }
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      const int t = tb + 64 * k + lane;
      if (t < t1)
        for (int c = 0; c < 2; ++c) part[((size_t)slot * 2 + c) * N + t] = S[k][c];
    }
  }
}

template <class T, int P>
__global__ __launch_bounds__(64, sizeof(T) == 4 ? 3 : 2) void k_m2p_tasks(int ntask, const int *__restrict__ tasks,
                                                  const int *__restrict__ slots,
                                                  const int *__restrict__ boxes,
                                                  const double *__restrict__ center,
                                                  const T *__restrict__ words,
                                                  const T *__restrict__ tgt, int N,
                                                  T kappa, T nk, double *__restrict__ part) {
  constexpr int kStage = m2p_stage<T, P>();
  __shared__ __align__(16) T sh[kStage * Orders<P>::NS];
  __shared__ T scen[kStage * 3];
  __shared__ int sbox[kStage];
  const int task = xcd_task(ntask);
  if (task < 0) return;
  const int t0 = tasks[4 * task], t1 = tasks[4 * task + 1];
  const int lb = tasks[4 * task + 2], le = tasks[4 * task + 3];
  const int slot = slots[task];
  // TPT up to 3 in FP32 and 2 in FP64 (on 144500 panels at P 5, bounds of 1, 2
  // and 3: 155, 159, 149 us and 333, 326, 375 us; three FP64 targets spill)
  constexpr int kMax = sizeof(T) == 4 ? 3 : 2;
  const int nt = t1 - t0, passes = (nt + 64 * kMax - 1) / (64 * kMax);
  const int tpt = (nt + 64 * passes - 1) / (64 * passes);
#define PBMP_MB(K)                                                                             \
  m2p_body<T, P, K>(t0, t1, lb, le, boxes, center, words, tgt, N, kappa, nk, slot, part, sh,   \
                    scen, sbox)
  if (tpt <= 1) PBMP_MB(1);
  else if (tpt == 2) PBMP_MB(2);
  else PBMP_MB(kMax);
#undef PBMP_MB
}

// y = A x from the far-field slots and the near/self corrections.  Four
// lanes per row (a wave takes 16 rows): lane u of a row sums the row's slots
// u, u + 4, ... and its correction entries u, u + 4, ..., so that the
// four lanes read neighbouring entries together and a launch holds four
// times as many waves to hide the latency of the scattered reads of x;
// the lanes' sums are then added in a fixed order (lane shuffles).
constexpr int kFinLanes = 4;
constexpr int kFinBlock = 256;

__global__ __launch_bounds__(kFinBlock) void k_finish_slots(
    int N, const int *__restrict__ tslots, const double *__restrict__ part,
    const int *__restrict__ rowptr, const int *__restrict__ col,
    const double *__restrict__ val, const double *__restrict__ x, double eps_ratio,
    const int *__restrict__ perm, double *__restrict__ y) {
  const int t = blockIdx.x * kFinBlock + (int)threadIdx.x;
  const int i = t / kFinLanes, u = t % kFinLanes;
  const bool live = i < N;
  const int il = live ? i : N - 1;
  double S[2] = {0.0, 0.0};
  const int ns = tslots[il];
  for (int c = u; c < ns; c += kFinLanes)
#pragma unroll
    for (int k = 0; k < 2; ++k) S[k] += part[((size_t)c * 2 + k) * N + il];
  const int e1 = rowptr[il + 1];
  for (int e = rowptr[il] + u; e < e1; e += kFinLanes) {
    const int j = col[e];
    const double ph = x[j], dp = x[N + j];
    const double *v = val + 4 * (size_t)e;
    S[0] += v[1] * ph - v[0] * dp;
    S[1] += eps_ratio * v[2] * dp - v[3] * ph;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    S[k] += __shfl_xor(S[k], 1, kFinLanes);
    S[k] += __shfl_xor(S[k], 2, kFinLanes);
  }
  if (!live || u != 0) return;
  const double ph = x[i];
  const int o = perm ? perm[i] : i;
  y[o] = 0.5 * ph + S[0];
  y[N + o] = 0.5 * ph + S[1];
}

template <class T, int P>
void launch_m2p_p(Tree &t, hipStream_t s, const T *words, const T *tgt, int N, T kappa, T nk,
                  double *part) {
  const int nb = ((t.n_m2p_tasks + 7) / 8) * 8;
  hipLaunchKernelGGL((k_m2p_tasks<T, P>), dim3(nb), dim3(64), 0, s, t.n_m2p_tasks,
                     t.d_m2p_task.p, t.d_m2p_slot.p, t.d_m2p_box.p, t.d_center.p, words,
                     tgt, N, kappa, nk, part);
}

template <int P>
void launch_moments_p(Tree &t, hipStream_t s, int nf, const double *src64, bool fp64,
                      double eps_ratio) {
  if (t.n_mom_tasks == 0) return;
  const HarmOut ho{t.d_hoff.p, t.d_hk.p, t.d_hpos.p, t.d_hc.p, eps_ratio,
                   fp64 ? t.d_harm64.p : nullptr, fp64 ? nullptr : t.d_harm32.p};
  const int direct = t.n_mom_tasks == t.nleaf;  // no leaf split into slices
  hipLaunchKernelGGL(k_p2m_tasks<P>, dim3(t.n_mom_tasks), dim3(256), 0, s, nf,
                     t.d_mom_task.p, t.d_center.p, src64, t.d_monos.p, t.d_mom_part.p, direct,
                     t.d_mom64.p, ho);
  if (!direct)
    hipLaunchKernelGGL(k_mom_reduce<P>, dim3(t.nbox), dim3(128), 0, s, t.d_mom_first.p,
                       t.d_mom_count.p, t.d_mom_part.p, t.d_mom64.p, 1, ho);
  if (t.n_shift_tasks > 0) {
    hipLaunchKernelGGL(k_shift_tasks<P>, dim3(t.n_shift_tasks), dim3(64 * kShiftWaves), 0, s,
                       t.d_shift_task.p, t.d_leaves.p, t.d_center.p, t.d_monos.p,
                       t.d_shift_toff.p, t.d_shift_term.p, t.d_mom64.p, t.d_shift_count.p,
                       t.d_shift_part.p, ho);
    if (t.shift_multi)
      hipLaunchKernelGGL(k_mom_reduce<P>, dim3(t.nbox), dim3(128), 0, s, t.d_shift_first.p,
                         t.d_shift_count.p, t.d_shift_part.p, t.d_mom64.p, 2, ho);
  }
}

#define PBMP_BY_ORDER(CALL)                                            \
  switch (t.prm.order) {                                               \
    case 1: CALL(1); break;                                            \
    case 2: CALL(2); break;                                            \
    case 3: CALL(3); break;                                            \
    case 4: CALL(4); break;                                            \
    case 5: CALL(5); break;                                            \
    case 6: CALL(6); break;                                            \
    default: throw Error(PBMP_EARG, "treecode order must be 1..6");    \
  }

template <class T>
void launch_m2p(Tree &t, hipStream_t s, const T *words, const T *tgt, int N, T kappa, T nk,
                double *part) {
#define PBMP_CALL(P) launch_m2p_p<T, P>(t, s, words, tgt, N, kappa, nk, part)
  PBMP_BY_ORDER(PBMP_CALL)
#undef PBMP_CALL
}

// Cartesian moments of every leaf and accepted box, FP64, and their harmonic
// words in the product's precision
void launch_moments(Tree &t, hipStream_t s, int nf, const double *src64, bool fp64,
                    double eps_ratio) {
#define PBMP_CALL(P) launch_moments_p<P>(t, s, nf, src64, fp64, eps_ratio)
  PBMP_BY_ORDER(PBMP_CALL)
#undef PBMP_CALL
}


// ===================================================== transposed product
// A^T z for the adjoint solve, the exact transpose of the treecode product
// above: P2P^T runs the forward P2P pairs with sources on lanes; M2P^T
// gathers, for every accepted box B, local coefficients
//   L_B,k = sum over the targets i of the leaves that accepted B of z_i a_k(x_i - c_B)
// (Laplace coefficients with the first component of z, Yukawa with the
// second); L2P evaluates at every node y the expansions of all boxes that
// contain it, h = y - c_B,
//   V^T: sum_k L_k h^k,   K^T: n . grad_h sum_k L_k h^k,
// the transpose of forming every box's moments from its nodes.

template <class T, int NF, int SPT, bool FLOOR>
__device__ void p2pT_body(const T *__restrict__ src, const T *__restrict__ tgt,
                          const double *__restrict__ z, const double *__restrict__ geo, int N,
                          int s0, int s1, const int *__restrict__ ranges, int lb, int le,
                          const Screen<T> &sc, double eps_ratio, int slot,
                          double *__restrict__ part, T *sh, int G, int L) {
  const int lane = (int)threadIdx.x;
  const int gi = lane / L, li = lane - gi * L;
  const bool active = gi < G;
  for (int sb = s0; sb < s1; sb += L * SPT) {
    T rec[SPT][12];
    int sj[SPT];
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      sj[k] = sb + k * L + li;
      const int jl = min(sj[k], s1 - 1);
      for (int c = 0; c < 12; ++c) rec[k][c] = src[16 * (size_t)jl + c];
    }
    double S[SPT][2];
#pragma unroll
    for (int k = 0; k < SPT; ++k) S[k][0] = S[k][1] = 0.0;
    for (int l = lb; l < le; ++l) {
      const int a0 = ranges[2 * l], a1 = ranges[2 * l + 1];
      for (int it = a0; it < a1; it += 64) {
        const int nt = min(64, a1 - it);
        __syncthreads();
        if (lane < nt) {
          const int i = it + lane;
          sh[8 * lane] = tgt[i];
          sh[8 * lane + 1] = tgt[N + i];
          sh[8 * lane + 2] = tgt[2 * N + i];
          sh[8 * lane + 3] = (T)z[i];
          sh[8 * lane + 4] = (T)z[N + i];
          sh[8 * lane + 5] = (T)(eps_ratio * z[N + i]);
        }
        __syncthreads();
        T a[SPT][2][kAcc<T, NF>];
#pragma unroll
        for (int k = 0; k < SPT; ++k)
          for (int c = 0; c < 2; ++c)
            for (int q = 0; q < kAcc<T, NF>; ++q) a[k][c][q] = T(0);
        for (int e = active ? gi : nt; e < nt; e += G) {
          const T *r = sh + 8 * e;
#pragma unroll
          for (int k = 0; k < SPT; ++k)
            panel_columns<NF, FLOOR>(rec[k], r[0], r[1], r[2], r[3], r[4], r[5], sc, a[k]);
        }
#pragma unroll
        for (int k = 0; k < SPT; ++k)
          for (int c = 0; c < 2; ++c)
            for (int q = 0; q < kAcc<T, NF>; ++q) S[k][c] += (double)a[k][c][q];
      }
    }
    if (G > 1) {
#pragma unroll
      for (int k = 0; k < SPT; ++k)
        for (int c = 0; c < 2; ++c) {
          const double v = S[k][c];
          double acc = v;
          for (int g = 1; g < G; ++g) acc += __shfl(v, li + g * L, 64);
          S[k][c] = acc;
        }
    }
    if (gi == 0)
#pragma unroll
      for (int k = 0; k < SPT; ++k)
        if (sj[k] < s1) {
          const double wA = geo[6 * (size_t)N + sj[k]] * kInv4PiT / NF;
          for (int c = 0; c < 2; ++c) part[((size_t)slot * 2 + c) * N + sj[k]] = wA * S[k][c];
        }
  }
}

template <class T, int NF, bool FLOOR>
__global__ __launch_bounds__(64) void k_p2pT_tasks(int ntask, const int *__restrict__ tasks,
                                                   const int *__restrict__ range,
                                                   const int *__restrict__ subs,
                                                   const T *__restrict__ src,
                                                   const T *__restrict__ tgt,
                                                   const double *__restrict__ z,
                                                   const double *__restrict__ geo, int N,
                                                   T kappa, double eps_ratio,
                                                   double *__restrict__ part) {
  __shared__ __align__(16) T sh[64 * 8];
  __shared__ double etab[sizeof(T) == 8 ? 64 : 1];
  const Screen<T> sc = make_screen(kappa, etab);
  const int task = xcd_task(ntask);
  if (task < 0) return;
  const int B = tasks[4 * task], lb = tasks[4 * task + 1], le = tasks[4 * task + 2];
  const int slot = tasks[4 * task + 3];
  const int s0 = range[2 * B], s1 = range[2 * B + 1];
  // up to three panels per lane (two, three, four: 452, 368, 365 us in FP64 and
  // 195, 156, 162 us in FP32 on 30420 panels: lane fill against registers)
  constexpr int kMax = 3;
  const LaneSplit ls = lane_split(s1 - s0, kMax);
#define PBMP_BODY(K)                                                                           \
  p2pT_body<T, NF, K, FLOOR>(src, tgt, z, geo, N, s0, s1, subs, lb, le, sc, eps_ratio, slot, part, \
                             sh, ls.G, ls.L)
  switch (ls.tpt) {
    case 1: PBMP_BODY(1); break;
    case 2: PBMP_BODY(2); break;
    default: PBMP_BODY(kMax); break;
  }
#undef PBMP_BODY
}

// M2P^T: per task (box B, target sub-ranges) the partial local coefficients
// in harmonic form (FAM 0 Laplace with z1, 1 Yukawa with z2, 2 both at once:
// the FP64 words of both do not leave registers for the rest).
template <class T, int P, int FAM>
__global__ __launch_bounds__(64) void k_m2pT_tasks(int ntask, const int *__restrict__ tasks,
                                                   const int *__restrict__ subs,
                                                   const double *__restrict__ center,
                                                   const T *__restrict__ tgt,
                                                   const double *__restrict__ z, int N,
                                                   T kappa, T nk, double *__restrict__ Lpart) {
  constexpr int NS = Orders<P>::NS;
  constexpr int NA = FAM == 2 ? NS : (NS / 2 + 3) / 4 * 4;
  const int task = xcd_task(ntask);
  if (task < 0) return;
  const int B = tasks[4 * task], lb = tasks[4 * task + 1], le = tasks[4 * task + 2];
  const T c[3] = {(T)center[3 * B], (T)center[3 * B + 1], (T)center[3 * B + 2]};
  T acc[NA];
#pragma unroll
  for (int k = 0; k < NA; ++k) acc[k] = T(0);
  for (int l = lb; l < le; ++l) {
    const int a0 = subs[2 * l], a1 = subs[2 * l + 1];
    for (int t = a0 + (int)threadIdx.x; t < a1; t += 64) {
      const T D[3] = {tgt[t] - c[0], tgt[N + t] - c[1], tgt[2 * N + t] - c[2]};
      const T R2 = D[0] * D[0] + D[1] * D[1] + D[2] * D[2];
      const T ri = rsqrt_t<T>(R2);
      const T ek = FAM == 0 ? T(0) : expneg_t<T>(nk, kappa, R2 * ri);
      harmonic_m2p_T<T, P + 1, FAM>(D, ri, ek, kappa, (T)z[t], (T)z[N + t], acc);
    }
  }
  double *out = Lpart + (size_t)task * NS;
  wave_sums(acc, [&](int k, double v) {
    const int pos = FAM == 2 ? k : 2 * k + FAM;
    if (pos < NS) out[pos] = v;
  });
}

// L_B, Cartesian [Laplace | Yukawa], from the partials of B's tasks (four
// interleaved runs of them, added in order; through the transposed map of
// harmonic_words); zero without tasks
template <int P>
__global__ __launch_bounds__(512) void k_l_reduce(const int *__restrict__ count,
                                                  const int *__restrict__ off,
                                                  const double *__restrict__ Lpart,
                                                  const int *__restrict__ koff,
                                                  const int *__restrict__ kpos,
                                                  const double *__restrict__ kc,
                                                  double *__restrict__ Lb) {
  constexpr int NK = Orders<P>::NK, NS = Orders<P>::NS;
  static_assert(NS <= 128, "a lane per word");
  __shared__ double run[4][NS];
  __shared__ double h[NS];
  const int B = blockIdx.x, t0 = off[B], nt = count[2 * B + 1];
  const int e = (int)threadIdx.x & 127, r = (int)threadIdx.x >> 7;
  if (e < NS) {
    double v = 0.0;
#pragma unroll 4
    for (int t = t0 + r; t < t0 + nt; t += 4) v += Lpart[(size_t)t * NS + e];
    run[r][e] = v;
  }
  __syncthreads();
  if (r == 0 && e < NS) h[e] = run[0][e] + run[1][e] + run[2][e] + run[3][e];
  __syncthreads();
  for (int k = threadIdx.x; k < NK; k += 512) {
    double a = 0.0, b = 0.0;
    for (int q = koff[k]; q < koff[k + 1]; ++q) {
      a += kc[2 * q] * h[kpos[q]];
      b += kc[2 * q + 1] * h[kpos[q] + 1];
    }
    Lb[(size_t)B * 2 * NK + k] = a;
    Lb[(size_t)B * 2 * NK + NK + k] = b;
  }
}

// local coefficients of every box for the weights z, in T
template <class T, int P>
void launch_locals(Tree &t, hipStream_t s, const T *tgt, const double *z, int N, T kappa, T nk) {
  constexpr int NK = Orders<P>::NK, NS = Orders<P>::NS;
  t.d_Lpart.reserve((size_t)std::max(1, t.n_m2pT_tasks) * NS);
  t.d_L.reserve((size_t)t.nbox * 2 * NK);
  if (t.n_m2pT_tasks > 0) {
    const dim3 grid(((t.n_m2pT_tasks + 7) / 8) * 8);
#define PBMP_ML(FAM)                                                                         \
  hipLaunchKernelGGL((k_m2pT_tasks<T, P, FAM>), grid, dim3(64), 0, s, t.n_m2pT_tasks,        \
                     t.d_m2pT_task.p, t.d_m2pT_sub.p, t.d_center.p, tgt, z, N, kappa, nk, \
                     t.d_Lpart.p)
    if constexpr (sizeof(T) == 4) {
      PBMP_ML(2);
    } else {
      PBMP_ML(0);
      PBMP_ML(1);
    }
#undef PBMP_ML
  }
  hipLaunchKernelGGL(k_l_reduce<P>, dim3(t.nbox), dim3(512), 0, s, t.d_m2pT_count.p,
                     t.d_m2pT_off.p, t.d_Lpart.p, t.d_koff.p, t.d_kpos.p, t.d_kc.p, t.d_L.p);
}

// L2P at the leaves: every node takes the local expansions of all boxes
// on its leaf's path to the root, each about its own centre (the direct
// counterpart of shifting them down level by level), lanes over the leaf's
// panels and a wave per node, FP64 (latency bound: one wave for all nodes took
// 31 us on 30420 panels).  Boxes that no leaf accepted carry zero coefficients
// and are skipped.
constexpr int kMaxChain = 24;

template <int P, int NF>
__global__ __launch_bounds__(64 * NF) void k_l2p(const int *__restrict__ leaves,
                                            const int *__restrict__ range,
                                            const int *__restrict__ parent,
                                            const int *__restrict__ ntask,
                                            const double *__restrict__ center,
                                            const double *__restrict__ Lb,
                                            const double *__restrict__ src64,
                                            const double *__restrict__ geo,
                                            const int *__restrict__ tslotsT, int N,
                                            double eps_ratio, double *__restrict__ part) {
  constexpr Multi<P> mi{};
  constexpr Multi<P + 1> miK{};
  constexpr int NC = Orders<P>::NV, NK = Orders<P>::NK;
  __shared__ double lp[kMaxChain][2 * NK];
  __shared__ double lc[kMaxChain][3];
  __shared__ int chain[kMaxChain];
  __shared__ int nchain;
  __shared__ double red[NF][64][2];
  const int B = leaves[blockIdx.x];
  if (threadIdx.x == 0) {
    int n = 0;
    for (int a = B; a >= 0 && n < kMaxChain; a = parent[a])
      if (ntask[2 * a + 1] > 0) chain[n++] = a;
    nchain = n;
  }
  __syncthreads();
  const int nc = nchain;
  for (int e = threadIdx.x; e < nc * 2 * NK; e += 64 * NF) {
    const int a = e / (2 * NK), k = e % (2 * NK);
    // the two sums a node takes: K_L - K_Y and eps V_Y - V_L
    const double *Lc = Lb + (size_t)chain[a] * 2 * NK;
    lp[a][k] = k < NK ? Lc[k] - Lc[NK + k] : eps_ratio * Lc[k] - Lc[k - NK];
  }
  for (int e = threadIdx.x; e < nc * 3; e += 64 * NF) lc[e / 3][e % 3] = center[3 * chain[e / 3] + e % 3];
  __syncthreads();
  const int lane = (int)threadIdx.x & 63, q = (int)threadIdx.x >> 6;
  for (int jb = range[2 * B]; jb < range[2 * B + 1]; jb += 64) {
    const int j = jb + lane;
    double out[2] = {0.0, 0.0};
    if (j < range[2 * B + 1]) {
      const double *r = src64 + 16 * (size_t)j;
      const double n[3] = {r[9], r[10], r[11]};
      const double y[3] = {r[3 * q], r[3 * q + 1], r[3 * q + 2]};
      for (int a = 0; a < nc; ++a) {
        const double h[3] = {y[0] - lc[a][0], y[1] - lc[a][1], y[2] - lc[a][2]};
        double mono[NC];
        mono[0] = 1.0;
#pragma unroll
        for (int k = 1; k < NC; ++k) {
          const int d = mi.e[k][0] ? 0 : (mi.e[k][1] ? 1 : 2);
          mono[k] = mono[mi.m1[k][d]] * h[d];
        }
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          double dn = 0.0;
#pragma unroll
          for (int d = 0; d < 3; ++d)
            if (miK.m1[k][d] >= 0) dn += miK.e[k][d] * n[d] * mono[miK.m1[k][d]];
          if (k < NC) out[1] += lp[a][NK + k] * mono[k];
          out[0] += lp[a][k] * dn;
        }
      }
    }
    __syncthreads();
    for (int c = 0; c < 2; ++c) red[q][lane][c] = out[c];
    __syncthreads();
    if (q == 0 && j < range[2 * B + 1]) {
      const double wA = geo[6 * (size_t)N + j] * kInv4PiT / NF;
      const int slot = tslotsT[j] - 1;
      for (int c = 0; c < 2; ++c) {
        double v = red[0][lane][c];
        for (int w = 1; w < NF; ++w) v += red[w][lane][c];
        part[((size_t)slot * 2 + c) * N + j] = wA * v;
      }
    }
  }
}

// (A^T z) from the transposed partial slots, the transposed near/self
// correction and the identity terms; lanes per row as in k_finish_slots
__global__ __launch_bounds__(kFinBlock) void k_finish_T_slots(
    int N, const int *__restrict__ tslotsT, const double *__restrict__ part,
    const int *__restrict__ trow, const int *__restrict__ tcol, const int *__restrict__ tent,
    const double *__restrict__ val, const double *__restrict__ z, double eps_ratio,
    const int *__restrict__ perm, double *__restrict__ y) {
  const int t = blockIdx.x * kFinBlock + (int)threadIdx.x;
  const int j = t / kFinLanes, u = t % kFinLanes;
  const int jl = min(j, N - 1);
  double S[2] = {0.0, 0.0};
  const int ns = tslotsT[jl];
  for (int c = u; c < ns; c += kFinLanes)
#pragma unroll
    for (int k = 0; k < 2; ++k) S[k] += part[((size_t)c * 2 + k) * N + jl];
  const int e1 = trow[jl + 1];
  for (int e = trow[jl] + u; e < e1; e += kFinLanes) {
    const int i = tcol[e];
    const double *v = val + 4 * (size_t)tent[e];
    const double z1 = z[i], z2 = z[N + i];
    S[0] += v[1] * z1 - v[3] * z2;
    S[1] += eps_ratio * v[2] * z2 - v[0] * z1;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    S[k] += __shfl_xor(S[k], 1, kFinLanes);
    S[k] += __shfl_xor(S[k], 2, kFinLanes);
  }
  if (j >= N || u != 0) return;
  const int o = perm ? perm[j] : j;
  y[o] = 0.5 * z[j] + 0.5 * z[N + j] + S[0];
  y[N + o] = S[1];
}

template <class T, int P>
void tree_T_far(Tree &t, hipStream_t s, int nf, int N, const double *geo,
                const double *src64, const T *src, const T *tgt, const double *z, T kappa,
                T nk, double eps_ratio, double *part, bool floor_r2) {
  // P2P^T
  const int nbp = ((t.n_p2pT_tasks + 7) / 8) * 8;
#define PBMP_TPT(NFV, FL)                                                                 \
  hipLaunchKernelGGL((k_p2pT_tasks<T, NFV, FL>), dim3(nbp), dim3(64), 0, s, t.n_p2pT_tasks, \
                     t.d_p2pT_task.p, t.d_range.p, t.d_p2pT_sub.p, src, tgt, z, geo, N,     \
                     kappa, eps_ratio, part)
  if (nf == 3 && floor_r2) PBMP_TPT(3, true);
  else if (nf == 3) PBMP_TPT(3, false);
  else if (floor_r2) PBMP_TPT(1, true);
  else PBMP_TPT(1, false);
#undef PBMP_TPT
  // M2P^T with per-box sums, L2P at the leaves
  launch_locals<T, P>(t, s, tgt, z, N, kappa, nk);
  if (nf == 3)
    hipLaunchKernelGGL((k_l2p<P, 3>), dim3(t.nleaf), dim3(192), 0, s, t.d_leaves.p,
                       t.d_range.p, t.d_parent.p, t.d_m2pT_count.p, t.d_center.p, t.d_L.p,
                       src64, geo, t.d_tslotsT.p, N, eps_ratio, part);
  else
    hipLaunchKernelGGL((k_l2p<P, 1>), dim3(t.nleaf), dim3(64), 0, s, t.d_leaves.p,
                       t.d_range.p, t.d_parent.p, t.d_m2pT_count.p, t.d_center.p, t.d_L.p,
                       src64, geo, t.d_tslotsT.p, N, eps_ratio, part);
  PBMP_HIP(hipGetLastError());
}

template <class T>
void tree_T_far_p(Tree &t, hipStream_t s, int nf, int N, const double *geo,
                  const double *src64, const T *src, const T *tgt, const double *z, T kappa,
                  T nk, double eps_ratio, double *part, bool floor_r2) {
  switch (t.prm.order) {
#define PBMP_TF(P)                                                                          \
  case P:                                                                                   \
    tree_T_far<T, P>(t, s, nf, N, geo, src64, src, tgt, z, kappa, nk, eps_ratio, part, floor_r2); \
    break;
    PBMP_TF(1)
    PBMP_TF(2)
    PBMP_TF(3)
    PBMP_TF(4)
    PBMP_TF(5)
    PBMP_TF(6)
#undef PBMP_TF
    default: throw Error(PBMP_EARG, "treecode order must be 1..6");
  }
}


// ======================================================= mesh adjoint
// Far-field part of the gradient of lambda . A x with respect to the
// collocation points c_i (target side) and to the far nodes y_g, normals n_j
// and areas A_j (source side), with the same octree, lists and expansions
// as the treecode product, so that the vertex gradient costs what a
// product costs.  Per target i the form is
//   l1_i (S_KL - S_VL) + l2_i (eps S_VY - S_KY)
// (the strengths s_V, s_K of the forward solution packed in the records).
// Exact derivatives of the discrete treecode operator with the expansion
// centres held fixed: direct pairs through op_pair; an accepted box's
// expansion, differentiated in the target, d/dx_i a_k(x - c) =
// -(k_i + 1) a_{k + e_i} (coefficients to degree P + 2); in the sources, the
// local expansions L_k = sum_i lambda_i a_k(x_i - c) of every box on a
// leaf's path (as in the transposed product) differentiated in the node
// h = y - c: the node's share of the form is
//   s_K n.grad_h P_K(h) + s_V P_V(h),
//   P_K = sum_{|k|<=P+1} (L^L_k - L^Y_k) h^k,  P_V = sum_{|k|<=P} (eps L^Y_k - L^L_k) h^k,
// with gradients in h, in n and in the area (the strengths are linear in A).

// target side, direct pairs: per forward P2P task, g_i = d/dc_i of the form
// over the task's source panels; partial slots [slot][4][N] (components 0..2)
template <int NF>
__global__ __launch_bounds__(64) void k_p2p_grad_tasks(int ntask, const int *__restrict__ tasks,
                                                       const int *__restrict__ slots,
                                                       const int *__restrict__ ranges,
                                                       const double *__restrict__ src64,
                                                       const double *__restrict__ geo,
                                                       const double *__restrict__ lam, int N,
                                                       double kappa, double eps_ratio,
                                                       double *__restrict__ part) {
  constexpr int kTileG = 64;
  __shared__ __align__(16) double sh[kTileG * 16];
  __shared__ double etab[64];
  const Screen<double> sc = make_screen(kappa, etab);
  const int task = xcd_task(ntask);
  if (task < 0) return;
  const int t0 = tasks[4 * task], t1 = tasks[4 * task + 1];
  const int lb = tasks[4 * task + 2], le = tasks[4 * task + 3];
  const int slot = slots[task];
  const int lane = (int)threadIdx.x;
  for (int tb = t0; tb < t1; tb += 64) {
    const int t = tb + lane, tl = min(t, t1 - 1);
    const double c[3] = {geo[tl], geo[N + tl], geo[2 * N + tl]};
    const double l1 = lam[tl], l2 = eps_ratio * lam[N + tl], l2k = lam[N + tl];
    double g[3] = {0.0, 0.0, 0.0};
    for (int l = lb; l < le; ++l) {
      const int s0 = ranges[2 * l], s1 = ranges[2 * l + 1];
      for (int jt = s0; jt < s1; jt += kTileG) {
        const int nj = min(kTileG, s1 - jt);
        __syncthreads();
        stage_records<double, kTileG>(src64 + (size_t)jt * 16, sh, nj, lane);
        __syncthreads();
        for (int jj = 0; jj < nj; ++jj) {
          const double *r = sh + 16 * jj;
#pragma unroll
          for (int q = 0; q < NF; ++q) {
            const double R[3] = {c[0] - r[3 * q], c[1] - r[3 * q + 1], c[2] - r[3 * q + 2]};
            double gR[3], gn[3];
            op_pair(R, r + 9, sc, l1 * r[14], l1 * r[13], l2k * r[14], l2 * r[13], gR, gn);
            for (int d = 0; d < 3; ++d) g[d] += gR[d];
          }
        }
      }
    }
    if (t < t1)
      for (int d = 0; d < 3; ++d) part[((size_t)slot * 4 + d) * N + t] = g[d];
  }
}

// target side, expansions: per forward M2P task (FP64 moments),
// d/dx of sum_k a_k m_k = - sum_k (k_d + 1) a_{k + e_d} m_k
template <int P>
__global__ __launch_bounds__(64) void k_m2p_grad_tasks(int ntask, const int *__restrict__ tasks,
                                                       const int *__restrict__ slots,
                                                       const int *__restrict__ boxes,
                                                       const double *__restrict__ center,
                                                       const double *__restrict__ mom,
                                                       const double *__restrict__ geo,
                                                       const double *__restrict__ lam, int N,
                                                       double kappa, double eps_ratio,
                                                       double *__restrict__ part) {
  constexpr Multi<P + 2> mi{};
  constexpr int NC = Orders<P>::NV, NK = Orders<P>::NK, NM = Orders<P>::NM;
  constexpr int NG = Multi<P + 2>::n;
  __shared__ double smom[kM2PChunkBoxes * NM];
  __shared__ double scen[kM2PChunkBoxes * 3];
  __shared__ int sbox[kM2PChunkBoxes];
  const int task = xcd_task(ntask);
  if (task < 0) return;
  const int t0 = tasks[4 * task], t1 = tasks[4 * task + 1];
  const int lb = tasks[4 * task + 2], le = tasks[4 * task + 3];
  const int slot = slots[task];
  for (int tb = t0; tb < t1; tb += 64) {
    const int t = tb + (int)threadIdx.x, tl = min(t, t1 - 1);
    const double x[3] = {geo[tl], geo[N + tl], geo[2 * N + tl]};
    const double l1 = lam[tl], l2 = lam[N + tl];
    double g[3] = {0.0, 0.0, 0.0};
    for (int cb = lb; cb < le; cb += kM2PChunkBoxes) {
    const int nb = min(kM2PChunkBoxes, le - cb);
    __syncthreads();
    if (threadIdx.x < nb) sbox[threadIdx.x] = boxes[cb + threadIdx.x];
    __syncthreads();
    for (int e = threadIdx.x; e < nb * NM; e += 64)
      smom[e] = mom[(size_t)sbox[e / NM] * NM + e % NM];
    for (int e = threadIdx.x; e < nb * 3; e += 64) scen[e] = center[3 * sbox[e / 3] + e % 3];
    __syncthreads();
    for (int b = 0; b < nb; ++b) {
      const double D[3] = {x[0] - scen[3 * b], x[1] - scen[3 * b + 1], x[2] - scen[3 * b + 2]};
      const double R2 = D[0] * D[0] + D[1] * D[1] + D[2] * D[2];
      const double ri = rsqrt_fp64(R2), iR2 = ri * ri;
      const double ek = exp_fp64(-kappa * R2 * ri);
      double a[NG], ay[NG], by[NG];
      a[0] = ri;
      by[0] = ek;
      ay[0] = ek * ri;
#pragma unroll
      for (int k = 1; k < NG; ++k) {
        const int sd = mi.deg[k];
        double S1 = 0, S2 = 0, Y1 = 0, Y2 = 0, B1 = 0, B2 = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          if (mi.m1[k][d] >= 0) {
            S1 += D[d] * a[mi.m1[k][d]];
            Y1 += D[d] * ay[mi.m1[k][d]];
            B1 += D[d] * by[mi.m1[k][d]];
          }
          if (mi.m2[k][d] >= 0) {
            S2 += a[mi.m2[k][d]];
            Y2 += ay[mi.m2[k][d]];
            B2 += by[mi.m2[k][d]];
          }
        }
        const double c1 = double(2 * sd - 1) / sd, c2 = double(sd - 1) / sd, ks = kappa / sd;
        a[k] = (c1 * S1 - c2 * S2) * iR2;
        by[k] = ks * (Y1 - Y2);
        ay[k] = (c1 * Y1 - c2 * Y2 + ks * (B1 - B2)) * iR2;
      }
      const double *m = smom + b * NM;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double vl = 0, kl = 0, vy = 0, ky = 0;
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          const int kp = mi.p1[k][d];
          const double w = -double(mi.e[k][d] + 1);
          if (k < NC) {
            vl += w * a[kp] * m[k];
            vy += w * ay[kp] * m[k];
          }
          kl += w * a[kp] * m[NC + k];
          ky += w * ay[kp] * m[NC + k];
        }
        g[d] += l1 * (kl - vl) + l2 * (eps_ratio * vy - ky);
      }
    }
    }
    if (t < t1)
      for (int d = 0; d < 3; ++d) part[((size_t)slot * 4 + d) * N + t] = g[d];
  }
}

// gc_i = sum of the target's forward slots
__global__ void k_grad_slots_reduce(int N, int ncomp, int stride, const int *__restrict__ nslots,
                                    int extra, const double *__restrict__ part,
                                    double *__restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int ns = nslots[i] + extra;
  for (int c = 0; c < ncomp; ++c) {
    double v = 0.0;
    for (int sl = 0; sl < ns; ++sl) v += part[((size_t)sl * stride + c) * N + i];
    out[(size_t)ncomp * i + c] = v;
  }
}

// gy (3 per node), gn, gA of a panel = sum of its transposed slots
__global__ void k_grad_src_reduce(int N, const int *__restrict__ nslots,
                                  const double *__restrict__ part, double *__restrict__ gy,
                                  double *__restrict__ gn, double *__restrict__ gA) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  const int ns = nslots[j];
  double v[13];
  for (int c = 0; c < 13; ++c) v[c] = 0.0;
  for (int sl = 0; sl < ns; ++sl)
    for (int c = 0; c < 13; ++c) v[c] += part[((size_t)sl * 13 + c) * N + j];
  for (int c = 0; c < 9; ++c) gy[9 * (size_t)j + c] = v[c];
  for (int c = 0; c < 3; ++c) gn[3 * (size_t)j + c] = v[9 + c];
  gA[j] = v[12];
}

// source side, direct pairs: per P2P^T task (sources of one leaf on the
// lanes, the task's targets through LDS), per source panel the 13 values
// d/dy_q (3 per node), d/dn (3), d/dA (1); slots [slot][13][N]
constexpr int kGradT = 13;

template <int NF>
__global__ __launch_bounds__(64) void k_p2pT_grad_tasks(int ntask, const int *__restrict__ tasks,
                                                        const int *__restrict__ range,
                                                        const int *__restrict__ subs,
                                                        const double *__restrict__ src64,
                                                        const double *__restrict__ geo,
                                                        const double *__restrict__ lam, int N,
                                                        double kappa, double eps_ratio,
                                                        double *__restrict__ part) {
  __shared__ double sh[64 * 5];
  __shared__ double etab[64];
  const Screen<double> sc = make_screen(kappa, etab);
  const int task = xcd_task(ntask);
  if (task < 0) return;
  const int B = tasks[4 * task], lb = tasks[4 * task + 1], le = tasks[4 * task + 2];
  const int slot = tasks[4 * task + 3];
  const int s0 = range[2 * B], s1 = range[2 * B + 1];
  const int lane = (int)threadIdx.x;
  for (int sb = s0; sb < s1; sb += 64) {
    const int j = sb + lane, jl = min(j, s1 - 1);
    double rec[15];
    for (int c = 0; c < 15; ++c) rec[c] = src64[16 * (size_t)jl + c];
    double acc[kGradT];
    for (int c = 0; c < kGradT; ++c) acc[c] = 0.0;
    for (int l = lb; l < le; ++l) {
      const int a0 = subs[2 * l], a1 = subs[2 * l + 1];
      for (int it = a0; it < a1; it += 64) {
        const int nt = min(64, a1 - it);
        __syncthreads();
        if (lane < nt) {
          const int i = it + lane;
          sh[5 * lane] = geo[i];
          sh[5 * lane + 1] = geo[N + i];
          sh[5 * lane + 2] = geo[2 * N + i];
          sh[5 * lane + 3] = lam[i];
          sh[5 * lane + 4] = lam[N + i];
        }
        __syncthreads();
        for (int e = 0; e < nt; ++e) {
          const double *r = sh + 5 * e;
#pragma unroll
          for (int q = 0; q < NF; ++q) {
            const double R[3] = {r[0] - rec[3 * q], r[1] - rec[3 * q + 1], r[2] - rec[3 * q + 2]};
            double gR[3], gn[3];
            const double f = op_pair(R, rec + 9, sc, r[3] * rec[14], r[3] * rec[13],
                                     r[4] * rec[14], eps_ratio * r[4] * rec[13], gR, gn);
            for (int d = 0; d < 3; ++d) {
              acc[3 * q + d] -= gR[d];
              acc[9 + d] += gn[d];
            }
            acc[12] += f;
          }
        }
      }
    }
    if (j < s1) {
      const double iA = 1.0 / geo[6 * (size_t)N + j];
      acc[12] *= iA;
      for (int c = 0; c < kGradT; ++c) part[((size_t)slot * kGradT + c) * N + j] = acc[c];
    }
  }
}

// source side, expansions: at every node the local expansions of the
// boxes on its leaf's path to the root (FP64 L from the M2P^T kernels with
// z = lambda); slot tslotsT[j] - 1
template <int P, int NF>
__global__ __launch_bounds__(64) void k_l2p_grad(const int *__restrict__ leaves,
                                                 const int *__restrict__ range,
                                                 const int *__restrict__ parent,
                                                 const int *__restrict__ ntask,
                                                 const double *__restrict__ center,
                                                 const double *__restrict__ Lb,
                                                 const double *__restrict__ src64,
                                                 const double *__restrict__ geo,
                                                 const int *__restrict__ tslotsT, int N,
                                                 double eps_ratio, double *__restrict__ part) {
  constexpr Multi<P> mi{};
  constexpr Multi<P + 1> miK{};
  constexpr int NC = Orders<P>::NV, NK = Orders<P>::NK;
  __shared__ double lp[kMaxChain][2 * NK];
  __shared__ double lc[kMaxChain][3];
  __shared__ int chain[kMaxChain];
  __shared__ int nchain;
  const int B = leaves[blockIdx.x];
  if (threadIdx.x == 0) {
    int n = 0;
    for (int a = B; a >= 0 && n < kMaxChain; a = parent[a])
      if (ntask[2 * a + 1] > 0) chain[n++] = a;
    nchain = n;
  }
  __syncthreads();
  const int nc = nchain;
  for (int e = threadIdx.x; e < nc * 2 * NK; e += 64) {
    const int a = e / (2 * NK), k = e % (2 * NK);
    lp[a][k] = Lb[(size_t)chain[a] * 2 * NK + k];
  }
  for (int e = threadIdx.x; e < nc * 3; e += 64) lc[e / 3][e % 3] = center[3 * chain[e / 3] + e % 3];
  __syncthreads();
  for (int j = range[2 * B] + (int)threadIdx.x; j < range[2 * B + 1]; j += 64) {
    const double *r = src64 + 16 * (size_t)j;
    const double n[3] = {r[9], r[10], r[11]};
    const double sv = r[13], sk = r[14];
    double acc[kGradT];
    for (int c = 0; c < kGradT; ++c) acc[c] = 0.0;
    for (int a = 0; a < nc; ++a) {
      for (int q = 0; q < NF; ++q) {
        const double h[3] = {r[3 * q] - lc[a][0], r[3 * q + 1] - lc[a][1], r[3 * q + 2] - lc[a][2]};
        double mono[NC];
        mono[0] = 1.0;
#pragma unroll
        for (int k = 1; k < NC; ++k) {
          const int d = mi.e[k][0] ? 0 : (mi.e[k][1] ? 1 : 2);
          mono[k] = mono[mi.m1[k][d]] * h[d];
        }
        double pv = 0.0, gv[3] = {0, 0, 0}, gk[3] = {0, 0, 0};
        double hk[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          const double cK = lp[a][k] - lp[a][NK + k];
          if (k < NC) {
            const double cV = eps_ratio * lp[a][NK + k] - lp[a][k];
            pv += cV * mono[k];
#pragma unroll
            for (int d = 0; d < 3; ++d)
              if (mi.m1[k][d] >= 0) gv[d] += cV * mi.e[k][d] * mono[mi.m1[k][d]];
          }
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            const int k1 = miK.m1[k][d];
            if (k1 < 0) continue;
            gk[d] += cK * miK.e[k][d] * mono[k1];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
              const int k2 = miK.m1[k1][e];
              if (k2 < 0) continue;
              hk[d][e] += cK * miK.e[k][d] * miK.e[k1][e] * mono[k2];
            }
          }
        }
        const double qk = n[0] * gk[0] + n[1] * gk[1] + n[2] * gk[2];
        for (int e = 0; e < 3; ++e) {
          const double hn = n[0] * hk[0][e] + n[1] * hk[1][e] + n[2] * hk[2][e];
          acc[3 * q + e] += sk * hn + sv * gv[e];
          acc[9 + e] += sk * gk[e];
        }
        acc[12] += sk * qk + sv * pv;
      }
    }
    const double iA = 1.0 / geo[6 * (size_t)N + j];
    acc[12] *= iA;
    const int slot = tslotsT[j] - 1;
    for (int c = 0; c < kGradT; ++c) part[((size_t)slot * kGradT + c) * N + j] = acc[c];
  }
}

template <int P>
void tree_mesh_adjoint_far_p(Tree &t, hipStream_t s, int nf, int N, const double *geo,
                             const double *src64, const double *lam, double kappa,
                             double eps_ratio, double *part, double *partT, double *gc,
                             double *gy, double *gn, double *gA) {
  // the moments of the strengths that the records hold now: those in d_mom64 are
  // the last product's, whatever vector that was
  launch_moments_p<P>(t, s, nf, src64, true, eps_ratio);
  // target side: direct pairs and expansions into the forward slots
  const int nbp = ((t.n_p2p_tasks + 7) / 8) * 8;
  if (nf == 3)
    hipLaunchKernelGGL(k_p2p_grad_tasks<3>, dim3(nbp), dim3(64), 0, s, t.n_p2p_tasks,
                       t.d_p2p_task.p, t.d_p2p_slot.p, t.d_p2p_src.p, src64, geo, lam, N,
                       kappa, eps_ratio, part);
  else
    hipLaunchKernelGGL(k_p2p_grad_tasks<1>, dim3(nbp), dim3(64), 0, s, t.n_p2p_tasks,
                       t.d_p2p_task.p, t.d_p2p_slot.p, t.d_p2p_src.p, src64, geo, lam, N,
                       kappa, eps_ratio, part);
  if (t.n_m2p_tasks > 0 && t.n_m2p_entries > 0) {
    const int nbm = ((t.n_m2p_tasks + 7) / 8) * 8;
    hipLaunchKernelGGL((k_m2p_grad_tasks<P>), dim3(nbm), dim3(64), 0, s, t.n_m2p_tasks,
                       t.d_m2p_task.p, t.d_m2p_slot.p, t.d_m2p_box.p, t.d_center.p,
                       t.d_mom64.p, geo, lam, N, kappa, eps_ratio, part);
  }
  hipLaunchKernelGGL(k_grad_slots_reduce, dim3((N + 255) / 256), dim3(256), 0, s, N, 3, 4,
                     t.d_tslots.p, 0, part, gc);
  // source side: transposed direct pairs, local expansions at the nodes
  const int nbt = ((t.n_p2pT_tasks + 7) / 8) * 8;
  if (nf == 3)
    hipLaunchKernelGGL(k_p2pT_grad_tasks<3>, dim3(nbt), dim3(64), 0, s, t.n_p2pT_tasks,
                       t.d_p2pT_task.p, t.d_range.p, t.d_p2pT_sub.p, src64, geo, lam, N,
                       kappa, eps_ratio, partT);
  else
    hipLaunchKernelGGL(k_p2pT_grad_tasks<1>, dim3(nbt), dim3(64), 0, s, t.n_p2pT_tasks,
                       t.d_p2pT_task.p, t.d_range.p, t.d_p2pT_sub.p, src64, geo, lam, N,
                       kappa, eps_ratio, partT);
  launch_locals<double, P>(t, s, geo, lam, N, kappa, 0.0);
  if (nf == 3)
    hipLaunchKernelGGL((k_l2p_grad<P, 3>), dim3(t.nleaf), dim3(64), 0, s, t.d_leaves.p,
                       t.d_range.p, t.d_parent.p, t.d_m2pT_count.p, t.d_center.p, t.d_L.p,
                       src64, geo, t.d_tslotsT.p, N, eps_ratio, partT);
  else
    hipLaunchKernelGGL((k_l2p_grad<P, 1>), dim3(t.nleaf), dim3(64), 0, s, t.d_leaves.p,
                       t.d_range.p, t.d_parent.p, t.d_m2pT_count.p, t.d_center.p, t.d_L.p,
                       src64, geo, t.d_tslotsT.p, N, eps_ratio, partT);
  hipLaunchKernelGGL(k_grad_src_reduce, dim3((N + 255) / 256), dim3(256), 0, s, N,
                     t.d_tslotsT.p, partT, gy, gn, gA);
  PBMP_HIP(hipGetLastError());
}

}  // namespace

void tree_upload_exponents(Tree &t, hipStream_t s) {
  std::vector<int> ex;
  for (int d = 0; d <= t.prm.order + 1; ++d)
    for (int i = d; i >= 0; --i)
      for (int j = d - i; j >= 0; --j) ex.insert(ex.end(), {i, j, d - i - j});
  t.d_monos.upload(ex.data(), ex.size(), s);
  // shift terms per coefficient k: (j, k - j, C(k, j)) for every j <= k
  auto index = [](int i, int j, int l) {
    const int d = i + j + l;
    return d * (d + 1) * (d + 2) / 6 + (d - i) * (d - i + 1) / 2 + (d - i - j);
  };
  auto binom = [](int n, int r) {
    double c = 1.0;
    for (int u = 1; u <= r; ++u) c = c * (n - r + u) / u;
    return c;
  };
  const int nc = (int)ex.size() / 3;
  std::vector<int> off(nc + 1, 0);
  std::vector<unsigned> term;  // j | (k - j) << 8 | C(k, j) << 16 (at most 119, 119, 35)
  for (int k = 0; k < nc; ++k) {
    const int kx = ex[3 * k], ky = ex[3 * k + 1], kz = ex[3 * k + 2];
    for (int jx = 0; jx <= kx; ++jx)
      for (int jy = 0; jy <= ky; ++jy)
        for (int jz = 0; jz <= kz; ++jz) {
          const double c = binom(kx, jx) * binom(ky, jy) * binom(kz, jz);
          term.push_back((unsigned)index(jx, jy, jz) |
                         (unsigned)index(kx - jx, ky - jy, kz - jz) << 8 |
                         (unsigned)std::lround(c) << 16);
        }
    off[k + 1] = (int)term.size();
  }
  t.d_shift_toff.upload(off.data(), off.size(), s);
  t.d_shift_term.upload(term.data(), term.size(), s);
  PBMP_HIP(hipStreamSynchronize(s));
}

// Tables of the harmonic form of order P (harmonic.hpp) for degrees up to
// L = P + 1: per harmonic its terms over the Cartesian indices, and per
// Cartesian index its terms over the harmonics' word positions (the
// transposed map of the local coefficients), each with the Laplace and the
// Yukawa constant.  The split of the degree-n monomials into |xi|^{2j} times
// harmonics is the inverse of the matrix whose columns are those products'
// monomial coefficients (at most 36 x 36, extended precision).
template <int L> static void harmonic_positions(std::vector<int> &pos) {
  for (int l = 0; l <= L; ++l)
    for (int m = -l; m <= l; ++m)
      pos.push_back(m == 0  ? Harm<L>::pole(l)
                    : m > 0 ? Harm<L>::group(l, m)
                            : Harm<L>::group(l, -m) + 2);
}

void tree_upload_harmonics(Tree &t, hipStream_t s) {
  using ld = long double;
  const double kappa = t.prm.kappa;
  const int L = t.prm.order + 1, D = L + 1;
  auto at = [&](int i, int j, int k) { return (i * D + j) * D + k; };
  using Poly = std::vector<ld>;
  auto zero = [&] { return Poly((size_t)D * D * D, 0.0L); };
  auto mul = [&](const Poly &a, int i, int j, int k, ld c, Poly &out) {  // out += c x^i y^j z^k a
    for (int x = 0; x + i < D; ++x)
      for (int y = 0; y + j < D; ++y)
        for (int z = 0; z + k < D; ++z)
          if (a[at(x, y, z)] != 0.0L) out[at(x + i, y + j, z + k)] += c * a[at(x, y, z)];
  };
  auto r2 = [&](const Poly &a, ld c, Poly &out) {
    mul(a, 2, 0, 0, c, out);
    mul(a, 0, 2, 0, c, out);
    mul(a, 0, 0, 2, c, out);
  };
  // harm[l][m + l]: the harmonic polynomials, m < 0 the sines
  std::vector<std::vector<Poly>> harm(L + 1);
  for (int l = 0; l <= L; ++l) harm[l].resize(2 * l + 1);
  Poly c = zero(), sn = zero();
  c[at(0, 0, 0)] = 1.0L;
  for (int m = 0; m <= L; ++m) {
    if (m > 0) {
      Poly nc = zero(), ns = zero();
      mul(c, 1, 0, 0, 1.0L, nc);
      mul(sn, 0, 1, 0, -1.0L, nc);
      mul(sn, 1, 0, 0, 1.0L, ns);
      mul(c, 0, 1, 0, 1.0L, ns);
      c = nc;
      sn = ns;
    }
    for (int sg = 0; sg < (m ? 2 : 1); ++sg) {
      Poly p0 = zero(), p1 = sg ? sn : c;
      harm[m][sg ? 0 : 2 * m] = p1;
      for (int l = m; l < L; ++l) {
        Poly p2 = zero();
        mul(p1, 0, 0, 1, 1.0L, p2);
        r2(p0, -(ld)(l * l - m * m) / (ld)(4 * l * l - 1), p2);
        harm[l + 1][l + 1 + (sg ? -m : m)] = p2;
        p0 = p1;
        p1 = p2;
      }
    }
  }
  std::vector<std::vector<int>> ex;  // Cartesian indices in storage order
  std::vector<int> first(L + 2, 0);
  for (int n = 0; n <= L; ++n) {
    for (int i = n; i >= 0; --i)
      for (int j = n - i; j >= 0; --j) ex.push_back({i, j, n - i - j});
    first[n + 1] = (int)ex.size();
  }
  auto fact = [](int n) {
    ld f = 1.0L;
    for (int i = 2; i <= n; ++i) f *= i;
    return f;
  };
  const int NH = (L + 1) * (L + 1), NK = (int)ex.size();
  std::vector<std::vector<int>> hk(NH), kh(NK);
  std::vector<std::vector<double>> hc(NH), kc(NK);
  for (int n = 0; n <= L; ++n) {
    const int n0 = first[n], dim = first[n + 1] - n0;
    struct Col {
      int l, m, j;
    };
    std::vector<Col> cols;
    std::vector<ld> A((size_t)dim * 2 * dim, 0.0L);  // [products | identity]
    for (int j = 0; 2 * j <= n; ++j) {
      const int l = n - 2 * j;
      for (int m = -l; m <= l; ++m) {
        Poly p = harm[l][m + l];
        for (int u = 0; u < j; ++u) {
          Poly q = zero();
          r2(p, 1.0L, q);
          p = q;
        }
        for (int k = 0; k < dim; ++k) {
          const auto &e = ex[n0 + k];
          A[(size_t)k * 2 * dim + cols.size()] = p[at(e[0], e[1], e[2])];
        }
        cols.push_back({l, m, j});
      }
    }
    for (int k = 0; k < dim; ++k) A[(size_t)k * 2 * dim + dim + k] = 1.0L;
    for (int k = 0; k < dim; ++k) {  // Gauss-Jordan with row pivoting
      int piv = k;
      for (int r = k + 1; r < dim; ++r)
        if (std::fabs(A[(size_t)r * 2 * dim + k]) > std::fabs(A[(size_t)piv * 2 * dim + k])) piv = r;
      for (int q = 0; q < 2 * dim; ++q)
        std::swap(A[(size_t)k * 2 * dim + q], A[(size_t)piv * 2 * dim + q]);
      const ld inv = 1.0L / A[(size_t)k * 2 * dim + k];
      for (int q = 0; q < 2 * dim; ++q) A[(size_t)k * 2 * dim + q] *= inv;
      for (int r = 0; r < dim; ++r) {
        const ld f = A[(size_t)r * 2 * dim + k];
        if (r == k || f == 0.0L) continue;
        for (int q = 0; q < 2 * dim; ++q)
          A[(size_t)r * 2 * dim + q] -= f * A[(size_t)k * 2 * dim + q];
      }
    }
    for (int q = 0; q < dim; ++q) {
      const Col &cq = cols[q];
      ld dfact = 1.0L;  // (2l - 1)!!
      for (int u = 2 * cq.l - 1; u > 1; u -= 2) dfact *= u;
      const ld kap = std::pow((ld)kappa, 2 * cq.j);
      for (int k = 0; k < dim; ++k) {
        const ld v = A[(size_t)q * 2 * dim + dim + k];
        if (std::fabs(v) < 1e-12L) continue;  // the true ones are simple fractions
        const auto &e = ex[n0 + k];
        const ld w = v * dfact / (fact(e[0]) * fact(e[1]) * fact(e[2]));
        const int h = cq.l * cq.l + cq.m + cq.l;
        const double cl = cq.j == 0 ? (double)w : 0.0, cy = (double)(w * kap);
        if (cl == 0.0 && cy == 0.0) continue;
        hk[h].push_back(n0 + k);
        hc[h].insert(hc[h].end(), {cl, cy});
        kh[n0 + k].push_back(h);
        kc[n0 + k].insert(kc[n0 + k].end(), {cl, cy});
      }
    }
  }
  std::vector<int> pos;
  switch (L) {
    case 2: harmonic_positions<2>(pos); break;
    case 3: harmonic_positions<3>(pos); break;
    case 4: harmonic_positions<4>(pos); break;
    case 5: harmonic_positions<5>(pos); break;
    case 6: harmonic_positions<6>(pos); break;
    case 7: harmonic_positions<7>(pos); break;
    default: throw Error(PBMP_EARG, "treecode order must be 1..6");
  }
  auto flat = [&](const std::vector<std::vector<int>> &ix,
                  const std::vector<std::vector<double>> &co, bool to_pos, Dbuf<int> &off,
                  Dbuf<int> &idx, Dbuf<double> &coef) {
    std::vector<int> o(1, 0), f;
    std::vector<double> v;
    for (size_t a = 0; a < ix.size(); ++a) {
      for (int b : ix[a]) f.push_back(to_pos ? pos[b] : b);
      v.insert(v.end(), co[a].begin(), co[a].end());
      o.push_back((int)f.size());
    }
    off.upload(o.data(), o.size(), s);
    idx.upload(f.data(), f.size(), s);
    coef.upload(v.data(), v.size(), s);
    PBMP_HIP(hipStreamSynchronize(s));
  };
  flat(hk, hc, false, t.d_hoff, t.d_hk, t.d_hc);
  flat(kh, kc, true, t.d_koff, t.d_kpos, t.d_kc);
  t.d_hpos.upload(pos.data(), pos.size(), s);
  const size_t words = 4 * (size_t)(L * (L + 1) / 2 + (L + 2) / 2);
  t.d_harm64.alloc((size_t)t.nbox * words);
  t.d_harm32.alloc((size_t)t.nbox * words);
  PBMP_HIP(hipMemsetAsync(t.d_harm64.p, 0, sizeof(double) * t.nbox * words, s));
  PBMP_HIP(hipMemsetAsync(t.d_harm32.p, 0, sizeof(float) * t.nbox * words, s));
  PBMP_HIP(hipStreamSynchronize(s));
}

void tree_apply(Tree &t, hipStream_t s, bool fp64, int nf, int N, const double *geo,
                const double *src64, const float *src32, const float *tgt32,
                double eps_ratio, double *part, KernelClock &clk, bool floor_r2) {
  const double kappa = t.prm.kappa;
  // The harmonic form holds kappa^2j (words) and kappa^l (radial factors) apart
  // from e^{-kappa r}, which vanishes long before their product's kappa^(P+1)
  // leaves the FP32 range; infinity times that zero would be NaN.  Beyond 1e10
  // (kappa of 27 at P 6, 100 at P 4, above any electrolyte's 3 per A) the
  // expansions are evaluated in FP64, where kappa <= kMaxKappa keeps them finite:
  // a test of e^{-kappa r} per pair took the product of 144500 panels in mixed
  // precision from 905 to 914 us.
  const bool m2p64 = fp64 || std::pow(kappa, t.prm.order + 1) > 1e10;
  hipEvent_t e0 = clk.on ? clk.begin(s) : nullptr;
  launch_moments(t, s, nf, src64, m2p64, eps_ratio);
  PBMP_HIP(hipGetLastError());
  if (clk.on) clk.end(s, e0, KernelClock::P2M, 0.0);

  e0 = clk.on ? clk.begin(s) : nullptr;
  const int nbp = ((t.n_p2p_tasks + 7) / 8) * 8;
#define PBMP_TP(TT, NFV, FL, SRC, TGT)                                                   \
  hipLaunchKernelGGL((k_p2p_tasks<TT, NFV, FL>), dim3(nbp), dim3(64), 0, s, t.n_p2p_tasks, \
                     t.d_p2p_task.p, t.d_p2p_slot.p, t.d_p2p_src.p, SRC, TGT, N,           \
                     kap, part)
#define PBMP_TPR(TT, SRC, TGT)                            \
  if (nf == 3 && floor_r2) PBMP_TP(TT, 3, true, SRC, TGT); \
  else if (nf == 3) PBMP_TP(TT, 3, false, SRC, TGT);       \
  else if (floor_r2) PBMP_TP(TT, 1, true, SRC, TGT);       \
  else PBMP_TP(TT, 1, false, SRC, TGT)
  if (fp64) {
    const double kap = kappa;
    PBMP_TPR(double, src64, geo);
  } else {
    const float kap = kappa32(kappa);
    PBMP_TPR(float, src32, tgt32);
  }
#undef PBMP_TPR
#undef PBMP_TP
  PBMP_HIP(hipGetLastError());
  if (clk.on) clk.end(s, e0, KernelClock::P2P, t.direct_pairs);

  if (t.n_m2p_tasks > 0 && t.n_m2p_entries > 0) {
    e0 = clk.on ? clk.begin(s) : nullptr;
    if (m2p64)
      launch_m2p<double>(t, s, t.d_harm64.p, geo, N, kappa, 0.0, part);
    else
      launch_m2p<float>(t, s, t.d_harm32.p, tgt32, N, (float)kappa,
                        (float)(-kappa * 1.4426950408889634), part);
    PBMP_HIP(hipGetLastError());
    if (clk.on) clk.end(s, e0, KernelClock::M2P, t.m2p_pairs);
  }
}

void launch_finish_slots(hipStream_t s, int N, const int *tslots, const double *part,
                         const int *rowptr, const int *col, const double *val,
                         const double *x, double eps_ratio, const int *perm, double *y) {
  const int rows_per_block = kFinBlock / kFinLanes;
  hipLaunchKernelGGL(k_finish_slots, dim3((N + rows_per_block - 1) / rows_per_block),
                     dim3(kFinBlock), 0, s, N, tslots, part, rowptr, col, val, x, eps_ratio, perm, y);
  PBMP_HIP(hipGetLastError());
}

void tree_mesh_adjoint_far(Tree &t, hipStream_t s, int nf, int N, const double *geo,
                           const double *src64, const double *lam, double eps_ratio,
                           double *part, double *partT, double *gc, double *gy, double *gn,
                           double *gA) {
  const double kappa = t.prm.kappa;
  switch (t.prm.order) {
#define PBMP_MA(P)                                                                          \
  case P:                                                                                   \
    tree_mesh_adjoint_far_p<P>(t, s, nf, N, geo, src64, lam, kappa, eps_ratio, part, partT, \
                               gc, gy, gn, gA);                                             \
    break;
    PBMP_MA(1)
    PBMP_MA(2)
    PBMP_MA(3)
    PBMP_MA(4)
    PBMP_MA(5)
    PBMP_MA(6)
#undef PBMP_MA
    default: throw Error(PBMP_EARG, "treecode order must be 1..6");
  }
}

void tree_apply_transpose(Tree &t, hipStream_t s, bool fp64, int nf, int N, const double *geo,
                          const double *src64, const float *src32, const float *tgt32,
                          const double *z, double *part, const int *trow, const int *tcol,
                          const int *tent, const double *val, double eps_ratio,
                          const int *perm, double *y, bool floor_r2) {
  const double kappa = t.prm.kappa;
  if (fp64)
    tree_T_far_p<double>(t, s, nf, N, geo, src64, src64, geo, z, kappa, 0.0, eps_ratio, part,
                         floor_r2);
  else
    // (the transposed radial factors start from e^{-kappa r}: kappa^2 finite is enough)
    tree_T_far_p<float>(t, s, nf, N, geo, src64, src32, tgt32, z, kappa32(kappa),
                        (float)(-kappa * 1.4426950408889634), eps_ratio, part, floor_r2);
  const int rows = kFinBlock / kFinLanes;
  hipLaunchKernelGGL(k_finish_T_slots, dim3((N + rows - 1) / rows), dim3(kFinBlock), 0, s, N,
                     t.d_tslotsT.p, part, trow, tcol, tent, val, z, eps_ratio, perm, y);
  PBMP_HIP(hipGetLastError());
}

}  // namespace pbmp
