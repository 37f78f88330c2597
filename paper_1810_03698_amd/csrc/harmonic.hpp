// Solid-harmonic form of the truncated Cartesian Taylor series of the
// treecode, the same polynomial regrouped (no further approximation).
//
// A box's series is sum_k a_k(D) m_k with a_k = (-1)^|k| / k! d^k G(D), D =
// target - centre.  A monomial xi^k splits into sum_j |xi|^{2j} H(xi) with
// harmonic H of degree l = |k| - 2j; applied to G as a differential operator,
// |xi|^2 is the Laplacian, which multiplies G by kappa^2 (0 for 1/r), and
// H(d) f(r) = H(D) (1/r d/dr)^l f (Hobson).  Hence
//   sum_k a_k m_k = sum_l g_l(r) sum_m Y_lm(D/r) M_lm,
// (L + 1)^2 terms instead of C(L + 3, 3), with one set of harmonics for both
// kernels and the radial factors
//   Laplace g_l = r^-(l+1),
//   Yukawa  g_l = e^{-kappa r} / r tau_l,  tau_0 = 1, tau_1 = 1/r + kappa,
//           tau_{l+1} = tau_l / r + kappa^2 / (4 l^2 - 1) tau_{l-1}
// (the reverse Bessel polynomials), the constants (2l - 1)!! kappa^{2j}
// being part of M_lm = sum_k C_{lm,k} m_k.
//
// Harmonics: Y_lm = Q_lm(z) Re or Im (x + iy)^m with the monic Q: Q_mm = 1,
// Q_{l+1,m} = z Q_lm - (l^2 - m^2)/(4 l^2 - 1) Q_{l-1,m}.
//
// A box's words: groups of four (cosine: Laplace, Yukawa; sine: Laplace,
// Yukawa) for m >= 1, m outer, then pairs (Laplace, Yukawa) for m = 0.
#pragma once

#include <hip/hip_runtime.h>

namespace pbmp {

template <int L> struct Harm {
  static constexpr int NH = (L + 1) * (L + 1);
  static constexpr int NP = L * (L + 1) / 2;            // (l, m) with m >= 1
  static constexpr int S = 4 * (NP + (L + 2) / 2);      // words of a box
  static constexpr __host__ __device__ int group(int l, int m) {
    return 4 * ((m - 1) * (L + 1) - m * (m - 1) / 2 + (l - m));
  }
  static constexpr __host__ __device__ int pole(int l) { return 4 * NP + 2 * l; }
};

constexpr __host__ __device__ double harm_beta(int l, int m) {
  return double(l * l - m * m) / double(4 * l * l - 1);
}

// Adds one box's two rows (Laplace words to acc[k][0], Yukawa words to
// acc[k][1]) at TPT targets per lane: D from the box centre, M its words.
template <class T, int L, int TPT>
__device__ __forceinline__ void harmonic_m2p(const T *M, const T (&D)[TPT][3],
                                             const T (&ri)[TPT], const T (&ek)[TPT], T kappa,
                                             T (&acc)[TPT][2]) {
  using H = Harm<L>;
  typedef T v4 __attribute__((ext_vector_type(4), aligned(16)));
  T u[TPT][3], AL[TPT][L + 1], AY[TPT][L + 1];
#pragma unroll
  for (int k = 0; k < TPT; ++k)
    for (int d = 0; d < 3; ++d) u[k][d] = D[k][d] * ri[k];
  {
    T q0[TPT], q1[TPT];
#pragma unroll
    for (int l = 0; l <= L; ++l) {
      const T ml = M[H::pole(l)], my = M[H::pole(l) + 1];
#pragma unroll
      for (int k = 0; k < TPT; ++k) {
        T q = T(1);
        if (l == 1) q = u[k][2];
        if (l > 1) q = u[k][2] * q1[k] - T(harm_beta(l - 1, 0)) * q0[k];
        AL[k][l] = l == 0 ? ml : q * ml;
        AY[k][l] = l == 0 ? my : q * my;
        q0[k] = q1[k];
        q1[k] = q;
      }
    }
  }
  T cm[TPT], sm[TPT];
#pragma unroll
  for (int m = 1; m <= L; ++m) {
    T q0[TPT], q1[TPT];
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      const T c = m == 1 ? u[k][0] : u[k][0] * cm[k] - u[k][1] * sm[k];
      const T s = m == 1 ? u[k][1] : u[k][0] * sm[k] + u[k][1] * cm[k];
      cm[k] = c;
      sm[k] = s;
    }
#pragma unroll
    for (int l = m; l <= L; ++l) {
      const v4 w = *reinterpret_cast<const v4 *>(M + H::group(l, m));
#pragma unroll
      for (int k = 0; k < TPT; ++k) {
        T q = T(1);
        if (l == m + 1) q = u[k][2];
        if (l > m + 1) q = u[k][2] * q1[k] - T(harm_beta(l - 1, m)) * q0[k];
        const T yc = l == m ? cm[k] : q * cm[k];
        const T ys = l == m ? sm[k] : q * sm[k];
        AL[k][l] += yc * w[0] + ys * w[2];
        AY[k][l] += yc * w[1] + ys * w[3];
        q0[k] = q1[k];
        q1[k] = q;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    T sl = AL[k][L];
#pragma unroll
    for (int l = L - 1; l >= 0; --l) sl = sl * ri[k] + AL[k][l];
    acc[k][0] += ri[k] * sl;
    T t0 = T(1), t1 = ri[k] + kappa, sy = AY[k][0] + t1 * AY[k][1];
#pragma unroll
    for (int l = 1; l < L; ++l) {
      const T t2 = ri[k] * t1 + kappa * kappa * T(1.0 / (4 * l * l - 1)) * t0;
      sy += t2 * AY[k][l + 1];
      t0 = t1;
      t1 = t2;
    }
    acc[k][1] += ek[k] * ri[k] * sy;
  }
}

// Adds one target's weighted coefficients to a box's words (the transpose of
// harmonic_m2p): w1 times the Laplace coefficients, w2 times the Yukawa
// ones.  FAM: 0 Laplace words only, 1 Yukawa words only (acc[pos / 2]), 2
// both (acc[pos]).
template <class T, int L, int FAM, int N>
__device__ __forceinline__ void harmonic_m2p_T(const T (&D)[3], T ri, T ek, T kappa, T w1, T w2,
                                               T (&acc)[N]) {
  using H = Harm<L>;
  const T u[3] = {D[0] * ri, D[1] * ri, D[2] * ri};
  T gl[L + 1], gy[L + 1];
  if constexpr (FAM != 1) {
    gl[0] = w1 * ri;
#pragma unroll
    for (int l = 1; l <= L; ++l) gl[l] = gl[l - 1] * ri;
  }
  if constexpr (FAM != 0) {
    gy[0] = w2 * ek * ri;
    gy[1] = gy[0] * (ri + kappa);
#pragma unroll
    for (int l = 1; l < L; ++l)
      gy[l + 1] = ri * gy[l] + kappa * kappa * T(1.0 / (4 * l * l - 1)) * gy[l - 1];
  }
  auto add = [&](int pos, int l, T y) {
    if constexpr (FAM == 2) {
      acc[pos] += gl[l] * y;
      acc[pos + 1] += gy[l] * y;
    } else if constexpr (FAM == 0) {
      acc[pos / 2] += gl[l] * y;
    } else {
      acc[pos / 2] += gy[l] * y;
    }
  };
  T c = T(1), s = T(0);
#pragma unroll
  for (int m = 0; m <= L; ++m) {
    if (m == 1) {
      c = u[0];
      s = u[1];
    } else if (m > 1) {
      const T cc = u[0] * c - u[1] * s;
      s = u[0] * s + u[1] * c;
      c = cc;
    }
    T q0 = T(0), q1 = T(0);
#pragma unroll
    for (int l = m; l <= L; ++l) {
      T q = T(1);
      if (l == m + 1) q = u[2];
      if (l > m + 1) q = u[2] * q1 - T(harm_beta(l - 1, m)) * q0;
      if (m == 0) {
        add(H::pole(l), l, q);
      } else {
        add(H::group(l, m), l, l == m ? c : q * c);
        add(H::group(l, m) + 2, l, l == m ? s : q * s);
      }
      q0 = q1;
      q1 = q;
    }
  }
}

// Sums of N values (a multiple of four) over the 64 lanes, fixed order:
// lane 16 r of the wave ends with the sum of v[4 i + 2 (r & 1) + (r >> 1)] in
// v[i].  The first two steps fold two values into one (the lane-swap
// instructions exchange the halves that the other value keeps), so that only
// N / 4 values pass through the last four.
__device__ __forceinline__ double fold_swap32(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi =
      __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
         __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

__device__ __forceinline__ double fold_swap16(double a, double b) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi =
      __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
         __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

template <class T, int N, class F>
__device__ __forceinline__ void wave_sums(const T (&v)[N], F &&out) {
  static_assert(N % 4 == 0, "wave_sums takes a multiple of four values");
  const int lane = (int)threadIdx.x & 63, row = lane >> 4;
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    const double a = fold_swap32((double)v[i], (double)v[i + 1]);
    const double b = fold_swap32((double)v[i + 2], (double)v[i + 3]);
    double s = fold_swap16(a, b);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((lane & 15) == 0) out(i + 2 * (row & 1) + (row >> 1), s);
  }
}

}  // namespace pbmp
