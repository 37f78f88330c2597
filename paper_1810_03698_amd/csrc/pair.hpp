// Far-field pair terms of the four boundary-integral kernels, shared by the
// forward and transposed source-target products and by the near/self
// correction.  The correction takes 1/r and e^{-k r} from the same operation
// sequence as the product (no contraction), so that for tiny panels their
// rounding cancels instead of being amplified by 1/r^3.
#pragma once

#include <hip/hip_runtime.h>

namespace pbmp {

// FP32 cut-off on r^2 (r < 1e-4 A): such a pair adds nothing.  Pairs that
// close only occur between a panel and itself (the one-node rule puts the
// node on the centroid), a near neighbour, or a panel of another sheet in
// contact, and the near correction removes exactly the value the product added,
// so skipping them is exact; it keeps coincident FP32 points finite without
// 1/r-sized terms in FP32 sums.
constexpr float kMinR2f = 1e-8f;
// The FP64 products skip pairs closer than 1e-10 A: a one-node rule's node on
// its own panel's centroid (the node and the centroid are computed with
// different roundings, so they need not coincide exactly), or a node on a
// centroid of another sheet in contact; from every other centroid of its own
// sheet a node is at least a sixth of an altitude away.  A mesh where no node
// comes near either cut-off takes the kernels without the test (FLOOR false).
constexpr double kMinR2d = 1e-20;

// 1/sqrt(rr) in FP64: the hardware estimate y0 (1 - rr y0^2 = e, |e| < 2^-23
// measured over two binades) and one step of the binomial series
// y0 (1 + e/2 + 3 e^2/8), whose next term is below 2^-70; also r = sqrt(rr)
// from the same factors.  Two Newton steps took two more operations.  rr must
// be positive and normal.
__device__ __forceinline__ double rsqrt_fp64(double rr, double &r) {
  const double y = __builtin_amdgcn_rsq(rr);
  const double t = rr * y;
  const double e = fma(-t, y, 1.0);
  const double c = e * fma(0.375, e, 0.5);
  r = fma(t, c, t);
  return fma(y, c, y);
}

__device__ __forceinline__ double rsqrt_fp64(double rr) {
  double r;
  return rsqrt_fp64(rr, r);
}

// e^x in FP64 for x <= 0 (the screening factor e^{-kappa r}; no overflow
// or NaN handling).  Cody-Waite reduction x = n ln2 + f, |f| <= ln2/2, with
// ln2 split into a 32-bit head (n * head is exact for |n| < 2^21) and the
// rounded tail; e^f by its Taylor series to degree 13 (remainder below
// 0.35^14/14! < 5e-18) in Horner form; then scaled by 2^n (e^x below the
// smallest subnormal comes out as zero).
__device__ __forceinline__ double exp_fp64(double x) {
  constexpr double kLog2e = 1.4426950408889634;
  constexpr double kLn2Hi = 0x1.62e42ffp-1;
  constexpr double kLn2Lo = -0x1.718432a1b0e26p-35;
  const double n = rint(x * kLog2e);
  double f = fma(-n, kLn2Hi, x);
  f = fma(-n, kLn2Lo, f);
  constexpr double kFact[14] = {1.0, 1.0, 2.0, 6.0, 24.0, 120.0, 720.0, 5040.0, 40320.0,
                                362880.0, 3628800.0, 39916800.0, 479001600.0,
                                6227020800.0};
  double p = 1.0 / kFact[13];
#pragma unroll
  for (int k = 12; k >= 0; --k) p = fma(p, f, 1.0 / kFact[k]);
  return ldexp(p, (int)n);
}

// 2^(j/64), correctly rounded
__device__ const double kExp2Table[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0,
    0x1.0874518759bc8p+0, 0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0,
    0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0, 0x1.172b83c7d517bp+0,
    0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0,
    0x1.2d285a6e4030bp+0, 0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0,
    0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0, 0x1.3dea64c123422p+0,
    0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0,
    0x1.56f4736b527dap+0, 0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0,
    0x1.6247eb03a5585p+0, 0x1.6623882552225p+0, 0x1.6a09e667f3bcdp+0,
    0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0,
    0x1.868d99b4492edp+0, 0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0,
    0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0, 0x1.9c49182a3f090p+0,
    0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0,
    0x1.bcc1e904bc1d2p+0, 0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0,
    0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0, 0x1.d5818dcfba487p+0,
    0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0,
    0x1.fa7c1819e90d8p+0};

// Screening constants of the pair kernels.  FP64: e^{-kappa r} =
// 2^(n/64) 2^(f/64) with n + f = -64 kappa r / ln 2, |f| <= 1/2: 2^(n/64) from
// the 64-entry table (a copy in LDS, one gather) and a shift of the exponent,
// 2^(f/64) by its Taylor series to degree 5 (remainder below 4e-17), the
// table-driven method of P. T. P. Tang (ACM TOMS 15, 1989); 11
// operations where the series over |x| <= ln 2 / 2 to degree 13 takes 20.
// Results below the smallest subnormal come out as zero; WIDE bounds the
// argument for kappa r beyond the integers of the reduction (1e7).
template <class T> struct Screen;
template <> struct Screen<float> {
  float kappa, nk;  // nk = -kappa log2(e)
};
template <> struct Screen<double> {
  double kappa, c, far;  // c = -64 kappa / ln 2; e^{-kappa far} = 0
  const double *table;
  template <bool WIDE> __device__ __forceinline__ double exp(double r) const {
    if (WIDE) r = fmin(r, far);
    constexpr double kShift = 0x1.8p52;  // rounds to an integer in the low word
    const double t = fma(r, c, kShift);
    const double f = fma(r, c, kShift - t);
    const int n = (int)(uint32_t)__builtin_bit_cast(uint64_t, t);
    constexpr double b = 0.6931471805599453 / 64;
    double p = fma(f, b * b * b * b * b / 120, b * b * b * b / 24);
    p = fma(p, f, b * b * b / 6);
    p = fma(p, f, b * b / 2);
    p = fma(p, f, b);
    const double s = table[n & 63];
    return ldexp(fma(p * f, s, s), n >> 6);
  }
};

// one wave or more of a block fills the block's copy of the table; the caller
// synchronises before the first use
__device__ __forceinline__ Screen<double> make_screen(double kappa, double *lds_table) {
  if (threadIdx.x < 64) lds_table[threadIdx.x] = kExp2Table[threadIdx.x];
  return Screen<double>{kappa, kappa * -92.33248261689366, 1e5 / kappa, lds_table};
}
// kappa of the FP32 pairs, bounded where it is passed to the kernels (bounding it
// in them took the direct product of 19220 panels from 514 to 523 us): beyond
// 1e18 every e^{-kappa r} past the cut-off vanishes, and kappa / r stays finite
__host__ __device__ inline float kappa32(double kappa) {
  return (float)(kappa < 1e18 ? kappa : 1e18);
}
__device__ __forceinline__ Screen<float> make_screen(float kappa, double *) {
  Screen<float> sc{kappa, kappa * -1.44269504f};
  // kappa in a vector register: an FMA with a scalar operand issues at two
  // thirds of the rate (direct product of 19220 panels 570 -> 534 us)
  asm volatile("" : "+v"(sc.kappa));
  return sc;
}

// n.(p - y0): the nodes of a flat panel share its plane, so this is n.R
// for every node; taken from the difference vector (error eps |p - y0|).
__device__ __forceinline__ float normal_dist(float nx, float ny, float nz,
                                             float dx, float dy, float dz) {
#pragma clang fp contract(off)
  return fmaf(nx, dx, fmaf(ny, dy, nz * dz));
}

__device__ __forceinline__ double normal_dist(double nx, double ny, double nz,
                                              double dx, double dy, double dz) {
#pragma clang fp contract(off)
  return nx * dx + ny * dy + nz * dz;
}

// 1/r and e^{-k r} of one node for the difference (dx, dy, dz); FLOOR: with the
// cut-offs for coincident points (and for kappa r beyond the FP64 exponential's
// range), which give the same values where they do not apply.
template <bool FLOOR>
__device__ __forceinline__ void pair_node(float dx, float dy, float dz, const Screen<float> &sc,
                                          float &ri, float &ek) {
#pragma clang fp contract(off)
  const float rr = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
  ri = __builtin_amdgcn_rsqf(rr);
  if (FLOOR) ri = rr < kMinR2f ? 0.0f : ri;
  ek = __builtin_amdgcn_exp2f(sc.nk * (rr * ri));
}

template <bool FLOOR>
__device__ __forceinline__ void pair_node(double dx, double dy, double dz,
                                          const Screen<double> &sc, double &ri, double &ek) {
#pragma clang fp contract(off)
  double rr = fma(dx, dx, fma(dy, dy, dz * dz)), rad;
  const bool on = FLOOR && rr < kMinR2d;  // a node on the target adds nothing
  if (FLOOR) rr = on ? 1.0 : rr;
  ri = rsqrt_fp64(rr, rad);
  if (FLOOR) ri = on ? 0.0 : ri;
  ek = sc.exp<FLOOR>(rad);
}

// Node sums of one panel (NF nodes and the normal of record r) at p, for the
// near correction: vl = sum 1/r, kl = sum 1/r^3, vy = sum e/r, ky = sum (1 + k r)
// e/r^3 with e = e^{-k r}, and n.R.
template <int NF, class T>
__device__ __forceinline__ void panel_sums(const T *r, T px, T py, T pz, const Screen<T> &sc,
                                           T &vl, T &kl, T &vy, T &ky, T &nR) {
  vl = kl = vy = ky = T(0);
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    const T dx = px - r[3 * q], dy = py - r[3 * q + 1], dz = pz - r[3 * q + 2];
    if (q == 0) nR = normal_dist(r[9], r[10], r[11], dx, dy, dz);
    T ri, ek;
    pair_node<true>(dx, dy, dz, sc, ri, ek);
    const T er = ek * ri, ri2 = ri * ri;
    vl += ri;
    vy += er;
    kl = fma(ri2, ri, kl);
    ky = fma(er, fma(sc.kappa, ri, ri2), ky);
  }
}

// accumulators per row: one per node in FP32 (no chain of dependent additions),
// one in FP64 (registers)
template <class T, int NF> constexpr int kAcc = sizeof(T) == 4 ? NF : 1;

// One panel's share of the two rows of y = A x at target p, from its record
// (s_V, s_K, eps s_V in words 13..15), node q to its own accumulators a[0][q],
// a[1][q]:
//   a0 += (s_K n.R / r^2 - s_V) / r,
//   a1 += (eps s_V - s_K n.R (1/r + k) / r) e / r.
// Combining the layers per node takes 18.3 VALU instructions per node with
// n.R, against 19.8 with the four node sums weighted once per panel.
template <int NF, bool FLOOR, class T>
__device__ __forceinline__ void panel_rows(const T *r, T px, T py, T pz, const Screen<T> &sc,
                                           T (&a)[2][kAcc<T, NF>]) {
  T d[NF][3], b[2] = {T(0), T(0)};
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    d[q][0] = px - r[3 * q];
    d[q][1] = py - r[3 * q + 1];
    d[q][2] = pz - r[3 * q + 2];
  }
  const T skn = r[14] * normal_dist(r[9], r[10], r[11], d[0][0], d[0][1], d[0][2]);
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    T ri, ek;
    pair_node<FLOOR>(d[q][0], d[q][1], d[q][2], sc, ri, ek);
    const T ri2 = ri * ri;
    T *p0 = kAcc<T, NF> == NF ? &a[0][q] : &b[0], *p1 = kAcc<T, NF> == NF ? &a[1][q] : &b[1];
    *p0 = fma(ri, fma(skn, ri2, -r[13]), *p0);
    *p1 = fma(ek * ri, fma(-skn, fma(sc.kappa, ri, ri2), r[15]), *p1);
  }
  if (kAcc<T, NF> != NF) {
    a[0][0] += b[0];
    a[1][0] += b[1];
  }
}

// The transposed share: target p with weights z = (z1, z2, eps z2) adds to the
// sums of panel r (nodes and normal), node q to a[0][q] and a[1][q].
template <int NF, bool FLOOR, class T>
__device__ __forceinline__ void panel_columns(const T *r, T px, T py, T pz, T z1, T z2, T ez2,
                                              const Screen<T> &sc, T (&a)[2][kAcc<T, NF>]) {
  T d[NF][3], b[2] = {T(0), T(0)};
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    d[q][0] = px - r[3 * q];
    d[q][1] = py - r[3 * q + 1];
    d[q][2] = pz - r[3 * q + 2];
  }
  const T nR = normal_dist(r[9], r[10], r[11], d[0][0], d[0][1], d[0][2]);
  const T y1 = nR * z1, y2 = nR * z2;
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    T ri, ek;
    pair_node<FLOOR>(d[q][0], d[q][1], d[q][2], sc, ri, ek);
    const T ri2 = ri * ri;
    T *p0 = kAcc<T, NF> == NF ? &a[0][q] : &b[0], *p1 = kAcc<T, NF> == NF ? &a[1][q] : &b[1];
    *p0 = fma(ri, fma(-(y2 * ek), fma(sc.kappa, ri, ri2), y1 * ri2), *p0);
    *p1 = fma(ri, fma(ez2, ek, -z1), *p1);
  }
  if (kAcc<T, NF> != NF) {
    a[0][0] += b[0];
    a[1][0] += b[1];
  }
}

// Far-rule pair function of the operator for R = c_i - y (one node):
//   f = a1 n.R/r^3 - a2/r - a3 n.R (1 + k r) e/r^3 + a4 e/r,  e = e^{-k r}
// with a1 = l1_i phi_j, a2 = l1_i dphi_j, a3 = l2_i phi_j, a4 = eps l2_i dphi_j
// (the pair's share of lambda_x . A x; with the panel's packed strengths
// s_K, s_V in place of phi_j, dphi_j the weight and area are included).
// Returns f, df/dR, df/dn.
__device__ inline double op_pair(const double R[3], const double n[3], const Screen<double> &sc,
                                 double a1, double a2, double a3, double a4, double gR[3],
                                 double gn[3]) {
  const double rr = R[0] * R[0] + R[1] * R[1] + R[2] * R[2];
  if (rr < kMinR2d) {  // a node on the target (one-node rule, self panel): no term
    for (int d = 0; d < 3; ++d) gR[d] = gn[d] = 0.0;
    return 0.0;
  }
  double r;
  const double ri = rsqrt_fp64(rr, r), kappa = sc.kappa;
  const double ri3 = ri * ri * ri, ri5 = ri3 * ri * ri;
  const double e = sc.exp<true>(r);
  const double nR = n[0] * R[0] + n[1] * R[1] + n[2] * R[2];
  const double ky = (1.0 + kappa * r) * e;
  const double f = a1 * nR * ri3 - a2 * ri - a3 * nR * ky * ri3 + a4 * e * ri;
  const double c3 = e * (3.0 + 3.0 * kappa * r + kappa * kappa * rr);
  for (int d = 0; d < 3; ++d) {
    gR[d] = a1 * (n[d] * ri3 - 3.0 * nR * R[d] * ri5) + a2 * R[d] * ri3 -
            a3 * (ky * n[d] * ri3 - nR * c3 * R[d] * ri5) - a4 * ky * R[d] * ri3;
    gn[d] = a1 * R[d] * ri3 - a3 * ky * R[d] * ri3;
  }
  return f;
}

}  // namespace pbmp
