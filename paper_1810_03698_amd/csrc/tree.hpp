// Octree over the panels (internal Morton order) for the treecode product,
// built on the device (k_treebuild.hip).
#pragma once

#include <vector>

#include "common.hpp"

namespace pbmp {

// P2P tasks: source tile in LDS, targets per lane bound, lane groups on/off
#ifndef PBMP_P2P_TILE
#define PBMP_P2P_TILE 128
#endif
#ifndef PBMP_P2P_MAXTPT
#define PBMP_P2P_MAXTPT 5
#endif
#ifndef PBMP_P2P_GROUPS
#define PBMP_P2P_GROUPS 1
#endif

struct LaneSplit {
  int G, L, tpt;
};

// Lanes of a one-wave P2P task for nt targets (or sources, transposed): G groups
// of L = 64 / G lanes, tpt targets per lane, maximising the useful fraction
// G nt / (64 tpt) with tpt <= maxtpt (ties: fewer groups; more than 64 maxtpt
// targets take several passes of equal size with G = 1)
__host__ __device__ inline LaneSplit lane_split(int nt, int maxtpt) {
  const int passes = (nt + 64 * maxtpt - 1) / (64 * maxtpt);
  LaneSplit best{1, 64, (nt + 64 * passes - 1) / (64 * passes)};
  float be = (float)nt / (64.0f * best.tpt * passes);
  for (int G = 2; G <= 16 * PBMP_P2P_GROUPS; ++G) {
    const int L = 64 / G;
    const int tpt = (nt + L - 1) / L;
    if (tpt > maxtpt) continue;
    const float e = (float)(G * nt) / (64.0f * tpt);
    if (e > be) {
      be = e;
      best = LaneSplit{G, L, tpt};
    }
  }
  return best;
}

// boxes of an M2P task at most, and those whose words pass through LDS (and
// whose FP32 sums run) together, at most kM2PStageBytes of them
constexpr int kM2PTaskBoxes = 64;
constexpr int kM2PChunkBoxes = 16;
constexpr int kM2PStageBytes = 8192;
// work per task, in target-source pairs: a leaf of nt targets gets tasks of
// about p2p_task_work(N) / nt source panels (P2P) and m2p_task_work(N) / nt
// boxes (M2P, at most kM2PTaskBoxes), so that tasks take about the same time.
//
// P2P: a surface of N panels has some 3500 N panel pairs in leaves of 300 and
// the chip holds some 5000 waves of the kernel (LDS), so 12288 pairs per task
// leave 20480 panels barely one task per wave and 28880 a second round half
// full; smaller tasks fill it and shorten the tail until their slots cost the
// finish kernel more (whole products at 4096, 6144, 8192, 12288 pairs: 20480
// panels in FP32 191, 195, 193, 207 us; 28880 252, 251, 258, 263 us; 30420
// transposed in FP64 413, 418, 427, 440 us; 60500 in FP32 355, 349, 345, 352 us
// and transposed in FP64 811, 737, 713, 718 us; 144500, kernels alone, 1346,
// 1322, 1310, 1297 us).  Below 14336 panels it is 2048 (5120 panels in leaves of
// 50 at 1024, 2048, 4096, 12288: 95, 97, 107, 116 us in FP32, of 300 in FP64 138,
// 136, 134, 150 us).  Where a round of tasks just overflows the chip the larger
// ones win: 14580 transposed, N / 7 against 12288 pairs, 206 against 162 us in FP32.
// The vertex gradient runs on the same tasks; its whole share of a backward pass
// takes 3.0 ms at N / 7 and 4.1 at 12288 pairs on 8820 panels, 4.0 and 4.5 on 20480,
// 5.4 and 5.4 on 28880, 9.3 and 9.4 on 60500.
inline int p2p_task_work(int N) { return N / 7 < 2048 ? 2048 : N / 7 > 12288 ? 12288 : N / 7; }
// A surface of N panels has 100-200 N M2P pairs: N / 48 per task gives the
// largest ones some 8000 tasks (eight waves per SIMD, short tail) without more
// partial-sum slots than that needs (144500 panels: N / 24, 48, 96 took 163,
// 149, 153 us); below 1024 pairs the staging and the finish kernel's slots
// cost more than the shorter tasks gain (28880 panels: 59, 56 and 69 us for
// both kernels at 512, 1024 and 256)
inline int m2p_task_work(int N) { return N / 48 < 1024 ? 1024 : N / 48 > 4096 ? 4096 : N / 48; }
// Panels per moment task: longer leaves are cut into slices, which cost a
// reduction launch.
constexpr int kMomChunkPanels = 1024;
// leaves per shift task (moments of the boxes above the leaves), one round of
// a task: the boxes with more leaves (up to some 64 on surfaces cut into leaves
// of 300) take a reduction launch, which costs less than their rounds in turn
// (16, 32, 64 leaves: 13, 16, 18 us with it on 28880 panels, 27, 34, 54 us on
// 144500)
constexpr int kShiftLeaves = 16;
// target panels per M2P^T task (adjoint product)
constexpr int kM2PTChunkTargets = 512;

// Beyond this e^{-kappa r} vanishes at every distance that the pair cut-offs
// leave, and (kMaxKappa)^7, the highest power at order 6, is finite in FP64.
constexpr double kMaxKappa = 1e20;

struct TreeParams {
  double theta = 0.5;
  double kappa = 0.0;  // the only one of a tree (its tables hold powers of it), <= kMaxKappa
  int order = 4;
  int leaf = 300;
};

class Tree {
 public:
  TreeParams prm;
  // coefficient counts: ncoef = C(P+3, 3) single-layer terms (|k| <= P),
  // ncoefK = C(P+4, 3) double-layer terms (|k| <= P + 1: the double-layer
  // moment of degree |k| holds h^(|k|-1), so both layers reach degree P in
  // h); moments and local coefficients of a box are [ncoef | ncoefK]
  int nbox = 0, nleaf = 0, ncoef = 0, ncoefK = 0, nmom = 0, depth = 0;
  std::vector<int> level_start;  // boxes of level l are [level_start[l], level_start[l+1])
  // tasks and list sizes
  int n_p2p_tasks = 0, n_m2p_tasks = 0, max_slots = 0;
  int n_m2p_entries = 0, n_p2p_entries = 0;
  double direct_pairs = 0.0, m2p_pairs = 0.0;  // per product (nodes / boxes)

  // boxes (ids level by level, key order within a level)
  Dbuf<int> d_start, d_end, d_level, d_parent, d_first, d_nchild;
  Dbuf<int> d_range;      // [2*nbox] start, end
  Dbuf<int> d_child;      // [8*nbox] child ids (-1 none)
  Dbuf<double> d_center;  // [3*nbox] expansion centres
  Dbuf<double> d_radius;  // [2*nbox] R_B (far nodes), R_T (centroids)
  Dbuf<int> d_leaves;     // [nleaf] leaf box ids (the target leaves)
  // lists per target leaf (CSR over the leaf index)
  Dbuf<int> d_m2p_ptr, d_m2p_box;  // accepted boxes
  Dbuf<int> d_p2p_ptr, d_p2p_box;  // leaves summed directly
  // tasks
  Dbuf<int> d_p2p_task;   // [4*n] t0, t1, sub-range begin, end
  Dbuf<int> d_p2p_slot;
  Dbuf<int> d_p2p_src;    // source sub-ranges of the P2P tasks: [2*len] start, end
  Dbuf<int> d_m2p_task;   // [4*n] t0, t1, list begin, end
  Dbuf<int> d_m2p_slot;
  Dbuf<int> d_tslots;     // [N] number of slots of the target's leaf
  // transposed (adjoint) product: P2P^T tasks per source leaf and M2P^T
  // tasks per accepted box, each over target sub-ranges;
  // task = (box, sub begin, sub end, slot)
  Dbuf<int> d_p2pT_sub, d_p2pT_task, d_p2pT_count;  // count[2*box] = (subs, tasks)
  Dbuf<int> d_m2pT_sub, d_m2pT_task, d_m2pT_count, d_m2pT_off;  // off: first task of a box
  Dbuf<int> d_tslotsT;    // [N] transposed slots of the panel's leaf (tasks + 1)
  int n_p2pT_tasks = 0, n_m2pT_tasks = 0, max_slots_T = 1;
  Dbuf<double> d_Lpart, d_L;  // local coefficients: per M2P^T task (harmonic), per box [2][ncoefK]
  // moment tasks: the panels of every leaf in slices of at most
  // kMomChunkPanels; task = (box, s0, s1); a box's slices are consecutive
  int n_mom_tasks = 0;
  Dbuf<int> d_mom_task, d_mom_first, d_mom_count;
  Dbuf<double> d_mom_part;  // [n_mom_tasks][nmom]
  // shift tasks: the leaves under an accepted box with children in runs of
  // at most kShiftLeaves; task = (box, first leaf index, end leaf index)
  int n_shift_tasks = 0;
  bool shift_multi = false;  // some box has several shift tasks
  Dbuf<int> d_shift_task, d_shift_first, d_shift_count;
  Dbuf<double> d_shift_part;  // [n_shift_tasks][nmom]
  Dbuf<int> d_shift_toff;       // per coefficient k: terms [toff[k], toff[k+1])
  Dbuf<unsigned> d_shift_term;  // j | (k - j) << 8 | C(k, j) << 16 of each term
  Dbuf<double> d_mom64;   // [nbox][nmom]
  // harmonic form (harmonic.hpp): words per box, and the tables of the maps
  // from the Cartesian moments and (transposed) to the Cartesian locals
  Dbuf<double> d_harm64;
  Dbuf<float> d_harm32;
  Dbuf<int> d_hoff, d_hk, d_hpos, d_koff, d_kpos;
  Dbuf<double> d_hc, d_kc;  // (Laplace, Yukawa) constant per term
  Dbuf<int> d_monos;      // [3*ncoefK] exponents up to degree P + 1

  // Build from the Morton keys of the panels in internal (sorted) order,
  // the centroids (geo SoA) and far nodes (src64 records), all on device.
  void build_device(int N, int nf, const uint64_t *key, const double *geo,
                    const double *src64, hipStream_t s);

 private:
  hipStream_t stream_ = nullptr;
  void build_transposed(int N, const int *owner, Dbuf<char> &tmp);
};

// Morton order of the panels on the device: perm[i] = caller's index of the
// i-th panel, key_sorted[i] its key (tri_user: the caller's triangles)
void morton_order_device(hipStream_t s, int N, const double *verts, const int *tri_user,
                         int *perm, uint64_t *key_sorted);

// upload the multi-index exponent table of the chosen order (d_monos)
void tree_upload_exponents(Tree &t, hipStream_t s);
// tables and buffers of the harmonic form for the chosen order and kappa
void tree_upload_harmonics(Tree &t, hipStream_t s);

}  // namespace pbmp
