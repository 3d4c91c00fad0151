// HIP kernels of the EGT hot path for gfx950 (CDNA4, 64-lane wavefronts).
//
//  * sbr_fused_kernel  : for small trees (fits_fused), a whole smoothed
//    best response (Section 4, Eq. 4 and the leaf / internal-simplex
//    derivation) in one launch: bottom-up over every level, root-value
//    partial sums, then the top-down rebuild q_i = q_{p_j} q_bar_i with the
//    convex-combination epilogue of Algorithm 2 (x_hat, y_+, x_+);
//    mu = 0 gives the best response;
//  * the same steps one level per launch for large trees:
//    bottom_up_leaf_pair_kernel (lowest level) or bottom_up_level_kernel
//    (its one-hand-per-lane form, for few nodes or unaligned rows), bottom_up_wide_kernel (levels of many nodes
//    with children, a wavefront per node) or bottom_up_internal_kernel (of few,
//    a wavefront per action, at most 8), top_down_kernel, and root_sums_kernel
//    where no top-down pass takes the root sums along;
//  * small helpers (uniform point, a*x + b*y, max |x|).
//
// Every vector is double[rows][ld], hands (slots) fastest, so consecutive
// lanes read consecutive doubles of one row.  Reductions use fixed orders, so
// results are bitwise repeatable run to run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "egt_device.h"
#include "egt_internal.h"

namespace egt {

namespace {

constexpr int kPassThreads = 64;       // per-level pass: one wavefront per (node, 64 hands)
constexpr int kDownWaves = 4;           // top-down pass: wavefronts per block
constexpr int kLeafRegs = 4;           // lowest level: actions of a node held in registers
constexpr int kInternalWaves = 8;       // level path: wavefronts per node block (4 blocks fill a CU's 32 wave slots)

// The per-information-set arithmetic of Section 4's smoothed best response in
// the association of its formulas, every operation rounded on its own (the
// library is built without floating-point contraction), so that every pass
// form below rounds exactly like a plain evaluation of those formulas:
//   weight of action a   w_a = exp((m - g~_a) / (mu beta)), m = min_a g~_a,
//                        so the largest weight is exactly 1;
//   node value           V = (m - mu beta log S) + mu beta log n, S = sum_a w_a
//                        added in action order;
//   local probability    q_bar_a = w_a / S.
// The precision form takes the exponential in FP32 of the FP64 shift times
// 1/temp, keeps S, the logarithm and V in FP64, and forms q_bar with the FP32
// reciprocal of S (itemp and rsum are used by the precision form only).
template <class TG>
__device__ inline double lse_weight(double m, double g, double temp, double itemp) {
  if constexpr (std::is_same<TG, float>::value)
    return (double)expf((float)((m - g) * itemp));
  else
    return exp((m - g) / temp);
}
template <class TG>
__device__ inline double inv_or_zero(double x) {
  return std::is_same<TG, float>::value ? 1.0 / x : 0.0;
}
template <class TG>
__device__ inline double qbar(double w, double sum, double rsum) {
  if constexpr (std::is_same<TG, float>::value)
    return (double)((float)w * (float)rsum);
  else
    return w / sum;
}
__device__ inline double lse_value(double m, double temp, double sum, double logn) {
  return (m - temp * log(sum)) + temp * logn;
}

// FP64 weights with temp's reciprocal known before the shift is: for y = 1/temp rounded, q0 = x y is within two ulps of x/temp, and two
// corrections by the exact remainder, q <- q + (x - temp q) y, give the rounded
// quotient (Markstein; the second starts within one ulp) -- 5 dependent
// operations of 5 cycles where a division takes 106 cycles of a chain that
// nothing else runs beside.  Exact remainders need temp in [2^-900, 2^900]
// (temp_inverse is 0 outside, and the wavefront divides) and x above some
// 2^-960, below which the quotient's exponential is 1 whatever its last bit.  A
// quotient below -1e4 (an overflowed one has no remainder) is left as q0: its
// exponential is 0.
template <class TG>
__device__ inline double temp_inverse(double temp) {
  return std::is_same<TG, float>::value || (temp >= 0x1p-900 && temp <= 0x1p900) ? 1.0 / temp : 0.0;
}
template <class TG>
__device__ inline double lse_weight_by_inverse(double m, double g, double temp, double itemp) {
  if constexpr (std::is_same<TG, float>::value) {
    return lse_weight<TG>(m, g, temp, itemp);
  } else {
    const double x = m - g;
    double q;
    if (__any(itemp == 0.0)) {
      q = x / temp;
    } else {
      const double q0 = x * itemp;
      q = __builtin_fma(__builtin_fma(-temp, q0, x), itemp, q0);
      q = __builtin_fma(__builtin_fma(-temp, q, x), itemp, q);
      q = q0 < -1e4 ? q0 : q;
    }
    return exp(q);
  }
}
// cA a + cB b (the mixed gradient of the prox, or a single scaled gradient).
__device__ inline double lin2(double cA, double a, double cB, double b) { return cA * a + cB * b; }

// ---------------------------------------------------------------------------
// One information set (node v, hand h) of a bottom-up pass:
//   g~_a = cA gA[v,a] + cB gB[v,a] + sum_{k in D(v,a)} V[k]
//   smoothed (mu > 0, temp = mu beta_v):
//     m = min_a g~_a,  w_a = exp((m - g~_a) / temp),  S = sum_a w_a
//     V[v] = m - temp log S + temp log n_v,  q_bar_a = w_a / S
//   best response (mu = 0): V[v] = min_a g~_a.
// The action with the smallest g~ has the largest q_bar (weight exactly 1), so
// V is the value g~_i + temp log q_bar_i + temp log n_v at that action, and
// every exponent is <= 0.  Both pass forms below evaluate exactly this through
// lse_weight / lse_value, the children of an action added in betting order
// (the order of the child CSR).
// ---------------------------------------------------------------------------

// ---------------------------------------------------------------------------
// Fused pass for small trees (fits_fused): block = (tree k, HB hands).
//
// A launch moves a few MB; its time is the chain of dependent steps of each
// level and the instructions around them: index arithmetic, loops over a node's
// actions, look-ups of tables (cycle stamps of a form that kept the tables in
// LDS, on the 223-sequence tree: of 24,000 cycles a block, 14,000 in three
// levels whose own chain -- minimum, division, exponential, logarithm -- takes
// about 1,000 each).  So a thread keeps the records of its (sequence, hand)
// pairs and of its node task in registers, and whatever the next level does not
// wait for is left until the levels are done.  223 sequences x 1081 hands, one
// tree: 14.3 -> 11.1 us; with the best responses beside, two trees: 17.9 ->
// 15.1 us; Leduc hold'em, which fits since a block may hold one hand: 20.4 ->
// 10.7 us for one tree against a launch per level.
//   1. Staging: every thread loads the records of its K sequences and of its
//      node and, at the same time, the combined gradient cA gA + cB gB and the
//      epilogue's x_prev; the gradient goes to LDS.
//   2. Bottom-up, a block barrier after each phase of a level:
//      (a) sequences above the lowest level: g~_s = g_s + the values of the
//          child nodes of s, read from their contiguous value slots;
//      (b) nodes: minimum, weights (to LDS), their sum (to LDS) and the node
//          value, by two lanes per (node, hand) on the lowest level (its nodes
//          have few actions, and the block's 512 threads are then one task
//          each on a tree of 63 such nodes) and by four above it.
//   3. The block's partial root sum (the tree value is a sum over (root, hand)).
//   4. q_bar = weight / sum, one sequence per thread, then top-down, level by
//      level from the roots, q[s] = q[parent] * q_bar[s], and the epilogue
//      (1 - tau) x_prev + tau q.  Slots h >= n (the row padding) are written 0.
// The additions, minima and products are those of one thread evaluating a node
// by itself, in its order, so the bits are too.
//
// The grid is one-dimensional over (tree, hand block) and spread so that each
// XCD (workgroups go round-robin over the 8 XCDs) gets a contiguous range of
// hand blocks: neighbouring blocks share cache lines of every row, and those
// then meet in one L2.
// ---------------------------------------------------------------------------
struct FusedTree {
  const SeqRec* seq;
  const NodeRec* node;
  const void* gA;
  const void* gB;
  const void* x_prev;
  void* q_out;
  void* comb_out;
  void* g_out;
  void* qb_out;
  double cA, cB, mu, tau, g_scale;
  int S, N, C, n_roots, n_levels, n_leaf, dual;  // n_leaf: nodes of the lowest level
};

struct FusedArgs {
  FusedTree t[kMaxTrees];
  double* partial;  // [trees (and dual trees)][n_hblocks] or null (device or pinned host memory)
  int count, n, ld, n_hblocks;  // hand blocks per tree
  int cap_nodes, cap_seqs;
};

// A double moved within every aligned quad of lanes (DPP quad permute).
template <int CTRL>
__device__ inline double quad_move(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// One (node, hand) task of the node phase by 2 or (quad) 4 adjacent lanes, b the
// lane's place: g~ of the node's actions at G, lane b taking actions b, b + 2 or
// b + 4, ...; the minimum crosses the lanes by DPP.
template <int HB>
__device__ __forceinline__ double lanes_min(const double* G, int na, int b, bool quad) {
  const int step = quad ? 4 : 2;
  double m = G[min(b, na - 1) * HB];
  for (int a = b + step; a < na; a += step) m = fmin(m, G[a * HB]);
  m = fmin(m, quad_move<0xb1>(m));             // lanes 1 0 3 2
  if (quad) m = fmin(m, quad_move<0x4e>(m));  // lanes 2 3 0 1
  return m;
}

// Smoothed: weights to W, their sum (every lane adds them in action order, the
// lanes' weights by DPP) and the node value returned.
template <class TG, int HB>
__device__ __forceinline__ double lanes_node(const double* G, double* W, int na, int b, bool quad, double temp,
                                             double itemp, double logn, double* sum_out) {
  const double m = lanes_min<HB>(G, na, b, quad);
  const int step = quad ? 4 : 2;
  double sum = 0.0;
#pragma unroll 1
  for (int a = 0; a < na; a += step) {
    const int own = a + b;
    const double w = lse_weight_by_inverse<TG>(m, G[min(own, na - 1) * HB], temp, itemp);
    if (own < na) W[own * HB] = w;
    if (quad) {
      const double w0 = quad_move<0x00>(w), w1 = quad_move<0x55>(w), w2 = quad_move<0xaa>(w), w3 = quad_move<0xff>(w);
      sum += w0;
      if (a + 1 < na) sum += w1;
      if (a + 2 < na) sum += w2;
      if (a + 3 < na) sum += w3;
    } else {
      const double w0 = quad_move<0xa0>(w), w1 = quad_move<0xf5>(w);  // lanes 0 0 2 2, 1 1 3 3
      sum += w0;
      if (a + 1 < na) sum += w1;
    }
  }
  *sum_out = sum;
  return lse_value(m, temp, sum, logn);
}

template <int HB, int K, class TG>
__global__ __launch_bounds__(kFusedThreads, K <= 2 ? 8 : K <= 3 ? 5 : 4) void sbr_fused_kernel(FusedArgs a) {
  extern __shared__ __align__(16) double fused_lds[];
  const int nb = a.n_hblocks;
  const int P = xcd_spread((int)blockIdx.x, (int)gridDim.x);
  const int k = P / nb, hblk = P % nb;
  const FusedTree& t = a.t[k];
  const int S = t.S, N = t.N, n = a.n, n_levels = t.n_levels, ld = a.ld;
  const double mu = t.mu;
  const bool smooth = mu > 0.0;
  // a dual tree (every tree of the launch is then dual) also takes the best
  // response to the same gradient: its g~ and node values beside
  const bool dual = t.dual != 0;
  const int sl = (a.cap_seqs + kFusedPad) * HB, nl = (a.cap_nodes + kFusedPad) * HB;
  double* Gl = fused_lds;  // [seqs][HB] gradient, then g~
  double* Wl = Gl + sl;    // [seqs][HB] weights, then q_bar and q
  double* Vs = Wl + sl;    // [nodes][HB] node values by slot
  double* Sl = Vs + nl;    // [nodes][HB] weight sums by slot
  double* GBl = Sl + nl;   // [seqs][HB] dual: gradient, then the best response's g~
  double* VBs = GBl + sl;  // [nodes][HB] dual: best-response node values
  const int tid = threadIdx.x, T = blockDim.x;
  const int h0 = hblk * HB;
  const TG* gA = (const TG*)t.gA;
  const TG* gB = (const TG*)t.gB;
  const TG* x_prev = (const TG*)t.x_prev;
  TG* g_out = (TG*)t.g_out;
  TG* q_out = (TG*)t.q_out;
  TG* comb_out = (TG*)t.comb_out;
  TG* qb_out = (TG*)t.qb_out;
  const bool want_q = (q_out || comb_out || qb_out) && smooth;

  // 1. this thread's (sequence, hand) pairs j = u T + tid, as LDS indices
  // packed in pairs (a block has at most kFusedTasks * kFusedThreads of them)
  constexpr unsigned kNone = 0xffffu;
  unsigned child[K];     // first child's value slot, number of children
  unsigned par_slot[K];  // parent (kNone at a root), own node's slot
  int lev[K];            // level, -1: no pair here
  double vx[K];
  double va[K], vb[K];
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int j = u * T + tid, s = j / HB, hl = j % HB, h = h0 + hl;
    va[u] = vb[u] = vx[u] = 0.0;
    child[u] = par_slot[u] = 0u;
    lev[u] = -1;
    if (s < S && h < n) {
      const size_t idx = (size_t)s * ld + h;
      const SeqRec r = t.seq[s];
      va[u] = (double)gA[idx];
      if (gB) vb[u] = (double)gB[idx];
      if (comb_out) vx[u] = (double)x_prev[idx];
      child[u] = (unsigned)(r.c0 * HB + hl) | ((unsigned)r.n_child << 16);
      par_slot[u] = (r.parent >= 0 ? (unsigned)(r.parent * HB + hl) : kNone) | ((unsigned)(r.slot * HB + hl) << 16);
      lev[u] = r.level;
    }
  }
  // Node tasks, numbered through: two per (node, hand) of the lowest level, then
  // four per (node, hand) of the others, where there are fewer.  The thread's
  // first one stays in registers; a tree with more tasks than threads reads the
  // others' records when their level comes.
  const int n_leaf = t.n_leaf, leaf_tasks = n_leaf * HB * 2, quad0 = (leaf_tasks + 3) & ~3;
  const int n_tasks = quad0 + (N - n_leaf) * HB * 4;
  struct Task {
    int na_level, at_slot;  // level -1: none here; LDS indices
    double temp, itemp, logn;
  };
  auto task_of = [&](int q) {
    const bool quad = q >= quad0;
    const int i = quad ? (q - quad0) / 4 : q / 2, v = (quad ? n_leaf : 0) + i / HB, hl = i % HB;
    Task d{1 | (-1 << 8), 0, 1.0, 1.0, 0.0};
    if ((quad ? q < n_tasks : q < leaf_tasks) && h0 + hl < n) {
      const NodeRec r = t.node[v];
      const double temp = mu * r.beta;
      d = Task{r.na | (r.level << 8), (r.first * HB + hl) | ((r.slot * HB + hl) << 16), temp,
               smooth ? temp_inverse<TG>(temp) : 0.0, r.logn};
    }
    return d;
  };
  const Task own = task_of(tid);
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int j = u * T + tid, s = j / HB;
    if (s < S) {
      double x = gB ? lin2(t.cA, va[u], t.cB, vb[u]) : t.cA * va[u];
      if (dual) GBl[j] = x;
      if (g_out) {
        g_out[(size_t)s * ld + h0 + j % HB] = (TG)(x * t.g_scale);  // 0 in the padding
        x = (double)(TG)x;  // continue with the stored gradient (g_scale = +-1)
      }
      Gl[j] = x;
    }
  }
  __syncthreads();

  // 2. bottom-up
  auto run_task = [&](const Task& d, bool quad, int b) {
    const int na = d.na_level & 0xff, at = d.at_slot & 0xffff, slot = (int)((unsigned)d.at_slot >> 16);
    if (dual || !smooth) {
      const double m = lanes_min<HB>((dual ? GBl : Gl) + at, na, b, quad);
      if (b == 0) (dual ? VBs : Vs)[slot] = m;
      if (!smooth) return;
    }
    double sum;
    const double v = lanes_node<TG, HB>(Gl + at, Wl + at, na, b, quad, d.temp, d.itemp, d.logn, &sum);
    if (b == 0) {
      Vs[slot] = v;
      Sl[slot] = sum;
    }
  };
  for (int l = 0; l < n_levels; ++l) {
    if (l > 0) {
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int j = u * T + tid, c0 = (int)(child[u] & 0xffffu), cn = (int)(child[u] >> 16);
        if (lev[u] != l || cn == 0) continue;
        Gl[j] = add_run<HB>(Gl[j], Vs + c0, cn);
        if (dual) GBl[j] = add_run<HB>(GBl[j], VBs + c0, cn);  // the same additions on the best-response values
      }
      __syncthreads();
    }
    Task d = own;
#pragma unroll 1
    for (int q = tid;;) {
      if ((d.na_level >> 8) == l) run_task(d, l > 0, q & (l > 0 ? 3 : 1));
      if ((q += T) >= n_tasks) break;
      d = task_of(q);
    }
    __syncthreads();
  }

  // 3. partial root sums, in the block's last HB threads: the tree's, and a
  // dual tree's best response after the launch's trees
  const int rt = tid - (T - HB);
  if (a.partial && rt >= 0) {
    double sv = 0.0, sb = 0.0;
    if (h0 + rt < n) {
      sv = add_run<HB>(0.0, Vs + t.C * HB + rt, t.n_roots);
      if (dual) sb = add_run<HB>(0.0, VBs + t.C * HB + rt, t.n_roots);
    }
#pragma unroll
    for (int off = HB / 2; off > 0; off >>= 1) {
      sv += __shfl_down(sv, off, HB);
      sb += __shfl_down(sb, off, HB);
    }
    if (rt == 0) {
      a.partial[(size_t)k * nb + hblk] = sv;
      if (dual) a.partial[(size_t)(a.count + k) * nb + hblk] = sb;
    }
  }

  // 4. local strategies, top-down and epilogue (0 in the padding)
  if (want_q) {
    double qv[K];
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const int j = u * T + tid, s = j / HB;
      qv[u] = 0.0;
      if (lev[u] >= 0) {
        const double sum = Sl[par_slot[u] >> 16];
        qv[u] = (double)(TG)qbar<TG>(Wl[j], sum, inv_or_zero<TG>(sum));
      }
      if (qb_out && s < S) qb_out[(size_t)s * ld + h0 + j % HB] = (TG)qv[u];
    }
    if (q_out || comb_out) {
#pragma unroll
      for (int u = 0; u < K; ++u)
        if (lev[u] > 0) Wl[u * T + tid] = qv[u];  // the lowest level has no children
      for (int l = n_levels - 2; l >= 0; --l) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < K; ++u) {
          const unsigned par = par_slot[u] & 0xffffu;
          if (lev[u] != l || par == kNone) continue;
          qv[u] = (double)((TG)Wl[par] * (TG)qv[u]);
          if (l > 0) Wl[u * T + tid] = qv[u];
        }
      }
      const TG tau = (TG)t.tau, one_m_tau = (TG)(1.0 - t.tau);
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int j = u * T + tid, s = j / HB;
        if (s >= S) continue;
        const size_t idx = (size_t)s * ld + h0 + j % HB;
        const TG q = (TG)qv[u];
        if (q_out) q_out[idx] = q;
        if (comb_out) comb_out[idx] = one_m_tau * (TG)vx[u] + tau * q;
      }
    }
  }

  // one live slot (HB = 1, one block per tree): the block also writes the rows' padding
  if constexpr (HB == 1) {
    const int pad = ld - 1;
    TG* outs[4] = {g_out, want_q ? qb_out : nullptr, q_out, comb_out};
    for (int o = 0; o < 4; ++o)
      if (outs[o])
        for (int i = tid; i < S * pad; i += T) outs[o][(size_t)(i / pad) * ld + 1 + i % pad] = (TG)0;
  }
}

// Large trees: one launch per level over all trees of the set; block = one
// wavefront for (node, 64 hands); node values (by value slot) and q_bar in
// global memory.  The node's record and parameters come from the table image
// (block-uniform loads), a sequence's children from contiguous value slots.
// With g_out the launch also writes g_scale (cA gA + cB gB) of every sequence
// it reads.
template <class TG>
__global__ __launch_bounds__(kPassThreads) void bottom_up_level_kernel(PassSet a) {
  int y = blockIdx.y, k = 0;
  while (k < a.count - 1 && y >= a.level_cnt[k]) {
    y -= a.level_cnt[k];
    ++k;
  }
  const TreePass& t = a.t[k];
  const int h = blockIdx.x * kPassThreads + threadIdx.x;
  if (h >= a.n) return;
  const size_t ld = a.ld;
  const int v = t.level_begin[a.level] + y;
  const LevelTabLayout L = level_tab_layout(t.P.n_nodes, t.P.n_seq);
  const unsigned char* tab = (const unsigned char*)t.P.level_tab;
  const int4 r = ((const int4*)(tab + L.rec))[v];
  const double2 p0 = ((const double2*)(tab + L.prm))[2 * v], p1 = ((const double2*)(tab + L.prm))[2 * v + 1];
  const int* cbeg = (const int*)(tab + L.cbeg);
  const int s0 = r.x, na = r.y;
  const TG* gA = (const TG*)t.gA;
  const TG* gB = (const TG*)t.gB;
  TG* g_out = (TG*)t.g_out;
  double g[kMaxActions];
  double m = INFINITY;
#pragma unroll
  for (int j = 0; j < kMaxActions; ++j) {
    if (j < na) {
      const size_t idx = (size_t)(s0 + j) * ld + h;
      double x = gB ? lin2(t.cA, (double)gA[idx], t.cB, (double)gB[idx]) : t.cA * (double)gA[idx];
      if (g_out) {
        g_out[idx] = (TG)(x * t.g_scale);
        x = (double)(TG)x;  // continue with the stored gradient (g_scale = +-1)
      }
      const int c1 = cbeg[s0 + j + 1];
      for (int c = cbeg[s0 + j]; c < c1; ++c) x += t.V[(size_t)c * ld + h];
      g[j] = x;
      m = fmin(m, x);
    }
  }
  if (!(t.mu > 0.0)) {
    t.V[(size_t)r.z * ld + h] = m;
    return;
  }
  // dual pass: below a node without child nodes the best response's g~ is
  // the same, so its value is the minimum
  if (t.VB) t.VB[(size_t)r.z * ld + h] = m;
  const double temp = t.mu * p0.x, itemp = inv_or_zero<TG>(temp);
  double sum = 0.0;
#pragma unroll
  for (int j = 0; j < kMaxActions; ++j) {
    if (j < na) {
      g[j] = lse_weight<TG>(m, g[j], temp, itemp);
      sum += g[j];
    }
  }
  t.V[(size_t)r.z * ld + h] = lse_value(m, temp, sum, p1.x);
  if (t.QB) {
    const double rs = inv_or_zero<TG>(sum);
#pragma unroll
    for (int j = 0; j < kMaxActions; ++j)
      if (j < na) ((TG*)t.QB)[(size_t)(s0 + j) * ld + h] = (TG)qbar<TG>(g[j], sum, rs);
  }
}

// The lowest level (no node has children) with two adjacent hands per lane:
// one 16-byte access per gradient row (8 bytes in FP32), half the wavefronts.
// Used for levels of many nodes when every row pointer is aligned to two elements;
// per hand the arithmetic is the one above, and slots h >= n are not written.
//
// A wavefront's rows are all requested before the first is used, and only the
// first kLeafRegs actions of a node live in registers (most nodes have two;
// further ones pass through LDS, a lane's own column), which makes 60 registers
// and 8 wavefronts per SIMD of 102 and 4.  1777 nodes x 1081 hands (90 MB, 17.6
// us at the rate of a large copy): 32 -> 27.5 us, in FP32 22.6 -> 19.9; two
// trees with their best responses 61 -> 48.7.  What is left is latency and the
// vector units, 68% busy, side by side: leaving the exponential of the
// smallest action out (it is 1), 2 to 8 wavefronts per block or fewer registers
// changed nothing.
template <class TG>
__device__ inline void store_pair(TG* p, double x0, double x1, bool both) {
  using V2 = typename std::conditional<std::is_same<TG, float>::value, float2, double2>::type;
  if (both) {
    V2 o;
    o.x = (TG)x0;
    o.y = (TG)x1;
    *(V2*)p = o;
  } else {
    p[0] = (TG)x0;
  }
}

template <class TG>
__global__ __launch_bounds__(kPassThreads, 8) void bottom_up_leaf_pair_kernel(PassSet a) {
  extern __shared__ double2 leaf_more[];
  using V2 = typename std::conditional<std::is_same<TG, float>::value, float2, double2>::type;
  int y = blockIdx.y, k = 0;
  while (k < a.count - 1 && y >= a.level_cnt[k]) {
    y -= a.level_cnt[k];
    ++k;
  }
  const TreePass& t = a.t[k];
  const int h = 2 * (blockIdx.x * kPassThreads + threadIdx.x);
  if (h >= a.n) return;
  const bool both = h + 1 < a.n;
  const size_t ld = a.ld;
  const int v = t.level_begin[a.level] + y;
  const LevelTabLayout L = level_tab_layout(t.P.n_nodes, t.P.n_seq);
  const unsigned char* tab = (const unsigned char*)t.P.level_tab;
  const int4 r = ((const int4*)(tab + L.rec))[v];
  const double2 p0 = ((const double2*)(tab + L.prm))[2 * v], p1 = ((const double2*)(tab + L.prm))[2 * v + 1];
  const int s0 = r.x, na = r.y;
  const TG* gA = (const TG*)t.gA + (size_t)s0 * ld + h;
  const TG* gB = t.gB ? (const TG*)t.gB + (size_t)s0 * ld + h : nullptr;
  TG* g_out = t.g_out ? (TG*)t.g_out + (size_t)s0 * ld + h : nullptr;
  TG* QB = t.QB ? (TG*)t.QB + (size_t)s0 * ld + h : nullptr;
  double2* more = leaf_more + threadIdx.x;  // g~ and weights of the actions from kLeafRegs on
  double m0 = INFINITY, m1 = INFINITY;
  auto combine = [&](int j, const V2& A, const V2& B, double& x0, double& x1) {
    x0 = gB ? lin2(t.cA, (double)A.x, t.cB, (double)B.x) : t.cA * (double)A.x;
    x1 = gB ? lin2(t.cA, (double)A.y, t.cB, (double)B.y) : t.cA * (double)A.y;
    if (g_out) {
      store_pair(g_out + j * ld, x0 * t.g_scale, x1 * t.g_scale, both);
      x0 = (double)(TG)x0;  // continue with the stored gradient (g_scale = +-1)
      x1 = (double)(TG)x1;
    }
    m0 = fmin(m0, x0);
    m1 = fmin(m1, x1);
  };
  double g0[kLeafRegs], g1[kLeafRegs];
  {
    V2 A[kLeafRegs], B[kLeafRegs];
#pragma unroll
    for (int j = 0; j < kLeafRegs; ++j)
      if (j < na) {
        A[j] = *(const V2*)(gA + j * ld);
        if (gB) B[j] = *(const V2*)(gB + j * ld);
      }
#pragma unroll
    for (int j = 0; j < kLeafRegs; ++j)
      if (j < na) combine(j, A[j], B[j], g0[j], g1[j]);
  }
#pragma unroll 2
  for (int j = kLeafRegs; j < na; ++j) {
    V2 B;
    if (gB) B = *(const V2*)(gB + j * ld);
    double2 x;
    combine(j, *(const V2*)(gA + j * ld), B, x.x, x.y);
    more[(j - kLeafRegs) * kPassThreads] = x;
  }
  double* Vrow = t.V + (size_t)r.z * ld + h;
  if (!(t.mu > 0.0)) {
    store_pair(Vrow, m0, m1, both);
    return;
  }
  if (t.VB) store_pair(t.VB + (size_t)r.z * ld + h, m0, m1, both);  // dual pass: the best response's value
  const double temp = t.mu * p0.x, itemp = temp_inverse<TG>(temp);
  double sum0 = 0.0, sum1 = 0.0;
#pragma unroll
  for (int j = 0; j < kLeafRegs; ++j)
    if (j < na) {
      g0[j] = lse_weight_by_inverse<TG>(m0, g0[j], temp, itemp);
      g1[j] = lse_weight_by_inverse<TG>(m1, g1[j], temp, itemp);
      sum0 += g0[j];
      sum1 += g1[j];
    }
  for (int j = kLeafRegs; j < na; ++j) {
    double2 x = more[(j - kLeafRegs) * kPassThreads];
    x.x = lse_weight_by_inverse<TG>(m0, x.x, temp, itemp);
    x.y = lse_weight_by_inverse<TG>(m1, x.y, temp, itemp);
    sum0 += x.x;
    sum1 += x.y;
    more[(j - kLeafRegs) * kPassThreads] = x;
  }
  store_pair(Vrow, lse_value(m0, temp, sum0, p1.x), lse_value(m1, temp, sum1, p1.x), both);
  if (QB) {
    const double rs0 = inv_or_zero<TG>(sum0), rs1 = inv_or_zero<TG>(sum1);
#pragma unroll
    for (int j = 0; j < kLeafRegs; ++j)
      if (j < na) store_pair(QB + j * ld, qbar<TG>(g0[j], sum0, rs0), qbar<TG>(g1[j], sum1, rs1), both);
    for (int j = kLeafRegs; j < na; ++j) {
      const double2 w = more[(j - kLeafRegs) * kPassThreads];
      store_pair(QB + j * ld, qbar<TG>(w.x, sum0, rs0), qbar<TG>(w.y, sum1, rs1), both);
    }
  }
}

// Levels above the lowest (every node has child nodes): the same evaluation
// with the actions in parallel, for levels of few nodes.  Block = (node, 64
// hands) x `blockDim.y` wavefronts (the level's most actions, at most
// kInternalWaves); wavefront j takes actions j, j + blockDim.y, ...: its
// gradients and its children, whose value slots [cbeg[s], cbeg[s + 1]) are
// read in batches of kChildBatch so that one round trip covers them all and
// added in slot order.  The node's g~ and weights meet in LDS; the minimum,
// the weight sum and the value are then formed in the same order as above, so
// per hand the result is bitwise the one the one-wavefront form gives.
template <class TG>
__global__ __launch_bounds__(kPassThreads * kInternalWaves) void bottom_up_internal_kernel(PassSet a) {
  constexpr int kChildBatch = 8;
  __shared__ double gl[kMaxActions][kPassThreads];
  __shared__ double wl[kMaxActions][kPassThreads];
  int y = blockIdx.y, k = 0;
  while (k < a.count - 1 && y >= a.level_cnt[k]) {
    y -= a.level_cnt[k];
    ++k;
  }
  const TreePass& t = a.t[k];
  const int lane = threadIdx.x, j = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
  const int h = blockIdx.x * kPassThreads + lane;
  const size_t ld = a.ld;
  const int v = t.level_begin[a.level] + y;
  const LevelTabLayout L = level_tab_layout(t.P.n_nodes, t.P.n_seq);
  const unsigned char* tab = (const unsigned char*)t.P.level_tab;
  const int4 r = ((const int4*)(tab + L.rec))[v];
  const double2 p0 = ((const double2*)(tab + L.prm))[2 * v], p1 = ((const double2*)(tab + L.prm))[2 * v + 1];
  const int* cbeg = (const int*)(tab + L.cbeg);
  const int s0 = r.x, na = r.y;
  const bool live = h < a.n;
  const bool act = live && j < na;  // this wavefront owns actions j, j + blockDim.y, ...
  const int nw = (int)blockDim.y;
  const TG* gA = (const TG*)t.gA;
  const TG* gB = (const TG*)t.gB;
  TG* g_out = (TG*)t.g_out;
  for (int jj = j; live && jj < na; jj += nw) {
    const size_t idx = (size_t)(s0 + jj) * ld + h;
    const int c0 = cbeg[s0 + jj], c1 = cbeg[s0 + jj + 1];
    double cv[kChildBatch];
    auto load_children = [&](int c) {
#pragma unroll
      for (int u = 0; u < kChildBatch; ++u)
        if (c + u < c1) cv[u] = t.V[(size_t)(c + u) * ld + h];
    };
    // the gradient and the first children are requested together
    const TG A = gA[idx], B = gB ? gB[idx] : (TG)0;
    load_children(c0);
    double x = gB ? lin2(t.cA, (double)A, t.cB, (double)B) : t.cA * (double)A;
    if (g_out) {
      g_out[idx] = (TG)(x * t.g_scale);
      x = (double)(TG)x;  // continue with the stored gradient (g_scale = +-1)
    }
    for (int c = c0; c < c1; c += kChildBatch) {
      if (c > c0) load_children(c);
#pragma unroll
      for (int u = 0; u < kChildBatch; ++u)
        if (c + u < c1) x += cv[u];
    }
    gl[jj][lane] = x;
  }
  __syncthreads();
  // four actions of the node per LDS round trip (the last one repeated)
  double m = INFINITY;
  if (act)
    for (int i = 0; i < na; i += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) m = fmin(m, gl[min(i + u, na - 1)][lane]);
  double* Vrow = t.V + (size_t)r.z * ld + h;
  if (!(t.mu > 0.0)) {
    if (act && j == 0) Vrow[0] = m;
    return;
  }
  const double temp = t.mu * p0.x, itemp = temp_inverse<TG>(temp);
  for (int jj = j; live && jj < na; jj += nw) wl[jj][lane] = lse_weight_by_inverse<TG>(m, gl[jj][lane], temp, itemp);
  __syncthreads();
  if (act) {
    // rows up to the next multiple of four are read, never added
    const double sum = add_run<kPassThreads>(0.0, &wl[0][lane], na);
    if (j == 0) Vrow[0] = lse_value(m, temp, sum, p1.x);
    if (t.QB) {
      const double rs = inv_or_zero<TG>(sum);
      for (int jj = j; jj < na; jj += nw)
        ((TG*)t.QB)[(size_t)(s0 + jj) * ld + h] = (TG)qbar<TG>(wl[jj][lane], sum, rs);
    }
  }
}

// A wide level above the lowest: block = one wavefront for (node, 64 x HP
// hands), as on the lowest level.  The node's gradient rows and its first
// children are requested together; g~ and then the weights of its actions pass
// through LDS, a lane's own column.  Per hand the operations and their order are
// those above.
template <class TG, int HP>
__global__ __launch_bounds__(kPassThreads, HP == 2 ? 4 : 7) void bottom_up_wide_kernel(PassSet a) {
  typedef TG VH __attribute__((ext_vector_type(HP)));
  typedef double DH __attribute__((ext_vector_type(HP)));
  constexpr int kRows = 4, kChildBatch = 8;
  extern __shared__ double wide_rows[];  // [actions][64] DH: g~, then the weights; a lane's own column
  DH* row = (DH*)wide_rows + threadIdx.x;
  int y = blockIdx.y, k = 0;
  while (k < a.count - 1 && y >= a.level_cnt[k]) {
    y -= a.level_cnt[k];
    ++k;
  }
  const TreePass& t = a.t[k];
  const int h = HP * (blockIdx.x * kPassThreads + threadIdx.x);
  if (h >= a.n) return;
  const bool both = HP == 2 && h + 1 < a.n;
  const size_t ld = a.ld;
  const int v = t.level_begin[a.level] + y;
  const LevelTabLayout L = level_tab_layout(t.P.n_nodes, t.P.n_seq);
  const unsigned char* tab = (const unsigned char*)t.P.level_tab;
  const int4 r = ((const int4*)(tab + L.rec))[v];
  const double2 p0 = ((const double2*)(tab + L.prm))[2 * v], p1 = ((const double2*)(tab + L.prm))[2 * v + 1];
  const int s0 = r.x, na = r.y;
  const int* cend = (const int*)(tab + L.cbeg) + s0 + 1;
  const TG* gA = (const TG*)t.gA + (size_t)s0 * ld + h;
  const TG* gB = t.gB ? (const TG*)t.gB + (size_t)s0 * ld + h : nullptr;
  TG* g_out = t.g_out ? (TG*)t.g_out + (size_t)s0 * ld + h : nullptr;
  auto store = [&](auto* p, const DH& x) {
    if constexpr (HP == 2)
      store_pair(p, x[0], x[1], both);
    else
      p[0] = (std::remove_pointer_t<decltype(p)>)x[0];
  };
  const int c_first = cend[-1], c_last = cend[na - 1];
  const double* Vc = t.V + h;
  DH cv[kChildBatch];
  auto load_children = [&](int c) {
#pragma unroll
    for (int u = 0; u < kChildBatch; ++u)
      if (c + u < c_last) cv[u] = *(const DH*)(Vc + (size_t)(c + u) * ld);
  };
  load_children(c_first);
  for (int j = 0; j < na; j += kRows) {
    VH A[kRows], B[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      if (j + u < na) {
        A[u] = *(const VH*)(gA + (size_t)(j + u) * ld);
        if (gB) B[u] = *(const VH*)(gB + (size_t)(j + u) * ld);
      }
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      if (j + u < na) {
        DH x;
#pragma unroll
        for (int e = 0; e < HP; ++e)
          x[e] = gB ? lin2(t.cA, (double)A[u][e], t.cB, (double)B[u][e]) : t.cA * (double)A[u][e];
        if (g_out) {
          store(g_out + (size_t)(j + u) * ld, x * t.g_scale);
#pragma unroll
          for (int e = 0; e < HP; ++e) x[e] = (double)(TG)x[e];  // continue with the stored gradient (g_scale = +-1)
        }
        row[(j + u) * kPassThreads] = x;
      }
  }
  // the children of all actions are consecutive value slots: added one after
  // the other, on to the next action where an action's end
  DH x = row[0], m = (DH)INFINITY;
  int j = 0, end = cend[0];
  auto close = [&]() {  // action j is complete
    row[j * kPassThreads] = x;
#pragma unroll
    for (int e = 0; e < HP; ++e) m[e] = fmin(m[e], x[e]);
    if (++j < na) {
      x = row[j * kPassThreads];
      end = cend[j];
    }
  };
  for (int c = c_first; c < c_last; c += kChildBatch) {
    if (c > c_first) load_children(c);
#pragma unroll
    for (int u = 0; u < kChildBatch; ++u)
      if (c + u < c_last) {
        while (c + u >= end) close();
        x += cv[u];
      }
  }
  while (j < na) close();
  double* Vrow = t.V + (size_t)r.z * ld + h;
  if (!(t.mu > 0.0)) {
    store(Vrow, m);
    return;
  }
  const double temp = t.mu * p0.x, itemp = temp_inverse<TG>(temp);
  DH sum = (DH)0.0;
  for (int i = 0; i < na; ++i) {
    DH w = row[i * kPassThreads];
#pragma unroll
    for (int e = 0; e < HP; ++e) w[e] = lse_weight_by_inverse<TG>(m[e], w[e], temp, itemp);
    row[i * kPassThreads] = w;
    sum += w;
  }
  DH val;
#pragma unroll
  for (int e = 0; e < HP; ++e) val[e] = lse_value(m[e], temp, sum[e], p1.x);
  store(Vrow, val);
  if (t.QB) {
    DH rs;
#pragma unroll
    for (int e = 0; e < HP; ++e) rs[e] = inv_or_zero<TG>(sum[e]);
    TG* QB = (TG*)t.QB + (size_t)s0 * ld + h;
#pragma unroll 2
    for (int i = 0; i < na; ++i) {
      DH w = row[i * kPassThreads];
#pragma unroll
      for (int e = 0; e < HP; ++e) w[e] = qbar<TG>(w[e], sum[e], rs[e]);
      store(QB + (size_t)i * ld, w);
    }
  }
}

// Root sums of the level path (rows of n slots, n <= 2048): the hands are dealt
// to 256 places h mod 256, a place adds root by root with h ascending; 64 places
// are then added by halves, and the four sums in order.  That order is the
// result's definition.  By itself the sum of one root of 1081 hands took 4.5 us,
// nearly all of it the launch, so it rides on the first blocks of a top-down
// pass where there is one.
struct RootSum {
  const double* rows;  // the first root's values
  double* out;
  int n_roots;
};
struct RootSums {
  RootSum job[kMaxTrees];
  int count, n, ld;
};
// The sum of 64 places, from place 64 w on, in lane 0.
__device__ inline double root_sum_quarter(const RootSum& r, int n, int ld, int w, int lane) {
  constexpr int kBatch = 8;  // loads in flight: the place's hands of one root, then the next root's
  const int steps = (n + 255) / 256, total = r.n_roots * steps;
  const int h0 = kPassThreads * w + lane;
  double s = 0.0;
  int q = 0, m = 0;  // root and step of the next load
  for (int i = 0; i < total; i += kBatch) {
    double v[kBatch];
    bool in[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int h = h0 + 256 * m;
      in[u] = i + u < total && h < n;
      v[u] = in[u] ? r.rows[(size_t)q * ld + h] : 0.0;
      if (++m == steps) {
        m = 0;
        ++q;
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (in[u]) s += v[u];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  return s;
}
// The sum by the block's first four wavefronts (256 threads).
__device__ inline void root_sum(const RootSum& r, int n, int ld, int w, int lane) {
  __shared__ double part[4];
  const double s = root_sum_quarter(r, n, ld, w, lane);
  if (lane == 0) part[w] = s;
  __syncthreads();
  if (w == 0 && lane == 0) *r.out = ((part[0] + part[1]) + part[2]) + part[3];
}

__global__ __launch_bounds__(kPassThreads * kDownWaves) void root_sums_kernel(RootSums a) {
  root_sum(a.job[blockIdx.x], a.n, a.ld, (int)threadIdx.y, (int)threadIdx.x);
}

// out[k] = sum of partial[k][0 .. nb) in order, block k = tree k.  The order of
// the additions is the result's definition, so one lane adds; what the launch
// took was that lane's loads, one round trip each (272 partials of 1081 hands:
// 20 us).  All partials are loaded at once into LDS and the chain reads them
// from there (2.6 us).
__global__ __launch_bounds__(256) void sum_partials_kernel(const double* partial, int nb, double* out) {
  __shared__ double part[kMaxPartials];
  const double* p = partial + (size_t)blockIdx.x * nb;
  for (int b = threadIdx.x; b < nb; b += 256) part[b] = p[b];
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = sum_in_order(part, nb);
}

// ---------------------------------------------------------------------------
// Top-down pass of the level path: q[s] = q_bar[root] * ... * q_bar[s] along
// the sequence's path, multiplied from the root down, then the epilogue
// comb = (1 - tau) x_prev + tau q.  Padding slots are written 0.
//
// One wavefront per (up to kDownRows sequences of a node, 64 x HP hands), HP the
// hands of a 16-byte access: the sequences of a node share the path above them,
// so its product is formed once and every sequence costs its own row (on a large
// tree, a wavefront per sequence spent its time on instructions, 149 vector and 117
// scalar ones for three or four products; a wavefront per node left those of
// ten actions to four rounds of loads: 33.8 us with the epilogue).  The path (root
// first) and the item are wavefront-uniform loads, and every row of the item and
// of the first kPathStep ancestors is in flight before the first product.  Bound by
// memory: 5938 sequences x 1081 hands, 102 MB, 21.8 -> 18.9 us with the root sums
// (18.1 -> 11.0 in FP32, which read 8 bytes per lane); with the epilogue, 154 to
// 206 MB, 32 -> 29.0 us (with the compiler's own 80 registers, 6 wavefronts per
// SIMD instead of 8: 19.7, 12.1 and 29.4).
// ---------------------------------------------------------------------------
struct DownArgs {
  const int* anc;
  int anc_stride;
  const int2* items;  // first sequence, sequences of one node; null: every sequence by itself
  const void* QB;
  int n, ld, n_items;
  void* q_out;
  const void* x_prev;
  double tau;
  void* comb_out;
  RootSums sums;  // root sums that ride along, on the grid's first blocks
};

template <class TS, int HP>
__global__ __launch_bounds__(kPassThreads * kDownWaves, 7) void top_down_kernel(DownArgs a) {
  typedef TS VH __attribute__((ext_vector_type(HP)));
  const TS* QB = (const TS*)a.QB;
  TS* q_out = (TS*)a.q_out;
  TS* comb_out = (TS*)a.comb_out;
  const TS* x_prev = (const TS*)a.x_prev;
  // (hand block, node) pairs in hand-block-major order, kDownWaves a block, dealt
  // to the XCDs in contiguous ranges: the blocks of one XCD share hand blocks,
  // so the ancestor rows are re-read from that XCD's L2
  const int n_sums = a.sums.count, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
  if ((int)blockIdx.x < n_sums) {
    root_sum(a.sums.job[blockIdx.x], a.sums.n, a.sums.ld, wave, (int)threadIdx.x);
    return;
  }
  const int pos = xcd_spread((int)blockIdx.x - n_sums, (int)gridDim.x - n_sums) * kDownWaves + wave;
  const int hb = pos / a.n_items;
  const int h = HP * (hb * kPassThreads + (int)threadIdx.x);
  if (h >= a.ld) return;  // ld is a multiple of HP
  const int2 item = a.items ? a.items[pos - hb * a.n_items] : make_int2(pos - hb * a.n_items, 1);
  const int s0 = item.x, rows = item.y;
  const size_t ld = a.ld, i0 = (size_t)s0 * ld + h;
  const int* path = a.anc + (size_t)s0 * a.anc_stride;
  VH own[kDownRows], xp[kDownRows];
#pragma unroll
  for (int u = 0; u < kDownRows; ++u)
    if (u < rows) {
      own[u] = *(const VH*)(QB + i0 + u * ld);
      if (comb_out) xp[u] = *(const VH*)(x_prev + i0 + u * ld);
    }
  VH above = (VH)(TS)1;
  for (int j = 0; j < a.anc_stride; j += kPathStep) {  // a multiple of kPathStep
    VH f[kPathStep];
    bool in[kPathStep];
#pragma unroll
    for (int u = 0; u < kPathStep; ++u) {
      const int q = path[j + u];  // s0 closes the path, -1 after it
      in[u] = q >= 0 && q != s0;
      if (in[u]) f[u] = *(const VH*)(QB + (size_t)q * ld + h);
    }
#pragma unroll
    for (int u = 0; u < kPathStep; ++u)
      if (in[u]) above *= f[u];
    if (!in[kPathStep - 1]) break;
  }
#pragma unroll
  for (int u = 0; u < kDownRows; ++u)
    if (u < rows) {
      const VH val = above * own[u];
      VH q, c;
#pragma unroll
      for (int e = 0; e < HP; ++e) {
        const bool live = h + e < a.n;
        q[e] = live ? val[e] : (TS)0;
        if (comb_out) c[e] = live ? (TS)(1.0 - a.tau) * xp[u][e] + (TS)a.tau * val[e] : (TS)0;
      }
      if (q_out) *(VH*)(q_out + i0 + u * ld) = q;
      if (comb_out) *(VH*)(comb_out + i0 + u * ld) = c;
    }
}

// The uniform point: q[s] = q[parent] / n for every sequence s of a node with n
// actions, from the root down along the sequence's root-first path.
struct UniformArgs {
  const int* anc;
  int anc_stride;
  const int* seq_nact;
  int n, ld;
  double* out;
};

__global__ __launch_bounds__(kPassThreads) void uniform_kernel(UniformArgs a) {
  const int h = blockIdx.x * kPassThreads + threadIdx.x;
  const int s = blockIdx.y;
  if (h >= a.ld) return;
  const int* path = a.anc + (size_t)s * a.anc_stride;
  double val = 1.0;
  for (int j = 0; j < a.anc_stride && path[j] >= 0; ++j) val = val / (double)a.seq_nact[path[j]];
  a.out[(size_t)s * a.ld + h] = h < a.n ? val : 0.0;
}

// max |X| into *out, which holds +0.0 beforehand.  |x| >= 0, so the bit
// patterns order as the values do; a NaN (positive after fabs) orders above
// every number and so reaches the result instead of being skipped.
__global__ __launch_bounds__(256) void max_abs_kernel(int64_t count, const double* X, unsigned long long* out) {
  __shared__ unsigned long long wmax[4];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  unsigned long long m = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(X[i]));
    m = b > m ? b : m;
  }
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(m, off);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) m = wmax[w] > m ? wmax[w] : m;
    atomicMax(out, m);
  }
}

__global__ __launch_bounds__(64) void zero_kernel(double* p) {
  if (threadIdx.x == 0) p[0] = 0.0;
}

template <class T>
__global__ __launch_bounds__(256) void axpby_kernel(int64_t count, double a, const T* X, double b, const T* Y,
                                                    T* out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const T ta = (T)a, tb = (T)b;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
    out[i] = Y ? ta * X[i] + tb * Y[i] : ta * X[i];
}

template <class TI, class TO>
__global__ __launch_bounds__(256) void convert_kernel(int64_t count, const TI* in, TO* out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) out[i] = (TO)in[i];
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

static void fill_pass_set(const egt_game* g, const Pass* p, int count, PassSet& a) {
  a.count = count;
  a.n = g->n;
  a.ld = g->ld;
  a.level = 0;
  for (int k = 0; k < kMaxTrees; ++k) {
    a.level_cnt[k] = 0;
    TreePass& t = a.t[k];
    if (k >= count) {
      t = a.t[0];
      continue;
    }
    const HostPlayer& hp = g->hp[p[k].player];
    t.P = g->dp[p[k].player];
    t.gA = p[k].gA;
    t.cA = p[k].cA;
    t.gB = p[k].gB;
    t.cB = p[k].cB;
    t.mu = p[k].mu;
    t.V = p[k].V;
    t.VB = p[k].VB;
    t.QB = p[k].QB;
    t.g_out = nullptr;
    t.g_scale = 0.0;
    t.n_levels = hp.n_levels;
    for (int l = 0; l <= kMaxDepth; ++l) {
      t.level_begin[l] = hp.level_begin[std::min(l, hp.n_levels)];
    }
  }
}

// Hand blocks of the fused pass: every slot of a row is in one; a general
// game's one live slot is a block of its own, which writes the padding too.
int fused_hblocks(const egt_game* g) { return g->fused_hands == 1 ? 1 : g->ld / g->fused_hands; }

int n_partials(const egt_game* g) { return g->fused_passes ? fused_hblocks(g) : 1; }

size_t fused_lds_bytes(int hands, int cap_nodes, int cap_seqs, bool dual) {
  const size_t seqs = (size_t)(cap_seqs + kFusedPad) * hands, nodes = (size_t)(cap_nodes + kFusedPad) * hands;
  return sizeof(double) * (dual ? 3 * seqs + 3 * nodes : 2 * seqs + 2 * nodes);
}

// The fused pass or a launch per level.  A block's time grows with the
// (sequence, hand) pairs K per thread, the level path's with its levels (four
// or five launches of at least 4 us each) until its launches fill the chip.
// Where the fused pass has a block for every compute unit and more, and in its
// one block of a general game, the paths meet near K = 3 (one step of EGT; 1081
// hands: 286 sequences 94 against 110 us, 520 sequences 158 against 127;
// general: 744 sequences 69 against 81 us, 936 sequences 84 against 92, 1240
// sequences 89 against 92); with blocks for part of the chip only, near K = 6
// (105 and 351 hands, 520 sequences: 82 against 96 and 86 against 105 us; 967
// sequences: 112 against 106 and 118 against 119).
bool fits_fused(const egt_game* g) {
  const int seqs = std::max(g->hp[0].n_seq, g->hp[1].n_seq), nodes = std::max(g->hp[0].n_nodes, g->hp[1].n_nodes);
  const bool part = g->fused_hands > 1 && 2 * fused_hblocks(g) <= g->n_cu;
  const int tasks = part ? kFusedTasks : 3;
  return seqs * g->fused_hands <= tasks * kFusedThreads &&
         fused_lds_bytes(g->fused_hands, nodes, seqs, false) <= (size_t)g->lds_per_block;
}

// 1, 2, 3 or 5 (sequence, hand) pairs per thread, the fewest that 512 threads
// allow; more than three only with four hands per block (fits_fused).
template <int HB, class TG>
static hipError_t fused_launch_hands(const FusedArgs& a, int pairs, dim3 grid, size_t lds, hipStream_t s) {
  const dim3 block((unsigned)std::min(kFusedThreads, std::max(256, (pairs + 63) / 64 * 64)));
  if (pairs > (HB == 4 ? kFusedTasks : 3) * kFusedThreads) return hipErrorInvalidValue;
  if (pairs <= kFusedThreads)
    hipLaunchKernelGGL((sbr_fused_kernel<HB, 1, TG>), grid, block, lds, s, a);
  else if (pairs <= 2 * kFusedThreads)
    hipLaunchKernelGGL((sbr_fused_kernel<HB, 2, TG>), grid, block, lds, s, a);
  else if (HB != 4 || pairs <= 3 * kFusedThreads)
    hipLaunchKernelGGL((sbr_fused_kernel<HB, 3, TG>), grid, block, lds, s, a);
  else if constexpr (HB == 4)
    hipLaunchKernelGGL((sbr_fused_kernel<HB, kFusedTasks, TG>), grid, block, lds, s, a);
  return hipGetLastError();
}

// All passes in one launch of the fused kernel.
template <class TG>
static hipError_t fused_launch(const egt_game* g, const Pass* p, int count, const Epilogue* epi, double* partial,
                               hipStream_t s) {
  const int hb = g->fused_hands;
  FusedArgs a;
  a.cap_nodes = std::max(g->hp[0].n_nodes, g->hp[1].n_nodes);
  a.cap_seqs = std::max(g->hp[0].n_seq, g->hp[1].n_seq);
  // dual passes inside the kernel when every pass is dual, every one is
  // smoothed and the extra LDS fits; otherwise each becomes a second tree
  // with mu = 0 after the others
  bool any_dual = false;
  bool in_kernel = fused_lds_bytes(hb, a.cap_nodes, a.cap_seqs, true) <= (size_t)g->lds_per_block;
  for (int k = 0; k < count; ++k) {
    any_dual = any_dual || p[k].VB;
    in_kernel = in_kernel && p[k].VB && p[k].mu > 0.0;
  }
  int nt = 0;
  auto add = [&](const Pass& q, double mu, const Epilogue& e) {
    const HostPlayer& hp = g->hp[q.player];
    FusedTree& t = a.t[nt++];
    t.seq = g->dp[q.player].seq_rec;
    t.node = g->dp[q.player].node_rec;
    t.gA = q.gA;
    t.gB = q.gB;
    t.x_prev = e.x_prev;
    t.q_out = e.q_out;
    t.comb_out = e.comb_out;
    t.g_out = e.g_out;
    t.qb_out = e.qb_out;
    t.cA = q.cA;
    t.cB = q.cB;
    t.mu = mu;
    t.tau = e.tau;
    t.g_scale = e.g_scale;
    t.S = hp.n_seq;
    t.N = hp.n_nodes;
    t.C = (int)hp.child.size();
    t.n_roots = (int)hp.roots.size();
    t.n_levels = hp.n_levels;
    t.n_leaf = hp.n_levels > 0 ? hp.level_begin[1] : 0;
    t.dual = in_kernel;
  };
  const Epilogue none{nullptr, nullptr, 0.0, nullptr, nullptr, 0.0};
  for (int k = 0; k < count; ++k) add(p[k], p[k].mu, epi ? epi[k] : none);
  for (int k = 0; any_dual && !in_kernel && k < count; ++k) {
    if (!p[k].VB) continue;
    if (nt >= kMaxTrees) return hipErrorInvalidValue;
    add(p[k], 0.0, none);
  }
  a.partial = partial;
  a.count = nt;
  a.n = g->n;
  a.ld = g->ld;
  a.n_hblocks = fused_hblocks(g);
  const dim3 grid((unsigned)(a.n_hblocks * nt));
  const size_t lds = fused_lds_bytes(hb, a.cap_nodes, a.cap_seqs, in_kernel);
  const int pairs = a.cap_seqs * hb;
  return hb == 4    ? fused_launch_hands<4, TG>(a, pairs, grid, lds, s)
         : hb == 16 ? fused_launch_hands<16, TG>(a, pairs, grid, lds, s)
                    : fused_launch_hands<1, TG>(a, pairs, grid, lds, s);
}

// A wavefront for every sequence while that is at most 16 per compute unit: there
// a part's rows one after the other take longer than their shared path saves
// (whole pass, parts against sequences: 967 sequences x 105 hands, 4 per unit, 19.8
// against 19.5 us; 520 x 1081, 18 per unit, 21.7 and 21.5; 5938 x 105, 23 per unit,
// 29.3 both, in FP32 25.4 and 25.7; 1684 x 595, 33 per unit, 30.8 and 31.2).
template <class TS, int HP>
static hipError_t top_down_launch(DownArgs a, int n_seq, int n_cu, hipStream_t s) {
  const int nbx = (a.ld / HP + kPassThreads - 1) / kPassThreads;
  if ((int64_t)nbx * n_seq <= 16 * (int64_t)n_cu) {
    a.items = nullptr;
    a.n_items = n_seq;
  }
  const dim3 grid((unsigned)(a.sums.count + (nbx * a.n_items + kDownWaves - 1) / kDownWaves));
  hipLaunchKernelGGL((top_down_kernel<TS, HP>), grid, dim3(kPassThreads, kDownWaves), 0, s, a);
  return hipGetLastError();
}

// Takes the root sums along (and clears the list) unless the tree is empty.
static hipError_t top_down(const egt_game* g, int player, const void* QB, void* q_out, const void* x_prev, double tau,
                           void* comb_out, hipStream_t s, Prec prec, RootSums& sums) {
  const DPlayer& P = g->dp[player];
  DownArgs a;
  a.anc = P.anc;
  a.anc_stride = P.anc_stride;
  a.items = P.down;
  a.QB = QB;
  a.n = g->n;
  a.ld = g->ld;
  a.q_out = q_out;
  a.x_prev = x_prev;
  a.tau = tau;
  a.comb_out = comb_out;
  a.n_items = P.n_down;
  if (a.n_items == 0) return hipSuccess;
  a.sums = sums;
  sums.count = 0;
  // the widest access of up to 16 bytes that every row allows
  const size_t elem = prec == kF32 ? sizeof(float) : sizeof(double);
  const uintptr_t bits = (uintptr_t)QB | (uintptr_t)q_out | (uintptr_t)x_prev | (uintptr_t)comb_out;
  auto fits = [&](int hands) { return g->ld % hands == 0 && bits % (hands * elem) == 0; };
  if (prec == kF32)
    return fits(4)   ? top_down_launch<float, 4>(a, P.n_seq, g->n_cu, s)
           : fits(2) ? top_down_launch<float, 2>(a, P.n_seq, g->n_cu, s)
                     : top_down_launch<float, 1>(a, P.n_seq, g->n_cu, s);
  return fits(2) ? top_down_launch<double, 2>(a, P.n_seq, g->n_cu, s) : top_down_launch<double, 1>(a, P.n_seq, g->n_cu, s);
}

template <class TG>
static hipError_t passes_launch(const egt_game* g, const Pass* p, int count, const Epilogue* epi, double* partial,
                                hipStream_t s) {
  if (g->fused_passes) return fused_launch<TG>(g, p, count, epi, partial, s);
  bool any_dual = false;
  for (int k = 0; k < count; ++k) any_dual = any_dual || p[k].VB != nullptr;
  PassSet a;
  fill_pass_set(g, p, count, a);
  for (int k = 0; k < count; ++k) {
    if (epi && (epi[k].q_out || epi[k].comb_out) && !p[k].QB) return hipErrorInvalidValue;
    a.t[k].g_out = epi ? epi[k].g_out : nullptr;
    a.t[k].g_scale = epi ? epi[k].g_scale : 0.0;
  }
  int max_levels = 0;
  for (int k = 0; k < count; ++k) max_levels = std::max(max_levels, a.t[k].n_levels);
  const unsigned bx = (unsigned)((g->n + kPassThreads - 1) / kPassThreads);
  const unsigned bx_pair = (unsigned)(((g->n + 1) / 2 + kPassThreads - 1) / kPassThreads);
  // two hands per lane when every row is 2-element aligned
  bool pair = g->ld % 2 == 0;
  {
    const size_t pb = 2 * (std::is_same<TG, float>::value ? sizeof(float) : sizeof(double));
    auto ok = [&](const void* ptr) { return ((uintptr_t)ptr % pb) == 0; };
    for (int k = 0; k < count; ++k) {
      const TreePass& t = a.t[k];
      pair = pair && ok(t.gA) && ok(t.gB) && ok(t.g_out) && ok(t.QB) && ((uintptr_t)t.V % 16) == 0 &&
             ((uintptr_t)t.VB % 16) == 0;
    }
  }
  // Dual passes: the lowest level takes the best response with the smoothed
  // pass (the same minimum); above it the best responses run as trees of
  // their own (mu = 0, node values in VB, their children's values read from
  // there), after the given ones in the same launches.
  PassSet ax = a;
  if (any_dual) {
    int nx = count;
    for (int k = 0; k < count; ++k) {
      ax.t[k].VB = nullptr;
      if (!p[k].VB) continue;
      if (nx >= kMaxTrees) return hipErrorInvalidValue;
      TreePass& b = ax.t[nx++];
      b = a.t[k];
      b.mu = 0.0;
      b.V = p[k].VB;
      b.VB = nullptr;
      b.QB = nullptr;
      b.g_out = nullptr;
      b.g_scale = 0.0;
    }
    ax.count = nx;
  }
  for (int l = 0; l < max_levels; ++l) {
    PassSet& cur = l == 0 ? a : ax;
    unsigned total = 0;
    for (int k = 0; k < cur.count; ++k) {
      const TreePass& t = cur.t[k];
      cur.level_cnt[k] = l < t.n_levels ? t.level_begin[l + 1] - t.level_begin[l] : 0;
      total += (unsigned)cur.level_cnt[k];
    }
    if (total == 0) continue;
    cur.level = l;
    // Two hands per lane from 16 (node, 128 hands) wavefronts per compute unit on.
    // Below, a pass with exponentials is faster with one hand per lane, whose
    // actions all stay in registers (whole pass, two against one: 315 nodes x 105
    // hands 21.9 against 19.8 us, in FP32 19.2 and 18.0; 168 nodes x 1081 hands,
    // 6 per unit, 23.1 and 21.7, FP32 19.6 and 19.2; 949 nodes x 595 hands, 19 per
    // unit, 35.0 and 33.8, FP32 28.0 and 28.3; 1777 nodes x 1081 hands, 62 per unit,
    // 69.4 and 69.2, FP32 52.3 and 54.4).  Best responses only load and compare: two
    // hands are the faster form at every size (15.1 against 17.3 us at the first).
    bool smooth = true;
    for (int k = 0; k < count; ++k) smooth = smooth && a.t[k].mu > 0.0;
    if (l == 0 && pair && (!smooth || (size_t)bx_pair * total >= 16 * (size_t)g->n_cu)) {
      int more = 0;  // actions beyond the registers
      for (int k = 0; k < count; ++k)
        if (a.t[k].n_levels > 0) more = std::max(more, g->hp[p[k].player].level_max_act[0] - kLeafRegs);
      hipLaunchKernelGGL(bottom_up_leaf_pair_kernel<TG>, dim3(bx_pair, total), dim3(kPassThreads),
                         (size_t)more * kPassThreads * sizeof(double2), s, a);
    } else if (l == 0) {
      hipLaunchKernelGGL(bottom_up_level_kernel<TG>, dim3(bx, total), dim3(kPassThreads), 0, s, a);
    } else {
      // above the lowest level every node has children
      int max_act = 1;
      for (int k = 0; k < count; ++k)
        if (l < a.t[k].n_levels) max_act = std::max(max_act, g->hp[p[k].player].level_max_act[l]);
      const size_t row = kPassThreads * sizeof(double) * (size_t)max_act;
      const int wa = std::min(max_act, kInternalWaves);  // a wavefront takes actions j, j + wa, ... beyond that
      // A wavefront per node once the level has 8 (node, 64 hands) pairs for every
      // compute unit: there a wavefront per action waits at its barriers in a second
      // round of blocks (195 nodes x 1081 hands, 13 per unit: 17.2 -> 16.5 us, in FP32
      // 14.2 -> 12.0); below, a node's children and exponentials one after the other
      // take longer (61 nodes x 1081 hands, 4 per unit: one step of EGT 209 against 214
      // us; 51 nodes of ten actions: 289 against 304).  With 32 and more, two hands per lane
      // (780 nodes, four trees, 52 per unit: 39.0 -> 32.9 us).
      if (pair && (size_t)bx * total >= 32 * (size_t)g->n_cu)
        hipLaunchKernelGGL((bottom_up_wide_kernel<TG, 2>), dim3(bx_pair, total), dim3(kPassThreads), 2 * row, s, ax);
      else if ((size_t)bx * total >= 8 * (size_t)g->n_cu)
        hipLaunchKernelGGL((bottom_up_wide_kernel<TG, 1>), dim3(bx, total), dim3(kPassThreads), row, s, ax);
      else
        hipLaunchKernelGGL(bottom_up_internal_kernel<TG>, dim3(bx, total), dim3(kPassThreads, wa), 0, s, ax);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  RootSums sums;
  sums.count = 0;
  sums.n = g->n;
  sums.ld = g->ld;
  for (int k = 0; partial && k < ax.count; ++k) {
    const TreePass& t = ax.t[k];
    // the r-th root's value slot follows the children's
    sums.job[sums.count++] = RootSum{t.V + (size_t)(t.P.n_nodes - t.P.n_roots) * g->ld, partial + k, t.P.n_roots};
  }
  for (int k = 0; epi && k < count; ++k) {
    if (!epi[k].q_out && !epi[k].comb_out) continue;
    const hipError_t e = top_down(g, p[k].player, p[k].QB, epi[k].q_out, epi[k].x_prev, epi[k].tau, epi[k].comb_out, s,
                                  std::is_same<TG, float>::value ? kF32 : kF64, sums);
    if (e != hipSuccess) return e;
  }
  if (sums.count) {  // no top-down pass took them
    hipLaunchKernelGGL(root_sums_kernel, dim3(sums.count), dim3(kPassThreads, kDownWaves), 0, s, sums);
    return hipGetLastError();
  }
  return hipSuccess;
}

hipError_t launch_passes(const egt_game* g, const Pass* p, int count, const Epilogue* epi, double* partial,
                         hipStream_t s, Prec prec) {
  if (count < 1 || count > kMaxTrees) return hipErrorInvalidValue;
  return prec == kF32 ? passes_launch<float>(g, p, count, epi, partial, s)
                      : passes_launch<double>(g, p, count, epi, partial, s);
}

hipError_t launch_sum_partials(const egt_game* g, const double* partial, int count, double* out, hipStream_t s) {
  hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)count), dim3(256), 0, s, partial, n_partials(g), out);
  return hipGetLastError();
}

hipError_t launch_value(const egt_game* g, const Pass& p, const Epilogue* epi, double* scratch, double* value_out,
                        hipStream_t s, Prec prec) {
  // one partial: it is the value (a sum that started from 0)
  const bool direct = !value_out || n_partials(g) == 1;
  const hipError_t e = launch_passes(g, &p, 1, epi, direct ? value_out : scratch, s, prec);
  if (e != hipSuccess || direct) return e;
  return launch_sum_partials(g, scratch, 1, value_out, s);
}

hipError_t launch_top_down(const egt_game* g, int player, const void* QB, void* q_out, const void* x_prev,
                           double tau, void* comb_out, hipStream_t s, Prec prec) {
  RootSums none;
  none.count = 0;
  return top_down(g, player, QB, q_out, x_prev, tau, comb_out, s, prec, none);
}

hipError_t launch_uniform(const egt_game* g, int player, double* out, hipStream_t s) {
  UniformArgs a;
  a.anc = g->dp[player].anc;
  a.anc_stride = g->dp[player].anc_stride;
  a.seq_nact = g->dp[player].seq_nact;
  a.n = g->n;
  a.ld = g->ld;
  a.out = out;
  if (g->dp[player].n_seq == 0) return hipSuccess;
  const unsigned bx = (unsigned)((g->ld + kPassThreads - 1) / kPassThreads);
  hipLaunchKernelGGL(uniform_kernel, dim3(bx, g->dp[player].n_seq), dim3(kPassThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_axpby(int64_t count, double a, const void* X, double b, const void* Y, void* out, hipStream_t s,
                        Prec prec) {
  if (count <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<int64_t>((count + 255) / 256, 4096);
  if (prec == kF32)
    hipLaunchKernelGGL(axpby_kernel<float>, dim3(blocks), dim3(256), 0, s, count, a, (const float*)X, b,
                       (const float*)Y, (float*)out);
  else
    hipLaunchKernelGGL(axpby_kernel<double>, dim3(blocks), dim3(256), 0, s, count, a, (const double*)X, b,
                       (const double*)Y, (double*)out);
  return hipGetLastError();
}

hipError_t launch_convert(int64_t count, const void* in, Prec in_prec, void* out, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<int64_t>((count + 255) / 256, 4096);
  if (in_prec == kF32)
    hipLaunchKernelGGL((convert_kernel<float, double>), dim3(blocks), dim3(256), 0, s, count, (const float*)in,
                       (double*)out);
  else
    hipLaunchKernelGGL((convert_kernel<double, float>), dim3(blocks), dim3(256), 0, s, count, (const double*)in,
                       (float*)out);
  return hipGetLastError();
}

hipError_t launch_max_abs(int64_t count, const double* X, double* out, hipStream_t s) {
  hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(64), 0, s, out);
  const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>((count + 255) / 256, 2048));
  hipLaunchKernelGGL(max_abs_kernel, dim3(blocks), dim3(256), 0, s, count, X, (unsigned long long*)out);
  return hipGetLastError();
}

}  // namespace egt
