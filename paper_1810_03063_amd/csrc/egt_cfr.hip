// Counterfactual regret minimisation on the same payoff kernels: CFR with
// regret matching, CFR with regret matching+ and CFR+, the regret-based
// methods Section 7 compares EGT with (two gradient computations per
// iteration).
//
// Per player p and iteration, on p's loss gradient g (A y for player 1,
// -A^T x for player 2, computed by the product kernels):
//   bottom-up over the treeplex, one launch per level, one lane per
//   information set (node v, hand h) and its actions in order:
//     g~_a  = g[v, a] + sum of the values of a's child sets (betting order),
//     V[v]  = sum_a q_bar_a g~_a            (q_bar the current local strategy),
//     r_a   = V[v] - g~_a, or 0 within 1e-12 of |V[v]| + |g~_a| + S, S the
//             largest |g| entry (an exact tie, or actions no opponent mass
//             reaches, whose sign the products' rounding would otherwise
//             decide),
//     R_a  <- R_a + r_a                     (regret matching+: then max(R_a, 0)),
//     q_bar_a = max(R_a, 0) / sum_a' max(R_a', 0), or 1 / n_v when no R_a is positive;
//   top-down, x[s] = x[parent] q_bar[s] (the pass the smoothed best response uses).
// Both players update against the strategies of the same iteration (CFR,
// CFR(RM+)), or player 2 against player 1's new strategy (CFR+).  Before the
// update the current strategies join the averages, avg <- (1 - tau) avg +
// tau x_t with tau = w_t / sum_{t' <= t} w_t' (w_t = 1, or t under CFR+); the
// saddle gap of the averages is evaluated with the FP64 products and
// best-response passes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

#include "egt_device.h"
#include "egt_internal.h"

namespace egt {

namespace {

constexpr int kLanes = 64;

struct RegretArgs {
  const void* tab;  // the player's table image (LevelTabLayout)
  int n_nodes, n_seq;
  int node0;        // first node of the level
  int n, ld;
  const double* g;  // p's gradient (times gsign)
  double gsign;
  double* V;        // node values by value slot
  double* R;        // cumulative regrets [n_seq][ld]
  double* QB;       // local strategy [n_seq][ld], read then overwritten
  const double* gscale;  // max |g| over the real hands (device scalar)
  int plus;         // regret matching+
};

// *out = the largest of p[0 .. n), all >= 0.
__global__ __launch_bounds__(256) void max_kernel(const double* p, int n, double* out) {
  __shared__ double wmax[4];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) m = fmax(m, p[i]);
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) *out = fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3]));
}

__global__ __launch_bounds__(kLanes) void regret_level_kernel(RegretArgs a) {
  const int h = blockIdx.x * kLanes + threadIdx.x;
  if (h >= a.n) return;
  const int v = a.node0 + (int)blockIdx.y;
  const size_t ld = a.ld;
  const LevelTabLayout L = level_tab_layout(a.n_nodes, a.n_seq);
  const unsigned char* tab = (const unsigned char*)a.tab;
  const int4 r = ((const int4*)(tab + L.rec))[v];
  const int* cbeg = (const int*)(tab + L.cbeg);
  const int s0 = r.x, na = r.y;
  double gt[kMaxActions];
  double val = 0.0;
#pragma unroll
  for (int j = 0; j < kMaxActions; ++j) {
    if (j < na) {
      const size_t idx = (size_t)(s0 + j) * ld + h;
      double x = a.gsign * a.g[idx];
      const int c1 = cbeg[s0 + j + 1];
      for (int c = cbeg[s0 + j]; c < c1; ++c) x += a.V[(size_t)c * ld + h];
      gt[j] = x;
      val += a.QB[idx] * x;
    }
  }
  a.V[(size_t)r.z * ld + h] = val;
  const double S = *a.gscale;
  double pos[kMaxActions];
  double tot = 0.0;
#pragma unroll
  for (int j = 0; j < kMaxActions; ++j) {
    if (j < na) {
      const size_t idx = (size_t)(s0 + j) * ld + h;
      double r = val - gt[j];
      if (fabs(r) <= 1e-12 * (fabs(val) + fabs(gt[j]) + S)) r = 0.0;  // an exact tie
      double R = a.R[idx] + r;
      if (a.plus) R = fmax(R, 0.0);
      a.R[idx] = R;
      pos[j] = fmax(R, 0.0);
      tot += pos[j];
    }
  }
#pragma unroll
  for (int j = 0; j < kMaxActions; ++j)
    if (j < na) a.QB[(size_t)(s0 + j) * ld + h] = tot > 0.0 ? pos[j] / tot : 1.0 / (double)na;
}

// The whole update of one player in one launch, for trees that take the fused
// smoothed best response: block = HB hands, a thread per (sequence, hand), up to
// K of them, and per (node, hand).  The averages' update and the top-down pass
// go with it.  What it replaces were 8 dependent launches of 4 to 9 us each per
// player on the 223-sequence tree of 1081 hands: an iteration of CFR+ (two products and
// two updates) 120 -> 44 us, this launch 11 us.
//   1. records, gradient, regrets, q_bar, the old strategy and the average of
//      the thread's sequences, all loads in flight together; the average takes
//      the old strategy;
//   2. per level: g~ and q_bar g~ (to LDS), then per node their sum in action
//      order, the node value;
//   3. regrets of every level at once, their positive parts (to LDS), per node
//      the sum in action order, the new q_bar;
//   4. top-down to the new strategy.
// Per element the operations are those of regret_level_kernel, the top-down
// pass and axpby, in their order.
struct RegretFusedArgs {
  const SeqRec* seq;
  const NodeRec* node;
  int S, N, n_levels, n, ld;
  int cap;  // LDS rows of the sequences
  const double* g;
  double gsign;
  double* R;
  double* QB;
  double* X;
  double* AVG;
  double tau;
  const double* gmax;  // [n_gmax] largest |g| of each block of the product
  int n_gmax;
  int plus;
};

template <int HB, int K>
__global__ __launch_bounds__(kFusedThreads, K <= 2 ? 8 : K <= 3 ? 6 : 4) void regret_fused_kernel(RegretFusedArgs a) {
  extern __shared__ __align__(16) double lds[];
  __shared__ double wmax[kFusedThreads / 64];
  const int S = a.S, N = a.N, n = a.n, n_levels = a.n_levels;
  double* Wl = lds;                            // [seqs][HB] q_bar g~, then max(R, 0), then q
  double* Vs = Wl + (a.cap + kFusedPad) * HB;  // [nodes][HB] values by slot
  double* Tl = Vs + (N + kFusedPad) * HB;      // [nodes][HB] sums of max(R, 0) by slot
  const int tid = threadIdx.x, T = blockDim.x;
  const int h0 = xcd_spread((int)blockIdx.x, (int)gridDim.x) * HB;
  constexpr unsigned kNone = 0xffffu;
  unsigned child[K], par_slot[K];  // LDS indices: first child's slot and their number; parent and own slot
  int lev_na[K];                   // level (-1: no pair here), actions
  double gt[K], R[K], q[K];
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int j = u * T + tid, s = j / HB, hl = j % HB, h = h0 + hl;
    child[u] = par_slot[u] = 0u;
    lev_na[u] = -1;
    gt[u] = R[u] = q[u] = 0.0;
    if (s < S && h < n) {
      const size_t idx = (size_t)s * a.ld + h;
      const SeqRec r = a.seq[s];
      const double g = a.g[idx], x = a.X[idx], avg = a.AVG[idx];
      R[u] = a.R[idx];
      q[u] = a.QB[idx];
      a.AVG[idx] = (1.0 - a.tau) * avg + a.tau * x;
      gt[u] = a.gsign * g;
      child[u] = (unsigned)(r.c0 * HB + hl) | ((unsigned)r.n_child << 16);
      par_slot[u] = (r.parent >= 0 ? (unsigned)(r.parent * HB + hl) : kNone) | ((unsigned)(r.slot * HB + hl) << 16);
      lev_na[u] = (r.level << 8) | r.na;
    }
  }
  // The thread's first node stays in registers; a tree with more (node, hand)
  // pairs than threads reads the others' records when their level comes.
  struct Task {
    int level, na, at, slot;  // level -1: none here
  };
  const int n_tasks = N * HB;
  auto task_of = [&](int i) {
    Task d{-1, 0, 0, 0};
    if (i < n_tasks && h0 + i % HB < n) {
      const NodeRec r = a.node[i / HB];
      d = Task{r.level, r.na, r.first * HB + i % HB, r.slot * HB + i % HB};
    }
    return d;
  };
  const Task own = task_of(tid);
  {  // S, the largest |g|: the product's block maxima, met in LDS by the first barrier
    double m = 0.0;
    for (int i = tid; i < a.n_gmax; i += T) m = fmax(m, a.gmax[i]);
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if ((tid & 63) == 0) wmax[tid >> 6] = m;
  }
  for (int l = 0; l < n_levels; ++l) {
#pragma unroll
    for (int u = 0; u < K; ++u) {
      if ((lev_na[u] >> 8) != l) continue;
      const int c0 = (int)(child[u] & 0xffffu), cn = (int)(child[u] >> 16);
      if (cn > 0) gt[u] = add_run<HB>(gt[u], Vs + c0, cn);
      Wl[u * T + tid] = q[u] * gt[u];
    }
    __syncthreads();
    Task d = own;
#pragma unroll 1
    for (int i = tid;;) {
      if (d.level == l) Vs[d.slot] = add_run<HB>(0.0, Wl + d.at, d.na);
      if ((i += T) >= n_tasks) break;
      d = task_of(i);
    }
    __syncthreads();
  }
  double scale = 0.0;
  for (int v = 0; v < T / 64; ++v) scale = fmax(scale, wmax[v]);
#pragma unroll
  for (int u = 0; u < K; ++u) {
    if (lev_na[u] < 0) continue;
    const int j = u * T + tid;
    const double val = Vs[par_slot[u] >> 16];
    double r = val - gt[u];
    if (fabs(r) <= 1e-12 * (fabs(val) + fabs(gt[u]) + scale)) r = 0.0;  // an exact tie
    R[u] += r;
    if (a.plus) R[u] = fmax(R[u], 0.0);
    a.R[(size_t)(j / HB) * a.ld + h0 + j % HB] = R[u];
    Wl[j] = fmax(R[u], 0.0);
  }
  __syncthreads();
  {
    Task d = own;
#pragma unroll 1
    for (int i = tid;;) {
      if (d.level >= 0) Tl[d.slot] = add_run<HB>(0.0, Wl + d.at, d.na);
      if ((i += T) >= n_tasks) break;
      d = task_of(i);
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < K; ++u) {
    if (lev_na[u] < 0) continue;
    const int j = u * T + tid;
    const double tot = Tl[par_slot[u] >> 16];
    q[u] = tot > 0.0 ? Wl[j] / tot : 1.0 / (double)(lev_na[u] & 0xff);
    a.QB[(size_t)(j / HB) * a.ld + h0 + j % HB] = q[u];
    if (lev_na[u] >> 8 > 0) Wl[j] = q[u];  // the lowest level has no children
  }
  for (int l = n_levels - 2; l >= 0; --l) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const unsigned par = par_slot[u] & 0xffffu;
      if ((lev_na[u] >> 8) != l || par == kNone) continue;
      q[u] = Wl[par] * q[u];
      if (l > 0) Wl[u * T + tid] = q[u];
    }
  }
#pragma unroll
  for (int u = 0; u < K; ++u) {  // the padding stays as the first strategies have it
    const int j = u * T + tid;
    if (lev_na[u] >= 0) a.X[(size_t)(j / HB) * a.ld + h0 + j % HB] = q[u];
  }
}

// Uniform local strategy: q_bar = 1 / n_v on every action (0 in the padding).
__global__ __launch_bounds__(kLanes) void uniform_local_kernel(const int* seq_nact, int n, int ld, double* QB) {
  const int h = blockIdx.x * kLanes + threadIdx.x;
  if (h >= ld) return;
  const int s = blockIdx.y;
  QB[(size_t)s * ld + h] = h < n ? 1.0 / (double)seq_nact[s] : 0.0;
}

__global__ __launch_bounds__(256) void fill_kernel(double* p, int64_t count, double v) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = v;
}

}  // namespace

int64_t vec_elems_of(const egt_game* g, int p) { return (int64_t)g->hp[p].n_seq * g->ld; }

}  // namespace egt

struct egt_cfr {
  const egt_game* g = nullptr;
  int variant = EGT_CFR_PLUS;
  int64_t t = 0;
  double wsum = 0.0;
  double* R[2] = {};
  double* QB[2] = {};
  double* X[2] = {};    // current strategies x_t, y_t
  double* AVG[2] = {};  // averages
  double* G[2] = {};    // gradient scratch
  double* V[2] = {};    // node values
  double* Vb[2] = {};   // node values of the gap's best responses
  double* part = nullptr;    // device partial sums [2][kMaxPartials]
  double* scal = nullptr;    // device sums [2]
  double* gmax[2] = {};      // device: the products' block maxima of |g| [absmax_capacity], and their largest (level path)
  double* gtop[2] = {};
  int n_gmax[2] = {0, 0};
  double* hscal = nullptr;   // pinned host copy
  void* block = nullptr;
};

using namespace egt;

namespace {

// Pairs per thread as in the fused smoothed best response.
template <int HB>
hipError_t launch_regret_fused(const RegretFusedArgs& a, dim3 grid, size_t lds, int pairs, hipStream_t s) {
  const dim3 block((unsigned)std::min(kFusedThreads, std::max(256, (pairs + 63) / 64 * 64)));
  if (pairs > (HB == 4 ? kFusedTasks : 3) * kFusedThreads) return hipErrorInvalidValue;
  if (pairs <= kFusedThreads)
    hipLaunchKernelGGL((regret_fused_kernel<HB, 1>), grid, block, lds, s, a);
  else if (pairs <= 2 * kFusedThreads)
    hipLaunchKernelGGL((regret_fused_kernel<HB, 2>), grid, block, lds, s, a);
  else if (HB != 4 || pairs <= 3 * kFusedThreads)
    hipLaunchKernelGGL((regret_fused_kernel<HB, 3>), grid, block, lds, s, a);
  else if constexpr (HB == 4)
    hipLaunchKernelGGL((regret_fused_kernel<HB, kFusedTasks>), grid, block, lds, s, a);
  return hipGetLastError();
}

// One update of player p; its current strategy joins the average with
// weight tau first.
int cfr_update(egt_cfr* c, int p, double tau, hipStream_t s) {
  const egt_game* g = c->g;
  const HostPlayer& hp = g->hp[p];
  if (g->fused_passes) {  // the trees of the fused smoothed best response, by the same measure
    const int hb = g->fused_hands, pairs = hp.n_seq * hb;
    RegretFusedArgs a;
    a.seq = g->dp[p].seq_rec;
    a.node = g->dp[p].node_rec;
    a.S = a.cap = hp.n_seq;
    a.N = hp.n_nodes;
    a.n_levels = hp.n_levels;
    a.n = g->n;
    a.ld = g->ld;
    a.g = c->G[p];
    a.gsign = p == 0 ? 1.0 : -1.0;
    a.R = c->R[p];
    a.QB = c->QB[p];
    a.X = c->X[p];
    a.AVG = c->AVG[p];
    a.tau = tau;
    a.gmax = c->gmax[p];
    a.n_gmax = c->n_gmax[p];
    a.plus = c->variant != EGT_CFR_RM;
    const size_t lds = sizeof(double) * (size_t)hb * ((size_t)hp.n_seq + 2 * (size_t)hp.n_nodes + 3 * kFusedPad);
    const dim3 grid((unsigned)fused_hblocks(g));
    EGT_HIP(hb == 4    ? launch_regret_fused<4>(a, grid, lds, pairs, s)
            : hb == 16 ? launch_regret_fused<16>(a, grid, lds, pairs, s)
                       : launch_regret_fused<1>(a, grid, lds, pairs, s));
    return EGT_OK;
  }
  EGT_HIP(launch_axpby(vec_elems_of(g, p), 1.0 - tau, c->AVG[p], tau, c->X[p], c->AVG[p], s));
  const unsigned bx = (unsigned)((g->n + kLanes - 1) / kLanes);
  RegretArgs a;
  a.tab = g->dp[p].level_tab;
  a.n_nodes = hp.n_nodes;
  a.n_seq = hp.n_seq;
  a.n = g->n;
  a.ld = g->ld;
  a.g = c->G[p];
  a.gsign = p == 0 ? 1.0 : -1.0;
  a.V = c->V[p];
  a.R = c->R[p];
  a.QB = c->QB[p];
  a.plus = c->variant != EGT_CFR_RM;
  a.gscale = c->gtop[p];
  hipLaunchKernelGGL(max_kernel, dim3(1), dim3(256), 0, s, (const double*)c->gmax[p], c->n_gmax[p], c->gtop[p]);
  EGT_HIP(hipGetLastError());
  for (int l = 0; l < hp.n_levels; ++l) {
    a.node0 = hp.level_begin[l];
    const int cnt = hp.level_begin[l + 1] - hp.level_begin[l];
    if (cnt == 0) continue;
    hipLaunchKernelGGL(regret_level_kernel, dim3(bx, (unsigned)cnt), dim3(kLanes), 0, s, a);
    EGT_HIP(hipGetLastError());
  }
  EGT_HIP(launch_top_down(g, p, c->QB[p], c->X[p], nullptr, 0.0, nullptr, s));
  return EGT_OK;
}

int cfr_iteration(egt_cfr* c, hipStream_t s) {
  const egt_game* g = c->g;
  const int64_t t = c->t + 1;
  const double w = c->variant == EGT_CFR_PLUS ? (double)t : 1.0;
  c->wsum += w;
  const double tau = w / c->wsum;
  auto product = [&](int p) {
    return launch_gradient(g, p, c->X[1 - p], c->G[p], s, c->gmax[p], &c->n_gmax[p]);
  };
  // player 1 against y_t; player 2 against x_t (simultaneous) or x_{t+1} (CFR+)
  EGT_HIP(product(0));
  if (c->variant != EGT_CFR_PLUS) EGT_HIP(product(1));
  int rc = cfr_update(c, 0, tau, s);
  if (rc) return rc;
  if (c->variant == EGT_CFR_PLUS) EGT_HIP(product(1));
  rc = cfr_update(c, 1, tau, s);
  if (rc) return rc;
  c->t = t;
  return EGT_OK;
}

// Saddle gap of the averages: FP64 products and best responses.
int cfr_gap(egt_cfr* c, double* gap, double* brmax, double* brmin, hipStream_t s) {
  const egt_game* g = c->g;
  EGT_HIP(launch_gradient(g, 0, c->AVG[1], c->G[0], s));
  EGT_HIP(launch_gradient(g, 1, c->AVG[0], c->G[1], s));
  const Pass ps[2] = {{0, c->G[0], 1.0, nullptr, 0.0, 0.0, c->Vb[0], nullptr},
                      {1, c->G[1], -1.0, nullptr, 0.0, 0.0, c->Vb[1], nullptr}};
  EGT_HIP(launch_passes(g, ps, 2, nullptr, c->part, s));
  EGT_HIP(launch_sum_partials(g, c->part, 2, c->scal, s));
  EGT_HIP(hipMemcpyAsync(c->hscal, c->scal, 2 * sizeof(double), hipMemcpyDeviceToHost, s));
  EGT_HIP(hipStreamSynchronize(s));
  if (!std::isfinite(c->hscal[0]) || !std::isfinite(c->hscal[1]))
    return fail(EGT_ENUMERIC, "non-finite value in the CFR gap");
  if (gap) *gap = -c->hscal[1] - c->hscal[0];
  if (brmax) *brmax = -c->hscal[1];
  if (brmin) *brmin = c->hscal[0];
  return EGT_OK;
}

}  // namespace

extern "C" {

int egt_cfr_create(const egt_game* g, int32_t variant, hipStream_t s, egt_cfr** out) {
  if (!g || !out) return fail(EGT_EINVAL, "null argument");
  *out = nullptr;
  if (variant != EGT_CFR_RM && variant != EGT_CFR_RMPLUS && variant != EGT_CFR_PLUS)
    return fail(EGT_EINVAL, "unknown CFR variant");
  std::unique_ptr<egt_cfr> c(new (std::nothrow) egt_cfr());
  if (!c) return fail(EGT_ENOMEM, "host allocation failed");
  c->g = g;
  c->variant = variant;
  size_t bytes = 0;
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  for (int p = 0; p < 2; ++p) {
    bytes += 5 * al(sizeof(double) * (size_t)vec_elems_of(g, p));
    bytes += 2 * al(sizeof(double) * (size_t)g->hp[p].n_nodes * g->ld);
  }
  bytes += al(sizeof(double) * 2 * kMaxPartials) + al(2 * sizeof(double)) +
           2 * (al(sizeof(double) * (size_t)absmax_capacity(g)) + al(sizeof(double)));
  hipError_t e = hipMalloc(&c->block, bytes);
  if (e != hipSuccess) return fail(EGT_ENOMEM, std::string("hipMalloc (CFR state): ") + hipGetErrorString(e));
  e = hipHostMalloc((void**)&c->hscal, 2 * sizeof(double), hipHostMallocDefault);
  if (e != hipSuccess) {
    (void)hipFree(c->block);
    return fail(EGT_ENOMEM, std::string("hipHostMalloc (CFR state): ") + hipGetErrorString(e));
  }
  unsigned char* cur = (unsigned char*)c->block;
  auto take = [&](size_t nb) {
    void* r = cur;
    cur += al(nb);
    return (double*)r;
  };
  for (int p = 0; p < 2; ++p) {
    const size_t vb = sizeof(double) * (size_t)vec_elems_of(g, p);
    c->R[p] = take(vb);
    c->QB[p] = take(vb);
    c->X[p] = take(vb);
    c->AVG[p] = take(vb);
    c->G[p] = take(vb);
    c->V[p] = take(sizeof(double) * (size_t)g->hp[p].n_nodes * g->ld);
    c->Vb[p] = take(sizeof(double) * (size_t)g->hp[p].n_nodes * g->ld);
  }
  c->part = take(sizeof(double) * 2 * kMaxPartials);
  c->scal = take(2 * sizeof(double));
  for (int p = 0; p < 2; ++p) {
    c->gmax[p] = take(sizeof(double) * (size_t)absmax_capacity(g));
    c->gtop[p] = take(sizeof(double));
  }
  // zero regrets, uniform local strategies, x_1 = the uniform point, avg = x_1
  for (int p = 0; p < 2; ++p) {
    const int64_t cnt = vec_elems_of(g, p);
    const unsigned fb = (unsigned)std::min<int64_t>((cnt + 255) / 256, 4096);
    if (cnt > 0) hipLaunchKernelGGL(fill_kernel, dim3(fb), dim3(256), 0, s, c->R[p], cnt, 0.0);
    const unsigned bx = (unsigned)((g->ld + kLanes - 1) / kLanes);
    if (g->hp[p].n_seq > 0)
      hipLaunchKernelGGL(uniform_local_kernel, dim3(bx, (unsigned)g->hp[p].n_seq), dim3(kLanes), 0, s,
                         g->dp[p].seq_nact, g->n, g->ld, c->QB[p]);
    EGT_HIP(hipGetLastError());
    EGT_HIP(launch_uniform(g, p, c->X[p], s));
    EGT_HIP(hipMemcpyAsync(c->AVG[p], c->X[p], sizeof(double) * (size_t)cnt, hipMemcpyDeviceToDevice, s));
  }
  EGT_HIP(hipStreamSynchronize(s));
  *out = c.release();
  return EGT_OK;
}

int egt_cfr_destroy(egt_cfr* c) {
  if (!c) return EGT_OK;
  int rc = EGT_OK;
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess && c->block) e = hipFree(c->block);
  if (e == hipSuccess && c->hscal) e = hipHostFree(c->hscal);
  if (e != hipSuccess) rc = hip_fail(e, "egt_cfr_destroy");
  delete c;
  return rc;
}

int egt_cfr_step(egt_cfr* c, int32_t iters, hipStream_t s) {
  if (!c || iters < 0) return fail(EGT_EINVAL, "null state or negative count");
  for (int32_t k = 0; k < iters; ++k) {
    const int rc = cfr_iteration(c, s);
    if (rc) return rc;
  }
  return EGT_OK;
}

int egt_cfr_gap(egt_cfr* c, double* gap, double* br_max_y, double* br_min_x, hipStream_t s) {
  if (!c) return fail(EGT_EINVAL, "null state");
  return cfr_gap(c, gap, br_max_y, br_min_x, s);
}

int egt_cfr_get(const egt_cfr* c, double* x_avg, double* y_avg, double* x_cur, double* y_cur, int64_t* iters,
                hipStream_t s) {
  if (!c) return fail(EGT_EINVAL, "null state");
  const egt_game* g = c->g;
  double* dst[4] = {x_avg, y_avg, x_cur, y_cur};
  const double* src[4] = {c->AVG[0], c->AVG[1], c->X[0], c->X[1]};
  for (int k = 0; k < 4; ++k)
    if (dst[k])
      EGT_HIP(hipMemcpyAsync(dst[k], src[k], sizeof(double) * (size_t)vec_elems_of(g, k % 2),
                             hipMemcpyDeviceToDevice, s));
  if (iters) *iters = c->t;
  return EGT_OK;
}

int egt_cfr_solve(const egt_game* g, int32_t variant, double eps, int64_t max_iters, int32_t gap_every,
                  egt_result* res, hipStream_t s) {
  if (!g || !res) return fail(EGT_EINVAL, "null argument");
  if (max_iters < 0) return fail(EGT_EINVAL, "max_iters < 0");
  std::memset(res, 0, sizeof(*res));
  if (eps <= 0) eps = 1e-3 * g->pot;
  if (gap_every < 1) gap_every = 1;
  const auto t0 = std::chrono::steady_clock::now();
  egt_cfr* c = nullptr;
  int rc = egt_cfr_create(g, variant, s, &c);
  if (rc) return rc;
  std::unique_ptr<egt_cfr, int (*)(egt_cfr*)> guard(c, egt_cfr_destroy);
  double gap = 0, brmax = 0, brmin = 0;
  bool converged = false;
  for (;;) {
    if ((rc = cfr_gap(c, &gap, &brmax, &brmin, s))) return rc;
    if (gap <= eps) {
      converged = true;
      break;
    }
    if (c->t >= max_iters) break;
    const int64_t k = std::min<int64_t>(gap_every, max_iters - c->t);
    if ((rc = egt_cfr_step(c, (int32_t)k, s))) return rc;
  }
  res->iters = c->t;
  res->products = 2 * c->t;
  res->gap = gap;
  res->br_max_y = brmax;
  res->br_min_x = brmin;
  res->converged = converged ? 1 : 0;
  // value of the averages: x_avg^T A y_avg with A y_avg from the last gap evaluation
  const int64_t n0 = vec_elems_of(g, 0);
  std::vector<double> hx((size_t)n0 * 2);
  EGT_HIP(hipMemcpyAsync(hx.data(), c->AVG[0], sizeof(double) * n0, hipMemcpyDeviceToHost, s));
  EGT_HIP(hipMemcpyAsync(hx.data() + n0, c->G[0], sizeof(double) * n0, hipMemcpyDeviceToHost, s));
  EGT_HIP(hipStreamSynchronize(s));
  double v = 0.0;
  for (int64_t i = 0; i < n0; ++i) v += hx[(size_t)i] * hx[(size_t)(n0 + i)];
  res->value_p1 = -v;
  res->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return converged ? EGT_OK : fail(EGT_ENOTCONV, "iteration cap reached before the target gap");
}

}  // extern "C"
