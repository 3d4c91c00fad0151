// Payoff products A y and A^T x (Section 2's gradient operators) on the fold
// and showdown terminals of a river endgame, O(n) per terminal, for gfx950;
// for a general game, a CSR SpMV over the explicit operator.
//
// For a terminal z with opponent sequence sigma_o(z) the opponent's reach is
// r(h') = b_o(h') v_o[sigma_o(z)][h'] over the strength-ordered hands, and
//   fold:     sum of r over hands compatible with h = T - C[a] - C[b] + r(h)
//             (T the total, C[c] the mass of the hands holding card c; hand h
//             holds both of its cards, so it is removed twice and added back);
//   showdown: (compatible mass stronger) - (compatible mass weaker): the
//             weaker mass is the exclusive prefix over strength order at the
//             start of h's tie group minus, per card of h, the exclusive
//             prefix over the strength-ordered hands holding that card; the
//             stronger mass mirrors it from the end of the tie group; hands of
//             the tie group count as neither.
// out[s][h] = b_own(h) / Z * sum over the terminals z at s of u(z) op_z(h),
// the showdown op negated for player 2 (W^T = -W).
//
// A block holds one or two wave groups of 256 threads; a group evaluates one
// terminal per round.  A round:
//   1. stage: each thread writes the reach of its strided hands into R (the
//      strength order) and into the hand's two slots of E, the card lists laid
//      end to end (card c's strength-ordered hands, then one slot for its
//      total), so every card list is contiguous in LDS;
//   2. the per-card exclusive prefixes, in place in E (four lanes per card,
//      each a contiguous quarter of the list, the quarter offsets added in a
//      fixed order), and beside them the strength-order scan of the group;
//   3. the exclusive strength prefix written in place over R;
//   4. every thread evaluates its contiguous hands from its own 16-byte
//      per-hand table of indices into R and E (kept in registers).
// While a round runs, the opponent row of the group's next round is already
// being loaded into registers, and the terminal record of the round after.  When blocks loop over many sequences they walk
// work items (TermItem): two-terminal sequences whole (one terminal per group,
// the two results added), one-terminal sequences in pairs (one per group).
// Every sum is taken in a fixed order, so results are bitwise repeatable.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "egt_internal.h"

namespace egt {

namespace {

constexpr int kGroupThreads = 256;  // one wave group evaluates one terminal per round
constexpr int kQR = 12;             // card-list quarters up to this long stay in registers

// A double moved across lanes by a DPP control (VALU, no LDS round trip);
// lanes whose source is out of range or whose row is masked get 0.
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_move(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Inclusive scan over the 64 lanes of a wavefront (every lane active): within
// each row of 16 lanes by shifts of 1, 2, 4, 8, then each row's total carried
// to the rows after it (row broadcasts of lanes 15 and 31).  The additions are
// fixed, so the result is repeatable.
__device__ inline double wave_inclusive_scan(double x) {
  x += dpp_move<0x111, 0xf>(x);  // row_shr:1
  x += dpp_move<0x112, 0xf>(x);  // row_shr:2
  x += dpp_move<0x114, 0xf>(x);  // row_shr:4
  x += dpp_move<0x118, 0xf>(x);  // row_shr:8
  x += dpp_move<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
  x += dpp_move<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}

// The largest x >= 0 over the wavefront, in every lane.
__device__ inline double wave_max(double x) {
  for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off));
  return x;
}

template <class TV, class TO>
struct ProdArgs {
  DPlayer own;
  const double* b_opp;
  DHands H;
  const TV* v_opp;
  TO* out;
  double show_sign;
  int groups;
  const TermItem* items;   // work items instead of whole sequences, or null
  int n_items;
  double* absmax;  // MAX: each block's largest |entry|
};

// HPT = hands per thread (n <= 256 HPT).  MINW = waves per SIMD the register
// allocation leaves room for (4: two blocks of two groups share a compute unit).
// TAB = the per-hand tables (index table, own prior) staged once per block in
// LDS behind the groups' arrays, which leaves the registers to the staging
// and the accumulators (used when the device's LDS per block allows it).
// MAX = also the block's largest |entry| (one store per block: atomics of every
// wavefront on one word took 19 us at 223 sequences).
template <class TV, class TO, int HPT, int MINW, bool TAB, bool MAX>
__global__ __launch_bounds__(2 * kGroupThreads, MINW) void product_kernel(ProdArgs<TV, TO> a) {
  extern __shared__ __align__(16) double lds[];
  __shared__ double wave_total[2][kGroupThreads / 64];
  const int n = a.H.n, ld = a.H.ld, cph = a.H.cph;
  const int groups = a.groups;
  const int rlen = (n + 2) / 2 * 2;            // R: n + 1 doubles, rounded up to keep E 16-byte aligned
  const int per_group = rlen + a.H.n_card_slots;
  const int tid = threadIdx.x;
  const int grp = tid / kGroupThreads, gt = tid % kGroupThreads;
  const int lane = tid & 63, wig = gt >> 6;
  double* R = lds + (size_t)grp * per_group;
  double* E = R + rlen;

  const int MT = a.own.term_stride, n_seq = a.own.n_seq;
  const int chunk = (n + kGroupThreads - 1) / kGroupThreads;
  const int beg = min(gt * chunk, n), end = min(beg + chunk, n), cnt = end - beg;
  const TermRec none{-1, -1, 0.0};
  const bool by_items = a.items != nullptr;
  const int n_work = by_items ? a.n_items : n_seq;
  const int rounds = by_items ? 1 : (MT + groups - 1) / groups;

  // the terminal of (unit w, round rd) for this group, and the row it writes
  auto term_of = [&](int w, int rd, TermRec& t, int& so, bool& comb) {
    if (by_items) {
      const TermItem& it = a.items[w];
      t = it.t[grp];
      so = it.seq[grp];
      comb = it.seq[0] == it.seq[1];
    } else {
      const int j = rd * groups + grp;
      t = j < MT ? a.own.term_rec[(size_t)w * MT + j] : none;
      so = w;
      comb = groups == 2;
    }
  };

  // per-thread constants, kept for every round: the indices of this thread's
  // own hands (16-bit fields: E index of the card-a prefix at the tie group's
  // start and end and of card a's total, the same for card b, then the tie
  // group [glo, ghi) in R), the opponent's prior at the strided hands it
  // stages, and those hands' two slots in E
  uint4 ht[TAB ? 1 : HPT];
  double bown[TAB ? 1 : HPT];
  double bo[HPT];
  unsigned hp[HPT];
  uint4* htab_l = (uint4*)(lds + ((size_t)groups * per_group + 1) / 2 * 2);  // TAB: [n], 16-byte aligned
  double* bown_l = (double*)(htab_l + n);                      // TAB: [n]
  if constexpr (TAB) {
    for (int i = tid; i < n; i += (int)blockDim.x) {
      htab_l[i] = a.H.htab[i];
      bown_l[i] = a.own.belief[i];
    }
  } else {
#pragma unroll
    for (int k = 0; k < HPT; ++k) {
      ht[k] = k < cnt ? a.H.htab[beg + k] : make_uint4(0u, 0u, 0u, 0u);
      bown[k] = k < cnt ? a.own.belief[beg + k] : 0.0;
    }
  }
#pragma unroll
  for (int k = 0; k < HPT; ++k) {
    const int i = gt + k * kGroupThreads;
    bo[k] = i < n ? a.b_opp[i] : 0.0;
    hp[k] = i < n ? a.H.hpos[i] : 0u;
  }
  // this lane's first card list (four lanes per card): start in E and length
  const int c_first = gt >> 2;
  const int cb_first = c_first < a.H.n_cards ? a.H.card_begin[c_first] : 0;
  const int len_first = c_first < a.H.n_cards ? a.H.card_begin[c_first + 1] - cb_first : 0;

  // The rounds of this block, in order: (unit w, round rd).  The terminal
  // records run two rounds ahead and the opponent rows one round ahead of
  // the round being evaluated, so neither load waits on the other.
  auto advance = [&](int& w_, int& rd_) {
    if (++rd_ >= rounds) {
      rd_ = 0;
      w_ += (int)gridDim.x;
    }
  };
  int w = blockIdx.x, rd = 0;
  TermRec tr = none;
  int s_out = -1;
  bool combine = false;
  if (w < n_work) term_of(w, 0, tr, s_out, combine);
  int w1 = w, rd1 = rd;
  advance(w1, rd1);
  TermRec tr1 = none;
  int s1 = -1;
  bool comb1 = false;
  if (w1 < n_work) term_of(w1, rd1, tr1, s1, comb1);
  double vv[HPT];
  auto load_row = [&](const TermRec& t, double* v) {
    const TV* row = t.opp >= 0 ? a.v_opp + (size_t)t.opp * ld : nullptr;
#pragma unroll
    for (int k = 0; k < HPT; ++k) {
      const int i = gt + k * kGroupThreads;
      v[k] = (row && i < n) ? (double)row[i] : 1.0;
    }
  };
  load_row(tr, vv);

  double acc[HPT];
#pragma unroll
  for (int k = 0; k < HPT; ++k) acc[k] = 0.0;
  double top = 0.0;  // MAX: this thread's largest |entry|
  while (w < n_work) {
    // uniform within a group
    const bool active = tr.kind >= 0;
    const int kind = tr.kind;
    const double coef = tr.coef;
    // 1. stage the reach into R (strength order) and E (card lists)
    if (active) {
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        const int i = gt + k * kGroupThreads;
        if (i < n) {
          const double r = bo[k] * vv[k];
          R[i] = r;
          E[hp[k] & 0xffffu] = r;
          if (cph == 2) E[hp[k] >> 16] = r;
        }
      }
    }
    // the next round's row, and the terminal two rounds ahead, loaded while this round runs
    load_row(tr1, vv);
    int w2 = w1, rd2 = rd1;
    advance(w2, rd2);
    TermRec tr2 = none;
    int s2 = -1;
    bool comb2 = false;
    if (w2 < n_work) term_of(w2, rd2, tr2, s2, comb2);
    __syncthreads();

    double rloc[HPT];
    double local = 0.0, incl = 0.0;
    if (active) {
      // 2a. per-card exclusive prefixes in place over each contiguous list
      const int sub = gt & 3;
      for (int c = c_first; c - c_first < a.H.n_cards; c += kGroupThreads / 4) {
        const bool valid = c < a.H.n_cards;
        const bool first = c == c_first;
        const int cb = first ? cb_first : valid ? a.H.card_begin[c] : 0;
        const int len = first ? len_first : valid ? a.H.card_begin[c + 1] - cb : 0;
        double* L = E + cb + c;
        const int qlen = (len + 3) >> 2;
        const int lo = min(sub * qlen, len), hi = min(lo + qlen, len);
        // the card's four lanes form an aligned quad: the quarter totals
        // cross lanes by DPP quad permutes
        if (qlen <= kQR) {  // uniform over the quad: the quarter stays in registers
          double v[kQR];
          double part = 0.0;
#pragma unroll
          for (int j = 0; j < kQR; ++j) v[j] = lo + j < hi ? L[lo + j] : 0.0;
#pragma unroll
          for (int j = 0; j < kQR; ++j)
            if (lo + j < hi) part += v[j];
          const double p0 = dpp_move<0x00, 0xf>(part), p1 = dpp_move<0x55, 0xf>(part), p2 = dpp_move<0xaa, 0xf>(part);
          double run = sub == 0 ? 0.0 : sub == 1 ? p0 : sub == 2 ? p0 + p1 : (p0 + p1) + p2;
#pragma unroll
          for (int j = 0; j < kQR; ++j) {
            if (lo + j < hi) {
              L[lo + j] = run;
              run += v[j];
            }
          }
          if (valid && sub == 3) L[len] = run;
        } else {  // long lists: two passes over the quarter in batches of kQ
          constexpr int kQ = 4;
          double part = 0.0;
          for (int k0 = lo; k0 < hi; k0 += kQ) {
            double v[kQ];
#pragma unroll
            for (int j = 0; j < kQ; ++j) v[j] = k0 + j < hi ? L[k0 + j] : 0.0;
#pragma unroll
            for (int j = 0; j < kQ; ++j)
              if (k0 + j < hi) part += v[j];
          }
          const double p0 = dpp_move<0x00, 0xf>(part), p1 = dpp_move<0x55, 0xf>(part), p2 = dpp_move<0xaa, 0xf>(part);
          double run = sub == 0 ? 0.0 : sub == 1 ? p0 : sub == 2 ? p0 + p1 : (p0 + p1) + p2;
          for (int k0 = lo; k0 < hi; k0 += kQ) {
            double v[kQ];
#pragma unroll
            for (int j = 0; j < kQ; ++j) v[j] = k0 + j < hi ? L[k0 + j] : 0.0;
#pragma unroll
            for (int j = 0; j < kQ; ++j) {
              if (k0 + j < hi) {
                L[k0 + j] = run;
                run += v[j];
              }
            }
          }
          if (valid && sub == 3) L[len] = run;
        }
      }
      // 2b. the strength-order scan of this thread's contiguous hands
#pragma unroll
      for (int k = 0; k < HPT; ++k) rloc[k] = k < cnt ? R[beg + k] : 0.0;
#pragma unroll
      for (int k = 0; k < HPT; ++k) local += rloc[k];
      incl = wave_inclusive_scan(local);
      if (lane == 63) wave_total[grp][wig] = incl;
    }
    __syncthreads();
    // 3. exclusive strength prefix in place over R, R[n] = total
    if (active) {
      double run = incl - local;
      for (int q = 0; q < wig; ++q) run += wave_total[grp][q];
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        if (k < cnt) {
          R[beg + k] = run;
          run += rloc[k];
        }
      }
      if (cnt > 0 && end == n) R[n] = run;
    }
    __syncthreads();
    // 4. evaluate this thread's hands
    if (active) {
      const double T = R[n];
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        if (k < cnt) {
          const uint4 t = TAB ? htab_l[beg + k] : ht[k];
          double op;
          if (kind == 0) {
            op = T - E[t.y & 0xffffu];
            if (cph == 2) op = op - E[t.z >> 16] + rloc[k];
          } else {
            double weaker = R[t.w & 0xffffu] - E[t.x & 0xffffu];
            double stronger = (T - R[t.w >> 16]) - (E[t.y & 0xffffu] - E[t.x >> 16]);
            if (cph == 2) {
              weaker -= E[t.y >> 16];
              stronger -= E[t.z >> 16] - E[t.z & 0xffffu];
            }
            op = a.show_sign * (stronger - weaker);
          }
          acc[k] += coef * op;
        }
      }
    }
    // the unit's last round: combine the two groups' results and write the row
    if (rd + 1 >= rounds) {
      if (combine) {
        __syncthreads();  // both groups are done reading their R
        if (grp == 1) {
#pragma unroll
          for (int k = 0; k < HPT; ++k)
            if (k < cnt) R[beg + k] = acc[k];
        }
        __syncthreads();
        if (grp == 0) {
          const double* R1 = lds + per_group;
#pragma unroll
          for (int k = 0; k < HPT; ++k)
            if (k < cnt) acc[k] += R1[beg + k];
        }
      }
      if ((!combine || grp == 0) && s_out >= 0) {
        TO* row = a.out + (size_t)s_out * ld;
#pragma unroll
        for (int k = 0; k < HPT; ++k)
          if (k < cnt) {
            const TO x = (TO)(acc[k] * ((TAB ? bown_l[beg + k] : bown[k]) * a.H.invZ));
            row[beg + k] = x;
            if constexpr (MAX) top = fmax(top, fabs((double)x));
          }
        for (int i = n + gt; i < ld; i += kGroupThreads) row[i] = (TO)0;
      }
#pragma unroll
      for (int k = 0; k < HPT; ++k) acc[k] = 0.0;
    }
    __syncthreads();  // the next round rewrites R and E of both groups
    w = w1;
    rd = rd1;
    tr = tr1;
    if (rd == 0) {
      s_out = s1;
      combine = comb1;
    }
    w1 = w2;
    rd1 = rd2;
    tr1 = tr2;
    s1 = s2;
    comb1 = comb2;
  }
  if constexpr (MAX) {
    top = wave_max(top);
    if (lane == 0) wave_total[grp][wig] = top;  // the last round ended in a barrier
    __syncthreads();
    if (tid == 0) {
      for (int v = 1; v < (int)blockDim.x / 64; ++v) top = fmax(top, wave_total[v / (kGroupThreads / 64)][v % (kGroupThreads / 64)]);
      a.absmax[blockIdx.x] = top;
    }
  }
}

// Large trees: two terminals of one kind per round.
//
// A block is one wave group; a round takes a terminal of each of two sequences,
// their reaches side by side in LDS as {first, second}, so that every index, LDS
// instruction, bank conflict and barrier of the evaluation above serves both
// (it is bound by LDS: of a showdown's 3,300 cycles of LDS pipe two thirds are
// the evaluation's scattered reads).  A pair of sequences has its folds and
// showdowns added by the same threads, with no second group to meet, and a fold
// round forms only the totals.  The card lists are gathered from the strength
// order (a thread's quarter of a list, at most kQR slots, sits in registers as
// indices), so nothing is scattered.  Rounds are dealt to the blocks at build
// (ProdRound), a compute unit holding as many blocks as its LDS lets in, at most four
// up to 512 hands and three above.  With more than two hands per thread
// the evaluation deals them strided over the block, although the scan takes
// them contiguous: neighbouring lanes then read neighbouring slots of R (fewer
// bank conflicts) and store whole lines of the row, and a fold reads its reach
// back from R, which it leaves as it was (1081 hands, strided instead of
// contiguous: 5938 sequences 3.7 us less, 1684 sequences 2.1).
// 5938 sequences, one player's product repeated, product_kernel against this one:
// 1081 hands 53.0 -> 40.2 us (player 2's 52.2 -> 38.7; the two in turn, each behind the
// other's vectors, 44 each), 595 hands 41.3 -> 30.2, 351 hands 32.1 -> 19.6, 105 hands
// 24.8 -> 14.6.  LDS and VALU are each busy a third of the time (counters at 1081
// hands), the rest is the latency of a round's chain between barriers at, for five
// hands per thread, 12 wavefronts per compute unit, which its LDS and registers allow
// (16 wavefronts, two blocks of 512 threads with half the hands each, took 5.8 us
// more; 24 of them spill and took 17 more).
// Every sum is the one product_kernel takes, in its order.
struct RoundArgs {
  DPlayer own;
  const double* b_opp;
  DHands H;
  const double* v_opp;
  double* out;
  double show_sign;
  double* absmax;  // MAX: each block's largest |entry|
};

__device__ inline double2 operator+(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 operator-(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

template <int HPT, int MINW, bool MAX>
__global__ __launch_bounds__(kGroupThreads, MINW) void product_pairs_kernel(RoundArgs a) {
  extern __shared__ __align__(16) double2 lds2[];
  __shared__ double2 wave_total[kGroupThreads / 64];
  const int n = a.H.n, ld = a.H.ld, cph = a.H.cph;
  double2* R = lds2;          // [n + 1] reach, then its exclusive prefix and total, in strength order
  double2* E = lds2 + n + 1;  // [n_card_slots] exclusive prefixes and totals by card
  const int gt = threadIdx.x, lane = gt & 63, wig = gt >> 6;
  const int chunk = (n + kGroupThreads - 1) / kGroupThreads;
  const int beg = min(gt * chunk, n), cnt = min(beg + chunk, n) - beg;
  // the k-th hand this thread evaluates
  constexpr bool strided = HPT > 2;
  auto hand = [&](int k) { return strided ? gt + k * kGroupThreads : beg + k; };
  auto has = [&](int k) { return strided ? gt + k * kGroupThreads < n : k < cnt; };

  double bo[HPT];
#pragma unroll
  for (int k = 0; k < HPT; ++k) bo[k] = gt + k * kGroupThreads < n ? a.b_opp[gt + k * kGroupThreads] : 0.0;
  // this thread's quarter of card gt / 4's list: slots, two to a word
  const int card = gt >> 2, sub = gt & 3;
  const bool has_card = card < a.H.n_cards;
  const int cb = has_card ? a.H.card_begin[card] : 0, len = has_card ? a.H.card_begin[card + 1] - cb : 0;
  const int qlen = (len + 3) >> 2, lo = min(sub * qlen, len), ql = min(lo + qlen, len) - lo;
  unsigned slots[kQR / 2];
#pragma unroll
  for (int j = 0; j < kQR / 2; ++j) {
    const unsigned s0 = 2 * j < ql ? a.H.card_slot[cb + lo + 2 * j] : 0u;
    const unsigned s1 = 2 * j + 1 < ql ? a.H.card_slot[cb + lo + 2 * j + 1] : 0u;
    slots[j] = s0 | (s1 << 16);
  }
  double2* L = E + cb + card;  // the card's list in E, its total behind

  const ProdRound* rounds = a.own.rounds;
  int ri = a.own.round_begin[blockIdx.x];
  const int rend = a.own.round_begin[blockIdx.x + 1];
  double v0[HPT], v1[HPT];
  auto load_rows = [&](int r) {
    const int o0 = rounds[r].opp[0], o1 = rounds[r].opp[1];
    const double* p0 = o0 >= 0 ? a.v_opp + (size_t)o0 * ld : nullptr;
    const double* p1 = o1 >= 0 ? a.v_opp + (size_t)o1 * ld : nullptr;
#pragma unroll
    for (int k = 0; k < HPT; ++k) {
      const int i = gt + k * kGroupThreads;
      v0[k] = (p0 && i < n) ? p0[i] : 1.0;
      v1[k] = (p1 && i < n) ? p1[i] : 1.0;
    }
  };
  if (ri < rend) load_rows(ri);
  double2 acc[HPT];
#pragma unroll
  for (int k = 0; k < HPT; ++k) acc[k] = make_double2(0.0, 0.0);
  double top = 0.0;  // MAX: this thread's largest |entry|
  for (; ri < rend; ++ri) {
    const ProdRound rd = rounds[ri];  // uniform
    if (rd.kind >= 0) {
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        const int i = gt + k * kGroupThreads;
        if (i < n) R[i] = make_double2(bo[k] * v0[k], bo[k] * v1[k]);
      }
    }
    if (ri + 1 < rend) load_rows(ri + 1);  // in flight while this round runs
    if (rd.kind >= 0) {
      __syncthreads();
      // per-card prefixes (folds: totals), the quarter totals by DPP within the
      // card's quad
      if (has_card) {
        double2 part = make_double2(0.0, 0.0);
        double2 v[kQR];
#pragma unroll
        for (int j = 0; j < kQR; j += 2) {
          unsigned w = slots[j / 2];
          asm volatile("" : "+v"(w));  // unpacked here each round: kept unpacked the indices would spill
          v[j] = j < ql ? R[w & 0xffffu] : make_double2(0.0, 0.0);
          v[j + 1] = j + 1 < ql ? R[w >> 16] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int j = 0; j < kQR; ++j)
          if (j < ql) part = part + v[j];
        const double2 p0 = make_double2(dpp_move<0x00, 0xf>(part.x), dpp_move<0x00, 0xf>(part.y));
        const double2 p1 = make_double2(dpp_move<0x55, 0xf>(part.x), dpp_move<0x55, 0xf>(part.y));
        const double2 p2 = make_double2(dpp_move<0xaa, 0xf>(part.x), dpp_move<0xaa, 0xf>(part.y));
        double2 run = sub == 0 ? make_double2(0.0, 0.0) : sub == 1 ? p0 : sub == 2 ? p0 + p1 : (p0 + p1) + p2;
#pragma unroll
        for (int j = 0; j < kQR; ++j) {
          if (j < ql) {
            if (rd.kind == 1) L[lo + j] = run;
            run = run + v[j];
          }
        }
        if (sub == 3) L[len] = run;
      }
      __builtin_amdgcn_sched_barrier(0);  // what follows takes the lists' registers
      // the index table from the cache, each round: it arrives behind the scan
      uint4 ht[HPT];
#pragma unroll
      for (int k = 0; k < HPT; ++k) ht[k] = has(k) ? a.H.htab[hand(k)] : make_uint4(0u, 0u, 0u, 0u);
      // strength order: this thread's contiguous hands, and the group's scan
      double2 rloc[HPT];
      double2 local = make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < HPT; ++k) rloc[k] = k < cnt ? R[beg + k] : make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < HPT; ++k) local = local + rloc[k];
      const double2 incl = make_double2(wave_inclusive_scan(local.x), wave_inclusive_scan(local.y));
      if (lane == 63) wave_total[wig] = incl;
      __syncthreads();
      {
        double2 run = incl - local;
        for (int q = 0; q < wig; ++q) run = run + wave_total[q];
#pragma unroll
        for (int k = 0; k < HPT; ++k) {
          if (k < cnt) {
            if (rd.kind == 1) R[beg + k] = run;
            run = run + rloc[k];
          }
        }
        if (cnt > 0 && beg + cnt == n) R[n] = run;
      }
      __syncthreads();
      const double2 T = R[n];
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        if (has(k)) {
          const uint4 t = ht[k];
          double2 op;
          if (rd.kind == 0) {
            op = T - E[t.y & 0xffffu];
            if (cph == 2) op = op - E[t.z >> 16] + (strided ? R[hand(k)] : rloc[k]);  // a fold leaves the reaches in R
          } else {
            double2 weaker = R[t.w & 0xffffu] - E[t.x & 0xffffu];
            double2 stronger = (T - R[t.w >> 16]) - (E[t.y & 0xffffu] - E[t.x >> 16]);
            if (cph == 2) {
              weaker = weaker - E[t.y >> 16];
              stronger = stronger - (E[t.z >> 16] - E[t.z & 0xffffu]);
            }
            op = stronger - weaker;
            op.x = a.show_sign * op.x;
            op.y = a.show_sign * op.y;
          }
          acc[k].x += rd.coef[0] * op.x;
          acc[k].y += rd.coef[1] * op.y;
        }
      }
      __syncthreads();  // the next round rewrites R and E
    }
    if (rd.last) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (rd.seq[j] < 0) continue;
        double* row = a.out + (size_t)rd.seq[j] * ld;
#pragma unroll
        for (int k = 0; k < HPT; ++k) {
          if (has(k)) {
            const int i = hand(k);
            const double x = (j == 0 ? acc[k].x : acc[k].y) * (a.own.belief[i] * a.H.invZ);
            row[i] = x;
            if constexpr (MAX) top = fmax(top, fabs(x));
          }
        }
        for (int i = n + gt; i < ld; i += kGroupThreads) row[i] = 0.0;
      }
#pragma unroll
      for (int k = 0; k < HPT; ++k) acc[k] = make_double2(0.0, 0.0);
    }
  }
  if constexpr (MAX) {
    top = wave_max(top);
    __syncthreads();
    if (lane == 0) wave_total[wig].x = top;
    __syncthreads();
    if (gt == 0) {
      for (int v = 1; v < kGroupThreads / 64; ++v) top = fmax(top, wave_total[v].x);
      a.absmax[blockIdx.x] = top;
    }
  }
}

// Precision form, fold terminals, in FP32, after the showdown GEMM: W = 4 fold
// terminals per round, one of each of four sequences, their reaches side by side
// in LDS, so that an index, an LDS instruction and a barrier serve four (one
// terminal per block and round was bound by its barriers and loads); W = 1 while
// there are fewer sequences than blocks to take them (1081 hands, whole product:
// 28 sequences 17.1 with W = 4, 14.4 us with W = 1; 223 sequences 18.6, 15.7).
// A round: the reaches r(h') to LDS in strength order; the card totals C[c],
// four lanes per card, each summing its quarter of the list, the quarters added
// in a fixed order; the total T (each thread's hands, then the wavefronts in
// order); then
//   op(h) = T - C[a] - C[b] + r(h)      (hand h holds cards a and b)
// for the thread's own hands, whose reach is still in registers, accumulated
// with the terminal's chips.  With its last round a row takes b_own(h)/Z times
// the sum: added to the showdown part where there is one, written elsewhere.
// 3958 folds on 5938 sequences x 1081 hands: 25.8 -> 16.8 us.
struct FoldArgs {
  DPlayer own;
  const double* b_opp;
  DHands H;
  const unsigned short* card_slot;
  const unsigned* hand_cards;
  const void* rounds;  // FoldRound<W>
  int n_rounds;
  const float* v_opp;
  float* out;
};

// W floats side by side (one LDS access of 4 W bytes).
template <int W>
struct alignas(4 * W) Lanes {
  float x[W];
};
template <int W, class F>
__device__ inline Lanes<W> lanes_of(F f) {
  Lanes<W> r;
#pragma unroll
  for (int j = 0; j < W; ++j) r.x[j] = f(j);
  return r;
}
template <int W>
__device__ inline Lanes<W> operator+(const Lanes<W>& a, const Lanes<W>& b) {
  return lanes_of<W>([&](int j) { return a.x[j] + b.x[j]; });
}
template <int W>
__device__ inline Lanes<W> operator-(const Lanes<W>& a, const Lanes<W>& b) {
  return lanes_of<W>([&](int j) { return a.x[j] - b.x[j]; });
}
template <int CTRL>
__device__ inline float quad_float(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

template <int HPT, int W>
__global__ __launch_bounds__(kGroupThreads) void fold_kernel(FoldArgs a) {
  using V = Lanes<W>;
  extern __shared__ __align__(16) float fold_lds[];
  __shared__ V wtot[kGroupThreads / 64];
  const V zero = lanes_of<W>([](int) { return 0.0f; });
  const int n = a.H.n, ld = a.H.ld, cph = a.H.cph;
  const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
  V* R = (V*)fold_lds;  // [n]
  V* C = R + n;         // [n_cards]
  float bo[HPT];
  unsigned cards[HPT];
#pragma unroll
  for (int k = 0; k < HPT; ++k) {
    const int i = tid + k * kGroupThreads;
    bo[k] = i < n ? (float)a.b_opp[i] : 0.0f;
    cards[k] = i < n ? a.hand_cards[i] : 0u;
  }
  // rounds in contiguous ranges, whole items (a group of sequences' rounds, the
  // last marked) per block: a range starts behind a last round
  const int per = (a.n_rounds + (int)gridDim.x - 1) / (int)gridDim.x;
  const FoldRound<W>* rounds = (const FoldRound<W>*)a.rounds;
  auto item_start = [&](int r) {
    r = min(r, a.n_rounds);
    while (r > 0 && r < a.n_rounds && !(rounds[r - 1].flags & kFoldLast)) ++r;
    return r;
  };
  int ri = item_start((int)blockIdx.x * per);
  const int rend = item_start(((int)blockIdx.x + 1) * per);
  // this thread's quarter of card tid / 4's list: its first slots stay in registers
  unsigned slots[kQR / 2];
  {
    const int c = tid >> 2;
    const int cb = c < a.H.n_cards ? a.H.card_begin[c] : 0, len = c < a.H.n_cards ? a.H.card_begin[c + 1] - cb : 0;
    const int qlen = (len + 3) >> 2, lo = min((tid & 3) * qlen, len), hi = min(lo + qlen, len);
#pragma unroll
    for (int j = 0; j < kQR / 2; ++j) {
      const unsigned s0 = lo + 2 * j < hi ? a.card_slot[cb + lo + 2 * j] : 0u;
      const unsigned s1 = lo + 2 * j + 1 < hi ? a.card_slot[cb + lo + 2 * j + 1] : 0u;
      slots[j] = s0 | (s1 << 16);
    }
  }
  V acc[HPT];
#pragma unroll
  for (int k = 0; k < HPT; ++k) acc[k] = zero;
  for (; ri < rend; ++ri) {
    const FoldRound<W> rd = rounds[ri];  // uniform
    if (!(rd.flags & kFoldNone)) {
      V r[HPT];
      V loc = zero;
      float v[W][HPT];
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const float* p = rd.opp[j] >= 0 ? a.v_opp + (size_t)rd.opp[j] * ld : nullptr;
#pragma unroll
        for (int k = 0; k < HPT; ++k) {
          const int i = tid + k * kGroupThreads;
          v[j][k] = (p && i < n) ? p[i] : 1.0f;
        }
      }
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        const int i = tid + k * kGroupThreads;
        r[k] = i < n ? lanes_of<W>([&](int j) { return bo[k] * v[j][k]; }) : zero;
        if (i < n) R[i] = r[k];
      }
#pragma unroll
      for (int k = 0; k < HPT; ++k) loc = loc + r[k];
      for (int off = 32; off > 0; off >>= 1) loc = loc + lanes_of<W>([&](int j) { return __shfl_xor(loc.x[j], off, 64); });
      if (lane == 0) wtot[wv] = loc;
      __syncthreads();
      for (int c0 = 0; c0 < a.H.n_cards; c0 += kGroupThreads / 4) {
        const int c = c0 + (tid >> 2), sub = tid & 3;
        const bool valid = c < a.H.n_cards;
        const int cb = valid ? a.H.card_begin[c] : 0, len = valid ? a.H.card_begin[c + 1] - cb : 0;
        const int qlen = (len + 3) >> 2, lo = min(sub * qlen, len), hi = min(lo + qlen, len);
        V part = zero;
        int k = lo;
        if (c0 == 0) {
#pragma unroll
          for (int j = 0; j < kQR; ++j)
            if (lo + j < hi) part = part + R[(slots[j / 2] >> (16 * (j & 1))) & 0xffffu];
          k = lo + kQR;
        }
        for (; k < hi; ++k) part = part + R[a.card_slot[cb + k]];
        const V p0 = lanes_of<W>([&](int j) { return quad_float<0x00>(part.x[j]); });
        const V p1 = lanes_of<W>([&](int j) { return quad_float<0x55>(part.x[j]); });
        const V p2 = lanes_of<W>([&](int j) { return quad_float<0xaa>(part.x[j]); });
        const V p3 = lanes_of<W>([&](int j) { return quad_float<0xff>(part.x[j]); });
        if (valid && sub == 0) C[c] = ((p0 + p1) + p2) + p3;
      }
      const V T = ((wtot[0] + wtot[1]) + wtot[2]) + wtot[3];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        V op = T - C[cards[k] & 0xffffu];
        if (cph == 2) op = (op - C[cards[k] >> 16]) + r[k];
        acc[k] = acc[k] + lanes_of<W>([&](int j) { return rd.coef[j] * op.x[j]; });
      }
      if (ri + 1 < rend) __syncthreads();  // the next round rewrites R and C
    }
    if (rd.flags & kFoldLast) {
      float scale[HPT];
#pragma unroll
      for (int k = 0; k < HPT; ++k) {
        const int i = tid + k * kGroupThreads;
        scale[k] = i < n ? (float)(a.own.belief[i] * a.H.invZ) : 0.0f;
      }
      float cur[W][HPT];  // the showdown parts, all loads in flight before the first store
#pragma unroll
      for (int j = 0; j < W; ++j)
#pragma unroll
        for (int k = 0; k < HPT; ++k) {
          const int i = tid + k * kGroupThreads;
          cur[j][k] = ((rd.flags >> j) & 1) && rd.seq[j] >= 0 && i < n ? a.out[(size_t)rd.seq[j] * ld + i] : 0.0f;
        }
#pragma unroll
      for (int j = 0; j < W; ++j) {
        if (rd.seq[j] < 0) continue;
        const bool add = (rd.flags >> j) & 1;
        float* out = a.out + (size_t)rd.seq[j] * ld;
#pragma unroll
        for (int k = 0; k < HPT; ++k) {
          const int i = tid + k * kGroupThreads;
          const float x = acc[k].x[j] * scale[k];
          if (i < n) out[i] = add ? x + cur[j][k] : x;
        }
        if (!add)
          for (int i = n + tid; i < ld; i += kGroupThreads) out[i] = 0.0f;
      }
#pragma unroll
      for (int k = 0; k < HPT; ++k) acc[k] = zero;
    }
  }
}

size_t align2(size_t x) { return (x + 1) / 2 * 2; }

// General games (Section 6's explicit sparse operator): one wavefront per CSR
// row; lane l takes the row's entries l, l + 64, ... in column order, then a
// fixed xor butterfly (every lane ends with the same sum); the row's slot 0
// gets the sum and its padding slots 1 .. ld - 1 are written 0.
__global__ __launch_bounds__(256) void spmv_kernel(const int64_t* ptr, const int* col, const double* val,
                                                   const double* v, int ld, int n_rows, double* out,
                                                   double* absmax) {
  __shared__ double top[4];
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const bool live = row < n_rows;
  const int64_t k0 = live ? ptr[row] : 0, k1 = live ? ptr[row + 1] : 0;
  double acc = 0.0;
  for (int64_t k = k0 + lane; k < k1; k += 64) acc += val[k] * v[(size_t)col[k] * ld];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  double* o = out + (size_t)row * ld;
  for (int i = lane; live && i < ld; i += 64) o[i] = i == 0 ? acc : 0.0;
  if (absmax) {  // the block's largest |entry|
    if (lane == 0) top[threadIdx.x >> 6] = fabs(acc);
    __syncthreads();
    if (threadIdx.x == 0) absmax[blockIdx.x] = fmax(fmax(fmax(fmax(0.0, top[0]), top[1]), top[2]), top[3]);
  }
}

}  // namespace

hipError_t launch_spmv(const egt_game* g, int player, const double* v_opp, double* grad_out, hipStream_t s,
                       double* absmax, int* blocks) {
  const DPlayer& P = g->dp[player];
  if (!g->general || !P.sp_ptr) return hipErrorInvalidValue;
  if (blocks) *blocks = (P.n_seq + 3) / 4;
  if (P.n_seq == 0) return hipSuccess;
  hipLaunchKernelGGL(spmv_kernel, dim3((unsigned)((P.n_seq + 3) / 4)), dim3(256), 0, s, P.sp_ptr, P.sp_col, P.sp_val,
                     v_opp, g->ld, P.n_seq, grad_out, absmax);
  return hipGetLastError();
}

// Doubles of LDS one wave group of the product kernel takes.
size_t product_group_doubles(const egt_game* g) { return align2((size_t)g->n + 1) + (size_t)g->dh.n_card_slots; }
// Bytes of the per-hand tables the kernel can stage in LDS (16-byte index table, own prior).
size_t product_table_bytes(const egt_game* g) { return (16 + 8) * (size_t)g->n; }

template <class TV, class TO>
static hipError_t product_launch(const egt_game* g, int player, const TV* v_opp, TO* grad_out, hipStream_t s,
                                 double* absmax, int* n_blocks) {
  ProdArgs<TV, TO> a;
  a.own = g->dp[player];
  a.b_opp = g->dp[1 - player].belief;
  a.H = g->dh;
  a.v_opp = v_opp;
  a.out = grad_out;
  a.show_sign = player == 0 ? 1.0 : -1.0;
  a.items = nullptr;
  a.n_items = 0;
  a.absmax = absmax;
  // two blocks per compute unit: each takes at most half of the CU's LDS
  const size_t budget = (size_t)g->lds_per_cu / 2;
  auto lds_bytes = [&](int gr) { return sizeof(double) * align2(gr * product_group_doubles(g)); };
  int groups = g->hp[player].max_terms_per_seq >= 2 ? 2 : 1;
  if (groups == 2 && lds_bytes(2) > std::min(budget, (size_t)g->lds_per_block)) groups = 1;
  a.groups = groups;
  const bool tab = lds_bytes(groups) + product_table_bytes(g) <= std::min(budget, (size_t)g->lds_per_block);
  const size_t lds = lds_bytes(groups) + (tab ? product_table_bytes(g) : 0);
  // one block per sequence up to two blocks per compute unit; beyond that each
  // block loops over work items that keep both groups busy
  const bool looping = g->dp[player].n_seq > g->n_cu;
  if (looping && groups == 2 && g->dp[player].term_items) {
    a.items = g->dp[player].term_items;
    a.n_items = g->dp[player].n_items;
  }
  const int units = a.items ? a.n_items : g->dp[player].n_seq;
  const int blocks = std::min(units, 2 * g->n_cu);
  if (n_blocks) *n_blocks = blocks;
  if (units == 0) return hipSuccess;
  const dim3 grid(blocks), block(kGroupThreads * groups);
  auto launch = [&](auto hpt, auto minw) {
    constexpr int H = decltype(hpt)::value, W = decltype(minw)::value;
    if (absmax && tab)
      hipLaunchKernelGGL((product_kernel<TV, TO, H, W, true, true>), grid, block, lds, s, a);
    else if (absmax)
      hipLaunchKernelGGL((product_kernel<TV, TO, H, W, false, true>), grid, block, lds, s, a);
    else if (tab)
      hipLaunchKernelGGL((product_kernel<TV, TO, H, W, true, false>), grid, block, lds, s, a);
    else
      hipLaunchKernelGGL((product_kernel<TV, TO, H, W, false, false>), grid, block, lds, s, a);
  };
  if (g->n <= 2 * kGroupThreads)
    launch(std::integral_constant<int, 2>(), std::integral_constant<int, 4>());
  else if (g->n <= 5 * kGroupThreads)
    launch(std::integral_constant<int, 5>(), std::integral_constant<int, 4>());
  else
    launch(std::integral_constant<int, 8>(), std::integral_constant<int, 2>());
  return hipGetLastError();
}

// LDS of one block of the paired kernel.
static size_t paired_lds(int n, int n_card_slots) { return sizeof(double2) * ((size_t)n + 1 + n_card_slots); }

int paired_product_blocks(const egt_game* g, const std::vector<int>& card_begin) {
  int longest = 0;
  for (int c = 0; c < g->n_cards; ++c) longest = std::max(longest, card_begin[c + 1] - card_begin[c]);
  // its registers hold five hands and a quarter list of kQR slots per thread, a
  // card's quad is one of 64
  if (g->n > 5 * kGroupThreads || longest > 4 * kQR || g->n_cards > kGroupThreads / 4) return 0;
  // Few sequences leave a pair's fold and showdown waiting for each other in one
  // block where two groups took them side by side: the kernels cross between
  // 520 and 808 sequences (1081 hands: 9.7 against 11.7 us, then 13.5 against
  // 12.3; 595 hands: 8.3 against 9.4, then 10.5 against 9.6).
  const int seqs = std::min(g->hp[0].n_seq, g->hp[1].n_seq);
  if (2 * seqs <= 5 * g->n_cu) return 0;
  const size_t lds = paired_lds(g->n, card_begin[g->n_cards] + g->n_cards);
  const int fit = (int)std::min<size_t>(g->n <= 2 * kGroupThreads ? 4 : 3, (size_t)g->lds_per_cu / (lds + 256));
  return fit >= 2 ? fit * g->n_cu : 0;
}

int absmax_capacity(const egt_game* g) {
  return std::max(4 * g->n_cu, (std::max(g->hp[0].n_seq, g->hp[1].n_seq) + 3) / 4);
}

hipError_t launch_gradient(const egt_game* g, int player, const double* v_opp, double* grad_out, hipStream_t s,
                           double* absmax, int* blocks) {
  if (g->general) return launch_spmv(g, player, v_opp, grad_out, s, absmax, blocks);
  const DPlayer& P = g->dp[player];
  if (P.rounds) {
    RoundArgs a{P, g->dp[1 - player].belief, g->dh, v_opp, grad_out, player == 0 ? 1.0 : -1.0, absmax};
    if (blocks) *blocks = P.n_round_blocks;
    const size_t lds = paired_lds(g->n, g->dh.n_card_slots);
    const dim3 grid((unsigned)P.n_round_blocks), block(kGroupThreads);
    if (g->n <= 2 * kGroupThreads && absmax)
      hipLaunchKernelGGL((product_pairs_kernel<2, 4, true>), grid, block, lds, s, a);
    else if (g->n <= 2 * kGroupThreads)
      hipLaunchKernelGGL((product_pairs_kernel<2, 4, false>), grid, block, lds, s, a);
    else if (absmax)
      hipLaunchKernelGGL((product_pairs_kernel<5, 3, true>), grid, block, lds, s, a);
    else
      hipLaunchKernelGGL((product_pairs_kernel<5, 3, false>), grid, block, lds, s, a);
    return hipGetLastError();
  }
  return product_launch<double, double>(g, player, v_opp, grad_out, s, absmax, blocks);
}

hipError_t launch_gradient_fold_f32(const egt_game* g, int player, const float* v_opp, float* grad_out,
                                    hipStream_t s) {
  if (g->general) return hipErrorInvalidValue;  // the precision form is river-only
  const DPlayer& P = g->dp[player];
  if (P.n_seq == 0) return hipSuccess;
  FoldArgs a;
  a.own = P;
  a.b_opp = g->dp[1 - player].belief;
  a.H = g->dh;
  a.card_slot = g->mx.card_slot;
  a.hand_cards = g->mx.hand_cards;
  a.rounds = g->mx.folds[player];
  a.n_rounds = g->mx.n_folds[player];
  a.v_opp = v_opp;
  a.out = grad_out;
  if (a.n_rounds == 0) return hipSuccess;
  const int w = g->mx.fold_width[player];
  const size_t lds = sizeof(float) * w * ((size_t)g->n + g->n_cards);
  const dim3 grid((unsigned)std::min(a.n_rounds, 4 * g->n_cu)), block(kGroupThreads);
  auto launch = [&](auto hpt) {
    constexpr int H = decltype(hpt)::value;
    if (w == 1)
      hipLaunchKernelGGL((fold_kernel<H, 1>), grid, block, lds, s, a);
    else
      hipLaunchKernelGGL((fold_kernel<H, 4>), grid, block, lds, s, a);
  };
  if (g->n <= 2 * kGroupThreads)
    launch(std::integral_constant<int, 2>());
  else if (g->n <= 5 * kGroupThreads)
    launch(std::integral_constant<int, 5>());
  else
    launch(std::integral_constant<int, 8>());
  return hipGetLastError();
}

}  // namespace egt
