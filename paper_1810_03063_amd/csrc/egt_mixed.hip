// Precision form of the payoff product: every showdown terminal of one
// player stacked into one dense contraction on the BF16 matrix cores.
//
// With hands in strength order, a showdown terminal z of player p contributes
//   out[s_p(z)][h] += b_p(h)/Z * u(z) * sign_p * sum_h' W[h][h'] r_z(h'),
//   W[h][h'] = [h, h' share no card] * sgn(s(h') - s(h))  in {-1, 0, +1},
//   r_z(h')  = b_o(h') v_o[s_o(z)][h']
// (Section 2's gradient operators, Eq. 2's payoff matrix restricted to the
// showdown leaves; W^T = -W, so player 2 uses the same W with sign -1).  All
// showdown columns r_z form Y (n x L), and C = W Y is computed as
// W Y_hi + W Y_lo with Y_hi = bf16(Y) and Y_lo = bf16(Y - Y_hi): W is exact in
// BF16, each BF16 x BF16 product is exact in FP32, the accumulation is FP32.
// Each own sequence has at most one showdown terminal (checked when the tables
// are built), so the GEMM writes every element of a row it has; the fold
// terminals keep their O(n) per-card evaluation (in FP32) in
// launch_gradient_fold_f32, which then adds to those rows and writes the others.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "egt_internal.h"

namespace egt {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 mfma_bf16x8;

constexpr int kTile = 32;     // output hands x showdown columns per block (one 32x32 MFMA tile)
constexpr int kKWaves = 16;   // waves per block, each contracting every 16th k-step of 16 hands
constexpr int kBatch = 3;     // k-steps whose operands a wave loads before multiplying
constexpr int kRedStride = kTile + 1;
constexpr int kTiledMinColumns = 512;  // without the column-block form: from this many showdown columns on, the tiled one

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

// Two floats to BF16, round to nearest with ties to even (gfx950 converts a
// pair in one instruction), packed low element first.
__device__ inline unsigned bf16x2_rn(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2v));
}

// Eight FP32 reaches split into BF16 hi = bf16(r) and lo = bf16(r - hi).
__device__ inline void split8(const float r[8], bf16x8& hi, bf16x8& lo) {
  unsigned h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    h[e] = bf16x2_rn(r[2 * e], r[2 * e + 1]);
    l[e] = bf16x2_rn(r[2 * e] - __uint_as_float(h[e] << 16), r[2 * e + 1] - __uint_as_float(h[e] & 0xffff0000u));
  }
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}

// Four floats of a caller's vector.  Its rows need not be 16-byte aligned (callers
// promise 8 bytes); on gfx950 the access is one 16-byte instruction all the same.
typedef float rowx4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ inline float4 load_row4(const float* p) {
  const rowx4 x = *(const rowx4*)p;
  return make_float4(x.x, x.y, x.z, x.w);
}

// Reach 0 for the hands of k .. k + 7 past the last one: what an input holds in its
// padding is not read as a value (0 x NaN would reach every row).
__device__ inline void clear_padding(float r[8], int k, int n) {
  if (k + 8 > n)
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = k + e < n ? r[e] : 0.0f;
}

struct GemmArgs {
  const unsigned short* W;  // [ld][ld] BF16 bits, row h, contiguous h'
  int n, ld;
  int L;                    // showdown columns of the own player
  const int* col_own;       // [L] own sequence of the column
  const int* col_opp;       // [L] opponent sequence (-1 = empty sequence)
  const double* col_coef;   // [L] player-2 chips at the terminal
  const float* b_opp32;     // [ld] opponent prior in FP32
  const double* b_own;      // [ld]
  double scale;             // sign / Z
  const float* v_opp;       // opponent strategy [S_o][ld]
  float* out;               // own gradient [S_own][ld]
};

// One 32 x 32 output tile (hands m0.., columns n0..) per block.  The k-steps
// of 16 hands are dealt round-robin to the 16 waves; each wave loads the
// operands of kBatch steps straight into registers (no reuse inside a block,
// so no LDS staging), forms the FP32 reach, splits it into BF16 hi + lo and
// issues two 32x32x16 MFMAs per step.  The 16 partial tiles are summed
// through LDS in wave order, and one lane per output element applies the
// epilogue.
// Operand layouts of v_mfma_f32_32x32x16_bf16 (lane l, element e < 8):
//   A[l % 32][8 (l / 32) + e], B[8 (l / 32) + e][l % 32];
//   accumulator r: row (r / 4) 8 + (l / 32) 4 + r % 4, column l % 32.
__global__ __launch_bounds__(64 * kKWaves) void show_gemm_kernel(GemmArgs a) {
  __shared__ float red[kKWaves * kTile * kRedStride];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.y * kTile, n0 = blockIdx.x * kTile;
  const int half = lane >> 5, l32 = lane & 31;
  const int col = n0 + l32;
  const float* vrow = nullptr;
  const bool cvalid = col < a.L;
  if (cvalid) {
    const int o = a.col_opp[col];
    vrow = o >= 0 ? a.v_opp + (size_t)o * a.ld : nullptr;
  }
  const unsigned short* wrow = a.W + (size_t)(m0 + l32) * a.ld + 8 * half;
  const int nk = a.ld / 16;

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  for (int base = wave; base < nk; base += kKWaves * kBatch) {
    uint4 av[kBatch];
    float4 v0[kBatch], v1[kBatch], b0[kBatch], b1[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int ks = base + u * kKWaves;
      av[u] = make_uint4(0u, 0u, 0u, 0u);
      v0[u] = v1[u] = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
      b0[u] = b1[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (ks < nk) {
        const int k0 = ks * 16 + 8 * half;
        av[u] = *(const uint4*)(wrow + ks * 16);
        if (cvalid) {
          if (vrow) {
            v0[u] = load_row4(vrow + k0);
            v1[u] = load_row4(vrow + k0 + 4);
          }
          b0[u] = *(const float4*)(a.b_opp32 + k0);
          b1[u] = *(const float4*)(a.b_opp32 + k0 + 4);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (base + u * kKWaves >= nk) break;  // uniform within the wave
      // FP32 reach of the 8 hands, split into BF16 hi + lo
      float r[8] = {b0[u].x * v0[u].x, b0[u].y * v0[u].y, b0[u].z * v0[u].z, b0[u].w * v0[u].w,
                    b1[u].x * v1[u].x, b1[u].y * v1[u].y, b1[u].z * v1[u].z, b1[u].w * v1[u].w};
      clear_padding(r, (base + u * kKWaves) * 16 + 8 * half, a.n);
      bf16x8 hi, lo;
      split8(r, hi, lo);
      const bf16x8 am = *(const bf16x8*)&av[u];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, hi, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, lo, acc, 0, 0, 0);
    }
  }
  // partial tiles to LDS as red[wave][column][row]
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = (r >> 2) * 8 + half * 4 + (r & 3);
    red[(wave * kTile + l32) * kRedStride + row] = acc[r];
  }
  __syncthreads();
  // one lane per output element: hands fastest, so each row is written coalesced
  const int h = m0 + (tid & 31), cl = tid >> 5, j = n0 + cl;
  if (j < a.L) {
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < kKWaves; ++w) sum += red[(w * kTile + cl) * kRedStride + (tid & 31)];
    const double c = a.col_coef[j] * a.scale;
    float* row = a.out + (size_t)a.col_own[j] * a.ld;
    row[h] = h < a.n ? (float)(c * a.b_own[h] * (double)sum) : 0.0f;
  }
}

// Many showdown columns where the column-block form below is left out (more than
// kColsMaxLd hands, or a player with fewer columns): a tiled GEMM with operand reuse.
// Block = 128 output hands x 64 columns, four waves, wave w owning rows
// 32 w .. 32 w + 31 of the tile as two 32 x 32 MFMA tiles.  K (the opponent's
// hands) advances in steps of kTK = 32 (ld is a multiple of 32): the block
// stages W[128 x 32] and the column reaches split into BF16 hi and lo
// ([64 columns x 32], k contiguous) in two LDS buffers, and the global loads
// run two steps ahead in registers, so each load has two steps of work to
// land behind.  The opponent's FP32 prior is staged in LDS once.  The hi and
// lo products accumulate in separate tiles (independent MFMA chains), added
// in the epilogue, which goes through LDS so that every output row is updated
// with coalesced accesses.  Tiles are numbered column block major and dealt to
// the XCDs in contiguous ranges, so the row blocks that share a column block's
// reaches meet in one L2.
constexpr int kTM = 128, kTN = 64, kTK = 32;
constexpr int kTKS = kTK + 8;  // LDS row stride (BF16 elements) of the staged operands
constexpr int kTCS = kTM + 1;  // LDS column stride (floats) of the output tile

struct TiledStage {
  unsigned short a[kTM * kTKS];   // W rows, k contiguous
  unsigned short bh[kTN * kTKS];  // reach hi, per column, k contiguous
  unsigned short bl[kTN * kTKS];  // reach lo
};
static_assert(sizeof(TiledStage) % 16 == 0, "the stages and the prior stay 16-byte aligned");
static_assert(kTCS * kTN * sizeof(float) <= 2 * sizeof(TiledStage), "the output tile fits the stages");

size_t tiled_lds_bytes(int ld) { return 2 * sizeof(TiledStage) + sizeof(float) * (size_t)ld; }

// Launch index -> tile, each XCD (launch indices go round-robin over the 8
// XCDs) taking a contiguous range of tiles.
__device__ inline int tile_of_launch(int b, int total) {
  const int q = total / 8, r = total % 8;
  const int x = b % 8, j = b / 8;
  return x * q + min(x, r) + j;
}

__global__ __launch_bounds__(256) void show_gemm_tiled_kernel(GemmArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  TiledStage* st = (TiledStage*)smem;                     // [2]
  float* bopp = (float*)(smem + 2 * sizeof(TiledStage));  // [ld]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int n_rb = (a.ld + kTM - 1) / kTM;
  const int t = tile_of_launch((int)blockIdx.x, (int)gridDim.x);
  const int m0 = (t % n_rb) * kTM, n0 = (t / n_rb) * kTN;
  const int nst = a.ld / kTK;

  // per thread and step: 16 k of one W row, 8 k of one column's reach
  const int arow = tid >> 1, ak = (tid & 1) * 16;
  const bool arow_ok = m0 + arow < a.ld;
  const unsigned short* wsrc = a.W + (size_t)(m0 + arow) * a.ld + ak;
  const int bcol = tid >> 2, bk = (tid & 3) * 8;
  const int jcol = n0 + bcol;
  const bool bcol_ok = jcol < a.L;
  const float* vsrc = nullptr;
  if (bcol_ok) {
    const int o = a.col_opp[jcol];
    vsrc = o >= 0 ? a.v_opp + (size_t)o * a.ld : nullptr;
  }
  for (int i = tid; i < a.ld; i += 256) bopp[i] = a.b_opp32[i];
  struct StepRegs {
    uint4 a0, a1;
    float4 v0, v1;
  };
  auto load_step = [&](StepRegs& q, int s) {
    const int k0 = s * kTK;
    q.a0 = q.a1 = make_uint4(0u, 0u, 0u, 0u);
    if (arow_ok) {
      q.a0 = *(const uint4*)(wsrc + k0);
      q.a1 = *(const uint4*)(wsrc + k0 + 8);
    }
    // a column past the last one has reach 0; the empty sequence has v = 1
    const float vfill = bcol_ok ? 1.0f : 0.0f;
    q.v0 = q.v1 = make_float4(vfill, vfill, vfill, vfill);
    if (vsrc) {
      q.v0 = load_row4(vsrc + k0 + bk);
      q.v1 = load_row4(vsrc + k0 + bk + 4);
    }
  };
  auto store_step = [&](const StepRegs& q, int s, TiledStage& d) {
    *(uint4*)&d.a[arow * kTKS + ak] = q.a0;
    *(uint4*)&d.a[arow * kTKS + ak + 8] = q.a1;
    const int kb = s * kTK + bk;
    const float4 b0 = *(const float4*)&bopp[kb], b1 = *(const float4*)&bopp[kb + 4];
    float r[8] = {b0.x * q.v0.x, b0.y * q.v0.y, b0.z * q.v0.z, b0.w * q.v0.w,
                  b1.x * q.v1.x, b1.y * q.v1.y, b1.z * q.v1.z, b1.w * q.v1.w};
    clear_padding(r, kb, a.n);
    bf16x8 hi, lo;
    split8(r, hi, lo);
    *(bf16x8*)&d.bh[bcol * kTKS + bk] = hi;
    *(bf16x8*)&d.bl[bcol * kTKS + bk] = lo;
  };

  f32x16 acc_hi[2], acc_lo[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc_hi[c][r] = 0.0f;
      acc_lo[c][r] = 0.0f;
    }
  const int arow_w = (wave * 32 + l32) * kTKS + 8 * half;  // this lane's A operand row
  const int bcol_w = l32 * kTKS + 8 * half;                // this lane's B operand column (tile 0)
  auto multiply = [&](const TiledStage& c) {
#pragma unroll
    for (int kk = 0; kk < kTK; kk += 16) {
      const bf16x8 am = *(const bf16x8*)&c.a[arow_w + kk];
#pragma unroll
      for (int ct = 0; ct < 2; ++ct) {
        const bf16x8 bh = *(const bf16x8*)&c.bh[bcol_w + 32 * ct * kTKS + kk];
        const bf16x8 bl = *(const bf16x8*)&c.bl[bcol_w + 32 * ct * kTKS + kk];
        acc_hi[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bh, acc_hi[ct], 0, 0, 0);
        acc_lo[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bl, acc_lo[ct], 0, 0, 0);
      }
    }
  };
  // Step s is multiplied from st[s & 1] while step s + 1 waits in registers
  // for the other buffer and step s + 2 is being loaded.
  StepRegs q0, q1;
  load_step(q0, 0);
  __syncthreads();  // the prior is staged
  store_step(q0, 0, st[0]);
  if (nst > 1) load_step(q0, 1);
  __syncthreads();
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    // st[0] holds step s, q0 step s + 1
    if (s + 2 < nst) load_step(q1, s + 2);
    multiply(st[0]);
    store_step(q0, s + 1, st[1]);
    __syncthreads();
    // st[1] holds step s + 1, q1 step s + 2
    if (s + 3 < nst) load_step(q0, s + 3);
    multiply(st[1]);
    if (s + 2 < nst) store_step(q1, s + 2, st[0]);
    __syncthreads();
  }
  if (s < nst) {  // an odd number of steps ends in st[0]
    multiply(st[0]);
    __syncthreads();  // the output tile below overwrites the stages
  }
  // output tile through LDS as ct[column][row] (the stage is free now)
  float* ct = (float*)smem;
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = wave * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
      const int col = 32 * c + l32;
      ct[col * kTCS + row] = acc_hi[c][r] + acc_lo[c][r];
    }
  __syncthreads();
  // each thread writes one hand of every second column
  constexpr int kColsPerSweep = 256 / kTM;  // columns covered by one sweep of the threads
  const int row = tid % kTM, h = m0 + row;
  if (h >= a.ld) return;
  const bool live = h < a.n;  // the padding is written 0
  const double bo = a.b_own[h];
#pragma unroll 4
  for (int col = tid / kTM; col < kTN; col += kColsPerSweep) {
    const int j = n0 + col;
    if (j >= a.L) break;
    const double c = a.col_coef[j] * a.scale;
    a.out[(size_t)a.col_own[j] * a.ld + h] = live ? (float)(c * bo * (double)ct[col * kTCS + row]) : 0.0f;
  }
}

// Many columns and at most kColsMaxLd hands: a block per 32 columns and part of
// the hands, no barrier in the contraction.
//
// The tiled form above moves every operand through LDS in 34 steps with a
// barrier each and splits each reach nine times (once per row block); its MFMA
// pipes were busy 16% of the time.  Here the block forms the reaches of its 32
// columns once, for all opponent hands, and keeps them in LDS as BF16 hi and lo
// (32 columns x 1088 hands x 4 bytes = 139 KB of the 160); each of its 12
// wavefronts owns MT tiles of 16 hands and runs over K on its own: its W
// operands come straight from L2 in the order the instruction takes them (W is
// stored that way: 1 KB contiguous per 16 hands x 32), two steps ahead in
// registers, the reaches from LDS.  MT is the smallest for which a block per
// compute unit is enough (3958 columns x 1088 hands: MT = 3, 248 blocks).
// That product: 51.0 -> 28 us, of which 13 in the contraction (8.3 at the MFMA
// peak) and 5 forming the reaches.
// Operand layouts of v_mfma_f32_16x16x32_bf16 (lane l, element e < 8):
//   A[l % 16][8 (l / 16) + e], B[8 (l / 16) + e][l % 16];
//   accumulator r: row 4 (l / 16) + r, column l % 16.
// LDS holds 16-byte units of 8 hands of a column at kc * 32 + (column ^ (kc % 8)),
// kc = hand / 8: writes (consecutive kc of a column) and reads (16 columns of a
// kc) both spread over the banks.
constexpr int kColsBlock = 32, kColsWaves = 12;
constexpr int kColsMinColumns = 256;
constexpr int kColsMaxLd = 1216;  // the reaches of a block fit LDS

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

size_t cols_lds_bytes(int ld) { return (size_t)kColsBlock * ld * 4; }

template <int MT>
__global__ __launch_bounds__(64 * kColsWaves, 3) void show_gemm_cols_kernel(GemmArgs a, int parts) {
  extern __shared__ __align__(16) uint4 bsm[];
  const int nk8 = a.ld / 8, nks = a.ld / 32;
  uint4* Bh = bsm;                     // [nk8][32] reach hi
  uint4* Bl = bsm + kColsBlock * nk8;  // reach lo
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = ((int)blockIdx.x / parts) * kColsBlock, part = (int)blockIdx.x % parts;
  // the block's reaches
  constexpr int kU = 3;  // units in flight per thread
  const int total = kColsBlock * nk8;
  for (int base = tid; base < total; base += 64 * kColsWaves * kU) {
    float4 v[kU][2], b[kU][2];
    int at[kU], k0[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = base + u * 64 * kColsWaves;
      const int col = i / nk8, kc = i - col * nk8, j = n0 + col;
      at[u] = i < total ? kc * kColsBlock + (col ^ (kc & 7)) : -1;
      k0[u] = 8 * kc;
      const bool ok = i < total && j < a.L;
      const float fill = ok ? 1.0f : 0.0f;  // the empty sequence has v = 1; no column has reach 0
      v[u][0] = v[u][1] = make_float4(fill, fill, fill, fill);
      b[u][0] = b[u][1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (ok) {
        const int o = a.col_opp[j];
        if (o >= 0) {
          const float* p = a.v_opp + (size_t)o * a.ld + 8 * kc;
          v[u][0] = load_row4(p);
          v[u][1] = load_row4(p + 4);
        }
        const float4* q = (const float4*)(a.b_opp32 + 8 * kc);
        b[u][0] = q[0];
        b[u][1] = q[1];
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (at[u] < 0) continue;
      const float4 b0 = b[u][0], b1 = b[u][1], v0 = v[u][0], v1 = v[u][1];
      float r[8] = {b0.x * v0.x, b0.y * v0.y, b0.z * v0.z, b0.w * v0.w,
                    b1.x * v1.x, b1.y * v1.y, b1.z * v1.z, b1.w * v1.w};
      clear_padding(r, k0[u], a.n);
      bf16x8 hi, lo;
      split8(r, hi, lo);
      Bh[at[u]] = __builtin_bit_cast(uint4, hi);
      Bl[at[u]] = __builtin_bit_cast(uint4, lo);
    }
  }
  __syncthreads();
  const int n_rt = a.ld / 16, rt0 = (part * kColsWaves + wave) * MT;
  if (rt0 >= n_rt) return;
  // W in operand order: [row tile][k step][lane], 16 bytes each; tiles past the
  // last one repeat it and are not written
  const uint4* A[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) A[t] = (const uint4*)a.W + (size_t)min(rt0 + t, n_rt - 1) * nks * 64 + lane;
  f32x4 hi[MT][2], lo[MT][2];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int c = 0; c < 2; ++c) hi[t][c] = lo[t][c] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int kAhead = 2;  // W steps in flight
  uint4 w[kAhead + 1][MT];
#pragma unroll
  for (int q = 0; q < kAhead; ++q)
#pragma unroll
    for (int t = 0; t < MT; ++t) w[q][t] = A[t][(size_t)min(q, nks - 1) * 64];
  for (int ks0 = 0; ks0 < nks; ks0 += kAhead + 1) {
#pragma unroll
    for (int q = 0; q < kAhead + 1; ++q) {
      const int ks = ks0 + q;
      if (ks >= nks) break;
      const int kn = min(ks + kAhead, nks - 1);
#pragma unroll
      for (int t = 0; t < MT; ++t) w[(q + kAhead) % (kAhead + 1)][t] = A[t][(size_t)kn * 64];
      const int kc = 4 * ks + (lane >> 4), col = lane & 15;
      const uint4* bh = Bh + kc * kColsBlock;
      const uint4* bl = Bl + kc * kColsBlock;
      const int c0 = col ^ (kc & 7), c1 = (16 + col) ^ (kc & 7);
      const mfma_bf16x8 h0 = __builtin_bit_cast(mfma_bf16x8, bh[c0]), h1 = __builtin_bit_cast(mfma_bf16x8, bh[c1]);
      const mfma_bf16x8 l0 = __builtin_bit_cast(mfma_bf16x8, bl[c0]), l1 = __builtin_bit_cast(mfma_bf16x8, bl[c1]);
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const mfma_bf16x8 am = __builtin_bit_cast(mfma_bf16x8, w[q][t]);
        hi[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, h0, hi[t][0], 0, 0, 0);
        hi[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, h1, hi[t][1], 0, 0, 0);
        lo[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, l0, lo[t][0], 0, 0, 0);
        lo[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, l1, lo[t][1], 0, 0, 0);
      }
    }
  }
  // every element of a row has one writer; the padding is written 0
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int j = n0 + 16 * c + (lane & 15);
    if (j >= a.L) continue;
    const double cf = a.col_coef[j] * a.scale;
    float* row = a.out + (size_t)a.col_own[j] * a.ld;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (rt0 + t >= n_rt) continue;
      const int h = 16 * (rt0 + t) + 4 * (lane >> 4);
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = (float)(cf * a.b_own[h + r] * (double)(hi[t][c][r] + lo[t][c][r]));
      if (h + 4 > a.n)  // on its own: selected with the products, their loads became conditional (28 -> 30.6 us)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = h + r < a.n ? x[r] : 0.0f;
      *(rowx4*)(row + h) = (rowx4){x[0], x[1], x[2], x[3]};
    }
  }
}

}  // namespace

// Column blocks wherever the tiled form would do (same bits: each element adds its
// hi and its lo products in the same order), and from kColsMinColumns on once the K-split
// form's tiles are more than one per compute unit; up to there those are all done
// at once and it is the faster form (whole product, columns against K-split: 595
// hands 209 tiles 14.3 against 11.9 us, 741 hands 264 tiles 16.0 and 19.0; 1081 hands
// 204 tiles 18.1 and 15.8, 374 tiles 19.0 and 26.1).
bool takes_column_gemm(const egt_game* g) {
  auto fits = [&](int p) {
    const std::vector<int>& kinds = g->hp[p].term_kind;
    const int64_t columns = std::count(kinds.begin(), kinds.end(), 1);
    const int64_t tiles = (columns + kTile - 1) / kTile * (g->ld / kTile);
    return columns >= kTiledMinColumns || (columns >= kColsMinColumns && tiles > g->n_cu);
  };
  return g->ld <= kColsMaxLd && fits(0) && fits(1);
}

// W (BF16 bits; in the column-block GEMM's operand order when both players take
// it), and per player the FP32 prior, the showdown column lists and the fold
// rounds, as one host image: W at 0, the rest at `off`.
int mixed_tables_image(const egt_game* g, std::vector<unsigned char>& img, MixedOffsets* off) {
  if (g->general) return fail(EGT_EINVAL, "the precision form needs a river endgame");
  const int n = g->n;
  const int kpad = g->ld;  // rows and columns padded like every vector
  std::vector<int> own[2], opp[2];
  std::vector<double> coef[2];
  std::vector<FoldRound<1>> folds1[2];
  std::vector<FoldRound<4>> folds4[2];
  for (int p = 0; p < 2; ++p) {
    const HostPlayer& hp = g->hp[p];
    std::vector<std::vector<int>> by_folds;  // by_folds[k]: sequences with k fold terminals
    std::vector<char> has_show(hp.n_seq, 0);
    for (int s = 0; s < hp.n_seq; ++s) {
      int shows = 0, nf = 0;
      for (int t = hp.term_begin[s]; t < hp.term_begin[s + 1]; ++t) {
        if (hp.term_kind[t] != 1) {
          ++nf;
          continue;
        }
        if (++shows > 1) return fail(EGT_EINVAL, "precision form needs at most one showdown per sequence");
        own[p].push_back(s);
        opp[p].push_back(hp.term_opp[t]);
        coef[p].push_back(hp.term_coef[t]);
      }
      has_show[s] = shows > 0;
      if (nf == 0 && shows > 0) continue;  // the GEMM writes the row
      if ((int)by_folds.size() <= nf) by_folds.resize(nf + 1);
      by_folds[nf].push_back(s);
    }
    // sequences with the same number of folds, four at a time where one each
    // would be more than four blocks per compute unit
    const size_t w = hp.n_seq > 4 * g->n_cu ? 4 : 1;
    off->p[p].fold_width = (int)w;
    auto deal = [&](auto& rounds, auto width) {
      constexpr int W = decltype(width)::value;
      for (size_t nf = 0; nf < by_folds.size(); ++nf)
        for (size_t i = 0; i < by_folds[nf].size(); i += W)
          for (size_t k = 0; k < std::max<size_t>(nf, 1); ++k) {
            FoldRound<W> r{};
            r.flags = (nf ? 0 : kFoldNone) | (k + 1 >= nf ? kFoldLast : 0);
            for (int j = 0; j < W; ++j) {
              r.opp[j] = r.seq[j] = -1;
              if (i + j >= by_folds[nf].size()) continue;
              const int s = by_folds[nf][i + j];
              r.seq[j] = s;
              if (has_show[s]) r.flags |= 1 << j;
              size_t seen = 0;
              for (int t = hp.term_begin[s]; t < hp.term_begin[s + 1]; ++t)
                if (hp.term_kind[t] == 0 && seen++ == k) {
                  r.opp[j] = hp.term_opp[t];
                  r.coef[j] = (float)hp.term_coef[t];
                }
            }
            rounds.push_back(r);
          }
    };
    if (w == 4)
      deal(folds4[p], std::integral_constant<int, 4>());
    else
      deal(folds1[p], std::integral_constant<int, 1>());
  }
  std::vector<unsigned> hand_cards(n);
  for (int i = 0; i < n; ++i)
    hand_cards[i] = (unsigned)g->slot_cards[(size_t)i * g->cph] |
                    (g->cph == 2 ? (unsigned)g->slot_cards[(size_t)i * g->cph + 1] << 16 : 0u);
  // slot order: strength ascending; compatibility from the cards of the slots
  off->by_columns = takes_column_gemm(g);
  std::vector<unsigned short> W((size_t)kpad * kpad, 0);
  for (int i = 0; i < n; ++i) {
    for (int k = 0; k < n; ++k) {
      bool share = false;
      for (int x = 0; x < g->cph && !share; ++x)
        for (int y = 0; y < g->cph; ++y)
          if (g->slot_cards[(size_t)i * g->cph + x] == g->slot_cards[(size_t)k * g->cph + y]) share = true;
      if (share) continue;
      const int si = g->slot_strength[i], sk = g->slot_strength[k];
      const size_t at = !off->by_columns ? (size_t)i * kpad + k
                                         : (((size_t)(i / 16) * (kpad / 32) + k / 32) * 64 + k % 32 / 8 * 16 + i % 16) * 8 + k % 8;
      W[at] = sk > si ? 0x3F80 : (sk < si ? 0xBF80 : 0);
    }
  }
  // FP32 copies of the priors (the reach b v is formed in FP32)
  std::vector<float> b32[2];
  for (int p = 0; p < 2; ++p) b32[p].assign(g->hbelief[p].begin(), g->hbelief[p].end());
  size_t total = 0;
  auto add = [&](size_t bytes) {
    const size_t at = total;
    total += (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
    return at;
  };
  add(sizeof(unsigned short) * W.size());
  for (int p = 0; p < 2; ++p) {
    MixedOffsets::Player& o = off->p[p];
    o.b32 = add(sizeof(float) * b32[p].size());
    o.own = add(sizeof(int) * own[p].size());
    o.opp = add(sizeof(int) * opp[p].size());
    o.coef = add(sizeof(double) * coef[p].size());
    o.folds = add(sizeof(FoldRound<1>) * folds1[p].size() + sizeof(FoldRound<4>) * folds4[p].size());
    o.n_show = (int)own[p].size();
    o.n_folds = (int)(folds1[p].size() + folds4[p].size());
  }
  off->cslot = add(sizeof(unsigned short) * g->card_slot.size());
  off->hcard = add(sizeof(unsigned) * hand_cards.size());
  img.assign(total, 0);
  auto put = [&](size_t at, const void* src, size_t bytes) {
    if (bytes) std::memcpy(img.data() + at, src, bytes);
  };
  put(0, W.data(), sizeof(unsigned short) * W.size());
  for (int p = 0; p < 2; ++p) {
    const MixedOffsets::Player& o = off->p[p];
    put(o.b32, b32[p].data(), sizeof(float) * b32[p].size());
    put(o.own, own[p].data(), sizeof(int) * own[p].size());
    put(o.opp, opp[p].data(), sizeof(int) * opp[p].size());
    put(o.coef, coef[p].data(), sizeof(double) * coef[p].size());
    put(o.folds, folds1[p].data(), sizeof(FoldRound<1>) * folds1[p].size());
    put(o.folds, folds4[p].data(), sizeof(FoldRound<4>) * folds4[p].size());
  }
  put(off->cslot, g->card_slot.data(), sizeof(unsigned short) * g->card_slot.size());
  put(off->hcard, hand_cards.data(), sizeof(unsigned) * hand_cards.size());
  return EGT_OK;
}

static void point_mixed_tables(egt_game* g, const MixedOffsets& off, void* dev, bool owned) {
  const unsigned char* base = (const unsigned char*)dev;
  g->mx.kpad = g->ld;
  g->mx.W = (const unsigned short*)dev;
  g->mx.by_columns = off.by_columns;
  for (int p = 0; p < 2; ++p) {
    const MixedOffsets::Player& o = off.p[p];
    g->mx.L[p] = o.n_show;
    g->mx.col_own[p] = (const int*)(base + o.own);
    g->mx.col_opp[p] = (const int*)(base + o.opp);
    g->mx.col_coef[p] = (const double*)(base + o.coef);
    g->mx.belief32[p] = (const float*)(base + o.b32);
    g->mx.folds[p] = base + o.folds;
    g->mx.n_folds[p] = o.n_folds;
    g->mx.fold_width[p] = o.fold_width;
  }
  g->mx.card_slot = (const unsigned short*)(base + off.cslot);
  g->mx.hand_cards = (const unsigned*)(base + off.hcard);
  g->mx.owned = owned;
  g->mx.block = dev;
}

int mixed_tables_upload(egt_game* g, const std::vector<unsigned char>& img, const MixedOffsets& off, void* dev,
                        bool owned, hipStream_t s) {
  EGT_HIP(hipMemcpyAsync(dev, img.data(), img.size(), hipMemcpyHostToDevice, s));
  point_mixed_tables(g, off, dev, owned);
  return EGT_OK;
}

// Builds and uploads the precision-form tables once per game, on first use
// (synchronous upload).
int ensure_mixed_tables(const egt_game* cg) {
  egt_game* g = const_cast<egt_game*>(cg);  // cached tables owned by the game
  if (g->mx.block) return EGT_OK;
  std::vector<unsigned char> img;
  MixedOffsets off{};
  int rc = mixed_tables_image(g, img, &off);
  if (rc) return rc;
  void* dev = nullptr;
  hipError_t e = hipMalloc(&dev, img.size());
  if (e != hipSuccess) return fail(EGT_ENOMEM, std::string("hipMalloc (precision tables): ") + hipGetErrorString(e));
  e = hipMemcpy(dev, img.data(), img.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(dev);
    return hip_fail(e, "upload of precision tables");
  }
  point_mixed_tables(g, off, dev, true);
  return EGT_OK;
}

hipError_t launch_show_gemm(const egt_game* g, int player, const float* v_opp, float* grad_out, hipStream_t s) {
  const MixedTables& m = g->mx;
  if (m.L[player] == 0) return hipSuccess;
  GemmArgs a;
  a.W = m.W;
  a.n = g->n;
  a.ld = g->ld;
  a.L = m.L[player];
  a.col_own = m.col_own[player];
  a.col_opp = m.col_opp[player];
  a.col_coef = m.col_coef[player];
  a.b_opp32 = m.belief32[1 - player];
  a.b_own = g->dp[player].belief;
  a.scale = (player == 0 ? 1.0 : -1.0) / g->Z;
  a.v_opp = v_opp;
  a.out = grad_out;
  if (m.by_columns) {
    const int col_blocks = (a.L + kColsBlock - 1) / kColsBlock, n_rt = g->ld / 16;
    const size_t lds = cols_lds_bytes(g->ld);
    // blocks a compute unit holds: LDS, and two blocks' wavefronts
    const int fit = g->n_cu * std::max(1, std::min(2, (int)((size_t)g->lds_per_cu / lds)));
    auto parts_of = [&](int mt) { return (n_rt + kColsWaves * mt - 1) / (kColsWaves * mt); };
    int mt = 1;
    while (mt < 3 && col_blocks * parts_of(mt) > fit) ++mt;
    const dim3 grid((unsigned)(col_blocks * parts_of(mt))), block(64 * kColsWaves);
    if (mt == 1)
      hipLaunchKernelGGL(show_gemm_cols_kernel<1>, grid, block, lds, s, a, parts_of(1));
    else if (mt == 2)
      hipLaunchKernelGGL(show_gemm_cols_kernel<2>, grid, block, lds, s, a, parts_of(2));
    else
      hipLaunchKernelGGL(show_gemm_cols_kernel<3>, grid, block, lds, s, a, parts_of(3));
    return hipGetLastError();
  }
  if (a.L >= kTiledMinColumns) {
    // enough columns for operand reuse to pay: the tiled form
    const unsigned tiles = (unsigned)(((a.L + kTN - 1) / kTN) * ((g->ld + kTM - 1) / kTM));
    hipLaunchKernelGGL(show_gemm_tiled_kernel, dim3(tiles), dim3(256), tiled_lds_bytes(g->ld), s, a);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((a.L + kTile - 1) / kTile), (unsigned)(g->ld / kTile));
  hipLaunchKernelGGL(show_gemm_kernel, grid, dim3(64 * kKWaves), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gradient_mixed(const egt_game* g, int player, const float* v_opp, float* grad_out, hipStream_t s) {
  hipError_t e = launch_show_gemm(g, player, v_opp, grad_out, s);
  if (e != hipSuccess) return e;
  return launch_gradient_fold_f32(g, player, v_opp, grad_out, s);
}

}  // namespace egt
