// sblm_mlp.hip -- learned proposal network for seeding the EA population.
//
// Not part of the paper's method (its neural network is a competing fitter,
// Sec. 4.1); the network only proposes starting points, and the EA's chi^2
// (Sec. 4.1, 4.4) still decides.  Contents:
//   * sblm_resample: a lightcurve -> 256 normalised bins;
//   * mlp_make_data: training lightcurves drawn from the EA's parameter
//     domain and observed at bin level through the forward model (Sec. 2.2);
//   * the network 256 -> 512 -> 512 -> 120 (ReLU hidden layers) whose output
//     is a K = 8 mixture of diagonal Gaussians over 7 targets, trained by its
//     own BF16 MFMA forward and backward GEMMs, an FP64 mixture-likelihood
//     kernel, deterministic column sums and Adam on FP32 master weights.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>

#include "sblm_internal.h"
#include "sblm_rng.h"

namespace sblm {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NB = MLP_NBINS;      // 256 input bins
constexpr int NH = MLP_HIDDEN;     // 512 hidden units
constexpr int NO = MLP_NOUT;       // 120 outputs
constexpr int NOP = MLP_NOUT_PAD;  // 128 (padded output width)
constexpr int KM = MLP_K, DM = MLP_D;

// Device parameter layout (FP32 master copy, BF16 shadow and Adam moments):
// W1 [256][512], b1 [512], W2 [512][512], b2 [512], W3 [512][128], b3 [128];
// the 8 pad columns of W3 and b3 hold zeros and receive zero gradient.
constexpr int64_t OFF_W1 = 0;
constexpr int64_t OFF_B1 = OFF_W1 + (int64_t)NB * NH;
constexpr int64_t OFF_W2 = OFF_B1 + NH;
constexpr int64_t OFF_B2 = OFF_W2 + (int64_t)NH * NH;
constexpr int64_t OFF_W3 = OFF_B2 + NH;
constexpr int64_t OFF_B3 = OFF_W3 + (int64_t)NH * NOP;
constexpr int64_t NP_DEV = OFF_B3 + NOP;

constexpr uint64_t P_MLP_INIT = 32;  // Philox purposes of this file (key
constexpr uint64_t P_DATA = 33;      // word 1 = sample index or 0)

// ------------------------------------------------------------------ BF16

__device__ __forceinline__ uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)0x7fc0;  // NaN
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);      // RNE
}

// ------------------------------------------------------------------ GEMM
//
// The weight gradients: C[M][N] = A[M][K] * B[N][K]^T on BF16 operands, k (the
// batch row) contiguous in both, with FP32 accumulation in the 32x32x16
// matrix-core instruction, k ascending (every output is the same chain of
// instructions in any tiling below).  A workgroup of four waves owns a TILE x
// TILE tile of C, K advancing through LDS in stages of TKS (row stride padded
// by 8: conflict-free 16-byte reads of a lane's 8 consecutive k).  At batch
// 1024 (eight ranges of 128 rows) one stage holds a range (NBUF = 1): a
// tile's loads are all in flight at once and one barrier separates them from
// the products; longer sums go through two buffers, the next stage's loads in
// flight during the products.  32 x 32 tiles replace 64 x 64 ones that would
// leave half of the compute units without work (batches below 256).
// Requires M, N % 64 == 0, K % (32 * ksplit) == 0.  With ksplit > 1 each K range
// writes its own partial, and splitk_reduce_kernel or the Adam kernel adds
// them in order.
struct GemmArgs {
  const uint16_t* A;  // [M][lda]
  int64_t lda;
  const uint16_t* B;  // [N][ldb]
  int64_t ldb;
  int M, N, K;
  float* C;           // [M][N] (with ksplit > 1: [ksplit][M][N])
  int ksplit;         // K is cut into ksplit equal ranges (blockIdx.z), 0/1: none
};

// Column sums that ride along in a GEMM launch (colsum_block): the work of
// tiles * CS_RC extra blocks.
constexpr int CS_RC = 16;
struct ColSeg {
  const float* X;
  int64_t ld;
  int ncol;
  float* out;
};
struct ColSegs {
  ColSeg s[4];
  int nseg;
  int tile0[5];  // first 64-column tile of each segment
  int col0[5];   // first column of each segment in the partial array
  int nrow;
};

// Column sums out[c] = sum_r X[r][c] of up to four matrices (bias gradients
// and the loss).  Stage 1: block (column tile of 64, row chunk rc) sums its
// rows in four interleaved groups combined in a fixed order into
// part[rc][column]; stage 2 adds the RC chunks in order.  Deterministic.
__device__ __forceinline__ void colsum_block(const ColSegs& cs, float* part, int tile, int rc,
                                             float (*red)[64]) {
  const int ncol_all = cs.col0[cs.nseg];
  int sg = 0;
  while (sg + 1 < cs.nseg && tile >= cs.tile0[sg + 1]) ++sg;
  const ColSeg& g = cs.s[sg];
  const int c = (tile - cs.tile0[sg]) * 64 + (threadIdx.x & 63);
  const int grp = threadIdx.x >> 6;
  const int per = (cs.nrow + CS_RC - 1) / CS_RC;
  const int r0 = rc * per, r1 = min(cs.nrow, r0 + per);
  float acc = 0.0f;
  if (c < g.ncol) {
#pragma unroll 4
    for (int r = r0 + grp; r < r1; r += 4) acc += g.X[(int64_t)r * g.ld + c];
  }
  red[grp][threadIdx.x & 63] = acc;
  __syncthreads();
  if (grp == 0 && c < g.ncol) {
    const int j = threadIdx.x;
    part[(int64_t)rc * ncol_all + cs.col0[sg] + c] =
        ((red[0][j] + red[1][j]) + red[2][j]) + red[3][j];
  }
}

__global__ void colsum_stage2(ColSegs cs, const float* part, int ncol_all) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncol_all) return;
  int sg = 0;
  while (sg + 1 < cs.nseg && c >= cs.col0[sg + 1]) ++sg;
  float t = part[c];
  for (int rc = 1; rc < CS_RC; ++rc) t += part[(int64_t)rc * ncol_all + c];
  cs.s[sg].out[c - cs.col0[sg]] = t;
}

// Up to three independent products of one shape class in one launch (the
// three weight gradients of a step): blockIdx.x runs over the output tiles
// of problem 0, then 1, then 2 (first[p] = its first block), blockIdx.z over
// the K ranges, which all problems share; the blocks from first[nprob] on
// take the column sums (cs.nseg > 0).
struct GemmGroup {
  GemmArgs g[3];
  int first[4];
  int nprob;
  ColSegs cs;
  float* cpart;
};

// One K stage of a TILE-row operand tile in 16-byte chunks, consecutive
// threads on consecutive chunks of a row.
template <int TILE, int TKS>
constexpr int STAGE_CHUNKS = TILE * TKS / 8 / 256;

template <int TILE, int TKS>
__device__ __forceinline__ void load_tile(const uint16_t* __restrict__ X, int64_t ld, int r0,
                                          int k0, uint4* v) {
#pragma unroll
  for (int j = 0; j < STAGE_CHUNKS<TILE, TKS>; ++j) {
    const int q = threadIdx.x + 256 * j;
    v[j] = *(const uint4*)(X + (int64_t)(r0 + q / (TKS / 8)) * ld + k0 + (q % (TKS / 8)) * 8);
  }
}

template <int TILE, int TKS>
__device__ __forceinline__ void store_tile(uint16_t* S, const uint4* v) {
#pragma unroll
  for (int j = 0; j < STAGE_CHUNKS<TILE, TKS>; ++j) {
    const int q = threadIdx.x + 256 * j;
    *(uint4*)(S + (q / (TKS / 8)) * (TKS + 8) + (q % (TKS / 8)) * 8) = v[j];
  }
}

template <int TILE, int TKS, int NBUF>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmGroup gg) {
  constexpr int STRIDE = TKS + 8;  // padded LDS row (elements)
  __shared__ __attribute__((aligned(16))) uint16_t sA[NBUF][TILE * STRIDE];
  __shared__ __attribute__((aligned(16))) uint16_t sB[NBUF][TILE * STRIDE];
  if ((int)blockIdx.x >= gg.first[gg.nprob]) {  // the whole block
    const int id = ((int)blockIdx.x - gg.first[gg.nprob]) * gridDim.z + blockIdx.z;
    const int tiles = gg.cs.tile0[gg.cs.nseg];
    if (id < tiles * CS_RC)
      colsum_block(gg.cs, gg.cpart, id % tiles, id / tiles, (float(*)[64])(void*)sA);
    return;
  }
  int prob = 0;
  while (prob + 1 < gg.nprob && (int)blockIdx.x >= gg.first[prob + 1]) ++prob;
  const GemmArgs& g = gg.g[prob];
  const int tile = (int)blockIdx.x - gg.first[prob], ntn = g.N / TILE;
  const int m0 = (tile / ntn) * TILE, n0 = (tile % ntn) * TILE;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // (32 x 32 tiles: the first wave multiplies, all four load)
  const int wm = TILE == 64 ? (wave >> 1) * 32 : 0, wn = TILE == 64 ? (wave & 1) * 32 : 0;
  const bool multiplies = TILE == 64 || wave == 0;
  const int nst = NBUF == 1 ? 1 : g.K / TKS / gridDim.z;  // stages of this K range
  const int kb = blockIdx.z * nst * TKS;                  // its first k

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

  // the MFMAs of the stage in LDS buffer `buf`
  auto mfma_stage = [&](int buf) {
    if (!multiplies) return;
    const uint16_t* pa = sA[buf] + (wm + (lane & 31)) * STRIDE + 8 * (lane >> 5);
    const uint16_t* pb = sB[buf] + (wn + (lane & 31)) * STRIDE + 8 * (lane >> 5);
#pragma unroll
    for (int kk = 0; kk < TKS; kk += 16) {
      const bf16x8 a = *(const bf16x8*)(pa + kk);
      const bf16x8 b = *(const bf16x8*)(pb + kk);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
  };
  constexpr int NC = STAGE_CHUNKS<TILE, TKS>;
  uint4 ra[NC], rb[NC];
  load_tile<TILE, TKS>(g.A, g.lda, m0, kb, ra);
  load_tile<TILE, TKS>(g.B, g.ldb, n0, kb, rb);
  store_tile<TILE, TKS>(sA[0], ra);
  store_tile<TILE, TKS>(sB[0], rb);
  __syncthreads();
  // software pipeline: the next stage's loads are in flight during this
  // stage's MFMAs; the last stage is peeled off, so the staging registers
  // are written on every pass of the loop (a conditional load kept them in
  // scratch memory, and the loads were waited for at once)
  if constexpr (NBUF > 1) {
    for (int s = 0; s + 1 < nst; ++s) {
      const int cur = s & 1;
      load_tile<TILE, TKS>(g.A, g.lda, m0, kb + (s + 1) * TKS, ra);
      load_tile<TILE, TKS>(g.B, g.ldb, n0, kb + (s + 1) * TKS, rb);
      mfma_stage(cur);
      store_tile<TILE, TKS>(sA[cur ^ 1], ra);
      store_tile<TILE, TKS>(sB[cur ^ 1], rb);
      __syncthreads();
    }
  }
  mfma_stage((nst - 1) & 1);
  if (!multiplies) return;

  // lane l, register r holds C[(r%4) + 8(r/4) + 4(l/32)][l%32] of the wave
  float* C = g.C + (int64_t)blockIdx.z * g.M * g.N + n0 + wn + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r)
    C[(int64_t)(m0 + wm + (r & 3) + 8 * (r >> 2) + 4 * (lane >> 5)) * g.N] = acc[r];
}

// C = A B^T for n (1..3) problems with the same K, K split and tile size, and
// the column sums cs (nullable) in the same launch.
hipError_t gemm_group(const GemmArgs* gs, int n, hipStream_t st, const ColSegs* cs = nullptr,
                      float* cpart = nullptr) {
  const int ks = gs[0].ksplit > 1 ? gs[0].ksplit : 1;
  const int K = gs[0].K / ks;
  int64_t tiles64 = 0;
  for (int i = 0; i < n; ++i) tiles64 += (int64_t)(gs[i].N / 64) * (gs[i].M / 64);
  const int tile = tiles64 * ks < 128 && K % 64 == 0 ? 32 : 64;
  GemmGroup gg;
  memset(&gg, 0, sizeof(gg));
  gg.nprob = n;
  gg.first[0] = 0;
  for (int i = 0; i < n; ++i) {
    gg.g[i] = gs[i];
    gg.first[i + 1] = gg.first[i] + (gs[i].N / tile) * (gs[i].M / tile);
  }
  int extra = 0;
  if (cs) {
    gg.cs = *cs;
    gg.cpart = cpart;
    extra = (cs->tile0[cs->nseg] * CS_RC + ks - 1) / ks;
  }
  const dim3 grid(gg.first[n] + extra, 1, ks);
  auto run = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, gg);
    return hipGetLastError();
  };
  if (tile == 64) {
    if (K == 128) return run(gemm_bf16_kernel<64, 128, 1>);
    if (K % 128 == 0) return run(gemm_bf16_kernel<64, 128, 2>);
    return run(gemm_bf16_kernel<64, 32, 2>);
  }
  if (K == 128) return run(gemm_bf16_kernel<32, 128, 1>);
  return run(gemm_bf16_kernel<32, 64, 2>);
}

// --------------------------------------------------- mixture likelihood
//
// Eight threads per sample, thread k owning mixture component k.  Output row
// O = (8 logits, 8x7 means, 8x7 log standard deviations, 8 pad); target row
// y[7], target 3 periodic on [0, 1).  loss_row = -log p(y)/n and dO = d loss
// / dO (pad entries 0), in FP64:
//   log pi_k = logit_k - logsumexp(logit),  r_kd = y_d - mu_kd (wrapped),
//   a_k = log pi_k + sum_d [-r^2/(2 s^2) - log s - log(2 pi)/2],
//   gamma_k = exp(a_k - logsumexp(a)),
//   dlogit_k = (pi_k - gamma_k)/n, dmu = -gamma r/s^2/n,
//   dlog s = -gamma (r^2/s^2 - 1)/n.
// The maxima and sums over the eight components are butterflies inside each
// group of eight lanes (a fixed order, so the result is deterministic).
__device__ __forceinline__ double grp8_max(double v) {
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) v = fmax(v, __shfl_xor(v, m, 8));
  return v;
}
__device__ __forceinline__ double grp8_sum(double v) {
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) v += __shfl_xor(v, m, 8);
  return v;
}

// One sample's row in LDS: its outputs on entry, dO on return (thread k reads
// and writes component k's entries only).  Returns the row's loss.
__device__ __forceinline__ float nll_row(float* o, const float* y, int k, double inv_n) {
  const double HALF_LOG_2PI = 0.91893853320467274178;
  const double logit = (double)o[k];
  const double lse_l = [&] {
    const double m = grp8_max(logit);
    return m + log(grp8_sum(exp(logit - m)));
  }();
  double r[DM], is2[DM];
  double a = logit - lse_l;
#pragma unroll
  for (int d = 0; d < DM; ++d) {
    double rr = (double)y[d] - (double)o[KM + k * DM + d];
    if (d == MLP_PERIODIC) rr -= floor(rr + 0.5);
    const double ls = (double)o[KM + KM * DM + k * DM + d];
    is2[d] = exp(-2.0 * ls);
    r[d] = rr;
    a += -0.5 * rr * rr * is2[d] - ls - HALF_LOG_2PI;
  }
  const double amax = grp8_max(a);
  const double lp = amax + log(grp8_sum(exp(a - amax)));
  const double gam = exp(a - lp);
  const double pi = exp(logit - lse_l);
  o[k] = (float)((pi - gam) * inv_n);
#pragma unroll
  for (int d = 0; d < DM; ++d) {
    o[KM + k * DM + d] = (float)(-gam * r[d] * is2[d] * inv_n);
    o[KM + KM * DM + k * DM + d] = (float)(-gam * (r[d] * r[d] * is2[d] - 1.0) * inv_n);
  }
  o[NO + k] = 0.0f;  // the eight pad columns
  return (float)(-lp * inv_n);
}

// ------------------------------------------------------- rows of a batch
//
// Everything that a sample's row goes through on its own: the three layers,
// and in training the likelihood and the gradients of the two hidden layers.
// A block of 16 waves takes 32 rows and keeps their activations in LDS; each
// wave owns 32 of a layer's 512 columns (the output's 128: four waves) and
// streams their weights from L2 in the order in which its matrix instructions
// take them ("fragments": 64 lanes x 16 bytes per 32 columns x 16 k), eight
// fragments in flight, a layer's first ones issued before the barrier that
// ends the layer before.  k ascends, so every output is the same chain of
// instructions as in a product of its own.  Bound by the weights' way into
// the block (0.9 MB forward, 1.6 MB with the gradients) and by the chain of
// five products; with a launch per product (7 to 11 us each, most of it the
// launch and one round trip to memory) 1024 rows took 24 us forward and 54 us
// with the gradients, here 16 and 29.
// Written for the weight gradients (training): inputs, activations and
// gradients transposed [columns][ldt]; for the bias gradients the FP32
// gradients; the rows' losses.
constexpr int FRAG = 512;  // elements of a fragment
// fragment arrays of the weights: W1, W2, W3 by (output column, input k), and
// for the gradients W2, W3 by (input column, output k)
constexpr int64_t OFF_F1 = 0;
constexpr int64_t OFF_F2 = OFF_F1 + (int64_t)NB * NH;
constexpr int64_t OFF_F3 = OFF_F2 + (int64_t)NH * NH;
constexpr int64_t OFF_R2 = OFF_F3 + (int64_t)NH * NOP;
constexpr int64_t OFF_R3 = OFF_R2 + (int64_t)NH * NH;
constexpr int64_t N_FRAG = OFF_R3 + (int64_t)NH * NOP;

struct RowArgs {
  const uint16_t* x;  // [rows][256]
  int64_t rows;
  const uint16_t* wf;  // fragments
  const float* p;      // parameters (the biases)
  float* out;          // [rows][128] (inference)
  // training
  const float* y;      // [rows][7]
  uint16_t *xT, *h1T, *h2T, *dobT, *dz2T, *dz1T;  // [columns][ldt]
  int64_t ldt;
  float *dof, *dz2f, *dz1f, *lrow;
  // captured training: rows [k mod per) * rows ... of (x, y), k = dstep[0],
  // which is noted in dstep[1] for the kernels after this one (the Adam
  // kernel moves dstep[0] on)
  int64_t* dstep;
  int64_t per;
};

constexpr int RB = 32;                       // rows of a block
constexpr int SX = NB + 8, SH = NH + 8, SD = NOP + 8, SO = NOP + 4;  // padded LDS rows
constexpr int PF = 8;                        // fragments in flight
constexpr int ROW_THREADS = 1024;            // threads of a block
// Rows of a launch at most (2^31 threads; a grid must stay below 2^32).
constexpr int64_t ROWS_MAX = (int64_t)1 << 26;
static_assert(ROWS_MAX % RB == 0 && ROWS_MAX / RB * ROW_THREADS < (int64_t)1 << 32, "grid");

__device__ __forceinline__ void frag_load(uint4* pre, const uint4* __restrict__ f) {
#pragma unroll
  for (int i = 0; i < PF; ++i) pre[i] = f[i * 64];
}
// acc += (32 rows at pa, a lane's row and half of 16 k) x (KB fragments at f,
// the first PF of them in pre)
template <int KB>
__device__ __forceinline__ f32x16 frag_mul(const uint16_t* pa, const uint4* __restrict__ f,
                                           uint4* pre) {
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const bf16x8 a = *(const bf16x8*)(pa + 16 * kb);
    const uint4 w = pre[kb % PF];
    if (kb + PF < KB) pre[kb % PF] = f[(kb + PF) * 64];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, w), acc, 0, 0, 0);
  }
  return acc;
}
// Row of accumulator register r in lane l: (r % 4) + 8 (r / 4) + 4 (l / 32);
// its column: l % 32.
__device__ __forceinline__ int acc_row(int r, int lane) {
  return (r & 3) + 8 * (r >> 2) + 4 * (lane >> 5);
}
// Four consecutive rows of a lane's column, transposed to global memory.
__device__ __forceinline__ void store_t(uint16_t* T, int64_t ldt, int n, int64_t row,
                                        const uint16_t* h) {
  *(ushort4*)(T + (int64_t)n * ldt + row) = {h[0], h[1], h[2], h[3]};
}

template <bool TRAIN>
__global__ __launch_bounds__(ROW_THREADS) void net_rows_kernel(RowArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t sX[RB * SX], sH1[RB * SH], sH2[RB * SH];
  __shared__ __attribute__((aligned(16))) float sO[TRAIN ? RB * SO : 4];
  __shared__ __attribute__((aligned(16))) uint16_t sD[TRAIN ? RB * SD : 8];
  __shared__ __attribute__((aligned(16))) uint16_t sZ[TRAIN ? RB * SH : 8];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int64_t row0 = (int64_t)blockIdx.x * RB;
  int64_t r0 = 0;
  if (TRAIN && a.dstep) {
    r0 = (a.dstep[0] % a.per) * a.rows;
    if (blockIdx.x == 0 && t == 0) a.dstep[1] = a.dstep[0];
  }
  const uint4* wf = (const uint4*)a.wf + lane;
  const uint4* f1 = wf + (OFF_F1 + (int64_t)wave * (NB / 16) * FRAG) / 8;
  const uint4* f2 = wf + (OFF_F2 + (int64_t)wave * (NH / 16) * FRAG) / 8;
  const uint4* f3 = wf + (OFF_F3 + (int64_t)(wave & 3) * (NH / 16) * FRAG) / 8;
  const uint4* g2 = wf + (OFF_R2 + (int64_t)wave * (NH / 16) * FRAG) / 8;
  const uint4* g3 = wf + (OFF_R3 + (int64_t)wave * (NOP / 16) * FRAG) / 8;
  const int pr = lane & 31, pk = 8 * (lane >> 5);  // the lane's row and k in LDS
  const int n = 32 * wave + pr;                    // its column in a hidden layer
  uint4 pre[PF];
  frag_load(pre, f1);
  {
    const int64_t r = row0 + (t >> 5);
    const uint4 v =
        *(const uint4*)(a.x + (r0 + (r < a.rows ? r : a.rows - 1)) * NB + (t & 31) * 8);
    *(uint4*)(sX + (t >> 5) * SX + (t & 31) * 8) = v;
  }
  __syncthreads();
  // hidden layers: bias, ReLU
  auto hidden = [&](const f32x16& acc, float bias, uint16_t* sH, uint16_t* T) {
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      uint16_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        h[i] = f2bf(fmaxf(acc[4 * r4 + i] + bias, 0.0f));
        sH[acc_row(4 * r4 + i, lane) * SH + n] = h[i];
      }
      if (TRAIN) store_t(T, a.ldt, n, row0 + acc_row(4 * r4, lane), h);
    }
  };
  {
    const float b1 = a.p[OFF_B1 + n];
    const f32x16 acc = frag_mul<NB / 16>(sX + pr * SX + pk, f1, pre);
    frag_load(pre, f2);
    hidden(acc, b1, sH1, a.h1T);
  }
  if (TRAIN) {  // the inputs transposed: 8 rows of a column per thread
    const int c = t >> 2, rb = (t & 3) * 8;
    uint16_t o[8] __attribute__((aligned(16)));
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = sX[(rb + i) * SX + c];
    *(uint4*)(a.xT + (int64_t)c * a.ldt + row0 + rb) = *(const uint4*)o;
  }
  __syncthreads();
  {
    const float b2 = a.p[OFF_B2 + n];
    const f32x16 acc = frag_mul<NH / 16>(sH1 + pr * SH + pk, f2, pre);
    if (wave < 4)
      frag_load(pre, f3);
    else if (TRAIN)
      frag_load(pre, g3);
    hidden(acc, b2, sH2, a.h2T);
  }
  __syncthreads();
  if (wave < 4) {
    const float b3 = a.p[OFF_B3 + n];
    const f32x16 acc = frag_mul<NH / 16>(sH2 + pr * SH + pk, f3, pre);
    if (TRAIN) frag_load(pre, g3);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = acc_row(r, lane);
      if constexpr (TRAIN)
        sO[m * SO + n] = acc[r] + b3;
      else if (row0 + m < a.rows)
        a.out[(row0 + m) * NOP + n] = acc[r] + b3;
    }
  }
  if constexpr (TRAIN) {
    __syncthreads();
    if (wave < 4) {
      const int i = t >> 3, k = t & 7;
      const float l = nll_row(sO + i * SO, a.y + (r0 + row0 + i) * DM, k, 1.0 / (double)a.rows);
      if (k == 0) a.lrow[row0 + i] = l;
    }
    __syncthreads();
    {  // dO in FP32, in BF16 for the product below and transposed
      const int i = t >> 5, c = (t & 31) * 4;
      const float4 v = *(const float4*)(sO + i * SO + c);
      *(float4*)(a.dof + (row0 + i) * NOP + c) = v;
      *(ushort4*)(sD + i * SD + c) = {f2bf(v.x), f2bf(v.y), f2bf(v.z), f2bf(v.w)};
      const int ct = t >> 3, rt = (t & 7) * 4;
      uint16_t h[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) h[j] = f2bf(sO[(rt + j) * SO + ct]);
      store_t(a.dobT, a.ldt, ct, row0 + rt, h);
    }
    __syncthreads();
    // dZ = (gradient of the layer above) W^T * [H > 0]
    auto grad = [&](const f32x16& acc, const uint16_t* sH, uint16_t* sZ_, float* F, uint16_t* T) {
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        uint16_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = acc_row(4 * r4 + i, lane);
          const uint16_t act = sH[m * SH + n];
          const float v = (act == 0 || (act & 0x8000u)) ? 0.0f : acc[4 * r4 + i];
          h[i] = f2bf(v);
          if (sZ_) sZ_[m * SH + n] = h[i];
          F[(row0 + m) * NH + n] = v;
        }
        store_t(T, a.ldt, n, row0 + acc_row(4 * r4, lane), h);
      }
    };
    {
      const f32x16 acc = frag_mul<NOP / 16>(sD + pr * SD + pk, g3, pre);
      frag_load(pre, g2);
      grad(acc, sH2, sZ, a.dz2f, a.dz2T);
    }
    __syncthreads();
    const f32x16 acc = frag_mul<NH / 16>(sZ + pr * SH + pk, g2, pre);
    grad(acc, sH1, nullptr, a.dz1f, a.dz1T);
  }
}

// Sum of ks partial matrices part[z][i], z in order (split-K reduction).
__global__ void splitk_reduce_kernel(const float* part, int ks, int64_t n, float* out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    float t = part[i];
    for (int z = 1; z < ks; ++z) t += part[(int64_t)z * n + i];
    out[i] = t;
  }
}

// The three weight matrices in 32 x 32 tiles, then the biases: the tiles that
// the kernels writing the BF16 weights in both orders take, one per block.
constexpr int WT1 = (NB / 32) * (NH / 32), WT2 = (NH / 32) * (NH / 32),
              WT3 = (NH / 32) * (NOP / 32);
constexpr int W_TILES = WT1 + WT2 + WT3;
constexpr int N_BIAS = NH + NH + NOP;
constexpr int W_BLOCKS = W_TILES + (N_BIAS + 255) / 256;
struct WTile {
  int64_t off;         // the matrix in the parameters
  int64_t off_f;       // its fragments for the forward pass and, if any, for
  int64_t off_r;       // the gradients (-1: none)
  int rows, cols;      // [rows = inputs][cols = outputs]
  int r0, c0;          // the tile's first row and column
  int tensor;          // 0: W3, 1: W2, 2: W1 (the order of KParts)
};
__device__ __forceinline__ WTile weight_tile(int b) {
  WTile w;
  if (b < WT1)
    w = {OFF_W1, OFF_F1, -1, NB, NH, 0, 0, 2};
  else if (b < WT1 + WT2)
    w = {OFF_W2, OFF_F2, OFF_R2, NH, NH, 0, 0, 1}, b -= WT1;
  else
    w = {OFF_W3, OFF_F3, OFF_R3, NH, NOP, 0, 0, 0}, b -= WT1 + WT2;
  w.r0 = b / (w.cols / 32) * 32;
  w.c0 = b % (w.cols / 32) * 32;
  return w;
}
// Parameter index of bias entry e (b1, b2, b3 one after another).
__device__ __forceinline__ int64_t bias_index(int e) {
  return e < NH ? OFF_B1 + e : e < 2 * NH ? OFF_B2 + (e - NH) : OFF_B3 + (e - 2 * NH);
}

// Element (column n, k) of a fragment array with KB fragments per 32 columns.
__device__ __forceinline__ int64_t frag_index(int n, int k, int KB) {
  return ((int64_t)(n / 32 * KB + k / 16) * 64 + (n & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
}

// The BF16 weights of a 32 x 32 tile into the fragment arrays: thread t holds
// row t / 8, columns 4 (t % 8) .. + 3 in h.
__device__ __forceinline__ void store_frags(const WTile& w, ushort4 h, uint16_t* wf,
                                            uint16_t (*sh)[36]) {
  const int t = threadIdx.x, r = t >> 3, c = (t & 7) * 4;
  if (w.off_r >= 0)
    *(ushort4*)(wf + w.off_r + frag_index(w.r0 + r, w.c0 + c, w.cols / 16)) = h;
  sh[c][r] = h.x;
  sh[c + 1][r] = h.y;
  sh[c + 2][r] = h.z;
  sh[c + 3][r] = h.w;
  __syncthreads();
  *(ushort4*)(wf + w.off_f + frag_index(w.c0 + r, w.r0 + c, w.rows / 16)) =
      *(const ushort4*)&sh[r][c];
}

// The BF16 weights of the FP32 parameters.
__global__ __launch_bounds__(256) void shadow_kernel(const float* p, uint16_t* wf) {
  __shared__ __attribute__((aligned(8))) uint16_t sh[32][36];
  const int t = threadIdx.x;
  const WTile w = weight_tile(blockIdx.x);
  const int64_t i = w.off + (int64_t)(w.r0 + (t >> 3)) * w.cols + w.c0 + (t & 7) * 4;
  const float4 x = *(const float4*)(p + i);
  store_frags(w, {f2bf(x.x), f2bf(x.y), f2bf(x.z), f2bf(x.w)}, wf, sh);
}

// Adam (Kingma & Ba 2015) with bias correction factors c1 = 1/(1 - b1^t),
// c2 = 1/(1 - b2^t):  p -= lr * (m c1) / (sqrt(v c2) + eps).  1 - b1 and 1 - b2
// come from the host in double (1.0f - 0.999f would carry a 1e-5 relative
// error into v).
struct AdamArgs {
  float *p, *m, *v;
  float b1, b2, omb1, omb2, eps;
};
__device__ __forceinline__ float adam_update(const AdamArgs& a, float p, float gi, float& m,
                                             float& v, float lr, float c1, float c2) {
  const float mi = a.b1 * m + a.omb1 * gi;
  const float vi = a.b2 * v + a.omb2 * (gi * gi);
  m = mi;
  v = vi;
  return p - lr * (mi * c1) / (sqrtf(vi * c2) + a.eps);
}

// The split-K partials of the three weight gradients of one step (a buffer
// each), for the graph form of training: the Adam kernel sums them.
struct KParts {
  const float* part[3];  // W3, W2, W1
  int ks;                // partials per tensor (1: none, the GEMM wrote the gradient)
};

// The column-sum partials of one step: the three bias gradients (b3, b2, b1)
// and the loss.
struct CParts {
  const float* part;  // [CS_RC][ncol_all]
  int ncol_all;
  int col0[3];        // first columns of b3, b2, b1 in part
  int loss_col;
};

// One Adam step, writing the BF16 weights' fragments.  Alone (dstep null)
// it takes the gradient g and the given learning rate and correction factors.
// In the captured training graph the step's learning rate and correction
// factors are sched[3k .. 3k+2] (k = dstep[1]); a weight tensor's gradient is
// first summed over its split-K partials, in range order (as splitk_reduce
// sums them), a bias gradient and the loss over their column-sum partials,
// in row-chunk order (as colsum_stage2 sums them); the gradients are stored
// to g, the loss to losses[k], and the counter moves on (dstep[0] = k + 1,
// which no block of this launch reads).
__global__ __launch_bounds__(256) void adam_kernel(AdamArgs a, float* g, uint16_t* wf,
                                                   float lr, float c1, float c2,
                                                   const float* sched, int64_t* dstep, KParts kp,
                                                   CParts cp, float* losses) {
  __shared__ __attribute__((aligned(8))) uint16_t sh[32][36];
  const int b = blockIdx.x, t = threadIdx.x;
  if (dstep) {
    const int64_t k = dstep[1];
    lr = sched[3 * k];
    c1 = sched[3 * k + 1];
    c2 = sched[3 * k + 2];
    if (b == W_TILES && t == 0) {
      float sum = cp.part[cp.loss_col];
      for (int rc = 1; rc < CS_RC; ++rc) sum += cp.part[(int64_t)rc * cp.ncol_all + cp.loss_col];
      losses[k] = sum;
      dstep[0] = k + 1;
    }
  }
  if (b >= W_TILES) {
    const int e = (b - W_TILES) * 256 + t;
    if (e >= N_BIAS) return;
    const int64_t i = bias_index(e);
    float gi;
    if (dstep) {
      const int c = e < NH ? cp.col0[2] + e : e < 2 * NH ? cp.col0[1] + (e - NH)
                                                         : cp.col0[0] + (e - 2 * NH);
      gi = cp.part[c];
      for (int rc = 1; rc < CS_RC; ++rc) gi += cp.part[(int64_t)rc * cp.ncol_all + c];
      g[i] = gi;
    } else {
      gi = g[i];
    }
    float m = a.m[i], v = a.v[i];
    const float x = adam_update(a, a.p[i], gi, m, v, lr, c1, c2);
    a.p[i] = x;
    a.m[i] = m;
    a.v[i] = v;
    return;
  }
  const WTile w = weight_tile(b);
  const int64_t j = (int64_t)(w.r0 + (t >> 3)) * w.cols + w.c0 + (t & 7) * 4, i = w.off + j;
  float4 gi;
  if (dstep && kp.ks > 1) {
    const float* part = kp.part[w.tensor];
    const int64_t mn = (int64_t)w.rows * w.cols;
    gi = *(const float4*)(part + j);
#pragma unroll 8
    for (int z = 1; z < kp.ks; ++z) {
      const float4 q = *(const float4*)(part + z * mn + j);
      gi.x += q.x;
      gi.y += q.y;
      gi.z += q.z;
      gi.w += q.w;
    }
    *(float4*)(g + i) = gi;
  } else {
    gi = *(const float4*)(g + i);
  }
  float4 x = *(const float4*)(a.p + i), m = *(const float4*)(a.m + i), v = *(const float4*)(a.v + i);
  x.x = adam_update(a, x.x, gi.x, m.x, v.x, lr, c1, c2);
  x.y = adam_update(a, x.y, gi.y, m.y, v.y, lr, c1, c2);
  x.z = adam_update(a, x.z, gi.z, m.z, v.z, lr, c1, c2);
  x.w = adam_update(a, x.w, gi.w, m.w, v.w, lr, c1, c2);
  *(float4*)(a.p + i) = x;
  *(float4*)(a.m + i) = m;
  *(float4*)(a.v + i) = v;
  store_frags(w, {f2bf(x.x), f2bf(x.y), f2bf(x.z), f2bf(x.w)}, wf, sh);
}

// He-normal weights (std sqrt(2/fan_in); output layer std 0.01), zero
// biases.  Normal deviates by the Box-Muller transform of two Philox words.
__global__ void mlp_init_kernel(float* p, uint64_t seed) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < NP_DEV;
       i += (int64_t)gridDim.x * blockDim.x) {
    float val = 0.0f;
    double sd = 0.0;
    if (i < OFF_B1) sd = sqrt(2.0 / NB);
    else if (i >= OFF_W2 && i < OFF_B2) sd = sqrt(2.0 / NH);
    else if (i >= OFF_W3 && i < OFF_B3 && (i - OFF_W3) % NOP < NO) sd = 0.01;
    if (sd > 0.0) {
      const u64x4 w = philox4x64_10(0, P_MLP_INIT, (uint64_t)i, 0, seed, 0);
      const double u1 = u01(w.v[0]), u2 = u01(w.v[1]);
      val = (float)(sd * sqrt(-2.0 * log(u1)) * cos(2.0 * M_PI * u2));
    }
    p[i] = val;
  }
}

// ------------------------------------------------------------ resampling
//
// Shared by sblm_resample and mlp_make_data; 256 threads, thread j owns
// bin j.  On entry v is the thread's bin value and `filled` its flag.
// Empty bins take the linear interpolation of the nearest filled bins on
// either side, evaluated as v_l + (v_h - v_l)(j - l)/(h - l) (the nearest
// filled value beyond the last filled bin at either end); then the bins are
// normalised as (v - median)/max(max - median, 1e-12), the median of 256
// values being the mean of the two central order statistics.
struct BinScratch {
  double val[NB], srt[NB];
  unsigned long long filled[NB / 64];  // bit j % 64 of word j / 64: bin j
};

// Nearest filled bin below / above j (-1 / NB: none).
__device__ __forceinline__ int filled_below(const unsigned long long* f, int j) {
  int w = j >> 6;
  unsigned long long m = f[w] & ((1ull << (j & 63)) - 1ull);
  while (!m && w > 0) m = f[--w];
  return m ? 64 * w + 63 - __builtin_clzll(m) : -1;
}
__device__ __forceinline__ int filled_above(const unsigned long long* f, int j) {
  int w = j >> 6;
  unsigned long long m = (f[w] >> (j & 63)) >> 1 << (j & 63) << 1;
  while (!m && w < NB / 64 - 1) m = f[++w];
  return m ? 64 * w + __builtin_ctzll(m) : NB;
}

__device__ __forceinline__ void finish_bins(BinScratch& sc, double v, bool filled, float* xf,
                                            uint16_t* xb) {
  const int j = threadIdx.x;
  const unsigned long long fw = __ballot(filled);
  if ((j & 63) == 0) sc.filled[j >> 6] = fw;
  sc.val[j] = v;
  __syncthreads();
  if (!(sc.filled[0] | sc.filled[1] | sc.filled[2] | sc.filled[3])) {
    if (xf) xf[j] = 0.0f;
    if (xb) xb[j] = 0;
    return;
  }
  if (!filled) {
    const int l = filled_below(sc.filled, j), h = filled_above(sc.filled, j);
    if (l >= 0 && h < NB)
      v = sc.val[l] + (sc.val[h] - sc.val[l]) * (double)(j - l) / (double)(h - l);
    else
      v = (l >= 0) ? sc.val[l] : sc.val[h];
  }
  sc.srt[j] = v;
  __syncthreads();
  // bitonic sort of srt[0..255], ascending; exchanges at a distance below 64
  // stay within a wave's own 64 entries and need no barrier (3 of 36 cross)
  for (int k = 2; k <= NB; k <<= 1) {
    for (int s = k >> 1; s > 0; s >>= 1) {
      const int p = j ^ s;
      if (p > j) {
        const double x = sc.srt[j], y = sc.srt[p];
        const bool up = (j & k) == 0;
        if ((x > y) == up) {
          sc.srt[j] = y;
          sc.srt[p] = x;
        }
      }
      if (s >= 64 || (s == 1 && k >= 64))
        __syncthreads();
      else
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
  const double med = (sc.srt[NB / 2 - 1] + sc.srt[NB / 2]) / 2.0;
  const double div = fmax(sc.srt[NB - 1] - med, 1e-12);
  const double r = (v - med) / div;
  if (xf) xf[j] = (float)r;
  if (xb) xb[j] = f2bf((float)r);
}

__device__ __forceinline__ int bin_of(double t, double t_a, double span) {
  if (span <= 0.0) return 0;
  const double u = (t - t_a) / span * (double)NB;
  return (int)fmin(u, (double)(NB - 1));
}

// One block of 256 threads per lightcurve (t ascending within each).  The
// epochs pass through LDS in chunks of 1024, loaded coalesced (the next
// chunk in flight while this one is summed); the thread that finds the first
// epoch of a bin notes it, and thread j then sums bin j's epochs in order.
// Bound by latency: one chain per lightcurve of a chunk's loads and the sum of
// its fullest bin.  1024 lightcurves of 200-5000 epochs: 71 -> 30 us (before,
// every bin searched the epochs in global memory and summed from there).
constexpr int RS_PER = 4, RS_CHUNK = 256 * RS_PER;

__global__ __launch_bounds__(256) void resample_kernel(const int64_t* off,
                                                       const double* __restrict__ t,
                                                       const double* __restrict__ y,
                                                       const double* __restrict__ w, float* xf,
                                                       uint16_t* xb) {
  __shared__ BinScratch sc;
  __shared__ double sw_[RS_CHUNK], swy_[RS_CHUNK];
  __shared__ int bin[RS_CHUNK], start[NB + 1];
  const int lc = blockIdx.x, j = threadIdx.x;
  const int64_t o0 = off[lc], o1 = off[lc + 1];
  const int64_t L = o1 - o0;
  float* xfl = xf ? xf + (int64_t)lc * NB : nullptr;
  uint16_t* xbl = xb ? xb + (int64_t)lc * NB : nullptr;
  double sw = 0.0, swy = 0.0;
  if (L > 0) {
    const double t_a = t[o0], span = t[o1 - 1] - t_a;
    double rt[RS_PER], rw[RS_PER], ry[RS_PER];
    auto fetch = [&](int64_t c0) {
#pragma unroll
      for (int i = 0; i < RS_PER; ++i) {
        const int64_t e = c0 + i * 256 + j;
        const bool in = e < L;
        rt[i] = in ? t[o0 + e] : 0.0;
        rw[i] = in ? w[o0 + e] : 0.0;
        ry[i] = in ? y[o0 + e] : 0.0;
      }
    };
    fetch(0);
    for (int64_t c0 = 0; c0 < L; c0 += RS_CHUNK) {
      const int n = (int)(L - c0 < RS_CHUNK ? L - c0 : RS_CHUNK);
      start[j] = n;
      if (j == 0) start[NB] = n;
#pragma unroll
      for (int i = 0; i < RS_PER; ++i) {
        const int e = i * 256 + j;
        if (e < n) {
          bin[e] = max(bin_of(rt[i], t_a, span), 0);
          sw_[e] = rw[i];
          swy_[e] = rw[i] * ry[i];
        }
      }
      __syncthreads();
      if (c0 + RS_CHUNK < L) fetch(c0 + RS_CHUNK);
      // first epoch of bin >= b for every bin b
      if (j <= bin[0]) start[j] = 0;
#pragma unroll
      for (int i = 0; i < RS_PER; ++i) {
        const int e = i * 256 + j;
        if (e > 0 && e < n) {
          const int b = bin[e];
          for (int k = bin[e - 1] + 1; k <= b; ++k) start[k] = e;
        }
      }
      __syncthreads();
      const int e1 = start[j + 1];
#pragma unroll 4
      for (int e = start[j]; e < e1; ++e) {
        sw += sw_[e];
        swy += swy_[e];
      }
      __syncthreads();
    }
  }
  finish_bins(sc, sw > 0.0 ? swy / sw : 0.0, sw > 0.0, xfl, xbl);
}

// ------------------------------------------------------- training data
//
// Sample s uses Philox key (seed, s), counter (0, P_DATA, row, j / 4):
//   row 0: words 0..5 the parameters (uniform over the domain below, in the
//          library's plane order), word 6 Fb ~ U[0, 0.5] (Fs = 1), word 7
//          the noise fraction s ~ U[0.005, 0.03], word 8 the epoch count
//          L ~ U{200..5000}, words 9, 10 the start and the end of the
//          observing window, t0 + a tE and t0 + b tE with a ~ U(-3, -2) and
//          b ~ U(2, 3) (the random start and end of Sec. 4.2);
//   row 1 + j: words 0..3 for bin j (Poisson count, two normal deviates).
// The observing window is seen through nightly windows
// [n + 0.1, n + 0.1 + 1/3] days; t_first, t_last are its first and last
// observable instants and span = t_last - t_first.  Bin j covers
// [t_first + span j/256, t_first + span (j+1)/256]; its expected epoch count
// is c_j = n_sched o_j / sum(o) + n_dense d_j / (0.2 tE), with o_j its
// overlap with the nightly windows, d_j its overlap with t0 +- 0.1 tE,
// n_dense = round(L/10), n_sched = L - n_dense; the count is Poisson(c_j)
// (inversion for c_j <= 64, else the rounded normal approximation).  A
// counted bin holds F = Fs A(t_j) + Fb plus N(0, (s F)^2 / count) noise, A
// from the forward model at the bin centre; then empty bins and
// normalisation as for sblm_resample.
//
// Targets: (log10 q + 3)/3, (d - 0.5)/1.5, u0/0.5, alpha/(2 pi),
// (t0 - t_first)/span, tE/span, Fs/(Fs + Fb).
constexpr double NIGHT0 = 0.1, NIGHT_LEN = 1.0 / 3.0;

__device__ void data_window(double t0, double tE, double a, double b, double& t_first,
                            double& t_last) {
  const double ta = t0 + a * tE, tb = t0 + b * tE;
  const double na = floor(ta - NIGHT0);
  t_first = (ta <= na + NIGHT0 + NIGHT_LEN) ? ta : na + 1.0 + NIGHT0;
  const double nb = floor(tb - NIGHT0);
  t_last = (tb <= nb + NIGHT0 + NIGHT_LEN) ? tb : nb + NIGHT0 + NIGHT_LEN;
}

// aux row per sample: t_first, span, t0, tE, Fb, s, L
constexpr int NAUX = 8;

__global__ void data_draw_kernel(uint64_t seed, int64_t first, int n, double* theta,
                                 double* aux, float* y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double DLO[6] = {-3.0, 0.5, 0.0, 0.0, 10.0, -10.0};
  const double DHI[6] = {0.0, 2.0, 0.5, 2.0 * M_PI, 100.0, 10.0};
  const uint64_t s = (uint64_t)(first + i);
  const u64x4 w0 = philox4x64_10(0, P_DATA, 0, 0, seed, s);
  const u64x4 w1 = philox4x64_10(0, P_DATA, 0, 1, seed, s);
  const u64x4 w2 = philox4x64_10(0, P_DATA, 0, 2, seed, s);
  const uint64_t wd[9] = {w0.v[0], w0.v[1], w0.v[2], w0.v[3], w1.v[0],
                          w1.v[1], w1.v[2], w1.v[3], w2.v[0]};
  double th[6];
  for (int g = 0; g < 6; ++g) th[g] = DLO[g] + (DHI[g] - DLO[g]) * u01(wd[g]);
  const double Fb = 0.5 * u01(wd[6]);
  const double sn = 0.005 + 0.025 * u01(wd[7]);
  const double L = (double)(200u + below(wd[8], 4801u));
  const double wa = -3.0 + u01(w2.v[1]), wb = 2.0 + u01(w2.v[2]);
  double t_first, t_last;
  data_window(th[5], th[4], wa, wb, t_first, t_last);
  const double span = t_last - t_first;
  for (int g = 0; g < 4; ++g) theta[(int64_t)g * n + i] = th[g];
  theta[(int64_t)4 * n + i] = th[4] / span;
  theta[(int64_t)5 * n + i] = (th[5] - t_first) / span;
  double* a = aux + (int64_t)i * NAUX;
  a[0] = t_first;
  a[1] = span;
  a[2] = th[5];
  a[3] = th[4];
  a[4] = Fb;
  a[5] = sn;
  a[6] = L;
  a[7] = 0.0;
  float* yy = y + (int64_t)i * DM;
  yy[0] = (float)((th[0] + 3.0) / 3.0);
  yy[1] = (float)((th[1] - 0.5) / 1.5);
  yy[2] = (float)(th[2] / 0.5);
  yy[3] = (float)(th[3] / (2.0 * M_PI));
  yy[4] = (float)((th[5] - t_first) / span);
  yy[5] = (float)(th[4] / span);
  yy[6] = (float)(1.0 / (1.0 + Fb));
}

__device__ __forceinline__ double overlap(double a0, double a1, double b0, double b1) {
  return fmax(0.0, fmin(a1, b1) - fmax(a0, b0));
}

__global__ __launch_bounds__(256) void data_finish_kernel(uint64_t seed, int64_t first,
                                                          const double* aux,
                                                          const double* A, float* xf,
                                                          uint16_t* xb) {
  __shared__ BinScratch sc;
  __shared__ double red[NB], inv[NB];
  const int i = blockIdx.x, j = threadIdx.x;
  const uint64_t s = (uint64_t)(first + i);
  const double* a = aux + (int64_t)i * NAUX;
  const double t_first = a[0], span = a[1], t0 = a[2], tE = a[3], Fb = a[4],
               sn = a[5], L = a[6];
  const double b0 = t_first + span * (double)j / NB;
  const double b1 = t_first + span * (double)(j + 1) / NB;
  double o = 0.0;
  for (double nt = floor(b0) - 1.0; nt <= floor(b1); nt += 1.0)
    o += overlap(b0, b1, nt + NIGHT0, nt + NIGHT0 + NIGHT_LEN);
  const double dj = overlap(b0, b1, t0 - 0.1 * tE, t0 + 0.1 * tE);
  red[j] = o;
  inv[j] = 1.0 / (double)(j + 1);  // for the counts below
  __syncthreads();
  for (int h = NB / 2; h > 0; h >>= 1) {  // fixed-order tree sum
    if (j < h) red[j] += red[j + h];
    __syncthreads();
  }
  const double osum = red[0];
  const double n_dense = floor(0.1 * L + 0.5), n_sched = L - n_dense;
  const double c = (osum > 0.0 ? n_sched * o / osum : 0.0) + n_dense * dj / (0.2 * tE);
  const u64x4 wb = philox4x64_10(0, P_DATA, 1 + (uint64_t)j, 0, seed, s);
  const double r1 = u01(wb.v[1]), r2 = u01(wb.v[2]);
  const double rad = sqrt(-2.0 * log(r1));
  double sn2, cs2;
  sincos(2.0 * M_PI * r2, &sn2, &cs2);
  const double z1 = rad * cs2, z2 = rad * sn2;
  double cnt;
  if (c <= 64.0) {
    // smallest count whose distribution function reaches u: the number of
    // values F_0, F_1, ... (ascending) below u, four per pass (the lanes of a
    // wave count in step, so the reciprocals are broadcast reads)
    const double u = u01(wb.v[0]);
    double p = exp(-c), F = p;
    int n = 0;
    for (int k = 0; u > F && k < 1000; k += 4) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        n += u > F ? 1 : 0;
        p = p * c * (k + m < NB ? inv[k + m] : 1.0 / (double)(k + m + 1));
        F += p;
      }
    }
    cnt = (double)n;
  } else {
    cnt = fmax(0.0, floor(c + sqrt(c) * z2 + 0.5));
  }
  const double flux = A[(int64_t)i * NB + j] + Fb;
  finish_bins(sc, cnt > 0.0 ? flux + sn * flux / sqrt(cnt) * z1 : 0.0, cnt > 0.0,
              xf ? xf + (int64_t)i * NB : nullptr, xb ? xb + (int64_t)i * NB : nullptr);
}

__global__ void bin_centres_kernel(double* u) {
  u[threadIdx.x] = ((double)threadIdx.x + 0.5) / NB;
}

}  // namespace
}  // namespace sblm

using namespace sblm;

// ------------------------------------------------------------- network

struct mlp_net {
  int device = 0;
  int batch_max = 0;
  int64_t step = 0;
  float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
  uint16_t* wf = nullptr;     // BF16 weights in fragments
  uint16_t* xbuf = nullptr;   // [batch_max][256] (rows at an odd address)
  // the batch transposed, [columns][batch_max]: inputs, activations, gradients
  uint16_t *xT = nullptr, *h1T = nullptr, *h2T = nullptr;
  uint16_t *dobT = nullptr, *dz2T = nullptr, *dz1T = nullptr;
  float* dof = nullptr;       // [batch_max][128]
  float *dz2f = nullptr, *dz1f = nullptr;  // [batch_max][512]
  float* lrow = nullptr;      // [batch_max]
  float* kpart = nullptr;     // split-K partials: [KSPLIT_MAX][512 * 512], the
                              // first of three buffers (W2, then W3, W1)
  float* cpart = nullptr;     // column-sum partials, [CS_RC][COLS_ALL] + a loss slot
  // the training graph (mlp_train) and what it reads
  int64_t* dstep = nullptr;   // [2] the graph's step counter, the running step
  float* sched = nullptr;     // [sched_cap][3]: learning rate, c1, c2 per step
  float* losses = nullptr;    // [sched_cap]
  int64_t sched_cap = 0;
  hipStream_t work = nullptr;
  hipEvent_t ev_in = nullptr, ev_out = nullptr;
  hipGraphExec_t train_exec = nullptr;    // one step
  hipGraphExec_t train_exec_n = nullptr;  // GRAPH_STEPS of them
  int64_t train_key[5] = {0, 0, 0, 0, 0};  // batch, x, y, steps per epoch, sched buffer
};

constexpr int KSPLIT_MAX = 8;
constexpr int COLS_ALL = NOP + NH + NH + 1;  // b3, b2, b1 gradients and the loss

// Split-K partial buffers of the three weight gradients (one block).
constexpr int64_t KPART_W2 = 0;
constexpr int64_t KPART_W3 = KPART_W2 + (int64_t)KSPLIT_MAX * NH * NH;
constexpr int64_t KPART_W1 = KPART_W3 + (int64_t)KSPLIT_MAX * NH * NOP;
constexpr int64_t KPART_ALL = KPART_W1 + (int64_t)KSPLIT_MAX * NB * NH;

static void net_free(mlp_net* n) {
  if (n->train_exec) (void)hipGraphExecDestroy(n->train_exec);
  if (n->train_exec_n) (void)hipGraphExecDestroy(n->train_exec_n);
  void* ptrs[] = {n->p,    n->g,    n->m,    n->v,    n->wf,    n->xbuf,  n->xT,
                  n->h1T,  n->h2T,  n->dobT, n->dz2T, n->dz1T,  n->dof,   n->dz2f,
                  n->dz1f, n->lrow, n->kpart, n->cpart, n->dstep, n->sched, n->losses};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  if (n->ev_in) (void)hipEventDestroy(n->ev_in);
  if (n->ev_out) (void)hipEventDestroy(n->ev_out);
  if (n->work) (void)hipStreamDestroy(n->work);
}

static int grid_for(int64_t n) {
  return (int)std::min<int64_t>((n + 255) / 256, 4096);
}

// The BF16 weights from the FP32 parameters (null stream).
static hipError_t shadow(mlp_net* n) {
  hipLaunchKernelGGL(shadow_kernel, dim3(W_TILES), dim3(256), 0, nullptr, n->p, n->wf);
  return hipGetLastError();
}

extern "C" int mlp_create(int32_t batch_max, uint64_t seed, mlp_net** out) {
  if (!out) return set_error(SBLM_EINVAL, "mlp_create: null out");
  *out = nullptr;
  if (batch_max < 64 || batch_max % 64 != 0)
    return set_error(SBLM_EINVAL, "mlp_create: batch_max = %d is not a positive multiple of 64",
                     batch_max);
  if (batch_max > (1 << 20))
    return set_error(SBLM_ERANGE, "mlp_create: batch_max = %d beyond 2^20", batch_max);
  mlp_net* n = new (std::nothrow) mlp_net();
  if (!n) return set_error(SBLM_ENOMEM, "mlp_create: host allocation");
  n->batch_max = batch_max;
  if (hipGetDevice(&n->device) != hipSuccess) {
    delete n;
    return set_error(SBLM_EDEVICE, "mlp_create: hipGetDevice");
  }
  const size_t B = (size_t)batch_max;
  bool ok = hipMalloc(&n->p, NP_DEV * 4) == hipSuccess &&
            hipMalloc(&n->g, NP_DEV * 4) == hipSuccess &&
            hipMalloc(&n->m, NP_DEV * 4) == hipSuccess &&
            hipMalloc(&n->v, NP_DEV * 4) == hipSuccess &&
            hipMalloc(&n->wf, N_FRAG * 2) == hipSuccess &&
            hipMalloc(&n->xT, B * NB * 2) == hipSuccess &&
            hipMalloc(&n->h1T, B * NH * 2) == hipSuccess &&
            hipMalloc(&n->h2T, B * NH * 2) == hipSuccess &&
            hipMalloc(&n->dobT, B * NOP * 2) == hipSuccess &&
            hipMalloc(&n->dz2T, B * NH * 2) == hipSuccess &&
            hipMalloc(&n->dz1T, B * NH * 2) == hipSuccess &&
            hipMalloc(&n->xbuf, B * NB * 2) == hipSuccess &&
            hipMalloc(&n->dof, B * NOP * 4) == hipSuccess &&
            hipMalloc(&n->dz2f, B * NH * 4) == hipSuccess &&
            hipMalloc(&n->dz1f, B * NH * 4) == hipSuccess &&
            hipMalloc(&n->lrow, B * 4) == hipSuccess &&
            hipMalloc(&n->kpart, (size_t)KPART_ALL * 4) == hipSuccess &&
            hipMalloc(&n->cpart, ((size_t)CS_RC * COLS_ALL + 1) * 4) == hipSuccess &&
            hipMalloc(&n->dstep, 16) == hipSuccess &&
            hipStreamCreateWithFlags(&n->work, hipStreamNonBlocking) == hipSuccess &&
            hipEventCreateWithFlags(&n->ev_in, hipEventDisableTiming) == hipSuccess &&
            hipEventCreateWithFlags(&n->ev_out, hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    net_free(n);
    delete n;
    return set_error(SBLM_ENOMEM, "mlp_create: device allocation");
  }
  hipLaunchKernelGGL(mlp_init_kernel, dim3(grid_for(NP_DEV)), dim3(256), 0, nullptr, n->p, seed);
  int rc = check_hip(hipGetLastError(), "mlp_create: init launch");
  if (rc == SBLM_OK) rc = check_hip(shadow(n), "mlp_create: shadow launch");
  if (rc == SBLM_OK)
    rc = check_hip(hipMemset(n->g, 0, NP_DEV * 4), "mlp_create: memset");
  if (rc == SBLM_OK)
    rc = check_hip(hipMemset(n->m, 0, NP_DEV * 4), "mlp_create: memset");
  if (rc == SBLM_OK)
    rc = check_hip(hipMemset(n->v, 0, NP_DEV * 4), "mlp_create: memset");
  if (rc == SBLM_OK) rc = check_hip(hipDeviceSynchronize(), "mlp_create: init");
  if (rc != SBLM_OK) {
    net_free(n);
    delete n;
    return rc;
  }
  *out = n;
  return SBLM_OK;
}

extern "C" void mlp_destroy(mlp_net* n) {
  if (!n) return;
  (void)hipDeviceSynchronize();
  net_free(n);
  delete n;
}

// canonical (host) order: W1 [256][512], b1, W2 [512][512], b2, W3 [512][120], b3 [120]
static void canon_map(int64_t* dst_of_src) {
  int64_t k = 0;
  for (int64_t i = 0; i < OFF_W3; ++i) dst_of_src[k++] = i;
  for (int r = 0; r < NH; ++r)
    for (int c = 0; c < NO; ++c) dst_of_src[k++] = OFF_W3 + (int64_t)r * NOP + c;
  for (int c = 0; c < NO; ++c) dst_of_src[k++] = OFF_B3 + c;
}

static int copy_canonical(mlp_net* n, float* dev, float* host, bool to_host,
                          const char* who) {
  float* tmp = (float*)calloc(NP_DEV, sizeof(float));
  int64_t* map = (int64_t*)malloc(MLP_NPARAMS * sizeof(int64_t));
  if (!tmp || !map) {
    free(tmp);
    free(map);
    return set_error(SBLM_ENOMEM, "%s: host allocation", who);
  }
  canon_map(map);
  int rc = SBLM_OK;
  if (to_host) {
    rc = check_hip(hipMemcpy(tmp, dev, NP_DEV * 4, hipMemcpyDeviceToHost), who);
    if (rc == SBLM_OK)
      for (int64_t i = 0; i < MLP_NPARAMS; ++i) host[i] = tmp[map[i]];
  } else {
    for (int64_t i = 0; i < MLP_NPARAMS; ++i) tmp[map[i]] = host[i];
    rc = check_hip(hipMemcpy(dev, tmp, NP_DEV * 4, hipMemcpyHostToDevice), who);
  }
  free(tmp);
  free(map);
  (void)n;
  return rc;
}

extern "C" int mlp_set_params(mlp_net* n, const float* params) {
  if (!n || !params) return set_error(SBLM_EINVAL, "mlp_set_params: null argument");
  // (queued steps and forward passes read and write what is replaced here)
  int rc = check_hip(hipDeviceSynchronize(), "mlp_set_params");
  if (rc != SBLM_OK) return rc;
  rc = copy_canonical(n, n->p, (float*)params, false, "mlp_set_params");
  if (rc != SBLM_OK) return rc;
  rc = check_hip(shadow(n), "mlp_set_params: launch");
  if (rc == SBLM_OK) rc = check_hip(hipMemset(n->m, 0, NP_DEV * 4), "mlp_set_params");
  if (rc == SBLM_OK) rc = check_hip(hipMemset(n->v, 0, NP_DEV * 4), "mlp_set_params");
  if (rc == SBLM_OK) rc = check_hip(hipDeviceSynchronize(), "mlp_set_params");
  n->step = 0;
  return rc;
}

extern "C" int mlp_get_params(mlp_net* n, float* params) {
  if (!n || !params) return set_error(SBLM_EINVAL, "mlp_get_params: null argument");
  int rc = check_hip(hipDeviceSynchronize(), "mlp_get_params");
  if (rc != SBLM_OK) return rc;
  return copy_canonical(n, n->p, params, true, "mlp_get_params");
}

extern "C" int mlp_get_grad(mlp_net* n, float* grad) {
  if (!n || !grad) return set_error(SBLM_EINVAL, "mlp_get_grad: null argument");
  int rc = check_hip(hipDeviceSynchronize(), "mlp_get_grad");
  if (rc != SBLM_OK) return rc;
  return copy_canonical(n, n->g, grad, true, "mlp_get_grad");
}

extern "C" int mlp_set_grad(mlp_net* n, const float* grad) {
  if (!n || !grad) return set_error(SBLM_EINVAL, "mlp_set_grad: null argument");
  int rc = check_hip(hipDeviceSynchronize(), "mlp_set_grad");
  if (rc != SBLM_OK) return rc;
  return copy_canonical(n, n->g, (float*)grad, false, "mlp_set_grad");
}

static hipError_t launch_rows(mlp_net* n, RowArgs& a, bool train, hipStream_t st) {
  a.wf = n->wf;
  a.p = n->p;
  const dim3 grid((unsigned)((a.rows + RB - 1) / RB));
  if (train)
    hipLaunchKernelGGL((net_rows_kernel<true>), grid, dim3(ROW_THREADS), 0, st, a);
  else
    hipLaunchKernelGGL((net_rows_kernel<false>), grid, dim3(ROW_THREADS), 0, st, a);
  return hipGetLastError();
}

extern "C" int mlp_forward(mlp_net* n, const uint16_t* x, int64_t rows, float* out,
                           void* stream) {
  if (!n) return set_error(SBLM_ESTATE, "mlp_forward: null network");
  if (rows < 0) return set_error(SBLM_EINVAL, "mlp_forward: rows < 0");
  if (rows == 0) return SBLM_OK;
  if (!x || !out) return set_error(SBLM_EINVAL, "mlp_forward: null x or out");
  hipStream_t st = (hipStream_t)stream;
  RowArgs a;
  memset(&a, 0, sizeof(a));
  // the kernel reads the caller's rows in 16-byte pieces: as many as a launch
  // takes where their address allows it, else chunks of batch_max from a copy
  const bool aligned = ((uintptr_t)x & 15) == 0;
  const int64_t chunk = aligned ? ROWS_MAX : n->batch_max;
  for (int64_t r0 = 0; r0 < rows; r0 += chunk) {
    a.rows = std::min<int64_t>(chunk, rows - r0);
    a.x = x + r0 * NB;
    a.out = out + r0 * NOP;
    hipError_t e = hipSuccess;
    if (!aligned) {
      e = hipMemcpyAsync(n->xbuf, a.x, (size_t)a.rows * NB * 2, hipMemcpyDeviceToDevice, st);
      a.x = n->xbuf;
    }
    if (e == hipSuccess) e = launch_rows(n, a, false, st);
    if (e != hipSuccess) return check_hip(e, "mlp_forward");
  }
  return SBLM_OK;
}

// K ranges of the weight-gradient products for a batch of `rows`: at least
// 128 rows each (more workgroups, shorter chains).
static int ksplit_for(int rows) {
  int ks = 1;
  while (ks < KSPLIT_MAX && rows % (64 * ks) == 0 && rows / (2 * ks) >= 128) ks *= 2;
  return ks;
}

// Loss and gradient of a batch.  `dstep` (captured training): the batch is the
// step's rows of (x, y), and the weight gradients are left as split-K partials,
// the bias gradients and the loss as column-sum partials (all summed by
// adam_kernel) instead of being reduced here.
static hipError_t loss_grad(mlp_net* n, const uint16_t* x, const float* y, int rows,
                            float* loss, hipStream_t st, int64_t* dstep = nullptr,
                            int64_t per = 1) {
  const bool fold = dstep != nullptr;
  const int64_t ldt = n->batch_max;
  RowArgs a;
  memset(&a, 0, sizeof(a));
  a.x = x;
  a.rows = rows;
  a.y = y;
  a.xT = n->xT; a.h1T = n->h1T; a.h2T = n->h2T;
  a.dobT = n->dobT; a.dz2T = n->dz2T; a.dz1T = n->dz1T;
  a.ldt = ldt;
  a.dof = n->dof; a.dz2f = n->dz2f; a.dz1f = n->dz1f; a.lrow = n->lrow;
  a.dstep = dstep;
  a.per = per;
  hipError_t e = launch_rows(n, a, true, st);
  if (e != hipSuccess) return e;
  // weight gradients: gW = (layer input)^T dZ, a contraction over the batch,
  // cut into K ranges of at least 128 rows (more workgroups, shorter chains);
  // the three products in one launch (independent once dZ1 is known), with
  // the column sums (bias gradients and the loss) beside them
  const int ks = ksplit_for(rows);
  struct { const uint16_t *A, *B; int M, N; float *out, *part; } wg[3] = {
      {n->h2T, n->dobT, NH, NOP, n->g + OFF_W3, n->kpart + KPART_W3},
      {n->h1T, n->dz2T, NH, NH, n->g + OFF_W2, n->kpart + KPART_W2},
      {n->xT, n->dz1T, NB, NH, n->g + OFF_W1, n->kpart + KPART_W1}};
  GemmArgs gw[3];
  for (int i = 0; i < 3; ++i) {
    memset(&gw[i], 0, sizeof(gw[i]));
    gw[i].A = wg[i].A; gw[i].lda = ldt; gw[i].B = wg[i].B; gw[i].ldb = ldt;
    gw[i].M = wg[i].M; gw[i].N = wg[i].N; gw[i].K = rows;
    gw[i].ksplit = ks;
    gw[i].C = ks > 1 ? wg[i].part : wg[i].out;
  }
  ColSegs cs;
  memset(&cs, 0, sizeof(cs));
  cs.s[0] = {n->dof, NOP, NOP, n->g + OFF_B3};
  cs.s[1] = {n->dz2f, NH, NH, n->g + OFF_B2};
  cs.s[2] = {n->dz1f, NH, NH, n->g + OFF_B1};
  cs.s[3] = {n->lrow, 1, 1, loss ? loss : n->cpart};  // unused slot when no loss
  cs.nseg = loss ? 4 : 3;
  cs.nrow = rows;
  for (int i = 0; i < cs.nseg; ++i) {
    cs.tile0[i + 1] = cs.tile0[i] + (cs.s[i].ncol + 63) / 64;
    cs.col0[i + 1] = cs.col0[i] + cs.s[i].ncol;
  }
  if ((e = gemm_group(gw, 3, st, &cs, n->cpart)) != hipSuccess || fold) return e;
  for (int i = 0; i < 3 && ks > 1; ++i) {
    const int64_t mn = (int64_t)gw[i].M * gw[i].N;
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3(grid_for(mn)), dim3(256), 0, st, wg[i].part, ks,
                       mn, wg[i].out);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int ncol_all = cs.col0[cs.nseg];
  hipLaunchKernelGGL(colsum_stage2, dim3((ncol_all + 255) / 256), dim3(256), 0, st, cs, n->cpart,
                     ncol_all);
  return hipGetLastError();
}

extern "C" int mlp_loss_grad(mlp_net* n, const uint16_t* x, const float* y, int32_t rows,
                             float* loss, void* stream) {
  if (!n) return set_error(SBLM_ESTATE, "mlp_loss_grad: null network");
  if (!x || !y) return set_error(SBLM_EINVAL, "mlp_loss_grad: null x or y");
  if (rows < 64 || rows % 64 != 0 || rows > n->batch_max)
    return set_error(SBLM_EINVAL,
                     "mlp_loss_grad: rows = %d must be a multiple of 64 in [64, %d]", rows,
                     n->batch_max);
  return check_hip(loss_grad(n, x, y, rows, loss, (hipStream_t)stream), "mlp_loss_grad");
}

static AdamArgs adam_args(mlp_net* n) {
  const double b1 = 0.9, b2 = 0.999;
  return {n->p, n->m, n->v, (float)b1, (float)b2, (float)(1.0 - b1), (float)(1.0 - b2), 1e-8f};
}

static hipError_t adam(mlp_net* n, float lr, hipStream_t st) {
  const double b1 = 0.9, b2 = 0.999;
  n->step += 1;
  const double c1 = 1.0 / (1.0 - pow(b1, (double)n->step));
  const double c2 = 1.0 / (1.0 - pow(b2, (double)n->step));
  hipLaunchKernelGGL(adam_kernel, dim3(W_BLOCKS), dim3(256), 0, st, adam_args(n), n->g, n->wf,
                     lr, (float)c1, (float)c2, nullptr, nullptr, KParts{}, CParts{},
                     nullptr);
  return hipGetLastError();
}

extern "C" int mlp_adam_step(mlp_net* n, float lr, void* stream) {
  if (!n) return set_error(SBLM_ESTATE, "mlp_adam_step: null network");
  if (!(lr >= 0.0f)) return set_error(SBLM_EINVAL, "mlp_adam_step: lr must be >= 0");
  return check_hip(adam(n, lr, (hipStream_t)stream), "mlp_adam_step");
}

// The captured training steps, each: the batch's rows (forward, likelihood,
// backward), the weight gradients with the column sums, Adam with the split-K
// and column sums, the loss and the step counter.  It holds the net's buffers
// and the caller's (x, y), of which the step's index picks the batch, so one
// graph serves every step of a call and later calls with the same data.
static hipError_t capture_train(mlp_net* n, const uint16_t* x, const float* y, int64_t per,
                                int batch, int steps, hipGraphExec_t* exec) {
  hipStream_t w = n->work;
  hipGraph_t graph = nullptr;
  hipError_t e = hipStreamBeginCapture(w, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return e;
  float* loss_slot = n->cpart + (int64_t)CS_RC * COLS_ALL;
  for (int k = 0; k < steps && e == hipSuccess; ++k) {
    e = loss_grad(n, x, y, batch, loss_slot, w, n->dstep, per);
    if (e != hipSuccess) break;
    KParts kp;
    kp.part[0] = n->kpart + KPART_W3;
    kp.part[1] = n->kpart + KPART_W2;
    kp.part[2] = n->kpart + KPART_W1;
    kp.ks = ksplit_for(batch);
    // the column sums' partials as loss_grad left them (b3, b2, b1, loss)
    CParts cp;
    cp.part = n->cpart;
    cp.ncol_all = COLS_ALL;
    cp.col0[0] = 0;
    cp.col0[1] = NOP;
    cp.col0[2] = NOP + NH;
    cp.loss_col = NOP + 2 * NH;
    hipLaunchKernelGGL(adam_kernel, dim3(W_BLOCKS), dim3(256), 0, w, adam_args(n), n->g, n->wf,
                       0.0f, 0.0f, 0.0f, n->sched, n->dstep, kp, cp, n->losses);
    e = hipGetLastError();
  }
  const hipError_t e_end = hipStreamEndCapture(w, &graph);
  if (e == hipSuccess) e = e_end;
  if (e == hipSuccess) {
    if (*exec) (void)hipGraphExecDestroy(*exec);
    *exec = nullptr;
    e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
  }
  if (graph) (void)hipGraphDestroy(graph);
  return e;
}

// Steps per graph of a long training call.  The GPU idles for some 5 us between
// two graph launches and 1 us between two kernels of one graph: 48 steps of 1024
// rows took 2750 us one by one and take 2540 so.
constexpr int GRAPH_STEPS = 8;

extern "C" int mlp_train(mlp_net* n, const uint16_t* x, const float* y, int64_t rows,
                         int32_t batch, int32_t epochs, float lr0, float lr1,
                         float* loss, void* stream) {
  if (!n) return set_error(SBLM_ESTATE, "mlp_train: null network");
  if (!x || !y) return set_error(SBLM_EINVAL, "mlp_train: null x or y");
  if (batch < 64 || batch % 64 != 0 || batch > n->batch_max)
    return set_error(SBLM_EINVAL, "mlp_train: batch = %d must be a multiple of 64 in [64, %d]",
                     batch, n->batch_max);
  if (epochs < 0 || rows < batch)
    return set_error(SBLM_EINVAL, "mlp_train: epochs = %d, rows = %lld (< batch?)", epochs,
                     (long long)rows);
  if (!(lr0 >= 0.0f) || !(lr1 >= 0.0f))
    return set_error(SBLM_EINVAL, "mlp_train: learning rates must be >= 0");
  const int64_t per = rows / batch;
  const int64_t total = per * epochs;
  if (total > ((int64_t)1 << 31))
    return set_error(SBLM_ERANGE, "mlp_train: %lld steps beyond 2^31", (long long)total);
  if (total == 0) return SBLM_OK;
  hipStream_t st = (hipStream_t)stream;
  // the step schedule on the host, as mlp_adam_step computes it: cosine
  // learning rate, bias corrections of step t = (steps so far) + k + 1
  float* sched_h = (float*)malloc((size_t)total * 3 * sizeof(float));
  if (!sched_h) return set_error(SBLM_ENOMEM, "mlp_train: host allocation");
  const double b1 = 0.9, b2 = 0.999;
  for (int64_t k = 0; k < total; ++k) {
    const double fr = total > 1 ? (double)k / (double)(total - 1) : 0.0;
    const double t = (double)(n->step + k + 1);
    sched_h[3 * k] = (float)(lr1 + 0.5 * (lr0 - lr1) * (1.0 + cos(M_PI * fr)));
    sched_h[3 * k + 1] = (float)(1.0 / (1.0 - pow(b1, t)));
    sched_h[3 * k + 2] = (float)(1.0 / (1.0 - pow(b2, t)));
  }
  // The steps of the call before, which may still be queued on the net's own
  // stream, read the schedule and run the graphs that this call replaces.
  int rc = check_hip(hipStreamSynchronize(n->work), "mlp_train: synchronise");
  // the net's work stream follows the caller's
  if (!rc) rc = check_hip(hipEventRecord(n->ev_in, st), "mlp_train: event");
  if (!rc) rc = check_hip(hipStreamWaitEvent(n->work, n->ev_in, 0), "mlp_train: wait");
  if (!rc && total > n->sched_cap) {
    // larger step buffers: the graph holds the old ones, so it is captured again
    if (n->sched) (void)hipFree(n->sched);
    if (n->losses) (void)hipFree(n->losses);
    n->sched = nullptr;
    n->losses = nullptr;
    n->sched_cap = 0;
    n->train_key[0] = 0;  // (also where the new buffers take the old addresses)
    if (hipMalloc(&n->sched, (size_t)total * 3 * sizeof(float)) != hipSuccess ||
        hipMalloc(&n->losses, (size_t)total * sizeof(float)) != hipSuccess) {
      (void)hipGetLastError();
      rc = set_error(SBLM_ENOMEM, "mlp_train: device allocation");
    } else {
      n->sched_cap = total;
    }
  }
  if (!rc)
    rc = check_hip(hipMemcpy(n->sched, sched_h, (size_t)total * 3 * sizeof(float),
                             hipMemcpyHostToDevice),
                   "mlp_train: schedule");
  free(sched_h);
  const int64_t key[5] = {batch, (int64_t)(uintptr_t)x, (int64_t)(uintptr_t)y, per,
                          (int64_t)(uintptr_t)n->sched};
  if (!rc && (!n->train_exec || memcmp(key, n->train_key, sizeof(key)) != 0)) {
    if (n->train_exec_n) (void)hipGraphExecDestroy(n->train_exec_n);
    n->train_exec_n = nullptr;
    rc = check_hip(capture_train(n, x, y, per, batch, 1, &n->train_exec), "mlp_train: capture");
    if (!rc) memcpy(n->train_key, key, sizeof(key));
  }
  if (!rc && !n->train_exec_n && total >= 4 * GRAPH_STEPS)
    rc = check_hip(capture_train(n, x, y, per, batch, GRAPH_STEPS, &n->train_exec_n),
                   "mlp_train: capture");
  // the step counter restarts at 0 (outside the graph)
  if (!rc) rc = check_hip(hipMemsetAsync(n->dstep, 0, 8, n->work), "mlp_train: counter");
  int64_t k = 0;
  for (; !rc && n->train_exec_n && k + GRAPH_STEPS <= total; k += GRAPH_STEPS)
    rc = check_hip(hipGraphLaunch(n->train_exec_n, n->work), "mlp_train: steps");
  for (; !rc && k < total; ++k)
    rc = check_hip(hipGraphLaunch(n->train_exec, n->work), "mlp_train: step");
  if (!rc && loss)
    rc = check_hip(hipMemcpyAsync(loss, n->losses, (size_t)total * sizeof(float),
                                  hipMemcpyDeviceToDevice, n->work),
                   "mlp_train: losses");
  if (!rc) n->step += total;
  if (!rc) rc = check_hip(hipEventRecord(n->ev_out, n->work), "mlp_train: event");
  if (!rc) rc = check_hip(hipStreamWaitEvent(st, n->ev_out, 0), "mlp_train: wait");
  return rc;
}

// ---------------------------------------------------------- resampling

extern "C" int sblm_resample(const sblm_lcs* lcs, float* xf, uint16_t* xb, void* stream) {
  if (!lcs || !lcs->off || !lcs->t || !lcs->y || !lcs->w)
    return set_error(SBLM_EINVAL, "sblm_resample: null lightcurve descriptor or array");
  if (lcs->n_lc < 1) return set_error(SBLM_EINVAL, "sblm_resample: n_lc < 1");
  if (lcs->n_lc > (1 << 24)) return set_error(SBLM_ERANGE, "sblm_resample: n_lc beyond 2^24");
  if (!xf && !xb) return set_error(SBLM_EINVAL, "sblm_resample: no output");
  hipLaunchKernelGGL(resample_kernel, dim3(lcs->n_lc), dim3(NB), 0, (hipStream_t)stream,
                     lcs->off, lcs->t, lcs->y, lcs->w, xf, xb);
  return check_hip(hipGetLastError(), "sblm_resample launch");
}

extern "C" int mlp_make_data(uint64_t seed, int64_t first, int64_t n, uint16_t* xb,
                             float* xf, float* y, void* stream) {
  if (n < 0 || first < 0) return set_error(SBLM_EINVAL, "mlp_make_data: negative range");
  if (n == 0) return SBLM_OK;
  if (!y || (!xb && !xf)) return set_error(SBLM_EINVAL, "mlp_make_data: null output");
  if (n > (1LL << 26)) return set_error(SBLM_ERANGE, "mlp_make_data: n beyond 2^26");
  hipStream_t st = (hipStream_t)stream;
  const int64_t chunk = std::min<int64_t>(n, 1 << 16);
  double *theta = nullptr, *aux = nullptr, *A = nullptr, *u = nullptr;
  bool ok = hipMalloc(&theta, (size_t)chunk * 6 * 8) == hipSuccess &&
            hipMalloc(&aux, (size_t)chunk * NAUX * 8) == hipSuccess &&
            hipMalloc(&A, (size_t)chunk * NB * 8) == hipSuccess &&
            hipMalloc(&u, NB * 8) == hipSuccess;
  int rc = SBLM_OK;
  if (!ok) {
    (void)hipGetLastError();
    rc = set_error(SBLM_ENOMEM, "mlp_make_data: device allocation");
  }
  if (rc == SBLM_OK) {
    hipLaunchKernelGGL(bin_centres_kernel, dim3(1), dim3(NB), 0, st, u);
    rc = check_hip(hipGetLastError(), "mlp_make_data: launch");
  }
  for (int64_t s0 = 0; rc == SBLM_OK && s0 < n; s0 += chunk) {
    const int nc = (int)std::min<int64_t>(chunk, n - s0);
    hipLaunchKernelGGL(data_draw_kernel, dim3((nc + 255) / 256), dim3(256), 0, st, seed,
                       first + s0, nc, theta, aux, y + s0 * DM);
    rc = check_hip(hipGetLastError(), "mlp_make_data: draw launch");
    if (rc == SBLM_OK) rc = sblm_magnify(theta, nc, u, NB, SBLM_FP64, A, nullptr, nullptr, st);
    if (rc == SBLM_OK) {
      hipLaunchKernelGGL(data_finish_kernel, dim3(nc), dim3(NB), 0, st, seed, first + s0,
                         aux, A, xf ? xf + s0 * NB : nullptr, xb ? xb + s0 * NB : nullptr);
      rc = check_hip(hipGetLastError(), "mlp_make_data: finish launch");
    }
  }
  // the temporaries are released once the queued work has used them
  if (hipStreamSynchronize(st) != hipSuccess && rc == SBLM_OK)
    rc = check_hip(hipGetLastError(), "mlp_make_data: synchronise");
  if (theta) (void)hipFree(theta);
  if (aux) (void)hipFree(aux);
  if (A) (void)hipFree(A);
  if (u) (void)hipFree(u);
  return rc;
}
