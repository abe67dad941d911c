// sblm_ea.hip -- the evolutionary algorithm of Rajpaul (2012), Appendix A,
// on the device, plus the ea_* entry points of the C ABI.
//
// One workgroup per lightcurve runs a whole generation of its population:
// the old population and its fitness are staged in LDS, rows are ranked
// (stable, NaN last), the tournaments and crossover weights of all pairings
// are drawn one Philox block per thread, then one thread per (offspring, two
// genes) crosses and mutates them, writing the next population in place;
// thread 0 keeps the per-lightcurve record (best-ever individual, best-chi^2
// history, jump probability, stagnation flags, restarts).
//
// Random numbers: Philox4x64-10 (Salmon et al. 2011), key (seed, lc),
// counter (generation, purpose, row, j/4), word j%4, so every draw is a pure
// function of its coordinates.  All arithmetic on encoded genes is written
// with explicit fused multiply-adds and compiled without contraction, so the
// result is the same on any IEEE-754 machine given the same fitness.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>

#include "sblm_internal.h"
#include "sblm_rng.h"

namespace sblm {

// 2^-v, v in [0, 64): Taylor polynomial of 2^-f = exp(-f ln 2) on f in
// [0,1) through f^16 (error < 6e-18), coefficients (-ln 2)^n/n! rounded to
// nearest, Horner with fma, then an exact power-of-two scaling.
__device__ __forceinline__ double exp2_neg(double v) {
  const double T[17] = {
      0x1.0000000000000p+0,   -0x1.62e42fefa39efp-1, 0x1.ebfbdff82c58fp-3,
      -0x1.c6b08d704a0c0p-5,  0x1.3b2ab6fba4e77p-7,  -0x1.5d87fe78a6731p-10,
      0x1.430912f86c787p-13,  -0x1.ffcbfc588b0c7p-17, 0x1.62c0223a5c824p-20,
      -0x1.b5253d395e7c4p-24, 0x1.e4cf5158b8ecap-28, -0x1.e8cac7351bb25p-32,
      0x1.c3bd650fc2986p-36,  -0x1.816193166d0f9p-40, 0x1.314964d5878a9p-44,
      -0x1.c36e843b04022p-49, 0x1.38e89ae79f8b4p-53};
  const double k = floor(v);
  const double f = v - k;
  double s = T[16];
#pragma unroll
  for (int n = 15; n >= 0; --n) s = fma(s, f, T[n]);
  return ldexp(s, -(int)k);
}

__device__ __forceinline__ double clamp01(double x) {
  return x < 0.0 ? 0.0 : (x > 1.0 ? 1.0 : x);
}

enum { P_INIT = EA_PURPOSE_INIT, P_TOURN = EA_PURPOSE_TOURN,
       P_MODE = EA_PURPOSE_MODE, P_CREEP = EA_PURPOSE_CREEP,
       P_JUMP = EA_PURPOSE_JUMP, P_SEED = EA_PURPOSE_SEED };

#define EA_HIST 64

// Per-lightcurve record, device resident.
struct EaLc {
  int64_t gen, gen_restart, best_gen;
  double p_mut;
  int32_t stag_count, n_restarts;
  double best_chi2, best_Fs, best_Fb;
  double best_p[SBLM_NPAR];
  double hist[EA_HIST];  // best chi^2 of generation g at hist[g % (window+1)]
};

// One EA population per "virtual lightcurve": with islands (Sec. 5.3),
// island i of lightcurve k is virtual lightcurve k * n_isl + i, and n_lc
// counts virtual lightcurves.
struct EaParams {
  int32_t n_lc, pop, n_tourn, window, restart_after;
  int32_t n_isl;  // islands per lightcurve
  double p_mut0, p_mut_min, p_mut_max, stag_frac;
  uint64_t seed;
  int64_t n_ind;  // n_lc * pop (all islands)
  // [n_lc / n_isl] nonzero: the lightcurve is frozen (ea_freeze) and its
  // generations, migrations and fitness evaluations are skipped
  const int32_t* frozen = nullptr;
};

// Sec. A.1: rows i < pop/2 uniform, row i + pop/2 = 1 - row i, odd last row
// uniform; draws keyed by generation `gen`.  Writes rows of P for
// lightcurve lc with the threads of one block, one Philox block (four genes,
// then two) per thread and pass.
__device__ void init_rows(const EaParams& p, double* P, int64_t lc,
                          int64_t gen) {
  const int half = p.pop / 2, drawn = half + (p.pop & 1);
  const int64_t base = lc * p.pop;
  for (int e = threadIdx.x; e < 2 * drawn; e += blockDim.x) {
    const int q = e >= drawn ? 1 : 0, i = e - q * drawn;
    const bool odd_last = (i == half);
    const int row = odd_last ? p.pop - 1 : i;
    const u64x4 w = philox4x64_10((uint64_t)gen, P_INIT, (uint64_t)row, (uint64_t)q, p.seed,
                                  (uint64_t)lc);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int g = 4 * q + m;
      if (g >= SBLM_NPAR) break;
      const double x = u01(w.v[m]);
      P[g * p.n_ind + base + row] = x;
      if (!odd_last) P[g * p.n_ind + base + i + half] = 1.0 - x;
    }
  }
}

__global__ void ea_init_kernel(EaParams p, double* P, EaLc* lcs) {
  const int64_t lc = blockIdx.x;
  init_rows(p, P, lc, 0);
  if (threadIdx.x == 0) {
    EaLc& s = lcs[lc];
    s.gen = 0;
    s.gen_restart = 0;
    s.best_gen = -1;
    s.p_mut = p.p_mut0;
    s.stag_count = 0;
    s.n_restarts = 0;
    s.best_chi2 = INFINITY;
    s.best_Fs = 0.0;
    s.best_Fb = 0.0;
    for (int g = 0; g < SBLM_NPAR; ++g) s.best_p[g] = 0.0;
    for (int h = 0; h < EA_HIST; ++h) s.hist[h] = INFINITY;
  }
}

__device__ __forceinline__ double rank_key(double c) {
  return isnan(c) ? INFINITY : c;
}

// Proposal seeding: row `row` < n_seed of lightcurve lc becomes a draw from
// the mixture that the proposal network output O[lc][0..119] describes (8
// logits, 8x7 means, 8x7 log standard deviations over the network's target
// map), decoded to physical parameters on the lightcurve's observed span
// and re-encoded (clamped) into the EA's domain.  Draws: key (seed, lc),
// counter (gen, EA_PURPOSE_SEED, row, j / 4); word 0 picks the component by
// inversion of the softmax weights, words 1..8 give four Box-Muller pairs.
struct Proposals {
  const float* O;  // [n_lc][ld] network outputs, or null (no seeding)
  int32_t ld;
  int32_t n_seed;
  int32_t window_only;  // 1: rows from the observation window alone (O unused)
  const int64_t* off;
  const double* t;
  double lo[SBLM_NPAR], span[SBLM_NPAR];
};

// Row `row`'s draw from the network's proposal mixture o (K logits, K x D
// means, K x D log standard deviations): component by the first Philox word,
// then a Gaussian draw by four Box-Muller pairs; x_3 reduced mod 1.
__device__ void seed_mixture(const float* o, const Stream& rs, int row, double* x) {
  const int K = MLP_K, D = MLP_D;
  double lmax = (double)o[0];
  for (int k = 1; k < K; ++k) lmax = fmax(lmax, (double)o[k]);
  double S = 0.0;
  for (int k = 0; k < K; ++k) S += exp((double)o[k] - lmax);
  const double u = u01(rs.draw(P_SEED, (uint64_t)row, 0));
  int comp = K - 1;
  double acc = 0.0;
  for (int k = 0; k < K; ++k) {
    acc += exp((double)o[k] - lmax);
    if (u * S < acc) {
      comp = k;
      break;
    }
  }
  double z[8];
  for (int i = 0; i < 4; ++i) {
    const double u1 = u01(rs.draw(P_SEED, (uint64_t)row, (uint64_t)(1 + 2 * i)));
    const double u2 = u01(rs.draw(P_SEED, (uint64_t)row, (uint64_t)(2 + 2 * i)));
    const double rad = sqrt(-2.0 * log(u1));
    z[2 * i] = rad * cos(2.0 * M_PI * u2);
    z[2 * i + 1] = rad * sin(2.0 * M_PI * u2);
  }
  for (int d = 0; d < D; ++d)
    x[d] = (double)o[K + comp * D + d] + exp((double)o[K + K * D + comp * D + d]) * z[d];
  x[MLP_PERIODIC] -= floor(x[MLP_PERIODIC]);
}

// (Out of line: its exponentials and cosines would cost the generation kernel,
// which calls it at restarts only, its registers.)
__device__ __noinline__ void seed_row(const EaParams& p, double* P, const Proposals& pr,
                                      int64_t lc, int row, int64_t gen) {
  const int64_t k = lc / p.n_isl;  // the lightcurve of this island
  const int64_t o0 = pr.off[k], o1 = pr.off[k + 1];
  if (o1 <= o0) return;
  const double t_first = pr.t[o0], tspan = pr.t[o1 - 1] - t_first;
  const Stream rs = {p.seed, (uint64_t)lc, (uint64_t)gen};
  double x[MLP_D];
  if (pr.window_only) {
    // the ablation of the learned form: t0 at the middle of the observed
    // span, tE a quarter of it, the other genes uniform over their range
    for (int d = 0; d < 4; ++d) x[d] = u01(rs.draw(P_SEED, (uint64_t)row, (uint64_t)(1 + d)));
    x[4] = 0.5;
    x[5] = 0.25;
  } else {
    seed_mixture(pr.O + k * (int64_t)pr.ld, rs, row, x);
  }
  double th[SBLM_NPAR];
  th[0] = -3.0 + 3.0 * x[0];
  th[1] = 0.5 + 1.5 * x[1];
  th[2] = 0.5 * x[2];
  th[3] = 2.0 * M_PI * x[3];
  th[4] = tspan * x[5];
  th[5] = t_first + tspan * x[4];
  const int64_t col = lc * p.pop + row;
  for (int g = 0; g < SBLM_NPAR; ++g) {
    const double e = (th[g] - pr.lo[g]) / pr.span[g];
    P[g * p.n_ind + col] = fmin(fmax(e, 0.0), 1.0);
  }
}

// One thread per (lightcurve, seeded row); keyed by each lightcurve's
// current generation.
__global__ void ea_seed_kernel(EaParams p, double* P, const EaLc* lcs, Proposals pr) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)p.n_lc * pr.n_seed) return;
  const int64_t lc = idx / pr.n_seed;
  seed_row(p, P, pr, lc, (int)(idx % pr.n_seed), lcs[lc].gen);
}

// The largest population.
#define EA_POP_MAX 1024

// Populations up to this size are ranked by counting, larger ones sorted.
#define EA_COUNT_RANK 256

// Entries of the ranking's arrays: N, or the next power of two for the sort.
__host__ __device__ inline int rank_room(int N) {
  if (N <= EA_COUNT_RANK) return N;
  int M = 2 * EA_COUNT_RANK;
  while (M < N) M *= 2;
  return M;
}

// Ranks of the keys (ascending, equal keys in row order) into perm[rank] =
// row; key[0] is then the lowest key if they were sorted.  Counting needs N^2 compares spread over the block and no barrier, the
// bitonic sort log^2 N barriers of N/2 exchanges: at N = 256 about 1 us
// against 4, at N = 1000 about 13 us against 6.  The sort needs room for
// the next power of two.
__device__ void rank_rows(double* key, int* perm, int N) {
  if (N <= EA_COUNT_RANK) {
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
      const double ki = key[i];
      int r = 0;
#pragma unroll 4
      for (int j = 0; j < N; ++j) {
        const double kj = key[j];
        r += (kj < ki || (kj == ki && j < i)) ? 1 : 0;
      }
      perm[r] = i;
    }
    __syncthreads();
    return;
  }
  const int M = rank_room(N);
  for (int i = threadIdx.x; i < M; i += blockDim.x) {
    perm[i] = i;
    if (i >= N) key[i] = INFINITY;  // (after every row: higher index)
  }
  __syncthreads();
  for (int k = 2; k <= M; k <<= 1) {
    for (int s = k >> 1; s > 0; s >>= 1) {
      for (int e = threadIdx.x; e < M / 2; e += blockDim.x) {
        const int i = 2 * e - (e & (s - 1)), j = i + s;  // i has bit s clear
        const double a = key[i], b = key[j];
        const int ia = perm[i], ib = perm[j];
        const bool gt = a > b || (a == b && ia > ib);
        if (gt == ((i & k) == 0)) {
          key[i] = b;
          key[j] = a;
          perm[i] = ib;
          perm[j] = ia;
        }
      }
      // exchanges at a distance of at most 64 stay within the 128 entries of
      // one wave; wider ones cross waves (the next distance after 1 is k)
      if (s > 64 || (s == 1 && k > 64))
        __syncthreads();
      else
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
}

// One generation (Sec. A.3-A.7) for lightcurve blockIdx.x.  Bound by the
// Philox blocks (ten rounds of two 64-bit products, quarter-rate integer
// multiplies) and, for small populations, by the length of the chain
// load - rank - draw - mutate.  Every block of four words is computed once:
// the tournament words of a pairing one block per thread (their minimum by
// an LDS atomic), its crossover weights in LDS for both children, the creep
// and jump words of two genes by the thread that mutates them.  256
// lightcurves x pop 1000: 252 -> 67 us a call; a fit of one lightcurve, pop
// 48: 72 -> 54 us a generation, fitness included (before: one thread per
// pairing and a Philox block for every word).
__global__ __launch_bounds__(1024) void ea_generation_kernel(
    EaParams p, double* P, EaLc* lcs, const double* chi2, const double* Fs, const double* Fb,
    int32_t* parents_out, Proposals pr) {
  extern __shared__ double smem[];
  const int N = p.pop, npair = N / 2, nt = p.n_tourn;
  const int Nr = rank_room(N);
  double* sP = smem;                            // [6][N] old population
  double* key = sP + SBLM_NPAR * N;             // [Nr]
  double* wgt = key + Nr;                       // [6][npair] crossover weights
  int* perm = (int*)(wgt + SBLM_NPAR * npair);  // [Nr] rank -> row
  int* par = perm + Nr;                         // [2][npair] parent ranks
  __shared__ double s_pmut;
  __shared__ int s_restart;

  const int64_t lc = blockIdx.x;
  if (p.frozen && p.frozen[lc / p.n_isl]) return;  // the whole block
  const int64_t base = lc * N;
  EaLc& st = lcs[lc];
  const int64_t gen = st.gen;
  const uint64_t ulc = (uint64_t)lc, ugen = (uint64_t)gen;
  // the record's fields that thread 0 needs after the ranking (loads in
  // flight meanwhile)
  const int W = p.window;
  double r_best = 0.0, r_old = 0.0, r_pmut = 0.0;
  int64_t r_gen0 = 0;
  int r_stag = 0;
  if (threadIdx.x == 0) {
    r_best = st.best_chi2;
    r_pmut = st.p_mut;
    r_gen0 = st.gen_restart;
    r_stag = st.stag_count;
    r_old = st.hist[(gen + 1) % (W + 1)];  // generation gen - W
  }

  for (int i = threadIdx.x; i < N; i += blockDim.x) key[i] = rank_key(chi2[base + i]);
  for (int i = threadIdx.x; i < N; i += blockDim.x)
#pragma unroll
    for (int g = 0; g < SBLM_NPAR; ++g) sP[g * N + i] = P[g * p.n_ind + base + i];
  for (int i = threadIdx.x; i < 2 * npair; i += blockDim.x) par[i] = N;
  __syncthreads();
  // (A.4) tournaments: parent rank = min of nt draws from {0..N-1}; words 0
  // .. nt-1 choose the first parent, nt .. 2 nt - 1 the second
  const int nq = (2 * nt + 3) / 4;
  for (int e = threadIdx.x; e < npair * nq; e += blockDim.x) {
    const int q = e / npair, k = e - q * npair;
    const u64x4 w = philox4x64_10(ugen, P_TOURN, (uint64_t)k, (uint64_t)q, p.seed, ulc);
    int ra = N, rb = N;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int j = 4 * q + m, x = (int)below(w.v[m], (uint32_t)N);
      if (j < nt)
        ra = x < ra ? x : ra;
      else if (j < 2 * nt)
        rb = x < rb ? x : rb;
    }
    if (ra < N) atomicMin(&par[k], ra);
    if (rb < N) atomicMin(&par[npair + k], rb);
  }
  // (A.5) weighting mode of every pairing: U(0,1), Bin(1,1/2) or ones
  for (int k = blockDim.x - 1 - threadIdx.x; k < npair; k += blockDim.x) {
    const u64x4 mb0 = philox4x64_10(ugen, P_MODE, (uint64_t)k, 0, p.seed, ulc);
    const u64x4 mb1 = philox4x64_10(ugen, P_MODE, (uint64_t)k, 1, p.seed, ulc);
    const int mode = (int)below(mb0.v[0], 3u);
#pragma unroll
    for (int g = 0; g < SBLM_NPAR; ++g) {
      const uint64_t x = (g < 3) ? mb0.v[1 + g] : mb1.v[g - 3];
      wgt[g * npair + k] = (mode == 0) ? u01(x) : (mode == 1 ? ((x >> 63) ? 1.0 : 0.0) : 1.0);
    }
  }
  // (A.3) stable rank
  rank_rows(key, perm, N);

  if (threadIdx.x == 0) {
    const int top = perm[0];
    const double b = key[N <= EA_COUNT_RANK ? top : 0];
    s_pmut = r_pmut;  // mutation of this generation uses the current value
    if (b < r_best) {
      st.best_chi2 = b;
      st.best_Fs = Fs[base + top];
      st.best_Fb = Fb[base + top];
      for (int g = 0; g < SBLM_NPAR; ++g) st.best_p[g] = sP[g * N + top];
      st.best_gen = gen;
    }
    st.hist[gen % (W + 1)] = b;
    // (A.7) stagnation test on the best chi^2 of `window` generations ago
    int restart = 0;
    if (gen - r_gen0 >= W) {
      const bool improved =
          isinf(r_old) ? (b < r_old) : ((r_old - b) > p.stag_frac * r_old);
      if (improved) {
        r_pmut = fmax(0.5 * r_pmut, p.p_mut_min);
        r_stag = 0;
      } else {
        r_pmut = fmin(1.5 * r_pmut, p.p_mut_max);
        r_stag += 1;
      }
      if (r_stag >= p.restart_after) {
        restart = 1;
        r_pmut = p.p_mut0;
        r_stag = 0;
        st.gen_restart = gen + 1;
        st.n_restarts += 1;
      }
      st.p_mut = r_pmut;
      st.stag_count = r_stag;
    }
    st.gen = gen + 1;
    s_restart = restart;
  }
  __syncthreads();

  if (s_restart) {  // fresh population keyed by the next generation
    init_rows(p, P, lc, gen + 1);
    if (pr.O || pr.window_only) {  // attached proposals re-seed their rows
      __syncthreads();
      for (int r = threadIdx.x; r < pr.n_seed; r += blockDim.x) seed_row(p, P, pr, lc, r, gen + 1);
    }
    return;
  }
  const double pm = s_pmut;
  if (threadIdx.x < SBLM_NPAR) {  // (A.5) elitism: row 0 keeps the fittest
    const int g = threadIdx.x;
    P[g * p.n_ind + base] = sP[g * N + perm[0]];
  }
  if (parents_out)
    for (int k = threadIdx.x; k < npair; k += blockDim.x) {
      parents_out[lc * 2 * npair + 2 * k] = par[k];
      parents_out[lc * 2 * npair + 2 * k + 1] = par[npair + k];
    }
  // offspring 2k+1, 2k+2 of pairing k, genes 2h and 2h+1 per thread
  const int n_off = 2 * npair < N - 1 ? 2 * npair : N - 1;
  for (int e = threadIdx.x; e < 3 * n_off; e += blockDim.x) {
    const int h = e / n_off, slot = 1 + e - h * n_off;
    const int k = (slot - 1) >> 1;
    const bool second = ((slot - 1) & 1) != 0;
    const int ia = perm[par[k]], ib = perm[par[npair + k]];
    const u64x4 cb = philox4x64_10(ugen, P_CREEP, (uint64_t)slot, (uint64_t)h, p.seed, ulc);
    const u64x4 jb = philox4x64_10(ugen, P_JUMP, (uint64_t)slot, (uint64_t)h, p.seed, ulc);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int g = 2 * h + m;
      const double f = wgt[g * npair + k], omf = 1.0 - f;
      const double pa = sP[g * N + (second ? ib : ia)], pb = sP[g * N + (second ? ia : ib)];
      double v = clamp01(fma(f, pa, omf * pb));
      // (A.6) creep: p -> p + (1-p) X or p - p X, ln X ~ U(ln 2^-52, 0)
      const double X = exp2_neg(52.0 * u01(cb.v[2 * m + 1]));
      v = (cb.v[2 * m] >> 63) ? fma(1.0 - v, X, v) : fma(-v, X, v);
      v = clamp01(v);
      // (A.6) jump: with probability p_mut replace by a fresh uniform
      if (u01(jb.v[2 * m]) < pm) v = u01(jb.v[2 * m + 1]);
      P[g * p.n_ind + base + slot] = v;
    }
  }
}

__global__ void ea_draws_kernel(uint64_t seed, uint64_t lc, uint64_t gen,
                                uint64_t purpose, uint64_t row, uint64_t j0,
                                int64_t n, uint64_t* out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const Stream rs = {seed, lc, gen};
  out[k] = rs.draw(purpose, row, j0 + (uint64_t)k);
}

// Record of lightcurve k: that of its island with the lowest best chi^2,
// the lowest island index among equals (records are never NaN).
__device__ __forceinline__ int64_t best_island(const EaLc* lcs, int64_t k, int n_isl) {
  int64_t v = k * n_isl;
  for (int i = 1; i < n_isl; ++i)
    if (lcs[k * n_isl + i].best_chi2 < lcs[v].best_chi2) v = k * n_isl + i;
  return v;
}

// The record's fittest solution as a [6][n_lc] encoded array (n_lc
// lightcurves, not islands).
__global__ void ea_best_kernel(const EaLc* lcs, int32_t n_lc, int32_t n_isl, double* x,
                               double* chi2) {
  const int lc = blockIdx.x * blockDim.x + threadIdx.x;
  if (lc >= n_lc) return;
  const EaLc& r = lcs[best_island(lcs, lc, n_isl)];
  for (int g = 0; g < SBLM_NPAR; ++g) x[(int64_t)g * n_lc + lc] = r.best_p[g];
  if (chi2) chi2[lc] = r.best_chi2;
}

// Replaces every record (one per island) whose refined solution is fitter.
__global__ void ea_improve_kernel(EaLc* lcs, int32_t n_rec, const double* x, const double* chi2,
                                  const double* Fs, const double* Fb) {
  const int lc = blockIdx.x * blockDim.x + threadIdx.x;
  if (lc >= n_rec) return;
  EaLc& r = lcs[lc];
  if (chi2[lc] < r.best_chi2) {
    r.best_chi2 = chi2[lc];
    r.best_Fs = Fs[lc];
    r.best_Fb = Fb[lc];
    for (int g = 0; g < SBLM_NPAR; ++g) r.best_p[g] = x[(int64_t)g * n_rec + lc];
    r.best_gen = r.gen;
  }
}

// Island migration (Sec. 5.3; timing, ring and replacement rule as stated
// with ea_config).  Two launches so that every island sends from the state
// before any receives: the first ranks each island (stable counting rank on
// the rank key) and copies its m fittest rows, with their fitness, to slots
// 0..m-1 of its own outbox and notes the rows of ranks pop-1 .. pop-m; the
// second copies the outbox of the island before it on the ring over those
// rows.  Every island of a state has the same generation count, so both
// launches agree on whether the migration is due.
struct MigArgs {
  double* chi2;     // [n_ind] fitness of the current rows, updated in place
  double* Fs;
  double* Fb;
  double* out;      // [n_lc][m][9] outbox: 6 genes, chi^2, Fs, Fb
  int32_t* least;   // [n_lc][m] row of rank pop - 1 - r
  int32_t m, every, force;
};

__device__ __forceinline__ bool migration_due(const MigArgs& a, int64_t gen) {
  return a.force || (gen > 0 && gen % a.every == 0);
}

__global__ void ea_emigrate_kernel(EaParams p, const double* P, const EaLc* lcs, MigArgs a) {
  extern __shared__ double skey[];  // [pop]
  const int64_t v = blockIdx.x;
  if (!migration_due(a, lcs[v].gen) || (p.frozen && p.frozen[v / p.n_isl])) return;
  const int N = p.pop;
  const int64_t base = v * N;
  for (int i = threadIdx.x; i < N; i += blockDim.x) skey[i] = rank_key(a.chi2[base + i]);
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += blockDim.x) {
    const double ki = skey[i];
    int r = 0;
    for (int j = 0; j < N; ++j) {
      const double kj = skey[j];
      r += (kj < ki || (kj == ki && j < i)) ? 1 : 0;
    }
    if (r < a.m) {
      double* o = a.out + (v * a.m + r) * 9;
      for (int g = 0; g < SBLM_NPAR; ++g) o[g] = P[g * p.n_ind + base + i];
      o[6] = a.chi2[base + i];
      o[7] = a.Fs[base + i];
      o[8] = a.Fb[base + i];
    }
    if (r >= N - a.m) a.least[v * a.m + (N - 1 - r)] = i;
  }
}

__global__ void ea_immigrate_kernel(EaParams p, double* P, const EaLc* lcs, MigArgs a) {
  const int64_t v = blockIdx.x;
  if (!migration_due(a, lcs[v].gen) || (p.frozen && p.frozen[v / p.n_isl])) return;
  const int64_t k = v / p.n_isl;
  const int i = (int)(v - k * p.n_isl);
  const int64_t src = k * p.n_isl + (i + p.n_isl - 1) % p.n_isl;
  const int64_t base = v * p.pop;
  for (int r = threadIdx.x; r < a.m; r += blockDim.x) {
    const int row = a.least[v * a.m + r];
    const double* o = a.out + (src * a.m + r) * 9;
    for (int g = 0; g < SBLM_NPAR; ++g) P[g * p.n_ind + base + row] = o[g];
    a.chi2[base + row] = o[6];
    a.Fs[base + row] = o[7];
    a.Fb[base + row] = o[8];
  }
}

// ---------------------------------------------------------------- host side

struct EaStateImpl {
  ea_config cfg;
  EaParams prm;
  sblm_lcs lcs;
  int device;
  double* P = nullptr;
  double* chi2 = nullptr;
  double* Fs = nullptr;
  double* Fb = nullptr;
  EaLc* lc = nullptr;
  hipStream_t work = nullptr;
  hipEvent_t ev_in = nullptr, ev_out = nullptr;
  hipGraphExec_t graph = nullptr;    // one generation
  hipGraphExec_t graph_n = nullptr;  // GRAPH_GENS of them (see ea_fit)
  sblm_stats* graph_stats = nullptr;
  // fitness schedule: lanes per individual (default_lanes at creation),
  // waves per block, persistent launch with work counters (these two chosen by
  // ea_autotune), stepping (kept and reported; both run the one kernel there is)
  int lanes = 16;
  int wpb = 4;
  int persistent = 1;
  int async = 0;
  int32_t* order = nullptr;    // item -> individual, longest lightcurves first
  unsigned int* queue = nullptr;  // 8 work counters, one per XCD
  int64_t* xcd_start = nullptr;   // [9] order positions owned by each XCD
  Proposals prop = {};         // attached by ea_seed(..., EA_SEED_AT_RESTARTS)
  int n_phys = 0;              // lightcurves (prm.n_lc counts islands)
  int32_t* frozen = nullptr;   // [n_phys] ea_freeze's mask
  // the workload as the schedule cache keys it (ea_autotune_cached)
  char sig[320] = {0};
  double* mig_out = nullptr;   // migration outboxes (islands with migrants)
  int32_t* mig_least = nullptr;
  bool mig_in_fit = false;     // ea_fit migrates when due
  // fitness timing (ea_time_fitness): device wall-clock ticks summed over the
  // timed launches [0], the start stamp of the current one [1], launches [2]
  unsigned long long* ticks = nullptr;
  int time_fitness = 0;
};

// Device wall-clock stamps around the fitness kernel (one thread): the
// start stamp, then at the end the interval is added to the sum.  Kernels on
// one stream run in order, so the interval spans the fitness kernel and the
// dispatch gaps on either side of it (a few microseconds).
__global__ void fitness_stamp_kernel(unsigned long long* t, int end) {
  if (threadIdx.x != 0) return;
  const unsigned long long now = (unsigned long long)wall_clock64();
  if (end) {
    t[0] += now - t[1];
    t[2] += 1;
  } else {
    t[1] = now;
  }
}

__global__ void ticks_clear_kernel(unsigned long long* t) {
  if (threadIdx.x < 4) t[threadIdx.x] = 0ull;
}

__global__ void queue_reset_kernel(unsigned int* q) {
  if (threadIdx.x < 8) q[threadIdx.x] = 0u;
}

static size_t gen_smem(int pop) {
  const size_t half = pop / 2, room = rank_room(pop);
  return SBLM_NPAR * (pop + half) * sizeof(double) + room * (sizeof(double) + sizeof(int)) +
         2 * half * sizeof(int);
}

// Threads of a generation's block: one per (offspring, two genes) task up to
// 256, where several blocks share a compute unit; 512 and 1024 for the
// populations whose LDS (44 KB at 512, 88 KB at 1024) leaves room for three
// blocks or one.
static int gen_block(int pop) {
  int b = 64;
  while (b < 3 * pop && b < 256) b *= 2;
  while (b < pop && b < 1024) b *= 2;
  return b;
}

static hipError_t enqueue_generation(EaStateImpl* s, const double* chi2,
                                     const double* Fs, const double* Fb,
                                     int32_t* parents, hipStream_t st) {
  hipLaunchKernelGGL(ea_generation_kernel, dim3(s->prm.n_lc),
                     dim3(gen_block(s->prm.pop)), gen_smem(s->prm.pop), st, s->prm,
                     s->P, s->lc, chi2, Fs, Fb, parents, s->prop);
  return hipGetLastError();
}

static hipError_t enqueue_migration(EaStateImpl* s, double* chi2, double* Fs, double* Fb,
                                    int force, hipStream_t st) {
  MigArgs a;
  a.chi2 = chi2;
  a.Fs = Fs;
  a.Fb = Fb;
  a.out = s->mig_out;
  a.least = s->mig_least;
  a.m = s->cfg.n_migrants;
  a.every = s->cfg.mig_every > 0 ? s->cfg.mig_every : 1;
  a.force = force;
  hipLaunchKernelGGL(ea_emigrate_kernel, dim3(s->prm.n_lc), dim3(gen_block(s->prm.pop)),
                     (size_t)s->prm.pop * sizeof(double), st, s->prm, s->P, s->lc, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ea_immigrate_kernel, dim3(s->prm.n_lc), dim3(64), 0, st, s->prm, s->P,
                     s->lc, a);
  return hipGetLastError();
}

static hipError_t enqueue_evaluate(EaStateImpl* s, sblm_stats* stats,
                                   hipStream_t st, bool stamped = false) {
  FitArgs a;
  memset(&a, 0, sizeof(a));
  a.theta = s->P;
  a.n_ind = s->prm.n_ind;
  a.encoded = 1;
  for (int j = 0; j < SBLM_NPAR; ++j) {
    a.lo[j] = s->cfg.lo[j];
    a.span[j] = s->cfg.hi[j] - s->cfg.lo[j];
  }
  a.off = s->lcs.off;
  a.pop = s->prm.pop * s->prm.n_isl;  // all islands of a lightcurve together
  a.t = s->lcs.t;
  a.y = s->lcs.y;
  a.w = s->lcs.w;
  a.chi2 = s->chi2;
  a.Fs = s->Fs;
  a.Fb = s->Fb;
  a.stats = stats;
  a.lanes_per_ind = s->lanes;
  a.order = s->order;
  a.skip = s->frozen;  // a frozen lightcurve's rows are evaluated as empty
  a.skip_per = a.pop;
  if (s->persistent) {
    a.queue = s->queue;
    a.xcd_start = s->xcd_start;
    hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(64), 0, st, s->queue);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (!stamped) return launch_fitness(a, s->cfg.mode, true, st, s->wpb);
  hipLaunchKernelGGL(fitness_stamp_kernel, dim3(1), dim3(64), 0, st, s->ticks, 0);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_fitness(a, s->cfg.mode, true, st, s->wpb);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fitness_stamp_kernel, dim3(1), dim3(64), 0, st, s->ticks, 1);
  return hipGetLastError();
}

}  // namespace sblm

using namespace sblm;

struct ea_state {
  EaStateImpl impl;
};

static int capture_graph(EaStateImpl& s, sblm_stats* stats);

extern "C" void ea_default_config(ea_config* c) {
  if (!c) return;
  memset(c, 0, sizeof(*c));
  c->pop = 256;
  c->n_tourn = 0;
  c->p_mut0 = 0.01;
  c->p_mut_min = 1e-4;
  c->p_mut_max = 0.5;
  c->stag_frac = 0.01;
  c->stag_window = 10;
  c->restart_after = 10;
  const double lo[SBLM_NPAR] = {-3.0, 0.5, 0.0, 0.0, 10.0, -10.0};
  const double hi[SBLM_NPAR] = {0.0, 2.0, 0.5, 6.283185307179586, 100.0, 10.0};
  for (int j = 0; j < SBLM_NPAR; ++j) {
    c->lo[j] = lo[j];
    c->hi[j] = hi[j];
  }
  c->mode = SBLM_FP64;
  c->n_islands = 1;  // no islands, no migration
}

static int validate(const ea_config* c) {
  if (c->pop < 2 || c->pop > EA_POP_MAX)
    return set_error(SBLM_ERANGE, "ea_config: pop = %d outside [2, %d]", c->pop, EA_POP_MAX);
  if (c->n_tourn < 0 || c->n_tourn > c->pop)
    return set_error(SBLM_EINVAL, "ea_config: n_tourn = %d", c->n_tourn);
  if (!(c->p_mut0 >= 0.0 && c->p_mut0 <= 1.0) || !(c->p_mut_min >= 0.0) ||
      !(c->p_mut_max <= 1.0) || !(c->p_mut_min <= c->p_mut_max))
    return set_error(SBLM_EINVAL, "ea_config: jump probabilities out of [0,1]");
  if (!(c->stag_frac >= 0.0))
    return set_error(SBLM_EINVAL, "ea_config: stag_frac < 0");
  if (c->stag_window < 1 || c->stag_window > EA_HIST - 1)
    return set_error(SBLM_ERANGE, "ea_config: stag_window = %d outside [1, %d]",
                     c->stag_window, EA_HIST - 1);
  if (c->restart_after < 1)
    return set_error(SBLM_EINVAL, "ea_config: restart_after < 1");
  for (int j = 0; j < SBLM_NPAR; ++j)
    if (!(c->lo[j] < c->hi[j]) || !isfinite(c->lo[j]) || !isfinite(c->hi[j]))
      return set_error(SBLM_EINVAL, "ea_config: empty or non-finite domain %d", j);
  if (!(c->lo[4] > 0.0))
    return set_error(SBLM_EINVAL, "ea_config: tE domain must be positive");
  if (c->mode != SBLM_FP64 && c->mode != SBLM_MIXED)
    return set_error(SBLM_EINVAL, "ea_config: unknown mode %d", c->mode);
  if (c->n_islands < 1 || c->n_islands > 256)
    return set_error(SBLM_ERANGE, "ea_config: n_islands = %d outside [1, 256]", c->n_islands);
  if (c->mig_every < 0) return set_error(SBLM_EINVAL, "ea_config: mig_every < 0");
  if (c->n_migrants < 0 || 2 * c->n_migrants > c->pop)
    return set_error(SBLM_EINVAL, "ea_config: n_migrants = %d outside [0, pop/2]",
                     c->n_migrants);
  return SBLM_OK;
}

extern "C" void ea_destroy(ea_state* st) {
  if (!st) return;
  EaStateImpl& s = st->impl;
  int prev = 0;
  (void)hipGetDevice(&prev);
  (void)hipSetDevice(s.device);
  if (s.work) (void)hipStreamSynchronize(s.work);
  if (s.graph) (void)hipGraphExecDestroy(s.graph);
  if (s.graph_n) (void)hipGraphExecDestroy(s.graph_n);
  if (s.ev_in) (void)hipEventDestroy(s.ev_in);
  if (s.ev_out) (void)hipEventDestroy(s.ev_out);
  if (s.work) (void)hipStreamDestroy(s.work);
  (void)hipFree(s.P);
  (void)hipFree(s.chi2);
  (void)hipFree(s.Fs);
  (void)hipFree(s.Fb);
  (void)hipFree(s.lc);
  (void)hipFree(s.order);
  (void)hipFree(s.queue);
  (void)hipFree(s.xcd_start);
  (void)hipFree(s.ticks);
  (void)hipFree(s.mig_out);
  (void)hipFree(s.mig_least);
  (void)hipFree(s.frozen);
  (void)hipSetDevice(prev);
  st->~ea_state();
  free(st);
}

extern "C" int ea_create(const ea_config* cfg, const sblm_lcs* lcs, uint64_t seed,
                         ea_state** out) {
  if (!cfg || !lcs || !out) return set_error(SBLM_EINVAL, "ea_create: null argument");
  *out = nullptr;
  int rc = validate(cfg);
  if (rc) return rc;
  if (!lcs->off || !lcs->t || !lcs->y || !lcs->w)
    return set_error(SBLM_EINVAL, "ea_create: null lightcurve array");
  if (lcs->n_lc < 1 || lcs->n_lc > (1 << 20))
    return set_error(SBLM_ERANGE, "ea_create: n_lc = %d", lcs->n_lc);
  if ((int64_t)lcs->n_lc * cfg->n_islands * cfg->pop > (1LL << 31) - 1)
    return set_error(SBLM_ERANGE, "ea_create: n_lc * n_islands * pop too large");
  void* mem = malloc(sizeof(ea_state));
  if (!mem) return set_error(SBLM_ENOMEM, "ea_create: host allocation");
  ea_state* st = new (mem) ea_state();
  EaStateImpl& s = st->impl;
  s.cfg = *cfg;
  s.lcs = *lcs;
  (void)hipGetDevice(&s.device);
  EaParams& p = s.prm;
  s.n_phys = lcs->n_lc;
  p.n_isl = cfg->n_islands;
  p.n_lc = lcs->n_lc * cfg->n_islands;
  p.pop = cfg->pop;
  p.n_tourn = cfg->n_tourn > 0 ? cfg->n_tourn : (cfg->pop + 24) / 25;
  p.window = cfg->stag_window;
  p.restart_after = cfg->restart_after;
  p.p_mut0 = cfg->p_mut0;
  p.p_mut_min = cfg->p_mut_min;
  p.p_mut_max = cfg->p_mut_max;
  p.stag_frac = cfg->stag_frac;
  p.seed = seed;
  p.n_ind = (int64_t)p.n_lc * p.pop;
  // Lanes per individual: each lane owns one contiguous chunk of a
  // lightcurve's epochs and warm-starts along it, so this number fixes where
  // the chains of warm starts begin and the merge of the lanes' sums -- it is
  // part of what the fit computes, and ea_autotune leaves it alone (the
  // knobs it tunes do not change a bit).  Rule: the fewest of 8 ... 64 lanes
  // that give the launch 2^20 lanes of work (eight residencies of the chip;
  // fewer lanes mean longer chunks, so fewer cold starts); a small state,
  // whose 64-lane groups would not fill one residency, takes the widest
  // group (up to 256 lanes, over several waves) that fits one, spread over
  // the four waves of a block on the one-shot grid.
  s.lanes = default_lanes(p.n_ind);
  if (s.lanes > 64) s.persistent = 0;
  // (the limit belongs to the kernel, which all states share: always the same,
  // that of the largest population)
  rc = check_hip(hipFuncSetAttribute((const void*)ea_generation_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)gen_smem(EA_POP_MAX)),
                 "ea_create: LDS");
  if (rc) {
    ea_destroy(st);
    return rc;
  }
  const size_t nb = (size_t)p.n_ind * sizeof(double);
  // longest-processing-time order of the work items: lightcurves by length,
  // longest first (stable), the individuals of each lightcurve (all its
  // islands) together
  const int nl = s.n_phys;
  const int popf = p.pop * p.n_isl;
  int64_t xcd_start_h[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  int64_t* off_h = (int64_t*)malloc((size_t)(nl + 1) * sizeof(int64_t));
  int32_t* order_h = (int32_t*)malloc((size_t)p.n_ind * sizeof(int32_t));
  int32_t* lcs_sorted = (int32_t*)malloc((size_t)nl * sizeof(int32_t));
  if (!off_h || !order_h || !lcs_sorted) {
    free(off_h);
    free(order_h);
    free(lcs_sorted);
    ea_destroy(st);
    return set_error(SBLM_ENOMEM, "ea_create: host allocation");
  }
  rc = check_hip(hipMemcpy(off_h, lcs->off, (size_t)(nl + 1) * sizeof(int64_t),
                           hipMemcpyDeviceToHost),
                 "ea_create offsets");
  if (!rc)
    for (int k = 0; k < nl; ++k)
      if (off_h[k + 1] < off_h[k] || off_h[0] != 0) {
        rc = set_error(SBLM_EINVAL, "ea_create: offsets not non-decreasing from 0");
        break;
      }
  if (!rc) {
    // workload signature: precision form, population, islands, lightcurves,
    // and how many lightcurves have floor(log2(L + 1)) = b
    int hist[64] = {0};
    for (int k = 0; k < nl; ++k) {
      uint64_t v = (uint64_t)(off_h[k + 1] - off_h[k]) + 1;
      int b = 0;
      while (v >>= 1) ++b;
      ++hist[b];
    }
    int n = snprintf(s.sig, sizeof(s.sig), "mode=%d pop=%d islands=%d n_lc=%d L2:",
                     cfg->mode, p.pop, p.n_isl, nl);
    for (int b = 0; b < 64 && n > 0 && n < (int)sizeof(s.sig) - 16; ++b)
      if (hist[b]) n += snprintf(s.sig + n, sizeof(s.sig) - n, " %d:%d", b, hist[b]);
  }
  if (!rc) {
    for (int k = 0; k < nl; ++k) lcs_sorted[k] = k;
    // stable bottom-up merge sort, longest first
    int32_t* tmp = (int32_t*)malloc((size_t)nl * sizeof(int32_t));
    for (int w = 1; tmp && w < nl; w *= 2)
      for (int lo = 0; lo < nl; lo += 2 * w) {
        int mid = lo + w < nl ? lo + w : nl;
        int hi = lo + 2 * w < nl ? lo + 2 * w : nl;
        int i = lo, j = mid, o = lo;
        while (i < mid && j < hi) {
          const int64_t li = off_h[lcs_sorted[i] + 1] - off_h[lcs_sorted[i]];
          const int64_t lj = off_h[lcs_sorted[j] + 1] - off_h[lcs_sorted[j]];
          tmp[o++] = (lj > li) ? lcs_sorted[j++] : lcs_sorted[i++];
        }
        while (i < mid) tmp[o++] = lcs_sorted[i++];
        while (j < hi) tmp[o++] = lcs_sorted[j++];
        for (int k = lo; k < hi; ++k) lcs_sorted[k] = tmp[k];
      }
    free(tmp);
    // lightcurves dealt to the 8 XCDs longest first, each to the XCD with the
    // least work so far (epochs x individuals, lowest index among equals);
    // the order lists XCD 0's lightcurves first (longest first), then XCD 1's
    int64_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int32_t* xcd_of = (int32_t*)malloc((size_t)nl * sizeof(int32_t));
    if (!xcd_of) rc = set_error(SBLM_ENOMEM, "ea_create: host allocation");
    for (int r = 0; !rc && r < nl; ++r) {
      const int k = lcs_sorted[r];
      const int64_t L = off_h[k + 1] - off_h[k];
      int x = 0;
      for (int y = 1; y < 8; ++y)
        if (load[y] < load[x]) x = y;
      xcd_of[k] = x;
      load[x] += (L > 0 ? L : 1) * popf;
    }
    int64_t pos = 0;
    for (int x = 0; !rc && x < 8; ++x) {
      xcd_start_h[x] = pos;
      for (int r = 0; r < nl; ++r) {
        const int k = lcs_sorted[r];
        if (xcd_of[k] != x) continue;
        for (int i = 0; i < popf; ++i) order_h[pos++] = k * popf + i;
      }
    }
    xcd_start_h[8] = pos;
    free(xcd_of);
  }
  free(off_h);
  free(lcs_sorted);
  if (rc) {
    free(order_h);
    ea_destroy(st);
    return rc;
  }
  if (hipMalloc(&s.P, SBLM_NPAR * nb) != hipSuccess || hipMalloc(&s.chi2, nb) != hipSuccess ||
      hipMalloc(&s.Fs, nb) != hipSuccess || hipMalloc(&s.Fb, nb) != hipSuccess ||
      hipMalloc(&s.lc, (size_t)p.n_lc * sizeof(EaLc)) != hipSuccess ||
      hipMalloc(&s.order, (size_t)p.n_ind * sizeof(int32_t)) != hipSuccess ||
      hipMalloc(&s.queue, 8 * sizeof(unsigned int)) != hipSuccess ||
      hipMalloc(&s.xcd_start, 9 * sizeof(int64_t)) != hipSuccess ||
      hipMalloc(&s.ticks, 4 * sizeof(unsigned long long)) != hipSuccess ||
      hipMalloc(&s.frozen, (size_t)s.n_phys * sizeof(int32_t)) != hipSuccess ||
      (p.n_isl > 1 && cfg->n_migrants > 0 &&
       (hipMalloc(&s.mig_out, (size_t)p.n_lc * cfg->n_migrants * 9 * sizeof(double)) !=
            hipSuccess ||
        hipMalloc(&s.mig_least, (size_t)p.n_lc * cfg->n_migrants * sizeof(int32_t)) !=
            hipSuccess))) {
    free(order_h);
    ea_destroy(st);
    return set_error(SBLM_ENOMEM, "ea_create: device allocation of %zu bytes failed",
                     (9 * nb + (size_t)p.n_lc * sizeof(EaLc)));
  }
  if ((rc = check_hip(hipStreamCreateWithFlags(&s.work, hipStreamNonBlocking),
                      "ea_create stream")) ||
      (rc = check_hip(hipEventCreateWithFlags(&s.ev_in, hipEventDisableTiming), "event")) ||
      (rc = check_hip(hipEventCreateWithFlags(&s.ev_out, hipEventDisableTiming), "event"))) {
    ea_destroy(st);
    return rc;
  }
  rc = check_hip(hipMemcpy(s.xcd_start, xcd_start_h, 9 * sizeof(int64_t),
                           hipMemcpyHostToDevice),
                 "ea_create order");
  if (!rc)
    rc = check_hip(hipMemcpy(s.order, order_h, (size_t)p.n_ind * sizeof(int32_t),
                             hipMemcpyHostToDevice),
                   "ea_create order");
  free(order_h);
  if (!rc)
    rc = check_hip(hipMemset(s.frozen, 0, (size_t)s.n_phys * sizeof(int32_t)), "ea_create mask");
  if (rc) {
    ea_destroy(st);
    return rc;
  }
  p.frozen = s.frozen;
  s.mig_in_fit = s.mig_out != nullptr && cfg->mig_every > 0;
  hipLaunchKernelGGL(ea_init_kernel, dim3(p.n_lc), dim3(gen_block(p.pop)), 0, s.work, p, s.P,
                     s.lc);
  rc = check_hip(hipGetLastError(), "ea_create init launch");
  if (!rc) rc = check_hip(hipStreamSynchronize(s.work), "ea_create init");
  if (!rc) rc = capture_graph(s, nullptr);
  if (rc) {
    ea_destroy(st);
    return rc;
  }
  *out = st;
  return SBLM_OK;
}

extern "C" int ea_generation(ea_state* st, const double* chi2, const double* Fs,
                             const double* Fb, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_generation: null state");
  if (!chi2 || !Fs || !Fb) return set_error(SBLM_EINVAL, "ea_generation: null fitness");
  return check_hip(enqueue_generation(&st->impl, chi2, Fs, Fb, nullptr, (hipStream_t)stream),
                   "ea_generation launch");
}

// Test hook: as ea_generation, also writing the selected parent ranks
// (int32 [n_lc][2*floor(pop/2)], device) of every pairing.
extern "C" int ea_generation_traced(ea_state* st, const double* chi2, const double* Fs,
                                    const double* Fb, int32_t* parents, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_generation_traced: null state");
  if (!chi2 || !Fs || !Fb || !parents)
    return set_error(SBLM_EINVAL, "ea_generation_traced: null argument");
  return check_hip(enqueue_generation(&st->impl, chi2, Fs, Fb, parents, (hipStream_t)stream),
                   "ea_generation launch");
}

extern "C" int ea_draws(uint64_t seed, uint64_t lc, uint64_t gen, uint64_t purpose,
                        uint64_t row, uint64_t j0, int64_t n, uint64_t* out, void* stream) {
  if (n < 0 || n > (1LL << 24)) return set_error(SBLM_ERANGE, "ea_draws: n = %lld", (long long)n);
  if (n == 0) return SBLM_OK;
  if (!out) return set_error(SBLM_EINVAL, "ea_draws: null output");
  hipLaunchKernelGGL(ea_draws_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, seed, lc, gen, purpose, row, j0, n, out);
  return check_hip(hipGetLastError(), "ea_draws launch");
}

static int capture_graph(EaStateImpl& s, sblm_stats* stats);

extern "C" int ea_seed(ea_state* st, const float* out, int32_t ld_out, int32_t n_seed,
                       int32_t flags, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_seed: null state");
  EaStateImpl& s = st->impl;
  if (flags & ~(EA_SEED_AT_RESTARTS | EA_SEED_WINDOW_ONLY))
    return set_error(SBLM_EINVAL, "ea_seed: unknown flags");
  const bool window = (flags & EA_SEED_WINDOW_ONLY) != 0;
  if (n_seed < 0 || n_seed > s.prm.pop)
    return set_error(SBLM_EINVAL, "ea_seed: n_seed = %d outside [0, pop = %d]", n_seed,
                     s.prm.pop);
  if (n_seed > 0 && !out && !window)
    return set_error(SBLM_EINVAL, "ea_seed: null network output");
  if (n_seed > 0 && !window && ld_out < MLP_NOUT)
    return set_error(SBLM_EINVAL, "ea_seed: ld_out = %d < %d", ld_out, MLP_NOUT);
  Proposals pr = {};
  pr.O = n_seed > 0 && !window ? out : nullptr;
  pr.ld = ld_out;
  pr.n_seed = n_seed;
  pr.window_only = n_seed > 0 && window ? 1 : 0;
  pr.off = s.lcs.off;
  pr.t = s.lcs.t;
  for (int g = 0; g < SBLM_NPAR; ++g) {
    pr.lo[g] = s.cfg.lo[g];
    pr.span[g] = s.cfg.hi[g] - s.cfg.lo[g];
  }
  if (n_seed > 0) {
    const int64_t n = (int64_t)s.prm.n_lc * n_seed;
    hipLaunchKernelGGL(ea_seed_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, s.prm, s.P, s.lc, pr);
    int rc = check_hip(hipGetLastError(), "ea_seed launch");
    if (rc) return rc;
  }
  const bool attach = (flags & EA_SEED_AT_RESTARTS) && n_seed > 0;
  const bool was = s.prop.O != nullptr || s.prop.window_only;
  s.prop = attach ? pr : Proposals{};
  if ((attach || was) && s.graph) return capture_graph(s, s.graph_stats);
  return SBLM_OK;
}

extern "C" int ea_freeze(ea_state* st, const int32_t* mask, int32_t n_lc, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_freeze: null state");
  if (!mask) return set_error(SBLM_EINVAL, "ea_freeze: null mask");
  EaStateImpl& s = st->impl;
  if (n_lc != s.n_phys)
    return set_error(SBLM_EINVAL, "ea_freeze: mask of %d entries for %d lightcurves", n_lc,
                     s.n_phys);
  const hipStream_t q = (hipStream_t)stream;
  int rc = check_hip(hipMemcpyAsync(s.frozen, mask, (size_t)s.n_phys * sizeof(int32_t),
                                    hipMemcpyHostToDevice, q),
                     "ea_freeze copy");
  if (!rc) rc = check_hip(hipStreamSynchronize(q), "ea_freeze synchronise");
  return rc;
}

extern "C" int ea_best(ea_state* st, double* x, double* chi2, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_best: null state");
  if (!x) return set_error(SBLM_EINVAL, "ea_best: null x");
  EaStateImpl& s = st->impl;
  hipLaunchKernelGGL(ea_best_kernel, dim3((s.n_phys + 255) / 256), dim3(256), 0,
                     (hipStream_t)stream, s.lc, s.n_phys, s.prm.n_isl, x, chi2);
  return check_hip(hipGetLastError(), "ea_best launch");
}

extern "C" int ea_records(ea_state* st, double* x, double* chi2, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_records: null state");
  if (!x) return set_error(SBLM_EINVAL, "ea_records: null x");
  EaStateImpl& s = st->impl;
  // one record per island: the best-of-islands rule over groups of one
  hipLaunchKernelGGL(ea_best_kernel, dim3((s.prm.n_lc + 255) / 256), dim3(256), 0,
                     (hipStream_t)stream, s.lc, s.prm.n_lc, 1, x, chi2);
  return check_hip(hipGetLastError(), "ea_records launch");
}

extern "C" int ea_refine(ea_state* st, const nm_config* cfg, int32_t* n_iter,
                         sblm_stats* stats, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_refine: null state");
  int rc = nm_check(cfg, "ea_refine");
  if (rc) return rc;
  EaStateImpl& s = st->impl;
  const int n = s.prm.n_lc;  // one simplex per island record
  hipStream_t hs = (hipStream_t)stream;
  double *x0 = nullptr, *x = nullptr, *c = nullptr, *fs = nullptr, *fb = nullptr;
  const size_t nn = (size_t)n;
  if (hipMalloc(&x0, nn * SBLM_NPAR * 8) != hipSuccess ||
      hipMalloc(&x, nn * SBLM_NPAR * 8) != hipSuccess || hipMalloc(&c, nn * 8) != hipSuccess ||
      hipMalloc(&fs, nn * 8) != hipSuccess || hipMalloc(&fb, nn * 8) != hipSuccess) {
    (void)hipGetLastError();
    rc = set_error(SBLM_ENOMEM, "ea_refine: device allocation");
  }
  if (rc == SBLM_OK) {
    hipLaunchKernelGGL(ea_best_kernel, dim3((n + 255) / 256), dim3(256), 0, hs, s.lc, n, 1,
                       x0, nullptr);
    rc = check_hip(hipGetLastError(), "ea_refine: launch");
  }
  double span[SBLM_NPAR];
  for (int g = 0; g < SBLM_NPAR; ++g) span[g] = s.cfg.hi[g] - s.cfg.lo[g];
  if (rc == SBLM_OK)
    rc = nm_run(s.lcs, s.prm.n_isl, s.cfg.lo, span, x0, *cfg, x, c, fs, fb, n_iter, stats, hs);
  if (rc == SBLM_OK) {
    hipLaunchKernelGGL(ea_improve_kernel, dim3((n + 255) / 256), dim3(256), 0, hs, s.lc, n, x,
                       c, fs, fb);
    rc = check_hip(hipGetLastError(), "ea_refine: launch");
  }
  if (hipStreamSynchronize(hs) != hipSuccess && rc == SBLM_OK)
    rc = check_hip(hipGetLastError(), "ea_refine: synchronise");
  double* bufs[] = {x0, x, c, fs, fb};
  for (double* b : bufs)
    if (b) (void)hipFree(b);
  return rc;
}

extern "C" int ea_evaluate(ea_state* st, sblm_stats* stats, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_evaluate: null state");
  return check_hip(enqueue_evaluate(&st->impl, stats, (hipStream_t)stream),
                   "ea_evaluate launch");
}

extern "C" int ea_migrate(ea_state* st, double* chi2, double* Fs, double* Fb, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_migrate: null state");
  EaStateImpl& s = st->impl;
  if (!s.mig_out) return set_error(SBLM_ESTATE, "ea_migrate: one island or no migrants");
  const int n_null = (chi2 == nullptr) + (Fs == nullptr) + (Fb == nullptr);
  if (n_null == 1 || n_null == 2)
    return set_error(SBLM_EINVAL, "ea_migrate: give all fitness arrays or none");
  if (n_null == 3) {
    chi2 = s.chi2;
    Fs = s.Fs;
    Fb = s.Fb;
  }
  return check_hip(enqueue_migration(&s, chi2, Fs, Fb, 1, (hipStream_t)stream),
                   "ea_migrate launch");
}

// Captures n generations (evaluate, migration when the state has it, and
// generation kernels on the state's work stream) into an executable graph
// bound to `stats`.
static int capture_generations(EaStateImpl& s, sblm_stats* stats, int n, hipGraphExec_t* exec) {
  int rc;
  hipGraph_t g;
  if ((rc = check_hip(hipStreamBeginCapture(s.work, hipStreamCaptureModeThreadLocal),
                      "ea graph capture")))
    return rc;
  hipError_t e1 = hipSuccess;
  for (int k = 0; k < n && e1 == hipSuccess; ++k) {
    e1 = enqueue_evaluate(&s, stats, s.work, s.time_fitness != 0);
    if (e1 == hipSuccess && s.mig_in_fit)
      e1 = enqueue_migration(&s, s.chi2, s.Fs, s.Fb, 0, s.work);
    if (e1 == hipSuccess) e1 = enqueue_generation(&s, s.chi2, s.Fs, s.Fb, nullptr, s.work);
  }
  hipError_t e3 = hipStreamEndCapture(s.work, &g);
  if ((rc = check_hip(e1 != hipSuccess ? e1 : e3, "ea graph capture"))) return rc;
  hipError_t e4 = hipGraphInstantiate(exec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  return check_hip(e4, "ea graph instantiate");
}

// The graph of one generation, anew; that of several goes with the old one.
static int capture_graph(EaStateImpl& s, sblm_stats* stats) {
  if (s.graph) {
    int rc0 = check_hip(hipStreamSynchronize(s.work), "ea graph re-capture");
    if (rc0) return rc0;
    if (s.graph_n) (void)hipGraphExecDestroy(s.graph_n);
    s.graph_n = nullptr;
    (void)hipGraphExecDestroy(s.graph);
    s.graph = nullptr;
  }
  const int rc = capture_generations(s, stats, 1, &s.graph);
  if (rc) return rc;
  s.graph_stats = stats;
  return SBLM_OK;
}

// Generations per graph of a long fit.  The GPU idles for some 5 us between two
// graph launches and 1 us between two kernels of one graph: 100 generations of
// a population of 48 on one curve of 400 epochs took 4.69 ms one by one and take
// 4.37 so (wall time of a call; the first call, which captures, 4.78 and 4.54).
// A fit of four of these graphs repays the capture.
constexpr int GRAPH_GENS = 8;

extern "C" int ea_fit(ea_state* st, int32_t n_gen, sblm_stats* stats, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_fit: null state");
  if (n_gen < 0) return set_error(SBLM_EINVAL, "ea_fit: n_gen < 0");
  EaStateImpl& s = st->impl;
  int rc;
  if (!s.graph || s.graph_stats != stats)
    if ((rc = capture_graph(s, stats))) return rc;
  hipStream_t caller = (hipStream_t)stream;
  if (!s.graph_n && (n_gen == 0 || n_gen >= 4 * GRAPH_GENS)) {
    // (not inside a capture of the caller's: its one-generation launches are
    // recorded there as ever)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(caller, &cap) != hipSuccess) {
      (void)hipGetLastError();
      cap = hipStreamCaptureStatusActive;
    }
    if (cap == hipStreamCaptureStatusNone &&
        (rc = capture_generations(s, stats, GRAPH_GENS, &s.graph_n)))
      return rc;
  }
  if (n_gen == 0) return SBLM_OK;
  if ((rc = check_hip(hipEventRecord(s.ev_in, caller), "ea_fit event")) ||
      (rc = check_hip(hipStreamWaitEvent(s.work, s.ev_in, 0), "ea_fit wait")))
    return rc;
  int g = 0;
  for (; s.graph_n && g + GRAPH_GENS <= n_gen; g += GRAPH_GENS)
    if ((rc = check_hip(hipGraphLaunch(s.graph_n, s.work), "ea_fit graph launch"))) return rc;
  for (; g < n_gen; ++g)
    if ((rc = check_hip(hipGraphLaunch(s.graph, s.work), "ea_fit graph launch"))) return rc;
  if ((rc = check_hip(hipEventRecord(s.ev_out, s.work), "ea_fit event")) ||
      (rc = check_hip(hipStreamWaitEvent(caller, s.ev_out, 0), "ea_fit wait")))
    return rc;
  return SBLM_OK;
}

extern "C" int ea_time_fitness(ea_state* st, int32_t enable, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_time_fitness: null state");
  if (enable != 0 && enable != 1)
    return set_error(SBLM_EINVAL, "ea_time_fitness: enable = %d", enable);
  EaStateImpl& s = st->impl;
  int rc;
  if ((rc = check_hip(hipEventRecord(s.ev_in, (hipStream_t)stream), "ea_time_fitness event")) ||
      (rc = check_hip(hipStreamWaitEvent(s.work, s.ev_in, 0), "ea_time_fitness wait")))
    return rc;
  hipLaunchKernelGGL(ticks_clear_kernel, dim3(1), dim3(64), 0, s.work, s.ticks);
  if ((rc = check_hip(hipGetLastError(), "ea_time_fitness clear"))) return rc;
  if ((rc = check_hip(hipEventRecord(s.ev_out, s.work), "ea_time_fitness event")) ||
      (rc = check_hip(hipStreamWaitEvent((hipStream_t)stream, s.ev_out, 0),
                      "ea_time_fitness wait")))
    return rc;
  if (s.time_fitness == enable && s.graph) return SBLM_OK;
  s.time_fitness = enable;
  return capture_graph(s, s.graph_stats);
}

extern "C" int ea_fitness_time(ea_state* st, double* ms, int64_t* launches) {
  if (!st || !ms || !launches) return set_error(SBLM_EINVAL, "ea_fitness_time: null argument");
  EaStateImpl& s = st->impl;
  int rc;
  unsigned long long t[4];
  int khz = 0;
  if ((rc = check_hip(hipStreamSynchronize(s.work), "ea_fitness_time sync")) ||
      (rc = check_hip(hipMemcpy(t, s.ticks, sizeof(t), hipMemcpyDeviceToHost),
                      "ea_fitness_time copy")) ||
      (rc = check_hip(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, s.device),
                      "ea_fitness_time clock rate")))
    return rc;
  if (khz <= 0) return set_error(SBLM_EDEVICE, "ea_fitness_time: wall clock rate %d kHz", khz);
  *ms = (double)t[0] / (double)khz;
  *launches = (int64_t)t[2];
  return SBLM_OK;
}

extern "C" int ea_get_schedule(ea_state* st, int32_t* sched) {
  if (!st || !sched) return set_error(SBLM_EINVAL, "ea_get_schedule: null argument");
  sched[0] = st->impl.lanes;
  sched[1] = st->impl.wpb;
  sched[2] = st->impl.persistent;
  sched[3] = st->impl.async;
  return SBLM_OK;
}

extern "C" int ea_set_schedule(ea_state* st, const int32_t* sched) {
  if (!st || !sched) return set_error(SBLM_EINVAL, "ea_set_schedule: null argument");
  const bool wide = sched[0] == 128 || sched[0] == 256;
  if ((sched[0] != 8 && sched[0] != 16 && sched[0] != 32 && sched[0] != 64 && !wide) ||
      (sched[1] != 1 && sched[1] != 2 && sched[1] != 4) || (sched[2] != 0 && sched[2] != 1) ||
      (sched[3] != 0 && sched[3] != 1) ||
      (wide && (sched[1] % (sched[0] / 64) != 0 || sched[2] != 0 || sched[3] != 0)))
    return set_error(SBLM_EINVAL, "ea_set_schedule: bad schedule (%d, %d, %d, %d)", sched[0],
                     sched[1], sched[2], sched[3]);
  EaStateImpl& s = st->impl;
  s.lanes = sched[0];
  s.wpb = sched[1];
  s.persistent = sched[2];
  s.async = sched[3];
  return capture_graph(s, s.graph_stats);
}

// Times one evaluation of the state's population with the current schedule
// (one untimed launch, then the mean of `reps`), on the work stream.
static int time_evaluate(EaStateImpl& s, hipEvent_t e0, hipEvent_t e1, int reps, float* ms) {
  int rc;
  if ((rc = check_hip(enqueue_evaluate(&s, nullptr, s.work), "ea_autotune launch"))) return rc;
  if ((rc = check_hip(hipEventRecord(e0, s.work), "ea_autotune event"))) return rc;
  for (int r = 0; r < reps; ++r)
    if ((rc = check_hip(enqueue_evaluate(&s, nullptr, s.work), "ea_autotune launch"))) return rc;
  if ((rc = check_hip(hipEventRecord(e1, s.work), "ea_autotune event")) ||
      (rc = check_hip(hipEventSynchronize(e1), "ea_autotune sync")) ||
      (rc = check_hip(hipEventElapsedTime(ms, e0, e1), "ea_autotune time")))
    return rc;
  *ms /= (float)reps;
  return SBLM_OK;
}

extern "C" int ea_autotune(ea_state* st, char* report, size_t report_len, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_autotune: null state");
  EaStateImpl& s = st->impl;
  int rc;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if ((rc = check_hip(hipEventRecord(s.ev_in, (hipStream_t)stream), "ea_autotune event")) ||
      (rc = check_hip(hipStreamWaitEvent(s.work, s.ev_in, 0), "ea_autotune wait")) ||
      (rc = check_hip(hipEventCreate(&e0), "ea_autotune event")) ||
      (rc = check_hip(hipEventCreate(&e1), "ea_autotune event"))) {
    if (e0) (void)hipEventDestroy(e0);
    return rc;
  }
  char buf[2048];
  int len = 0;
  buf[0] = 0;
  // coordinate descent over the knobs that leave every result bit as it is:
  // waves per block, persistent vs one-shot grid.  The lanes per individual stay
  // (see ea_create), and so does the epoch stepping, asynchronous or lockstep: one
  // kernel serves both, whose time stands in the report for either.
  int best[4] = {s.lanes, s.wpb, s.persistent, s.async};
  float best_ms = INFINITY;
  rc = time_evaluate(s, e0, e1, 2, &best_ms);
  if (!rc)
    len += snprintf(buf + len, sizeof(buf) - len,
                    "start: lanes=%d wpb=%d persistent=%d async=%d: %.3f ms\n", best[0], best[1],
                    best[2], best[3], best_ms);
  // (128 or 256 lanes spread an individual over several waves: those go
  // with whole individuals per block, the one-shot grid and lockstep
  // stepping, and candidates that break this are skipped)
  const int wpb_c[3] = {1, 2, 4}, bin_c[2] = {1, 0};
  const int stage_field[3] = {3, 1, 2};
  for (int stage = 0; stage < 3 && !rc; ++stage) {
    const int field = stage_field[stage];
    const int nc = field == 1 ? 3 : 2;
    for (int k = 0; k < nc && !rc; ++k) {
      int cand[4] = {best[0], best[1], best[2], best[3]};
      cand[field] = field == 1 ? wpb_c[k] : bin_c[k];
      if (cand[0] > 64 && (cand[1] % (cand[0] / 64) != 0 || cand[2] != 0 || cand[3] != 0))
        continue;
      s.lanes = cand[0];
      s.wpb = cand[1];
      s.persistent = cand[2];
      s.async = cand[3];
      float ms = best_ms;
      if (field != 3) rc = time_evaluate(s, e0, e1, 2, &ms);
      if (rc) break;
      if (len < (int)sizeof(buf) - 100)
        len += snprintf(buf + len, sizeof(buf) - len,
                        "lanes=%d wpb=%d persistent=%d async=%d: %.3f ms\n", cand[0], cand[1],
                        cand[2], cand[3], ms);
      // a candidate replaces the current schedule only when it is faster by
      // more than 2% (timings of one schedule vary by ~1% from one try to the
      // next), so that the choice is stable from one run to the next; the
      // current schedule keeps its best time
      const bool same = cand[0] == best[0] && cand[1] == best[1] && cand[2] == best[2] &&
                        cand[3] == best[3];
      if (same) {
        best_ms = ms < best_ms ? ms : best_ms;
      } else if (ms < 0.98f * best_ms) {
        best_ms = ms;
        for (int f = 0; f < 4; ++f) best[f] = cand[f];
      }
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  s.lanes = best[0];
  s.wpb = best[1];
  s.persistent = best[2];
  s.async = best[3];
  if (!rc) rc = capture_graph(s, s.graph_stats);
  if (!rc && len < (int)sizeof(buf) - 100)
    snprintf(buf + len, sizeof(buf) - len,
             "chosen: lanes=%d wpb=%d persistent=%d async=%d (%.3f ms)\n", best[0], best[1],
             best[2], best[3], best_ms);
  if (report && report_len) {
    strncpy(report, buf, report_len - 1);
    report[report_len - 1] = 0;
  }
  if (!rc) rc = check_hip(hipEventRecord(s.ev_out, s.work), "ea_autotune event");
  if (!rc) rc = check_hip(hipStreamWaitEvent((hipStream_t)stream, s.ev_out, 0), "ea_autotune wait");
  return rc;
}

// 64-bit FNV-1a hash of a string.
static uint64_t fnv1a64(const char* x, uint64_t h = 0xcbf29ce484222325ull) {
  for (; *x; ++x) h = (h ^ (uint64_t)(unsigned char)*x) * 0x100000001b3ull;
  return h;
}

extern "C" int ea_autotune_cached(ea_state* st, const char* path, int32_t* tuned, char* report,
                                  size_t report_len, void* stream) {
  if (!st) return set_error(SBLM_ESTATE, "ea_autotune_cached: null state");
  if (!path || !path[0]) return set_error(SBLM_EINVAL, "ea_autotune_cached: null path");
  EaStateImpl& s = st->impl;
  hipDeviceProp_t prop;
  int rc = check_hip(hipGetDeviceProperties(&prop, s.device), "ea_autotune_cached device");
  if (rc) return rc;
  char dev[160];
  snprintf(dev, sizeof(dev), "%s cu=%d lanes=%d ", prop.gcnArchName, prop.multiProcessorCount,
           s.lanes);
  const uint64_t key = fnv1a64(s.sig, fnv1a64(dev));
  // look the key up: lines "<16 hex digits> lanes wpb persistent async ..."
  FILE* f = fopen(path, "r");
  if (f) {
    char line[640];
    while (fgets(line, sizeof(line), f)) {
      unsigned long long k = 0;
      int32_t sc[4];
      if (sscanf(line, "%16llx %d %d %d %d", &k, &sc[0], &sc[1], &sc[2], &sc[3]) != 5 ||
          (uint64_t)k != key)
        continue;
      fclose(f);
      if (sc[0] != s.lanes)  // another rule's lanes: a different fit, not a schedule
        return set_error(SBLM_EINVAL, "ea_autotune_cached: %s: entry %016llx has lanes %d, "
                         "the state %d", path, k, sc[0], s.lanes);
      if ((rc = ea_set_schedule(st, sc))) return rc;
      if (tuned) *tuned = 0;
      if (report && report_len)
        snprintf(report, report_len, "kept: lanes=%d wpb=%d persistent=%d async=%d\n", sc[0],
                 sc[1], sc[2], sc[3]);
      return SBLM_OK;
    }
    fclose(f);
  }
  if ((rc = ea_autotune(st, report, report_len, stream))) return rc;
  if (tuned) *tuned = 1;
  f = fopen(path, "a");
  if (!f) return set_error(SBLM_EINVAL, "ea_autotune_cached: cannot append to %s", path);
  const int ok = fprintf(f, "%016llx %d %d %d %d %s%s\n", (unsigned long long)key, s.lanes,
                         s.wpb, s.persistent, s.async, dev, s.sig) > 0;
  if (fclose(f) != 0 || !ok)
    return set_error(SBLM_EINVAL, "ea_autotune_cached: cannot append to %s", path);
  return SBLM_OK;
}

extern "C" int ea_buffers(ea_state* st, double** P, double** chi2, double** Fs,
                          double** Fb) {
  if (!st) return set_error(SBLM_ESTATE, "ea_buffers: null state");
  if (P) *P = st->impl.P;
  if (chi2) *chi2 = st->impl.chi2;
  if (Fs) *Fs = st->impl.Fs;
  if (Fb) *Fb = st->impl.Fb;
  return SBLM_OK;
}

extern "C" int ea_summary(ea_state* st, ea_lc_summary* out, void* stream) {
  if (!st || !out) return set_error(SBLM_EINVAL, "ea_summary: null argument");
  EaStateImpl& s = st->impl;
  const int n = s.prm.n_lc;
  EaLc* h = (EaLc*)malloc((size_t)n * sizeof(EaLc));
  if (!h) return set_error(SBLM_ENOMEM, "ea_summary: host allocation");
  int rc = check_hip(hipMemcpyAsync(h, s.lc, (size_t)n * sizeof(EaLc), hipMemcpyDeviceToHost,
                                    (hipStream_t)stream),
                     "ea_summary copy");
  if (!rc) rc = check_hip(hipStreamSynchronize((hipStream_t)stream), "ea_summary sync");
  if (!rc)
    for (int k = 0; k < s.n_phys; ++k) {
      const int ni = s.prm.n_isl;
      int v = k * ni;  // the island holding the best record, lowest index first
      for (int i = 1; i < ni; ++i)
        if (h[k * ni + i].best_chi2 < h[v].best_chi2) v = k * ni + i;
      ea_lc_summary& o = out[k];
      o.best_chi2 = h[v].best_chi2;
      o.best_Fs = h[v].best_Fs;
      o.best_Fb = h[v].best_Fb;
      for (int j = 0; j < SBLM_NPAR; ++j)
        o.best_theta[j] = s.cfg.lo[j] + (s.cfg.hi[j] - s.cfg.lo[j]) * h[v].best_p[j];
      o.best_gen = h[v].best_gen;
      o.p_mut = h[v].p_mut;
      o.stag_count = h[v].stag_count;
      o.n_restarts = h[v].n_restarts;
      o.gen = h[v].gen;
      o.gen_restart = h[v].gen_restart;
    }
  free(h);
  return rc;
}

// Snapshot: header, population [6][n_lc*pop] doubles, per-lightcurve records.
struct SnapHeader {
  uint64_t magic;  // "SBLMEA01"
  uint64_t seed;
  int32_t n_lc, pop;
  ea_config cfg;
  uint64_t rec_size;
};
static const uint64_t SNAP_MAGIC = 0x3130414D4C424253ULL;

extern "C" int ea_save(ea_state* st, void* buf, size_t* len, void* stream) {
  if (!st || !len) return set_error(SBLM_EINVAL, "ea_save: null argument");
  EaStateImpl& s = st->impl;
  const size_t np = (size_t)SBLM_NPAR * s.prm.n_ind * sizeof(double);
  const size_t nl = (size_t)s.prm.n_lc * sizeof(EaLc);
  const size_t need = sizeof(SnapHeader) + np + nl;
  if (!buf) {
    *len = need;
    return SBLM_OK;
  }
  if (*len < need) return set_error(SBLM_EINVAL, "ea_save: buffer of %zu < %zu bytes", *len, need);
  SnapHeader hd;
  memset(&hd, 0, sizeof(hd));
  hd.magic = SNAP_MAGIC;
  hd.seed = s.prm.seed;
  hd.n_lc = s.prm.n_lc;
  hd.pop = s.prm.pop;
  hd.cfg = s.cfg;
  hd.rec_size = sizeof(EaLc);
  char* b = (char*)buf;
  memcpy(b, &hd, sizeof(hd));
  hipStream_t str = (hipStream_t)stream;
  int rc = check_hip(hipMemcpyAsync(b + sizeof(hd), s.P, np, hipMemcpyDeviceToHost, str),
                     "ea_save copy");
  if (!rc)
    rc = check_hip(hipMemcpyAsync(b + sizeof(hd) + np, s.lc, nl, hipMemcpyDeviceToHost, str),
                   "ea_save copy");
  if (!rc) rc = check_hip(hipStreamSynchronize(str), "ea_save sync");
  *len = need;
  return rc;
}

extern "C" int ea_load(ea_state* st, const void* buf, size_t len, void* stream) {
  if (!st || !buf) return set_error(SBLM_EINVAL, "ea_load: null argument");
  EaStateImpl& s = st->impl;
  const size_t np = (size_t)SBLM_NPAR * s.prm.n_ind * sizeof(double);
  const size_t nl = (size_t)s.prm.n_lc * sizeof(EaLc);
  SnapHeader hd;
  if (len < sizeof(hd) + np + nl) return set_error(SBLM_ESTATE, "ea_load: snapshot too short");
  memcpy(&hd, buf, sizeof(hd));
  if (hd.magic != SNAP_MAGIC || hd.seed != s.prm.seed || hd.n_lc != s.prm.n_lc ||
      hd.pop != s.prm.pop || hd.rec_size != sizeof(EaLc) ||
      memcmp(&hd.cfg, &s.cfg, sizeof(ea_config)) != 0)
    return set_error(SBLM_ESTATE, "ea_load: snapshot does not match this state");
  const char* b = (const char*)buf;
  hipStream_t str = (hipStream_t)stream;
  int rc = check_hip(hipMemcpyAsync(s.P, b + sizeof(hd), np, hipMemcpyHostToDevice, str),
                     "ea_load copy");
  if (!rc)
    rc = check_hip(hipMemcpyAsync(s.lc, b + sizeof(hd) + np, nl, hipMemcpyHostToDevice, str),
                   "ea_load copy");
  if (!rc) rc = check_hip(hipStreamSynchronize(str), "ea_load sync");
  return rc;
}
