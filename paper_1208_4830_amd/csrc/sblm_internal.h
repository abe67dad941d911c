// sblm_internal.h -- declarations shared by the library's translation units
// (kernels and host entry points).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/sblm.h"

namespace sblm {

// Thread-local last-error message; returns `code` for convenient chaining.
int set_error(int code, const char* fmt, ...);
int check_hip(hipError_t e, const char* what);

// Doubles a lane saves of its first epoch (see FitArgs::root_cache).
constexpr int ROOT_CACHE = 10;

// Arguments of the batched fitness kernels (one wave per individual).
struct FitArgs {
  // population: theta[j * n_ind + i] decoded, or encoded P with lo/hi
  const double* theta;
  int64_t n_ind;
  int32_t encoded;
  double lo[SBLM_NPAR], span[SBLM_NPAR];
  // epochs: either shared (off == nullptr, n_t epochs of t) or CSR per
  // lightcurve (individual i uses lightcurve i / pop)
  const int64_t* off;
  int32_t pop;
  const double* t;
  const double* y;
  const double* w;
  int64_t n_t;
  // outputs
  double* A;        // [n_ind][n_t] (magnify)
  int8_t* n_img;    // nullable (magnify)
  double* chi2;     // [n_ind] (chi2)
  double* Fs;
  double* Fb;
  sblm_stats* stats;  // nullable
  // schedule
  const int32_t* order;  // nullable: item -> individual permutation
  double* root_cache;     // nullable, G >= 64 only: [n_ind][G][ROOT_CACHE],
                          // the roots (tracked: three images) of each lane's
                          // first epoch, read as its start (when finite) and
                          // rewritten after it
  const int32_t* cold;    // nullable (with root_cache): individual i ignores
                          // the cache when cold[i / cold_per] != 0
  int64_t cold_per;
  int32_t lanes_per_ind;  // 64, 32, 16 or 8 (a power of two dividing 64), or
                          // 128 / 256: several waves per individual (one-shot
                          // lockstep, wpb a multiple of G/64); magnifications
                          // also 1, 2, 4 or any multiple of 64
  unsigned int* queue;    // nullable: persistent launch; one shared work
                          // counter, or with xcd_start one per XCD (8)
  const int64_t* xcd_start;  // nullable: [9] order positions; the items at
                             // [xcd_start[x], xcd_start[x+1]) belong to XCD x
                          // (must read 0 when the kernel starts)
  const int32_t* skip;    // nullable (CSR only): individual i is evaluated
  int32_t skip_per;       // as empty when skip[i / skip_per] != 0
  int32_t by_chain;       // 1: whether images are tracked follows from the chain
                          // alone (simplex_tracked), not from how many run
};

// Lanes of one residency of the chip: 256 compute units x 8 waves.
constexpr int64_t RESIDENT_LANES = 2048 * 64;

// Whether images are tracked along the chains of C epochs of an individual with
// L epochs, G lanes each of n_ind: where the epochs are dense enough that a step
// of a wave seldom needs a solve all the same, and the chain long enough to
// repay its dearer first epoch.  For epochs over a few tE, solved and tracked
// us FP64 in a launch of 8 residencies of the chip (65536 individuals, 16
// lanes): 638 and 720 for 80 epochs, 828 and 848 for 100, 1006 and 939 for 130,
// 1761 and 1265 for 300, 2962 and 1754 for 600.  Where little runs, the slowest
// wave decides, and it has most of the failures (4096 individuals, 32 lanes):
// 102 and 137 for 130, 126 and 148 for 200, 157 and 156 for 300, 196 and 186 for
// 400, 258 and 207 for 600; and in chains of three (256 individuals, 256 lanes,
// 600 epochs) 48 and 52.
inline __host__ __device__ bool tracked_chains(int64_t n_ind, int64_t G, int64_t L, int64_t C) {
  return n_ind * G >= 4 * RESIDENT_LANES ? L > 112 && C > 2 : L > 320 && C > 3;
}

// The same for the trial points of simplices, whose values depend on the points
// and the lanes, not on how many simplices a call has: by the chain alone.
// Times of 60 steps, solved and tracked ms, on 64 lanes: 64 simplices of 130
// epochs (chains of 3) 5.3 and 5.9, of 200 5.8 and 5.8, of 300 6.3 and 6.0; 4096
// of 130 26.5 and 24.8, of 200 32.6 and 28.1, of 300 38.1 and 30.4.
inline __host__ __device__ bool simplex_tracked(int64_t C) { return C > 3; }

// Launch the FP64 or mixed fitness kernel; chi2 = false writes A/n_img.
// Lanes per individual for a launch of n_ind individuals: the fewest of 8,
// 16, 32, 64 that give the launch 2^20 lanes of work (fewer lanes, longer
// chains of warm-started epochs per lane, fewer cold starts); a launch whose
// 64-lane groups would not fill one residency of the chip (2^17 lanes: 256
// compute units x 8 waves) takes the widest group, up to 256 lanes over
// several waves, that fits one.
inline int default_lanes(int64_t n_ind) {
  constexpr int64_t RESIDENT = RESIDENT_LANES;
  if (n_ind * 64 <= RESIDENT) {
    int g = 64;
    while (g < 256 && n_ind * (2 * g) <= RESIDENT) g *= 2;
    return g;
  }
  for (int g = 8; g < 64; g *= 2)
    if (n_ind * g >= 8 * RESIDENT) return g;
  return 64;
}

// In FitArgs::lanes_per_ind: magnifications with no chains of epochs, every pair
// (individual, epoch) by itself.
constexpr int MAGNIFY_PAIRS = 0;

// Lanes per individual for the magnifications of n individuals at n_t shared
// epochs, where no sum over the epochs ties the lanes together: the number of
// lowest modelled time, the fewest among equals.  A lane's chain of C epochs
// costs 2.5 for the cold start and w for every other one, w = 0.6 where images
// are tracked, else 1 for dense epochs, more (a poorer extrapolation) for few.
// The n G lanes are r = n G / 2^17 residencies of the chip; below one residency
// only the chain's length counts (a little slower when waves share a SIMD), above it the work grows
// with r and more, shorter waves even out what the slowest lane of each
// holds up (the factor, fitted to 1 <= r <= 32 at 4096 x 1000).  In us at G
// lanes against the rule's choice: 2^20 single epochs 1660 (8), 187 (1); one
// curve of 1000 epochs 18 (256), 11 (1024); 256 x 1000 46 (512), 41 (256);
// 16384 x 256 470 (8), 345 (32); 4096 x 1000 238 (32), 229 (64); 10^5 x 4 135
// (8), 85 (4); 16 x 5000 72 (256), 31 (8192); 65536 x 256 1191 (64), 980 (16).
//   Few epochs (taken as spread out, as above) and enough pairs: no chains at
// all (magnify_pairs_kernel).  In us by the rule below and so: 2^18 single
// epochs 60 and 68, 2^19 109 and 95, 2^20 204 and 147; 2^20 x 2 335 and 215,
// 2^19 x 4 339 and 232, 2^18 x 12 498 and 343, 2^20 x 16 2505 and 1562.
inline int64_t magnify_lanes(int64_t n, int64_t n_t) {
  if (n_t <= 16 && n * n_t >= 4 * RESIDENT_LANES) return MAGNIFY_PAIRS;
  const double w_solved = 1.0 + fmin(1.5, 12.0 / (double)n_t);
  int64_t best = 1;
  double best_cost = 0.0;
  for (int64_t g = 1;; g *= 2) {
    const double r = (double)n * (double)g / (double)RESIDENT_LANES;
    const int64_t C = (n_t + g - 1) / g;
    const double w = tracked_chains(n, g, n_t, C) ? 0.6 : w_solved;
    const double chain = 2.5 + w * (double)(C - 1);
    const double cost = chain * (r < 1.0 ? 1.3 + 0.8 * r : r + 1.1 * sqrt(r));
    if (g == 1 || cost < best_cost) {
      best = g;
      best_cost = cost;
    }
    if (g >= n_t) return best;
  }
}

hipError_t launch_fitness(const FitArgs& a, int mode, bool chi2,
                          hipStream_t stream, int waves_per_block);

// Batched downhill-simplex refinement (sblm_nm.hip): one simplex per
// lightcurve from x0 [6][n_lc] (encoded with lo/span); results as for
// nm_refine.  Allocates and frees its workspace; synchronises `st`.
// Iterated simplex (nm_iterated): `runs` random starts per slot and where
// the best per lightcurve goes.
struct NmIterated {
  uint64_t seed;
  int32_t runs;
  double* x;
  double* chi2;
  double* Fs;
  double* Fb;
  int64_t* n_iter;
};
// One simplex per (lightcurve, rep) from x0, or with `iter` the iterated
// form from drawn starts (x0 and the per-simplex outputs unused).
// `workspace` (nullable): a device block of nm_work_bytes(n_lc * reps) bytes
// that replaces the allocation of the simplices' state; with it the trial
// points take 64 lanes and no root cache, and nothing is allocated.
int nm_run(const sblm_lcs& lcs, int32_t reps, const double* lo, const double* span,
           const double* x0, const nm_config& cfg, double* x, double* chi2, double* Fs,
           double* Fb, int32_t* n_iter, sblm_stats* stats, hipStream_t st,
           const NmIterated* iter = nullptr, void* workspace = nullptr);
size_t nm_work_bytes(int64_t n_simplices);
int nm_check(const nm_config* cfg, const char* who);

}  // namespace sblm
