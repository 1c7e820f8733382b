// State and arguments shared by the CG kernels (solve.hip, cg_grid.hip).
#pragma once

#include <cstdint>

#include "mskm_internal.h"

namespace mskm {

// Per-level solve control and state (one struct per level).
struct CgLevel {
  double rtol2;   // rtol^2 (host)
  double bb;      // b.b
  double rr;      // r.r of the current iterate
  double alpha;   // step of the current iteration
  double beta;    // direction coefficient for the next spmv
  int32_t maxit;  // iteration cap (host)
  int32_t on;     // participates (host)
  int32_t iters;  // iterations done
  int32_t done;   // stopped (converged, capped or broken down)
  int32_t capped; // stopped by the cap or by non-finite data
  int32_t fallback; // flexible CG: 0 network in use, 2 just dropped (restart), 1 dropped
  double rr_prev;   // single-reduction form: r.r and step of the previous iteration
  double alpha_prev;
};

// Single-reduction step decision on the level's sums: gamma = r.z (z = r, or
// M^-1 r when preconditioned), delta = z.A z, rr = r.r. Stops on rr before
// the update; else beta = gamma / gamma_prev, alpha = gamma / (delta - beta
// gamma / alpha_prev). Returns true when the update is to be applied.
__device__ __forceinline__ bool cg1_decide(CgLevel& S, double gamma, double delta, double rr) {
  S.rr = rr;
  const bool finite = isfinite(rr) && isfinite(gamma) && isfinite(delta);
  if (finite && !(rr > S.rtol2 * S.bb)) {
    S.done = 1;
    return false;
  }
  if (!finite || S.iters >= S.maxit) {
    S.done = 1;
    S.capped = 1;
    return false;
  }
  const double beta = S.iters == 0 ? 0.0 : gamma / S.rr_prev;
  const double den = S.iters == 0 ? delta : delta - beta * gamma / S.alpha_prev;
  if (!(den > 0.0) || !isfinite(den) || !(gamma > 0.0)) {  // cannot happen for SPD A (and M) and r != 0
    S.done = 1;
    S.capped = 1;
    return false;
  }
  S.beta = beta;
  S.alpha = gamma / den;
  S.rr_prev = gamma;
  S.alpha_prev = S.alpha;
  S.iters += 1;
  return true;
}

constexpr int kWgSolveRows = 1024;  // largest level solved by one workgroup (k_cg_level_wg)
// Levels of at most this many rows together take the two-waves-per-slice product.
constexpr int64_t kSplitProductRows = 65536;

// Preconditioner arguments (block-Jacobi forms).
template <typename TX>
struct PcArgs {
  const int64_t* start;
  const int32_t* of_row;
  const int64_t* off;
  const TX* inv;
  TX* z;  // z = M^-1 r
};

// cg_grid.hip: the whole CG of levels lo..hi in one launch, their workgroups
// all on the GPU at once. cg_grid_ready decides (building the plan at its
// first use) whether these levels can take it, and with how many lanes per
// row (at most most_lanes; 0: they cannot).
mskm_status cg_grid_ready(mskm_hier* h, int lo, int hi, bool bj, int* lanes, int most_lanes = 2);
// Queues the solve A_l x_l = b_l (x0 = 0) of levels lo..hi; z0, z1, z2: three
// vectors of the hierarchy's length, scratch. st[l] receives the final
// states. *aborted (device, cleared by the caller before the first of several
// launches) is set, and x and st are unusable, when a workgroup's wait ran out;
// launches that find it set give up at once.
template <typename TX>
mskm_status cg_grid_launch(mskm_hier* h, int lo, int hi, bool bj, int lanes, const TX* val, const TX* b, TX* x,
                           TX* z0, TX* z1, TX* z2, CgLevel* st, int32_t* aborted, double rtol2, int maxit,
                           const PcArgs<TX>& pc);

// The same for nrhs right-hand sides (b, x: [N][R], R >= nrhs, zeros past them;
// z0, z1, z2: scratch of that size;
// states to st[l * R + r]), every column a system of its own. *how: 0 when it
// takes more launches than are worth it (nothing is queued), 1 queued, 2 queued
// and *aborted (cleared by the caller) has to be looked at.
struct MrState;
template <typename TX>
mskm_status cg_grid_columns(mskm_hier* h, int lo, int hi, bool bj, const TX* val, const TX* b, TX* x, TX* z0, TX* z1,
                            TX* z2, int nrhs, int R, MrState* st, int32_t* aborted, double rtol2, int maxit, const PcArgs<TX>& pc,
                            int* how);

// cg_stream.hip: the same for all levels of one depth, FP32, where they do not
// fit the registers. cg_stream_ready: *depth is that depth, or -1.
mskm_status cg_stream_ready(mskm_hier* h, int lo, int hi, bool bj, int* depth);
mskm_status cg_stream_launch(mskm_hier* h, int depth, bool bj, const float* b, float* x, float* z0, float* z1,
                             CgLevel* st, int32_t* aborted, double rtol2, int maxit, const PcArgs<float>& pc);

}  // namespace mskm
