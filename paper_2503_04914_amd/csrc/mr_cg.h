// Many-right-hand-side CG (mr_cg.hip) and its workspace.
#pragma once

#include <memory>
#include <vector>

#include "mr_tiles.h"
#include "mskm_internal.h"

namespace mskm {

constexpr int kMaxRPerLane = 8;  // R <= 64 * 8 = 512

struct MrCfg {
  int R, LR, RM;  // right-hand sides, lanes per row, right-hand sides per lane (row-by-row products)
};

// Per-(level, rhs) CG state (index l * R + r).
struct MrState {
  double rtol2, bb, rr, beta;
  double rz;      // r.z with z = M^-1 r (preconditioned), else r.r
  double alpha;   // step of the current iteration (0 once stopped)
  double xalpha;  // step of the last direction that x has not received yet
  int32_t maxit, iters, done, capped;
};

// Per-level statistics kept on the device over a solve.
struct MrLevStat {
  int64_t iters;  // sum over its CG solves and right-hand sides
  int32_t last;   // most iterations of a right-hand side in its last CG solve
  int32_t capped;
};

// Workspace of one many-right-hand-side call: one block of the context's cache.
struct MrWS {
  mskm_ctx* ctx = nullptr;
  MrCfg c{};
  int nrhs = 0;  // right-hand sides that are not padding
  const MrTiles *D = nullptr, *Lw = nullptr;  // tiles of the blocks (null: row by row)
  double *fi = nullptr, *ai = nullptr;        // FP64 f, alpha [N][R], internal order
  void *beta = nullptr, *t = nullptr, *r = nullptr, *p = nullptr, *q = nullptr, *z = nullptr;
  float *f32 = nullptr, *a32 = nullptr;
  double *part_s = nullptr, *part_v = nullptr, *part_z = nullptr;
  double* sums = nullptr;  // [2 L R] level sums of the residual
  bool pc = false;
  MrState* st = nullptr;
  int32_t* running = nullptr;  // [L] systems of each level still running
  int32_t* on = nullptr;       // [L]
  MrLevStat* stat = nullptr;   // [L]
  int32_t* aborted = nullptr;  // the persistent form gave up
  bool grid_off = false;       // no persistent launches (any more)
  int32_t* h_aborted = nullptr;
  int32_t* h_running[2] = {nullptr, nullptr};  // pinned copies behind the two chunks in flight
  hipEvent_t ev[2] = {nullptr, nullptr};
  void* base = nullptr;
  size_t bytes = 0;
  void* pinned = nullptr;
  size_t pinned_bytes = 0;
  struct Graph {
    int lo, hi;
    const void* x;
    hipGraphExec_t exec;
  };
  std::vector<Graph> graphs;  // captured iterations, by levels
  MrWS() = default;
  MrWS(const MrWS&) = delete;
  MrWS& operator=(const MrWS&) = delete;
  ~MrWS();
};

// Vectors a workspace holds: what 0 residual only, 1 FP64 solve, 2 mixed
// solve, 3 CG only (right-hand side in fi, solution the caller's).
mskm_status mr_workspace(mskm_hier* h, int nrhs, int R, int what, bool pc, MrWS& W);

// CG on A_l X_l = B_l (x0 = 0) for the levels with on[l], all right-hand sides
// at once. Queues the work; the host waits only to see when every system has
// stopped. Statistics go to W.stat.
template <typename TV, typename TX>
mskm_status mr_cg(mskm_hier* h, MrWS& W, const TV* dval, const std::vector<char>& on, const TX* b, TX* x, double rtol,
                  int maxit, int K);

// Coefficient vectors of Lagrange functions (Section 4; solve_mr.hip): columns
// of A_l^-1 by CG from zero with unit right-hand sides, `width` at a time. The
// workspace and the captured iterations serve every call of columns().
struct LagrangeSolver {
  mskm_hier* h = nullptr;
  int R = 0;
  std::unique_ptr<MrWS> W;
  mskm_status open(mskm_hier* h, int width);
  // Columns n0 .. n0 + R - 1 of level l: Z [N][R] FP64 device, internal order,
  // rows of level l written (columns past the level's end are zero).
  mskm_status columns(int l, int64_t n0, double rtol, int maxit, double* Z);
  // CG iterations so far (sum over all systems), and whether a cap stopped one.
  mskm_status totals(int64_t* iters, bool* capped);
};

// Row-by-row CG product (solve_mr.hip), where there are no tiles.
template <typename TV, typename TX>
void mr_cg_product_rows(mskm_hier* h, const MrCfg& c, int b0, int nb, const TV* dval, const TX* p, TX* q,
                        const int32_t* running, double* part);
// The CG product as the solver launches it, and the width of its chunks.
template <typename TV, typename TX>
void mr_cg_product(mskm_hier* h, const MrTiles* D, const MrCfg& c, int chunk, int b0, int nb, const TV* dval,
                   const TX* p, TX* q, const int32_t* running, double* part);
template <typename TV, typename TX>
int mr_chunk_for(mskm_hier* h, const MrTiles* D, const MrCfg& c, const TV* dval, const TX* p, TX* q, double* part,
                 const int32_t* running);

// out[l][R] = sums over level l's blocks of part[block][R] (fixed order).
void mr_level_sums(mskm_hier* h, const WorkTable& wt, const double* part, double* out, int R);

template <typename T>
void mr_fill(hipStream_t s, T* v, int64_t n, T x);

inline unsigned mr_nblk(int64_t n, int per) {
  const int64_t b = (n + per - 1) / per;
  return (unsigned)(b < 1 ? 1 : b > (1 << 30) ? (1 << 30) : b);
}

}  // namespace mskm
