// Many right-hand sides in the same launches: CG on A_l X_l = B_l for every
// (level, right-hand side) pair, Jacobi sweeps / forward substitution with a
// multi-vector SpMM, FP64 residuals per right-hand side. Vectors are
// point-major [N][R] in the internal order, so the R values gathered for one
// column are contiguous and a group of lanes reads them in one coalesced
// access; every matrix entry is loaded once per SpMM and applied to all R
// right-hand sides.
//
// Lane mapping: a group of LR lanes (LR = 64 for R >= 64, else the power of
// two >= R) handles one row; lane t of the group owns right-hand sides
// t, t + LR, ... (at most kMaxRPerLane of them).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>

#include "device_common.h"
#include "mr_cg.h"

namespace mskm {

// `cnt` columns of the caller's vectors in[n][stride], input order, into
// internal order [n][R], R >= cnt (columns past cnt are zero), and back.
template <typename TO>
__global__ void __launch_bounds__(kBlock) k_mr_to_internal(const double* __restrict__ in, const int32_t* __restrict__ perm,
                                                           TO* __restrict__ out, int64_t n, int stride, int cnt, int R) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n * R) return;
  const int64_t i = e / R;
  const int r = (int)(e - i * R);
  out[e] = r < cnt ? (TO)in[(int64_t)perm[i] * stride + r] : (TO)0;
}

template <typename TI>
__global__ void __launch_bounds__(kBlock) k_mr_to_input(const TI* __restrict__ in, const int32_t* __restrict__ perm,
                                                        double* __restrict__ out, int64_t n, int nrhs, int R) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n * nrhs) return;
  const int64_t i = e / nrhs;
  const int r = (int)(e - i * nrhs);
  out[(int64_t)perm[i] * nrhs + r] = (double)in[i * R + r];
}

// Y[i][:] = b[i][:] + sign * (A X)[i][:] for rows [r0, r1) (b nullable).
template <typename TV, typename TX>
__global__ void __launch_bounds__(kBlock)
    k_mr_spmm(const int64_t* __restrict__ rp, const int32_t* __restrict__ col, const TV* __restrict__ val,
              const TX* __restrict__ x, const TX* __restrict__ b, TX* __restrict__ y, TX sign, int64_t r0, int64_t r1,
              MrCfg c) {
  const int gl = threadIdx.x % c.LR;
  const int groups_per_block = kBlock / c.LR;
  const int64_t groups = (int64_t)gridDim.x * groups_per_block;
  for (int64_t i = r0 + (int64_t)blockIdx.x * groups_per_block + threadIdx.x / c.LR; i < r1; i += groups) {
    TX acc[kMaxRPerLane];
#pragma unroll
    for (int m = 0; m < kMaxRPerLane; ++m) acc[m] = 0;
    const int64_t ke = rp[i + 1];
    for (int64_t k = rp[i]; k < ke; ++k) {
      const TX v = (TX)val[k];
      const TX* xr = x + (int64_t)col[k] * c.R;
#pragma unroll
      for (int m = 0; m < kMaxRPerLane; ++m) {
        const int r = gl + m * c.LR;
        if (m < c.RM && r < c.R) acc[m] += v * xr[r];
      }
    }
#pragma unroll
    for (int m = 0; m < kMaxRPerLane; ++m) {
      const int r = gl + m * c.LR;
      if (m < c.RM && r < c.R) y[i * c.R + r] = (b ? b[i * c.R + r] : (TX)0) + sign * acc[m];
    }
  }
}

// Block partials of per-rhs sums: each lane holds acc[m] for rhs gl + m*LR;
// the block's row groups are combined in LDS; part[blk*R + r].
__device__ __forceinline__ void mr_block_partial(const double* acc, const MrCfg& c, double* sm, double* part,
                                                 int blk) {
  const int gl = threadIdx.x % c.LR, grp = threadIdx.x / c.LR, ngrp = kBlock / c.LR;
  for (int m = 0; m < c.RM; ++m) {
    const int r = gl + m * c.LR;
    if (r < c.R) sm[grp * c.R + r] = acc[m];
  }
  __syncthreads();
  for (int r = threadIdx.x; r < c.R; r += kBlock) {
    double s = 0.0;
    for (int g = 0; g < ngrp; ++g) s += sm[g * c.R + r];
    part[(size_t)blk * c.R + r] = s;
  }
  __syncthreads();
}

constexpr int kMrLds = kBlock * kMaxRPerLane;  // doubles of LDS for block partials

// Q = A P on the block's rows; partial p.q per rhs.
template <typename TV, typename TX>
__global__ void __launch_bounds__(kBlock)
    k_mr_cg_spmm(const WorkTable wt, int base, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                 const TV* __restrict__ val, const TX* __restrict__ p, TX* __restrict__ q,
                 const int32_t* __restrict__ running, double* __restrict__ pqp, MrCfg c) {
  __shared__ double sm[kMrLds];
  const int blk = base + xcd_block_id(gridDim.x);
  const int l = wt.lev[blk];
  if (running[l] == 0) return;
  const int gl = threadIdx.x % c.LR;
  double part[kMaxRPerLane];
#pragma unroll
  for (int m = 0; m < kMaxRPerLane; ++m) part[m] = 0.0;
  for (int64_t i = wt.row0[blk] + threadIdx.x / c.LR; i < wt.row1[blk]; i += kBlock / c.LR) {
    TX acc[kMaxRPerLane];
#pragma unroll
    for (int m = 0; m < kMaxRPerLane; ++m) acc[m] = 0;
    const int64_t ke = rp[i + 1];
    for (int64_t k = rp[i]; k < ke; ++k) {
      const TX v = (TX)val[k];
      const TX* pr = p + (int64_t)col[k] * c.R;
#pragma unroll
      for (int m = 0; m < kMaxRPerLane; ++m) {
        const int r = gl + m * c.LR;
        if (m < c.RM && r < c.R) acc[m] += v * pr[r];
      }
    }
#pragma unroll
    for (int m = 0; m < kMaxRPerLane; ++m) {
      const int r = gl + m * c.LR;
      if (m < c.RM && r < c.R) {
        q[i * c.R + r] = acc[m];
        part[m] += (double)p[i * c.R + r] * (double)acc[m];
      }
    }
  }
  mr_block_partial(part, c, sm, pqp, blk);
}

// FP64 residual per rhs over the level-aligned SpMV table: partials
// rr[blk][r], ff[blk][r]. Values: stored FP64, else the split FP32 values
// (hi + remainder; an FP32-only hierarchy stores the remainders).
__global__ void __launch_bounds__(kBlock)
    k_mr_residual(const WorkTable wt, const int64_t* __restrict__ drp, const int32_t* __restrict__ dc,
                  const double* __restrict__ dv, const int64_t* __restrict__ lrp, const int32_t* __restrict__ lc,
                  const double* __restrict__ lv, const float* __restrict__ dh, const float* __restrict__ dl,
                  const float* __restrict__ lh, const float* __restrict__ ll, const double* __restrict__ a,
                  const double* __restrict__ f, float* __restrict__ rout, double* __restrict__ rrp,
                  double* __restrict__ ffp, MrCfg c) {
  __shared__ double sm[kMrLds];
  const int blk = xcd_block_id(gridDim.x);
  const int gl = threadIdx.x % c.LR;
  double prr[kMaxRPerLane], pff[kMaxRPerLane];
  for (int m = 0; m < kMaxRPerLane; ++m) prr[m] = pff[m] = 0.0;
  for (int64_t i = wt.row0[blk] + threadIdx.x / c.LR; i < wt.row1[blk]; i += kBlock / c.LR) {
    double acc[kMaxRPerLane];
    for (int m = 0; m < kMaxRPerLane; ++m) acc[m] = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
      const int64_t* rp = pass == 0 ? drp : lrp;
      const int32_t* col = pass == 0 ? dc : lc;
      const double* val = pass == 0 ? dv : lv;
      const float* vh = pass == 0 ? dh : lh;
      const float* vl = pass == 0 ? dl : ll;
      for (int64_t k = rp[i]; k < rp[i + 1]; ++k) {
        const int64_t cc = col[k];
        const double v = val ? val[k] : (double)vh[k] + (double)vl[k];
        const double* ar = a + cc * c.R;
        for (int m = 0; m < c.RM; ++m) {
          const int r = gl + m * c.LR;
          if (r < c.R) acc[m] += v * ar[r];
        }
      }
    }
    for (int m = 0; m < c.RM; ++m) {
      const int r = gl + m * c.LR;
      if (r >= c.R) continue;
      const double fi = f[i * c.R + r];
      const double ri = fi - acc[m];
      if (rout) rout[i * c.R + r] = (float)ri;
      prr[m] += ri * ri;
      pff[m] += fi * fi;
    }
  }
  mr_block_partial(prr, c, sm, rrp, blk);
  mr_block_partial(pff, c, sm, ffp, blk);
}

// Residual of a = 0 (r = f): partials of f.f for both sums.
__global__ void __launch_bounds__(kBlock)
    k_mr_residual_zero(const WorkTable wt, const double* __restrict__ f, float* __restrict__ rout,
                       double* __restrict__ rrp, double* __restrict__ ffp, MrCfg c) {
  __shared__ double sm[kMrLds];
  const int blk = xcd_block_id(gridDim.x);
  const int gl = threadIdx.x % c.LR;
  double pff[kMaxRPerLane];
  for (int m = 0; m < kMaxRPerLane; ++m) pff[m] = 0.0;
  for (int64_t i = wt.row0[blk] + threadIdx.x / c.LR; i < wt.row1[blk]; i += kBlock / c.LR) {
    for (int m = 0; m < c.RM; ++m) {
      const int r = gl + m * c.LR;
      if (r >= c.R) continue;
      const double fi = f[i * c.R + r];
      if (rout) rout[i * c.R + r] = (float)fi;
      pff[m] += fi * fi;
    }
  }
  mr_block_partial(pff, c, sm, rrp, blk);
  mr_block_partial(pff, c, sm, ffp, blk);
}

__global__ void __launch_bounds__(kBlock) k_mr_axpy(const float* __restrict__ d, double* __restrict__ a, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) a[i] += (double)d[i];
}

template <typename TV, typename TX>
void mr_cg_product_rows(mskm_hier* h, const MrCfg& c, int b0, int nb, const TV* dval, const TX* p, TX* q,
                        const int32_t* running, double* part) {
  hipLaunchKernelGGL((k_mr_cg_spmm<TV, TX>), dim3(nb), dim3(kBlock), 0, h->ctx->stream, h->wt_spmv, b0,
                     h->diag.rowptr, h->diag.col, dval, p, q, running, part, c);
}
template void mr_cg_product_rows<float, float>(mskm_hier*, const MrCfg&, int, int, const float*, const float*, float*,
                                               const int32_t*, double*);
template void mr_cg_product_rows<double, double>(mskm_hier*, const MrCfg&, int, int, const double*, const double*,
                                                 double*, const int32_t*, double*);

// ------------------------------------------------------------------ driver

namespace {

// y = f - (T - D) t on the levels l0 .. l1 - 1.
template <typename TV, typename TX>
void mr_lower(mskm_hier* h, const MrWS& W, const TV* lval, const TX* t, const TX* f, TX* y, int l0, int l1) {
  const int64_t r0 = h->h_off[l0], r1 = h->h_off[l1];
  if (r1 <= r0) return;
  if (W.Lw) {
    const std::vector<int32_t>& lb = h->wt_spmv.h_lev_begin;
    mr_tile_lower<TX>(h, *W.Lw, W.c.R, lb[l0], lb[l1] - lb[l0], t, f, y);
    return;
  }
  hipLaunchKernelGGL((k_mr_spmm<TV, TX>), dim3(mr_nblk(r1 - r0, kBlock / W.c.LR)), dim3(kBlock), 0, h->ctx->stream,
                     h->lower.rowptr, h->lower.col, lval, t, f, y, (TX)-1, r0, r1, W.c);
}

template <typename TV, typename TX>
mskm_status mr_solve_internal(mskm_hier* h, MrWS& W, const TV* dval, const TV* lval, const TX* f, TX* alpha,
                              const mskm_solve_opts* o, int* sweeps_done) {
  hipStream_t s = h->ctx->stream;
  const int L = h->L;
  TX* beta = (TX*)W.beta;
  TX* t = (TX*)W.t;
  const size_t NR = (size_t)h->N * W.c.R;
  const int maxit = o->max_cg_iters > 0 ? o->max_cg_iters : 20000;
  const int K = o->check_every > 0 ? o->check_every : 8;
  std::vector<char> on(L, 0);
  if (o->algorithm == MSKM_ALG_SEQUENTIAL) {
    const int D = (int)h->h_depth_begin.size() - 1;
    for (int d = 0; d < D; ++d) {
      const int l0 = h->h_depth_begin[d], l1 = h->h_depth_begin[d + 1];
      mr_lower<TV, TX>(h, W, lval, alpha, f, beta, l0, l1);
      std::fill(on.begin(), on.end(), 0);
      for (int l = l0; l < l1; ++l) on[l] = 1;
      MSKM_TRY((mr_cg<TV, TX>(h, W, dval, on, beta, alpha, o->cg_rtol, maxit, K)));
    }
    *sweeps_done = 0;
    return MSKM_OK;
  }
  int Lmax = 0;
  for (int g = 0; g < h->ngroups; ++g) Lmax = std::max(Lmax, (int)h->h_group_levels[g]);
  const int S = o->sweeps > 0 ? o->sweeps : Lmax;
  MSKM_HIP_TRY(hipMemcpyAsync(beta, f, NR * sizeof(TX), hipMemcpyDeviceToDevice, s));
  for (int l = 0; l < L; ++l) on[l] = h->h_next[l] >= 0;
  for (int sw = 0; sw < S && Lmax > 1; ++sw) {
    MSKM_TRY((mr_cg<TV, TX>(h, W, dval, on, beta, t, o->cg_rtol, maxit, K)));
    mr_lower<TV, TX>(h, W, lval, t, f, beta, 0, L);
    *sweeps_done = sw + 1;
  }
  std::fill(on.begin(), on.end(), 1);
  MSKM_TRY((mr_cg<TV, TX>(h, W, dval, on, beta, alpha, o->cg_rtol, maxit, K)));
  return MSKM_OK;
}

// Per-rhs, per-group relative residuals (host rel[R][ngroups]) of a (null: a
// = 0); rout (nullable) receives the residual rounded to FP32.
mskm_status mr_residual(mskm_hier* h, MrWS& W, const double* a, const double* f, float* rout, std::vector<double>& rel) {
  hipStream_t s = h->ctx->stream;
  const MrCfg c = W.c;
  const WorkTable& wt = h->wt_spmv;
  const dim3 grid(wt.nblocks);
  const Csr &D = h->diag, &Lw = h->lower;
  if (!a)
    hipLaunchKernelGGL(k_mr_residual_zero, grid, dim3(kBlock), 0, s, wt, f, rout, W.part_s, W.part_v, c);
  else if (W.D && W.Lw)
    mr_tile_residual(h, *W.D, *W.Lw, c.R, a, f, rout, W.part_s, W.part_v);
  else
    hipLaunchKernelGGL(k_mr_residual, grid, dim3(kBlock), 0, s, wt, D.rowptr, D.col, D.val, Lw.rowptr, Lw.col, Lw.val,
                       D.val32, D.val32lo, Lw.val32, Lw.val32lo, a, f, rout, W.part_s, W.part_v, c);
  // per-level sums on the device, then per group on the host
  const size_t LR = (size_t)h->L * c.R;
  mr_level_sums(h, wt, W.part_s, W.sums, c.R);
  mr_level_sums(h, wt, W.part_v, W.sums + LR, c.R);
  std::vector<double> sums(2 * LR);
  MSKM_HIP_TRY(hipMemcpyAsync(sums.data(), W.sums, sums.size() * 8, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipStreamSynchronize(s));
  rel.assign((size_t)c.R * h->ngroups, 0.0);
  std::vector<double> rr((size_t)c.R * h->ngroups, 0.0), ff((size_t)c.R * h->ngroups, 0.0);
  for (int l = 0; l < h->L; ++l) {
    const int g = h->h_group[l];
    for (int r = 0; r < c.R; ++r) {
      rr[(size_t)r * h->ngroups + g] += sums[(size_t)l * c.R + r];
      ff[(size_t)r * h->ngroups + g] += sums[LR + (size_t)l * c.R + r];
    }
  }
  for (size_t i = 0; i < rel.size(); ++i) rel[i] = ff[i] > 0.0 ? std::sqrt(rr[i] / ff[i]) : std::sqrt(rr[i]);
  return MSKM_OK;
}

}  // namespace

bool mr_supported(int nrhs) { return nrhs >= 2 && nrhs <= 64 * kMaxRPerLane; }

mskm_status set_mr_chunk(mskm_hier* h, int R, int prec, int chunk) {
  if (!mr_supported(R) || R % 64) return fail(MSKM_EINVAL, "nrhs must be a multiple of 64 in [64, 512]");
  const bool fp32 = prec == MSKM_PREC_FP32;
  if (chunk < 64 || chunk > 512 || (chunk & (chunk - 1)) || R % chunk)
    return fail(MSKM_EINVAL, "chunk must be a power of two in [64, 512] dividing nrhs");
  h->mr_chunk[R / 64 - 1][fp32 ? 1 : 0] = chunk;
  return MSKM_OK;
}

// Mean device time of the many-right-hand-side CG product (q = A_l p for R
// right-hand sides with the partials p.q) on level `level` alone, in the
// chunk width the solver uses for R (tuned here if no solve has), launched
// `repeats` times between two events; vectors of the precision the solve
// uses for prec (FP32 values and vectors, or FP64), allocated here.
template <typename TV, typename TX>
static mskm_status time_mr_product_t(mskm_hier* h, const TV* dval, int level, int R, int repeats, float* avg_ms) {
  hipStream_t s = h->ctx->stream;
  R = mr_width(R);
  int LR = 1;
  while (LR < R && LR < 64) LR <<= 1;
  const MrCfg c{R, LR, (R + LR - 1) / LR};
  const MrTiles* D = nullptr;
  MSKM_TRY(mr_tiles(h, false, &D));
  const WorkTable& ws = h->wt_spmv;
  const int b0 = ws.h_lev_begin[level], nb = ws.h_lev_begin[level + 1] - b0;
  const size_t NR = (size_t)h->N * R;
  TX *p = nullptr, *q = nullptr;
  double* part = nullptr;
  int32_t* running = nullptr;
  Carve cv;
  cv.add(&p, NR);
  cv.add(&q, NR);
  cv.add(&part, (size_t)std::max(ws.nblocks, 1) * R);
  cv.add(&running, (size_t)h->L);
  void* base = nullptr;
  MSKM_TRY(cv.alloc(h->ctx, &base));
  CtxScratch scratch{h->ctx, base, cv.bytes};
  mr_fill<TX>(s, p, (int64_t)NR, (TX)1);
  mr_fill<int32_t>(s, running, (int64_t)h->L, 1);
  const int chunk = mr_chunk_for<TV, TX>(h, D, c, dval, (const TX*)p, q, part, running);
  MSKM_HIP_TRY(hipEventRecord(h->ctx->ev0, s));
  for (int k = 0; k < repeats; ++k) mr_cg_product<TV, TX>(h, D, c, chunk, b0, nb, dval, p, q, running, part);
  float ms = 0.f;
  MSKM_HIP_TRY(hipEventRecord(h->ctx->ev1, s));
  MSKM_HIP_TRY(hipEventSynchronize(h->ctx->ev1));
  MSKM_HIP_TRY(hipEventElapsedTime(&ms, h->ctx->ev0, h->ctx->ev1));
  MSKM_HIP_TRY(hipGetLastError());
  *avg_ms = ms / (float)repeats;
  return MSKM_OK;
}

mskm_status time_mr_product(mskm_hier* h, int level, int prec, int R, int repeats, float* avg_ms) {
  if (!mr_supported(R)) return fail(MSKM_EINVAL, "nrhs out of range for the many-right-hand-side product");
  if (prec == MSKM_PREC_FP32) {
    if (!h->diag.val32) return fail(MSKM_ESTATE, "FP32 values are not stored");
    return time_mr_product_t<float, float>(h, h->diag.val32, level, R, repeats, avg_ms);
  }
  if (!h->diag.val) return fail(MSKM_ESTATE, "FP64 values are not stored");
  return time_mr_product_t<double, double>(h, h->diag.val, level, R, repeats, avg_ms);
}

// Unit right-hand sides of level l: E[i][r] = 1 for i = off + n0 + r (r < nr).
__global__ void __launch_bounds__(kBlock) k_mr_unit(double* __restrict__ E, int64_t off, int64_t n0, int nr, int R) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r < nr) E[(off + n0 + r) * R + r] = 1.0;
}

mskm_status LagrangeSolver::open(mskm_hier* hier, int width) {
  h = hier;
  R = width;
  if (R < 1 || R > 64 * kMaxRPerLane || R != mr_width(R))
    return fail(MSKM_EINVAL, "Lagrange columns: the width must be 16 or a multiple of 32 up to 512");
  if (!h->diag.val) return fail(MSKM_ESTATE, "Lagrange columns: FP64 values are not stored");
  W.reset(new (std::nothrow) MrWS());
  if (!W) return fail(MSKM_ENOMEM, "host memory");
  MSKM_TRY(mr_workspace(h, R, R, 3, false, *W));
  return mr_tiles(h, false, &W->D);
}

mskm_status LagrangeSolver::columns(int l, int64_t n0, double rtol, int maxit, double* Z) {
  hipStream_t s = h->ctx->stream;
  const int64_t nl = h->h_off[l + 1] - h->h_off[l];
  const int nr = (int)std::max<int64_t>(0, std::min<int64_t>(R, nl - n0));
  MSKM_HIP_TRY(hipMemsetAsync(W->fi + (size_t)h->h_off[l] * R, 0, (size_t)nl * R * 8, s));
  if (nr > 0)
    hipLaunchKernelGGL(k_mr_unit, dim3((nr + kBlock - 1) / kBlock), dim3(kBlock), 0, s, W->fi, h->h_off[l], n0, nr, R);
  W->nrhs = std::max(nr, 1);
  std::vector<char> on(h->L, 0);
  on[l] = 1;
  return mr_cg<double, double>(h, *W, h->diag.val, on, W->fi, Z, rtol, maxit, 8);
}

mskm_status LagrangeSolver::totals(int64_t* iters, bool* capped) {
  hipStream_t s = h->ctx->stream;
  std::vector<MrLevStat> S(h->L);
  MSKM_HIP_TRY(hipMemcpyAsync(S.data(), W->stat, S.size() * sizeof(MrLevStat), hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipStreamSynchronize(s));
  *iters = 0;
  *capped = false;
  for (const MrLevStat& l : S) {
    *iters += l.iters;
    *capped |= l.capped != 0;
  }
  return MSKM_OK;
}

// Multi-rhs solve: f, alpha [N][nrhs] (input order; device if io_dev).
mskm_status solve_multi(mskm_hier* h, const double* f_in, int nrhs, const mskm_solve_opts* o, double* alpha_out,
                        mskm_report* rep) {
  hipStream_t s = h->ctx->stream;
  const bool io_dev = (o->flags & MSKM_IO_DEVICE) != 0;
  const bool mixed = o->precision == MSKM_PREC_FP32;
  if (mixed ? !h->diag.val32 : !h->diag.val) return fail(MSKM_ESTATE, "requested precision's values are not stored");
  const bool pc = o->precond == MSKM_PRECOND_BLOCK_JACOBI;
  if (pc) {
    MSKM_TRY(build_block_jacobi(h));
    MSKM_TRY(bj_wait(h, h->L - 1));
  }
  const int R = mr_width(nrhs);  // right-hand sides with padding
  const int64_t NR = h->N * R, NU = h->N * nrhs;  // internal vectors, the caller's
  MrWS W;
  MSKM_TRY(mr_workspace(h, nrhs, R, mixed ? 2 : 1, pc, W));
  MSKM_TRY(mr_tiles(h, false, &W.D));
  MSKM_TRY(mr_tiles(h, true, &W.Lw));
  const double* fdev = f_in;
  double* stage = nullptr;  // the caller's vectors, when they are host arrays (f, then alpha)
  const size_t stage_bytes = (size_t)NU * 8;
  if (!io_dev) {
    void* q = nullptr;
    MSKM_TRY(ctx_alloc(h->ctx, stage_bytes, &q));
    stage = static_cast<double*>(q);
  }
  CtxScratch stage_guard{h->ctx, stage, stage_bytes};
  if (!io_dev) {
    MSKM_HIP_TRY(hipMemcpyAsync(stage, f_in, stage_bytes, hipMemcpyHostToDevice, s));
    fdev = stage;
  }
  int sweeps_done = 0, refine = 0;
  std::vector<double> rel;
  MSKM_HIP_TRY(hipEventRecord(h->ctx->ev0, s));
  hipLaunchKernelGGL(k_mr_to_internal<double>, dim3(mr_nblk(NR, kBlock)), dim3(kBlock), 0, s, fdev, h->perm, W.fi, h->N,
                     nrhs, nrhs, R);
  if (!mixed) {
    MSKM_TRY((mr_solve_internal<double, double>(h, W, h->diag.val, h->lower.val, W.fi, W.ai, o, &sweeps_done)));
    MSKM_TRY(mr_residual(h, W, W.ai, W.fi, nullptr, rel));
  } else {
    const int maxref = o->max_refine > 0 ? o->max_refine : 10;
    MSKM_HIP_TRY(hipMemsetAsync(W.ai, 0, (size_t)NR * 8, s));
    for (;;) {
      MSKM_TRY(mr_residual(h, W, refine == 0 ? nullptr : W.ai, W.fi, W.f32, rel));  // alpha = 0 at the start
      const double worst = *std::max_element(rel.begin(), rel.end());
      if (worst <= o->target_rel_residual || refine >= maxref) break;
      mskm_solve_opts oi = *o;
      if (refine > 0) oi.cg_rtol = std::min(0.1, std::max(o->cg_rtol, 0.5 * o->target_rel_residual / worst));
      MSKM_TRY((mr_solve_internal<float, float>(h, W, h->diag.val32, h->lower.val32, W.f32, W.a32, &oi, &sweeps_done)));
      hipLaunchKernelGGL(k_mr_axpy, dim3(mr_nblk(NR, kBlock)), dim3(kBlock), 0, s, W.a32, W.ai, NR);
      ++refine;
    }
  }
  double* adev = io_dev ? alpha_out : stage;
  hipLaunchKernelGGL(k_mr_to_input<double>, dim3(mr_nblk(NU, kBlock)), dim3(kBlock), 0, s, (const double*)W.ai, h->perm,
                     adev, h->N, nrhs, R);
  MSKM_HIP_TRY(hipEventRecord(h->ctx->ev1, s));
  if (!io_dev) MSKM_HIP_TRY(hipMemcpyAsync(alpha_out, stage, stage_bytes, hipMemcpyDeviceToHost, s));
  std::vector<MrLevStat> stat(h->L);
  MSKM_HIP_TRY(hipMemcpyAsync(stat.data(), W.stat, h->L * sizeof(MrLevStat), hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipStreamSynchronize(s));
  float msec = 0.f;
  MSKM_HIP_TRY(hipEventElapsedTime(&msec, h->ctx->ev0, h->ctx->ev1));
  const double worst = rel.empty() ? 0.0 : *std::max_element(rel.begin(), rel.end());
  int64_t iters = 0;
  bool capped = false;
  for (const MrLevStat& S : stat) {
    iters += S.iters;
    capped = capped || S.capped;
  }
  const bool enoconv = mixed ? worst > o->target_rel_residual : capped;
  if (rep) {
    std::memset(rep, 0, sizeof(*rep));
    rep->levels = h->L;
    rep->sweeps_done = sweeps_done;
    rep->refine_steps = refine;
    rep->cg_iters_total = iters;
    for (int l = 0; l < std::min(h->L, 64); ++l) rep->cg_iters_last[l] = stat[l].last;
    rep->rel_residual = worst;
    rep->solve_ms = msec;
  }
  MSKM_HIP_TRY(hipGetLastError());
  return enoconv ? MSKM_ENOCONV : MSKM_OK;
}

// mskm_residual for several right-hand sides at once, on the tiles of the
// blocks: the matrix is read once for up to 512 of them instead of once each
// (349,504 points, 256 right-hand sides: 3.1 ms against 256 passes of 0.19 ms,
// each with two permutations and a host wait). The tiles cost about as much
// as 16 such passes to build, so fewer right-hand sides use them only when a
// solve has left them. *done stays false where this form does not apply (no
// tiles, no room for the vectors), and where a residual is not finite: the zeros
// of a tile times an infinite coefficient are NaN in rows that do not touch it, so
// an infinite residual is told from an undefined one by the products row by row.
mskm_status residual_multi(mskm_hier* h, const double* alpha, const double* f, int nrhs, double* rel_out, bool* done) {
  *done = false;
  constexpr int kBuildAt = 16, kSlab = 64 * kMaxRPerLane;
  if (nrhs < 2 || (nrhs < kBuildAt && !mr_tiles_built(h))) return MSKM_OK;
  hipStream_t s = h->ctx->stream;
  for (int r0 = 0; r0 < nrhs; r0 += kSlab) {
    const int cnt = std::min(kSlab, nrhs - r0), R = mr_width(cnt);
    MrWS W;
    const mskm_status st = mr_workspace(h, cnt, R, 0, false, W);
    if (st == MSKM_ENOMEM) return MSKM_OK;
    if (st < 0) return st;
    MSKM_TRY(mr_tiles(h, false, &W.D));
    MSKM_TRY(mr_tiles(h, true, &W.Lw));
    if (!W.D || !W.Lw) return MSKM_OK;
    const unsigned nb = mr_nblk(h->N * R, kBlock);
    hipLaunchKernelGGL(k_mr_to_internal<double>, dim3(nb), dim3(kBlock), 0, s, alpha + r0, h->perm, W.ai, h->N, nrhs,
                       cnt, R);
    hipLaunchKernelGGL(k_mr_to_internal<double>, dim3(nb), dim3(kBlock), 0, s, f + r0, h->perm, W.fi, h->N, nrhs, cnt,
                       R);
    std::vector<double> rel;
    MSKM_TRY(mr_residual(h, W, W.ai, W.fi, nullptr, rel));
    for (size_t i = 0; i < (size_t)cnt * h->ngroups; ++i)
      if (!std::isfinite(rel[i])) return MSKM_OK;
    std::memcpy(rel_out + (size_t)r0 * h->ngroups, rel.data(), (size_t)cnt * h->ngroups * sizeof(double));
  }
  *done = true;
  return MSKM_OK;
}

}  // namespace mskm
