// Preconditioned CG for many right-hand sides: one system per (level, right-hand
// side), all of them in each launch, textbook recurrences (Theorem cg) with
// per-system scalars. Vectors are point-major [N][R].
//
// An iteration is five launches: direction (p = z + beta p, with the step of x
// along the previous p, which is read here anyway), product (q = A p with p.q),
// alpha, update (r -= alpha q and z = M^-1 r in one pass, with r.r and r.z),
// beta and the stopping test. Per row and right-hand side that is 5 + 2 + 4
// vector words instead of the 13 of separate direction, step, residual and
// preconditioner passes: the vectors (268 MB each on 262,144 rows with 256
// right-hand sides in FP32) are what bounds a large level. The block inverses
// are small dense products and go through the matrix cores, block rows against
// right-hand sides, in the layout that the residual update already has them.
// Sums over a level's blocks run on one workgroup per 8 right-hand sides: with
// one per 64 they took 30-39 us an iteration on 262,144 rows.
#include <algorithm>
#include <cstring>

#include "cg_state.h"
#include "device_common.h"
#include "mr_cg.h"

namespace mskm {

constexpr int kUpdThreads = 256;  // workgroup of the preconditioned update: 4 waves over the blocks of its group

// Sum of right-hand side r0 + t's partials over blocks [b0, b1) in the threads
// t < 8 of a workgroup of kRedThreads; fixed order.
constexpr int kRedThreads = 1024;
constexpr int kRedRhs = 8;
__device__ __forceinline__ double rhs_sum(const double* __restrict__ part, int b0, int b1, int R, int r0, double* sm) {
  constexpr int kLanes = kRedThreads / kRedRhs, kWaves = kRedThreads / kWave;
  const int t = threadIdx.x, rl = t % kRedRhs, w = t / kWave;
  double v = 0.0;
#pragma unroll 4
  for (int b = b0 + t / kRedRhs; b < b1; b += kLanes) v += part[(size_t)b * R + r0 + rl];
  v += __shfl_xor(v, 8, kWave);
  v += __shfl_xor(v, 16, kWave);
  v += __shfl_xor(v, 32, kWave);
  if (t % kWave < kRedRhs) sm[w * kRedRhs + rl] = v;
  __syncthreads();
  double s = 0.0;
  if (t < kRedRhs)
    for (int k = 0; k < kWaves; ++k) s += sm[k * kRedRhs + t];
  __syncthreads();
  return s;
}

__global__ void __launch_bounds__(kRedThreads)
    k_mr_level_sums(const int32_t* __restrict__ lev_begin, const double* __restrict__ part, double* __restrict__ out,
                    int R) {
  __shared__ double sm[kRedThreads / kWave * kRedRhs];
  const int l = blockIdx.x, r = blockIdx.y * kRedRhs + (int)threadIdx.x;
  const double v = rhs_sum(part, lev_begin[l], lev_begin[l + 1], R, blockIdx.y * kRedRhs, sm);
  if (threadIdx.x < kRedRhs) out[(size_t)l * R + r] = v;
}

void mr_level_sums(mskm_hier* h, const WorkTable& wt, const double* part, double* out, int R) {
  hipLaunchKernelGGL(k_mr_level_sums, dim3(h->L, R / kRedRhs), dim3(kRedThreads), 0, h->ctx->stream, wt.lev_begin,
                     part, out, R);
}

// State before the first residual: nothing stopped, no step taken.
__global__ void __launch_bounds__(kBlock)
    k_mr_state(int lev0, int n, int R, double rtol2, int maxit, MrState* __restrict__ st, int32_t* __restrict__ running) {
  const int e = blockIdx.x * kBlock + threadIdx.x;
  if (e >= n * R) return;
  MrState& S = st[(size_t)lev0 * R + e];
  S.rtol2 = rtol2;
  S.alpha = S.xalpha = S.beta = 0.0;
  S.maxit = maxit;
  S.iters = S.capped = 0;
  S.done = 0;
  if (e % R == 0) running[lev0 + e / R] = 0;
}

// Initial sums (r = b, so rr = bb) and stopping test.
__global__ void __launch_bounds__(kRedThreads)
    k_mr_red_init(int lev0, const int32_t* __restrict__ lev_begin, const double* __restrict__ rrp,
                  const double* __restrict__ rzp, MrState* __restrict__ st, int32_t* __restrict__ running,
                  const int32_t* __restrict__ on, int R) {
  __shared__ double sm[kRedThreads / kWave * kRedRhs];
  const int l = lev0 + blockIdx.x, r0 = blockIdx.y * kRedRhs;
  const double bb = rhs_sum(rrp, lev_begin[l], lev_begin[l + 1], R, r0, sm);
  const double rz = rzp ? rhs_sum(rzp, lev_begin[l], lev_begin[l + 1], R, r0, sm) : bb;
  if (threadIdx.x >= kRedRhs) return;
  MrState& S = st[(size_t)l * R + r0 + threadIdx.x];
  S.bb = S.rr = bb;
  S.rz = rz;
  const bool finite = isfinite(bb);
  const bool conv = finite && !(bb > S.rtol2 * bb);
  S.capped = on[l] && !conv && (!finite || S.maxit <= 0);
  S.done = !on[l] || conv || S.capped;
  if (!S.done) atomicAdd(&running[l], 1);
}

// alpha = r.z / p.q.
__global__ void __launch_bounds__(kRedThreads)
    k_mr_red_a(int lev0, const int32_t* __restrict__ lev_begin, const double* __restrict__ pqp,
               MrState* __restrict__ st, const int32_t* __restrict__ running, int R) {
  __shared__ double sm[kRedThreads / kWave * kRedRhs];
  const int l = lev0 + blockIdx.x, r0 = blockIdx.y * kRedRhs;
  if (running[l] == 0) return;
  const double pq = rhs_sum(pqp, lev_begin[l], lev_begin[l + 1], R, r0, sm);
  if (threadIdx.x >= kRedRhs) return;
  MrState& S = st[(size_t)l * R + r0 + threadIdx.x];
  if (S.done) {  // its last step has reached x
    S.alpha = S.xalpha = 0.0;
  } else if (pq > 0.0 && isfinite(pq)) {
    S.alpha = S.xalpha = S.rz / pq;
  } else {
    S.alpha = S.xalpha = 0.0;
    S.done = 2;  // counted out by k_mr_red_b: `running` does not change while this kernel reads it
    S.capped = !(S.rr <= S.rtol2 * S.bb);
  }
}

// Stopping test and beta. A level whose last system stops here has steps that
// x still misses (xalpha); k_mr_dir's FLUSH form adds them after the last
// iteration.
__global__ void __launch_bounds__(kRedThreads)
    k_mr_red_b(int lev0, const int32_t* __restrict__ lev_begin, const double* __restrict__ rrp,
               const double* __restrict__ rzp, MrState* __restrict__ st, int32_t* __restrict__ running, int R) {
  __shared__ double sm[kRedThreads / kWave * kRedRhs];
  const int l = lev0 + blockIdx.x, r0 = blockIdx.y * kRedRhs;
  if (running[l] == 0) return;
  const double rr = rhs_sum(rrp, lev_begin[l], lev_begin[l + 1], R, r0, sm);
  const double rz = rzp ? rhs_sum(rzp, lev_begin[l], lev_begin[l + 1], R, r0, sm) : rr;
  if (threadIdx.x >= kRedRhs) return;
  MrState& S = st[(size_t)l * R + r0 + threadIdx.x];
  if (S.done == 2) {
    S.done = 1;
    atomicSub(&running[l], 1);
  }
  if (S.done) return;
  S.iters += 1;
  const double old = S.rz;
  S.rr = rr;
  S.rz = rz;
  if (isfinite(rr) && !(rr > S.rtol2 * S.bb)) {
    S.done = 1;
  } else if (!isfinite(rr) || !isfinite(rz) || S.iters >= S.maxit) {
    S.done = 1;
    S.capped = 1;
  } else {
    S.beta = rz / old;
  }
  if (S.done) atomicSub(&running[l], 1);
}

// Adds a level's states to its statistics (one block per level).
__global__ void __launch_bounds__(kBlock)
    k_mr_stats(int lev0, const MrState* __restrict__ st, const int32_t* __restrict__ on, MrLevStat* __restrict__ out,
               int R) {
  __shared__ int sum, most, capped;
  const int l = lev0 + blockIdx.x;
  if (threadIdx.x == 0) sum = most = capped = 0;
  __syncthreads();
  for (int r = threadIdx.x; r < R; r += kBlock) {
    const MrState& S = st[(size_t)l * R + r];
    atomicAdd(&sum, S.iters);
    atomicMax(&most, S.iters);
    if (S.capped || !S.done) capped = 1;
  }
  __syncthreads();
  if (threadIdx.x == 0 && on[l]) {
    out[l].iters += sum;
    out[l].last = most;
    out[l].capped |= capped;
  }
}

// x += xalpha p (the step along the previous direction), then p = z + beta p
// for running systems. FLUSH: the pending step only, whether or not the level
// still runs. Grid (64-row blocks, slices of 16 NT right-hand sides).
template <typename TX, int NT, bool FLUSH>
__global__ void __launch_bounds__(kBlock)
    k_mr_dir(const WorkTable wt, int base, const TX* __restrict__ z, TX* __restrict__ p, TX* __restrict__ x,
             const MrState* __restrict__ st, const int32_t* __restrict__ running, int ldr) {
  const int blk = base + xcd_block_id(gridDim.x);
  const int l = wt.lev[blk];
  if (!FLUSH && running[l] == 0) return;
  const int c = (int)blockIdx.y * 16 * NT + NT * (threadIdx.x % 16);
  TX beta[NT];
  double step[NT];
  bool run[NT];
  bool any = false;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const MrState& S = st[(size_t)l * ldr + c + u];
    run[u] = !S.done;
    beta[u] = (TX)S.beta;
    step[u] = S.xalpha;
    any = any || step[u] != 0.0 || (!FLUSH && run[u]);
  }
  if (!any) return;  // nothing to do for this thread's systems
  const int64_t r1 = wt.row1[blk];
#pragma unroll 4
  for (int64_t i = wt.row0[blk] + threadIdx.x / 16; i < r1; i += kBlock / 16) {
    const size_t e = (size_t)i * ldr + c;
    TX pv[NT], xv[NT];
    load_nt<NT>(p + e, pv);
    load_nt<NT>(x + e, xv);
    TX zv[NT];
    if constexpr (!FLUSH) load_nt<NT>(z + e, zv);
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (step[u] != 0.0) xv[u] = (TX)((double)xv[u] + step[u] * (double)pv[u]);
      if constexpr (!FLUSH)
        if (run[u]) pv[u] = zv[u] + beta[u] * pv[u];
    }
    store_nt<NT>(x + e, xv);
    if constexpr (!FLUSH) store_nt<NT>(p + e, pv);
  }
}

// Partial sums of the waves' values: lane (n, k) holds right-hand sides
// NT n + q of the slice; part[at + r].
template <int NT, int WAVES>
__device__ __forceinline__ void rhs_partial(double (&acc)[NT], double* sm, double* __restrict__ part, size_t at) {
  constexpr int R = 16 * NT;
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    acc[q] += __shfl_xor(acc[q], 16, kWave);
    acc[q] += __shfl_xor(acc[q], 32, kWave);
    if (lane < 16) sm[w * R + NT * lane + q] = acc[q];
  }
  __syncthreads();
  if (threadIdx.x < R) {
    double t = 0.0;
    for (int k = 0; k < WAVES; ++k) t += sm[k * R + threadIdx.x];
    part[at + threadIdx.x] = t;
  }
  __syncthreads();
}

// r -= alpha q with the partial r.r (64-row blocks; no preconditioner, z is
// r). INIT: r = b, x = p = 0.
template <typename TX, int NT, bool INIT>
__global__ void __launch_bounds__(kBlock)
    k_mr_update(const WorkTable wt, int base, const TX* __restrict__ b, TX* __restrict__ x, TX* __restrict__ p,
                TX* __restrict__ r, const TX* __restrict__ q, const MrState* __restrict__ st,
                const int32_t* __restrict__ running, double* __restrict__ rrp, int ldr) {
  __shared__ double sm[kBlock / kWave * 16 * NT];
  const int blk = base + xcd_block_id(gridDim.x);
  const int l = wt.lev[blk];
  if (!INIT && running[l] == 0) return;
  const int c0 = (int)blockIdx.y * 16 * NT, c = c0 + NT * (threadIdx.x % 16);
  double alpha[NT], acc[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    alpha[u] = INIT ? 0.0 : st[(size_t)l * ldr + c + u].alpha;
    acc[u] = 0.0;
  }
  const int64_t r1 = wt.row1[blk];
#pragma unroll 4
  for (int64_t i = wt.row0[blk] + threadIdx.x / 16; i < r1; i += kBlock / 16) {
    const size_t e = (size_t)i * ldr + c;
    TX rv[NT];
    if constexpr (INIT) {
      load_nt<NT>(b + e, rv);
      TX zero[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) zero[u] = (TX)0;
      store_nt<NT>(x + e, zero);
      store_nt<NT>(p + e, zero);
      store_nt<NT>(r + e, rv);
    } else {
      TX qv[NT];
      load_nt<NT>(r + e, rv);
      load_nt<NT>(q + e, qv);
#pragma unroll
      for (int u = 0; u < NT; ++u)
        if (alpha[u] != 0.0) rv[u] = (TX)((double)rv[u] - alpha[u] * (double)qv[u]);
      store_nt<NT>(r + e, rv);
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) acc[u] += (double)rv[u] * (double)rv[u];
  }
  rhs_partial<NT, kBlock / kWave>(acc, sm, rrp, (size_t)blk * ldr + c0);
}

// The same with z = M^-1 r over workgroups of whole preconditioner blocks
// (partials r.r and r.z): wave w takes blocks w, w + 4, ... of its group. A
// block's rows of r sit in the lanes as the matrix instruction's second
// operand, lane (n, k) holding rows k + 4 s of the 16 of step s: a row of the inverse
// is added in the order of its entries. The rows of the inverse are spread over
// the first operand so that lane (n, k) gets the same rows of z as it has of r. Bound by the four vectors
// it streams: 262,144 rows with 256 right-hand sides in FP32 take 191 us, 5.6
// TB/s. It took 315 us with rows loaded one by one under their bounds check and
// sixteen waves on the ten or so blocks of a group.
template <typename TX, int NT, bool INIT>
__global__ void __launch_bounds__(kUpdThreads, 3)
    k_mr_update_bj(const WorkTable wt, int base, const int64_t* __restrict__ start, const int32_t* __restrict__ of_row,
                   const int64_t* __restrict__ off, const TX* __restrict__ inv, const TX* __restrict__ b,
                   TX* __restrict__ x, TX* __restrict__ p, TX* __restrict__ r, const TX* __restrict__ q,
                   TX* __restrict__ z, const MrState* __restrict__ st, const int32_t* __restrict__ running,
                   double* __restrict__ rrp, double* __restrict__ rzp, int ldr) {
  constexpr int kWaves = kUpdThreads / kWave;
  __shared__ double sm[kWaves * 16 * NT];
  const int blk = base + xcd_block_id(gridDim.x);
  const int l = wt.lev[blk];
  if (!INIT && running[l] == 0) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int n = lane % 16, k4 = lane / 16;
  const int c0 = (int)blockIdx.y * 16 * NT, c = c0 + NT * n;
  double alpha[NT], arr[NT], arz[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    alpha[u] = INIT ? 0.0 : st[(size_t)l * ldr + c + u].alpha;
    arr[u] = arz[u] = 0.0;
  }
  const int32_t bfirst = of_row[wt.row0[blk]], blast = of_row[wt.row1[blk] - 1];
  for (int32_t bk = bfirst + w; bk <= blast; bk += kWaves) {
    const int64_t a = start[bk];
    const int m = (int)(start[bk + 1] - a);
    const TX* Mb = inv + off[bk];
    const TX *rb = INIT ? b : r;
    TX rv[2][4][NT], qv[2][4][NT], mv[2][2][4];
    // everything the block needs is asked for at once: rows and inverse entries
    // past its end are read at its last row and dropped (loads under a branch
    // would be waited for one by one)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
      if (16 * kt < m) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const size_t e = (size_t)(a + min(16 * kt + k4 + 4 * s, m - 1)) * ldr + c;
          load_nt<NT>(rb + e, rv[kt][s]);
          if constexpr (!INIT) load_nt<NT>(q + e, qv[kt][s]);
        }
      }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
        if (16 * mt < m && 16 * kt < m) {
#pragma unroll
          for (int s = 0; s < 4; ++s)
            mv[mt][kt][s] = Mb[min(16 * mt + Mma<TX>::spread(n), m - 1) * m + min(16 * kt + k4 + 4 * s, m - 1)];
        }
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int row = 16 * kt + k4 + 4 * s;
        if (row < m) {
          const size_t e = (size_t)(a + row) * ldr + c;
          if constexpr (INIT) {
            TX zero[NT];
#pragma unroll
            for (int u = 0; u < NT; ++u) zero[u] = (TX)0;
            store_nt<NT>(x + e, zero);
            store_nt<NT>(p + e, zero);
          } else {
#pragma unroll
            for (int u = 0; u < NT; ++u)
              if (alpha[u] != 0.0) rv[kt][s][u] = (TX)((double)rv[kt][s][u] - alpha[u] * (double)qv[kt][s][u]);
          }
          store_nt<NT>(r + e, rv[kt][s]);
#pragma unroll
          for (int u = 0; u < NT; ++u) arr[u] += (double)rv[kt][s][u] * (double)rv[kt][s][u];
        } else {
#pragma unroll
          for (int u = 0; u < NT; ++u) rv[kt][s][u] = (TX)0;
        }
      }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      if (16 * mt >= m) continue;
      typename Mma<TX>::acc d[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) d[u] = (typename Mma<TX>::acc)(TX)0;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        if (16 * kt >= m) continue;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const bool in = 16 * mt + Mma<TX>::spread(n) < m && 16 * kt + k4 + 4 * s < m;
          const TX av = in ? mv[mt][kt][s] : (TX)0;
#pragma unroll
          for (int u = 0; u < NT; ++u) d[u] = Mma<TX>::mul(av, rv[kt][s][u], d[u]);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * mt + k4 + 4 * i;
        if (row < m) {
          TX zv[NT];
#pragma unroll
          for (int u = 0; u < NT; ++u) {
            zv[u] = d[u][i];
            arz[u] += (double)rv[mt][i][u] * (double)zv[u];
          }
          store_nt<NT>(z + (size_t)(a + row) * ldr + c, zv);
        }
      }
    }
  }
  rhs_partial<NT, kWaves>(arr, sm, rrp, (size_t)blk * ldr + c0);
  rhs_partial<NT, kWaves>(arz, sm, rzp, (size_t)blk * ldr + c0);
}

// ------------------------------------------------------------------- driver

template <typename T>
__global__ void __launch_bounds__(kBlock) k_mr_fill(T* __restrict__ v, int64_t n, T x) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) v[i] = x;
}
template <typename T>
void mr_fill(hipStream_t s, T* v, int64_t n, T x) {
  hipLaunchKernelGGL(k_mr_fill<T>, dim3(mr_nblk(n, kBlock)), dim3(kBlock), 0, s, v, n, x);
}
template void mr_fill<float>(hipStream_t, float*, int64_t, float);
template void mr_fill<double>(hipStream_t, double*, int64_t, double);
template void mr_fill<int32_t>(hipStream_t, int32_t*, int64_t, int32_t);

MrWS::~MrWS() {
  for (hipEvent_t e : ev)
    if (e) {
      (void)hipEventSynchronize(e);  // a copy into the pinned block may be in flight
      (void)hipEventDestroy(e);
    }
  for (Graph& g : graphs) (void)hipGraphExecDestroy(g.exec);
  if (base) ctx_release(ctx, base, bytes);
  if (pinned) ctx_host_release(ctx, pinned, pinned_bytes);
}

mskm_status mr_workspace(mskm_hier* h, int nrhs, int R, int what, bool pc, MrWS& W) {
  W.nrhs = nrhs;
  W.ctx = h->ctx;
  W.pc = pc;
  W.grid_off = what != 0 && grid_resting(h->ctx);
  int LR = 1;
  while (LR < R && LR < 64) LR <<= 1;
  W.c = MrCfg{R, LR, (R + LR - 1) / LR};
  const size_t NR = (size_t)h->N * R, L = (size_t)h->L;
  const size_t xs = what == 2 ? 4 : 8;
  const size_t nb = (size_t)std::max(h->wt_spmv.nblocks, pc ? h->bj.wt.nblocks : 0) * R;
  Carve cv;
  cv.add(&W.fi, NR);
  if (what != 3) cv.add(&W.ai, NR);
  cv.add(&W.part_s, nb);
  cv.add(&W.part_v, nb);
  if (what != 3) cv.add(&W.sums, 2 * L * R);
  char *beta = nullptr, *t = nullptr, *r = nullptr, *p = nullptr, *q = nullptr, *z = nullptr;
  if (what != 0) {
    for (char** v : {&r, &p, &q}) cv.add(v, NR * xs);
    if (what != 3)
      for (char** v : {&beta, &t}) cv.add(v, NR * xs);
    if (pc) {
      cv.add(&z, NR * xs);
      cv.add(&W.part_z, nb);
    }
    if (what == 2) {
      cv.add(&W.f32, NR);
      cv.add(&W.a32, NR);
    }
    cv.add(&W.st, L * R);
    cv.add(&W.running, L);
    cv.add(&W.on, L);
    cv.add(&W.stat, L);
    cv.add(&W.aborted, 1);
  }
  MSKM_TRY(cv.alloc(h->ctx, &W.base));
  W.bytes = cv.bytes;
  W.beta = beta;
  W.t = t;
  W.r = r;
  W.p = p;
  W.q = q;
  W.z = z;
  if (what == 0) return MSKM_OK;
  W.pinned_bytes = (2 * L + 1) * sizeof(int32_t);
  MSKM_TRY(ctx_host_alloc(h->ctx, W.pinned_bytes, &W.pinned));
  W.h_running[0] = static_cast<int32_t*>(W.pinned);
  W.h_running[1] = W.h_running[0] + L;
  W.h_aborted = W.h_running[1] + L;
  for (hipEvent_t& e : W.ev) MSKM_HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  MSKM_HIP_TRY(hipMemsetAsync(W.stat, 0, L * sizeof(MrLevStat), h->ctx->stream));
  return MSKM_OK;
}

template <typename TV, typename TX>
void mr_cg_product(mskm_hier* h, const MrTiles* D, const MrCfg& c, int chunk, int b0, int nb, const TV* dval,
                   const TX* p, TX* q, const int32_t* running, double* part) {
  if (nb <= 0) return;
  if (D)
    mr_tile_cg<TX>(h, *D, c.R, chunk, b0, nb, p, q, running, part);
  else
    mr_cg_product_rows<TV, TX>(h, c, b0, nb, dval, p, q, running, part);
}
template void mr_cg_product<float, float>(mskm_hier*, const MrTiles*, const MrCfg&, int, int, int, const float*,
                                          const float*, float*, const int32_t*, double*);
template void mr_cg_product<double, double>(mskm_hier*, const MrTiles*, const MrCfg&, int, int, int, const double*,
                                            const double*, double*, const int32_t*, double*);

// Chunk width of the CG product for this R: the fastest of the candidates
// (64, 128, 256, 512, dividing R and not less than a workgroup's) timed once per hierarchy, R and precision on
// its largest level, then kept (the timing overwrites q and the partials,
// which the solve rewrites).
template <typename TV, typename TX>
int mr_chunk_for(mskm_hier* h, const MrTiles* D, const MrCfg& c, const TV* dval, const TX* p, TX* q, double* part,
                 const int32_t* running) {
  if (!D || c.R % 64) return c.R;
  int32_t& slot = h->mr_chunk[c.R / 64 - 1][sizeof(TX) == 4 ? 1 : 0];
  if (slot > 0) return slot;
  int big = 0;  // the largest level (a solve's first call may run only the coarsest)
  for (int l = 1; l < h->L; ++l)
    if (h->h_lev[l].n > h->h_lev[big].n) big = l;
  const WorkTable& ws = h->wt_spmv;
  const int b0 = ws.h_lev_begin[big], nb = ws.h_lev_begin[big + 1] - b0;
  hipStream_t s = h->ctx->stream;
  const int least = std::max(64, mr_cg_width<TX>(c.R));
  int best = least;
  float best_ms = 0.f;
  for (int ch = least; ch <= std::min(c.R, 512); ch *= 2) {
    if (c.R % ch) continue;
    mr_cg_product<TV, TX>(h, D, c, ch, b0, nb, dval, p, q, running, part);  // warm
    float ms = 0.f;
    if (hipEventRecord(h->ctx->ev0, s) != hipSuccess) return least;
    for (int k = 0; k < 2; ++k) mr_cg_product<TV, TX>(h, D, c, ch, b0, nb, dval, p, q, running, part);
    if (hipEventRecord(h->ctx->ev1, s) != hipSuccess || hipEventSynchronize(h->ctx->ev1) != hipSuccess ||
        hipEventElapsedTime(&ms, h->ctx->ev0, h->ctx->ev1) != hipSuccess)
      return least;
    if (ch == least || ms < best_ms) {
      best = ch;
      best_ms = ms;
    }
  }
  slot = best;
  return best;
}
template int mr_chunk_for<float, float>(mskm_hier*, const MrTiles*, const MrCfg&, const float*, const float*, float*,
                                        double*, const int32_t*);
template int mr_chunk_for<double, double>(mskm_hier*, const MrTiles*, const MrCfg&, const double*, const double*,
                                          double*, double*, const int32_t*);

namespace {

template <typename TX>
struct MrRun {  // one CG call's launches
  mskm_hier* h;
  MrWS& W;
  int lo, hi, chunk;
  const TX* b;
  TX* x;
  const TX* inv;

  template <int NT, bool INIT>
  void update_nt() const {
    hipStream_t s = h->ctx->stream;
    const int R = W.c.R;
    TX *r = (TX*)W.r, *p = (TX*)W.p, *q = (TX*)W.q, *z = (TX*)W.z;
    const WorkTable& wt = W.pc ? h->bj.wt : h->wt_spmv;
    const int b0 = wt.h_lev_begin[lo], nb = wt.h_lev_begin[hi + 1] - b0;
    if (nb <= 0) return;
    const dim3 grid(nb, R / (16 * NT));
    if (W.pc)
      hipLaunchKernelGGL((k_mr_update_bj<TX, NT, INIT>), grid, dim3(kUpdThreads), 0, s, wt, b0, h->bj.start,
                         h->bj.of_row, h->bj.off, inv, b, x, p, r, q, z, W.st, W.running, W.part_v, W.part_z, R);
    else
      hipLaunchKernelGGL((k_mr_update<TX, NT, INIT>), grid, dim3(kBlock), 0, s, wt, b0, b, x, p, r, q, W.st, W.running,
                         W.part_v, R);
  }
  template <int NT, bool FLUSH>
  void dir_nt() const {
    const WorkTable& wt = h->wt_spmv;
    const int b0 = wt.h_lev_begin[lo], nb = wt.h_lev_begin[hi + 1] - b0;
    if (nb <= 0) return;
    hipLaunchKernelGGL((k_mr_dir<TX, NT, FLUSH>), dim3(nb, W.c.R / (16 * NT)), dim3(kBlock), 0, h->ctx->stream, wt, b0,
                       W.pc ? (const TX*)W.z : (const TX*)W.r, (TX*)W.p, x, W.st, W.running, W.c.R);
  }
  template <bool INIT>
  void update() const {
    switch (mr_lane_rhs<TX>(W.c.R)) {
      case 4:
        if constexpr (sizeof(TX) == 4) update_nt<4, INIT>();
        break;
      case 2:
        update_nt<2, INIT>();
        break;
      default:
        update_nt<1, INIT>();
    }
  }
  template <bool FLUSH>
  void dir() const {
    switch (mr_lane_rhs<TX>(W.c.R)) {
      case 4:
        if constexpr (sizeof(TX) == 4) dir_nt<4, FLUSH>();
        break;
      case 2:
        dir_nt<2, FLUSH>();
        break;
      default:
        dir_nt<1, FLUSH>();
    }
  }
};

}  // namespace

template <typename TV, typename TX>
mskm_status mr_cg(mskm_hier* h, MrWS& W, const TV* dval, const std::vector<char>& on, const TX* b, TX* x, double rtol,
                  int maxit, int K) {
  hipStream_t s = h->ctx->stream;
  const int R = W.c.R, L = h->L;
  int lo = 0, hi = L - 1;
  while (lo < L && !on[lo]) ++lo;
  while (hi >= 0 && !on[hi]) --hi;
  if (lo > hi) return MSKM_OK;
  const int nlev = hi - lo + 1;
  const TX* inv = nullptr;
  if (W.pc) {
    if constexpr (sizeof(TX) == 8)
      inv = h->bj.inv;
    else
      inv = h->bj.inv32;
  }
  TX *p = (TX*)W.p, *q = (TX*)W.q;
  std::vector<int32_t> on32(on.begin(), on.end());
  MSKM_HIP_TRY(hipMemcpyAsync(W.on, on32.data(), L * 4, hipMemcpyHostToDevice, s));  // pageable: copied before return
  // small levels: every column solved by workgroups of its own in one launch
  // (cg_grid.hip). Launched, an iteration is five launches of 3-9 us however
  // small the level is.
  bool all_on = dval != nullptr && !W.grid_off;
  for (int l = lo; l <= hi; ++l) all_on = all_on && on[l];
  if (all_on) {
    int how = 0;
    MSKM_HIP_TRY(hipMemsetAsync(W.aborted, 0, 4, s));
    const PcArgs<TX> pc{h->bj.start, h->bj.of_row, h->bj.off, inv, nullptr};
    MSKM_TRY((cg_grid_columns<TX>(h, lo, hi, W.pc, dval, b, x, p, q, (TX*)W.r, W.nrhs, R, W.st, W.aborted, rtol * rtol,
                                 maxit, pc, &how)));
    *W.h_aborted = 0;
    if (how == 2) {
      MSKM_HIP_TRY(hipMemcpyAsync(W.h_aborted, W.aborted, 4, hipMemcpyDeviceToHost, s));
      MSKM_HIP_TRY(hipEventRecord(W.ev[0], s));
      MSKM_HIP_TRY(hipEventSynchronize(W.ev[0]));
      if (*W.h_aborted) {
        ++h->ctx->given_up;
        h->ctx->grid_rest = kGridRest;
        W.grid_off = true;
      }
    }
    if (how > 0 && *W.h_aborted == 0) {
      hipLaunchKernelGGL(k_mr_stats, dim3(nlev), dim3(kBlock), 0, s, lo, W.st, W.on, W.stat, R);
      MSKM_HIP_TRY(hipGetLastError());
      return MSKM_OK;
    }
  }
  // chunk width of the product (timed at the first solve with this R, every level running)
  mr_fill<int32_t>(s, W.running, L, 1);
  const int chunk = mr_chunk_for<TV, TX>(h, W.D, W.c, dval, p, q, W.part_s, W.running);
  const MrRun<TX> run{h, W, lo, hi, chunk, b, x, inv};
  hipLaunchKernelGGL(k_mr_state, dim3(mr_nblk((int64_t)nlev * R, kBlock)), dim3(kBlock), 0, s, lo, nlev, R,
                     rtol * rtol, maxit, W.st, W.running);
  run.template update<true>();
  const dim3 rgrid(nlev, R / kRedRhs), rblock(kRedThreads);
  const WorkTable& ws = h->wt_spmv;
  const int32_t* ulb = W.pc ? h->bj.wt.lev_begin : ws.lev_begin;  // blocks of the update's partials
  const double* rzp = W.pc ? W.part_z : nullptr;
  hipLaunchKernelGGL(k_mr_red_init, rgrid, rblock, 0, s, lo, ulb, W.part_v, rzp, W.st, W.running, W.on, R);
  // K iterations, captured once into a graph: its kernels read and update the
  // per-system state, so each replay continues the solve
  hipGraphExec_t exec = nullptr;
  for (const MrWS::Graph& g : W.graphs)
    if (g.lo == lo && g.hi == hi && g.x == x) exec = g.exec;
  if (!exec) {
    const int sb0 = ws.h_lev_begin[lo], sbn = ws.h_lev_begin[hi + 1] - sb0;
    hipGraph_t graph = nullptr;
    MSKM_HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    for (int k = 0; k < K; ++k) {
      run.template dir<false>();
      mr_cg_product<TV, TX>(h, W.D, W.c, chunk, sb0, sbn, dval, p, q, W.running, W.part_s);
      hipLaunchKernelGGL(k_mr_red_a, rgrid, rblock, 0, s, lo, ws.lev_begin, W.part_s, W.st, W.running, R);
      run.template update<false>();
      hipLaunchKernelGGL(k_mr_red_b, rgrid, rblock, 0, s, lo, ulb, W.part_v, rzp, W.st, W.running, R);
    }
    MSKM_HIP_TRY(hipStreamEndCapture(s, &graph));
    const hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return fail(MSKM_EDEVICE, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
    W.graphs.push_back(MrWS::Graph{lo, hi, x, exec});
  }
  // two replays in flight: the second runs while the host reads the first's
  // running counts; replays past the end are no-ops
  const int most = (maxit + K - 1) / K;
  int launched = 0, checked = 0;
  auto launch = [&]() -> mskm_status {
    const int k = launched & 1;
    MSKM_HIP_TRY(hipGraphLaunch(exec, s));
    MSKM_HIP_TRY(hipMemcpyAsync(W.h_running[k], W.running, L * 4, hipMemcpyDeviceToHost, s));
    MSKM_HIP_TRY(hipEventRecord(W.ev[k], s));
    ++launched;
    return MSKM_OK;
  };
  if (most > 0) MSKM_TRY(launch());
  while (checked < launched) {
    if (launched < most) MSKM_TRY(launch());
    MSKM_HIP_TRY(hipEventSynchronize(W.ev[checked & 1]));
    const int32_t* c = W.h_running[checked & 1];
    ++checked;
    bool any = false;
    for (int l = lo; l <= hi; ++l) any |= c[l] != 0;
    if (!any) break;
  }
  run.template dir<true>();  // steps of the last iteration
  hipLaunchKernelGGL(k_mr_stats, dim3(nlev), dim3(kBlock), 0, s, lo, W.st, W.on, W.stat, R);
  MSKM_HIP_TRY(hipGetLastError());
  return MSKM_OK;
}
template mskm_status mr_cg<float, float>(mskm_hier*, MrWS&, const float*, const std::vector<char>&, const float*,
                                         float*, double, int, int);
template mskm_status mr_cg<double, double>(mskm_hier*, MrWS&, const double*, const std::vector<char>&, const double*,
                                           double*, double, int, int);

}  // namespace mskm
