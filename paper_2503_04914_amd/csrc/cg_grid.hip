// CG on one or more middle-sized levels in one launch (x0 = 0; Theorem cg), plain
// or with the cell block-Jacobi preconditioner, with every workgroup of the
// levels on the GPU at once and every matrix entry, inverse entry and vector of its
// rows held on its CU.
//
// What bounds a level of 10^3 .. 10^5 rows is not its bytes but the chain of
// dependent steps of an iteration: as separate launches it took two to five
// kernels of 3-6 us each (the preconditioned FP32 form 12 us, the textbook
// FP64 form 17 us an iteration on 16,384 rows). Here an iteration is one or two
// exchanges between the level's workgroups, about 1.5 us each, plus the work on
// rows that never leave the CU.
//
// Three forms. FP32 and preconditioned solves take the single-reduction form of
// the launched kernels (kFormOneRed): z = M^-1 r anew in every iteration, exchanged
// for the halo, then q = A z and the sums z.q, r.z, r.r. Their FP32 arithmetic is
// the launched kernels' element by element, the order within a row included
// (GridSum): only the FP64 sums are added in another order, so a mixed solve
// leaves the coefficients that the launched kernels leave. (Carrying z along by
// z -= alpha M^-1 q instead saves the halo's exchange, 336 against 371 us for 58,000
// FP32 rows, but z then keeps the rounding of its first, large values: FP32 solves
// broke off at 1e-6 of the right-hand side, or ran to their cap, and FP64 ones at
// 1e-14.)
//
// FP64 without preconditioner (kFormPred) has one exchange an iteration: with q =
// A p in hand, a workgroup publishes p.q, r.r, q.r, q.q of its rows, and q. The sums
// give the step alpha = r.r / p.q, the stopping test on r.r, and r.r after the
// step, r.r - 2 alpha q.r + alpha^2 q.q, so that the next direction needs nothing
// more: the halo's r and direction are carried along by every workgroup that reads
// them, by the same operations as their owner's. r.r itself is summed anew every
// time, only beta uses the predicted value. Against the two exchanges of the textbook
// order: 22,000 rows 881 us a solve (1,333 before), 1,089 rows 399 us (545).
// Coefficients against 64 bits, 12 to 24 point sets of each of six sizes from 1,600 to
// 80,000 points: 0.95 to 1.05 times the launched kernels' error in the geometric mean
// of a size, 0.3 to 2.1 times in single cases (where the last iteration happens to
// stop).
//
// Columns of many right-hand sides, FP32 or preconditioned, take the textbook form
// of their launched kernels (kFormText), again in their order: r.r, r.z and the
// halo's z in one exchange, p.q in the other.
//
// Exchange without a barrier or a cache flush: every workgroup stores its
// partial sums into a slot of its own with device-coherent (agent scope)
// stores, and every workgroup polls all slots of its level with
// device-coherent loads until each holds something other than kEmptySlot, a
// bit pattern that no stored value has. The polled words carry the data, so
// nothing has to be ordered before them. The entries of w that a workgroup
// needs from its neighbours travel the same way. Agent-scope fences, which write
// back and invalidate a whole XCD's L2, are not used. Measured: 1.4 / 1.5 /
// 2.0 us an exchange for 64 / 128 / 256 workgroups with slots 64 bytes apart
// (2.3 / 2.8 / 3.3 us with adjacent slots; a counter barrier with fences 3.4 /
// 5.5 / 10.4 us).
//
// Reuse of the buffers. kFormPred: exchange m uses buffer m % 3 (exchange 0 has the
// halo's first r only). A workgroup empties its words of exchange m - 1 once it has
// received exchange m, which everybody published after leaving m - 1. All stores of
// a workgroup are waited for before it publishes m + 1, so whoever has received m +
// 1 sees the emptied words, and polls that buffer again only then, for m + 2.
// kFormOneRed: iteration n's z is in buffer n % 2, its sums in n % 3. Everybody
// publishes the sums after receiving z, and the sums after leaving the sums before:
// with the sums of n received, a workgroup empties its z of n and its sums of n - 1,
// waits for these stores before it publishes the sums of n + 1, and the words are
// polled again for z of n + 2 and the sums of n + 2, both after the sums of n + 1.
// kFormText: the sums with z (A) and p.q (B) of iteration n are in buffer n % 2; A
// and z of n are emptied after B of n, B of n - 1 after A of n, the stores waited
// for before B of n + 1 or n, and polled again after that.
//
// Waiting: every poll loop ends after `spin` polls, and a thread that has waited
// that long does not wait again. A workgroup that gives up sets *aborted and
// leaves, the others then give up the same way, the launches queued behind it
// give up at once, and the caller solves the levels by the launched kernels
// instead. All workgroups of
// a launch must be on the GPU together: at most one per CU is launched, and
// launches of this kernel from different streams of the process are ordered
// one after the other (another kernel only delays the start).
#include <algorithm>
#include <mutex>
#include <vector>

#include "cg_grid.h"
#include "cg_state.h"
#include "device_common.h"
#include "mr_cg.h"

namespace mskm {

constexpr int kGridE = 64;          // matrix entries per lane kept in registers (at most)
constexpr int kGridLocal = 4096;    // direction entries per workgroup: its rows and its halo
constexpr int64_t kGridLevelRows = 131072;  // column bitmap of the plan: 16 KiB of LDS

// Levels that can be solved this way with 512 / lanes rows per workgroup:
// workgroup w of level l takes `per` consecutive blocks of the level's
// work table (64-row blocks, or the preconditioner's workgroups of whole blocks).
struct CgGridDev {
  int32_t nwg = 0;
  int32_t* wg0 = nullptr;           // device [L + 1]
  int32_t* lev = nullptr;           // [nwg]
  int32_t* row0 = nullptr;          // [nwg] first row
  int32_t* nrow = nullptr;          // [nwg]
  int32_t* nhalo = nullptr;         // [nwg]
  int32_t* halo = nullptr;          // [nwg][kGridLocal] rows of the halo, ascending
  uint16_t* lidx = nullptr;         // [nwg][entry of the row][row] position of each entry's column, kGridE kGridThreads
  int32_t* stats = nullptr;         // [2 L] h_local, h_row
  int32_t nslot = 0;                // workgroups of one launch (at most)
  uint64_t* slots = nullptr;        // [3][nslot][kGridSlot]: three buffers
};
struct CgGridPlan {
  bool built = false;
  std::vector<int32_t> h_wg0;       // [L + 1] first workgroup of each level
  std::vector<int32_t> h_local;     // [L] most direction entries of one of its workgroups
  std::vector<int32_t> h_row;       // [L] longest row
  CgGridDev d;
};

struct CgGrid {
  CgGridPlan plan[2][2];  // [block-Jacobi][lanes per row 2, 1]
};

static void cg_grid_free(void* p) { delete static_cast<CgGrid*>(p); }

// --------------------------------------------------------------------- plan

// One workgroup per planned workgroup: its halo (columns of
// its rows outside its rows, ascending) by a bitmap over the level, and each
// entry's position in the workgroup's vector (own rows first, then the halo).
__global__ void __launch_bounds__(kGridThreads)
    k_grid_plan(const CgGridDev P, int L, int lanes, int per, const DevLevel* __restrict__ lev, const WorkTable wt,
                const int64_t* __restrict__ rp, const int32_t* __restrict__ col) {
  constexpr int kWords = (int)(kGridLevelRows / 32);
  constexpr int kPer = kWords / kGridThreads;  // bitmap words per thread in the scan
  __shared__ uint32_t bits[kWords];
  __shared__ uint32_t rank[kWords];
  __shared__ uint32_t ws[kGridThreads / kWave];
  __shared__ int maxlen;
  const int wg = blockIdx.x, t = threadIdx.x;
  const int l = P.lev[wg];
  const int64_t off = lev[l].off;
  const int b0 = wt.lev_begin[l] + (wg - P.wg0[l]) * per;
  const int b1 = min(b0 + per, wt.lev_begin[l + 1]);
  const int64_t r0 = wt.row0[b0];
  const int nr = (int)(wt.row1[b1 - 1] - r0);
  for (int w = t; w < kWords; w += kGridThreads) bits[w] = 0;
  if (t == 0) maxlen = 0;
  __syncthreads();
  const int64_t e0 = rp[r0], e1 = rp[r0 + nr];
  for (int64_t k = e0 + t; k < e1; k += kGridThreads) {
    const int64_t c = col[k];
    if (c < r0 || c >= r0 + nr) atomicOr(&bits[(c - off) >> 5], 1u << ((c - off) & 31));
  }
  __syncthreads();
  // rank[w] = set bits before word w
  uint32_t sum = 0;
  for (int q = 0; q < kPer; ++q) sum += __popc(bits[t * kPer + q]);
  uint32_t inc = sum;
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t v = __shfl_up(inc, o, kWave);
    if (t % kWave >= o) inc += v;
  }
  if (t % kWave == kWave - 1) ws[t / kWave] = inc;
  __syncthreads();
  uint32_t base = inc - sum, total = 0;
  for (int w = 0; w < kGridThreads / kWave; ++w) {
    if (w < t / kWave) base += ws[w];
    total += ws[w];
  }
  for (int q = 0; q < kPer; ++q) {
    const int w = t * kPer + q;
    rank[w] = base;
    base += __popc(bits[w]);
  }
  __syncthreads();
  for (int w = t; w < kWords; w += kGridThreads) {
    uint32_t m = bits[w];
    int pos = (int)rank[w];
    while (m) {
      const int b = __ffs(m) - 1;
      m &= m - 1;
      if (pos < kGridLocal) P.halo[(size_t)wg * kGridLocal + pos] = (int32_t)(off + 32 * w + b);
      ++pos;
    }
  }
  const int i = t / lanes, g = t % lanes;
  int len = 0;
  if (i < nr) {
    const int64_t s = rp[r0 + i], e = rp[r0 + i + 1];
    len = (int)min<int64_t>(e - s, INT32_MAX);
    for (int k = 0; k < kGridE; ++k) {
      const int64_t q = s + g + (int64_t)k * lanes;
      if (q >= e) break;
      const int64_t c = col[q];
      int p;
      if (c >= r0 && c < r0 + nr) {
        p = (int)(c - r0);
      } else {
        const int64_t d = c - off;
        p = nr + (int)(rank[d >> 5] + __popc(bits[d >> 5] & ((1u << (d & 31)) - 1u)));
      }
      P.lidx[(size_t)wg * kGridE * kGridThreads + (g + k * lanes) * (kGridThreads / lanes) + i] =
          (uint16_t)min(p, kGridLocal - 1);
    }
  }
  atomicMax(&maxlen, len);
  __syncthreads();
  if (t == 0) {
    P.row0[wg] = (int32_t)r0;
    P.nrow[wg] = nr;
    P.nhalo[wg] = (int32_t)min(total, (uint32_t)kGridLocal);
    atomicMax(&P.stats[l], nr + (int)total);
    atomicMax(&P.stats[L + l], maxlen);
  }
}

static mskm_status build_plan(mskm_hier* h, CgGridPlan& P, bool bj, int lanes) {
  const int L = h->L;
  const WorkTable& wt = bj ? h->bj.wt : h->wt_spmv;
  // the preconditioner's workgroups hold at most 256 rows on levels of up to kGridLevelRows
  const int per = bj ? (lanes == 2 ? 1 : 2) : kGridThreads / lanes / 64;
  CgGridDev& D = P.d;
  P.h_wg0.assign(L + 1, 0);
  P.h_local.assign(L, 0);
  P.h_row.assign(L, 0);
  std::vector<int32_t> lev;
  const int nd = (int)h->h_depth_begin.size() - 1;
  for (int d = 0; d < nd; ++d) {  // depths whose levels fit the GPU together
    const int l0 = h->h_depth_begin[d], l1 = h->h_depth_begin[d + 1];
    int64_t tot = 0, rows = 0;
    for (int l = l0; l < l1; ++l) {
      tot += (wt.h_lev_begin[l + 1] - wt.h_lev_begin[l] + per - 1) / per;
      rows = std::max<int64_t>(rows, h->h_lev[l].n);
    }
    const bool in = tot <= h->ctx->ncu && rows <= kGridLevelRows;
    for (int l = l0; l < l1; ++l) {
      P.h_wg0[l] = (int32_t)lev.size();
      const int nw = (wt.h_lev_begin[l + 1] - wt.h_lev_begin[l] + per - 1) / per;
      for (int w = 0; in && w < nw; ++w) lev.push_back(l);
    }
  }
  P.h_wg0[L] = (int32_t)lev.size();
  const size_t n = lev.size();
  if (n == 0) return MSKM_OK;
  D.nslot = h->ctx->ncu;
  Carve cv;
  cv.add(&D.wg0, (size_t)L + 1);
  cv.add(&D.lev, n);
  cv.add(&D.row0, n);
  cv.add(&D.nrow, n);
  cv.add(&D.nhalo, n);
  cv.add(&D.halo, n * kGridLocal);
  cv.add(&D.lidx, n * kGridE * kGridThreads);
  cv.add(&D.stats, 2 * (size_t)L);
  cv.add(&D.slots, 3 * (size_t)D.nslot * kGridSlot);
  MSKM_TRY(cv.alloc(h));
  hipStream_t s = h->ctx->stream;
  MSKM_TRY(upload_async(h, D.wg0, P.h_wg0.data(), P.h_wg0.size() * 4));
  MSKM_TRY(upload_async(h, D.lev, lev.data(), n * 4));
  MSKM_HIP_TRY(hipMemsetAsync(D.stats, 0, 2 * (size_t)L * 4, s));
  D.nwg = (int32_t)n;
  hipLaunchKernelGGL(k_grid_plan, dim3(D.nwg), dim3(kGridThreads), 0, s, D, L, lanes, per, h->d_lev, wt,
                     h->diag.rowptr, h->diag.col);
  std::vector<int32_t> st(2 * (size_t)L);
  MSKM_HIP_TRY(hipMemcpyAsync(st.data(), D.stats, st.size() * 4, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipStreamSynchronize(s));
  P.h_local.assign(st.begin(), st.begin() + L);
  P.h_row.assign(st.begin() + L, st.end());
  return MSKM_OK;
}

// Workgroups of levels lo..hi in this plan, 0 when one of them cannot be
// solved this way (not planned, a row or a halo too long) or they do not fit
// the GPU together.
static int plan_workgroups(const mskm_hier* h, const CgGridPlan& P, int lanes, int lo, int hi) {
  for (int l = lo; l <= hi; ++l)
    if (P.h_wg0[l + 1] == P.h_wg0[l] || P.h_row[l] > lanes * kGridE || P.h_local[l] > kGridLocal) return 0;
  const int n = P.h_wg0[hi + 1] - P.h_wg0[lo];
  return n <= h->ctx->ncu ? n : 0;
}

mskm_status cg_grid_ready(mskm_hier* h, int lo, int hi, bool bj, int* lanes, int most_lanes) {
  *lanes = 0;
  if (h->N >= INT32_MAX) return MSKM_OK;
  for (int l = lo; l <= hi; ++l)
    if (h->h_lev[l].n > kGridLevelRows || h->h_lev[l].n <= 0) return MSKM_OK;
  if (!h->cg_grid) {
    auto* g = new (std::nothrow) CgGrid();
    if (!g) return MSKM_OK;
    h->cg_grid = g;
    h->cg_grid_free = cg_grid_free;
  }
  CgGrid& g = *static_cast<CgGrid*>(h->cg_grid);
  // 256 rows per workgroup, two lanes a row, as long as the workgroups are at
  // most one per CU; else 512 rows, one lane a row. The latter first for levels
  // of up to 512 rows that it solves with one workgroup each: a solve of 342 rows
  // takes 74 us without exchanges, one of 1,366 rows in five workgroups 137 us
  // (k_cg_level_wg, which reads the matrix in every iteration: 259 us for 341).
  int64_t most = 0;
  for (int l = lo; l <= hi; ++l) most = std::max<int64_t>(most, h->h_lev[l].n);
  auto fits = [&](int ln, int* nw) -> mskm_status {
    CgGridPlan& P = g.plan[bj ? 1 : 0][ln == 2 ? 0 : 1];
    if (!P.built) {
      P.built = true;
      const size_t mark = h->allocs.size();
      const mskm_status st = build_plan(h, P, bj, ln);
      if (st == MSKM_ENOMEM) {  // no room for the plan: these levels stay launched
        halloc_undo(h, mark);
        P.h_wg0.assign(h->L + 1, 0);
      } else if (st < 0) {
        return st;
      }
    }
    *nw = plan_workgroups(h, P, ln, lo, hi);
    return MSKM_OK;
  };
  int nw = 0;
  if (most > kGridThreads / 2 && most <= kGridThreads) {
    MSKM_TRY(fits(1, &nw));
    if (nw == hi - lo + 1) {
      *lanes = 1;
      return MSKM_OK;
    }
  }
  for (int ln = most_lanes; ln >= 1 && *lanes == 0; --ln) {
    MSKM_TRY(fits(ln, &nw));
    if (nw > 0) *lanes = ln;
  }
  return MSKM_OK;
}

// -------------------------------------------------------------------- solve

// The row's entry of M^-1 times the block rb, in the block's order as the
// launched kernels add it; every lane of a row has it. The inverse row is in
// registers (N of them, zeros past the block) or read through the caches (N =
// 1). The reads of rb are unconditional, past the block its last entry: under a
// bounds check each was waited for by itself, 1,650 cycles for 16 of them
// instead of 550.
template <int N, typename TX>
__device__ __forceinline__ TX grid_precond(const TX (&iv)[N], const TX* Mi, int bm, const TX* rb) {
  TX a = 0;
  if constexpr (N > 1) {
    const int last = max(bm - 1, 0);
#pragma unroll
    for (int k = 0; k < N; ++k) a += iv[k] * rb[min(k, last)];
  } else {
#pragma unroll 4
    for (int j = 0; j < bm; ++j) a += Mi[j] * rb[j];
  }
  return a;
}

// Right-hand sides of one launch: column col0 + q of b and x (ld words a row)
// in the workgroups q nw, q nw + 1, ... of the launch, each column a system of
// its own. The z buffers hold a level's columns one after the other.
struct GridCols {
  int nw, ld, col0;
  MrState* st;  // [L][ld], instead of the per-level states
};

// Forms of the iteration. kFormPred: textbook with one exchange an iteration
// (FP64 without preconditioner). kFormOneRed: single reduction (FP32, or
// preconditioned). kFormText: textbook (columns of many right-hand sides, FP32 or
// preconditioned).
enum GridForm { kFormPred, kFormOneRed, kFormText };

constexpr int kSums = 4;  // kFormPred: p.q, r.r, q.r, q.q

// G lanes per row, 512 / G rows per workgroup, at most E matrix entries per
// lane. Thread t holds a share of row t / G's entries (grid_entry) and the
// row's part of its block inverse; all G lanes of a row hold its vectors'
// entries. SOLO: every level has one workgroup, which exchanges nothing and takes
// the sums from LDS.
template <int G>
__device__ __forceinline__ int grid_entry(int sum, int k, int g, int len) {  // the lane's k-th entry of the row
  if (G == 2 && sum == kSumHalves) return (k >> 2) * 8 + 4 * g + (k & 3);
  if (G == 2 && sum == kSumRow) {  // the row's first half, the rest
    const int h = (len + 1) / 2;
    return g == 0 ? (k < h ? k : INT32_MAX) : h + k;
  }
  return g + k * G;
}

template <typename TX, bool PC, int G, int E, bool SOLO, int FORM>
__global__ void __launch_bounds__(kGridThreads)
    k_cg_grid(const CgGridDev P, int wgb, int sum, const DevLevel* __restrict__ lev, const int64_t* __restrict__ rp,
              const TX* __restrict__ val, const TX* __restrict__ b, TX* __restrict__ x,
              typename GridWord<TX>::type* z0, typename GridWord<TX>::type* z1, typename GridWord<TX>::type* z2,
              CgLevel* __restrict__ st,
              int32_t* aborted, double rtol2, int maxit, int spin, const PcArgs<TX> pc,
              const GridCols gc) {
  static_assert(FORM != kFormPred || !PC, "z is r");
  using W = typename GridWord<TX>::type;
  constexpr int RW = kGridThreads / G;
  constexpr int kWaves = kGridThreads / kWave;
  constexpr int kH = kGridLocal / kGridThreads;  // halo entries per thread
  constexpr int kParts = kWaves * kWave / 16;    // sums over 16 lanes of a workgroup
  constexpr bool kInvRegs = PC && sizeof(TX) == 4;
  constexpr int kI = kInvRegs ? kBjMax : 1;
  constexpr bool kHaloZ = !SOLO && FORM == kFormPred;
  __shared__ TX pw[kGridLocal];    // what A multiplies (p, or z in kFormOneRed): own rows, then the halo
  __shared__ TX zw[kHaloZ ? kGridLocal : 1];  // z of the halo
  __shared__ int32_t hrow[SOLO ? 1 : kGridLocal];  // rows of the halo
  __shared__ TX rs[PC ? RW : 1];   // what the preconditioner is applied to
  __shared__ double sm[kSums][kParts], sp[kSums];
  __shared__ int bad;
  const int cq = blockIdx.x / gc.nw, col = gc.col0 + cq, wl = blockIdx.x - cq * gc.nw;
  const int wg = wgb + wl, t = threadIdx.x, w = t / kWave, lane = t % kWave;
  const int l = P.lev[wg], w0 = P.wg0[l], nw = P.wg0[l + 1] - w0;
  const int r0 = P.row0[wg], nr = P.nrow[wg], nh = P.nhalo[wg];
  const int i = t / G, g = t % G;
  const bool mine = i < nr, first = mine && g == 0;
  const int64_t row = r0 + (mine ? i : 0);
  const int me = wg - w0, nslot = P.nslot;
  // slot of workgroup wg0 + q of the level in buffer k: slot + (k * nslot + q) * kGridSlot
  uint64_t* const slot = P.slots + (size_t)((int)blockIdx.x - me) * kGridSlot;
  {
    const int64_t off = lev[l].off, zo = off * (gc.ld - 1) + (int64_t)col * lev[l].n;
    z0 += zo;
    z1 += zo;
    z2 += zo;
  }

  // matrix entries (past the row's end: value 0 at position 0)
  TX v[E];
  uint32_t ci[E / 2];
  int len;
  {
    const int64_t s = rp[row], e = rp[row + 1];
    len = mine ? (int)(e - s) : 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int q = grid_entry<G>(sum, k, g, len);
      v[k] = q < len ? val[s + q] : (TX)0;
      const uint32_t c = q < len ? P.lidx[(size_t)wg * kGridE * kGridThreads + q * RW + i] : 0u;
      if (k & 1)
        ci[k / 2] |= c << 16;
      else
        ci[k / 2] = c;
    }
  }
  // entries per lane of the wave's longest row
  int kmax = G == 2 && sum == kSumHalves ? (len + 7) / 8 * 4 : (len + G - 1) / G;
  for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, kWave));
  kmax = __builtin_amdgcn_readfirstlane(kmax);
  // the lane's products added to `from` in NA accumulators, these added in halves
  auto dot = [&](auto na, auto by_four, TX from = 0) {
    constexpr int NA = decltype(na)::value;
    TX a[NA];
#pragma unroll
    for (int u = 0; u < NA; ++u) a[u] = u == 0 ? from : (TX)0;
#pragma unroll
    for (int k0 = 0; k0 < E; k0 += 8)
      if (k0 < kmax) {
#pragma unroll
        for (int k = k0; k < k0 + 8; ++k)
          a[(decltype(by_four)::value ? k >> 2 : k) & (NA - 1)] +=
              v[k] * pw[k & 1 ? ci[k / 2] >> 16 : ci[k / 2] & 0xffffu];
      }
#pragma unroll
    for (int o = NA / 2; o > 0; o /= 2)
#pragma unroll
      for (int u = 0; u < o; ++u) a[u] += a[u + o];
    return a[0];
  };
  using std::bool_constant;
  using std::integral_constant;
  auto product = [&]() -> TX {
    TX q;
    if constexpr (FORM == kFormPred) {
      q = dot(integral_constant<int, 1>{}, bool_constant<false>{});
    } else if constexpr (G == 2) {
      if (sum == kSumLanes4)
        q = dot(integral_constant<int, 2>{}, bool_constant<false>{});
      else if (sum == kSumLanes8)
        q = dot(integral_constant<int, 4>{}, bool_constant<false>{});
      else if (sum == kSumLanes16)
        q = dot(integral_constant<int, 8>{}, bool_constant<false>{});
      else
        q = dot(integral_constant<int, 1>{}, bool_constant<false>{});
      if (sum == kSumRow) {  // the second lane goes on from the first one's sum
        q = dot(integral_constant<int, 1>{}, bool_constant<false>{}, dpp<kDppXor1>(q));
        const TX o = dpp<kDppXor1>(q);
        return g ? q : o;
      }
    } else {
      if (sum == kSumRow)
        q = dot(integral_constant<int, 1>{}, bool_constant<false>{});
      else if (sum == kSumHalves)
        q = dot(integral_constant<int, 2>{}, bool_constant<true>{});
      else
        q = dot(integral_constant<int, 8>{}, bool_constant<false>{});
    }
    return lanes_sum<G>(q);
  };
  // block inverse: the row's entries
  int ba = 0, bm = 0;
  const TX* Mi = nullptr;
  TX iv[kI];
  if constexpr (PC) {
    if (mine) {
      const int32_t bk = pc.of_row[row];
      const int64_t a = pc.start[bk];
      bm = (int)(pc.start[bk + 1] - a);
      ba = (int)(a - r0);
      Mi = pc.inv + pc.off[bk] + (row - a) * bm;
    }
  }
#pragma unroll
  for (int k = 0; k < kI; ++k) iv[k] = kInvRegs && k < bm ? Mi[k] : (TX)0;

  TX xi = 0, ri = mine ? b[row * gc.ld + col] : (TX)0, pi = 0, zi;
  if (t == 0) bad = !SOLO && get(aborted) != 0;  // a launch before this one has given up
  int left = spin;                               // polls that the thread still waits for
  auto precondition = [&] {  // z = M^-1 r
    if constexpr (PC) {
      if (first) rs[i] = ri;
      __syncthreads();
      zi = grid_precond<kI, TX>(iv, Mi, bm, rs + ba);
    } else {
      zi = ri;
    }
  };
  precondition();
  // halo entries t, t + kGridThreads, ... are the thread's; their rows stay in LDS
  for (int q = t; !SOLO && q < nh; q += kGridThreads) hrow[q] = P.halo[(size_t)wg * kGridLocal + q];

  // words of the halo
  W hz[SOLO ? 1 : kH];
  auto halo_words = [&](W* zc) {
#pragma unroll
    for (int q = 0; q < kH; ++q) {
      if (t + q * kGridThreads < nh && hz[q] == GridWord<TX>::empty)
        hz[q] = poll(&zc[hrow[t + q * kGridThreads]], GridWord<TX>::empty, left, &bad);
    }
  };
  auto halo_ask = [&](W* zc) {
#pragma unroll
    for (int q = 0; q < kH; ++q) {
      hz[q] = t + q * kGridThreads < nh ? get(&zc[hrow[t + q * kGridThreads]]) : (W)0;
    }
  };
  static_assert(kParts == 32, "two sums of 16");
  auto total = [&](int k) {
    const double s = lanes_sum<16>(sm[k][lane % kParts]);
    return readlane_f64(s, 0) + readlane_f64(s, 16);
  };
  auto parts = [&](int k, double a) {
    a = lanes_sum<16>(a);
    if (lane % 16 == 0) sm[k][t / 16] = a;
  };
  // wave w's sum over the level's workgroups: word w of buffer m
  auto level_sum = [&](int m, int word) {
    uint64_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      u[k] = lane + k * kWave < nw ? get(slot + (m * nslot + lane + k * kWave) * kGridSlot + word) : 0ull;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (u[k] == kEmptySlot)
        u[k] = poll(slot + (m * nslot + lane + k * kWave) * kGridSlot + word, kEmptySlot, left, &bad);
      s += value_of(u[k]);
    }
    s = wave64_sum(s);
    if (lane == 0) sp[word] = s;
  };
  double bb = 0.0, rr = 0.0;
  int n = 0, capped = 0;
  if constexpr (!SOLO) {
    __syncthreads();
    if (bad) left = 0;
    if (first) put(&z0[row], word_of(zi));
  }

  if constexpr (FORM == kFormPred) {
    // z of the halo (exchange 0), and the first direction
    if constexpr (!SOLO) {
      halo_ask(z0);
      halo_words(z0);
#pragma unroll
      for (int q = 0; q < kH; ++q)
        if (t + q * kGridThreads < nh) pw[nr + t + q * kGridThreads] = zw[t + q * kGridThreads] = value_of(hz[q]);
    }
    pi = zi;
    if (first) pw[i] = pi;
    for (int m = 1;; ++n, m = m == 2 ? 0 : m + 1) {  // m = (n + 1) % 3
      W* const zc = m == 0 ? z0 : m == 1 ? z1 : z2;
      W* const zp = m == 0 ? z2 : m == 1 ? z0 : z1;
      __syncthreads();
      if (bad) break;
      const TX q = product();
      // every earlier store of this workgroup is waited for before it publishes
      if constexpr (!SOLO) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (first) put(&zc[row], word_of(q));
      }
      parts(0, first ? (double)pi * (double)q : 0.0);
      parts(1, first ? (double)ri * (double)ri : 0.0);
      parts(2, first ? (double)q * (double)ri : 0.0);
      parts(3, first ? (double)q * (double)q : 0.0);
      __syncthreads();
      double pq, qr, qq;
      if constexpr (SOLO) {
        pq = total(0);
        rr = total(1);
        qr = total(2);
        qq = total(3);
      } else {
        if (w < 4) {
          const double s = total(w);
          if (lane == 0) put(slot + (m * nslot + me) * kGridSlot + w, word_of(s));
        }
        // the halo and the level's sums, whichever comes first
        halo_ask(zc);
        if (w < 4) level_sum(m, w);
        halo_words(zc);
        __syncthreads();
        if (bad) break;
        pq = sp[0];
        rr = sp[1];
        qr = sp[2];
        qq = sp[3];
      }
      if (n == 0) bb = rr;
      const bool conv = isfinite(rr) && !(rr > rtol2 * bb);
      if (conv || !isfinite(rr) || n >= maxit) {
        capped = conv ? 0 : 1;
        break;
      }
      if (!(pq > 0.0) || !isfinite(pq)) {  // cannot happen for SPD A and p != 0
        capped = 1;
        break;
      }
      // everybody has left the exchange before
      if constexpr (!SOLO) {
        if (first) put(&zp[row], GridWord<TX>::empty);
        if (w < 4 && lane == 0) put(slot + ((m == 0 ? 2 : m - 1) * nslot + me) * kGridSlot + w, kEmptySlot);
      }
      const double alpha = rr / pq;
      const double rrnew = rr - alpha * (2.0 * qr - alpha * qq);  // r.r after the step
      const TX beta = rrnew > 0.0 ? (TX)(rrnew / rr) : (TX)0;
      xi = (TX)((double)xi + alpha * (double)pi);
      ri = (TX)((double)ri - alpha * (double)q);
      pi = ri + beta * pi;
      if (first) pw[i] = pi;
      if constexpr (!SOLO) {
#pragma unroll
        for (int h = 0; h < kH; ++h) {
          if (t + h * kGridThreads < nh) {
            const int at = nr + t + h * kGridThreads;
            const TX zh = (TX)((double)zw[at - nr] - alpha * (double)value_of(hz[h]));
            zw[at - nr] = zh;
            pw[at] = zh + beta * pw[at];
          }
        }
      }
    }
  }

  if constexpr (FORM == kFormOneRed) {
    TX si = 0;  // A p
    CgLevel S{};
    S.rtol2 = rtol2;
    S.maxit = maxit;
    if (first) pw[i] = zi;
    for (int m = 0;; ++n, m = m == 2 ? 0 : m + 1) {  // m = n % 3
      W* const zc = n & 1 ? z1 : z0;
      W* const zn = n & 1 ? z0 : z1;
      if constexpr (!SOLO) {
        halo_ask(zc);
        halo_words(zc);
#pragma unroll
        for (int q = 0; q < kH; ++q)
          if (t + q * kGridThreads < nh) pw[nr + t + q * kGridThreads] = value_of(hz[q]);
      }
      __syncthreads();
      if (bad) break;
      const TX q = product();
      parts(0, first ? (double)zi * (double)q : 0.0);
      parts(1, first ? (double)zi * (double)ri : 0.0);
      if constexpr (PC) parts(2, first ? (double)ri * (double)ri : 0.0);
      constexpr int kWords = PC ? 3 : 2;
      // every earlier store of this workgroup is waited for before it publishes
      if constexpr (!SOLO) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      double delta, gamma;
      if constexpr (SOLO) {
        delta = total(0);
        gamma = total(1);
        rr = PC ? total(2) : gamma;
      } else {
        if (w < kWords) {
          const double s = total(w);
          if (lane == 0) put(slot + (m * nslot + me) * kGridSlot + w, word_of(s));
          level_sum(m, w);
        }
        __syncthreads();
        if (bad) break;
        delta = sp[0];
        gamma = sp[1];
        rr = PC ? sp[2] : gamma;
      }
      if (n == 0) S.bb = bb = rr;
      if (!cg1_decide(S, gamma, delta, rr)) {
        capped = S.capped;
        break;
      }
      if constexpr (!SOLO) {
        // everybody has this iteration's z, and has left the sums before
        if (first) put(&zc[row], GridWord<TX>::empty);
        if (w < kWords && lane == 0) put(slot + ((m == 0 ? 2 : m - 1) * nslot + me) * kGridSlot + w, kEmptySlot);
      }
      const TX beta = (TX)S.beta;
      pi = zi + beta * pi;
      si = q + beta * si;
      xi = (TX)((double)xi + S.alpha * (double)pi);
      ri = (TX)((double)ri - S.alpha * (double)si);
      precondition();
      if (first) {
        pw[i] = zi;
        if constexpr (!SOLO) put(&zn[row], word_of(zi));
      }
    }
  }

  if constexpr (FORM == kFormText) {
    if (first) pw[i] = (TX)0;
    for (int q = t; !SOLO && q < nh; q += kGridThreads) pw[nr + q] = (TX)0;
    double rzold = 0.0;
    for (;; ++n) {
      W* const zc = n & 1 ? z1 : z0;
      W* const zn = n & 1 ? z0 : z1;
      const int m = n & 1;
      // exchange A: r.r, r.z and z of the halo
      parts(0, first ? (double)ri * (double)ri : 0.0);
      parts(1, first ? (double)ri * (double)zi : 0.0);
      __syncthreads();
      double rz;
      if constexpr (SOLO) {
        rr = total(0);
        rz = total(1);
      } else {
        if (w < 2) {
          const double s = total(w);
          if (lane == 0) put(slot + (m * nslot + me) * kGridSlot + w, word_of(s));
        }
        halo_ask(zc);
        if (w < 2) level_sum(m, w);
        halo_words(zc);
        __syncthreads();
        if (bad) break;
        rr = sp[0];
        rz = sp[1];
      }
      if (n == 0) bb = rr;
      const bool conv = isfinite(rr) && !(rr > rtol2 * bb);
      if (conv || !isfinite(rr) || (n > 0 && !isfinite(rz)) || n >= maxit) {
        capped = conv ? 0 : 1;
        break;
      }
      // everybody has left the sum p.q before
      if constexpr (!SOLO)
        if (n > 0 && t == 0) put(slot + ((m ^ 1) * nslot + me) * kGridSlot + 2, kEmptySlot);
      const TX beta = n == 0 ? (TX)0 : (TX)(rz / rzold);
      rzold = rz;
      pi = zi + beta * pi;
      if (first) pw[i] = pi;
      if constexpr (!SOLO) {
#pragma unroll
        for (int h = 0; h < kH; ++h)
          if (t + h * kGridThreads < nh) {
            const int at = nr + t + h * kGridThreads;
            pw[at] = value_of(hz[h]) + beta * pw[at];
          }
      }
      __syncthreads();
      const TX q = product();
      // exchange B: p.q (every earlier store of this workgroup is waited for first)
      parts(2, first ? (double)pi * (double)q : 0.0);
      if constexpr (!SOLO) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      double pq;
      if constexpr (SOLO) {
        pq = total(2);
      } else {
        if (w == 0) {
          const double s = total(2);
          if (lane == 0) put(slot + (m * nslot + me) * kGridSlot + 2, word_of(s));
          level_sum(m, 2);
        }
        __syncthreads();
        if (bad) break;
        pq = sp[2];
      }
      if (!(pq > 0.0) || !isfinite(pq)) {  // cannot happen for SPD A and p != 0
        capped = !(rr <= rtol2 * bb);
        break;
      }
      if constexpr (!SOLO) {  // everybody has this iteration's z and sums
        if (first) put(&zc[row], GridWord<TX>::empty);
        if (w < 2 && lane == 0) put(slot + (m * nslot + me) * kGridSlot + w, kEmptySlot);
      }
      const double alpha = rz / pq;
      xi = (TX)((double)xi + alpha * (double)pi);
      ri = (TX)((double)ri - alpha * (double)q);
      precondition();
      if constexpr (!SOLO)
        if (first) put(&zn[row], word_of(zi));
    }
  }

  if (bad) {
    if (t == 0) atomicOr(aborted, 1);
    return;
  }
  if (first) x[row * gc.ld + col] = xi;
  if (t == 0 && wg == w0 && gc.st) {
    MrState* const o = gc.st + (size_t)l * gc.ld + col;
    o->iters = n;
    o->done = 1;
    o->capped = capped;
  } else if (t == 0 && wg == w0) {
    CgLevel* const o = st + l;
    o->rtol2 = rtol2;
    o->bb = bb;
    o->rr = rr;
    o->maxit = maxit;
    o->on = 1;
    o->iters = n;
    o->done = 1;
    o->capped = capped;
    o->fallback = 0;
  }
}

// `last` is the context that launched a persistent kernel last.
namespace {
struct GridOrder {
  std::mutex mu;
  mskm_ctx* last = nullptr;
};
constexpr int kGridDevices = 64;
GridOrder g_order[kGridDevices];
}  // namespace

int launched_sum(const mskm_hier* h, int lo, int hi, bool fp32) {
  int64_t most = 0;
  for (int l = lo; l <= hi; ++l) most = std::max<int64_t>(most, h->h_lev[l].n);
  if (most <= kWgSolveRows) return most <= 64 ? kSumLanes16 : most <= 256 ? kSumLanes4 : kSumLanes8;
  const int code = h->spmv_g[MSKM_OP_DIAG][fp32 ? 1 : 0];
  if (code == kSellCode && h->sell.col16)
    return h->h_off[hi + 1] - h->h_off[lo] <= kSplitProductRows ? kSumHalves : kSumRow;
  if (code == kSellCode || code == kSell32Code) return kSumRow;
  return kSumLanes8;
}

void cg_grid_forget(mskm_ctx* c) {
  if (c->device < 0 || c->device >= kGridDevices) return;
  GridOrder& o = g_order[c->device];
  std::lock_guard<std::mutex> lock(o.mu);
  if (o.last == c) o.last = nullptr;
}

mskm_status cg_grid_in_turn(mskm_ctx* c, const std::function<void()>& launch) {
  if (c->device < 0 || c->device >= kGridDevices) return fail(MSKM_ELIMIT, "device index beyond 63");
  GridOrder& o = g_order[c->device];
  std::lock_guard<std::mutex> lock(o.mu);
  if (o.last && o.last != c) MSKM_HIP_TRY(hipStreamWaitEvent(c->stream, o.last->ev_grid, 0));
  launch();
  MSKM_HIP_TRY(hipGetLastError());
  MSKM_HIP_TRY(hipEventRecord(c->ev_grid, c->stream));
  o.last = c;
  return MSKM_OK;
}

void cg_grid_set_spin(mskm_ctx* c, int spin) {
  c->grid_spin = spin;
  c->grid_rest = 0;
}

extern "C" int64_t mskm_test_given_up(const mskm_ctx* c) { return c->given_up; }

extern "C" void mskm_test_spin(mskm_ctx* c, int spin) { cg_grid_set_spin(c, spin); }

extern "C" void mskm_test_limits(mskm_ctx* c, uint64_t hier_bytes, uint64_t scratch_bytes) {
  c->limit_hier = hier_bytes;
  c->limit_scratch = scratch_bytes;
}

// Empties z0, z1 on the rows [r0, r0 + n) and every slot of the plan.
template <typename TX>
__global__ void __launch_bounds__(kBlock)
    k_grid_empty(typename GridWord<TX>::type* __restrict__ z0, typename GridWord<TX>::type* __restrict__ z1,
                 typename GridWord<TX>::type* __restrict__ z2, int64_t r0, int64_t n, uint64_t* __restrict__ slots,
                 int64_t ns) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) {
    z0[r0 + i] = GridWord<TX>::empty;
    z1[r0 + i] = GridWord<TX>::empty;
    if (z2) z2[r0 + i] = GridWord<TX>::empty;
  }
  if (i < ns) slots[i] = kEmptySlot;
}

template <typename TX>
void grid_empty(hipStream_t s, TX* z0, TX* z1, TX* z2, int64_t r0, int64_t n, uint64_t* slots, int64_t ns) {
  using W = typename GridWord<TX>::type;
  hipLaunchKernelGGL(k_grid_empty<TX>, dim3((unsigned)((std::max(n, ns) + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                     (W*)z0, (W*)z1, (W*)z2, r0, n, slots, ns);
}
template void grid_empty<float>(hipStream_t, float*, float*, float*, int64_t, int64_t, uint64_t*, int64_t);
template void grid_empty<double>(hipStream_t, double*, double*, double*, int64_t, int64_t, uint64_t*, int64_t);

// The order that a form with `lanes` lanes a row has for these levels.
static int grid_sum(const mskm_hier* h, int lo, int hi, int lanes, bool fp32) {
  const int sum = launched_sum(h, lo, hi, fp32);
  if (lanes == 2) return sum;
  return sum == kSumRow || sum == kSumHalves ? sum : kSumLanes8;
}

// The kernel for levels lo..hi with the columns of gc, `cols` of them.
template <typename TX, int FORM>
static void grid_launch(mskm_hier* h, int lo, int hi, bool bj, int lanes, const TX* val, const TX* b, TX* x, TX* z0,
                        TX* z1, TX* z2, CgLevel* st, int32_t* aborted, double rtol2, int maxit, const PcArgs<TX>& pc,
                        const GridCols& gc, int cols) {
  using W = typename GridWord<TX>::type;
  const CgGridPlan& P = static_cast<CgGrid*>(h->cg_grid)->plan[bj ? 1 : 0][lanes == 2 ? 0 : 1];
  const int w0 = P.h_wg0[lo];
  const bool solo = gc.nw == hi - lo + 1;
  const int sum = FORM == kFormOneRed ? grid_sum(h, lo, hi, lanes, sizeof(TX) == 4)
                  : FORM == kFormText ? kSumRow
                                      : kSumLanes8;  // kFormPred: any
  int longest = 0;
  for (int l = lo; l <= hi; ++l) longest = std::max(longest, P.h_row[l]);
#define MSKM_GRID_LAUNCH(PCF, GG, EE, SS)                                                                           \
  hipLaunchKernelGGL((k_cg_grid<TX, PCF, GG, EE, SS, FORM>), dim3((unsigned)gc.nw * cols), dim3(kGridThreads), 0,   \
                     h->ctx->stream, P.d, w0, sum, h->d_lev, h->diag.rowptr, val, b, x, (W*)z0, (W*)z1, (W*)z2, st, \
                     aborted, rtol2, maxit, h->ctx->grid_spin, pc, gc)
#define MSKM_GRID_SOLO(PCF, GG, EE)          \
  do {                                       \
    if (solo)                                \
      MSKM_GRID_LAUNCH(PCF, GG, EE, true);   \
    else                                     \
      MSKM_GRID_LAUNCH(PCF, GG, EE, false);  \
  } while (0)
#define MSKM_GRID_FORM(GG, EE)                                  \
  do {                                                          \
    if constexpr (FORM != kFormPred) {                          \
      if (bj) {                                                 \
        MSKM_GRID_SOLO(true, GG, EE);                           \
        return;                                                 \
      }                                                         \
    }                                                           \
    if constexpr (FORM == kFormPred || sizeof(TX) == 4)         \
      MSKM_GRID_SOLO(false, GG, EE);                            \
  } while (0)
  if (lanes == 2) {
    if (longest <= 64)
      MSKM_GRID_FORM(2, 32);
    else
      MSKM_GRID_FORM(2, 64);
    return;
  }
  if (longest <= 48)
    MSKM_GRID_FORM(1, 48);
  else
    MSKM_GRID_FORM(1, 64);
#undef MSKM_GRID_FORM
#undef MSKM_GRID_SOLO
#undef MSKM_GRID_LAUNCH
}

template <typename TX>
mskm_status cg_grid_launch(mskm_hier* h, int lo, int hi, bool bj, int lanes, const TX* val, const TX* b, TX* x,
                           TX* z0, TX* z1, TX* z2, CgLevel* st, int32_t* aborted, double rtol2, int maxit,
                           const PcArgs<TX>& pc) {
  const CgGridPlan& P = static_cast<CgGrid*>(h->cg_grid)->plan[bj ? 1 : 0][lanes == 2 ? 0 : 1];
  const int nw = P.h_wg0[hi + 1] - P.h_wg0[lo];
  const GridCols gc{nw, 1, 0, nullptr};
  // one workgroup per level: no words to empty, no launch to wait for
  const bool solo = nw == hi - lo + 1;
  if (!solo) {
    const int64_t r0 = h->h_off[lo], n = h->h_off[hi + 1] - r0;
    grid_empty<TX>(h->ctx->stream, z0, z1, z2, r0, n, P.d.slots, (int64_t)3 * P.d.nslot * kGridSlot);
  }
  auto launch = [&] {
    if constexpr (sizeof(TX) == 8)
      if (!bj) {
        grid_launch<TX, kFormPred>(h, lo, hi, bj, lanes, val, b, x, z0, z1, z2, st, aborted, rtol2, maxit, pc, gc, 1);
        return;
      }
    grid_launch<TX, kFormOneRed>(h, lo, hi, bj, lanes, val, b, x, z0, z1, z2, st, aborted, rtol2, maxit, pc, gc, 1);
  };
  if (!solo) return cg_grid_in_turn(h->ctx, launch);
  launch();
  MSKM_HIP_TRY(hipGetLastError());
  return MSKM_OK;
}
template mskm_status cg_grid_launch<float>(mskm_hier*, int, int, bool, int, const float*, const float*, float*, float*,
                                           float*, float*, CgLevel*, int32_t*, double, int, const PcArgs<float>&);
template mskm_status cg_grid_launch<double>(mskm_hier*, int, int, bool, int, const double*, const double*, double*,
                                            double*, double*, double*, CgLevel*, int32_t*, double, int,
                                            const PcArgs<double>&);

// Launches one after the other that the columns of a level may take: an
// iteration takes 4-5 us in each, launched for all columns at once 25-35 us.
// Measured for 21 right-hand sides: 4,096 rows in one launch 0.25 ms, 16,384 rows in
// four 1.4 ms; three solves of a hierarchy of 87,000 points and their residuals 19.9 ms
// (31.0 ms with every level launched).
constexpr int kGridRounds = 4;

// Columns past the right-hand sides: zero solutions, nothing done.
template <typename TX>
__global__ void __launch_bounds__(kBlock)
    k_grid_pad(TX* __restrict__ x, MrState* __restrict__ st, int64_t r0, int64_t n, int lev0, int nlev, int nrhs, int R) {
  const int w = R - nrhs;
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e < n * w) x[(r0 + e / w) * R + nrhs + e % w] = (TX)0;
  if (e < (int64_t)nlev * w) {
    MrState& S = st[(lev0 + e / w) * R + nrhs + e % w];
    S.iters = S.capped = 0;
    S.done = 1;
  }
}

template <typename TX>
mskm_status cg_grid_columns(mskm_hier* h, int lo, int hi, bool bj, const TX* val, const TX* b, TX* x, TX* z0, TX* z1,
                            TX* z2, int nrhs, int R, MrState* st, int32_t* aborted, double rtol2, int maxit, const PcArgs<TX>& pc,
                            int* how) {
  *how = 0;
  // the textbook form as the launched kernels have it, whose rows are added in
  // entry order: one lane a row, or two, one after the other, for rows past 64
  // entries; FP64 without preconditioner as in cg_grid_launch
  const bool text = bj || sizeof(TX) == 4;
  int lanes = 0;
  MSKM_TRY(cg_grid_ready(h, lo, hi, bj, &lanes, text ? 1 : 2));
  if (text && lanes == 0) MSKM_TRY(cg_grid_ready(h, lo, hi, bj, &lanes));
  if (lanes == 0) return MSKM_OK;
  const CgGridPlan& P = static_cast<CgGrid*>(h->cg_grid)->plan[bj ? 1 : 0][lanes == 2 ? 0 : 1];
  const int nw = P.h_wg0[hi + 1] - P.h_wg0[lo], ncu = h->ctx->ncu;
  const bool solo = nw == hi - lo + 1;
  const int per = ncu / nw;  // columns of a launch; alone on their level, workgroups may queue
  if ((nrhs + per - 1) / per > kGridRounds) return MSKM_OK;
  const int64_t r0 = h->h_off[lo], n = h->h_off[hi + 1] - r0;
  if (nrhs < R)
    hipLaunchKernelGGL(k_grid_pad<TX>, dim3(mr_nblk(n * (R - nrhs), kBlock)), dim3(kBlock), 0, h->ctx->stream, x, st, r0,
                       n, lo, hi - lo + 1, nrhs, R);
  auto launch = [&](const GridCols& gc, int cols) {
    if constexpr (sizeof(TX) == 8)
      if (!text) {
        grid_launch<TX, kFormPred>(h, lo, hi, bj, lanes, val, b, x, z0, z1, z2, nullptr, aborted, rtol2, maxit, pc, gc,
                                   cols);
        return;
      }
    grid_launch<TX, kFormText>(h, lo, hi, bj, lanes, val, b, x, z0, z1, z2, nullptr, aborted, rtol2, maxit, pc, gc,
                               cols);
  };
  if (solo) {
    launch(GridCols{nw, R, 0, st}, nrhs);
    MSKM_HIP_TRY(hipGetLastError());
    *how = 1;
    return MSKM_OK;
  }
  for (int c0 = 0; c0 < nrhs; c0 += per) {
    grid_empty<TX>(h->ctx->stream, z0, z1, z2, r0 * R, c0 == 0 ? n * R : 0, P.d.slots, (int64_t)3 * P.d.nslot * kGridSlot);
    const GridCols gc{nw, R, c0, st};
    MSKM_TRY(cg_grid_in_turn(h->ctx, [&] { launch(gc, std::min(per, nrhs - c0)); }));
  }
  *how = 2;
  return MSKM_OK;
}
template mskm_status cg_grid_columns<float>(mskm_hier*, int, int, bool, const float*, const float*, float*, float*,
                                            float*, float*, int, int, MrState*, int32_t*, double, int, const PcArgs<float>&, int*);
template mskm_status cg_grid_columns<double>(mskm_hier*, int, int, bool, const double*, const double*, double*,
                                             double*, double*, double*, int, int, MrState*, int32_t*, double, int,
                                             const PcArgs<double>&, int*);

}  // namespace mskm
