// FP32 CG on a depth of large levels in one launch (x0 = 0): the single-reduction
// form and the exchange of cg_grid.hip (kFormOneRed; its buffers and their reuse) for
// levels whose matrix does not fit the registers.
//
// One workgroup per CU owns up to 1,504 consecutive rows (three slots of 512). x,
// r, z on the columns its rows reach, the place of every row's block
// inverse and, where they fit, the inverses stay in LDS over the whole solve, the
// direction and A p in registers; the matrix of the first RES slots stays in
// registers, that of the rest in the LDS left over and, past it, is read once an
// iteration from L2.
//
// Bound: the sums' exchange between 256 workgroups (2 us) and the halo's z an
// iteration, and the LDS reads of the product, one word an entry. A solve of
// 262,144 rows with 45 entries a row in 55 iterations takes 0.87 ms (launched: 27
// us an iteration, 1.5 ms; the textbook form, which waits for two sums, 1.02 ms);
// a 3-D one of up to 100 entries a row, one resident slot, 3.3 ms (4.2 ms).
//
// The window is kept in runs of 64 columns, and only the runs that are used: in
// Morton order a workgroup's columns span up to 60,000 places of which it uses
// 2,500. Held whole, the window took the LDS of the inverses, and one of more
// than 24,576 columns left the level to the launched kernels.
//
// More rows per workgroup lose: 1,048,576 rows (4,096 a workgroup, seven of nine
// slots read every iteration by eight waves) took 137 us an iteration against
// 90 us launched, so such a level stays launched.
//
// The matrix is stored for this kernel in slices of 64 rows, as the sliced copy
// of the diagonal blocks is, but by workgroup and wave: slice (workgroup, wave w,
// slot j) holds rows 512 j + 64 w .. of the workgroup.
#include <algorithm>
#include <new>
#include <vector>

#include "cg_grid.h"
#include "cg_state.h"
#include "device_common.h"

namespace mskm {

constexpr int kStreamWaves = kGridThreads / kWave;
constexpr int kStreamWindow = 65536;                    // columns from the first to the last of a workgroup (at most)
constexpr int kStreamChunks = kStreamWindow / kWave;    // in runs of 64
constexpr int kStreamFlagWords = kStreamChunks / 32;
constexpr int kStreamRt = 3;                            // slots of 512 rows of a workgroup
constexpr int kStreamHalo = 4;                          // halo runs a wave asks for at a time

struct CgStreamDev {
  int32_t nwg = 0;                // workgroups
  int32_t* lev = nullptr;         // [nwg]
  int32_t* part = nullptr;        // [nwg] its number within its level
  int32_t* wg0 = nullptr;         // [nwg] first workgroup of its level
  int32_t* nw = nullptr;          // [nwg] workgroups of its level
  int32_t* row0 = nullptr;        // [nwg] first row
  int32_t* nrow = nullptr;        // [nwg]
  int32_t* wbase = nullptr;       // [nwg] first column of the window
  int32_t* wlen = nullptr;        // [nwg] its length: columns, of which the runs that are used are kept
  int64_t* size = nullptr;        // [nwg 8 kStreamRt + 1] entries of each slice
  int64_t* soff = nullptr;        // [nwg 8 kStreamRt + 1] their scan
  uint32_t* flags = nullptr;      // [nwg][kStreamFlagWords] runs of the window that hold columns or own rows
  uint16_t* rank = nullptr;       // [nwg][kStreamChunks] a run's place among them
  int32_t* nchunk = nullptr;      // [nwg] runs that lie (partly) outside the own rows
  uint32_t* chunk = nullptr;      // [nwg][kStreamChunks] those: place << 16 | run
  float* val = nullptr;           // entries in groups of four per row, as in the sliced copy
  uint16_t* idx = nullptr;        // position of each entry's column in the kept runs
  uint64_t* slots = nullptr;      // [3][nwg][kGridSlot]
  int32_t* stats = nullptr;       // [6] widest slice, longest window, most rows, inverse words, kept runs, halo runs
};

struct CgStreamPlan {
  bool built = false, ok = false;
  int32_t width = 0, window = 0, rows = 0;
  int32_t inv = 0;     // words of LDS for the block inverses (0: read from memory)
  int32_t chunks = 0;  // most halo runs
  int32_t nl = 0;      // streamed slices kept in LDS
  CgStreamDev d;
};

struct CgStream {
  std::vector<CgStreamPlan> depth[2];  // [block-Jacobi][depth]
};

// Bytes of LDS: the kept runs of the window, r, x and block places of the rows,
// the block inverses, the slices kept there, the halo runs.
static size_t stream_lds(const CgStreamPlan& P) {
  const size_t w = (size_t)(P.window + 3) / 4 * 4, r = (size_t)(P.rows + 3) / 4 * 4, c = (size_t)(P.chunks + 3) / 4 * 4;
  return 4 * w + 16 * r + 4 * (size_t)P.inv + 6 * (size_t)P.nl * P.width * kWave + 4 * c;
}
constexpr size_t kStreamLds = 159 * 1024;  // of 160 KiB, the rest for the reductions

static void cg_stream_free(void* p) { delete static_cast<CgStream*>(p); }

// --------------------------------------------------------------------- plan

// Rows of the workgroups: workgroup q of a level starts at the preconditioner
// block that holds the level's row q T (without blocks, at that row).
__global__ void __launch_bounds__(kBlock)
    k_stream_rows(const CgStreamDev P, int T, const DevLevel* __restrict__ lev, const int64_t* __restrict__ start,
                  const int32_t* __restrict__ of_row) {
  const int w = blockIdx.x * kBlock + threadIdx.x;
  if (w >= P.nwg) return;
  const DevLevel& Lv = lev[P.lev[w]];
  auto at = [&](int q) -> int64_t {
    if (q >= P.nw[w]) return Lv.off + Lv.n;
    const int64_t r = Lv.off + (int64_t)q * T;
    return of_row ? start[of_row[r]] : r;
  };
  const int64_t a = at(P.part[w]), e = at(P.part[w] + 1);
  P.row0[w] = (int32_t)a;
  P.nrow[w] = (int32_t)(e - a);
}

// Window and slice sizes of a workgroup (one block of 512 threads each).
__global__ void __launch_bounds__(kGridThreads)
    k_stream_scan(const CgStreamDev P, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                  const int32_t* __restrict__ of_row, const int64_t* __restrict__ off) {
  __shared__ int lo, hi, widest;
  const int wg = blockIdx.x, t = threadIdx.x, w = t / kWave, lane = t % kWave;
  const int64_t r0 = P.row0[wg];
  const int nr = P.nrow[wg];
  if (t == 0) {
    lo = INT32_MAX;
    hi = widest = 0;
  }
  __syncthreads();
  int mn = INT32_MAX, mx = 0, wide = 0;
  for (int j = 0; j < kStreamRt; ++j) {
    const int i = j * kGridThreads + t;
    int len = 0;
    if (i < nr) {
      const int64_t s = rp[r0 + i], e = rp[r0 + i + 1];
      len = (int)min<int64_t>(e - s, 1 << 20);
      if (len > 0) {  // columns ascend within a row
        mn = min(mn, col[s]);
        mx = max(mx, col[e - 1]);
      }
    }
    for (int o = 32; o > 0; o >>= 1) len = max(len, __shfl_xor(len, o, kWave));
    len = (len + 3) / 4 * 4;
    if (lane == 0) P.size[((int64_t)wg * kStreamWaves + w) * kStreamRt + j] = (int64_t)len * kWave;
    wide = max(wide, len);
  }
  atomicMin(&lo, mn);
  atomicMax(&hi, mx);
  atomicMax(&widest, wide);
  __syncthreads();
  if (t == 0) {
    const int base = min(lo, (int)r0), len = max(hi + 1, (int)r0 + nr) - base;
    P.wbase[wg] = base;
    P.wlen[wg] = len;
    atomicMax(&P.stats[0], widest);
    atomicMax(&P.stats[1], len);
    atomicMax(&P.stats[2], nr);
    if (of_row) atomicMax(&P.stats[3], (int)(off[of_row[r0 + nr - 1] + 1] - off[of_row[r0]]));
    if (wg == 0) P.size[(int64_t)P.nwg * kStreamRt * kStreamWaves] = 0;
  }
}

// Marks the runs that hold columns of one slice's rows, or the rows themselves.
__global__ void __launch_bounds__(kBlock)
    k_stream_flags(const CgStreamDev P, const int64_t* __restrict__ rp, const int32_t* __restrict__ col) {
  __shared__ uint32_t fl[kStreamFlagWords];
  const int wg = blockIdx.x / (kStreamRt * kStreamWaves), js = blockIdx.x % (kStreamRt * kStreamWaves);
  const int i0 = js * kWave, i1 = min(i0 + kWave, P.nrow[wg]);
  if (i0 >= i1) return;
  for (int k = threadIdx.x; k < kStreamFlagWords; k += kBlock) fl[k] = 0;
  __syncthreads();
  const int base = P.wbase[wg];
  const int64_t r0 = (int64_t)P.row0[wg] + i0;
  const int64_t e = rp[r0 + i1 - i0];
  for (int64_t k = rp[r0] + threadIdx.x; k < e; k += kBlock) {
    const int c = col[k] - base;
    atomicOr(&fl[c >> 11], 1u << ((c >> 6) & 31));
  }
  if ((int)threadIdx.x < i1 - i0) {
    const int c = (int)(r0 - base) + (int)threadIdx.x;
    atomicOr(&fl[c >> 11], 1u << ((c >> 6) & 31));
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kStreamFlagWords; k += kBlock)
    if (fl[k]) atomicOr(&P.flags[(int64_t)wg * kStreamFlagWords + k], fl[k]);
}

// Places of the marked runs, and the list of those (partly) outside the
// workgroup's rows, ascending.
__global__ void __launch_bounds__(kWave) k_stream_chunks(const CgStreamDev P) {
  const int wg = blockIdx.x, lane = threadIdx.x;
  const int own0 = P.row0[wg] - P.wbase[wg], own1 = own0 + P.nrow[wg];
  int n = 0, nh = 0;
  for (int c0 = 0; c0 < kStreamChunks; c0 += kWave) {
    const int c = c0 + lane;
    const bool on = P.flags[(int64_t)wg * kStreamFlagWords + (c >> 5)] >> (c & 31) & 1u;
    const bool halo = on && (c * kWave < own0 || (c + 1) * kWave > own1);
    const uint64_t m = __ballot(on), mh = __ballot(halo), below = (1ull << lane) - 1ull;
    const int rk = n + __popcll(m & below);
    P.rank[(int64_t)wg * kStreamChunks + c] = (uint16_t)rk;
    if (halo) P.chunk[(int64_t)wg * kStreamChunks + nh + __popcll(mh & below)] = (uint32_t)rk << 16 | (uint32_t)c;
    n += __popcll(m);
    nh += __popcll(mh);
  }
  if (lane == 0) {
    P.nchunk[wg] = nh;
    atomicMax(&P.stats[4], n);
    atomicMax(&P.stats[5], nh);
  }
}

// Entries of one slice (blocks of 256 threads): wave v takes rows 16 v .. 16 v +
// 15, lane = 4 * row + group reads four consecutive entries of a row (64
// contiguous bytes per row and step) and writes them as one group.
__global__ void __launch_bounds__(kBlock)
    k_stream_fill(const CgStreamDev P, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                  const float* __restrict__ val) {
  const int64_t s = blockIdx.x;
  const int64_t o0 = P.soff[s], o1 = P.soff[s + 1];
  if (o0 == o1) return;
  const int wg = (int)(s / (kStreamRt * kStreamWaves)), ws = (int)(s % (kStreamRt * kStreamWaves));
  const int js = ws % kStreamRt * kStreamWaves + ws / kStreamRt;  // 64-row run of the workgroup
  const int lane = threadIdx.x % kWave, t = 16 * (threadIdx.x / kWave) + lane / 4, g = lane % 4;
  const int i = js * kWave + t, base = P.wbase[wg];
  const uint16_t* const rank = P.rank + (int64_t)wg * kStreamChunks;
  const int width = (int)((o1 - o0) / kWave);
  const int64_t row = (int64_t)P.row0[wg] + i;
  const bool mine = i < P.nrow[wg];
  const int64_t b = mine ? rp[row] : 0, e = mine ? rp[row + 1] : 0;
  for (int k0 = 4 * g; k0 < width; k0 += 16) {
    float v[4];
    uint16_t x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t q = b + k0 + u;
      const bool in = q < e;
      const int c = in ? col[q] - base : mine ? (int)(row - base) : 0;
      v[u] = in ? val[q] : 0.0f;
      x[u] = in || mine ? (uint16_t)(rank[c >> 6] * kWave + (c & 63)) : (uint16_t)0;
    }
    const int64_t at = o0 + (int64_t)(k0 / 4) * 4 * kWave + 4 * t;
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef unsigned short u4 __attribute__((ext_vector_type(4)));
    *reinterpret_cast<f4*>(P.val + at) = f4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<u4*>(P.idx + at) = u4{x[0], x[1], x[2], x[3]};
  }
}

// Slots whose entries stay in registers, by the widest slice.
static int stream_resident(int width) { return width <= 48 ? 2 : width <= 96 ? 1 : 0; }

namespace {
mskm_status build_stream(mskm_hier* h, CgStreamPlan& P, int depth, bool bj) {
  const int l0 = h->h_depth_begin[depth], l1 = h->h_depth_begin[depth + 1], ncu = h->ctx->ncu;
  CgStreamDev& D = P.d;
  int64_t n = 0;
  for (int l = l0; l < l1; ++l) n += h->h_lev[l].n;
  // the fewest rows per workgroup with which the depth's levels fit the CUs
  const int64_t most = (int64_t)kGridThreads * kStreamRt - kBjMax;
  if (n > most * ncu || l1 - l0 > ncu) return MSKM_OK;
  auto wgs = [&](int64_t T) {
    int64_t w = 0;
    for (int l = l0; l < l1; ++l) w += (h->h_lev[l].n + T - 1) / T;
    return w;
  };
  int64_t a = std::max<int64_t>(1, n / ncu), e = most;
  if (wgs(e) > ncu) return MSKM_OK;
  while (a < e) {
    const int64_t m = (a + e) / 2;
    if (wgs(m) <= ncu)
      e = m;
    else
      a = m + 1;
  }
  const int64_t T = std::max<int64_t>(a, 2 * kBjMax);
  std::vector<int32_t> tab[4];  // lev, part, wg0, nw
  for (int l = l0; l < l1; ++l) {
    const int nw = (int)((h->h_lev[l].n + T - 1) / T), w0 = (int)tab[0].size();
    for (int q = 0; q < nw; ++q) {
      tab[0].push_back(l);
      tab[1].push_back(q);
      tab[2].push_back(w0);
      tab[3].push_back(nw);
    }
  }
  const size_t nwg = tab[0].size(), ns = nwg * kStreamRt * kStreamWaves;
  if (nwg == 0) return MSKM_OK;
  hipStream_t s = h->ctx->stream;
  int32_t** dst[4] = {&D.lev, &D.part, &D.wg0, &D.nw};
  Carve cv;
  for (int32_t** v : {&D.lev, &D.part, &D.wg0, &D.nw, &D.row0, &D.nrow, &D.wbase, &D.wlen, &D.nchunk}) cv.add(v, nwg);
  cv.add(&D.size, ns + 1);
  cv.add(&D.soff, ns + 1);
  cv.add(&D.flags, nwg * kStreamFlagWords);
  cv.add(&D.chunk, nwg * kStreamChunks);
  cv.add(&D.rank, nwg * kStreamChunks);
  cv.add(&D.slots, 3 * nwg * kGridSlot);
  cv.add(&D.stats, 6);
  MSKM_TRY(cv.alloc(h));
  for (int k = 0; k < 4; ++k) MSKM_TRY(upload_async(h, *dst[k], tab[k].data(), nwg * 4));
  D.nwg = (int32_t)nwg;
  void* part = nullptr;
  const size_t part_bytes = (size_t)scan_parts((int64_t)ns + 1) * 8;
  MSKM_TRY(ctx_alloc(h->ctx, part_bytes, &part));
  CtxScratch scratch{h->ctx, part, part_bytes};
  MSKM_HIP_TRY(hipMemsetAsync(D.stats, 0, 24, s));
  MSKM_HIP_TRY(hipMemsetAsync(D.flags, 0, nwg * kStreamFlagWords * 4, s));
  hipLaunchKernelGGL(k_stream_rows, dim3((unsigned)((nwg + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, D, (int)T,
                     h->d_lev, bj ? h->bj.start : nullptr, bj ? h->bj.of_row : nullptr);
  hipLaunchKernelGGL(k_stream_scan, dim3(D.nwg), dim3(kGridThreads), 0, s, D, h->diag.rowptr, h->diag.col,
                     bj ? h->bj.of_row : nullptr, bj ? h->bj.off : nullptr);
  MSKM_TRY(exclusive_scan_i64(s, D.size, D.soff, (int64_t)ns + 1, static_cast<int64_t*>(part)));
  int32_t st[6] = {};
  int64_t total = 0;
  MSKM_HIP_TRY(hipMemcpyAsync(st, D.stats, 16, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipMemcpyAsync(&total, D.soff + ns, 8, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipStreamSynchronize(s));
  if (st[1] > kStreamWindow || st[2] > kStreamRt * kGridThreads) return MSKM_OK;
  hipLaunchKernelGGL(k_stream_flags, dim3((unsigned)ns), dim3(kBlock), 0, s, D, h->diag.rowptr, h->diag.col);
  hipLaunchKernelGGL(k_stream_chunks, dim3(D.nwg), dim3(kWave), 0, s, D);
  Carve entries;
  entries.add(&D.val, (size_t)total);
  entries.add(&D.idx, (size_t)total);
  MSKM_TRY(entries.alloc(h));
  hipLaunchKernelGGL(k_stream_fill, dim3((unsigned)ns), dim3(kBlock), 0, s, D, h->diag.rowptr, h->diag.col,
                     h->diag.val32);
  MSKM_HIP_TRY(hipMemcpyAsync(st, D.stats, 24, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipStreamSynchronize(s));
  P.width = st[0];
  P.window = st[4] * kWave;
  P.rows = st[2];
  P.chunks = st[5];
  P.inv = (st[3] + 3) / 4 * 4;
  if (stream_lds(P) > kStreamLds) P.inv = 0;
  if (stream_lds(P) > kStreamLds) return MSKM_OK;
  // slices past the resident slots, in the order slot by slot, that fit the LDS left
  const int res = stream_resident(P.width), streamed = (P.rows + kWave - 1) / kWave - res * kStreamWaves;
  if (streamed > 0)
    P.nl = (int32_t)std::min<size_t>((size_t)streamed, (kStreamLds - stream_lds(P)) / (6 * (size_t)P.width * kWave));
  MSKM_HIP_TRY(hipGetLastError());
  P.ok = true;
  return MSKM_OK;
}
}  // namespace

// -------------------------------------------------------------------- solve

typedef float st_f4 __attribute__((ext_vector_type(4)));
typedef unsigned short st_u4 __attribute__((ext_vector_type(4)));

// kStreamRt slots of 512 rows, the first RES of them in registers (rows of at
// most E entries). Thread t holds row 512 j + t in slot j. The single-reduction
// form and the order of the launched kernels, so that a solve rounds as theirs
// does, element by element: SUM is the order of a row's products (kSumRow,
// kSumHalves or kSumLanes8), NA sums added in halves.
template <bool PC, int RES, int E, int SUM>
__global__ void __launch_bounds__(kGridThreads)
    k_cg_stream(const CgStreamDev P, int window, int rows, int ninv, int nl, int width, const float* __restrict__ b,
                float* __restrict__ x, uint32_t* z0, uint32_t* z1, CgLevel* __restrict__ st, int32_t* aborted,
                double rtol2, int maxit, int spin, const PcArgs<float> pc) {
  constexpr int RT = kStreamRt, NA = SUM == kSumRow ? 1 : SUM == kSumHalves ? 2 : 8;
  extern __shared__ __align__(16) char lds[];
  float* const zw = reinterpret_cast<float*>(lds);                 // z on the kept runs of the window
  float* const rs = zw + (window + 3) / 4 * 4;                     // r, x of the own rows
  float* const xs = rs + (rows + 3) / 4 * 4;
  int2* const bi = reinterpret_cast<int2*>(xs + (rows + 3) / 4 * 4);  // inverse offset, block start << 8 | size
  float* const li = reinterpret_cast<float*>(bi + (rows + 3) / 4 * 4);  // block inverses
  float* const lv = li + ninv;                                     // slices kept here: values, positions
  uint16_t* const lx = reinterpret_cast<uint16_t*>(lv + nl * width * kWave);
  uint32_t* const chunk = reinterpret_cast<uint32_t*>(lx + nl * width * kWave);
  __shared__ double sm[3][kStreamWaves], sp[kStreamWaves], sq[4];
  __shared__ int bad;
  const int wg = blockIdx.x, t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWave), lane = t % kWave;
  const int l = P.lev[wg], nw = P.nw[wg], me = P.part[wg], nslot = P.nwg;
  const int r0 = P.row0[wg], nr = P.nrow[wg], base = P.wbase[wg], wlen = P.wlen[wg], own0 = r0 - base;
  const int own = P.rank[(int64_t)wg * kStreamChunks + (own0 >> 6)] * kWave + (own0 & 63);  // own rows in the kept runs
  const int nchunk = P.nchunk[wg];
  uint64_t* const slot = P.slots + (size_t)P.wg0[wg] * kGridSlot;
  const int64_t* const so = P.soff + ((int64_t)wg * kStreamWaves + w) * RT;

  // resident entries
  constexpr int kRes = RES > 0 ? RES : 1, kE = RES > 0 ? E : 16;
  float v[kRes][kE];
  uint32_t ci[kRes][kE / 2];
  int wid[kRes];
#pragma unroll
  for (int j = 0; j < RES; ++j) {
    const int64_t o = so[j];
    wid[j] = __builtin_amdgcn_readfirstlane((int)((so[j + 1] - o) / kWave));
#pragma unroll
    for (int k = 0; k < kE; k += 4) {
      st_f4 a = {0.f, 0.f, 0.f, 0.f};
      st_u4 c = {0, 0, 0, 0};
      if (k < wid[j]) {
        a = *reinterpret_cast<const st_f4*>(P.val + o + (int64_t)k * kWave + 4 * lane);
        c = *reinterpret_cast<const st_u4*>(P.idx + o + (int64_t)k * kWave + 4 * lane);
      }
      v[j][k] = a.x;
      v[j][k + 1] = a.y;
      v[j][k + 2] = a.z;
      v[j][k + 3] = a.w;
      ci[j][k / 2] = (uint32_t)c.x | (uint32_t)c.y << 16;
      ci[j][k / 2 + 1] = (uint32_t)c.z | (uint32_t)c.w << 16;
    }
  }
  const float* inv = nullptr;
  if constexpr (PC) {
    const int32_t bfirst = pc.of_row[r0];
    const int64_t o0 = pc.off[bfirst];
    inv = pc.inv + o0;
    if (ninv > 0) {
      const int words = (int)(pc.off[pc.of_row[r0 + nr - 1] + 1] - o0);
      for (int k = t; k < words; k += kGridThreads) li[k] = inv[k];
    }
    for (int i = t; i < nr; i += kGridThreads) {
      const int32_t bk = pc.of_row[r0 + i];
      const int64_t a = pc.start[bk];
      bi[i] = make_int2((int)(pc.off[bk] - o0), (int)(a - r0) << 8 | (int)(pc.start[bk + 1] - a));
    }
  }
  for (int k = t; k < nchunk; k += kGridThreads) chunk[k] = P.chunk[(int64_t)wg * kStreamChunks + k];
  for (int k = t; k < window; k += kGridThreads) zw[k] = 0.0f;
  for (int q = w; q < nl; q += kStreamWaves) {  // streamed slice q: slot RES + q / 8 of wave q % 8
    const int64_t o = so[RES + q / kStreamWaves], e = so[RES + q / kStreamWaves + 1];
    for (int64_t d = o + 4 * lane; d < e; d += 4 * kWave) {
      *reinterpret_cast<st_f4*>(lv + q * width * kWave + (d - o)) = *reinterpret_cast<const st_f4*>(P.val + d);
      *reinterpret_cast<st_u4*>(lx + q * width * kWave + (d - o)) = *reinterpret_cast<const st_u4*>(P.idx + d);
    }
  }
  for (int i = t; i < nr; i += kGridThreads) {
    rs[i] = b[r0 + i];
    xs[i] = 0.0f;
  }
  if (t == 0) bad = get(aborted) != 0;  // a launch before this one has given up
  __syncthreads();
  int left = bad ? 0 : spin;            // polls that the thread still waits for

  float p[RT], s[RT];  // direction and A p of the own rows
#pragma unroll
  for (int j = 0; j < RT; ++j) p[j] = s[j] = 0.0f;
  // z = M^-1 r of the own rows (the inverses are symmetric: lane i of a block
  // reads column i, consecutive lanes consecutive words), published in zc
  auto precondition = [&](uint32_t* zc) {
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      const int i = j * kGridThreads + t;
      if (i < nr) {
        float zi = rs[i];
        if constexpr (PC) {
          const int2 q = bi[i];
          const int m = q.y & 255, ba = q.y >> 8;
          const float* rb = rs + ba;
          zi = 0.0f;
          if (ninv > 0) {
            const float* Mc = li + q.x + (i - ba);
#pragma unroll 4
            for (int k = 0; k < m; ++k) zi += Mc[k * m] * rb[k];
          } else {
            const float* Mc = inv + q.x + (i - ba);
#pragma unroll 8
            for (int k = 0; k < m; ++k) zi += Mc[k * m] * rb[k];
          }
        }
        zw[own + i] = zi;
        put(&zc[r0 + i], word_of(zi));
      }
    }
  };
  precondition(z0);

  CgLevel S{};
  S.rtol2 = rtol2;
  S.maxit = maxit;
  int n = 0;
  for (int m = 0;; ++n, m = m == 2 ? 0 : m + 1) {  // m = n % 3
    uint32_t* const zc = n & 1 ? z1 : z0;
    // z of the halo, four runs of a wave at a time
    for (int q0 = 0; q0 < nchunk; q0 += kStreamHalo * kStreamWaves) {
      uint32_t hz[kStreamHalo];
      int he[kStreamHalo], at[kStreamHalo];
#pragma unroll
      for (int q = 0; q < kStreamHalo; ++q) {
        const int k = q0 + q * kStreamWaves + w;
        he[q] = -1;
        if (k < nchunk) {
          const uint32_t ck = chunk[k];
          const int e = (int)(ck & 0xffffu) * kWave + lane;
          if (e < wlen && (e < own0 || e >= own0 + nr)) {
            he[q] = e;
            at[q] = (int)(ck >> 16) * kWave + lane;
            hz[q] = get(&zc[base + e]);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < kStreamHalo; ++q)
        if (he[q] >= 0) {
          if (hz[q] == kEmptyWord) hz[q] = poll(&zc[base + he[q]], kEmptyWord, left, &bad);
          zw[at[q]] = value_of(hz[q]);
        }
    }
    __syncthreads();
    if (bad) break;
    // q = A z (the empty asm statements keep the compiler from unpacking the
    // resident positions once and for all, into twice as many registers, and
    // from having the LDS reads of many groups in flight: both would spill)
    float qv[RT];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      float acc[NA];  // entry k in number k % 8, (k / 4) % 2 or 0
#pragma unroll
      for (int u = 0; u < NA; ++u) acc[u] = 0.0f;
      if (j < RES) {
#pragma unroll
        for (int k0 = 0; k0 < kE; k0 += 16) {
#pragma unroll
          for (int k = k0 / 2; k < k0 / 2 + 8; ++k) asm volatile("" : "+v"(ci[j < RES ? j : 0][k]));
#pragma unroll
          for (int k = k0; k < k0 + 16; ++k) {
            const uint32_t c = ci[j < RES ? j : 0][k / 2];
            acc[NA == 8 ? k & 7 : NA == 2 ? (k >> 2) & 1 : 0] +=
                v[j < RES ? j : 0][k] * zw[k & 1 ? c >> 16 : c & 0xffffu];
          }
          asm volatile("" ::: "memory");
        }
      } else {
        const int q = (j - RES) * kStreamWaves + w;
        const int64_t o = so[j];
        const int len = (int)(so[j + 1] - o);
        const bool here = q < nl;  // kept in LDS
        auto streamed = [&](const float* pv, const uint16_t* px) {
          auto group = [&](int d, auto odd) {
            constexpr int o = decltype(odd)::value ? NA / 2 : 0, s = NA == 8 ? 1 : 0;
            const st_f4 f = *reinterpret_cast<const st_f4*>(pv + d);
            const st_u4 u = *reinterpret_cast<const st_u4*>(px + d);
            acc[o] += f.x * zw[u.x];
            acc[o + s] += f.y * zw[u.y];
            acc[o + 2 * s] += f.z * zw[u.z];
            acc[o + 3 * s] += f.w * zw[u.w];
          };
          if constexpr (NA > 1) {  // unrolled twice the preconditioned form takes 61 ms where it takes 42, the
            int d = 0;             // other one 45 where once takes 53 (70,001 rows of 180 entries, 3,000 and 4,250 iterations)
#pragma unroll (PC ? 1 : 2)
            for (; d + 4 * kWave < len; d += 8 * kWave) {
              group(d, std::false_type{});
              group(d + 4 * kWave, std::true_type{});
            }
            if (d < len) group(d, std::false_type{});
          } else {
#pragma unroll 4
            for (int d = 0; d < len; d += 4 * kWave) group(d, std::false_type{});
          }
        };
        if (here)
          streamed(lv + q * width * kWave + 4 * lane, lx + q * width * kWave + 4 * lane);
        else
          streamed(P.val + o + 4 * lane, P.idx + o + 4 * lane);
      }
#pragma unroll
      for (int o = NA / 2; o > 0; o /= 2)
#pragma unroll
        for (int u = 0; u < o; ++u) acc[u] += acc[u + o];
      qv[j] = acc[0];
      const int i = j * kGridThreads + t;
      if (i < nr) {
        const double zi = (double)zw[own + i], ri = (double)rs[i];
        a0 += zi * (double)acc[0];
        a1 += zi * ri;
        a2 += ri * ri;
      }
    }
    // exchange of z.q, r.z and r.r (every earlier store of this workgroup is waited for first)
    a0 = wave64_sum(a0);
    a1 = wave64_sum(a1);
    if constexpr (PC) a2 = wave64_sum(a2);
    if (lane == 0) {
      sm[0][w] = a0;
      sm[1][w] = a1;
      sm[2][w] = a2;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (w < (PC ? 3 : 2)) {
      const double a = lanes_sum<kStreamWaves>(sm[w][lane % kStreamWaves]);
      if (lane == 0) put(slot + (m * nslot + me) * kGridSlot + w, word_of(a));
    }
    const uint64_t* const sa = slot + (size_t)(m * nslot) * kGridSlot;
    uint64_t u = 0, u2 = 0;  // word t / 256, and word 2
    if (t % 256 < nw) {
      u = get(sa + t % 256 * kGridSlot + t / 256);
      if (PC && t < 256) u2 = get(sa + t * kGridSlot + 2);
      if (u == kEmptySlot) u = poll(sa + t % 256 * kGridSlot + t / 256, kEmptySlot, left, &bad);
      if (PC && u2 == kEmptySlot) u2 = poll(sa + t * kGridSlot + 2, kEmptySlot, left, &bad);
    }
    const double s01 = wave64_sum(value_of(u));
    if (lane == 0) sp[w] = s01;
    if (PC && w < 4) {
      const double s2 = wave64_sum(value_of(u2));
      if (lane == 0) sq[w] = s2;
    }
    __syncthreads();
    if (bad) break;
    const double delta = (sp[0] + sp[1]) + (sp[2] + sp[3]), gamma = (sp[4] + sp[5]) + (sp[6] + sp[7]);
    const double rr = PC ? (sq[0] + sq[1]) + (sq[2] + sq[3]) : gamma;
    if (n == 0) S.bb = rr;
    if (!cg1_decide(S, gamma, delta, rr)) break;
    // everybody has this iteration's z, and has left the sums before
    if (w < (PC ? 3 : 2) && lane == 0) put(slot + ((m == 0 ? 2 : m - 1) * nslot + me) * kGridSlot + w, kEmptySlot);
    const float beta = (float)S.beta;
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      const int i = j * kGridThreads + t;
      if (i < nr) {
        p[j] = zw[own + i] + beta * p[j];
        s[j] = qv[j] + beta * s[j];
        xs[i] = (float)((double)xs[i] + S.alpha * (double)p[j]);
        rs[i] = (float)((double)rs[i] - S.alpha * (double)s[j]);
        put(&zc[r0 + i], kEmptyWord);
      }
    }
    if constexpr (PC) __syncthreads();
    precondition(n & 1 ? z0 : z1);
  }
  if (bad) {
    if (t == 0) atomicOr(aborted, 1);
    return;
  }
  for (int i = t; i < nr; i += kGridThreads) x[r0 + i] = xs[i];
  if (t == 0 && me == 0) {
    S.on = 1;
    S.done = 1;
    st[l] = S;
  }
}

mskm_status cg_stream_ready(mskm_hier* h, int lo, int hi, bool bj, int* depth) {
  *depth = -1;
  const int d = h->h_depth[lo];
  if (!h->diag.val32 || h->h_depth[hi] != d || h->h_depth_begin[d] != lo || h->h_depth_begin[d + 1] != hi + 1)
    return MSKM_OK;
  int64_t most = 0;
  for (int l = lo; l <= hi; ++l) {
    if (h->h_lev[l].n <= 0) return MSKM_OK;
    most = std::max<int64_t>(most, h->h_lev[l].n);
  }
  if (most <= 256) return MSKM_OK;  // one workgroup each (k_cg_level_wg), whose order there this kernel does not have
  if (!h->cg_stream) {
    auto* p = new (std::nothrow) CgStream();
    if (!p) return MSKM_OK;
    h->cg_stream = p;
    h->cg_stream_free = cg_stream_free;
  }
  auto& plans = static_cast<CgStream*>(h->cg_stream)->depth[bj ? 1 : 0];
  if (plans.empty()) plans.resize(h->h_depth_begin.size() - 1);
  CgStreamPlan& P = plans[d];
  if (!P.built) {
    P.built = true;
    const size_t mark = h->allocs.size();
    const mskm_status st = build_stream(h, P, d, bj);
    if (!P.ok) halloc_undo(h, mark);
    if (st < 0 && st != MSKM_ENOMEM) return st;
  }
  if (P.ok) *depth = d;
  return MSKM_OK;
}

mskm_status cg_stream_launch(mskm_hier* h, int depth, bool bj, const float* b, float* x, float* z0, float* z1,
                             CgLevel* st, int32_t* aborted, double rtol2, int maxit, const PcArgs<float>& pc) {
  CgStreamPlan& P = static_cast<CgStream*>(h->cg_stream)->depth[bj ? 1 : 0][depth];
  mskm_ctx* c = h->ctx;
  hipStream_t s = c->stream;
  const int64_t r0 = h->h_off[h->h_depth_begin[depth]], n = h->h_off[h->h_depth_begin[depth + 1]] - r0;
  grid_empty<float>(s, z0, z1, nullptr, r0, n, P.d.slots, (int64_t)3 * P.d.nwg * kGridSlot);
  const size_t lds = stream_lds(P);
  const int sum = launched_sum(h, h->h_depth_begin[depth], h->h_depth_begin[depth + 1] - 1, true);
  hipError_t e = hipSuccess;
  const mskm_status r = cg_grid_in_turn(c, [&] {
#define MSKM_STREAM(PCF, RES, EE, SS)                                                                                \
  do {                                                                                                              \
    auto* k = k_cg_stream<PCF, RES, EE, SS>;                                                                        \
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
    if (e == hipSuccess)                                                                                            \
      hipLaunchKernelGGL(k, dim3(P.d.nwg), dim3(kGridThreads), lds, s, P.d, P.window, P.rows, P.inv, P.nl, P.width, \
                         b, x, (uint32_t*)z0, (uint32_t*)z1, st, aborted, rtol2, maxit, c->grid_spin, pc);            \
  } while (0)
// (two sums a row in turn and 96 resident entries spill 100 registers)
#define MSKM_STREAM_RES(PCF, SS)                \
  do {                                          \
    if (P.width <= 48)                          \
      MSKM_STREAM(PCF, 2, 48, SS);              \
    else if (P.width <= 96 && SS != kSumHalves) \
      MSKM_STREAM(PCF, 1, 96, SS);              \
    else                                        \
      MSKM_STREAM(PCF, 0, 16, SS);              \
  } while (0)
#define MSKM_STREAM_SUM(PCF)                   \
  do {                                         \
    if (sum == kSumRow)                        \
      MSKM_STREAM_RES(PCF, kSumRow);           \
    else if (sum == kSumHalves)                \
      MSKM_STREAM_RES(PCF, kSumHalves);        \
    else                                       \
      MSKM_STREAM_RES(PCF, kSumLanes8);        \
  } while (0)
    if (bj)
      MSKM_STREAM_SUM(true);
    else
      MSKM_STREAM_SUM(false);
#undef MSKM_STREAM_SUM
#undef MSKM_STREAM_RES
#undef MSKM_STREAM
  });
  if (e != hipSuccess) return fail(MSKM_EDEVICE, std::string("persistent CG: ") + hipGetErrorString(e));
  return r;
}

}  // namespace mskm
