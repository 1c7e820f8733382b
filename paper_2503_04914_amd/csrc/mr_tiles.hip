// Products with many right-hand sides on the matrix cores.
//
// Neighbouring rows have most of their columns in common (the internal order
// is spatial): 16 consecutive rows of a 2-D level with 40 entries a row reach
// about 150 distinct columns, and their entries in a coarser level about 55
// for that level. One wave multiplies the dense 16 x columns tile of such rows
// with the listed rows of X, so a row of X is fetched once per tile instead
// of once per entry (4.3 times fewer for the diagonal blocks, 10 and more for
// the lower ones), and the arithmetic that the zeros of the tile add (73% of
// a diagonal tile) runs on matrix cores that were idle: FP32 products on
// v_mfma_f32_16x16x4_f32, FP64 ones on v_mfma_f64_16x16x4_f64, inputs and
// accumulation in the operator's precision.
//
// Layout. Lane (n, k) = (lane % 16, lane / 16). In one step of 16 listed
// columns, lane (n, k) reads places 4 k .. 4 k + 3 of row n of the tile (LDS) and
// NT consecutive right-hand sides NT n .. of the four rows of X that belong to
// the columns there (one vector load each, 256 contiguous bytes per 16
// lanes): 4 NT matrix instructions, the j-th on places {4 k + j}, right-hand
// sides {NT n + q}. The tile is built in LDS by its own wave (zeroed, the
// segment's entries scattered), 128 columns at a time in FP32 and 64 in FP64
// (8.4 KB a wave, 16 waves a CU); the rows of X for the next step are in
// flight while a step multiplies. What bounds it is the fetch of X through
// the caches.
#include <algorithm>
#include <new>
#include <vector>

#include "device_common.h"
#include "mr_tiles.h"

namespace mskm {

// --------------------------------------------------------------------- build

constexpr int kWinWords = 2048;            // bitmap window of 65536 columns
constexpr int kTileMaxCols = 65536;        // listed columns of one tile (at most)
constexpr int kTileMaxSegs = kTileMaxCols / kTileSeg;

// Place of listed column pos: within 16 listed columns, column 4 j + k goes to
// place 4 k + j, so that the matrix instruction j of a step, which takes places j,
// 4 + j, 8 + j and 12 + j, multiplies columns 4 j .. 4 j + 3. These are added in
// order, each with one rounding (checked against a chain of fused multiply-adds: no
// difference in 512,000 FP32 results), and the zeros of the tile add nothing: a
// row's products are summed in the order of its entries, as the row-by-row
// kernels of solve_mr.hip sum them, and a level's CG rounds as it does with those.
__device__ __forceinline__ int tile_place(int pos) { return (pos & ~15) | (pos & 3) << 2 | (pos >> 2 & 3); }

// Rows of tile t: [r0, r1) (empty past the end of its block).
__device__ __forceinline__ void tile_rows(const WorkTable& wt, int64_t t, int64_t& r0, int64_t& r1) {
  const int64_t b = t >> 2;
  r0 = min(wt.row0[b] + kTileRows * (t & 3), wt.row1[b]);
  r1 = min(r0 + kTileRows, wt.row1[b]);
}

// Walks the columns of entries [e0, e1) in ascending order by windows of 65536
// columns: fn(base, first, bits, rank) is called by all threads once per
// window that holds columns, with the window's bitmap, each word's number of
// set bits before it and the number of columns listed before the window.
// Returns the number of distinct columns.
template <typename F>
__device__ __forceinline__ int tile_windows(int64_t e0, int64_t e1, const int32_t* __restrict__ col, uint32_t* bits,
                                            uint32_t* rank, int* red, F&& fn) {
  constexpr int kPer = kWinWords / kBlock;
  const int t = threadIdx.x;
  int listed = 0;
  int64_t from = 0;
  for (;;) {
    // the smallest column not yet listed
    int lo = INT32_MAX;
    for (int64_t k = e0 + t; k < e1; k += kBlock) {
      const int c = col[k];
      if (c >= from) lo = min(lo, c);
    }
    for (int o = 32; o > 0; o >>= 1) lo = min(lo, __shfl_xor(lo, o, kWave));
    __syncthreads();
    if (t % kWave == 0) red[t / kWave] = lo;
    __syncthreads();
    for (int w = 0; w < kBlock / kWave; ++w) lo = min(lo, red[w]);
    if (lo == INT32_MAX) return listed;
    for (int w = t; w < kWinWords; w += kBlock) bits[w] = 0;
    __syncthreads();
    for (int64_t k = e0 + t; k < e1; k += kBlock) {
      const int64_t c = (int64_t)col[k] - lo;
      if (c >= 0 && c < 32 * kWinWords) atomicOr(&bits[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    uint32_t sum = 0;
    for (int q = 0; q < kPer; ++q) sum += __popc(bits[t * kPer + q]);
    uint32_t inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t v = __shfl_up(inc, o, kWave);
      if (t % kWave >= o) inc += v;
    }
    if (t % kWave == kWave - 1) red[t / kWave] = (int)inc;
    __syncthreads();
    uint32_t base = inc - sum, total = 0;
    for (int w = 0; w < kBlock / kWave; ++w) {
      if (w < t / kWave) base += (uint32_t)red[w];
      total += (uint32_t)red[w];
    }
    for (int q = 0; q < kPer; ++q) {
      rank[t * kPer + q] = base;
      base += __popc(bits[t * kPer + q]);
    }
    __syncthreads();
    fn(lo, listed);
    __syncthreads();
    listed += (int)total;
    from = (int64_t)lo + 32 * kWinWords;
  }
}

__global__ void __launch_bounds__(kBlock)
    k_tile_count(const WorkTable wt, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                 int64_t* __restrict__ ncol, int64_t* __restrict__ nseg, int64_t ntile, int32_t* __restrict__ most) {
  __shared__ uint32_t bits[kWinWords], rank[kWinWords];
  __shared__ int red[kBlock / kWave];
  const int64_t tile = blockIdx.x;
  int64_t r0, r1;
  tile_rows(wt, tile, r0, r1);
  const int n = tile_windows(rp[r0], rp[r1], col, bits, rank, red, [](int, int) {});
  if (threadIdx.x == 0) {
    ncol[tile] = (n + 15) / 16 * 16;
    nseg[tile] = (n + kTileSeg - 1) / kTileSeg;
    if (tile == 0) ncol[ntile] = nseg[ntile] = 0;
    if (n > kTileMaxCols) atomicMax(most, n);
  }
}

__global__ void __launch_bounds__(kBlock)
    k_tile_fill(const WorkTable wt, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                const double* __restrict__ val, const float* __restrict__ val32, const float* __restrict__ lo32,
                const MrTiles T) {
  __shared__ uint32_t bits[kWinWords], rank[kWinWords];
  __shared__ int red[kBlock / kWave];
  __shared__ int hist[kTileMaxSegs + 1];
  const int64_t tile = blockIdx.x;
  const int t = threadIdx.x;
  int64_t r0, r1;
  tile_rows(wt, tile, r0, r1);
  const int64_t e0 = rp[r0], e1 = rp[r1], c0 = T.cptr[tile], s0 = T.sptr[tile];
  const int ns = (int)(T.sptr[tile + 1] - s0), nc = (int)(T.cptr[tile + 1] - c0);
  for (int s = t; s <= ns; s += kBlock) hist[s] = 0;
  __syncthreads();
  auto place = [&](int64_t k, int base, int listed, int& pos) {  // position of entry k's column, if in this window
    const int64_t c = (int64_t)col[k] - base;
    if (c < 0 || c >= 32 * kWinWords) return false;
    pos = listed + (int)(rank[c >> 5] + __popc(bits[c >> 5] & ((1u << (c & 31)) - 1u)));
    return true;
  };
  const int n = tile_windows(e0, e1, col, bits, rank, red, [&](int base, int listed) {
    for (int w = t; w < kWinWords; w += kBlock) {
      uint32_t m = bits[w];
      int at = listed + (int)rank[w];
      while (m) {
        T.cols[c0 + tile_place(at++)] = base + 32 * w + __ffs(m) - 1;
        m &= m - 1;
      }
    }
    for (int64_t k = e0 + t; k < e1; k += kBlock) {
      int pos;
      if (place(k, base, listed, pos)) atomicAdd(&hist[pos / kTileSeg], 1);
    }
  });
  // segment starts (entries of a segment land in any order within it: each has its own place in the tile)
  if (t == 0) {
    int at = 0;
    for (int s = 0; s < ns; ++s) {
      const int c = hist[s];
      hist[s] = at;
      T.eptr[s0 + s] = e0 + at;
      at += c;
    }
    if (tile == T.ntile - 1) T.eptr[T.nseg] = T.nnz;
  }
  __threadfence_block();
  __syncthreads();
  for (int q = n + t; q < nc; q += kBlock) T.cols[c0 + tile_place(q)] = T.cols[c0 + tile_place(n - 1)];
  tile_windows(e0, e1, col, bits, rank, red, [&](int base, int listed) {
    for (int64_t k = e0 + t; k < e1; k += kBlock) {
      int pos;
      if (!place(k, base, listed, pos)) continue;
      int row = 0;  // the last row starting at or before entry k
      for (int b = kTileRows / 2; b > 0; b >>= 1)
        if (r0 + row + b < r1 && rp[r0 + row + b] <= k) row += b;
      const int64_t at = e0 + atomicAdd(&hist[pos / kTileSeg], 1);
      T.code[at] = (uint16_t)(row << 7 | (tile_place(pos) & 127));
      if (T.val) T.val[at] = val[k];
      if (T.val32) T.val32[at] = val32[k];
      if (T.lo) T.lo[at] = lo32[k];
    }
  });
}

namespace {
struct MrTileSet {
  bool tried[2] = {false, false}, ok[2] = {false, false};
  MrTiles t[2];
};
void tile_set_free(void* p) { delete static_cast<MrTileSet*>(p); }

mskm_status build_tiles(mskm_hier* h, const Csr& A, MrTiles& T, bool* ok) {
  *ok = false;
  hipStream_t s = h->ctx->stream;
  const WorkTable& wt = h->wt_spmv;
  T.ntile = 4 * (int64_t)wt.nblocks;
  if (T.ntile == 0 || T.ntile > INT32_MAX) return MSKM_OK;
  T.nnz = A.nnz;
  int64_t *ncol = nullptr, *nseg = nullptr, *part = nullptr;
  int32_t* most = nullptr;
  Carve cv;
  cv.add(&ncol, (size_t)T.ntile + 1);
  cv.add(&nseg, (size_t)T.ntile + 1);
  cv.add(&part, (size_t)scan_parts(T.ntile + 1));
  cv.add(&most, 1);
  void* base = nullptr;
  MSKM_TRY(cv.alloc(h->ctx, &base));
  CtxScratch scratch{h->ctx, base, cv.bytes};
  MSKM_TRY(halloc(h, &T.cptr, (size_t)T.ntile + 1));
  MSKM_TRY(halloc(h, &T.sptr, (size_t)T.ntile + 1));
  MSKM_HIP_TRY(hipMemsetAsync(most, 0, 4, s));
  hipLaunchKernelGGL(k_tile_count, dim3((unsigned)T.ntile), dim3(kBlock), 0, s, wt, A.rowptr, A.col, ncol, nseg,
                     T.ntile, most);
  MSKM_TRY(exclusive_scan_i64(s, ncol, T.cptr, T.ntile + 1, part));
  MSKM_TRY(exclusive_scan_i64(s, nseg, T.sptr, T.ntile + 1, part));
  int32_t over = 0;
  MSKM_HIP_TRY(hipMemcpyAsync(&T.ncol, T.cptr + T.ntile, 8, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipMemcpyAsync(&T.nseg, T.sptr + T.ntile, 8, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipMemcpyAsync(&over, most, 4, hipMemcpyDeviceToHost, s));
  MSKM_HIP_TRY(hipStreamSynchronize(s));
  if (over) return MSKM_OK;
  Carve tiles;
  tiles.add(&T.cols, (size_t)T.ncol);
  tiles.add(&T.eptr, (size_t)T.nseg + 1);
  tiles.add(&T.code, (size_t)T.nnz);
  if (A.val) tiles.add(&T.val, (size_t)T.nnz);
  if (A.val32) tiles.add(&T.val32, (size_t)T.nnz);
  if (A.val32lo) tiles.add(&T.lo, (size_t)T.nnz);
  MSKM_TRY(tiles.alloc(h));
  hipLaunchKernelGGL(k_tile_fill, dim3((unsigned)T.ntile), dim3(kBlock), 0, s, wt, A.rowptr, A.col, A.val, A.val32,
                     A.val32lo, T);
  MSKM_HIP_TRY(hipGetLastError());
  *ok = true;
  return MSKM_OK;
}
}  // namespace

mskm_status mr_tiles(mskm_hier* h, bool lower, const MrTiles** out) {
  *out = nullptr;
  if (!h->mr_tiles) {
    auto* p = new (std::nothrow) MrTileSet();
    if (!p) return MSKM_OK;
    h->mr_tiles = p;
    h->mr_tiles_free = tile_set_free;
  }
  MrTileSet& S = *static_cast<MrTileSet*>(h->mr_tiles);
  const int k = lower ? 1 : 0;
  if (!S.tried[k]) {
    S.tried[k] = true;
    const size_t mark = h->allocs.size();
    const mskm_status st = build_tiles(h, lower ? h->lower : h->diag, S.t[k], &S.ok[k]);
    if (!S.ok[k]) halloc_undo(h, mark);
    if (st < 0 && st != MSKM_ENOMEM) return st;
  }
  if (S.ok[k]) *out = &S.t[k];
  return MSKM_OK;
}

bool mr_tiles_built(const mskm_hier* h) {
  const auto* S = static_cast<const MrTileSet*>(h->mr_tiles);
  return S && S->ok[0] && S->ok[1];
}

// ------------------------------------------------------------------ products

// Values in the product's precision: entries i, i + step, ... from entry e on (past `last`: that one again).
template <typename T>
struct TileVals;
template <>
struct TileVals<float> {
  const float* v;
  template <int N>
  __device__ __forceinline__ void get(int64_t e, int i, int step, int last, float (&o)[N]) const {
#pragma unroll
    for (int u = 0; u < N; ++u) o[u] = (v + e)[(uint32_t)min(i + u * step, last)];
  }
};
template <>
struct TileVals<double> {
  const double* v;
  const float *hi, *lo;  // without FP64 values: FP32 value + remainder
  template <int N>
  __device__ __forceinline__ void get(int64_t e, int i, int step, int last, double (&o)[N]) const {
    if (v) {
#pragma unroll
      for (int u = 0; u < N; ++u) o[u] = (v + e)[(uint32_t)min(i + u * step, last)];
    } else {
      float a[N], b[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const uint32_t k = (uint32_t)min(i + u * step, last);
        a[u] = (hi + e)[k];
        b[u] = (lo + e)[k];
      }
#pragma unroll
      for (int u = 0; u < N; ++u) o[u] = (double)a[u] + (double)b[u];
    }
  }
};

// A wave's LDS: the tile's columns of a pass, and their rows of X.
template <typename TX>
struct TileLds {
  alignas(16) TX a[kTileRows * Mma<TX>::kStride];
  alignas(16) int32_t c[Mma<TX>::kCols];
};

// d += tile * X for right-hand sides c0 + NT n + q; S: the wave's LDS.
template <typename TX, int NT>
__device__ __forceinline__ void tile_mul(const MrTiles& T, int64_t tile, const TileVals<TX>& val, const TX* x, int ldr,
                                         int c0, TileLds<TX>& S, typename Mma<TX>::acc (&d)[NT]) {
  constexpr int CH = Mma<TX>::kCols, ST = Mma<TX>::kStride;
  const int lane = threadIdx.x % kWave, n = lane % 16, k4 = lane / 16;
  const int64_t s0 = T.sptr[tile], s1 = T.sptr[tile + 1], cb = T.cptr[tile];
  const int nc = (int)(T.cptr[tile + 1] - cb);
  const TX* xc = x + c0 + NT * n;
  for (int ch = 0; ch * CH < nc; ++ch) {
    const int steps = min(CH, nc - ch * CH) / 16;
    for (int z = lane; z < 16 * steps; z += kWave) S.c[z] = T.cols[cb + ch * CH + z];
    typedef typename VecN<TX, 16 / sizeof(TX)>::type zvec;
    for (int z = lane; z < kTileRows * ST * (int)sizeof(TX) / 16; z += kWave)
      reinterpret_cast<zvec*>(S.a)[z] = (zvec)(TX)0;
    __builtin_amdgcn_wave_barrier();
    // rows of X of the first step; columns of the step after the one asked for
    mi4 c = *reinterpret_cast<const mi4*>(S.c + 4 * k4);
    TX b0[4][NT], b1[4][NT];
    auto rows = [&](int next, TX (&bn)[4][NT]) {
#pragma unroll
      for (int j = 0; j < 4; ++j) load_nt<NT>(xc + (int64_t)c[j] * ldr, bn[j]);
      c = *reinterpret_cast<const mi4*>(S.c + 4 * k4 + 16 * min(next, steps - 1));
      asm volatile("" ::: "memory");
    };
    rows(1, b0);
    // the tile's columns of this pass
    const int64_t ea = T.eptr[s0 + ch * (CH / kTileSeg)];
    const int64_t ee = T.eptr[min(s0 + (ch + 1) * (CH / kTileSeg), s1)];
    const int ne = (int)(ee - ea);
    for (int e = lane; e < ne; e += 4 * kWave) {
      int cd[4];
      TX v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) cd[u] = (T.code + ea)[(uint32_t)min(e + u * kWave, ne - 1)];  // past the end: the last one again
      val.template get<4>(ea, e, kWave, ne - 1, v);
#pragma unroll
      for (int u = 0; u < 4; ++u) S.a[(cd[u] >> 7) * ST + (cd[u] & (CH - 1))] = v[u];
    }
    __builtin_amdgcn_wave_barrier();
    const TX* Ar = S.a + n * ST + 4 * k4;
    auto step = [&](int s, TX (&bc)[4][NT]) {
      TX a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = Ar[16 * s + j];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < NT; ++q) d[q] = Mma<TX>::mul(a[j], bc[j][q], d[q]);
    };
    // the loads are unconditional (past the end: the last step's rows again)
    // and held in place by the empty asm statement: under a branch, or sunk to
    // their use, the products would wait for the ones just issued
    for (int s = 0; s < steps; ++s) {
      rows(s + 2, b1);
      step(s, b0);
      if (++s >= steps) break;
      rows(s + 2, b0);
      step(s, b1);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Block sums of the waves' per-right-hand-side values: acc[q] of lane (n, k)
// belongs to right-hand side c0 + NT n + q; part[blk * ldr + ...].
template <int NT>
__device__ __forceinline__ void tile_partial(double (&acc)[NT], double (*sm)[16 * 4], double* __restrict__ part,
                                             size_t at) {
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave, n = lane % 16;
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    acc[q] += __shfl_xor(acc[q], 16, kWave);
    acc[q] += __shfl_xor(acc[q], 32, kWave);
    if (lane < 16) sm[w][NT * n + q] = acc[q];
  }
  __syncthreads();
  if (threadIdx.x < 16 * NT) {
    double t = 0.0;
    for (int k = 0; k < kBlock / kWave; ++k) t += sm[k][threadIdx.x];
    part[at + threadIdx.x] = t;
  }
  __syncthreads();
}

// Workgroup (block of the work table, slice of 16 NT right-hand sides): four
// waves, one tile each. blockIdx.x = block * sub + slice within the chunk,
// blockIdx.y the chunk.
template <typename TX, int NT>
__global__ void __launch_bounds__(kBlock, 4)
    k_mrt_cg(const WorkTable wt, int base, int sub, const MrTiles D, const TileVals<TX> val, const TX* p,
             TX* __restrict__ q, int ldr, const int32_t* __restrict__ running, double* __restrict__ part) {
  __shared__ TileLds<TX> As[kBlock / kWave];
  __shared__ double sm[kBlock / kWave][16 * 4];
  const int id = xcd_block_id(gridDim.x);
  const int blk = base + id / sub, c0 = ((int)blockIdx.y * sub + id % sub) * 16 * NT;
  if (running[wt.lev[blk]] == 0) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int n = lane % 16, k4 = lane / 16;
  const int64_t r0 = wt.row0[blk] + kTileRows * w, r1 = wt.row1[blk];
  double acc[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) acc[u] = 0.0;
  if (r0 < r1) {
    typename Mma<TX>::acc d[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) d[u] = (typename Mma<TX>::acc)(TX)0;
    tile_mul<TX, NT>(D, 4 * (int64_t)blk + w, val, p, ldr, c0, As[w], d);
    TX pi[4][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i) load_nt<NT>(p + min(r0 + Mma<TX>::row(k4, i), r1 - 1) * ldr + c0 + NT * n, pi[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = r0 + Mma<TX>::row(k4, i);
      if (row < r1) {
        TX qi[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          qi[u] = d[u][i];
          acc[u] += (double)pi[i][u] * (double)qi[u];
        }
        store_nt<NT>(q + row * ldr + c0 + NT * n, qi);
      }
    }
  }
  tile_partial<NT>(acc, sm, part, (size_t)blk * ldr + c0);
}

// The same for widths of whole groups of four slices: workgroup (block, group
// of slices), wave w slice w of the group, and four tiles one after the other.
// The four waves lay a tile's columns out in LDS together, once for four
// slices, in two buffers in turn, and the next one's entries are on their way
// in registers while one is multiplied. Sums stay in the wave's lanes over the
// four tiles: the workgroups of four neighbouring blocks take one tile of the
// same block at a time, so that the rows of p that an XCD works on (2 MB for
// 256 right-hand sides) stay in its L2: the counter of reads from beyond it
// (FETCH_SIZE) shows 502,000 KiB, and 811,000 with a block's tiles in one
// workgroup. Every row has its
// diagonal entry, so a tile with rows has columns.
// 262,144 rows with 256 right-hand sides in FP32: 237 us (k_mrt_cg 323 us, or
// 256 us with its loads in place); the matrix cores are busy for 103 us of it,
// the vectors' 540 MB take 116 us, and 2.3 GB of rows of p pass from L2 to L1.
template <typename TX, int NT>
__global__ void __launch_bounds__(kBlock, 4)
    k_mrt_cg4(const WorkTable wt, int base, int sub, const MrTiles T, const TileVals<TX> val, const TX* p,
              TX* __restrict__ q, int ldr, const int32_t* __restrict__ running, double* __restrict__ part) {
  constexpr int CH = Mma<TX>::kCols, ST = Mma<TX>::kStride, kE = kTileRows * CH / kBlock;
  constexpr int kVec = kTileRows * ST * (int)sizeof(TX) / 16;  // 16-byte words of a buffer
  typedef typename VecN<TX, 16 / sizeof(TX)>::type zvec;
  typedef uint32_t mu4 __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) TX As[2][kTileRows * ST];
  __shared__ __align__(16) uint32_t offs[2][CH];  // byte offsets of the columns' rows of p
  const int id = xcd_block_id(gridDim.x);
  const int blk = base + id / sub;
  const int lev = wt.lev[blk];
  if (running[lev] == 0) return;
  const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWave), lane = t % kWave;
  const int n = lane % 16, k4 = lane / 16;
  const int c0 = (((int)blockIdx.y * sub + id % sub) * (kBlock / kWave) + w) * 16 * NT + NT * n;
  const uint32_t rowb = (uint32_t)ldr * sizeof(TX), c0b = (uint32_t)c0 * sizeof(TX);
  // the set's blocks sb .. sb + ns - 1; this workgroup's tiles are j, j + ns, ... of its 4 ns
  const int lb = wt.lev_begin[lev], sb = lb + (blk - lb) / 4 * 4, ns = min(4, wt.lev_begin[lev + 1] - sb), j = blk - sb;
  const char* const pb = reinterpret_cast<const char*>(p);
  auto row_at = [&](uint32_t o) { return reinterpret_cast<const TX*>(pb + (uint32_t)(o + c0b)); };
  // the pass at hand: the i-th tile (rows r0 ..), its columns ch CH ..
  int64_t tile = 0, cb = 0, sg = 0, r0 = 0, r1 = 0;
  int nc = 0, i = -1, ch = 0, ne = 0;
  auto next_tile = [&] {  // one with rows, if there is one
    do {
      ++i;
      if (i >= 4) return;
      const int q = j + i * ns, b = sb + q / 4;
      tile = 4 * (int64_t)b + q % 4;
      r0 = wt.row0[b] + kTileRows * (q % 4);
      r1 = wt.row1[b];
    } while (r0 >= r1);
    ch = 0;
    cb = T.cptr[tile];
    sg = T.sptr[tile];
    nc = (int)(T.cptr[tile + 1] - cb);
  };
  uint32_t cd[kE];
  TX ev[kE];
  int32_t col = 0;
  auto entries = [&] {  // of the pass, to registers
    const int64_t ea = T.eptr[sg], ee = T.eptr[min(sg + CH / kTileSeg, T.sptr[tile + 1])];
    ne = (int)(ee - ea);
    col = T.cols[cb + ch * CH + min(t, min(CH, nc - ch * CH) - 1)];
    // past the end: the last one again
#pragma unroll
    for (int u = 0; u < kE; ++u) cd[u] = (T.code + ea)[(uint32_t)min(u * kBlock + t, ne - 1)];
    val.template get<kE>(ea, t, kBlock, ne - 1, ev);
    asm volatile("" ::: "memory");
  };
  next_tile();
  if (i < 4) entries();
  int buf = 0;
  for (int z = t; z < kVec; z += kBlock) reinterpret_cast<zvec*>(As[0])[z] = (zvec)(TX)0;
  double acc[NT];
  typename Mma<TX>::acc d[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    acc[u] = 0.0;
    d[u] = (typename Mma<TX>::acc)(TX)0;
  }
  while (i < 4) {
    __syncthreads();  // the buffer is clear, the other one read
    const int steps = min(CH, nc - ch * CH) / 16;
#pragma unroll
    for (int u = 0; u < kE; ++u)
      if (u * kBlock + t < ne) As[buf][(cd[u] >> 7) * ST + (cd[u] & (CH - 1))] = ev[u];
    if (t < 16 * steps) offs[buf][t] = (uint32_t)col * rowb;
    __syncthreads();
    const TX* Ar = As[buf] + n * ST + 4 * k4;
    const uint32_t* Or = offs[buf] + 4 * k4;
    TX b0[4][NT], b1[4][NT];
    mu4 o = *reinterpret_cast<const mu4*>(Or);
    auto rows = [&](int next, TX (&bn)[4][NT]) {  // of the step at o; then o of step `next`
#pragma unroll
      for (int j = 0; j < 4; ++j) load_nt<NT>(row_at(o[j]), bn[j]);
      o = *reinterpret_cast<const mu4*>(Or + 16 * min(next, steps - 1));
      asm volatile("" ::: "memory");
    };
    rows(1, b0);
    // the next pass
    const bool last = (ch + 1) * CH >= nc;
    const int64_t ra = r0, rb = r1;
    if (last) {
      next_tile();
    } else {
      ++ch;
      sg += CH / kTileSeg;
    }
    buf ^= 1;
    if (i < 4) {
      entries();
      for (int z = t; z < kVec; z += kBlock) reinterpret_cast<zvec*>(As[buf])[z] = (zvec)(TX)0;
    }
    auto step = [&](int s, TX (&bc)[4][NT]) {
      TX a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = Ar[16 * s + j];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int u = 0; u < NT; ++u) d[u] = Mma<TX>::mul(a[j], bc[j][u], d[u]);
    };
    for (int s = 0; s < steps; ++s) {
      rows(s + 2, b1);
      step(s, b0);
      if (++s >= steps) break;
      rows(s + 2, b0);
      step(s, b1);
    }
    if (last) {
#pragma unroll
      for (int g = 0; g < 4; g += 2) {
        TX pi[2][NT];
#pragma unroll
        for (int h = 0; h < 2; ++h)
          load_nt<NT>(row_at((uint32_t)min(ra + Mma<TX>::row(k4, g + h), rb - 1) * rowb), pi[h]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int64_t row = ra + Mma<TX>::row(k4, g + h);
          if (row < rb) {
            TX qi[NT];
#pragma unroll
            for (int u = 0; u < NT; ++u) {
              qi[u] = d[u][g + h];
              acc[u] += (double)pi[h][u] * (double)qi[u];
            }
            store_nt<NT>(q + row * ldr + c0, qi);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < NT; ++u) d[u] = (typename Mma<TX>::acc)(TX)0;
    }
  }
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    acc[u] += __shfl_xor(acc[u], 16, kWave);
    acc[u] += __shfl_xor(acc[u], 32, kWave);
    if (lane < 16) part[(size_t)blk * ldr + c0 + u] = acc[u];
  }
}

// y = f - L x.
template <typename TX, int NT>
__global__ void __launch_bounds__(kBlock, 4)
    k_mrt_lower(const WorkTable wt, int base, int sub, const MrTiles Lw, const TileVals<TX> val,
   const TX* x, const TX* __restrict__ f, TX* __restrict__ y, int ldr) {
  __shared__ TileLds<TX> As[kBlock / kWave];
  const int id = xcd_block_id(gridDim.x);
  const int blk = base + id / sub, c0 = (id % sub) * 16 * NT;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int n = lane % 16, k4 = lane / 16;
  const int64_t r0 = wt.row0[blk] + kTileRows * w, r1 = wt.row1[blk];
  if (r0 >= r1) return;
  typename Mma<TX>::acc d[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) d[u] = (typename Mma<TX>::acc)(TX)0;
  tile_mul<TX, NT>(Lw, 4 * (int64_t)blk + w, val, x, ldr, c0, As[w], d);
  TX fi[4][NT];
#pragma unroll
  for (int i = 0; i < 4; ++i) load_nt<NT>(f + min(r0 + Mma<TX>::row(k4, i), r1 - 1) * ldr + c0 + NT * n, fi[i]);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t row = r0 + Mma<TX>::row(k4, i);
    if (row < r1) {
      TX yi[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) yi[u] = fi[i][u] - d[u][i];
      store_nt<NT>(y + row * ldr + c0 + NT * n, yi);
    }
  }
}

// r = f - (L + D) a in FP64 with partials r.r and f.f.
template <int NT>
__global__ void __launch_bounds__(kBlock, 4)
    k_mrt_residual(const WorkTable wt, int sub, const MrTiles D, const MrTiles Lw, const TileVals<double> dval,
                   const TileVals<double> lval, const double* a, const double* __restrict__ f,
                   float* __restrict__ rout, double* __restrict__ rrp, double* __restrict__ ffp, int ldr) {
  __shared__ TileLds<double> As[kBlock / kWave];
  __shared__ double sm[kBlock / kWave][16 * 4];
  const int id = xcd_block_id(gridDim.x);
  const int blk = id / sub, c0 = (id % sub) * 16 * NT;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int n = lane % 16, k4 = lane / 16;
  const int64_t r0 = wt.row0[blk] + kTileRows * w, r1 = wt.row1[blk];
  double prr[NT], pff[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) prr[u] = pff[u] = 0.0;
  if (r0 < r1) {
    md4 d[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) d[u] = (md4)0.0;
    tile_mul<double, NT>(Lw, 4 * (int64_t)blk + w, lval, a, ldr, c0, As[w], d);
    tile_mul<double, NT>(D, 4 * (int64_t)blk + w, dval, a, ldr, c0, As[w], d);
    double fi[4][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i) load_nt<NT>(f + min(r0 + Mma<double>::row(k4, i), r1 - 1) * ldr + c0 + NT * n, fi[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = r0 + Mma<double>::row(k4, i);
      if (row < r1) {
        double ri[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          ri[u] = fi[i][u] - d[u][i];
          prr[u] += ri[u] * ri[u];
          pff[u] += fi[i][u] * fi[i][u];
        }
        if (rout) {
          float r32[NT];
#pragma unroll
          for (int u = 0; u < NT; ++u) r32[u] = (float)ri[u];
          store_nt<NT>(rout + row * ldr + c0 + NT * n, r32);
        }
      }
    }
  }
  tile_partial<NT>(prr, sm, rrp, (size_t)blk * ldr + c0);
  tile_partial<NT>(pff, sm, ffp, (size_t)blk * ldr + c0);
}

template <typename TX>
static TileVals<TX> tile_vals(const MrTiles& T);
template <>
TileVals<float> tile_vals<float>(const MrTiles& T) {
  return TileVals<float>{T.val32};
}
template <>
TileVals<double> tile_vals<double>(const MrTiles& T) {
  return TileVals<double>{T.val, T.val32, T.lo};
}

template <typename TX>
void mr_tile_cg(mskm_hier* h, const MrTiles& D, int ldr, int chunk, int b0, int nb, const TX* p, TX* q,
                const int32_t* running, double* part) {
  if (nb <= 0) return;
  const int nt = mr_lane_rhs<TX>(ldr);
  // k_mrt_cg4 takes a block's tiles one after the other and 32-bit offsets into
  // p: from kWideBlocks workgroups on
  // (4,096 of them: 237 us against 256; 1,024: 22.6 against 20.1; 256: 18 against 9)
  constexpr int kWideBlocks = 2048;
  const int four = mr_cg_width<TX>(ldr);
  const bool wide = four > 16 * nt && (int64_t)nb * (ldr / four) >= kWideBlocks &&
                    (uint64_t)h->N * ldr * sizeof(TX) <= UINT32_MAX;
  const int width = wide ? four : 16 * nt;
  if (chunk % width || ldr % chunk) chunk = ldr;
  const int sub = chunk / width;
  const dim3 grid(nb * sub, ldr / chunk);
  hipStream_t s = h->ctx->stream;
  const TileVals<TX> v = tile_vals<TX>(D);
#define MSKM_MRT(K, NTV) \
  hipLaunchKernelGGL((K<TX, NTV>), grid, dim3(kBlock), 0, s, h->wt_spmv, b0, sub, D, v, p, q, ldr, running, part)
  if constexpr (sizeof(TX) == 4) {
    if (nt == 4) {
      if (wide)
        MSKM_MRT(k_mrt_cg4, 4);
      else
        MSKM_MRT(k_mrt_cg, 4);
      return;
    }
  }
  if (nt == 2 && wide)
    MSKM_MRT(k_mrt_cg4, 2);
  else if (nt == 2)
    MSKM_MRT(k_mrt_cg, 2);
  else
    MSKM_MRT(k_mrt_cg, 1);
#undef MSKM_MRT
}
template void mr_tile_cg<float>(mskm_hier*, const MrTiles&, int, int, int, int, const float*, float*, const int32_t*,
                                double*);
template void mr_tile_cg<double>(mskm_hier*, const MrTiles&, int, int, int, int, const double*, double*,
                                 const int32_t*, double*);

template <typename TX>
void mr_tile_lower(mskm_hier* h, const MrTiles& Lw, int ldr, int b0, int nb, const TX* x, const TX* f, TX* y) {
  if (nb <= 0) return;
  const int nt = mr_lane_rhs<TX>(ldr), sub = ldr / (16 * nt);
  const dim3 grid(nb * sub);
  hipStream_t s = h->ctx->stream;
  const TileVals<TX> v = tile_vals<TX>(Lw);
#define MSKM_MRT(NTV) \
  hipLaunchKernelGGL((k_mrt_lower<TX, NTV>), grid, dim3(kBlock), 0, s, h->wt_spmv, b0, sub, Lw, v, x, f, y, ldr)
  if constexpr (sizeof(TX) == 4) {
    if (nt == 4) {
      MSKM_MRT(4);
      return;
    }
  }
  if (nt == 2)
    MSKM_MRT(2);
  else
    MSKM_MRT(1);
#undef MSKM_MRT
}
template void mr_tile_lower<float>(mskm_hier*, const MrTiles&, int, int, int, const float*, const float*, float*);
template void mr_tile_lower<double>(mskm_hier*, const MrTiles&, int, int, int, const double*, const double*, double*);

void mr_tile_residual(mskm_hier* h, const MrTiles& D, const MrTiles& Lw, int ldr, const double* a, const double* f,
                      float* rout, double* rrp, double* ffp) {
  const int nt = mr_lane_rhs<double>(ldr), sub = ldr / (16 * nt);
  const dim3 grid((unsigned)h->wt_spmv.nblocks * sub);
  hipStream_t s = h->ctx->stream;
  const TileVals<double> dv = tile_vals<double>(D), lv = tile_vals<double>(Lw);
  if (nt == 2)
    hipLaunchKernelGGL(k_mrt_residual<2>, grid, dim3(kBlock), 0, s, h->wt_spmv, sub, D, Lw, dv, lv, a, f, rout, rrp,
                       ffp, ldr);
  else
    hipLaunchKernelGGL(k_mrt_residual<1>, grid, dim3(kBlock), 0, s, h->wt_spmv, sub, D, Lw, dv, lv, a, f, rout, rrp,
                       ffp, ldr);
}

}  // namespace mskm
