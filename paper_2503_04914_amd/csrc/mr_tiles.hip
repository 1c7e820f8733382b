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
// columns, lane (n, k) reads entries A[n][4 k .. 4 k + 3] of the tile (LDS) and
// NT consecutive right-hand sides NT n .. of the four rows of X that belong to
// columns 4 k .. 4 k + 3 (one vector load each, 256 contiguous bytes per 16
// lanes): 4 NT matrix instructions, the j-th on columns {4 k + j}, right-hand
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
      int64_t at = c0 + listed + rank[w];
      while (m) {
        T.cols[at++] = base + 32 * w + __ffs(m) - 1;
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
  for (int q = n + t; q < nc; q += kBlock) T.cols[c0 + q] = T.cols[c0 + n - 1];
  tile_windows(e0, e1, col, bits, rank, red, [&](int base, int listed) {
    for (int64_t k = e0 + t; k < e1; k += kBlock) {
      int pos;
      if (!place(k, base, listed, pos)) continue;
      int row = 0;  // the last row starting at or before entry k
      for (int b = kTileRows / 2; b > 0; b >>= 1)
        if (r0 + row + b < r1 && rp[r0 + row + b] <= k) row += b;
      const int64_t at = e0 + atomicAdd(&hist[pos / kTileSeg], 1);
      T.code[at] = (uint16_t)(row << 7 | (pos & 127));
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
  MSKM_TRY(halloc(h, &T.cols, (size_t)T.ncol));
  MSKM_TRY(halloc(h, &T.eptr, (size_t)T.nseg + 1));
  MSKM_TRY(halloc(h, &T.code, (size_t)T.nnz));
  if (A.val) MSKM_TRY(halloc(h, &T.val, (size_t)T.nnz));
  if (A.val32) MSKM_TRY(halloc(h, &T.val32, (size_t)T.nnz));
  if (A.val32lo) MSKM_TRY(halloc(h, &T.lo, (size_t)T.nnz));
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

// Value of entry e in the product's precision.
template <typename T>
struct TileVals;
template <>
struct TileVals<float> {
  const float* v;
  __device__ __forceinline__ float operator()(int64_t e) const { return v[e]; }
};
template <>
struct TileVals<double> {
  const double* v;
  const float *hi, *lo;  // without FP64 values: FP32 value + remainder
  __device__ __forceinline__ double operator()(int64_t e) const { return v ? v[e] : (double)hi[e] + (double)lo[e]; }
};

// d += tile * X for right-hand sides c0 + NT n + q; As: the wave's LDS.
template <typename TX, int NT>
__device__ __forceinline__ void tile_mul(const MrTiles& T, int64_t tile, const TileVals<TX>& val,
                                         const TX* __restrict__ x, int ldr, int c0, TX* As,
                                         typename Mma<TX>::acc (&d)[NT]) {
  constexpr int CH = Mma<TX>::kCols, ST = Mma<TX>::kStride;
  const int lane = threadIdx.x % kWave, n = lane % 16, k4 = lane / 16;
  const int64_t s0 = T.sptr[tile], s1 = T.sptr[tile + 1], cb = T.cptr[tile];
  const int nc = (int)(T.cptr[tile + 1] - cb);
  const TX* xc = x + c0 + NT * n;
  for (int ch = 0; ch * CH < nc; ++ch) {
    const int steps = min(CH, nc - ch * CH) / 16;
    const int32_t* cl = T.cols + cb + ch * CH + 4 * k4;
    // rows of X of the first step, columns of the second
    mi4 c = *reinterpret_cast<const mi4*>(cl);
    TX b[4][NT];
#pragma unroll
    for (int j = 0; j < 4; ++j) load_nt<NT>(xc + (int64_t)c[j] * ldr, b[j]);
    if (steps > 1) c = *reinterpret_cast<const mi4*>(cl + 16);
    // the tile's columns of this pass
    typedef typename VecN<TX, 16 / sizeof(TX)>::type zvec;
    for (int z = lane; z < kTileRows * ST * (int)sizeof(TX) / 16; z += kWave) reinterpret_cast<zvec*>(As)[z] = (zvec)(TX)0;
    __builtin_amdgcn_wave_barrier();
    const int64_t ea = T.eptr[s0 + ch * (CH / kTileSeg)];
    const int64_t ee = T.eptr[min(s0 + (ch + 1) * (CH / kTileSeg), s1)];
    for (int64_t e = ea + lane; e < ee; e += kWave) {
      const int cd = T.code[e];
      As[(cd >> 7) * ST + (cd & (CH - 1))] = val(e);
    }
    __builtin_amdgcn_wave_barrier();
    const TX* Ar = As + n * ST + 4 * k4;
    for (int s = 0; s < steps; ++s) {
      TX a[4], bn[4][NT];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = Ar[16 * s + j];
      if (s + 1 < steps) {
#pragma unroll
        for (int j = 0; j < 4; ++j) load_nt<NT>(xc + (int64_t)c[j] * ldr, bn[j]);
        if (s + 2 < steps) c = *reinterpret_cast<const mi4*>(cl + 16 * (s + 2));
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < NT; ++q) d[q] = Mma<TX>::mul(a[j], b[j][q], d[q]);
      if (s + 1 < steps) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int q = 0; q < NT; ++q) b[j][q] = bn[j][q];
      }
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
__global__ void __launch_bounds__(kBlock)
    k_mrt_cg(const WorkTable wt, int base, int sub, const MrTiles D, const TileVals<TX> val, const TX* __restrict__ p,
             TX* __restrict__ q, int ldr, const int32_t* __restrict__ running, double* __restrict__ part) {
  __shared__ TX As[kBlock / kWave][kTileRows * Mma<TX>::kStride];
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
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = r0 + Mma<TX>::row(k4, i);
      if (row < r1) {
        TX pi[NT], qi[NT];
        load_nt<NT>(p + row * ldr + c0 + NT * n, pi);
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          qi[u] = d[u][i];
          acc[u] += (double)pi[u] * (double)qi[u];
        }
        store_nt<NT>(q + row * ldr + c0 + NT * n, qi);
      }
    }
  }
  tile_partial<NT>(acc, sm, part, (size_t)blk * ldr + c0);
}

// y = f - L x.
template <typename TX, int NT>
__global__ void __launch_bounds__(kBlock)
    k_mrt_lower(const WorkTable wt, int base, int sub, const MrTiles Lw, const TileVals<TX> val,
                const TX* __restrict__ x, const TX* __restrict__ f, TX* __restrict__ y, int ldr) {
  __shared__ TX As[kBlock / kWave][kTileRows * Mma<TX>::kStride];
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
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t row = r0 + Mma<TX>::row(k4, i);
    if (row < r1) {
      TX fi[NT], yi[NT];
      load_nt<NT>(f + row * ldr + c0 + NT * n, fi);
#pragma unroll
      for (int u = 0; u < NT; ++u) yi[u] = fi[u] - d[u][i];
      store_nt<NT>(y + row * ldr + c0 + NT * n, yi);
    }
  }
}

// r = f - (L + D) a in FP64 with partials r.r and f.f.
template <int NT>
__global__ void __launch_bounds__(kBlock)
    k_mrt_residual(const WorkTable wt, int sub, const MrTiles D, const MrTiles Lw, const TileVals<double> dval,
                   const TileVals<double> lval, const double* __restrict__ a, const double* __restrict__ f,
                   float* __restrict__ rout, double* __restrict__ rrp, double* __restrict__ ffp, int ldr) {
  __shared__ double As[kBlock / kWave][kTileRows * Mma<double>::kStride];
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
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = r0 + Mma<double>::row(k4, i);
      if (row < r1) {
        double fi[NT], ri[NT];
        load_nt<NT>(f + row * ldr + c0 + NT * n, fi);
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          ri[u] = fi[u] - d[u][i];
          prr[u] += ri[u] * ri[u];
          pff[u] += fi[u] * fi[u];
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
  const int nt = mr_lane_rhs<TX>(ldr), width = 16 * nt;
  if (chunk % width || ldr % chunk) chunk = ldr;
  const int sub = chunk / width;
  const dim3 grid(nb * sub, ldr / chunk);
  hipStream_t s = h->ctx->stream;
  const TileVals<TX> v = tile_vals<TX>(D);
#define MSKM_MRT(NTV)                                                                                             \
  hipLaunchKernelGGL((k_mrt_cg<TX, NTV>), grid, dim3(kBlock), 0, s, h->wt_spmv, b0, sub, D, v, p, q, ldr, running, \
                     part)
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
