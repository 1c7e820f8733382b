// Tiles of the many-right-hand-side products (mr_tiles.hip).
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "mskm_internal.h"

namespace mskm {

// Rows of one tile and columns of one segment of a tile's entries.
constexpr int kTileRows = 16;
constexpr int kTileSeg = 64;

// One CSR matrix in tiles of 16 rows: tile 4 b + w holds rows 16 w .. of block
// b of the 64-row SpMV work table. A tile lists the distinct columns of its
// rows, ascending (but for their places within 16, tile_place), padded to a
// multiple of 16 with its last column; its entries are grouped by segments of 64
// listed columns, each with its row and place in the list.
struct MrTiles {
  int64_t ntile = 0, nseg = 0, ncol = 0, nnz = 0;
  int64_t* cptr = nullptr;   // [ntile + 1] first listed column
  int32_t* cols = nullptr;   // [ncol]
  int64_t* sptr = nullptr;   // [ntile + 1] first segment
  int64_t* eptr = nullptr;   // [nseg + 1] first entry of each segment
  uint16_t* code = nullptr;  // [nnz] row << 7 | place % 128
  double* val = nullptr;     // [nnz] values in tile order, as stored by the hierarchy
  float* val32 = nullptr;
  float* lo = nullptr;
};

// The tiles of a hierarchy's blocks, built at the first call that needs them;
// *out is null where they are not available (a tile with more than 65536
// columns, or no memory): the caller takes the general products.
mskm_status mr_tiles(mskm_hier* h, bool lower, const MrTiles** out);
bool mr_tiles_built(const mskm_hier* h);  // both matrices' tiles are there

// Right-hand sides are padded to a width that the tiles' products take: 16,
// or a multiple of 32 (the padding solves zero systems, which stop at once).
// Refined mixed solves, row by row in their own width and padded (first call, with
// the tiles' build), in ms: two right-hand sides on 87,000 points 151 and 7.8 (15), on
// 1,398,080 729 and 138 (151), on 300,000 in 3-D 414 and 89 (92); nine 235 and 22 (23),
// 1,059 and 151 (164), 729 and 109 (111). The price is memory: 48 bytes a row and
// padded right-hand side in a mixed solve.
inline int mr_width(int nrhs) { return nrhs <= 16 ? 16 : (nrhs + 31) / 32 * 32; }

// q = A p on the blocks [b0, b0 + nb) of the SpMV work table with partials p.q
// part[block][ldr], A the diagonal blocks' tiles, p and q [N][ldr]; levels
// with running[l] = 0 are skipped. The right-hand sides go in slices of `chunk`
// (the slowest launch dimension; a multiple of mr_cg_width dividing ldr, or ldr).
template <typename TX>
void mr_tile_cg(mskm_hier* h, const MrTiles& D, int ldr, int chunk, int b0, int nb, const TX* p, TX* q,
                const int32_t* running, double* part);
// y = f - L x on blocks [b0, b0 + nb), L the lower blocks' tiles.
template <typename TX>
void mr_tile_lower(mskm_hier* h, const MrTiles& Lw, int ldr, int b0, int nb, const TX* x, const TX* f, TX* y);
// r = f - (L + D) a in FP64 over the whole work table, partials r.r and f.f
// [block][ldr]; rout (nullable) receives r rounded to FP32.
void mr_tile_residual(mskm_hier* h, const MrTiles& D, const MrTiles& Lw, int ldr, const double* a, const double* f,
                      float* rout, double* rrp, double* ffp);

// Right-hand sides per lane of the many-right-hand-side kernels: 16 bytes, as
// far as the width is a multiple of 16 lanes' worth.
template <typename TX>
inline int mr_lane_rhs(int ldr) {
  if (sizeof(TX) == 4 && ldr % 64 == 0) return 4;
  return ldr % 32 == 0 ? 2 : 1;
}

// Right-hand sides of one workgroup of mr_tile_cg, which its chunks are
// multiples of: four waves' slices where the width has whole groups of them
// (k_mrt_cg4), else one.
template <typename TX>
inline int mr_cg_width(int ldr) {
  const int one = 16 * mr_lane_rhs<TX>(ldr);
  return one >= 32 && ldr % (4 * one) == 0 ? 4 * one : one;
}

// ------------------------------------------------------------ device helpers

typedef float mf4 __attribute__((ext_vector_type(4)));
typedef double md4 __attribute__((ext_vector_type(4)));
typedef int mi4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Mma;
template <>
struct Mma<float> {
  using acc = mf4;
  static constexpr int kCols = 128, kStride = kCols + 4;  // columns of the tile in LDS, row stride
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int k, int i) { return 4 * k + i; }  // of accumulator element i
  // operand row n for which element i of lane (., k) becomes row k + 4 i
  static __device__ __forceinline__ int spread(int n) { return n / 4 + 4 * (n % 4); }
};
template <>
struct Mma<double> {
  using acc = md4;
  static constexpr int kCols = 64, kStride = kCols + 2;
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int k, int i) { return k + 4 * i; }
  static __device__ __forceinline__ int spread(int n) { return n; }
};

template <typename T, int NT>
struct VecN {
  typedef T type __attribute__((ext_vector_type(NT)));
};
template <typename T>
struct VecN<T, 1> {
  typedef T type;
};
template <int NT, typename T>
__device__ __forceinline__ void load_nt(const T* p, T (&v)[NT]) {
  const typename VecN<T, NT>::type u = *reinterpret_cast<const typename VecN<T, NT>::type*>(p);
  if constexpr (NT == 1) {
    v[0] = u;
  } else {
#pragma unroll
    for (int q = 0; q < NT; ++q) v[q] = u[q];
  }
}
template <int NT, typename T>
__device__ __forceinline__ void store_nt(T* p, const T (&v)[NT]) {
  typename VecN<T, NT>::type u;
  if constexpr (NT == 1) {
    u = v[0];
  } else {
#pragma unroll
    for (int q = 0; q < NT; ++q) u[q] = v[q];
  }
  *reinterpret_cast<typename VecN<T, NT>::type*>(p) = u;
}

}  // namespace mskm
