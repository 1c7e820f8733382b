// Parts shared by the persistent CG kernels (cg_grid.hip, cg_stream.hip): words
// exchanged between workgroups through device-coherent memory.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <functional>

#include "mskm_internal.h"

namespace mskm {

constexpr int kGridThreads = 512;
constexpr int kGridSlot = 8;  // 64-byte slots

__device__ constexpr uint64_t kEmptySlot = 0x7ff4deadbeef0001ull;  // signalling NaN patterns: arithmetic never
__device__ constexpr uint32_t kEmptyWord = 0x7fa4beefu;            // produces them (results are quieted)

// Queues launch() on the context's stream behind the last persistent launch of
// any other context on the device: two of them partly resident at the same time
// would wait for workgroups that cannot start.
mskm_status cg_grid_in_turn(mskm_ctx* c, const std::function<void()>& launch);

// Order in which a row's products are added, that of the product which the
// launched kernels take for the same levels: an FP32 solve then rounds as they
// do, element by element. Entry order; the two halves of the two-waves-per-slice
// product (every other group of four); 4, 8 or 16 lanes' shares, lane i's being
// entries i, i + 4, ....
enum GridSum { kSumRow = 0, kSumHalves = 1, kSumLanes4 = 4, kSumLanes8 = 8, kSumLanes16 = 16 };

// The order of the launched kernels for levels lo..hi (FP32; FP64 results do not
// depend on it to the accuracy asked for). The products of the CSR copy with
// other widths than its default of 8 lanes, which only an autotuned or chosen
// product has, are taken for that one and differ in rounding.
int launched_sum(const mskm_hier* h, int lo, int hi, bool fp32);

// Empties z0, z1 (and z2) on the rows [r0, r0 + n) and ns slot words.
template <typename TX>
void grid_empty(hipStream_t s, TX* z0, TX* z1, TX* z2, int64_t r0, int64_t n, uint64_t* slots, int64_t ns);

// lane-crossing moves within 16 lanes
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;                 // quad permutations
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;       // within 8 and 16 lanes
template <int G, typename T>
__device__ __forceinline__ T lanes_sum(T v) {  // over G (a power of two, at most 16) neighbouring lanes
  if constexpr (G >= 2) v += dpp<kDppXor1>(v);
  if constexpr (G >= 4) v += dpp<kDppXor2>(v);
  if constexpr (G >= 8) v += dpp<kDppHalfMirror>(v);
  if constexpr (G >= 16) v += dpp<kDppMirror>(v);
  return v;
}
__device__ __forceinline__ double readlane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ __forceinline__ double wave64_sum(double v) {
  v = lanes_sum<16>(v);
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// Device-coherent words. A value whose bits are the empty pattern (it can
// only be a signalling NaN from the caller's data) is published quieted.
__device__ __forceinline__ uint32_t word_of(float v) {
  const uint32_t b = __float_as_uint(v);
  return b == kEmptyWord ? b | 0x00400000u : b;
}
__device__ __forceinline__ uint64_t word_of(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  return b == kEmptySlot ? b | 0x0008000000000000ull : b;
}
__device__ __forceinline__ float value_of(uint32_t b) { return __uint_as_float(b); }
__device__ __forceinline__ double value_of(uint64_t b) { return __longlong_as_double((long long)b); }
template <typename T>
struct GridWord;
template <>
struct GridWord<float> {
  using type = uint32_t;
  static constexpr uint32_t empty = kEmptyWord;
};
template <>
struct GridWord<double> {
  using type = uint64_t;
  static constexpr uint64_t empty = kEmptySlot;
};
template <typename W>
__device__ __forceinline__ void put(W* p, W v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename W>
__device__ __forceinline__ W get(const W* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The word at p once it is there; *bad after `left` further polls, and then none
// are left for the thread's next waits.
template <typename W>
__device__ __forceinline__ W poll(const W* p, W empty, int& left, int* bad) {
  W u = get(p);
  for (int k = 0; u == empty && k < left; ++k) u = get(p);
  if (u == empty) {
    *bad = 1;
    left = 0;
  }
  return u;
}

}  // namespace mskm
