// wave.h -- cross-lane primitives of a 64-lane wave, workgroup sums, and how
// records are read; shared by the device code (kernels.hip, filter.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "launch.h"

namespace sc {

constexpr int NWAVE = NT / 64;

// record fields from its two 64-bit halves (little-endian sim_record)
struct Rec {
  uint64_t unit;
  uint32_t tid, epoch, action, space;
};
__device__ __forceinline__ Rec unpack_rec(ulonglong2 v) {
  Rec r;
  r.unit = v.x;
  r.tid = (uint32_t)v.y;
  r.epoch = (uint32_t)(v.y >> 32) & 0xFFFFu;
  r.action = (uint32_t)(v.y >> 48) & 0xFFu;
  r.space = (uint32_t)(v.y >> 56);
  return r;
}


// Cross-lane moves of the wave's data-parallel primitives (DPP): the value
// of another lane, or 0 where that lane is outside the pattern or the row
// is masked off.  Row = 16 lanes.
enum : int {
  DPP_ROW_SHR1 = 0x111, DPP_ROW_SHR2 = 0x112, DPP_ROW_SHR4 = 0x114, DPP_ROW_SHR8 = 0x118,
  DPP_WAVE_SHR1 = 0x138,   // lane i gets lane i - 1
  DPP_ROW_BCAST15 = 0x142, // last lane of each row to the next row
  DPP_ROW_BCAST31 = 0x143  // lane 31 to rows 2 and 3
};
// (`old` instead of 0 where the source lane is outside the pattern.)
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp(uint32_t v, uint32_t old = 0u) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint64_t dpp(uint64_t v, uint64_t old = 0ull) {
  return ((uint64_t)dpp<CTRL, ROWS>((uint32_t)(v >> 32), (uint32_t)(old >> 32)) << 32) |
         dpp<CTRL, ROWS>((uint32_t)v, (uint32_t)old);
}

__device__ __forceinline__ uint32_t readlane(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ uint64_t readlane(uint64_t v, int lane) {
  return ((uint64_t)readlane((uint32_t)(v >> 32), lane) << 32) | readlane((uint32_t)v, lane);
}
__device__ __forceinline__ uint64_t readlane_key(uint64_t v, int lane) { return readlane(v, lane); }
__device__ __forceinline__ u128 readlane_key(u128 v, int lane) {
  return ((u128)readlane((uint64_t)(v >> 64), lane) << 64) | readlane((uint64_t)v, lane);
}
__device__ __forceinline__ uint64_t readfirstlane(uint64_t v) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

// Reduction over the 64 lanes with an associative, commutative operator
// whose identity is `id`: the scan pattern below ends with the total in
// lane 63, which every lane then reads.
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, T id, Op op) {
  v = op(dpp<DPP_ROW_SHR1>(v, id), v);
  v = op(dpp<DPP_ROW_SHR2>(v, id), v);
  v = op(dpp<DPP_ROW_SHR4>(v, id), v);
  v = op(dpp<DPP_ROW_SHR8>(v, id), v);
  v = op(dpp<DPP_ROW_BCAST15, 0xa>(v, id), v);
  v = op(dpp<DPP_ROW_BCAST31, 0xc>(v, id), v);
  return readlane(v, 63);
}
template <typename T>
__device__ __forceinline__ T wave_min(T v) {
  return wave_reduce(v, (T)~(T)0, [](T a, T b) { return a < b ? a : b; });
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
  return wave_reduce(v, (T)0, [](T a, T b) { return a > b ? a : b; });
}

// Inclusive scan over the 64 lanes of a wave with an associative operator
// whose identity is 0: within rows (shifts 1, 2, 4, 8), then across rows
// (row 0's total into row 1 and row 2's into row 3, then lane 31's into
// rows 2 and 3).
template <typename T, typename Op>
__device__ __forceinline__ T wave_incl_scan(T v, Op op) {
  v = op(dpp<DPP_ROW_SHR1>(v), v);
  v = op(dpp<DPP_ROW_SHR2>(v), v);
  v = op(dpp<DPP_ROW_SHR4>(v), v);
  v = op(dpp<DPP_ROW_SHR8>(v), v);
  v = op(dpp<DPP_ROW_BCAST15, 0xa>(v), v);
  v = op(dpp<DPP_ROW_BCAST31, 0xc>(v), v);
  return v;
}

// Exclusive sum over a workgroup of NW waves; *total receives the sum of all
// values.  Every thread of the workgroup must call it (it holds barriers).
template <int NW>
__device__ uint32_t block_excl_sum_n(uint32_t v, uint32_t* lds /* NW */, uint32_t* total) {
  const uint32_t lane = __lane_id(), wave = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan(v, [](uint32_t a, uint32_t b) { return a + b; });
  if (lane == 63) lds[wave] = inc;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; w++) {
    const uint32_t x = lds[w];
    if (w < (int)wave) pre += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return pre + inc - v;
}

__device__ __forceinline__ uint32_t block_excl_sum(uint32_t v, uint32_t* lds /* NWAVE */, uint32_t* total) {
  return block_excl_sum_n<NWAVE>(v, lds, total);
}

// A tile's records, read through the pointer its table entry holds.  To the
// compiler that pointer is generic, so it would load through flat
// instructions, and a flat load also holds up every wait for an LDS
// operation.  Records are always in memory the GPU addresses as global, so
// they are read as global memory.
typedef uint64_t rec_words __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) rec_words* GRecords;
__device__ __forceinline__ GRecords global_records(const void* p) { return (GRecords)p; }
__device__ __forceinline__ ulonglong2 load_record(GRecords p, uint32_t j) {
  const rec_words v = p[j];
  return ulonglong2{v.x, v.y};
}

}  // namespace sc
