// Device helpers shared by the kernels of this library (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aires {
namespace kern {
namespace {

constexpr int WAVE = 64;

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Orders LDS traffic between the lanes of one wavefront (they execute in
// lockstep; this stops the compiler from moving LDS accesses across).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Cross-lane moves by DPP (data-parallel primitives of the GFX9 vector
// ALU, no LDS traffic): row_shr:n = 0x110 + n shifts within rows of 16
// lanes, row_bcast:15 = 0x142 and row_bcast:31 = 0x143 pass the last lane
// of a row (of two rows) on to the rows that ROW_MASK enables, wave_shr:1 =
// 0x138 shifts across the wavefront.  Lanes without a source read 0.
template <int CTRL, int ROW_MASK, typename T>
__device__ __forceinline__ T dpp_move(T x) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit lanes");
  if constexpr (sizeof(T) == 4) {
    return (T)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xf, false);
  } else {
    const uint64_t u = (uint64_t)x;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROW_MASK, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROW_MASK, 0xf, false);
    return (T)(((uint64_t)hi << 32) | lo);
  }
}

// Inclusive wavefront scan: Hillis-Steele steps 1, 2, 4, 8 inside rows of
// 16 lanes, then the row totals are carried to rows 1 and 3 and to rows 2
// and 3.  OP is + (SUM) or max (for non-negative values).
template <bool SUM, typename T>
__device__ __forceinline__ T wave_scan_op(T v) {
  auto op = [](T a, T b) { return SUM ? a + b : (a > b ? a : b); };
  v = op(v, dpp_move<0x111, 0xf>(v));
  v = op(v, dpp_move<0x112, 0xf>(v));
  v = op(v, dpp_move<0x114, 0xf>(v));
  v = op(v, dpp_move<0x118, 0xf>(v));
  v = op(v, dpp_move<0x142, 0xa>(v));
  v = op(v, dpp_move<0x143, 0xc>(v));
  return v;
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
  return wave_scan_op<true>(v);
}

// The value of lane 63 in every lane.
template <typename T>
__device__ __forceinline__ T wave_last(T x) {
  if constexpr (sizeof(T) == 4) {
    return (T)__builtin_amdgcn_readlane((int)x, WAVE - 1);
  } else {
    const uint64_t u = (uint64_t)x;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, WAVE - 1);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), WAVE - 1);
    return (T)(((uint64_t)hi << 32) | lo);
  }
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  return wave_last(wave_incl_scan(v));
}

// fp32 sum over the wavefront, in every lane (butterfly over lane pairs).
__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// C is written once and not read back by the kernels: stream it past the
// caches so that B's rows stay resident there.
template <typename T>
__device__ __forceinline__ void store_stream(T* p, T v) {
  __builtin_nontemporal_store(v, p);
}

template <typename RP>
__device__ __forceinline__ int64_t ld_rp(const void* rp, int64_t i) {
  return (int64_t)static_cast<const RP*>(rp)[i];
}

}  // namespace
}  // namespace kern
}  // namespace aires
