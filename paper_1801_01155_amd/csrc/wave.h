// Wave-level (64 lanes) helpers for device code. All lanes must be active.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

__device__ inline int wave_lane() { return (int)(threadIdx.x & 63); }

// Inclusive scans over the wave by DPP moves (row shifts, then the rows' last
// lanes broadcast): six register-to-register steps. A cross-lane read through
// the LDS pipe takes more than ten times as long, and the scans are serial
// chains in every step of a ray.
template <int kCtrl, int kRows>
__device__ inline uint32_t dpp_or_0(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRows, 0xF, false);
}

__device__ inline uint32_t wave_incl_sum(uint32_t v) {
  v += dpp_or_0<0x111, 0xF>(v);   // row_shr 1, 2, 4, 8
  v += dpp_or_0<0x112, 0xF>(v);
  v += dpp_or_0<0x114, 0xF>(v);
  v += dpp_or_0<0x118, 0xF>(v);
  v += dpp_or_0<0x142, 0xA>(v);   // row_bcast 15 into rows 1 and 3
  v += dpp_or_0<0x143, 0xC>(v);   // row_bcast 31 into rows 2 and 3
  return v;
}

__device__ inline uint32_t wave_incl_max(uint32_t v) {
  v = max(v, dpp_or_0<0x111, 0xF>(v));
  v = max(v, dpp_or_0<0x112, 0xF>(v));
  v = max(v, dpp_or_0<0x114, 0xF>(v));
  v = max(v, dpp_or_0<0x118, 0xF>(v));
  v = max(v, dpp_or_0<0x142, 0xA>(v));
  v = max(v, dpp_or_0<0x143, 0xC>(v));
  return v;
}

__device__ inline uint32_t wave_excl_scan(uint32_t v, uint32_t& total) {
  const uint32_t inc = wave_incl_sum(v);
  total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  return inc - v;
}

// The next lane's value; `last` (wave-uniform) in lane 63.
__device__ inline int32_t wave_next(int32_t v, int32_t last) {
  return __builtin_amdgcn_update_dpp(last, v, 0x130, 0xF, 0xF, false);   // wave_shl 1
}

// Inclusive sum over the lanes [seg0, lane], seg0 the same for the lanes of one
// contiguous segment.
template <int kCtrl, int kRows>
__device__ inline float dpp_or_0f(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, kRows, 0xF, false));
}

__device__ inline float wave_seg_sum(float v, int seg0) {
  const int lane = wave_lane();
  float y;
  y = dpp_or_0f<0x111, 0xF>(v);
  v += lane - 1 >= seg0 ? y : 0.f;
  y = dpp_or_0f<0x112, 0xF>(v);
  v += lane - 2 >= seg0 ? y : 0.f;
  y = dpp_or_0f<0x114, 0xF>(v);
  v += lane - 4 >= seg0 ? y : 0.f;
  y = dpp_or_0f<0x118, 0xF>(v);
  v += lane - 8 >= seg0 ? y : 0.f;
  y = dpp_or_0f<0x142, 0xA>(v);   // the end of the row before, into rows 1 and 3
  v += seg0 < (lane & 48) ? y : 0.f;
  y = dpp_or_0f<0x143, 0xC>(v);   // lane 31, into rows 2 and 3
  v += seg0 < 32 ? y : 0.f;
  return v;
}

// Owner of pair base + lane among the wave's pairs (lane r owns [P_r, P_r +
// n_r), in lane order): each owner marks its first pair of the chunk in the
// wave's 64 words of LDS, and a running maximum spreads the marks.
__device__ inline int chunk_owner(uint32_t* own, uint32_t P, uint32_t n, uint32_t base) {
  const int lane = wave_lane();
  own[lane] = 0u;
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  if (n != 0u && P < base + 64u && P + n > base) own[P > base ? P - base : 0u] = (uint32_t)lane;
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  return (int)wave_incl_max(own[lane]);
}

// Bits [a, b) of a 64-bit mask (0 <= a, b <= 64; none if a >= b).
__device__ inline unsigned long long lane_range(int a, int b) {
  if (a >= b) return 0ull;
  const unsigned long long hi = b >= 64 ? ~0ull : ((1ull << b) - 1ull);
  return hi & ~((1ull << a) - 1ull);
}

// Pair w's lane in the chunk [base, base + 64): 0 before it, 64 after it. (A wave's
// pairs may number 2^31 and more.)
__device__ inline int chunk_lane(uint32_t w, uint32_t base) {
  return (int)min(__builtin_elementwise_sub_sat(w, base), 64u);
}

// The chunk's lanes that hold pairs [P, P + n).
__device__ inline unsigned long long chunk_lanes(uint32_t P, uint32_t n, uint32_t base) {
  return lane_range(chunk_lane(P, base), chunk_lane(P + n, base));
}

}  // namespace
