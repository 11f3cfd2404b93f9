// Device helpers shared by the libmemattn kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace memattn {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Order-preserving map from fp32 to uint32: a < b (as floats, no NaN)
// exactly when f2ord(a) < f2ord(b).
__device__ __forceinline__ uint32_t f2ord(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ord2f(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

// Selection key: larger key = better candidate (score descending, then id
// ascending).  Key 0 marks an empty slot and is below every real candidate,
// including a score of -inf.
__device__ __forceinline__ uint64_t make_key(float s, uint32_t idx) {
  return (static_cast<uint64_t>(f2ord(s)) << 32) | static_cast<uint64_t>(0xFFFFFFFFu - idx);
}
__device__ __forceinline__ float key_score(uint64_t k) { return ord2f(static_cast<uint32_t>(k >> 32)); }

__device__ __forceinline__ uint32_t key_idx(uint64_t k) { return 0xFFFFFFFFu - static_cast<uint32_t>(k); }

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// Hardware base-2 exponential (v_exp_f32): exp2(-inf) = 0.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Write one selected key (slot r of query q) as id, score and probability;
// an empty key (fewer candidates than k) becomes id -1, score -inf, p 0.
__device__ __forceinline__ void write_selected(uint64_t key, float c2, float lse2, int64_t at, int32_t* idx,
                                               float* score, float* prob) {
  const bool have = key != 0;
  const float s = have ? key_score(key) : -INFINITY;
  idx[at] = have ? static_cast<int32_t>(key_idx(key)) : -1;
  if (score) score[at] = s;
  if (prob) prob[at] = have ? fast_exp2(s * c2 - lse2) : 0.f;
}

// Running softmax state in the log2 domain: m = max of x = scale*log2e*s
// seen so far, sum = sum of exp2(x - m).
struct SoftmaxState {
  float m;
  float sum;
};

// Reductions over a fully active wave, the same value in every lane: DPP steps
// combine each 16-lane row (lane ^ 1, lane ^ 2, then the half row and row
// mirrors), and the four rows' results are read out as scalars -- a few vector
// instructions instead of six dependent permutes through the LDS unit.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_f32(float x, int lane) {
  return __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(__float_as_uint(x)), lane)));
}
__device__ __forceinline__ float wave_max_f32(float x) {
  x = fmaxf(x, __uint_as_float(dpp_u32<0xB1>(__float_as_uint(x))));
  x = fmaxf(x, __uint_as_float(dpp_u32<0x4E>(__float_as_uint(x))));
  x = fmaxf(x, __uint_as_float(dpp_u32<0x141>(__float_as_uint(x))));
  x = fmaxf(x, __uint_as_float(dpp_u32<0x140>(__float_as_uint(x))));
  return fmaxf(fmaxf(lane_f32(x, 0), lane_f32(x, 16)), fmaxf(lane_f32(x, 32), lane_f32(x, 48)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint64_t lo = dpp_u32<CTRL>(static_cast<uint32_t>(u)), hi = dpp_u32<CTRL>(static_cast<uint32_t>(u >> 32));
  return __builtin_bit_cast(double, (hi << 32) | lo);
}
__device__ __forceinline__ double lane_f64(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(u)), lane));
  const uint64_t hi =
      static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(u >> 32)), lane));
  return __builtin_bit_cast(double, (hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum_f64(double x) {
  x += dpp_f64<0xB1>(x);
  x += dpp_f64<0x4E>(x);
  x += dpp_f64<0x141>(x);
  x += dpp_f64<0x140>(x);
  return (lane_f64(x, 0) + lane_f64(x, 16)) + (lane_f64(x, 32) + lane_f64(x, 48));
}

}  // namespace memattn
