// Element types and small device helpers shared by the LiSA kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lisa {

// Storage tags.  bf16 is kept as its raw 16 bits; half is the native _Float16.
struct bf16_t { uint16_t bits; };
typedef _Float16 half_t;

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t bits) {
  return __uint_as_float(bits << 16);
}
// Round-to-nearest-even float -> bf16 bits (NaN kept quiet).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t x = __float_as_uint(f);
  if ((x & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;
  x += 0x7fffu + ((x >> 16) & 1u);
  return x >> 16;
}
// Saturating float -> half: scores beyond the half range are clamped to +-65504 instead
// of becoming infinities that would poison the softmax of the next layer.
__device__ __forceinline__ half_t f32_to_half_sat(float f) {
  return (half_t)__builtin_amdgcn_fmed3f(f, -65504.0f, 65504.0f);   // one median-of-three
}

template <typename T> struct elem;
template <> struct elem<float> {
  static __device__ __forceinline__ float load(const float* p) { return *p; }
  static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct elem<bf16_t> {
  static __device__ __forceinline__ float load(const bf16_t* p) { return bf16_bits_to_f32(p->bits); }
  static __device__ __forceinline__ void store(bf16_t* p, float v) { p->bits = (uint16_t)f32_to_bf16_bits(v); }
};
template <> struct elem<half_t> {
  static __device__ __forceinline__ float load(const half_t* p) { return (float)*p; }
  static __device__ __forceinline__ void store(half_t* p, float v) { *p = f32_to_half_sat(v); }
};

// Number of keys visible to query row i.
__device__ __host__ __forceinline__ int n_visible(int i, int Lq, int Lk, int causal) {
  if (!causal) return Lk;
  int n = i + 1 + (Lk - Lq);
  return n < 0 ? 0 : (n > Lk ? Lk : n);
}

// Reductions over a wave, the result in every lane: rotations inside the rows of 16 lanes (DPP), then the row
// swaps of gfx950.  All on the vector ALU: a reduction through the LDS crossbar (shuffles) waits for it six
// times, and short kernels spend most of their softmax there.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, true));
}
template <class Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
  v = op(v, dpp_move<0x128>(v));                             // row_ror:8, 4, 2, 1
  v = op(v, dpp_move<0x124>(v));
  v = op(v, dpp_move<0x122>(v));
  v = op(v, dpp_move<0x121>(v));
  const unsigned u = __float_as_uint(v);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const unsigned w = __float_as_uint(v);
  auto q = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return op(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_reduce(v, [](float a, float b) { return a + b; });
}

}  // namespace lisa
