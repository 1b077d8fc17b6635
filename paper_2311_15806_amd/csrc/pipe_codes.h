// Device side of the activation codes, shared by the quantizers (pipe_quant.hip) and the depthwise layer
// (pipe_depthwise.hip).  Q(x) = clamp(rint(x / s), ...) with the correctly rounded fp32 quotient, half to even.  Written
// in explicitly rounded operations, which a file compiled with contraction (pipe_gemv.hip) leaves apart as well: a rounded product is the factor or the addend of
// a written fma, never a bare sum's.
#pragma once
#include "pipe_internal.h"

constexpr int CODES_BLK = 256;   // workgroup size that block_max and max_of assume

__device__ __forceinline__ float block_max(float v) {
  __shared__ float sm[CODES_BLK / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sm[0];
#pragma unroll
  for (int i = 1; i < CODES_BLK / 64; ++i) r = fmaxf(r, sm[i]);
  __syncthreads();
  return r;
}

// max(v, v of the lane that the data-parallel move CTRL names); rows outside ROWS and lanes without a source keep theirs
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max(float v) {
  const int b = (int)__float_as_uint(v);
  return fmaxf(v, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(b, b, CTRL, ROWS, 0xf, false)));
}
// The largest of a wave's non-negative values, in every lane: moves within the vector unit instead of six trips through LDS
__device__ __forceinline__ float wave_max(float v) {
  v = dpp_max<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: the last lane of 16 holds their maximum
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);   // row_bcast 15, 31: lane 63 holds the wave's
  v = dpp_max<0x143, 0xc>(v);
  return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 63));
}

// The value of a slot, by a whole wave
__device__ __forceinline__ float slot_max(const uint32_t* slot) {
  float m = __uint_as_float(slot[(threadIdx.x & (PIPE_SLOT_LINES - 1)) * PIPE_SLOT_WORDS]);
#pragma unroll
  for (int o = PIPE_SLOT_LINES / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  return m;
}

// The value of a max reduction: the largest of its parts.  Called by all threads of a workgroup.
__device__ __forceinline__ float max_of(const MaxOf& a) {
  if (a.n == 0) return slot_max(a.p);
  if (a.n == 1) return __uint_as_float(a.p[0]);
  float m = 0.f;
  for (int i = threadIdx.x; i < a.n; i += CODES_BLK) m = fmaxf(m, __uint_as_float(a.p[i]));
  return block_max(m);
}

// Two of them, requested together (one after the other they cost the quantizer of 1000 x 768 affine codes a microsecond of its 6)
__device__ __forceinline__ void max_of_two(const MaxOf& a, const MaxOf& b, float* va, float* vb) {
  if (a.n <= 1 || a.n != b.n) {
    *va = max_of(a);
    *vb = max_of(b);
    return;
  }
  __shared__ float sm[2][CODES_BLK / 64];
  float m = 0.f, n = 0.f;
  for (int i = threadIdx.x; i < a.n; i += CODES_BLK) {
    m = fmaxf(m, __uint_as_float(a.p[i]));
    n = fmaxf(n, __uint_as_float(b.p[i]));
  }
  m = wave_max(m);
  n = wave_max(n);
  if ((threadIdx.x & 63) == 0) { sm[0][threadIdx.x >> 6] = m; sm[1][threadIdx.x >> 6] = n; }
  __syncthreads();
  m = sm[0][0]; n = sm[1][0];
#pragma unroll
  for (int i = 1; i < CODES_BLK / 64; ++i) { m = fmaxf(m, sm[0][i]); n = fmaxf(n, sm[1][i]); }
  *va = m;
  *vb = n;
}

// The same found by every wave for itself, all parts requested together, no barrier: for kernels of short workgroups that have
// registers to spare (128 images of 64 x 56 x 56, 1 x 1 convolution: 148 us with the reduction over the workgroup, 145 with this one; the
// linear layers' quantizer, with eight loads of x in flight, would drop from five waves per SIMD to four).
__device__ __forceinline__ float max_of_by_wave(const MaxOf& a) {
  if (a.n == 0) return slot_max(a.p);
  if (a.n == 1) return __uint_as_float(a.p[0]);
  const int lane = threadIdx.x & 63;
  float v[PIPE_MAX_PARTS / 64];
#pragma unroll
  for (int j = 0; j < PIPE_MAX_PARTS / 64; ++j) {
    v[j] = 0.f;
    if (64 * j < a.n) v[j] = __uint_as_float(a.p[min(64 * j + lane, a.n - 1)]);
  }
#pragma unroll
  for (int j = 1; j < PIPE_MAX_PARTS / 64; ++j) v[0] = fmaxf(v[0], v[j]);
  return wave_max(v[0]);
}

// Correctly rounded quotients by one divisor.  The compiler's IEEE division is about 11 instructions per element; with
// y = RN(1/s) at hand, Markstein's two corrections q' = RN(q + RN(v - s q) y) of a first guess give RN(v/s) in five (P.
// Markstein, "Computation of elementary functions on the IBM RISC System/6000 processor", 1990: exact remainder, and a
// correctly rounded result from a faithful q).  The remainder is exact while nothing underflows, hence the range of
// s (quotients below 1/4 in magnitude may be inexact: they round to code 0 either way).  v is bounded by 1024 s first, far
// beyond the largest code, so that no quotient or remainder is infinite; NaN becomes the lower bound, and thus the smallest
// code, which is what the clamp of the codes makes of a NaN quotient.
struct Divisor {
  float s, y, bound;
  bool fast;
  __device__ __forceinline__ explicit Divisor(float s_)
      : s(s_), y(__fdiv_rn(1.f, s_)), bound(1024.f * s_), fast(s_ > 1e-27f && s_ < 1e27f) {}
  template <bool FAST>
  __device__ __forceinline__ float quotient(float v) const {
    if (!FAST) return __fdiv_rn(v, s);
    v = __builtin_amdgcn_fmed3f(v, -bound, bound);
    float q = __fmul_rn(v, y);
    q = __fmaf_rn(__fmaf_rn(-q, s, v), y, q);
    return __fmaf_rn(__fmaf_rn(-q, s, v), y, q);
  }
};

__device__ __forceinline__ uint32_t pack4(int a, int b, int c, int d) {
  return (uint32_t)(uint8_t)a | ((uint32_t)(uint8_t)b << 8) | ((uint32_t)(uint8_t)c << 16) |
         ((uint32_t)(uint8_t)d << 24);
}
