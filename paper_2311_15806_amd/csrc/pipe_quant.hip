// Activation quantization (App. B, Eq. (define_dre): Q(x) with a per-tensor scale lambda_x):
// absmax reduction, fp32 -> int8 into the fragment layout with per-token code sums, the
// im2col variant for convolutions, and the element-wise hidden activation of the MLP call.
//
// Q(x) = clamp(rint(x / s_x), -127, 127) with an IEEE fp32 division and round-half-to-even;
// this file is compiled with floating-point contraction off.
#include "pipe_codes.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int BLK = CODES_BLK;

__global__ void zero_u32_kernel(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// Shows every float4 of x4[0..n4) from x4[i] on, `stride` apart, to take() at least once, N 16-byte loads in flight to the end: for a
// maximum, the last one may stand in for those behind it (what was left of eight used to be loaded one by one: 333 x 4096, 7.98 loads a
// thread, 4.8 -> 4.0 us; sixteen in flight, or two sets of eight in turn, change nothing: 4096 x 4096 at 17 us).
template <int N, class Take>
__device__ __forceinline__ void scan4(const float4* __restrict__ x4, int64_t n4, int64_t i, int64_t stride, Take take) {
  for (; i < n4; i += N * stride) {
    float4 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = x4[min(i + u * stride, n4 - 1)];
#pragma unroll
    for (int u = 0; u < N; ++u) take(v[u]);
  }
}
__device__ __forceinline__ float absmax4(const float4& v) {
  return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)));
}

// max|x| over n elements, one value per workgroup (the quantizer that follows takes the maximum of them: a slot that all
// workgroups raise by atomics costs about 20 ns for each, 20 -> 31 -> 39 us for 256, 1024 and 2048 workgroups over 64 MiB);
// the maximum is order independent, so the result is exact.
// Also clears the per-token code sums the quantizer that follows accumulates into.
__global__ __launch_bounds__(BLK) void absmax_kernel(const float* __restrict__ x, int64_t n,
                                                     uint32_t* __restrict__ part,
                                                     int32_t* __restrict__ zero_me, int n_zero) {
  for (int i = blockIdx.x * BLK + threadIdx.x; i < n_zero; i += gridDim.x * BLK) zero_me[i] = 0;
  float m = 0.f;
  const int64_t stride = (int64_t)gridDim.x * BLK;
  const int64_t i0 = (int64_t)blockIdx.x * BLK + threadIdx.x;
  if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
    const int64_t n4 = n >> 2;
    scan4<8>(reinterpret_cast<const float4*>(x), n4, i0, stride, [&](const float4& v) { m = fmaxf(m, absmax4(v)); });
    for (int64_t i = (n4 << 2) + i0; i < n; i += stride) m = fmaxf(m, fabsf(x[i]));
  } else {
    for (int64_t i = i0; i < n; i += stride) m = fmaxf(m, fabsf(x[i]));
  }
  m = block_max(m);
  if (threadIdx.x == 0) part[blockIdx.x] = __float_as_uint(m);
}

// Largest activation code 2^(a-1)-1: 127 for int8 activations, 31 / 7 for 6 / 4 bits (the codes
// still travel as bytes).  Set by pipe_set_activation_bits through set_act_qmax below.
__constant__ float c_act_qmax = 127.f;

__device__ __forceinline__ float act_scale(float s_static, const MaxOf& amax) {
  if (s_static > 0.f) return s_static;
  return __fdiv_rn(max_of(amax), c_act_qmax);
}

// Q(x), symmetric: code = clamp(rint(x / s), -qmax, qmax)
struct SymCodes {
  Divisor d;
  float qmax;
  __device__ __forceinline__ explicit SymCodes(float s) : d(s), qmax(c_act_qmax) {}
  __device__ __forceinline__ bool live() const { return d.s > 0.f; }
  template <bool FAST>
  __device__ __forceinline__ int code(float v) const {
    return (int)fminf(fmaxf(rintf(d.quotient<FAST>(v)), -qmax), qmax);
  }
  int8_t* rows = nullptr;   // row-major copy of the codes, or nullptr
  __device__ __forceinline__ void row_major(int t, int k0, int T, int in, const int (&q)[16]) const {
    if (rows == nullptr || t >= T) return;
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (k0 + e < in) rows[(size_t)t * in + k0 + e] = (int8_t)q[e];
  }
};

__device__ __forceinline__ int quant1(float v, float s) {
  float q = rintf(__fdiv_rn(v, s));
  q = fminf(fmaxf(q, -c_act_qmax), c_act_qmax);
  return (int)q;
}

// One block: token block blockIdx.x (16 tokens), a range of 16-wide k-chunks given by
// blockIdx.y (whole 64-k steps).  FETCH(t, k) returns the fp32 activation (0 outside the valid
// region).  Rows that can be read 16 bytes at a time (xvec) take the wide path for every 64-k step
// that lies inside the row: a wave owns 16 tokens x 64 k, one load instruction reads 256 contiguous bytes of 4 rows
// (lane = row lane >> 4, 16 bytes lane & 15), the codes are turned through 1.25 KiB of LDS per wave and leave as one
// store of the whole 1-KiB fragment.  Everything else (ragged tail, padding, gathers) goes
// through the generic path: thread = (token tid & 15, chunk slot tid >> 4).
// MAKE() returns the quantizer (SymCodes, AsymCodes) once the scale is known; it is called by all threads, behind the
// first requests for x.
template <class Make, class Fetch>
__device__ __forceinline__ void quantize_block(Make make, Fetch fetch, int T, int in, int in_pad,
                                               uint8_t* __restrict__ qx_frag, int32_t* __restrict__ rowsum,
                                               const float* __restrict__ xvec) {
  const int tb = blockIdx.x;
  const int nks = in_pad >> 6;
  const int nchunk = in_pad >> 4;
  const int per = ((nchunk + (int)gridDim.y - 1) / (int)gridDim.y + 3) & ~3;
  const int c_lo = min(nchunk, (int)blockIdx.y * per);
  const int c_hi = min(nchunk, c_lo + per);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int NWAVE = BLK / 64;
  constexpr int STEPS = 2;       // 64-k steps of a wave requested together: eight 16-byte loads per lane in flight
  __shared__ uint4 turn[NWAVE][2][80];   // a fragment: 64-k quarter kc at kc * 320 bytes (no bank conflicts either way)
  __shared__ int wsum[2][NWAVE][16];

  // wide path
  const int r4 = lane >> 4, c4 = lane & 15;
  const int c_wide = xvec != nullptr ? max(c_lo, min(c_hi, (in >> 6) << 2)) : c_lo;
  const int ks_hi = c_wide >> 2;
  int ks = (c_lo >> 2) + wave;
  const float* row[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) row[i] = xvec + (size_t)min(tb * 16 + 4 * i + r4, T - 1) * in + c4 * 4;
  float4 f[STEPS][4];
  auto load_steps = [&]() {
#pragma unroll
    for (int u = 0; u < STEPS; ++u)
      if (ks + u * NWAVE < ks_hi) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[u][i] = *reinterpret_cast<const float4*>(row[i] + (ks + u * NWAVE) * 64);
      }
  };
  load_steps();
  const auto cd = make();
  const bool live = cd.live();
  int sum_w[4] = {0, 0, 0, 0};   // rows 4*i + (lane >> 4)
  auto walk = [&](auto fast) {
    constexpr bool FAST = decltype(fast)::value;
    uint8_t* dst = qx_frag + (size_t)tb * nks * 1024 + lane * 16;
    while (ks < ks_hi) {
#pragma unroll
      for (int u = 0; u < STEPS; ++u) {
        if (ks + u * NWAVE >= ks_hi) break;
        uint8_t* tw = reinterpret_cast<uint8_t*>(turn[wave][u & 1]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          int q0 = 0, q1 = 0, q2 = 0, q3 = 0;
          if (live && tb * 16 + 4 * i + r4 < T) {
            q0 = cd.template code<FAST>(f[u][i].x); q1 = cd.template code<FAST>(f[u][i].y);
            q2 = cd.template code<FAST>(f[u][i].z); q3 = cd.template code<FAST>(f[u][i].w);
          }
          sum_w[i] += q0 + q1 + q2 + q3;
          *reinterpret_cast<uint32_t*>(tw + (c4 >> 2) * 320 + (4 * i + r4) * 16 + (c4 & 3) * 4) = pack4(q0, q1, q2, q3);
        }
        __builtin_amdgcn_wave_barrier();   // a wave's own LDS accesses stay in order: enough between the turn's halves
        *reinterpret_cast<uint4*>(dst + (size_t)(ks + u * NWAVE) * 1024) = turn[wave][u & 1][(lane >> 4) * 20 + (lane & 15)];
        __builtin_amdgcn_wave_barrier();
      }
      ks += STEPS * NWAVE;
      load_steps();
    }
  };

  // generic path
  const int n = threadIdx.x & 15;
  const int t = tb * 16 + n;
  int sum = 0;
  auto rest = [&](auto fast) {
    constexpr bool FAST = decltype(fast)::value;
    for (int c = c_wide + (threadIdx.x >> 4); c < c_hi; c += BLK / 16) {
      int q[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = c * 16 + e;
        int v = 0;
        if (live && t < T && k < in) v = cd.template code<FAST>(fetch(t, k));
        q[e] = v;
        sum += v;
      }
      const int ks = c >> 2, kc = c & 3;
      uint4 w = make_uint4(pack4(q[0], q[1], q[2], q[3]), pack4(q[4], q[5], q[6], q[7]),
                           pack4(q[8], q[9], q[10], q[11]), pack4(q[12], q[13], q[14], q[15]));
      *reinterpret_cast<uint4*>(qx_frag + (((size_t)tb * nks + ks) * 64 + kc * 16 + n) * 16) = w;
      cd.row_major(t, c * 16, T, in, q);
    }
  };
  if (cd.d.fast) { walk(std::true_type{}); rest(std::true_type{}); }
  else { walk(std::false_type{}); rest(std::false_type{}); }
  // one atomic per token and workgroup.  Generic path: threads 16 apart hold the same token
  // (lane bits 4 and 5); wide path: the 16 lanes of a row; then the waves through LDS.
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) sum_w[i] += __shfl_xor(sum_w[i], o, 64);
  if (lane < 16) wsum[0][wave][lane] = sum;
  if ((lane & 15) == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) wsum[1][wave][4 * i + (lane >> 4)] = sum_w[i];
  }
  __syncthreads();
  if (threadIdx.x < 16) {
    int tot = 0;
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) tot += wsum[0][w][threadIdx.x] + wsum[1][w][threadIdx.x];
    if (t < T && tot != 0) atomicAdd(&rowsum[t], tot);
  }
}

// blockIdx.z = ensemble member: member m reads x + m*x_mstride with the scale slot m, and writes
// its own fragment buffer, code sums and scale.
__global__ __launch_bounds__(BLK) void quantize_act_kernel(const float* __restrict__ x_all, int64_t x_mstride, int T, int in,
                                                           int in_pad, float s_static, MaxOf amax,
                                                           uint8_t* __restrict__ qx_all, int64_t qx_mstride,
                                                           int32_t* __restrict__ rowsum_all, int rowsum_mstride,
                                                           int8_t* __restrict__ qx_rowmajor,
                                                           float* __restrict__ scale_out) {
  const int m = blockIdx.z;
  const float* x = x_all + (size_t)m * x_mstride;
  auto make = [&]() {
    const float s = act_scale(s_static, MaxOf{amax.p + m, amax.n});   // (parts: one member only)
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && scale_out) scale_out[m] = s;
    SymCodes cd(s);
    cd.rows = qx_rowmajor;
    return cd;
  };
  auto fetch = [=](int t, int k) { return x[(size_t)t * in + k]; };
  const bool vec = (in & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 && qx_rowmajor == nullptr;
  quantize_block(make, fetch, T, in, in_pad, qx_all + (size_t)m * qx_mstride, rowsum_all + (size_t)m * rowsum_mstride, vec ? x : nullptr);
}

// Decode-sized batches (up to 64 tokens): ONE launch does max|x|, scale, codes and code sums, so the
// forward path is two launches (this one and the contraction).  Workgroup (n, m) owns token n
// of member m: it first reduces max|x| over the member's whole input (every workgroup does,
// redundantly -- the input is a few hundred KiB and L2 resident, and it spares a grid-wide
// synchronization), then quantizes its own token and sums its codes without atomics.
constexpr int SBLK = 1024;   // a large workgroup: the scan for the maximum is the long part
__global__ __launch_bounds__(SBLK) void quantize_small_kernel(const float* __restrict__ x_all, int64_t x_mstride,
                                                              int T, int in, int in_pad, float s_static,
                                                              const uint32_t* __restrict__ amax_bits,
                                                              uint8_t* __restrict__ qx_all, int64_t qx_mstride,
                                                              int32_t* __restrict__ rowsum_all,
                                                              int8_t* __restrict__ qx_rowmajor,
                                                              float* __restrict__ scale_out) {
  const int n = blockIdx.x;      // token 0..T_pad-1 (T_pad = gridDim.x, a multiple of 16)
  const int nks = in_pad >> 6;
  const int m = blockIdx.y;
  const float* x = x_all + (size_t)m * x_mstride;
  uint8_t* qx_frag = qx_all + (size_t)m * qx_mstride;
  __shared__ float smax[SBLK / 64];
  __shared__ int ssum[SBLK / 64];
  float s = s_static;
  if (!(s_static > 0.f) && amax_bits != nullptr) {
    // the producer of x already reduced max|x| of member m
    s = __fdiv_rn(slot_max(&amax_bits[m]), c_act_qmax);
  } else if (!(s_static > 0.f)) {
    float mx = 0.f;
    const int64_t cnt = (int64_t)T * in;
    if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
      const int64_t n4 = cnt >> 2;
      // (every workgroup reads everything: eight loads for the last one or two would take 2 x 3072 from 4.3 to 4.9 us)
      const int64_t eights = (n4 + 6 * SBLK - 1) / (8 * SBLK) * (8 * SBLK);   // in batches of eight but for a rest of up to two a thread
      const float4* x4 = reinterpret_cast<const float4*>(x);
      auto take = [&](const float4& v) { mx = fmaxf(mx, absmax4(v)); };
      scan4<8>(x4, min(eights, n4), threadIdx.x, SBLK, take);
      scan4<2>(x4, n4, eights + threadIdx.x, SBLK, take);
      for (int64_t j = (n4 << 2) + threadIdx.x; j < cnt; j += SBLK) mx = fmaxf(mx, fabsf(x[j]));
    } else {
      for (int64_t j = threadIdx.x; j < cnt; j += SBLK) mx = fmaxf(mx, fabsf(x[j]));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = smax[0];
#pragma unroll
    for (int i = 1; i < SBLK / 64; ++i) mx = fmaxf(mx, smax[i]);
    s = __fdiv_rn(mx, c_act_qmax);
  }
  if (n == 0 && threadIdx.x == 0 && scale_out) scale_out[m] = s;
  const bool live = s > 0.f && n < T;
  const int nchunk = in_pad >> 4;
  const bool vec = (in & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
  int sum = 0;
  for (int c = threadIdx.x; c < nchunk; c += SBLK) {
    int q[16];
    if (live && vec && c * 16 + 15 < in) {
      const float4* row = reinterpret_cast<const float4*>(x + (size_t)n * in + c * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float4 v = row[e];
        q[4 * e] = quant1(v.x, s); q[4 * e + 1] = quant1(v.y, s); q[4 * e + 2] = quant1(v.z, s); q[4 * e + 3] = quant1(v.w, s);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) q[e] = (live && c * 16 + e < in) ? quant1(x[(size_t)n * in + c * 16 + e], s) : 0;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) sum += q[e];
    const int ks = c >> 2, kc = c & 3;
    const uint4 w = make_uint4(pack4(q[0], q[1], q[2], q[3]), pack4(q[4], q[5], q[6], q[7]),
                               pack4(q[8], q[9], q[10], q[11]), pack4(q[12], q[13], q[14], q[15]));
    *reinterpret_cast<uint4*>(qx_frag + (((size_t)(n >> 4) * nks + ks) * 64 + kc * 16 + (n & 15)) * 16) = w;
    if (qx_rowmajor != nullptr && n < T) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (c * 16 + e < in) qx_rowmajor[(size_t)n * in + c * 16 + e] = (int8_t)q[e];
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) ssum[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
#pragma unroll
    for (int i = 0; i < SBLK / 64; ++i) tot += ssum[i];
    rowsum_all[(size_t)m * gridDim.x + n] = tot;
  }
}

struct ConvGeom {
  int N, C, H, W, kh, kw, stride, pad, nhwc, Ho, Wo;
};

// Convolution input, step 1: every input element is quantized once, in the input's own layout
// (an element appears in up to kh*kw patches; the IEEE division is paid once, not per patch).
__global__ __launch_bounds__(BLK) void quantize_elem_kernel(const float* __restrict__ x, int64_t n, float s_static, MaxOf amax,
                                                            int8_t* __restrict__ q8, float* __restrict__ scale_out,
                                                            int32_t* __restrict__ zero_me, int n_zero) {
  // also clears the token code sums the gather that follows adds into
  for (int i = blockIdx.x * BLK + threadIdx.x; i < n_zero; i += gridDim.x * BLK) zero_me[i] = 0;
  const float s = act_scale(s_static, amax);
  if (blockIdx.x == 0 && threadIdx.x == 0 && scale_out) *scale_out = s;
  const bool live = s > 0.f;
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK)
    q8[i] = live ? (int8_t)quant1(x[i], s) : (int8_t)0;
}

// Step 2: patches of codes -> fragment layout and token code sums.  Token t = (n, ho, wo); column
// k = (c, r, q) as in a weight row flattened [C, kh, kw].  A thread owns 16 consecutive k of one
// token; (c, r, q) is split once per chunk and then stepped, not divided, element by element.
// pad_neg: nullptr (taps outside the image read code 0), or a device word whose negation is the code
// of the real value 0 (asymmetric codes: the zero point minus 2^(a-1)).
__global__ __launch_bounds__(BLK) void im2col_codes_kernel(const int8_t* __restrict__ q8, ConvGeom g, int T, int in,
                                                           int in_pad, uint8_t* __restrict__ qx_frag,
                                                           int32_t* __restrict__ rowsum, const int32_t* __restrict__ pad_neg) {
  const int padv = pad_neg != nullptr ? -pad_neg[0] : 0;
  const int tb = blockIdx.x;
  const int n16 = threadIdx.x & 15;
  const int t = tb * 16 + n16;
  const int nks = in_pad >> 6;
  const int nchunk = in_pad >> 4;
  const int per = (nchunk + gridDim.y - 1) / gridDim.y;
  const int c_lo = blockIdx.y * per;
  const int c_hi = min(nchunk, c_lo + per);
  const bool tok = t < T;
  const int wo = tok ? t % g.Wo : 0, ho = tok ? (t / g.Wo) % g.Ho : 0, nimg = tok ? t / (g.Wo * g.Ho) : 0;
  const int hi0 = ho * g.stride - g.pad, wi0 = wo * g.stride - g.pad;
  // offset = base_n + c * step_c + h * step_r + w * step_q in either layout
  const int step_q = g.nhwc ? g.C : 1, step_r = g.nhwc ? g.W * g.C : g.W, step_c = g.nhwc ? 1 : g.H * g.W;
  const int base_n = nimg * g.C * g.H * g.W;
  int sum = 0;
  for (int c = c_lo + (threadIdx.x >> 4); c < c_hi; c += BLK / 16) {
    int k = c * 16;
    int qq = k % g.kw, rr = (k / g.kw) % g.kh, cc = k / (g.kw * g.kh);
    // The element offset is stepped, not recomputed (32-bit: the input has fewer than 2^31 elements), and
    // all 16 byte loads are issued before the first one is used: offsets of taps that are not read are
    // clamped to element 0 and the value is replaced afterwards.
    int off = base_n + cc * step_c + (hi0 + rr) * step_r + (wi0 + qq) * step_q;
    int q[16];
    int offs[16];
    int kind[16];   // 0: code 0 (beyond the row or the batch), 1: read, 2: outside the image
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int hi = hi0 + rr, wi = wi0 + qq;
      const bool inside = hi >= 0 && hi < g.H && wi >= 0 && wi < g.W;
      kind[e] = (tok && k < in) ? (inside ? 1 : 2) : 0;
      offs[e] = kind[e] == 1 ? off : 0;
      ++k;
      off += step_q;
      if (++qq == g.kw) {
        qq = 0;
        off += step_r - g.kw * step_q;
        if (++rr == g.kh) { rr = 0; ++cc; off += step_c - g.kh * step_r; }
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) q[e] = q8[offs[e]];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      q[e] = kind[e] == 1 ? q[e] : (kind[e] == 2 ? padv : 0);
      sum += q[e];
    }
    const int ks = c >> 2, kc = c & 3;
    const uint4 w = make_uint4(pack4(q[0], q[1], q[2], q[3]), pack4(q[4], q[5], q[6], q[7]),
                               pack4(q[8], q[9], q[10], q[11]), pack4(q[12], q[13], q[14], q[15]));
    *reinterpret_cast<uint4*>(qx_frag + (((size_t)tb * nks + ks) * 64 + kc * 16 + n16) * 16) = w;
  }
  if (tok && sum != 0) atomicAdd(&rowsum[t], sum);
}

// h = act(y1) for every member, and max|h| per member (amax_neg set: max(h, 0) and max(-h, 0) apart, the range
// an asymmetric quantizer needs).
__global__ __launch_bounds__(BLK) void mlp_act_kernel(const float* __restrict__ y1, int T, int H, int act,
                                                      float* __restrict__ h, uint32_t* __restrict__ amax_bits,
                                                      uint32_t* __restrict__ amax_neg) {
  const int m = blockIdx.y;
  const int64_t n = (int64_t)T * H;
  const int O1 = act == PIPE_ACT_SILU_GATED ? 2 * H : H;
  const float* src = y1 + (size_t)m * T * O1;
  float* dst = h + (size_t)m * n;
  float mx = 0.f, mn = 0.f;
  const bool two_sided = amax_neg != nullptr;
  auto gate1 = [](float gte, float up) { return gte / (1.f + expf(-gte)) * up; };
  auto take = [&](float v) { mx = fmaxf(mx, two_sided ? v : fabsf(v)); mn = fmaxf(mn, -v); };
  if ((H & 3) == 0 && ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0) {
    // four neighbouring channels of a token per step: 16-byte loads and stores, 32-bit index arithmetic
    // (the host keeps T * H below 2^31), the same expression per element as below
    const int H4 = H >> 2, n4 = T * H4, O4 = O1 >> 2;
    const float4* s4 = reinterpret_cast<const float4*>(src);
    float4* d4 = reinterpret_cast<float4*>(dst);
    for (int i = blockIdx.x * BLK + threadIdx.x; i < n4; i += gridDim.x * BLK) {
      const int t = i / H4, c4 = i - t * H4;
      float4 v;
      if (act == PIPE_ACT_SILU_GATED) {
        const float4 g = s4[t * O4 + c4], u = s4[t * O4 + H4 + c4];
        v = make_float4(gate1(g.x, u.x), gate1(g.y, u.y), gate1(g.z, u.z), gate1(g.w, u.w));
      } else {
        const float4 a = s4[i];
        v = make_float4(gelu_erf(a.x), gelu_erf(a.y), gelu_erf(a.z), gelu_erf(a.w));
      }
      d4[i] = v;
      take(v.x); take(v.y); take(v.z); take(v.w);
    }
  } else {
    for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) {
      float v;
      if (act == PIPE_ACT_SILU_GATED) {
        const int64_t t = i / H;
        const int c = (int)(i - t * H);
        v = gate1(src[t * O1 + c], src[t * O1 + H + c]);
      } else {
        v = gelu_erf(src[i]);
      }
      dst[i] = v;
      take(v);
    }
  }
  mx = block_max(mx);
  if (threadIdx.x == 0) slot_raise(&amax_bits[m], mx);
  if (two_sided) {
    mn = block_max(mn);
    if (threadIdx.x == 0) slot_raise(&amax_neg[m], mn);
  }
}


// ---------------------------------------------------------------- asymmetric activation codes
// Sec. 4.3 compares under asymmetric quantization; the affine quantizer over [min(x,0), max(x,0)]:
//   s = (hi - lo) / (2^a - 1),  z = clamp(rint(-lo / s), 0, 2^a - 1),  Q(x) = clamp(rint(x / s) + z, 0, 2^a - 1).
// The contraction kernels multiply signed bytes, so the stored code is Q(x) - 2^(a-1); the exact
// accumulator is then acc' + (2^(a-1) - z) * (sum of the row's weight codes), a term without the
// token that the entry point folds into the bias.

// max(x, 0) and max(-x, 0), one value per workgroup (bit patterns; both order independent, hence exact).  Also clears the token
// code sums the quantizer that follows adds into.
__global__ __launch_bounds__(BLK) void minmax_kernel(const float* __restrict__ x, int64_t n, uint32_t* __restrict__ hi_part,
                                                     uint32_t* __restrict__ nlo_part, int32_t* __restrict__ zero_me, int n_zero) {
  for (int i = blockIdx.x * BLK + threadIdx.x; i < n_zero; i += gridDim.x * BLK) zero_me[i] = 0;
  float hi = 0.f, nlo = 0.f;
  auto take = [&](float v) { hi = fmaxf(hi, v); nlo = fmaxf(nlo, -v); };
  const int64_t stride = (int64_t)gridDim.x * BLK, i0 = (int64_t)blockIdx.x * BLK + threadIdx.x;
  int64_t done = 0;
  if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
    const int64_t n4 = n >> 2;
    scan4<8>(reinterpret_cast<const float4*>(x), n4, i0, stride, [&](const float4& v) { take(v.x); take(v.y); take(v.z); take(v.w); });
    done = n4 << 2;
  }
  for (int64_t i = done + i0; i < n; i += stride) take(x[i]);
  hi = block_max(hi);
  nlo = block_max(nlo);
  if (threadIdx.x == 0) {
    hi_part[blockIdx.x] = __float_as_uint(hi);
    nlo_part[blockIdx.x] = __float_as_uint(nlo);
  }
}

// Q(x), asymmetric, minus 2^(a-1): qa = 2^a - 1, shift = 2^(a-1)
struct AsymCodes {
  Divisor d;
  float qa, zf;
  int shift;
  uint8_t* rows = nullptr;   // row-major copy of the unsigned codes, or nullptr
  __device__ __forceinline__ AsymCodes(float hi, float nlo, float qa_, int shift_)
      : d(__fdiv_rn(__fadd_rn(hi, nlo), qa_)), qa(qa_), shift(shift_) {
    zf = live() ? fminf(fmaxf(rintf(__fdiv_rn(nlo, d.s)), 0.f), qa) : 0.f;
  }
  __device__ __forceinline__ bool live() const { return d.s > 0.f; }
  template <bool FAST>
  __device__ __forceinline__ int code(float v) const {
    return (int)fminf(fmaxf(__fadd_rn(rintf(d.quotient<FAST>(v)), zf), 0.f), qa) - shift;
  }
  __device__ __forceinline__ void row_major(int t, int k0, int T, int in, const int (&q)[16]) const {
    if (rows == nullptr || t >= T) return;
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (k0 + e < in) rows[(size_t)t * in + k0 + e] = live() ? (uint8_t)(q[e] + shift) : (uint8_t)0;
  }
};

// The same walk as quantize_act_kernel with the affine quantizer.  Writes the fragment layout, adds the token code sums
// (zero on entry), optionally the unsigned codes row-major, and (block 0,0) the scale and shift - z.  With `C` (the
// single layer) also the bias the contraction adds: bias_eff[o] = b[o] + (s * dz) * C[o], C[o] = sum_k s_k[o] * (sum_i
// q_k[o,i]) -- a launch of its own took 5 us.
__global__ __launch_bounds__(BLK) void quantize_asym_kernel(const float* __restrict__ x, int T, int in, int in_pad,
                                                            MaxOf hi_max, MaxOf nlo_max, float qa, int shift,
                                                            uint8_t* __restrict__ qx_frag, int32_t* __restrict__ rowsum,
                                                            uint8_t* __restrict__ qx_rowmajor, float* __restrict__ scale_out,
                                                            int32_t* __restrict__ dz_out, const float* __restrict__ bias,
                                                            const float* __restrict__ C, float* __restrict__ bias_eff, int n_out) {
  float off = 0.f;   // the scale times the zero point's distance from the codes' middle
  auto make = [&]() {
    float hi, nlo;
    max_of_two(hi_max, nlo_max, &hi, &nlo);
    AsymCodes cd(hi, nlo, qa, shift);
    cd.rows = qx_rowmajor;
    const int dz = cd.live() ? shift - (int)cd.zf : 0;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
      scale_out[0] = cd.d.s;
      dz_out[0] = dz;
    }
    off = cd.d.s * (float)dz;
    return cd;
  };
  auto fetch = [=](int t, int k) { return x[(size_t)t * in + k]; };
  const bool vec = (in & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 && qx_rowmajor == nullptr;
  quantize_block(make, fetch, T, in, in_pad, qx_frag, rowsum, vec ? x : nullptr);
  if (C != nullptr) {
    const int nb = gridDim.x * gridDim.y;
    for (int o = (blockIdx.y * gridDim.x + blockIdx.x) * BLK + threadIdx.x; o < n_out; o += nb * BLK)
      bias_eff[o] = (bias != nullptr ? bias[o] : 0.f) + off * C[o];
  }
}

// every element of a tensor once, in its own layout (the convolution's first step): code minus shift
__global__ __launch_bounds__(BLK) void quantize_elem_asym_kernel(const float* __restrict__ x, int64_t n,
                                                                 MaxOf hi_max, MaxOf nlo_max, float qa, int shift,
                                                                 int8_t* __restrict__ q8, float* __restrict__ scale_out,
                                                                 int32_t* __restrict__ dz_out, int32_t* __restrict__ zero_me,
                                                                 int n_zero) {
  for (int i = blockIdx.x * BLK + threadIdx.x; i < n_zero; i += gridDim.x * BLK) zero_me[i] = 0;
  const float hi = max_of(hi_max), nlo = max_of(nlo_max);
  const float s = __fdiv_rn(__fadd_rn(hi, nlo), qa);
  const bool live = s > 0.f;
  const float zf = live ? fminf(fmaxf(rintf(__fdiv_rn(nlo, s)), 0.f), qa) : 0.f;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scale_out[0] = s;
    dz_out[0] = live ? shift - (int)zf : 0;
  }
  for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLK) {
    int v = 0;
    if (live) v = (int)fminf(fmaxf(__fadd_rn(rintf(__fdiv_rn(x[i], s)), zf), 0.f), qa) - shift;
    q8[i] = (int8_t)v;
  }
}

// bias_eff[o] = b[o] + (s * dz) * C[o], C[o] = sum_k s_k[o] * (sum_i q_k[o,i])
__global__ void asym_bias_kernel(const float* __restrict__ bias, const float* __restrict__ C, const float* __restrict__ scale,
                                 const int32_t* __restrict__ dz, float* __restrict__ out, int n) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= n) return;
  const float f = scale[0] * (float)dz[0];
  out[o] = (bias != nullptr ? bias[o] : 0.f) + f * C[o];
}

// Members of a chain, each with its own scale and zero point: member m's offset vector is
// (s_m * dz_m) * sum_{k in member m, ascending} P[k][o], P[k][o] = s_k[o] * (sum_i q_k[o,i]); the layer's
// bias joins the first member.  reduce: one vector, the members' sum (ascending m) plus the bias.
__global__ void asym_bias_members_kernel(const float* __restrict__ bias, const float* __restrict__ P, const float* __restrict__ scale,
                                         int scale_stride, const int32_t* __restrict__ dz, int dz_stride, MemberRanges mr,
                                         int reduce, float* __restrict__ outv, int n) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= n) return;
  float tot = bias != nullptr ? bias[o] : 0.f;
  for (int m = 0; m < mr.M; ++m) {
    float c = 0.f;
    for (int k = mr.lo[m]; k <= mr.hi[m]; ++k) c += P[(size_t)k * n + o];
    const float f = scale[m * scale_stride] * (float)dz[m * dz_stride];
    if (reduce) {
      tot = fmaf(f, c, tot);
    } else {
      outv[(size_t)m * n + o] = fmaf(f, c, m == 0 ? tot : 0.f);
    }
  }
  if (reduce) outv[o] = tot;
}

// exact accumulators of the debug export: acc[k][t][o] += dz * wsum[k][o]
__global__ void asym_acc_fix_kernel(int32_t* __restrict__ acc, const int32_t* __restrict__ wsum, const int32_t* __restrict__ dz,
                                    int K, int T, int out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)K * T * out) return;
  const int o = (int)(i % out), k = (int)(i / ((int64_t)T * out));
  acc[i] += dz[0] * wsum[(size_t)k * out + o];
}

// sum of the codes of every stored row of one order -> wsum[o] (dense over output channels)
__global__ __launch_bounds__(BLK) void row_code_sums_kernel(const int8_t* __restrict__ codes, int in, int group,
                                                            const int32_t* __restrict__ gids, int32_t* __restrict__ wsum) {
  const int r = blockIdx.x, slot = r / group;
  const int o = gids[slot] * group + (r - slot * group);
  int s = 0;
  for (int i = threadIdx.x; i < in; i += BLK) s += codes[(size_t)r * in + i];
  __shared__ int sm[BLK];
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int w = BLK / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) wsum[o] = sm[0];
}

// Convolution input for the implicit GEMM: channels-last int8 codes [N, H, W, C] and, per pixel, the sum of its C codes (added into
// csum, zero on entry: one atomic per pixel and 64 channels).  A workgroup takes 1024 * U elements, 64 channels of 16 * U neighbouring pixels
// of an image, through LDS: reads run along the layout's own inner dimension, 16 bytes a lane where its rows allow (`vec`), writes are 16
// channels a lane.  Bound by the trip to memory: U loads a lane in flight, then one store (32 images of 256 x 14 x 14: tiles of 32 x 32, one byte
// a store, 7.2 us, these 4.7).
template <int U>
__global__ __launch_bounds__(BLK) void quantize_nhwc_sums_kernel(const float* __restrict__ x, int C, int HW, int nhwc, int vec,
                                                                 float s_static, MaxOf amax,
                                                                 int8_t* __restrict__ q8, int32_t* __restrict__ csum,
                                                                 float* __restrict__ scale_out) {
  constexpr int CH = 64, P = 1024 * U / CH, ROW = CH + 16;   // channels, pixels; bytes of a pixel in LDS (16 apart: other banks)
  __shared__ alignas(16) uint8_t tile[P * ROW];
  const int n = blockIdx.z, c0 = blockIdx.y * CH, p0 = blockIdx.x * P, tid = threadIdx.x;
  // four neighbours along the input's inner dimension: pixels of a channel, or channels of a pixel
  const int per_row = nhwc ? CH / 4 : P / 4, step = BLK / per_row;   // quads of a row, rows of a pass
  const int quad = (tid % per_row) * 4, row = tid / per_row;
  float xv[U][4];   // requested before the scale is known
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int r = row + j * step;
    const int c = nhwc ? c0 + quad : c0 + r, p = nhwc ? p0 + r : p0 + quad;
    const size_t at = nhwc ? ((size_t)n * HW + p) * C + c : ((size_t)n * C + c) * HW + p;
    if (vec) {
      const float4 v = p < HW ? *reinterpret_cast<const float4*>(x + at) : make_float4(0.f, 0.f, 0.f, 0.f);
      xv[j][0] = v.x; xv[j][1] = v.y; xv[j][2] = v.z; xv[j][3] = v.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) xv[j][i] = (nhwc ? p : p + i) < HW ? x[at + i] : 0.f;
    }
  }
  const float s = s_static > 0.f ? s_static : __fdiv_rn(max_of_by_wave(amax), c_act_qmax);
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && tid == 0 && scale_out) *scale_out = s;
  const SymCodes cd(s);
  const bool live = cd.live();
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int r = row + j * step;
    int q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = live ? (cd.d.fast ? cd.code<true>(xv[j][i]) : cd.code<false>(xv[j][i])) : 0;
    if (nhwc) {
      *reinterpret_cast<uint32_t*>(&tile[r * ROW + quad]) = pack4(q[0], q[1], q[2], q[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) tile[(quad + i) * ROW + r] = (uint8_t)q[i];
    }
  }
  __syncthreads();
  constexpr int CHUNKS = CH / 16;   // lanes of a pixel
  const int px = tid / CHUNKS, ck = tid % CHUNKS, p = p0 + px;
  if (px >= P) return;   // (whole pixels: their lanes leave together)
  const uint4 w = *reinterpret_cast<const uint4*>(&tile[px * ROW + ck * 16]);
  int sum = __builtin_amdgcn_sdot4((int)w.x, 0x01010101, 0, false);
  sum = __builtin_amdgcn_sdot4((int)w.y, 0x01010101, sum, false);
  sum = __builtin_amdgcn_sdot4((int)w.z, 0x01010101, sum, false);
  sum = __builtin_amdgcn_sdot4((int)w.w, 0x01010101, sum, false);
#pragma unroll
  for (int o = CHUNKS / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (p < HW) {
    *reinterpret_cast<uint4*>(q8 + ((size_t)n * HW + p) * C + c0 + ck * 16) = w;
    if (ck == 0 && sum != 0) atomicAdd(&csum[(size_t)n * HW + p], sum);
  }
}

}  // namespace

int launch_quantize_nhwc_sums(const float* x, int N, int C, int HW, int nhwc, float s_static, MaxOf amax,
                              int8_t* q8, int32_t* csum, float* scale_out, hipStream_t st) {
  if (C % 64 != 0) return PIPE_ESHAPE;
  // rows of whole 16-byte loads: pixels of a channel, or channels of a pixel, in a tensor that begins on 16 bytes
  const int vec = (reinterpret_cast<uintptr_t>(x) & 15) == 0 && (nhwc || HW % 4 == 0);
  // One load a lane while that leaves four workgroups a compute unit at most, then two, four for the largest.  Kernels, us, with 1 / 2 / 4: 1 image of 128 x 28 x 28
  // 3.5 / 4.0 / 4.9, 8 3.8 / 4.1 / 5.0, 16 4.6 / 4.5 / 5.2, 40 8.7 / 6.9 / 7.9; 128 of 64 x 56 x 56 34 / 22.8 / 22.9, 256 64 / 41.0 / 39.7.
  const int64_t elements = (int64_t)N * C * HW;
#define PIPE_NHWC(U)                                                                                                                      \
  PIPE_KLAUNCH(quantize_nhwc_sums_kernel<U>, dim3(ceil_div(HW, 16 * U), C / 64, N), dim3(BLK), 0, st, x, C, HW, nhwc, vec, s_static, amax, q8, csum, \
               scale_out)
  if (elements <= 1 << 20) PIPE_NHWC(1);
  else if (elements <= 16 << 20) PIPE_NHWC(2);
  else PIPE_NHWC(4);
#undef PIPE_NHWC
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int set_act_qmax(float qmax) {
  PIPE_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_act_qmax), &qmax, sizeof(float)));
  return PIPE_OK;
}

int launch_zero_u32(uint32_t* p, int n, hipStream_t st) {
  if (n <= 0) return PIPE_OK;
  PIPE_KLAUNCH(zero_u32_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, st, p, n);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

// Workgroups (and parts) of a max reduction over n elements: eight 16-byte loads per thread, two workgroups per compute unit
// at most (64 MiB: 20 us with 256 or 512; 12 MiB: 4.8 us, 7.5 with one atomic slot).
int max_parts(int64_t n) {
  const int64_t blocks = (n / 4 + BLK * 8 - 1) / (BLK * 8);
  return (int)std::min<int64_t>(std::max<int64_t>(blocks, 1), PIPE_MAX_PARTS);
}

int launch_absmax(const float* x, int64_t n, uint32_t* part, int32_t* zero_me, int n_zero, hipStream_t st) {
  if (n <= 0) return PIPE_OK;
  PIPE_KLAUNCH(absmax_kernel, dim3((unsigned)max_parts(n)), dim3(BLK), 0, st, x, n, part, zero_me, n_zero);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

static int ksplit_for(int T_pad, int in_pad) {
  // four workgroups per compute unit (64 MiB in, 16 MiB out: 18.7 us; split into 512, 2048 and 4096: 25.6, 25.0 and 29.3)
  const int tbs = T_pad / 16;
  int ks = 1;
  const int nchunk = in_pad / 16;
  while (tbs * ks < 1024 && ks * 2 * 16 <= nchunk) ks *= 2;
  return ks;
}

int launch_quantize_act(const float* x, int T, int in, int in_pad, int T_pad, float s_static,
                        MaxOf amax, uint8_t* qx_frag, int32_t* rowsum, bool rowsum_is_zero,
                        int8_t* qx_rowmajor, float* scale_out, hipStream_t st) {
  if (!rowsum_is_zero) {
    int rc = launch_zero_u32(reinterpret_cast<uint32_t*>(rowsum), T_pad, st);
    if (rc) return rc;
  }
  dim3 grid(T_pad / 16, ksplit_for(T_pad, in_pad));
  PIPE_KLAUNCH(quantize_act_kernel, grid, dim3(BLK), 0, st, x, (int64_t)0, T, in, in_pad, s_static, amax,
                     qx_frag, (int64_t)0, rowsum, 0, qx_rowmajor, scale_out);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_quantize_members(const float* x, int64_t x_mstride, int M, int T, int in, int in_pad, int T_pad,
                            const uint32_t* amax_bits, uint8_t* qx_frag, int64_t qx_mstride, int32_t* rowsum,
                            bool rowsum_is_zero, float* scale_out, hipStream_t st) {
  if (!rowsum_is_zero) {
    int rc = launch_zero_u32(reinterpret_cast<uint32_t*>(rowsum), M * T_pad, st);
    if (rc) return rc;
  }
  dim3 grid(T_pad / 16, ksplit_for(T_pad * M, in_pad), M);
  PIPE_KLAUNCH(quantize_act_kernel, grid, dim3(BLK), 0, st, x, x_mstride, T, in, in_pad, 0.f, MaxOf{amax_bits, 0},
                     qx_frag, qx_mstride, rowsum, T_pad, (int8_t*)nullptr, scale_out);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_quantize_small(const float* x, int64_t x_mstride, int M, int T, int in, int in_pad, float s_static,
                          const uint32_t* amax_bits, uint8_t* qx_frag, int64_t qx_mstride, int32_t* rowsum,
                          int8_t* qx_rowmajor, float* scale_out, hipStream_t st) {
  PIPE_KLAUNCH(quantize_small_kernel, dim3((unsigned)round_up64(T, 16), M), dim3(SBLK), 0, st, x, x_mstride, T, in, in_pad, s_static,
                     amax_bits, qx_frag, qx_mstride, rowsum, qx_rowmajor, scale_out);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_quantize_elem(const float* x, int64_t n, float s_static, MaxOf amax, int8_t* q8,
                         float* scale_out, hipStream_t st) {
  int64_t blocks = (n + BLK - 1) / BLK;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  PIPE_KLAUNCH(quantize_elem_kernel, dim3((unsigned)blocks), dim3(BLK), 0, st, x, n, s_static, amax, q8, scale_out,
                     (int32_t*)nullptr, 0);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_quantize_im2col(const float* x, int N, int C, int H, int W, int kh, int kw, int stride,
                           int pad, int nhwc, int Ho, int Wo, int in_pad, int T_pad,
                           float s_static, MaxOf amax, int8_t* q8_scratch, uint8_t* qx_frag,
                           int32_t* rowsum, float* scale_out, hipStream_t st) {
  const int64_t n = (int64_t)N * C * H * W;
  if (n >= ((int64_t)1 << 31)) return PIPE_ESHAPE;   // the gather steps 32-bit element offsets
  int64_t blocks = (n + BLK - 1) / BLK;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  PIPE_KLAUNCH(quantize_elem_kernel, dim3((unsigned)blocks), dim3(BLK), 0, st, x, n, s_static, amax,
                     q8_scratch, scale_out, rowsum, T_pad);
  ConvGeom g{N, C, H, W, kh, kw, stride, pad, nhwc, Ho, Wo};
  const int T = N * Ho * Wo, in = C * kh * kw;
  dim3 grid(T_pad / 16, ksplit_for(T_pad, in_pad));
  PIPE_KLAUNCH(im2col_codes_kernel, grid, dim3(BLK), 0, st, q8_scratch, g, T, in, in_pad, qx_frag, rowsum,
                     (const int32_t*)nullptr);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

// the same with asymmetric codes: every element once (code minus 2^(a-1), scale and 2^(a-1) - z to device
// memory), then the patches, whose taps outside the image hold the code of the real value 0
int launch_quantize_im2col_asym(const float* x, int N, int C, int H, int W, int kh, int kw, int stride, int pad, int nhwc,
                                int Ho, int Wo, int in_pad, int T_pad, MaxOf hi_max, MaxOf nlo_max,
                                int act_bits, int8_t* q8_scratch, uint8_t* qx_frag, int32_t* rowsum, float* scale_out,
                                int32_t* dz_out, hipStream_t st) {
  const int64_t n = (int64_t)N * C * H * W;
  if (n >= ((int64_t)1 << 31)) return PIPE_ESHAPE;   // the gather steps 32-bit element offsets
  int64_t blocks = (n + BLK - 1) / BLK;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  PIPE_KLAUNCH(quantize_elem_asym_kernel, dim3((unsigned)blocks), dim3(BLK), 0, st, x, n, hi_max, nlo_max,
                     (float)((1 << act_bits) - 1), 1 << (act_bits - 1), q8_scratch, scale_out, dz_out, rowsum, T_pad);
  ConvGeom g{N, C, H, W, kh, kw, stride, pad, nhwc, Ho, Wo};
  const int T = N * Ho * Wo, in = C * kh * kw;
  dim3 grid(T_pad / 16, ksplit_for(T_pad, in_pad));
  PIPE_KLAUNCH(im2col_codes_kernel, grid, dim3(BLK), 0, st, q8_scratch, g, T, in, in_pad, qx_frag, rowsum,
                     (const int32_t*)dz_out);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_mlp_act(const float* y1, int M, int T, int H, int act, float* h, uint32_t* amax_bits, uint32_t* amax_neg,
                   hipStream_t st) {
  const int64_t n = (int64_t)T * H;
  if (n <= 0) return PIPE_OK;
  if (n >= ((int64_t)1 << 31)) return PIPE_ESHAPE;   // the kernel's fast path indexes with 32 bits
  int64_t blocks = (n + BLK * 4 - 1) / (BLK * 4);
  if (blocks > 4096) blocks = 4096;
  PIPE_KLAUNCH(mlp_act_kernel, dim3((unsigned)blocks, M), dim3(BLK), 0, st, y1, T, H, act, h, amax_bits, amax_neg);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

// ---- asymmetric activation codes (host side) ----------------------------------------------
int launch_minmax(const float* x, int64_t n, uint32_t* hi_part, uint32_t* nlo_part, int32_t* zero_me, int n_zero, hipStream_t st) {
  PIPE_KLAUNCH(minmax_kernel, dim3((unsigned)max_parts(n)), dim3(BLK), 0, st, x, n, hi_part, nlo_part, zero_me, n_zero);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_quantize_asym(const float* x, int T, int in, int in_pad, int T_pad, MaxOf hi_max, MaxOf nlo_max,
                         int act_bits, uint8_t* qx_frag, int32_t* rowsum, bool rowsum_is_zero, uint8_t* qx_rowmajor, float* scale_out,
                         int32_t* dz_out, hipStream_t st, const float* bias, const float* C, float* bias_eff, int n_out) {
  if (!rowsum_is_zero) {
    int rc = launch_zero_u32(reinterpret_cast<uint32_t*>(rowsum), T_pad, st);
    if (rc) return rc;
  }
  dim3 grid(T_pad / 16, ksplit_for(T_pad, in_pad));
  PIPE_KLAUNCH(quantize_asym_kernel, grid, dim3(BLK), 0, st, x, T, in, in_pad, hi_max, nlo_max, (float)((1 << act_bits) - 1),
                     1 << (act_bits - 1), qx_frag, rowsum, qx_rowmajor, scale_out, dz_out, bias, C, bias_eff, n_out);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_asym_bias(const float* bias, const float* C, const float* scale, const int32_t* dz, float* out, int n,
                     hipStream_t st) {
  PIPE_KLAUNCH(asym_bias_kernel, dim3((n + 255) / 256), dim3(256), 0, st, bias, C, scale, dz, out, n);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_asym_bias_members(const float* bias, const float* P, const float* scale, int scale_stride, const int32_t* dz,
                             int dz_stride, int M, const int* lo, const int* hi, int reduce, float* outv, int n, hipStream_t st) {
  MemberRanges mr{};
  mr.M = M;
  for (int m = 0; m < M; ++m) { mr.lo[m] = lo[m]; mr.hi[m] = hi[m]; }
  PIPE_KLAUNCH(asym_bias_members_kernel, dim3((n + 255) / 256), dim3(256), 0, st, bias, P, scale, scale_stride,
               dz, dz_stride, mr, reduce, outv, n);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_asym_acc_fix(int32_t* acc, const int32_t* wsum, const int32_t* dz, int K, int T, int out, hipStream_t st) {
  const int64_t n = (int64_t)K * T * out;
  if (n == 0) return PIPE_OK;
  PIPE_KLAUNCH(asym_acc_fix_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, acc, wsum, dz, K, T, out);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_row_code_sums(const int8_t* codes, int rows, int in, int group, const int32_t* gids, int32_t* wsum, hipStream_t st) {
  if (rows == 0) return PIPE_OK;
  PIPE_KLAUNCH(row_code_sums_kernel, dim3(rows), dim3(BLK), 0, st, codes, in, group, gids, wsum);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}
