// Expanded depthwise convolution (App. H: a convolution whose filters see one input channel;
// the separable blocks of MobileNet / EfficientNet).  Not a dense contraction: every output is
// kh*kw multiply-adds per order, so the layer is bound by reading the input and writing y, and runs
// on the vector ALUs.  Two ways: depthwise3_kernel (3 x 3, one member of at most 4 orders, images that fill its
// workgroups) quantizes the fp32 input into LDS and multiplies a window column's three taps at once; everything else takes two launches,
// codes channels last first, then depthwise_kernel, whose thread owns one pixel and 4 channels, reads its window once and
// applies every stored order to it.  Arithmetic as everywhere: exact integer sums,
// fp32 sum over the orders of a member in ascending order, activation scale, bias.
#include <algorithm>
#include <type_traits>

#include "pipe_codes.h"

namespace {

constexpr int BLK = 256;
constexpr int MAX_WIN = 49;   // up to 7 x 7

// codes[k][i][o] (tap-major, channel-minor: the codes of four neighbouring channels for one
// tap are one 32-bit word) and scales[k][o] of one order, from its unpacked stored rows
__global__ void dense_order_kernel(const int8_t* __restrict__ rows_codes, const float* __restrict__ scales_all,
                                   const int32_t* __restrict__ pos, const int32_t* __restrict__ gids, int group, int in,
                                   int C, int8_t* __restrict__ codes_k, float* __restrict__ scales_k) {
  const int r = blockIdx.x;   // stored row
  const int slot = r / group;
  const int o = gids[slot] * group + (r - slot * group);
  for (int i = threadIdx.x; i < in; i += blockDim.x) codes_k[(size_t)i * C + o] = rows_codes[(size_t)r * in + i];
  if (threadIdx.x == 0) scales_k[o] = scales_all[(size_t)pos[r >> 4] * 16 + (r & 15)];
}

// fp32 [N,C,H,W] -> int8 codes [N,H,W,C]: 32 channels x 32 pixels at a time through LDS, so that reads run along the pixels
// and writes along the channels.  A workgroup takes the same tile of one image after another, the next one's values
// requested ahead: it finds the scale once for all of them (32768 images of 32 x 2 x 2, the whole layer 49.3 -> 34.7 us).
constexpr int NHWC_BLOCKS = 4096;
__global__ __launch_bounds__(256) void quantize_to_nhwc_kernel(const float* __restrict__ x, int N, int C, int HW, float s_static,
                                                               MaxOf amax, float qmax,
                                                               int8_t* __restrict__ q8, float* __restrict__ scale_out) {
  __shared__ int8_t tile[2][32][33];
  const int c0 = blockIdx.y * 32, p0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  const float* src = x + (size_t)blockIdx.z * C * HW + (size_t)(c0 + ty) * HW + p0 + tx;
  int8_t* dst = q8 + (size_t)blockIdx.z * C * HW + (size_t)(p0 + ty) * C + c0 + tx;
  const size_t step = (size_t)gridDim.z * C * HW;
  float xv[4];
  auto load = [&]() {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (c0 + ty + 8 * j < C && p0 + tx < HW) xv[j] = src[(size_t)(8 * j) * HW];
  };
  load();
  const float s = s_static > 0.f ? s_static : __fdiv_rn(max_of_by_wave(amax), qmax);
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0 && scale_out) *scale_out = s;
  const Divisor d(s);
  int buf = 0;
  for (int left = (N - 1 - (int)blockIdx.z) / (int)gridDim.z; left >= 0; --left) {
    auto put = [&](auto fast) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c0 + ty + 8 * j < C && p0 + tx < HW)
          tile[buf][ty + 8 * j][tx] = s > 0.f ? (int8_t)(int)fminf(fmaxf(rintf(d.quotient<decltype(fast)::value>(xv[j])), -qmax), qmax) : (int8_t)0;
    };
    if (d.fast) put(std::true_type{});
    else put(std::false_type{});
    src += step;
    if (left > 0) load();
    __syncthreads();   // (before anyone writes the other buffer again, everyone has read it and come here)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (c0 + tx < C && p0 + ty + 8 * j < HW) dst[(size_t)(8 * j) * C] = tile[buf][tx][ty + 8 * j];
    dst += step;
    buf ^= 1;
  }
}

// dense codes [K][9][C] of a 3 x 3 layer -> [K][3][C], the vertical taps of a window column in bytes 0-2 of a dword
__global__ void pack_columns_kernel(const int8_t* __restrict__ codes, int K, int C, uint32_t* __restrict__ cols) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= K * 3 * C) return;
  const int c = i % C, kq = i / C, k = kq / 3, q = kq - 3 * k;
  const int8_t* g = codes + ((size_t)k * 9 + q) * C + c;
  cols[i] = pack4(g[0], g[(size_t)3 * C], g[(size_t)6 * C], 0);
}

struct DwParams {
  const int8_t* q8;        // Q(x), channels last [N,H,W,C]
  const float* s_x;
  const int8_t* codes;     // [K][kk][C]
  const float* scales;     // [K][C]
  const float* bias;
  float* y;                // [T, C] or [M, T, C]
  int N, C, H, W, kh, kw, stride, pad, Ho, Wo;
  int K, M, reduce;
  int member_lo[PIPE_MAX_K], member_hi[PIPE_MAX_K];
};

__device__ __forceinline__ int byte_of(uint32_t w, int j) { return (int)(int8_t)(w >> (8 * j)); }

// A thread owns one pixel and four neighbouring channels (C is a multiple of 16): one 32-bit
// load per window tap, one per tap and order for the codes, 16-byte stores.  KH, KW > 0: the
// window is a compile-time size and lives in registers; 0: any size up to MAX_WIN.
template <int KH, int KW>
__global__ __launch_bounds__(BLK) void depthwise_kernel(const DwParams p) {
  const int C4 = p.C >> 2;
  const long long idx = (long long)blockIdx.x * BLK + threadIdx.x;   // (pixel, channel quad), quad fastest
  const long long n_pix = (long long)p.N * p.Ho * p.Wo;
  if (idx >= n_pix * C4) return;
  const int c = (int)(idx % C4) * 4;
  const long long pix = idx / C4;
  const int wo = (int)(pix % p.Wo), ho = (int)((pix / p.Wo) % p.Ho), n = (int)(pix / ((long long)p.Wo * p.Ho));
  const int kh = KH > 0 ? KH : p.kh, kw = KW > 0 ? KW : p.kw;
  const int kk = kh * kw;
  uint32_t win[KH > 0 ? KH * KW : MAX_WIN];
#pragma unroll
  for (int r = 0; r < (KH > 0 ? KH : MAX_WIN); ++r) {
    if (r >= kh) break;
#pragma unroll
    for (int q = 0; q < (KW > 0 ? KW : MAX_WIN); ++q) {
      if (q >= kw) break;
      const int hi = ho * p.stride - p.pad + r, wi = wo * p.stride - p.pad + q;
      uint32_t v = 0;
      if (hi >= 0 && hi < p.H && wi >= 0 && wi < p.W)
        v = *reinterpret_cast<const uint32_t*>(p.q8 + (((size_t)n * p.H + hi) * p.W + wi) * p.C + c);
      win[r * kw + q] = v;
    }
  }
  const float sx = p.s_x[0];
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  if (p.bias != nullptr) bias = *reinterpret_cast<const float4*>(p.bias + c);
  float ysum[4] = {0.f, 0.f, 0.f, 0.f};
  for (int m = 0; m < p.M; ++m) {
    float yacc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = p.member_lo[m]; k <= p.member_hi[m]; ++k) {
      const float4 s4 = *reinterpret_cast<const float4*>(p.scales + (size_t)k * p.C + c);
      if (s4.x == 0.f && s4.y == 0.f && s4.z == 0.f && s4.w == 0.f) continue;   // all four pruned at this order
      const int8_t* w = p.codes + (size_t)k * kk * p.C + c;
      int acc[4] = {0, 0, 0, 0};
      auto tap = [&](int i) __attribute__((always_inline)) {
        const uint32_t cw = *reinterpret_cast<const uint32_t*>(w + (size_t)i * p.C);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += byte_of(win[i], j) * byte_of(cw, j);
      };
      if (KH > 0) {
#pragma unroll
        for (int i = 0; i < KH * KW; ++i) tap(i);
      } else {
        for (int i = 0; i < kk; ++i) tap(i);
      }
      const float sv[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) yacc[j] = fmaf(sv[j], (float)acc[j], yacc[j]);   // a pruned channel has scale 0 and codes 0
    }
    const float bv[4] = {bias.x, bias.y, bias.z, bias.w};
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = fmaf(sx, yacc[j], m == 0 ? bv[j] : 0.f);
      ysum[j] = m == 0 ? v[j] : ysum[j] + v[j];
    }
    if (!p.reduce) *reinterpret_cast<float4*>(p.y + ((size_t)m * n_pix + pix) * p.C + c) = make_float4(v[0], v[1], v[2], v[3]);
  }
  if (p.reduce) *reinterpret_cast<float4*>(p.y + (size_t)pix * p.C + c) = make_float4(ysum[0], ysum[1], ysum[2], ysum[3]);
}

// 3 x 3 windows, stride 1 or 2, one member of at most 4 orders: quantizer and layer in one launch, no codes in memory.
// A workgroup takes 64 channels of RB output rows and up to XT output columns.  It reads the fp32 input once, quantizes
// it into LDS as one dword per channel, column and 4 rows (packed along the rows), then every lane walks the columns of its
// channel: 3 dwords of 3 vertical taps against 3 dwords of codes, v_dot4 each, so an output costs 3 instructions per order
// instead of 9 multiply-adds and byte extractions.  Stores are 256 contiguous bytes (64 channels of a pixel).
// Bound by memory, the read and the write phase of the workgroups one after the other: a 3 x 3 layer of 32 x 384 x 28 x 28, K = 3,
// takes 23.7 us for 51 MB in (8 rows for 6) and 38.5 MB out, after 7.7 us for the maximum; quantizer, vector-ALU layer and slot clearing
// took 16 + 42 + 4 us.
struct Dw3Params {
  const float* x;
  MaxOf amax;
  float s_static, qmax;
  const uint32_t* codes;   // [K][3][C]: the three vertical taps of a window column in bytes 0-2
  const float* scales;     // [K][C]
  const float* bias;
  float* y;                // [T, C]
  int N, C, H, W, Ho, Wo, pad, nhwc, vec;
  int bands, x_tiles;
};

// output rows and columns (at most) of a workgroup
constexpr int dw3_rows(int stride) { return stride == 1 ? 6 : 3; }
constexpr int dw3_columns(int stride) { return stride == 1 ? 32 : 16; }
// the input can be read 16 bytes at a time (C is a multiple of 16)
inline bool dw3_wide(const float* x, int W, int nhwc) { return (nhwc || W % 4 == 0) && (reinterpret_cast<uintptr_t>(x) & 15) == 0; }

template <int STRIDE, int K>
__global__ __launch_bounds__(BLK) void depthwise3_kernel(const Dw3Params p) {
  constexpr int ND = 2, R = 4 * ND;                        // input rows held (16 rows: 25.8 us against 23.7 on the layer above)
  constexpr int RB = dw3_rows(STRIDE), XT = dw3_columns(STRIDE);
  static_assert((RB - 1) * STRIDE + 3 <= R, "rows held");
  constexpr int COLS = (XT - 1) * STRIDE + 3;
  constexpr int PITCH = 65;                                // dwords per (column, 4 rows): 64 channels, rotated over the banks
  __shared__ uint32_t tile[COLS * ND * PITCH];

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int blk = blockIdx.x;
  const int xt = blk % p.x_tiles;
  blk /= p.x_tiles;
  const int band = blk % p.bands, n = blk / p.bands;
  const int c0 = blockIdx.y * 64, nc = min(64, p.C - c0);
  const int xo0 = xt * XT, nx = min(XT, p.Wo - xo0), ho0 = band * RB;
  const int cols = (nx - 1) * STRIDE + 3;
  const int ci0 = xo0 * STRIDE - p.pad, ri0 = ho0 * STRIDE - p.pad;   // input column and row of the tile's corner
  const int c = c0 + min(lane, nc - 1);

  // codes, scales and bias of this lane's channel: requested behind the input, used after it
  uint32_t w[K][3];
  float sc[K], bias = 0.f;
  auto request_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int q = 0; q < 3; ++q) w[k][q] = p.codes[((size_t)k * 3 + q) * p.C + c];
      sc[k] = p.scales[(size_t)k * p.C + c];
    }
    if (p.bias != nullptr) bias = p.bias[c];
  };

  // ---- input -> codes in LDS.  A unit is 4 rows of one channel at one column (vec: at 4 columns, 16-byte loads).
  auto row_ok = [&](int j, int i) { return (unsigned)(ri0 + 4 * j + i) < (unsigned)p.H; };
  float sx = p.s_static;
  if (p.vec) {
    // A unit is 4 rows x 4 neighbours in memory order, 16-byte loads: channels first, 4 columns of one channel; channels last,
    // 4 channels of one column.  Unit -> (channel or channel quad cc, row quad j, column quad or column g).
    const int g0 = p.nhwc ? max(ci0, 0) : max(ci0, 0) & ~3;
    const int span = min(ci0 + cols, p.W) - g0;                     // columns inside the image
    const int ng = p.nhwc ? span : (span + 3) >> 2, ncc = p.nhwc ? (nc + 3) >> 2 : nc;
    const int units = max(ncc * ND * ng, 0);
    auto split = [&](int u, int& cc, int& j, int& g) __attribute__((always_inline)) {
      if (p.nhwc) { cc = u % ncc; const int r = u / ncc; j = r % ND; g = r / ND; }
      else { g = u % ng; const int r = u / ng; j = r % ND; cc = r / ND; }
    };
    const ptrdiff_t row_step = p.nhwc ? (ptrdiff_t)p.W * p.C : p.W;
    float4 a[4], b[4];
    auto ld = [&](int u, float4(&v)[4]) {
      if (u >= units) return;
      int cc, j, g;
      split(u, cc, j, g);
      const int h = ri0 + 4 * j;
      const float* src = p.nhwc ? p.x + (((ptrdiff_t)n * p.H + h) * p.W + g0 + g) * p.C + c0 + 4 * cc
                                : p.x + (((ptrdiff_t)n * p.C + c0 + cc) * p.H + h) * p.W + g0 + 4 * g;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = row_ok(j, i) ? *reinterpret_cast<const float4*>(src + i * row_step) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    int u = threadIdx.x;
    ld(u, a);
    ld(u + BLK, b);
    request_weights();
    // the columns outside the image (at most the padding on either side)
    const int left = min(cols, max(0, -ci0)), right = min(cols, max(0, ci0 + cols - p.W));
    for (int i = threadIdx.x; i < (left + right) * ND * 64; i += BLK) {
      const int col = i / (ND * 64), rem = i - col * ND * 64;
      tile[((col < left ? col : cols - right + col - left) * ND + (rem >> 6)) * PITCH + (rem & 63)] = 0u;
    }
    if (!(p.s_static > 0.f)) sx = __fdiv_rn(max_of(p.amax), p.qmax);
    const Divisor d(sx);
    auto walk = [&](auto fast) {
      auto code = [&](float v) {
        return (int)fminf(fmaxf(rintf(d.quotient<decltype(fast)::value>(v)), -p.qmax), p.qmax);
      };
      auto st = [&](int u, const float4(&v)[4]) {
        if (u >= units) return;
        int cc, j, g;
        split(u, cc, j, g);
        const uint32_t q[4] = {pack4(code(v[0].x), code(v[1].x), code(v[2].x), code(v[3].x)),
                               pack4(code(v[0].y), code(v[1].y), code(v[2].y), code(v[3].y)),
                               pack4(code(v[0].z), code(v[1].z), code(v[2].z), code(v[3].z)),
                               pack4(code(v[0].w), code(v[1].w), code(v[2].w), code(v[3].w))};
        const int col = g0 - ci0 + (p.nhwc ? g : 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (p.nhwc) tile[(col * ND + j) * PITCH + 4 * cc + e] = sx > 0.f ? q[e] : 0u;   // nc is a multiple of 16
          else if ((unsigned)(col + e) < (unsigned)cols) tile[((col + e) * ND + j) * PITCH + cc] = sx > 0.f ? q[e] : 0u;
        }
      };
      while (u < units) {
        st(u, a);
        st(u + BLK, b);
        u += 2 * BLK;
        ld(u, a);
        ld(u + BLK, b);
      }
    };
    if (d.fast) walk(std::true_type{});
    else walk(std::false_type{});
  } else {
    request_weights();
    if (!(p.s_static > 0.f)) sx = __fdiv_rn(max_of(p.amax), p.qmax);
    const Divisor d(sx);
    auto walk = [&](auto fast) {
      for (int u = threadIdx.x; u < 64 * ND * cols; u += BLK) {
        // channels last: channel fastest; channels first: column fastest
        int cc, j, col;
        if (p.nhwc) { cc = u & 63; j = (u >> 6) % ND; col = (u >> 6) / ND; }
        else { col = u % cols; j = (u / cols) % ND; cc = u / (cols * ND); }
        const bool in_x = (unsigned)(ci0 + col) < (unsigned)p.W && cc < nc;
        int q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v = 0.f;
          if (in_x && row_ok(j, i)) {
            const int h = ri0 + 4 * j + i, wi = ci0 + col;
            v = p.x[p.nhwc ? (((size_t)n * p.H + h) * p.W + wi) * p.C + c0 + cc : (((size_t)n * p.C + c0 + cc) * p.H + h) * p.W + wi];
          }
          q[i] = (int)fminf(fmaxf(rintf(d.quotient<decltype(fast)::value>(v)), -p.qmax), p.qmax);
        }
        tile[(col * ND + j) * PITCH + cc] = sx > 0.f ? pack4(q[0], q[1], q[2], q[3]) : 0u;
      }
    };
    if (d.fast) walk(std::true_type{});
    else walk(std::false_type{});
  }
  __syncthreads();

  // ---- a wave takes a quarter of the columns; lane = channel
  const int per = (nx + 3) >> 2, x_lo = wave * per, x_hi = min(nx, x_lo + per);
  if (lane >= nc || x_lo >= x_hi) return;
  uint32_t col[3][2 * ND - 1];   // a column's dwords, then the dwords two rows further down
  auto column = [&](int q, int x) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < ND; ++j) col[q][j] = tile[(x * ND + j) * PITCH + lane];
#pragma unroll
    for (int j = 0; j + 1 < ND; ++j) col[q][ND + j] = __builtin_amdgcn_alignbyte(col[q][j + 1], col[q][j], 2);
  };
  if (STRIDE == 1) {
    column(1, x_lo);
    column(2, x_lo + 1);
  }
  for (int x = x_lo; x < x_hi; ++x) {
    if (STRIDE == 1) {
#pragma unroll
      for (int j = 0; j < 2 * ND - 1; ++j) { col[0][j] = col[1][j]; col[1][j] = col[2][j]; }
      column(2, x + 2);
    } else {
#pragma unroll
      for (int q = 0; q < 3; ++q) column(q, x * 2 + q);
    }
    float* dst = p.y + (((size_t)n * p.Ho + ho0) * p.Wo + xo0 + x) * p.C + c;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      // rows i*STRIDE .. +2 of the columns: bytes 0-2 or 1-3 of a dword, or of one two rows further down
      constexpr int S = STRIDE;
      const int off = i * S, j = (off & 2) ? ND + (off >> 2) : off >> 2;
      float acc_y = 0.f;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        int acc = 0;
#pragma unroll
        for (int q = 0; q < 3; ++q) acc = __builtin_amdgcn_sdot4((int)col[q][j], (int)((off & 1) ? w[k][q] << 8 : w[k][q]), acc, false);
        acc_y = fmaf(sc[k], (float)acc, acc_y);   // a pruned channel has scale 0 and codes 0
      }
      if (ho0 + i < p.Ho) dst[(size_t)i * p.Wo * p.C] = fmaf(sx, acc_y, bias);
    }
  }
}

template <int STRIDE>
int launch_depthwise3(Dw3Params& p, int K, hipStream_t st) {
  p.bands = ceil_div(p.Ho, dw3_rows(STRIDE));
  p.x_tiles = ceil_div(p.Wo, dw3_columns(STRIDE));
  const dim3 grid((unsigned)(p.N * p.bands * p.x_tiles), (unsigned)ceil_div(p.C, 64));
  switch (K) {
    case 1: PIPE_KLAUNCH((depthwise3_kernel<STRIDE, 1>), grid, dim3(BLK), 0, st, p); break;
    case 2: PIPE_KLAUNCH((depthwise3_kernel<STRIDE, 2>), grid, dim3(BLK), 0, st, p); break;
    case 3: PIPE_KLAUNCH((depthwise3_kernel<STRIDE, 3>), grid, dim3(BLK), 0, st, p); break;
    default: PIPE_KLAUNCH((depthwise3_kernel<STRIDE, 4>), grid, dim3(BLK), 0, st, p); break;
  }
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

}  // namespace

// Fills the tables of a depthwise layer, which the caller allocated
static int build_tables(const pipe_expansion* e, int8_t* codes, float* scales, uint32_t* cols, hipStream_t st) {
  const size_t n_codes = (size_t)e->K * e->out * e->in;
  PIPE_HIP(hipMemsetAsync(codes, 0, n_codes, st));
  PIPE_HIP(hipMemsetAsync(scales, 0, (size_t)e->K * e->out * sizeof(float), st));
  for (int k = 0; k < e->K; ++k) {
    const PipeOrder& o = e->orders[k];
    const int rows = o.n_kept * e->group;
    if (rows == 0) continue;
    int8_t* tmp = (int8_t*)pipe_ws_get(WS_DIAG_CODES, (size_t)rows * e->in);
    if (!tmp) return pipe_ws_error();
    int rc = launch_unpack_codes(e->codes_dev, o.pos_dev, e->bits, rows, e->in, e->in_pad, tmp, st);
    if (rc) return rc;
    PIPE_KLAUNCH(dense_order_kernel, dim3(rows), dim3(64), 0, st, tmp, e->scales_all_dev, o.pos_dev, o.gids_dev,
                       e->group, e->in, e->out, codes + (size_t)k * e->out * e->in, scales + (size_t)k * e->out);
    PIPE_HIP(hipGetLastError());
  }
  if (cols != nullptr) {
    PIPE_KLAUNCH(pack_columns_kernel, dim3(ceil_div(e->K * 3 * e->out, 256)), dim3(256), 0, st, codes, e->K, e->out, cols);
    PIPE_HIP(hipGetLastError());
  }
  PIPE_HIP(hipStreamSynchronize(st));   // the scratch rows are reused by other calls
  return PIPE_OK;
}

// The expansion holds all of a layer's tables or none: a call that fails on the way leaves nothing for the next to find.
int pipe_depthwise_prepare(pipe_expansion* e, hipStream_t st) {
  if (e->dw_codes_dev != nullptr) return PIPE_OK;
  if (pipe_capturing()) return PIPE_ENOTREADY;   // allocates and synchronizes: run the call once outside capture
  int8_t* codes = nullptr;
  float* scales = nullptr;
  uint32_t* cols = nullptr;
  const char* what = "hipMalloc(depthwise tables)";
  int rc = pipe_hip_ok(hipMalloc(&codes, (size_t)e->K * e->out * e->in), what) &&
           pipe_hip_ok(hipMalloc(&scales, (size_t)e->K * e->out * sizeof(float)), what) &&
           (e->in != 9 || pipe_hip_ok(hipMalloc(&cols, (size_t)e->K * 3 * e->out * sizeof(uint32_t)), what)) ? PIPE_OK : PIPE_ENOMEM;
  if (rc == PIPE_OK) rc = build_tables(e, codes, scales, cols, st);
  if (rc != PIPE_OK) {
    (void)hipStreamSynchronize(st);   // what was launched has ended
    if (codes) (void)hipFree(codes);
    if (scales) (void)hipFree(scales);
    if (cols) (void)hipFree(cols);
    return rc;
  }
  e->dw_codes_dev = codes; e->dw_scales_dev = scales; e->dw_cols_dev = cols;
  return PIPE_OK;
}

int launch_quantize_to_nhwc(const float* x, int N, int C, int HW, float s_static, MaxOf amax, float qmax,
                            int8_t* q8, float* scale_out, hipStream_t st) {
  const int64_t tiles = (int64_t)ceil_div(HW, 32) * ceil_div(C, 32);
  const int images = (int)std::min<int64_t>(N, std::max<int64_t>(1, std::min<int64_t>(NHWC_BLOCKS / tiles, 65535)));
  PIPE_KLAUNCH(quantize_to_nhwc_kernel, dim3(ceil_div(HW, 32), ceil_div(C, 32), images), dim3(256), 0, st, x, N, C, HW, s_static,
                     amax, qmax, q8, scale_out);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

int launch_depthwise(const pipe_expansion* e, const int8_t* q8, const float* s_x, int N, int C, int H, int W, int kh, int kw,
                     int stride, int pad, int Ho, int Wo, int M, const int* lo, const int* hi,
                     const float* bias, int reduce, float* y, hipStream_t st) {
  if (kh * kw > MAX_WIN || (C & 3) != 0) return PIPE_ESHAPE;
  DwParams p;
  p.q8 = q8; p.s_x = s_x; p.codes = e->dw_codes_dev; p.scales = e->dw_scales_dev; p.bias = bias; p.y = y;
  p.N = N; p.C = C; p.H = H; p.W = W; p.kh = kh; p.kw = kw; p.stride = stride; p.pad = pad; p.Ho = Ho; p.Wo = Wo;
  p.K = e->K; p.M = M; p.reduce = reduce;
  for (int m = 0; m < PIPE_MAX_K; ++m) { p.member_lo[m] = m < M ? lo[m] : 0; p.member_hi[m] = m < M ? hi[m] : -1; }
  const long long total = (long long)N * Ho * Wo * (C / 4);
  if (total <= 0) return PIPE_OK;
  const dim3 grid((unsigned)((total + BLK - 1) / BLK));
  if (kh == 3 && kw == 3) PIPE_KLAUNCH((depthwise_kernel<3, 3>), grid, dim3(BLK), 0, st, p);
  else if (kh == 5 && kw == 5) PIPE_KLAUNCH((depthwise_kernel<5, 5>), grid, dim3(BLK), 0, st, p);
  else if (kh == 7 && kw == 7) PIPE_KLAUNCH((depthwise_kernel<7, 7>), grid, dim3(BLK), 0, st, p);
  else PIPE_KLAUNCH((depthwise_kernel<0, 0>), grid, dim3(BLK), 0, st, p);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

// A workgroup of the fused kernel costs nearly as much for a few outputs as for all it has room for (64 channels, 6 or 3 rows, 32
// or 16 columns), while the two-step path runs through the pixels in full waves: many small images, or few channels of them, are
// quicker in two steps.  The lines by outputs a workgroup, 2049 to 24000 workgroups, 16 to 960 channels, 4 bit, K = 3, fused time
// over two-step time: channels last 0.44 to 1.04 from 1024 on (784 outputs of 32 x 7 x 7: up to 1.12, 256 of 64 x 2 x 2: 1.78);
// channels first with 16-byte rows, which two steps have to turn, 0.45 to 0.96 from 576 on (512 of 16 x 8 x 8: 1.46); element by
// element 0.63 to 0.96 from 1536 on (1045 of 16 x 14 x 14: 1.58).  Up to 2048 workgroups the chip is not full and the
// launch that is saved decides (0.41 to 1.02).
bool pipe_depthwise_fused(const pipe_expansion* e, const float* x, int kh, int kw, int stride, int M, int N, int W, int nhwc, int Ho, int Wo) {
  if (e->dw_cols_dev == nullptr || kh != 3 || kw != 3 || (stride != 1 && stride != 2) || M != 1 || e->K > 4) return false;
  const int C = e->out, groups = ceil_div(C, 64);
  const int64_t images = (int64_t)N * ceil_div(Ho, dw3_rows(stride)) * ceil_div(Wo, dw3_columns(stride));   // grid x
  if (images >= (int64_t)1 << 24 || groups > 65535) return false;   // a launch holds fewer than 2^32 threads along x
  const int64_t enough = !dw3_wide(x, W, nhwc) ? 1536 : (nhwc ? 1024 : 576);
  return images * groups <= 2048 || (int64_t)N * Ho * Wo * C >= enough * images * groups;
}

int launch_depthwise_fused(const pipe_expansion* e, const float* x, float s_static, MaxOf amax, float qmax, int N, int C, int H, int W,
                           int stride, int pad, int nhwc, int Ho, int Wo, const float* bias, float* y, hipStream_t st) {
  Dw3Params p;
  p.x = x; p.amax = amax; p.s_static = s_static; p.qmax = qmax;
  p.codes = e->dw_cols_dev; p.scales = e->dw_scales_dev; p.bias = bias; p.y = y;
  p.N = N; p.C = C; p.H = H; p.W = W; p.Ho = Ho; p.Wo = Wo; p.pad = pad; p.nhwc = nhwc;
  p.vec = dw3_wide(x, W, nhwc) ? 1 : 0;
  return stride == 1 ? launch_depthwise3<1>(p, e->K, st) : launch_depthwise3<2>(p, e->K, st);
}
