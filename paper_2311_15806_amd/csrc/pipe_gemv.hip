// Weight-streaming kernel of the expanded layer for decode-sized batches (T <= 16, and up to 128 where the dispatch finds it faster), where the
// path is bound by reading the packed codes from HBM once (App. B, Eq. (define_dre), same
// arithmetic as the tiled kernel).
//
// Work item = one stored row block (16 rows of one order, all of in_features).  A workgroup
// owns a bin of items that together hold every order of a few output row blocks; its waves
// split the k dimension (wave w takes packed tiles w, w+NW, ...), so each wave streams its
// own 1-KiB tiles straight from HBM into registers with fully coalesced 16-byte loads, widens
// them with a shift and a mask and feeds v_mfma_i32_16x16x64_i8 against the 16-token
// activation fragments (also read straight from L2: waves use disjoint k, nothing is shared,
// so the k loop has no LDS traffic and no barrier).  The waves' partial int32 tiles meet in
// LDS and are summed exactly; the epilogue then applies offsets, row scales, activation scale,
// bias and the member sum in a fixed order, so results are bit-reproducible.  A workgroup
// handles one 16-token block; larger batches (up to 128 tokens) run one workgroup per bin and
// token block, on the same XCD, so that the bin still comes from HBM once.  Expansions with more
// than 4 orders have bins of 8, 12 or 16 items: gemm_stream_multi_kernel streams them four at a
// time and keeps the integer tiles of the whole bin in LDS for one epilogue.
#include "pipe_codes.h"

#include <algorithm>
#include <type_traits>

int g_stream_ksplit = 0;   // 0: automatic

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int STREAM_SCALARS = 56;   // bytes of the scalar arguments ahead of the struct
constexpr int R = 4;  // items processed concurrently by a wave (independent load streams)

// byte k of a kernel-argument array, k uniform, without forcing the array into scratch memory
__device__ __forceinline__ int pick(const uint32_t (&a)[PIPE_MAX_K / 4], int k) {
  uint32_t v = a[0];
#pragma unroll
  for (int i = 1; i < PIPE_MAX_K / 4; ++i) v = (i == k >> 2) ? a[i] : v;
  return (int)(v >> (k & 3) * 8 & 255u);
}

struct StreamParams {
  const uint8_t* qx;
  int64_t qx_mstride;
  const int32_t* rowsum;
  int64_t rowsum_mstride;
  const float* s_x;
  int sx_mstride;
  const uint8_t* codes;    // stored row blocks in schedule order: bin b owns positions [b*cap, (b+1)*cap), cap = 4, 8, 12 or 16
  const float* scales;     // 16 row scales per position
  const StreamBin* bins;
  const float* bias;
  long long bias_mstride;  // 0: the first member's (or the sum's) vector; else one vector per member
  float* y;
  int32_t* acc_out;
  uint32_t* amax_out;
  uint32_t* amax_neg;      // if set: positive and negative parts of the range apart
  const float* res;        // skip tensor [res_members, T, out] or nullptr
  long long res_mstride;
  int res_members, res_pre_act;
  uint32_t* zero_after;
  int zero_n;
  uint32_t* zero_big;
  int zero_big_n;
  int T, out, nks, M, reduce, act;
  int ksplit;              // workgroups per bin: each takes a contiguous share of the k tiles
  int n_tb;                // 16-token blocks: one workgroup per (bin, k share, token block)
  int n_bins;
  float s_static;          // QFUSE: given activation scale, or <= 0 for max|x| / act_qmax
  float act_qmax;          // QFUSE: largest activation code
  int32_t* ws_sum;         // [n_bins][ksplit][cap][256] partial tiles of split bins
  uint32_t* ws_cnt;        // [n_bins] arrival counters, zero between launches
  uint32_t member_lo[PIPE_MAX_K / 4], member_hi[PIPE_MAX_K / 4], member_of[PIPE_MAX_K / 4];   // a byte each: a launch copies its arguments on the host
  __device__ __forceinline__ int lo(int m) const { return pick(member_lo, m); }
  __device__ __forceinline__ int hi(int m) const { return pick(member_hi, m); }
  __device__ __forceinline__ int of(int k) const { return pick(member_of, k); }
};

// Of a layer on its own, which quantizes its few tokens itself and has one member: the others of the fields above are what they are here.  With the
// scalars ahead of it 112 bytes, the most that a launch passes at the lower price: of small kernels back to back, launches with up to 112 bytes of arguments
// take 2.65 us each, with 120 and more 3.0 to 3.4.  256 x 256, 16 tokens, in a graph 4.87 us a call with the struct above and 3.90 with this one, eagerly, where the host
// is all there is, 7.9 and 7.7; 11008 x 4096 ternary, one token, 8.6 and 7.6.
struct StreamPlain {
  const float *scales, *bias;
  float* y;
  int32_t* ws_sum;
  uint32_t* ws_cnt;
  int out;
  float s_static, act_qmax;
  static constexpr int M = 1, reduce = 1, act = PIPE_ACT_NONE, zero_n = 0, zero_big_n = 0, res_members = 0, res_pre_act = 0;
  static constexpr long long qx_mstride = 0, bias_mstride = 0, res_mstride = 0;
  static constexpr uint32_t *amax_out = nullptr, *amax_neg = nullptr, *zero_after = nullptr, *zero_big = nullptr;
  static constexpr const float* res = nullptr;
  static constexpr int32_t* acc_out = nullptr;
  __device__ __forceinline__ int lo(int) const { return 0; }
  __device__ __forceinline__ int hi(int) const { return PIPE_MAX_K - 1; }
  __device__ __forceinline__ int of(int) const { return 0; }
};
static_assert(STREAM_SCALARS + sizeof(StreamPlain) <= 112, "arguments of a launch at the lower price");

// What the host passes ahead of the struct
struct StreamCall {
  StreamParams p;
  const float* x_f32;      // QFUSE: the fp32 input [T, in], quantized by every workgroup itself
  int in;                  // in_features (QFUSE: a multiple of 4)
  int thr0, thr1, thr2;    // bins of 4, fullest first: how many hold 4, at least 3, at least 2 items
};

// The sum over a wave whose lanes are all active, by data-parallel moves within the vector unit
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }
__device__ __forceinline__ int wave_sum(int v) {
  v = dpp_add<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: the last lane of 16 holds their sum
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);   // row_bcast 15, 31: lane 63 holds the wave's
  v = dpp_add<0x143, 0xc>(v);
  return __builtin_amdgcn_readlane(v, 63);
}

template <int BITS>
__device__ __forceinline__ void unpack_step(const uint4& w, int j, v4i& o) {
  if (BITS == 8) {
    o = v4i{(int)w.x, (int)w.y, (int)w.z, (int)w.w};
  } else if (BITS == 4) {
    const uint32_t a = j == 0 ? w.x : w.z, b = j == 0 ? w.y : w.w;
    o = v4i{(int)(a & 0x0F0F0F0Fu), (int)((a >> 4) & 0x0F0F0F0Fu), (int)(b & 0x0F0F0F0Fu), (int)((b >> 4) & 0x0F0F0F0Fu)};
  } else {
    const uint32_t a = j == 0 ? w.x : (j == 1 ? w.y : (j == 2 ? w.z : w.w));
    o = v4i{(int)(a & 0x03030303u), (int)((a >> 2) & 0x03030303u), (int)((a >> 4) & 0x03030303u), (int)((a >> 6) & 0x03030303u)};
  }
}

// A partial tile in LDS: 16 words left out behind each 64, so that the 4 tokens x 16 channels a wave sums lie in different banks
constexpr int PART_WORDS = 4 * 80;
__device__ __forceinline__ int part_word(int i) { return i + (i >> 6) * 16; }

// XM = number of distinct activation tensors the items of a bin can read: 1 (one input for all
// orders), or 2 / 4 (one input per ensemble member, at most XM members).
// XMASK: the batch does not fill its last 16-token block; the activation loads of that block are
// issued for the lanes of real tokens only.
// QFUSE (few tokens of few features, one activation tensor): there is no quantizer launch; every
// workgroup reduces max|x| over the few-KiB input itself, quantizes it into LDS with the same
// arithmetic as the quantizer kernels (IEEE division, round half to even) while its first codes are
// on their way, and builds its activation fragments from there.
constexpr int QF_T = 16, QF_IN = 8192;   // tokens; codes of all tokens
constexpr int QF_THREADS = 512;          // of a workgroup that quantizes, each up to QF_IN / 4 / QF_THREADS quads
// What the first loads need comes as scalar arguments ahead of the struct, two to a word: they are in registers with the launch, while the struct has to be
// read from memory first.
// D = tiles an item that a wave asks for together: see two_tiles.
template <int BITS, int NW, int XM, bool ACC_OUT, bool XMASK, bool QFUSE = false, class Params = StreamParams, int D = 1>
__global__ __launch_bounds__(NW * 64, (XM * (BITS == 2 ? 4 : (BITS == 4 ? 2 : 1)) <= 8) ? 4 : 2) void gemm_stream_kernel(
    const uint8_t* a_codes, const StreamBin* a_bins, const void* a_x, uint64_t a_nb_t0, uint64_t a_t1_t2, uint64_t a_in_mg, uint64_t a_sp_T,
    const Params p) {
  const int a_n_bins = (int)a_nb_t0, a_thr0 = (int)(a_nb_t0 >> 32), a_thr1 = (int)a_t1_t2, a_thr2 = (int)(a_t1_t2 >> 32);
  const int a_in = (int)a_in_mg, a_split = (int)a_sp_T, a_T = (int)(a_sp_T >> 32);
  const unsigned a_magic = (unsigned)(a_in_mg >> 32);
  static_assert(!QFUSE || (XM == 1 && !ACC_OUT && NW * 64 == QF_THREADS), "the fused quantizer serves one shared input");
  static_assert(D == 1 || D == 2, "tiles asked for together");
  __shared__ __attribute__((aligned(16))) uint8_t s_qx[QFUSE ? QF_IN : 16];
  __shared__ float s_red[NW];
  __shared__ int s_rs[QF_T];
  constexpr int OFF = BITS == 8 ? 0 : (BITS == 4 ? 8 : 1);
  constexpr int KSUP = 512 / BITS;
  constexpr int STEPS = KSUP / 64;      // 64-k steps per packed tile
  constexpr int NX = XM * STEPS;
  constexpr int BIN_WORDS = sizeof(StreamBin) / 4;
  static_assert(BIN_WORDS <= 64, "bin descriptor is fetched with one load per lane");
  __shared__ __attribute__((aligned(16))) int part[NW][R][PART_WORDS];   // each wave's partial tiles
  __shared__ unsigned s_mx[2 * R];   // the members' largest magnitudes (two-sided: largest values, then of their negatives), as the slots hold them
  __shared__ int s_last;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int in_pad_q = (a_in + 255) & ~255;
  const int n_tiles = in_pad_q / KSUP;

  // Block index -> (bin, k share, token block).  Blocks are handed to the XCDs round robin, so the
  // workgroups that stream the same bin (for different token blocks or k shares) get indices that
  // are equal modulo 8: they run on one XCD and the bin comes from HBM once, then from that L2.
  // A bin has several k shares or several token blocks, not both; a_magic divides by their number.
  const int ksplit = a_split & 255, n_tb = a_split >> 8, subs = ksplit * n_tb;
  const int g8 = (int)(blockIdx.x >> 3);
  const int grp = subs == 1 ? g8 : (int)__umulhi(g8, a_magic);
  const int bin = grp * 8 + (int)(blockIdx.x & 7), sub = g8 - grp * subs;
  const int ksp = ksplit > 1 ? sub : 0, tb = ksplit > 1 ? 0 : sub;
  if (bin >= a_n_bins) return;   // padding of the last group of eight bins

  // epilogue role of this thread: 256 threads per output row block, thread = (token t, channel ch)
  const int e = threadIdx.x & 255;
  const int t = e >> 4, ch = e & 15;   // token inside this workgroup's 16-token block
  const int tg = tb * 16 + t;          // token of the call
  const int fidx = part_word(((ch >> 2) * 16 + t) * 4 + (ch & 3));   // lane*4 + i of the MFMA result layout
  const int o_first = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  constexpr int O_STEP = (NW * 64) / 256;

  // ---- everything that does not depend on the bin descriptor is requested first: where the bin's
  // stored row blocks sit in the schedule-ordered buffers follows from the bin's index (below), so
  // the code stream (the HBM traffic that bounds this kernel) starts at once.  Wave w streams
  // tiles w, w+NW, ..., one tile per item in flight: with exact waits two, three and four were the slower the more (11008 x 4096 8 bit, 16 tokens,
  // call 24.2 us / 27.1 / 29.8 / 30.3; 4 bit, one token 12.2 / 14.2; six ternary layers of 2048, two members, 50 tokens 77.8 / 89.6).  At 8 bits two that are
  // asked for and waited for together can be faster, see two_tiles.
  // All loads go through buffer resources that end with this workgroup's share of the k tiles: an item that the bin does not have, a tile beyond
  // the share and a token beyond the batch read as zero without any access, so that with one tile at a time no load is behind a branch and every wait is an exact count.
  const int tile_lo = ksplit > 1 ? (int)__umulhi(n_tiles * ksp, a_magic) : 0;
  const int tile_hi = ksplit > 1 ? (int)__umulhi(n_tiles * (ksp + 1), a_magic) : n_tiles;
  // quantizing workgroups request their input before the codes: it is what they wait for first (results return in order)
  constexpr int XQ = QF_IN / 4 / QF_THREADS;
  v4f xq[QFUSE ? XQ : 1];
  const __amdgpu_buffer_rsrc_t l_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a_x), 0, (unsigned)(a_T * a_in * 4), 0x00020000);
  if constexpr (QFUSE) {
#pragma unroll
    for (int i = 0; i < XQ; ++i) xq[i] = (v4f)__builtin_amdgcn_raw_buffer_load_b128(l_q, (threadIdx.x + i * QF_THREADS) * 16, 0, 0);
  }
  auto load_d = [&]() __attribute__((always_inline)) { return reinterpret_cast<const int32_t*>(a_bins + bin)[min(lane, BIN_WORDS - 1)]; };
  int d0 = 0;
  if (XM > 1) d0 = load_d();   // says which activations an item multiplies
  // the bin's first position and item count, from its index: the bins lie without gaps, fullest first
  const int b3 = max(bin - a_thr0, 0), b2 = max(bin - a_thr1, 0), b1 = max(bin - a_thr2, 0);
  const int n_here = bin < a_thr0 ? 4 : (bin < a_thr1 ? 3 : (bin < a_thr2 ? 2 : 1));
  const int pos0 = 4 * bin - b3 - b2 - b1;
  __amdgpu_buffer_rsrc_t l_w[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    l_w[r] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a_codes) + (size_t)(pos0 + (r < n_here ? r : 0)) * n_tiles * 1024, 0,
                                               r < n_here ? (unsigned)tile_hi * 1024u : 0u, 0x00020000);
  v4u w[D][R];
  v4i x[D][NX];
  auto load_w = [&](int tl, v4u (&w)[R]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < R; ++r) w[r] = (v4u)__builtin_amdgcn_raw_buffer_load_b128(l_w[r], tl * 1024 + lane * 16, 0, 0);
  };
  // member m's activations
  const size_t x_tb = (size_t)tb * in_pad_q * 16;
  __amdgpu_buffer_rsrc_t l_x[XM];
  if constexpr (!QFUSE) {
#pragma unroll
    for (int m = 0; m < XM; ++m) {
      const bool on = m == 0 || m < p.M;
      l_x[m] = __builtin_amdgcn_make_buffer_rsrc((uint8_t*)const_cast<void*>(a_x) + (m > 0 && on ? (size_t)m * p.qx_mstride : 0) + x_tb, 0,
                                                 on ? (unsigned)(tile_hi * STEPS) * 1024u : 0u, 0x00020000);
    }
  }
  const unsigned x_off = !XMASK || tb * 16 + (lane & 15) < a_T ? lane * 16u : 0x80000000u;
  auto load_x = [&](int tl, v4i (&x)[NX]) __attribute__((always_inline)) {
    if constexpr (QFUSE) {
      // the fragment of a 64-k step: lane (kc, n) holds codes 16 kc .. 16 kc + 15 of token n (of the last one beyond it: never stored)
      const uint8_t* row = &s_qx[min(lane & 15, a_T - 1) * in_pad_q + (lane >> 4) * 16];
      const int at = min(tl, tile_hi - 1) * STEPS;
#pragma unroll
      for (int j = 0; j < STEPS; ++j) x[j] = *reinterpret_cast<const v4i*>(row + (at + j) * 64);
    } else {
#pragma unroll
      for (int m = 0; m < XM; ++m)
#pragma unroll
        for (int j = 0; j < STEPS; ++j) x[m * STEPS + j] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(l_x[m], x_off + (tl * STEPS + j) * 1024u, 0, 0);
    }
  };
  int tl = tile_lo + wave;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    load_w(tl + d * NW, w[d]);
    if (!QFUSE) load_x(tl + d * NW, x[d]);
  }
  __builtin_amdgcn_sched_barrier(0);
  request_arguments<sizeof(Params) + STREAM_SCALARS>();
  if (XM == 1) d0 = load_d();
  // epilogue operands that need no descriptor: row scales (same positions), and per member the
  // activation scale and this thread's token code sum
  const bool fold_sx = p.reduce && p.M > 1;
  float scv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) scv[r] = p.scales[(size_t)(pos0 + (r < n_here ? r : 0)) * 16 + ch];
  float sxm[R];
  int rsm[R];
  if constexpr (!QFUSE) {
#pragma unroll
    for (int m = 0; m < R; ++m) {       // at most R members (K <= R), and XM where each has its own input
      if (XM > 1 && m >= XM) { sxm[m] = 0.f; rsm[m] = 0; continue; }
      const int mm = m < p.M ? m : p.M - 1;
      sxm[m] = p.s_x[mm * p.sx_mstride];
      rsm[m] = OFF ? p.rowsum[(size_t)mm * p.rowsum_mstride + tg] : 0;
    }
  } else {
    // ---- quantize the input here (the codes already requested are on their way meanwhile)
    const int n4 = (a_T * a_in) >> 2;
    if ((int)threadIdx.x < QF_T) s_rs[threadIdx.x] = 0;
    float s_act = p.s_static;
    if (!(s_act > 0.f)) {
      float mx = 0.f;
#pragma unroll
      for (int i = 0; i < XQ; ++i) mx = fmaxf(mx, fmaxf(fmaxf(fabsf(xq[i].x), fabsf(xq[i].y)), fmaxf(fabsf(xq[i].z), fabsf(xq[i].w))));
      mx = wave_max(mx);
      if (lane == 0) s_red[wave] = mx;
      __syncthreads();
      mx = s_red[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_red[w]);
      s_act = __fdiv_rn(mx, p.act_qmax);
    } else {
      __syncthreads();   // the cleared code sums
    }
    const bool live_q = s_act > 0.f;
    const Divisor div(s_act);
    const float per_row = __builtin_amdgcn_rcpf((float)a_in);
    const bool by_wave = a_T == 1 || a_in % 256 == 0;   // a wave's 64 quads lie in one row (behind the input they are zero)
    auto quantize = [&](auto fast, int i, const v4f& v) __attribute__((always_inline)) {
      auto q1 = [&](float f) __attribute__((always_inline)) {
        const float q = fminf(fmaxf(rintf(div.template quotient<decltype(fast)::value>(f)), -p.act_qmax), p.act_qmax);
        return live_q ? (int)q : 0;
      };
      // in_features is a multiple of 4: one token per quad.  The estimate is exact: the quotient, up to 16, is at least 1/2 / 8192 from
      // the next whole number.
      const int tq = a_T == 1 ? 0 : min((int)(((float)(i * 4) + 0.5f) * per_row), a_T - 1);
      const int a = q1(v.x), b = q1(v.y), c = q1(v.z), d = q1(v.w);
      if (i < n4) *reinterpret_cast<uint32_t*>(&s_qx[tq * in_pad_q + i * 4 - tq * a_in]) = pack4(a, b, c, d);
      int sum = a + b + c + d;
      if (by_wave) sum = wave_sum(sum);
      if (by_wave ? lane == 0 : sum != 0) atomicAdd(&s_rs[tq], sum);
    };
    if (div.fast) {
#pragma unroll
      for (int u = 0; u < XQ; ++u)
        if (u * QF_THREADS + wave * 64 < n4) quantize(std::true_type{}, threadIdx.x + u * QF_THREADS, xq[u]);
    } else {
#pragma unroll 1
      for (int u = 0; u * QF_THREADS + wave * 64 < n4; ++u)
        quantize(std::false_type{}, threadIdx.x + u * QF_THREADS, (v4f)__builtin_amdgcn_raw_buffer_load_b128(l_q, (threadIdx.x + u * QF_THREADS) * 16, 0, 0));
    }
    // codes beyond in_features are zero
    const int pad4 = (in_pad_q - a_in) >> 2;
    for (int i = threadIdx.x; i < a_T * pad4; i += NW * 64) {
      const int tq = i / pad4, k = a_in + (i - tq * pad4) * 4;
      *reinterpret_cast<uint32_t*>(&s_qx[(size_t)tq * in_pad_q + k]) = 0u;
    }
    __syncthreads();
    const int rs_q = (OFF && tg < a_T) ? s_rs[min(tg, QF_T - 1)] : 0;
#pragma unroll
    for (int m = 0; m < R; ++m) { sxm[m] = s_act; rsm[m] = rs_q; }
  }

  // ---- the descriptor: scalar reads out of one vector register, with one input only behind the codes (it arrives after them)
  auto word = [&](int i) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(d0, i); };
  int itm[R];   // which activation tensor item r reads
#pragma unroll
  for (int r = 0; r < R; ++r) itm[r] = XM == 1 ? 0 : p.of(word(2 + (r < n_here ? r : 0)));

  v4i acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = v4i{0, 0, 0, 0};
  auto mul_tile = [&](v4u (&w)[R], v4i (&x)[NX]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v4i xf = x[j];
#pragma unroll
        for (int m = 1; m < XM; ++m) {   // uniform select, component by component
          const bool pickm = itm[r] == m;
#pragma unroll
          for (int c = 0; c < 4; ++c) xf[c] = pickm ? x[m * STEPS + j][c] : xf[c];
        }
        v4i wf;
        unpack_step<BITS>(make_uint4(w[r].x, w[r].y, w[r].z, w[r].w), j, wf);
        acc[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf, xf, acc[r], 0, 0, 0);
      }
    }
  };
  if constexpr (D == 1) {
    // The first tile stands apart: behind it are the epilogue's operands, of which the loop's waits know nothing.
    if (QFUSE) load_x(tl, x[0]);
    mul_tile(w[0], x[0]);
    for (tl += NW; tl < tile_hi; tl += NW) {
      load_w(tl, w[0]);
      load_x(tl, x[0]);
      mul_tile(w[0], x[0]);
    }
  } else {
    // The branches make the wait at the loop's head one for both tiles, and their loads leave back to back.  Without branches and with exact waits, so that one
    // tile is on its way while the other is multiplied, or with the loads of both mixed, 16384 x 4096, K = 4, 123 tokens took 137 to 140 us,
    // with one tile 136, in this form 125.
    if (QFUSE) { load_x(tl, x[0]); load_x(tl + NW, x[D - 1]); }
    for (; tl < tile_hi; tl += 2 * NW) {
      mul_tile(w[0], x[0]);
      if (tl + 2 * NW < tile_hi) { load_w(tl + 2 * NW, w[0]); load_x(tl + 2 * NW, x[0]); }
      if (tl + NW < tile_hi) {
        mul_tile(w[D - 1], x[D - 1]);
        if (tl + 3 * NW < tile_hi) { load_w(tl + 3 * NW, w[D - 1]); load_x(tl + 3 * NW, x[D - 1]); }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
    *reinterpret_cast<v4i*>(&part[wave][r][part_word(lane * 4)]) = acc[r];
  const int n_items = word(0), n_out = word(1);
  int itk[R], its[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool on = r < n_items;
    itk[r] = word(2 + (on ? r : 0));
    its[r] = on ? word(2 + STREAM_BIN_CAP + r) : -1;
  }
  auto out_rb = [&](int o) __attribute__((always_inline)) { return word(2 + 2 * STREAM_BIN_CAP + o); };
  if (blockIdx.x == 0 && p.zero_after != nullptr) slots_clear<NW * 64>(p.zero_after, p.zero_n);
  if (p.zero_big != nullptr)
    for (int i = (bin * subs + sub) * (NW * 64) + threadIdx.x; i < p.zero_big_n; i += a_n_bins * subs * (NW * 64)) p.zero_big[i] = 0u;
  if (threadIdx.x < 2 * R) s_mx[threadIdx.x] = 0u;
  __syncthreads();

  // A split bin: every workgroup writes its integer partial tiles to its own slice of the bin's
  // workspace with device-scope stores (written through to memory, no cache maintenance), waits
  // for them to complete (vmcnt counts stores) and then counts its arrival; the one that arrives
  // last reads all slices with device-scope loads, sums them (exact, order independent), resets
  // the counter and runs the epilogue.  Nobody waits for anybody.
  // What this relies on is the hardware's behaviour, not the language's memory model (all accesses
  // are relaxed): a device-scope store is written through to the memory-side cache all compute
  // units share, s_waitcnt vmcnt(0) returns only once every such store of the wave has been
  // acknowledged from there, the barrier extends that to the workgroup, and only then is the
  // counter raised; the reader's device-scope loads bypass its own caches.  A release/acquire pair
  // on the counter would express the same order in the model; its cache write-back and invalidate
  // measured 11 to 34 us per exchange on this chip, more than the kernel.
  if (ksplit > 1) {
    int32_t* ws = p.ws_sum + ((size_t)bin * ksplit + ksp) * (R * 256);
    for (int i = threadIdx.x; i < R * 256; i += NW * 64) {
      int a = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) a += part[w][i >> 8][part_word(i & 255)];
      __hip_atomic_store(&ws[i], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&p.ws_cnt[bin], 1u) == (unsigned)(ksplit - 1);
    __syncthreads();
    if (!s_last) return;
    const int32_t* wsb = p.ws_sum + (size_t)bin * ksplit * (R * 256);
    for (int i = threadIdx.x; i < R * 256; i += NW * 64) {
      int a = 0;
      for (int q = 0; q < ksplit; ++q) a += __hip_atomic_load(&wsb[(size_t)q * (R * 256) + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      part[0][i >> 8][part_word(i & 255)] = a;
#pragma unroll
      for (int w = 1; w < NW; ++w) part[w][i >> 8][part_word(i & 255)] = 0;
    }
    if (threadIdx.x == 0) __hip_atomic_store(&p.ws_cnt[bin], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
  }

  // epilogue: exact integer sum over the waves, then the fixed-order fp32 sum (same evaluation
  // order as the tiled kernel): one member, or members kept apart:
  //   y_m = s_x,m * (sum_k s_k * a_k) + b;  members summed: y = sum_m sum_k (s_k * s_x,m) * a_k + b.
  for (int o = o_first; o < n_out; o += O_STEP) {
    // a row block's items are adjacent, in ascending order k
    const int col = out_rb(o) * 16 + ch;
    const float bias = p.bias != nullptr ? p.bias[col] : 0.f;
    float yacc = 0.f;
#pragma unroll
    for (int m = 0; m < R; ++m) {
      if (m >= p.M) break;
      const int rs = rsm[m];
      const float sx = sxm[m];
      const int k_lo = p.lo(m), k_hi = p.hi(m);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (its[r] != o || itk[r] < k_lo || itk[r] > k_hi) continue;
        int a = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) a += part[w][r][fidx];
        a -= OFF * rs;
        const float sc = fold_sx ? scv[r] * sx : scv[r];
        yacc = fmaf(sc, (float)a, yacc);
        if (ACC_OUT) {
          if (tg < a_T) p.acc_out[((size_t)itk[r] * a_T + tg) * p.out + col] = a;
        }
      }
      if (ACC_OUT) continue;
      if (fold_sx && m + 1 < p.M) continue;
      const float bm = (m == 0 || fold_sx) ? bias : (p.bias_mstride != 0 && p.bias != nullptr ? p.bias[(size_t)m * p.bias_mstride + col] : 0.f);
      float v = fold_sx ? yacc + bm : fmaf(sx, yacc, bm);   // same rounding as the tiled kernel
      yacc = 0.f;
      float rsum = 0.f;
      if (p.res != nullptr) {
        // the members summed into this output each add their own skip tensor
        const int n_res = p.reduce ? p.res_members : (m < p.res_members ? 1 : 0);
        const float* rp = p.res + (size_t)(p.reduce ? 0 : m) * p.res_mstride + (size_t)min(tg, a_T - 1) * p.out + col;
        for (int mm = 0; mm < n_res; ++mm) rsum += rp[(size_t)mm * p.res_mstride];
      }
      if (p.res_pre_act) v += rsum;
      if (p.act == PIPE_ACT_GELU) v = gelu_erf(v);
      else if (p.act == PIPE_ACT_RELU) v = fmaxf(v, 0.f);
      if (!p.res_pre_act) v += rsum;
      if (p.amax_out != nullptr) {
        const bool two_sided = p.amax_neg != nullptr;
        float mx = tg < a_T ? (two_sided ? fmaxf(v, 0.f) : fabsf(v)) : 0.f;
        mx = wave_max(mx);
        if (lane == 0) atomicMax(&s_mx[m], __float_as_uint(mx));
        if (two_sided) {
          float mn = tg < a_T ? fmaxf(-v, 0.f) : 0.f;
          mn = wave_max(mn);
          if (lane == 0) atomicMax(&s_mx[R + m], __float_as_uint(mn));
        }
      }
      if (tg < a_T) p.y[((size_t)(p.reduce ? 0 : m) * a_T + tg) * p.out + col] = v;
    }
  }
  // One raise of a member's slot per workgroup.  By every wave and row block the raises were what a launch of many tokens waited for (waves that end
  // together all find the slot low), the longer the quicker the activation ran: MLP 1024-4096-1024 4 bit, K = 3 in 2 and 1, GELU, 32 tokens
  // 33.8 us with erff and 37.1 with the polynomial, 79 tokens 49.5; so 25.4 and 34.5; six 2048 x 2048 ternary layers of two members, 128 tokens 201 -> 131.
  if (!ACC_OUT && p.amax_out != nullptr) {
    __syncthreads();
    const int m = threadIdx.x & (R - 1), neg = threadIdx.x / R;
    if (neg < (p.amax_neg != nullptr ? 2 : 1) && m < p.M)
      slot_raise(neg ? &p.amax_neg[m] : &p.amax_out[m], __uint_as_float(s_mx[threadIdx.x]));
  }
}

// Bins of CAP = 4 * NCH items (expansions with 5 to 16 orders).  The workgroup streams the bin in
// chunks of R = 4 items exactly as above (waves split k, one tile per item in flight; with two, and every wave raising the maxima itself, seven layers of 2048
// ternary with two members of 4 orders took 138 us at 40 tokens instead of 92.7, 94.6 at 16 instead of 81.8; at 8 bits two, 400 calls of 5 to 12 orders -5 % in the mean:
// 1024 x 11008, K = 5, 69 tokens 37.3 us with one and 28.5 with two, 512 x 8192, 123 26.6 and 22.7, 4 layers of 3072, two members of 6, 49 167 and 178), reduces
// each chunk's per-wave tiles into isum and runs one epilogue over all items: per output row
// block and member the items are summed in ascending order k, the same fp32 order as everywhere.
// XM = 1: all items read one activation tensor; XM = 4: one stream per item of the chunk (its
// member's tensor; the streams need the bin descriptor, so it is fetched first).
template <int BITS, int NW, int XM, int NCH>
__global__ __launch_bounds__(NW * 64, 2) void gemm_stream_multi_kernel(const StreamParams p) {
  static_assert(XM == 1 || XM == R, "one stream, or one per item of a chunk");
  constexpr int CAP = R * NCH;
  constexpr int D = BITS == 8 ? 2 : 1;   // tiles that a wave asks for together
  constexpr int OFF = BITS == 8 ? 0 : (BITS == 4 ? 8 : 1);
  constexpr int KSUP = 512 / BITS;
  constexpr int STEPS = KSUP / 64;
  constexpr int NX = XM * STEPS;
  constexpr int BIN_WORDS = sizeof(StreamBin) / 4;
  static_assert(BIN_WORDS <= 64, "bin descriptor is fetched with one load per lane");
  __shared__ int part[NW][R][256];   // each wave's partial tiles of the current chunk
  __shared__ int isum[CAP][256];     // the bin's integer tiles, summed over the waves
  __shared__ unsigned s_mx[2 * PIPE_MAX_K];   // the members' largest magnitudes, as above
  __shared__ int s_last;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_tiles = (p.nks * 64) / KSUP;
  if (blockIdx.x == 0 && p.zero_after != nullptr) slots_clear<NW * 64>(p.zero_after, p.zero_n);
  if (p.zero_big != nullptr)
    for (int i = blockIdx.x * (NW * 64) + threadIdx.x; i < p.zero_big_n; i += gridDim.x * (NW * 64)) p.zero_big[i] = 0u;

  const int subs = p.ksplit * p.n_tb;
  const int grp = (int)blockIdx.x / (8 * subs), within = (int)blockIdx.x - grp * (8 * subs);
  const int bin = grp * 8 + (within & 7), sub = within >> 3;
  const int ksp = sub % p.ksplit, tb = sub / p.ksplit;
  if (bin >= p.n_bins) return;

  const int e = threadIdx.x & 255;
  const int t = e >> 4, ch = e & 15;
  const int tg = tb * 16 + t;
  const int fidx = ((ch >> 2) * 16 + t) * 4 + (ch & 3);
  const int o_first = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  constexpr int O_STEP = (NW * 64) / 256;
  const bool fold_sx = p.reduce && p.M > 1;
  const int tile_lo = (int)((long long)n_tiles * ksp / p.ksplit), tile_hi = (int)((long long)n_tiles * (ksp + 1) / p.ksplit);

  const int d0 = lane < BIN_WORDS ? reinterpret_cast<const int32_t*>(p.bins + bin)[lane] : 0;
  auto word = [&](int i) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(d0, i); };
  auto out_rb = [&](int o) __attribute__((always_inline)) { return word(2 + 2 * STREAM_BIN_CAP + o); };
  // epilogue operands, requested now and used (or staged in LDS) only after the code stream has
  // started: this thread's row scale of every item, and per member the activation scale and
  // the token's code sum
  float scv[CAP];
#pragma unroll
  for (int r = 0; r < CAP; ++r) scv[r] = p.scales[((size_t)bin * CAP + r) * 16 + ch];
  __shared__ float s_sx[PIPE_MAX_K];
  __shared__ int s_rs[PIPE_MAX_K][16];
  const float my_sx = (int)threadIdx.x < p.M ? p.s_x[threadIdx.x * p.sx_mstride] : 0.f;
  const int my_rs = (OFF && (int)threadIdx.x < p.M * 16)
                        ? p.rowsum[(size_t)(threadIdx.x >> 4) * p.rowsum_mstride + tb * 16 + (threadIdx.x & 15)] : 0;
  auto stage_member_operands = [&]() __attribute__((always_inline)) {
    if ((int)threadIdx.x < p.M) s_sx[threadIdx.x] = my_sx;
    if (OFF && (int)threadIdx.x < p.M * 16) s_rs[threadIdx.x >> 4][threadIdx.x & 15] = my_rs;
    if (threadIdx.x < 2 * PIPE_MAX_K) s_mx[threadIdx.x] = 0u;
  };

  // One chunk of R items streamed by WPC waves (wave slot wk of WPC takes tiles wk, wk+WPC, ...);
  // leaves the wave's partial tiles in part[wave].
  auto run_chunk = [&](int c, int wk, int wpc) __attribute__((always_inline)) {
    v4i acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = v4i{0, 0, 0, 0};
    {
      // The codes are requested before anything that needs the bin descriptor (their positions
      // follow from the block index; unused positions of a bin hold zeros and are streamed too).
      const size_t pos0 = (size_t)bin * CAP + (size_t)c * R;
      const uint8_t* wb[R];
#pragma unroll
      for (int r = 0; r < R; ++r) wb[r] = p.codes + (pos0 + r) * (size_t)n_tiles * 1024;
      uint4 w[D][R], x[D][NX];
      auto load_w = [&](int tl, uint4 (&w)[R]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < R; ++r) w[r] = reinterpret_cast<const uint4*>(wb[r] + (size_t)tl * 1024)[lane];
      };
#pragma unroll
      for (int d = 0; d < D; ++d)
#pragma unroll
        for (int r = 0; r < R; ++r) w[d][r] = make_uint4(0, 0, 0, 0);
      int tl = tile_lo + wk;
#pragma unroll
      for (int d = 0; d < D; ++d)
        if (tl + d * wpc < tile_hi) load_w(tl + d * wpc, w[d]);
      const int n_items = word(0);
      const uint8_t* xb[XM];
#pragma unroll
      for (int s = 0; s < XM; ++s) {
        // stream s feeds item s of the chunk: its member's tensor (items beyond the bin's last repeat it)
        const int it = min(c * R + s, n_items - 1);
        const int mem = XM == 1 ? 0 : p.of(word(2 + it));
        xb[s] = p.qx + (size_t)mem * p.qx_mstride + (size_t)tb * p.nks * 1024;
      }
      auto load_x = [&](int tl, uint4 (&x)[NX]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < XM; ++s)
#pragma unroll
          for (int j = 0; j < STEPS; ++j) x[s * STEPS + j] = reinterpret_cast<const uint4*>(xb[s] + (size_t)(tl * STEPS + j) * 1024)[lane];
      };
#pragma unroll
      for (int d = 0; d < D; ++d)
#pragma unroll
        for (int j = 0; j < NX; ++j) x[d][j] = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int d = 0; d < D; ++d)
        if (tl + d * wpc < tile_hi) load_x(tl + d * wpc, x[d]);
      auto mul_tile = [&](uint4 (&w)[R], uint4 (&x)[NX]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const uint4& xs = x[(XM == 1 ? 0 : r) * STEPS + j];
            const v4i xf = v4i{(int)xs.x, (int)xs.y, (int)xs.z, (int)xs.w};
            v4i wf;
            unpack_step<BITS>(w[r], j, wf);
            acc[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf, xf, acc[r], 0, 0, 0);
          }
        }
      };
      if constexpr (D == 1) {
        if (tl < tile_hi) mul_tile(w[0], x[0]);
        for (tl += wpc; tl < tile_hi; tl += wpc) {
          load_w(tl, w[0]);
          load_x(tl, x[0]);
          mul_tile(w[0], x[0]);
        }
      } else {
        for (; tl < tile_hi; tl += 2 * wpc) {
          mul_tile(w[0], x[0]);
          if (tl + 2 * wpc < tile_hi) { load_w(tl + 2 * wpc, w[0]); load_x(tl + 2 * wpc, x[0]); }
          if (tl + wpc < tile_hi) {
            mul_tile(w[D - 1], x[D - 1]);
            if (tl + 3 * wpc < tile_hi) { load_w(tl + 3 * wpc, w[D - 1]); load_x(tl + 3 * wpc, x[D - 1]); }
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
      *reinterpret_cast<v4i*>(&part[wave][r][lane * 4]) = acc[r];
  };
  if constexpr (NW % NCH == 0) {
    // the waves share out the chunks: NW / NCH waves per chunk, all chunks in flight at once
    constexpr int WPC = NW / NCH;
    run_chunk(wave / WPC, wave % WPC, WPC);
    stage_member_operands();
    __syncthreads();
    for (int i = threadIdx.x; i < CAP * 256; i += NW * 64) {
      const int c = i / (R * 256), j = i - c * (R * 256);
      int a = 0;
#pragma unroll
      for (int w = 0; w < WPC; ++w) a += (&part[c * WPC + w][0][0])[j];
      (&isum[0][0])[i] = a;
    }
    __syncthreads();
  } else {
    for (int c = 0; c < NCH; ++c) {
      if (c > 0 && c * R >= word(0)) continue;   // uniform; chunk 0 always holds items
      run_chunk(c, wave, NW);
      if (c == 0) stage_member_operands();
      __syncthreads();
      for (int i = threadIdx.x; i < R * 256; i += NW * 64) {
        int a = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) a += (&part[w][0][0])[i];
        (&isum[c * R][0])[i] = a;
      }
      __syncthreads();   // part is free for the next chunk, isum of this one complete
    }
  }

  const int n_items = word(0), n_out = word(1);
  // a split bin: as in the 4-item kernel, over the tiles of the bin's n_items items
  if (p.ksplit > 1) {
    const int n_words = n_items * 256;
    int32_t* ws = p.ws_sum + ((size_t)bin * p.ksplit + ksp) * (CAP * 256);
    for (int i = threadIdx.x; i < n_words; i += NW * 64)
      __hip_atomic_store(&ws[i], (&isum[0][0])[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&p.ws_cnt[bin], 1u) == (unsigned)(p.ksplit - 1);
    __syncthreads();
    if (!s_last) return;
    const int32_t* wsb = p.ws_sum + (size_t)bin * p.ksplit * (CAP * 256);
    for (int i = threadIdx.x; i < n_words; i += NW * 64) {
      int a = 0;
      for (int q = 0; q < p.ksplit; ++q) a += __hip_atomic_load(&wsb[(size_t)q * (CAP * 256) + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      (&isum[0][0])[i] = a;
    }
    if (threadIdx.x == 0) __hip_atomic_store(&p.ws_cnt[bin], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
  }

  // epilogue over all items of the bin (same arithmetic and order as the 4-item kernel)
  for (int o = o_first; o < n_out; o += O_STEP) {
    const int col = out_rb(o) * 16 + ch;
    const float bias = p.bias != nullptr ? p.bias[col] : 0.f;
    float yacc = 0.f;
    for (int m = 0; m < p.M; ++m) {
      const float sx = s_sx[m];
      const int rs = OFF ? s_rs[m][t] : 0;
      const int k_lo = p.lo(m), k_hi = p.hi(m);
#pragma unroll
      for (int r = 0; r < CAP; ++r) {
        const int kk = word(2 + r);
        if (r >= n_items || word(2 + STREAM_BIN_CAP + r) != o || kk < k_lo || kk > k_hi) continue;   // uniform
        const int a = isum[r][fidx] - OFF * rs;
        const float sc = fold_sx ? scv[r] * sx : scv[r];
        yacc = fmaf(sc, (float)a, yacc);
      }
      if (fold_sx && m + 1 < p.M) continue;
      const float bm = (m == 0 || fold_sx) ? bias : (p.bias_mstride != 0 && p.bias != nullptr ? p.bias[(size_t)m * p.bias_mstride + col] : 0.f);
      float v = fold_sx ? yacc + bm : fmaf(sx, yacc, bm);
      yacc = 0.f;
      float rsum = 0.f;
      if (p.res != nullptr) {
        const int n_res = p.reduce ? p.res_members : (m < p.res_members ? 1 : 0);
        const float* rp = p.res + (size_t)(p.reduce ? 0 : m) * p.res_mstride + (size_t)min(tg, p.T - 1) * p.out + col;
        for (int mm = 0; mm < n_res; ++mm) rsum += rp[(size_t)mm * p.res_mstride];
      }
      if (p.res_pre_act) v += rsum;
      if (p.act == PIPE_ACT_GELU) v = gelu_erf(v);
      else if (p.act == PIPE_ACT_RELU) v = fmaxf(v, 0.f);
      if (!p.res_pre_act) v += rsum;
      if (p.amax_out != nullptr) {
        const bool two_sided = p.amax_neg != nullptr;
        float mx = tg < p.T ? (two_sided ? fmaxf(v, 0.f) : fabsf(v)) : 0.f;
        mx = wave_max(mx);
        if (lane == 0) atomicMax(&s_mx[m], __float_as_uint(mx));
        if (two_sided) {
          float mn = tg < p.T ? fmaxf(-v, 0.f) : 0.f;
          mn = wave_max(mn);
          if (lane == 0) atomicMax(&s_mx[PIPE_MAX_K + m], __float_as_uint(mn));
        }
      }
      if (tg < p.T) p.y[((size_t)(p.reduce ? 0 : m) * p.T + tg) * p.out + col] = v;
    }
  }
  if (p.amax_out != nullptr) {   // one raise of a member's slot per workgroup
    __syncthreads();
    const int m = threadIdx.x & (PIPE_MAX_K - 1), neg = threadIdx.x / PIPE_MAX_K;
    if (neg < (p.amax_neg != nullptr ? 2 : 1) && m < p.M)
      slot_raise(neg ? &p.amax_neg[m] : &p.amax_out[m], __uint_as_float(s_mx[threadIdx.x]));
  }
}

template <int BITS, int NW, int NCH>
int launch_multi(const StreamParams& p, int n_bins, int xm, const GemmArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)((n_bins + 7) / 8 * 8 * p.ksplit * p.n_tb)), blk(NW * 64);
  if (xm == 1) PIPE_LAUNCH((gemm_stream_multi_kernel<BITS, NW, 1, NCH>), grid, blk, st, a.ev_start, a.ev_stop, p);
  else PIPE_LAUNCH((gemm_stream_multi_kernel<BITS, NW, R, NCH>), grid, blk, st, a.ev_start, a.ev_stop, p);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

template <int BITS>
int launch_multi_cap(const StreamParams& p, int n_bins, int cap, int xm, const GemmArgs& a, hipStream_t st) {
  switch (cap) {
    case 8: return launch_multi<BITS, 8, 2>(p, n_bins, xm, a, st);
    case 12: return launch_multi<BITS, 8, 3>(p, n_bins, xm, a, st);
    case 16: return launch_multi<BITS, 8, 4>(p, n_bins, xm, a, st);
    default: return PIPE_ESHAPE;
  }
}

// a bin's workgroups are subs = ksplit * n_tb, of which one factor is 1: the first whole number above (2^32 - 1) / subs, ceil(2^32 / subs), gives floor(i / subs) as the product's upper half while
// 7 i < 2^32
inline uint64_t two_words(int lo, uint32_t hi) { return (uint64_t)(uint32_t)lo | (uint64_t)hi << 32; }
#define PIPE_STREAM_ARGS(x, params)                                                                                      \
  p.codes, p.bins, (const void*)(x), two_words(p.n_bins, c.thr0), two_words(c.thr1, c.thr2),                             \
      two_words(c.in, 0xffffffffu / (unsigned)(p.ksplit * p.n_tb) + 1u), two_words(p.ksplit | p.n_tb << 8, p.T), params

// At 8 bits a tile is one multiplication an item behind 5 KiB of loads, and a wave with one tile at a time does not keep the caches busy.  Two at a time against
// one, calls of 1700 layers:
//   17 to 128 tokens -1 to -12 % in the mean of every class of bins, token blocks and steps of k (320 x 16384, K = 2, 107 tokens 30.6 -> 25.9 us, 8192 x 8192, K = 4, 111
//   122.7 -> 113.9; at worst 11008 x 4096, K = 2, 32 24.8 -> 26.8);
//   up to 16 tokens, where all codes come from HBM, from 1024 bins on -3 to -8 % (28672 x 3584, K = 3, 2 tokens 53.9 -> 49.6), from 512 on walks of 16 tiles a wave
//   -3 to -9 % (16384 x 8192, K = 3, 2 83.7 -> 75.7); fewer -2 to +3 %, single layers +10 % (28672 x 4096, K = 2, 16 45.1 -> 49.6);
//   one token that the launch quantizes itself, from 128 bins on walks of more than 8 tiles 0 to -16 % (28672 x 8192, K = 2 100 -> 84; 4096 x 8192 17.3 -> 15.4), above
//   1280 bins -1 to -11 %; 20480 x 4096, K = 2 +13 %, shorter walks -9 to +9 %.
// With an input for each member +6 to +16 % (chains of 1536 to 3072, 65 to 128 tokens: more registers, one workgroup less a compute unit); at 4 bits -4 to +3 %, at 2
// bits 0 to +5 % on walks of more than a tile a wave.
inline bool two_tiles(const StreamParams& p, bool fused) {
  if (fused) return p.n_bins > 1280 || (p.n_bins >= 128 && p.nks > 64);
  return p.n_tb > 1 || p.n_bins >= 1024 || (p.nks >= 128 && p.n_bins >= 512);
}

template <int BITS, int NW>
int launch_nw(const StreamCall& c, int n_bins, int xm, bool acc_out, const GemmArgs& a, hipStream_t st) {
  const StreamParams& p = c.p;
  const dim3 grid((unsigned)((n_bins + 7) / 8 * 8 * p.ksplit * p.n_tb)), blk(NW * 64);
  if (c.x_f32 != nullptr) {
    // no quantizer launch: the contraction quantizes its few tokens itself
    if (xm != 1 || acc_out || p.T > QF_T || p.T * p.nks * 64 > QF_IN || c.in % 4 != 0 || p.n_tb != 1) return PIPE_EINVAL;
#define PIPE_STREAM_LAUNCH_Q(PARAMS, params, D) \
  PIPE_LAUNCH((gemm_stream_kernel<BITS, NW, 1, false, true, true, PARAMS, D>), grid, blk, st, a.ev_start, a.ev_stop, PIPE_STREAM_ARGS(c.x_f32, params))
    const bool two = BITS == 8 && two_tiles(p, true);
    constexpr int D2 = BITS == 8 ? 2 : 1;
    if (p.M == 1 && p.act == PIPE_ACT_NONE && p.res == nullptr && p.amax_out == nullptr && p.zero_after == nullptr && p.zero_big == nullptr) {
      const StreamPlain q{p.scales, p.bias, p.y, p.ws_sum, p.ws_cnt, p.out, p.s_static, p.act_qmax};
      if (two) PIPE_STREAM_LAUNCH_Q(StreamPlain, q, D2);
      else PIPE_STREAM_LAUNCH_Q(StreamPlain, q, 1);
    } else {
      if (two) PIPE_STREAM_LAUNCH_Q(StreamParams, p, D2);
      else PIPE_STREAM_LAUNCH_Q(StreamParams, p, 1);
    }
#undef PIPE_STREAM_LAUNCH_Q
    PIPE_HIP(hipGetLastError());
    return PIPE_OK;
  }
  const bool xmask = p.T % 16 != 0, two = BITS == 8 && xm == 1 && two_tiles(p, false);
#define PIPE_STREAM_LAUNCH_D(XMV, ACC, MASK, D) \
  PIPE_LAUNCH((gemm_stream_kernel<BITS, NW, XMV, ACC, MASK, false, StreamParams, D>), grid, blk, st, a.ev_start, a.ev_stop, PIPE_STREAM_ARGS(p.qx, p))
#define PIPE_STREAM_LAUNCH(XMV, ACC, MASK)                                                              \
  do {                                                                                                  \
    if (two) PIPE_STREAM_LAUNCH_D(XMV, ACC, MASK, (BITS == 8 && (XMV) == 1 ? 2 : 1));                   \
    else PIPE_STREAM_LAUNCH_D(XMV, ACC, MASK, 1);                                                       \
  } while (0)
#define PIPE_STREAM_PICK(XMV)                                                     \
  do {                                                                            \
    if (acc_out) { if (xmask) PIPE_STREAM_LAUNCH(XMV, true, true); else PIPE_STREAM_LAUNCH(XMV, true, false); }   \
    else { if (xmask) PIPE_STREAM_LAUNCH(XMV, false, true); else PIPE_STREAM_LAUNCH(XMV, false, false); }         \
  } while (0)
  if (xm == 1) PIPE_STREAM_PICK(1);
  else if (xm == 2) PIPE_STREAM_PICK(2);
  else PIPE_STREAM_PICK(4);
#undef PIPE_STREAM_PICK
#undef PIPE_STREAM_LAUNCH
#undef PIPE_STREAM_LAUNCH_D
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

}  // namespace

int launch_gemm_stream(const GemmArgs& a, hipStream_t st) {
  const pipe_expansion* e = a.e;
  if (a.T <= 0) return PIPE_OK;
  if (a.T > PIPE_STREAM_MAX_T || a.T_pad != (int)round_up64(a.T, 16) || e->K > e->bin_cap || e->bin_cap % R != 0) return PIPE_ESHAPE;
  if (e->bin_cap != R && a.acc_out != nullptr) return PIPE_EINVAL;   // the integer export of wide bins goes through the tiled kernel
  StreamCall c;
  StreamParams& p = c.p;
  p.qx = a.qx; p.qx_mstride = a.qx_mstride;
  p.rowsum = a.rowsum; p.rowsum_mstride = a.rowsum_mstride;
  p.s_x = a.s_x; p.sx_mstride = a.sx_mstride;
  p.codes = e->codes_dev; p.scales = e->scales_all_dev;
  p.bins = e->bins_dev;
  p.bias = a.bias; p.bias_mstride = a.bias_mstride; p.y = a.y; p.acc_out = a.acc_out; p.amax_out = a.amax_out; p.amax_neg = a.amax_neg; p.res = a.res; p.res_mstride = a.res_mstride; p.res_members = a.res_members; p.res_pre_act = a.res_pre_act; p.zero_after = a.zero_after; p.zero_n = a.zero_n; p.zero_big = a.zero_big; p.zero_big_n = a.zero_big_n;
  p.T = a.T; p.out = e->out; p.nks = e->nks; p.M = a.M; p.reduce = a.reduce; p.act = a.act;
  p.s_static = a.s_static; p.act_qmax = g_act_qmax_host;
  c.x_f32 = a.x_f32; c.in = e->in;
  if (a.x_f32 != nullptr && e->bin_cap != R) return PIPE_EINVAL;
  // Fewer bins than half the CUs and a long k: split each bin over several workgroups (each still
  // with at least two tiles per wave).  With more bins a split only adds the exchange through
  // the workspace (measured on the 4096 x 11008 4-bit layer: 160 bins, 21.7 us unsplit, 23.5 us
  // split in three).
  {
    const int n_tiles = e->in_pad / (512 / e->bits);
    int ks;
    if (g_stream_ksplit > 0) ks = std::min(std::min(g_stream_ksplit, PIPE_MAX_SPLIT), n_tiles);   // forced (tests, tuning)
    else ks = std::min(256 / (e->n_bins > 0 ? e->n_bins : 1), std::min(PIPE_MAX_SPLIT, n_tiles / 16));
    p.n_tb = a.T_pad / 16;
    p.n_bins = e->n_bins;
    c.thr0 = e->bin_thr[0]; c.thr1 = e->bin_thr[1]; c.thr2 = e->bin_thr[2];
    if (p.n_tb > 1) ks = 1;   // several token blocks already multiply the workgroups
    p.ksplit = std::max(ks, 1);
    p.ws_sum = e->split_sum_dev; p.ws_cnt = e->split_cnt_dev;
  }
  static_assert(PIPE_MAX_K % 4 == 0 && PIPE_MAX_K <= 255, "members as bytes");
  for (int i = 0; i < PIPE_MAX_K / 4; ++i) p.member_lo[i] = p.member_hi[i] = p.member_of[i] = 0u;
  for (int m = 0; m < a.M; ++m) {
    p.member_lo[m >> 2] |= (uint32_t)a.member_lo[m] << (m & 3) * 8;
    p.member_hi[m >> 2] |= (uint32_t)a.member_hi[m] << (m & 3) * 8;
    for (int k = a.member_lo[m]; k <= a.member_hi[m]; ++k) p.member_of[k >> 2] |= (uint32_t)m << (k & 3) * 8;
  }
  // distinct activation tensors: one, or one per member
  const int xm = (a.qx_mstride == 0 || a.M <= 1) ? 1 : (a.M <= 2 ? 2 : 4);
  const bool acc_out = a.acc_out != nullptr;
  if (e->bin_cap != R) {
    const int xmm = (a.qx_mstride == 0 || a.M <= 1) ? 1 : R;
    switch (e->bits) {
      case 8: return launch_multi_cap<8>(p, e->n_bins, e->bin_cap, xmm, a, st);
      case 4: return launch_multi_cap<4>(p, e->n_bins, e->bin_cap, xmm, a, st);
      default: return launch_multi_cap<2>(p, e->n_bins, e->bin_cap, xmm, a, st);
    }
  }
  switch (e->bits) {
    case 8: return launch_nw<8, 8>(c, e->n_bins, xm, acc_out, a, st);
    case 4: return launch_nw<4, 8>(c, e->n_bins, xm, acc_out, a, st);
    default: return launch_nw<2, 8>(c, e->n_bins, xm, acc_out, a, st);
  }
}
