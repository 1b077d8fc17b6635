// Single-pass tiled contraction kernel of the expanded layer (App. B, Eq. (define_dre)), for layers whose members hold
// at most 4 orders:
//   y[t,o] = sum_m ( s_x,m * sum_{k in member m} s_k[o] * acc_k[t,o]  (+ b[o] if m = 0) ),  acc_k exact, int32.
//
// All orders of a row block multiply the same Q(x), so a wave takes a bin of 4 stored row blocks ("items") that holds
// EVERY order of its 1 to 4 output row blocks, and a tile is 4 such bins (the 4 waves) against 16*MTB tokens.  One walk
// along k per tile, whatever the orders:
//   - tiles differ by a quarter at most, so nothing waits for the tile with the most orders: 4 items are multiplied where a bin
//     of the tile has 4, 3 where none has more (a third of the work of dense layers of 3 orders: 11008 x 2048 ternary, 4096 tokens 266 ->
//     235 us), and none at all where every bin holds row blocks that its member pruned, which only get their bias;
//   - the activations of a tile are fetched once, not once per order;
//   - no fp32 running sum lives through the loop: int32 accumulators only, the orders are folded behind it.
// Data paths of a stage (SK 64-k steps, one or two packed code tiles per item), requested DP stages before it is multiplied:
//   - packed codes: L2 -> registers, 16 bytes per lane, DP + 1 register sets, widened to int8 between the MFMAs of the item before;
//   - activations: L2 -> LDS without passing through registers, already in the MFMA operand layout, DP + 1 slots.
// Bound by the matrix pipe and the issue slots around it (a ternary stage of 64 tokens: 64 MFMAs against 112 unpack instructions, 16
// LDS reads and 8 loads per wave), and by what a workgroup does outside its loop (4.3 of 27.5 us of a 16-stage tile), which other
// workgroups have to cover: 144 to 153 vector registers and 35 KB of LDS let three share a compute unit, and four where the fragments
// have one register set (128 registers, the most that four can have; see launch_cfg for which).  A third stage in flight costs the registers and a fifth more loads
// (each tile then requests stages behind its last) and gains nothing (11008 x 4096 ternary, 4096 tokens 203 us against 198 with two
// and 191 with two and four workgroups); a workgroup that walks several tiles loses (220 us: 768 fixed walks fill the chip worse than
// the dispatcher does); tiles of 128 tokens, two workgroups, lose on ternary codes (214) and win a little on 4 bits (gate||up
// 22016 x 4096, 2048 tokens 364 against 372).
// Where the chip holds more waves than the tiles bring: a full chip (four workgroups a unit) spends 4176 cycles on the four's 4096 MFMA cycles of
// a ternary stage; a tile alone spends 1560 on the 512 of a 4-bit stage of a convolution, 390 of them on its own loads after the barrier, at the 16 cycles
// per KiB that the unit's address path takes, 230 on the first fragments.  So (G = 2)
// two groups of 4 waves share a tile, half of k each, and (DP = 2) the loads of a stage two ahead are asked for one by one between
// the multiplies: through buffer resources, so that those behind the last stage read nothing and every wait stays an exact count.
// (Exact in the code that the compiler makes of it, too: see the loop.  With waits that reached into the loads in flight the calls took 1 to 4 %
// longer: 4096 x 11008 4 bit, 200 tokens 42.0 -> 40.5 us, ternary, 400 tokens 66.6 -> 64.1, 4096 x 4096 8 bit, 500 tokens 30.2 -> 29.3.)
// A stage of two groups, 1024 MFMA cycles, then takes 1490 at 4 bits (768 x 3072, 2000 tokens) and 2150 with a convolution's gathers (256 x 14 x 14, 32 images);
// one group with two stages in flight 840 and 1230 for its 512, one with one in flight 1180 and 1560; at 8 bits 890 and 1410.
// Measured against one pass per order (pipe_gemm.hip, same box): 11008 x 4096 ternary, K = 4, 4096 tokens 227 -> 203 us,
// 333 tokens 62 -> 30 us; 3x3 convolution 256 x 256 of 6272 pixels, 4 bit, K = 3 35.5 -> 18.4 us; 3072 x 768 and back, 4 bit,
// K = 3, 4096 tokens 81 -> 60 us; eight 2048 x 2048 ternary layers, two members of 4 orders, 4096 tokens 676 -> 591 us
// (550 with the hidden maxima in eight lines).
// One barrier per stage.  The activations are loaded through a buffer resource: unlike global LDS-direct loads, which the compiler
// counts as flat ones and waits for one and all, their waits are counted, and its range check serves tokens and taps outside.
#include <algorithm>
#include <type_traits>

#include "pipe_tile.h"

namespace {

constexpr int FRAG = 64;   // uint4 per fragment

struct BinsParams {
  const uint8_t* qx;
  int64_t qx_mstride;
  const int32_t* rowsum;
  int64_t rowsum_mstride;
  const float* s_x;
  int sx_mstride;
  const uint8_t* codes;
  const float* scales;
  const TileBin* bins;            // [4 * n_ct]
  const float* bias;
  long long bias_mstride;
  float* y;
  uint32_t* amax_out;
  uint32_t* amax_neg;
  uint32_t* zero_after;
  int zero_n;
  uint32_t* zero_big;
  int zero_big_n;
  int T, T_pad, out, nks;
  int apart;                      // 1: one output per member, y[M,T,out]
  int fold_sx;                    // 1: the activation scale joins the row scales (a sum over several members)
  int act;
  const float* res;               // MODE_CHAIN: skip tensor
  long long res_mstride;
  int res_members, res_pre_act;
  int hidden;                     // MODE_GATED: rows are gate [0,H) and up [H,2H), y is [M,T,H]
  int later;                      // 1: MODE_SUM
  int dead_ct, dead_gap;          // column tiles from dead_ct on lie dead_gap further on
  int three;                      // 1: tiles of 3 items walk with 3
  TileOrder order;
  const int8_t* cq8;              // CONV (implicit GEMM), as in pipe_gemm.hip
  const int32_t* ccsum;
  unsigned cbytes;
  int one_tap;                    // 1: a stage's 64-k steps share a tap (its address is stepped once: 2 to 4 % with two groups)
  int cC, cH, cW, ckh, ckw, cstride, cpad, cHo, cWo;
};

enum { MODE_PLAIN = 0, MODE_GELU = 2, MODE_GATED = 3, MODE_CHAIN = 4, MODE_RELU = 5,
       MODE_SUM = 6 };   // a member of a sum behind the first: y is read, its orders are added, y is written

// Packed codes of one item for one stage of SK 64-k steps.
template <int BITS, int SK>
struct Codes {
  static constexpr int N = SK * BITS / 8;   // uint4
  static_assert(N >= 1, "a stage is whole code tiles");
  v4u v[N];
};

template <int BITS, int SK>
__device__ __forceinline__ v4i widen(const Codes<BITS, SK>& w, int j) {
  constexpr int N = Codes<BITS, SK>::N;
  if (BITS == 8) return (v4i)w.v[j & (N - 1)];
  const v4u q = w.v[BITS == 4 ? (j >> 1) & (N - 1) : 0];
  if (BITS == 4) return (j & 1) ? widen4(q.z, q.w) : widen4(q.x, q.y);
  return widen2(j == 0 ? q.x : (j == 1 ? q.y : (j == 2 ? q.z : q.w)));
}

// Global -> LDS, 16 bytes per lane from base + lane's offset + scalar offset to dst + 16 * lane, both moved by OFFS.
template <int OFFS>
__device__ __forceinline__ void bload16(__amdgpu_buffer_rsrc_t base, v4i* dst, unsigned lane_off, unsigned off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(base, (__attribute__((address_space(3))) void*)dst, 16, lane_off, off, OFFS, 0);
}
// s_waitcnt: at most vm vector-memory and lgkm LDS / scalar operations outstanding
constexpr int wait_imm(int vm, int lgkm) { return (vm & 15) | (7 << 4) | (lgkm << 8) | ((vm >> 4) << 14); }

// G groups of 4 waves take a tile's walk along k in G parts, each with slots of its own; their sums meet in LDS behind the loop and
// every group finishes MTB / G of the token blocks.
template <int BITS, int MTB, int MINW, int MODE, bool CONV, int G, int DP>
__global__ __launch_bounds__(256 * G, MINW) void gemm_bins_kernel(const TileBin* __restrict__ a_bins, const uint8_t* __restrict__ a_codes, int a_n_ct, int a_n_tt,
                                                                  int a_strip, int a_toks, int a_dead_ct, int a_dead_gap, int a_nks, const BinsParams p) {
  constexpr int OFF = BITS == 8 ? 0 : (BITS == 4 ? 8 : 1);
  constexpr int SK = BITS == 2 || MTB == 1 || (G == 2 && MTB == 2) ? 4 : 2;   // 64-k steps per stage
  constexpr int XC = MTB * SK / 4;                    // activation fragments (1 KiB) a wave loads per stage
  constexpr int WN = Codes<BITS, SK>::N;
  constexpr int XF = MTB == 4 && MINW == 4 ? 1 : 2;   // register sets of activation fragments
  static_assert(TOK_TILE % (16 * MTB) == 0 && MTB % G == 0, "token tile");
  constexpr int MB = MTB / G;                         // token blocks a group finishes
  constexpr int SLOT = G * MTB * SK * FRAG;
  struct Side {
    float scl[4 * G][64];                             // per wave: row scales of its items
    float bias[4 * G][64];                            // ... bias of their output rows
    int rs[4 * G][64];                                // ... code sums of the tokens it finishes
  };
  // One array per slot: the compiler tells their LDS-direct loads and reads apart by the array, and so waits before a read
  // for nothing but the slot's own loads.
  __shared__ alignas(1024) v4i xs0[SLOT], xs1[SLOT], xs2[DP > 1 ? SLOT : 1];
  __shared__ Side lds;
  static_assert((DP + 1) * SLOT * 16 <= 65536, "LDS-direct loads reach the first 64 KiB");

  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = wid & 3, grp = G == 1 ? 0 : wid >> 2;
  // The tile's descriptor first, from arguments that come in registers with the launch: the others are on their way from host memory
  // meanwhile.
  int ct, tt;
  const bool mine = TileOrder{a_n_ct, a_n_tt, a_strip, a_toks}.tile(blockIdx.x, &ct, &tt);
  const int t0 = tt * (16 * MTB);
  if (ct >= a_dead_ct) ct += a_dead_gap;
  const TileBin* bin = a_bins + (mine ? ct : 0) * 4 + wave;
  const v4i pos = cload(&bin->pos, 0), spos = cload(&bin->spos, 0), rb = cload(&bin->rb, 0), info = cload(&bin->info, 0);
  if (p.zero_big != nullptr)
    for (int i = blockIdx.x * (256 * G) + threadIdx.x; i < p.zero_big_n; i += gridDim.x * (256 * G)) p.zero_big[i] = 0u;
  if (blockIdx.x == 0 && p.zero_after != nullptr) slots_clear<256 * G>(p.zero_after, p.zero_n);
  if (!mine) return;
  const int m = info[0], ends = info[1], ups = info[2];   // member; items that end a row block (and, << 4, that have codes); items of an up block
  const bool active = info[3] & 1;
  const int tile_items = info[3] >> 1;                    // items that any bin of the tile multiplies: 4, 3 or none

  // ---- load cursor: the stage requested next
  const int n_all = a_nks / SK, n_max = (n_all + G - 1) / G;   // stages of the tile, of a group
  const int s0 = grp * n_max, n_stage = G == 1 ? n_all : max(0, min(n_max, n_all - s0));
  const int tg = t0 + grp * (16 * MB);                         // first token that this group finishes
  const int64_t rb_bytes = (int64_t)a_nks * 8 * BITS * 16;   // packed codes of a row block
  const int xb = wave * XC / SK, xj = wave * XC - xb * SK;   // this wave's fragments: token block, first 64-k step
  // activations come through a buffer resource of the tile's fragments (of the whole image, CONV): base in scalar registers, a
  // lane's offset that does not change and the stage's offset in a scalar register
  const __amdgpu_buffer_rsrc_t l_x = __builtin_amdgcn_make_buffer_rsrc(
      CONV ? (void*)p.cq8 : (void*)(p.qx + (int64_t)m * p.qx_mstride + (int64_t)(t0 / 16) * a_nks * 1024), 0,
      CONV ? p.cbytes : (unsigned)(min(MTB, (p.T_pad - t0) / 16) * a_nks * 1024), 0x00020000);
  unsigned l_xlane = (unsigned)(xb * a_nks + xj + s0 * SK) * 1024 + lane * 16;
  unsigned l_xoff = 0;
  const uint8_t* l_wb[4];
  __amdgpu_buffer_rsrc_t l_w[4];   // groups: a resource of each item's codes, up to the end of the group's part
  unsigned l_woff = s0 * (WN * 1024) + lane * 16;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint8_t* c = a_codes + pos[r] * rb_bytes;
    if constexpr (DP == 1) l_wb[r] = c;
    else l_w[r] = __builtin_amdgcn_make_buffer_rsrc((void*)c, 0, (unsigned)((s0 + n_stage) * WN * 1024), 0x00020000);
  }
  constexpr int NCB = CONV ? XC : 1;
  int c_off = 0, c_h0 = 0, c_w0 = 0;         // CONV: this lane's pixel: offset of the window's first tap, its row and column
  int c_r[NCB], c_q[NCB], c_c0[NCB];         // wave-uniform: tap and first channel of the 64-k step each fragment loads next
  // ... and this lane's offset in it, ready a stage before the load (one tap a stage: all alike).  Chosen and range-checked beside every load, with
  // branches between the multiplies: convolution of 128 x 28 x 28, 16 images, 4 bit 21.2 -> 23.1 us, of 512 x 7 x 7, 32 images, 8 bit 27.3 -> 29.5
  unsigned c_at[NCB];
  const bool one_tap = CONV && p.one_tap;
  if constexpr (CONV) {
    const int t = t0 + xb * 16 + (lane & 15);
    const int wo = t % p.cWo, ho = (t / p.cWo) % p.cHo, img = t / (p.cWo * p.cHo);
    const int h0 = ho * p.cstride - p.cpad;
    c_h0 = t < p.T ? h0 : -(1 << 20);        // a token beyond the batch: every tap outside
    c_w0 = wo * p.cstride - p.cpad;
    c_off = ((img * p.cH + h0) * p.cW + c_w0) * p.cC + (lane >> 4) * 16;   // used only for taps inside the image
#pragma unroll
    for (int f = 0; f < XC; ++f) {
      const int tap = ((s0 * SK + xj + f) * 64) / p.cC;
      c_c0[f] = (s0 * SK + xj + f) * 64 - tap * p.cC;
      c_r[f] = tap / p.ckw;
      c_q[f] = tap - c_r[f] * p.ckw;
    }
  }
  // out of the resource's range (zeros) where the tap lies outside the image
  auto tap_at = [&](int r, int q) __attribute__((always_inline)) {
    const bool inside = r < p.ckh && (unsigned)(c_h0 + r) < (unsigned)p.cH && (unsigned)(c_w0 + q) < (unsigned)p.cW;
    return inside ? (unsigned)(c_off + (r * p.cW + q) * p.cC) : 0xFFF00000u;
  };
  if constexpr (CONV) {
#pragma unroll
    for (int f = 0; f < XC; ++f) c_at[f] = tap_at(c_r[f], c_q[f]);
  }
  // requests a stage: the items' codes (the i-th 16 bytes per lane), this wave's share of the activations (fragment f)
  auto ask_codes = [&](auto& w, int i) __attribute__((always_inline)) {
    w[i / WN].v[i % WN] = (v4u)__builtin_amdgcn_raw_buffer_load_b128(l_w[i / WN], l_woff + (i % WN) * 1024, 0, 0);
  };
  auto ask_acts = [&](v4i* slot, auto frag) __attribute__((always_inline)) {
    constexpr int f = decltype(frag)::value;
    v4i* dst = slot + (grp * MTB * SK + wave * XC) * FRAG;
    if constexpr (CONV) {
      bload16<0>(l_x, dst + f * FRAG, c_at[f], c_c0[f]);
    } else {   // a wave's fragments lie next to each other, here and there
      bload16<f * 1024>(l_x, dst, l_xlane, l_xoff);
    }
  };
  auto ask_next = [&]() __attribute__((always_inline)) {   // moves on to the next stage
    if constexpr (DP > 1) l_woff += WN * 1024;
    if constexpr (!CONV) {
      if (DP == 1) l_xoff += SK * 1024; else l_xlane += SK * 1024;
    } else if (one_tap) {
#pragma unroll
      for (int f = 0; f < XC; ++f) c_c0[f] += SK * 64;
      if (c_c0[XC - 1] >= p.cC) {
        if (++c_q[0] == p.ckw) { c_q[0] = 0; ++c_r[0]; }
        const unsigned at = tap_at(c_r[0], c_q[0]);
#pragma unroll
        for (int f = 0; f < XC; ++f) { c_c0[f] -= p.cC; c_at[f] = at; }
      }
    } else {
#pragma unroll
      for (int f = 0; f < XC; ++f) {   // the 64-k steps run tap-major, channel-minor (C is a multiple of 64); the position is stepped, not divided out
        c_c0[f] += SK * 64;
        while (c_c0[f] >= p.cC) {
          c_c0[f] -= p.cC;
          if (++c_q[f] == p.ckw) { c_q[f] = 0; ++c_r[f]; }
        }
        c_at[f] = tap_at(c_r[f], c_q[f]);
      }
    }
  };
  auto ask_part = [&](auto& w, v4i* slot, int i) __attribute__((always_inline)) {   // the i-th load of a stage
    if (i >= XC) ask_codes(w, i - XC);
    else if (i == 0) ask_acts(slot, std::integral_constant<int, 0>{});
    else if (i == 1) ask_acts(slot, std::integral_constant<int, (XC > 1 ? 1 : 0)>{});
    else if (i == 2) ask_acts(slot, std::integral_constant<int, (XC > 2 ? 2 : 0)>{});
    else ask_acts(slot, std::integral_constant<int, (XC > 2 ? 3 : 0)>{});
  };
  auto request = [&](auto& w, v4i* slot) __attribute__((always_inline)) {
    constexpr int NI = (int)std::extent<std::remove_reference_t<decltype(w)>>::value;
    if constexpr (DP == 1) {
      unsigned off = lane * 16;
      asm volatile("" : "+v"(off));   // a 32-bit offset next to the loads: they take the scalar base + offset form
#pragma unroll
      for (int r = 0; r < NI; ++r) {
#pragma unroll
        for (int q = 0; q < WN; ++q) w[r].v[q] = gload16(l_wb[r] + q * 1024 + off);
        l_wb[r] += WN * 1024;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < XC; ++i) ask_part(w, slot, i);
    } else {
#pragma unroll
      for (int i = 0; i < XC + NI * WN; ++i) ask_part(w, slot, i);
    }
    ask_next();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto wait_for = [&](auto left) __attribute__((always_inline)) {   // until all but the last `left` loads have arrived
    __builtin_amdgcn_s_waitcnt(wait_imm(decltype(left)::value, 0));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // ---- what the epilogue needs travels beside the first stage, into LDS of this wave
  float e_scl, e_bias = 0.f;
  int e_rs = 0;
  {
    const int r = lane >> 4;
    int sp = 0, br = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // selects on scalar registers (an indexed array would live in scratch memory)
      sp |= r == q ? spos[q] : 0;
      br |= r == q ? max(rb[q], 0) * 16 + ((ups >> q) & 1 ? p.hidden : 0) : 0;
    }
    e_scl = p.scales[(size_t)sp * 16 + (lane & 15)];
    if (p.bias != nullptr) e_bias = p.bias[(size_t)m * p.bias_mstride + br + (lane & 15)];
    if (OFF && !CONV) e_rs = p.rowsum[(size_t)m * p.rowsum_mstride + min(tg + lane, p.T_pad - 1)];
  }
  const float sx = p.s_x[m * p.sx_mstride];
  auto window_sums = [&]() __attribute__((always_inline)) {
    if constexpr (OFF != 0 && CONV) {
      // token code sum = the channel sums of the window's pixels that lie inside the image
      {
        const int t = tg + min(lane, 16 * MB - 1);
        const int wo = t % p.cWo, ho = (t / p.cWo) % p.cHo, img = t / (p.cWo * p.cHo);
        const int h0 = ho * p.cstride - p.cpad, w0_ = wo * p.cstride - p.cpad;
        // nine taps' loads in flight (one after the other they took 2.2 of the 14.5 us of a 3 x 3 layer's workgroup); a tap outside
        // reads the first sum and drops it
        int sum = 0, r = 0, q = 0;
        while (r < p.ckh) {
          int c[9];
          bool in[9];
#pragma unroll
          for (int i = 0; i < 9; ++i) {
            in[i] = t < p.T && r < p.ckh && (unsigned)(h0 + r) < (unsigned)p.cH && (unsigned)(w0_ + q) < (unsigned)p.cW;
            c[i] = r < p.ckh ? p.ccsum[in[i] ? (img * p.cH + h0 + r) * p.cW + w0_ + q : 0] : 0;
            if (++q == p.ckw) { q = 0; ++r; }
          }
#pragma unroll
          for (int i = 0; i < 9; ++i) sum += in[i] ? c[i] : 0;
        }
        e_rs = sum;
      }
    }
  };

  auto side = [&]() __attribute__((always_inline)) {
    lds.scl[wid][lane] = e_scl;
    lds.bias[wid][lane] = e_bias;
    if (OFF) lds.rs[wid][lane] = e_rs;
  };

  v4i acc[4][MTB];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int b = 0; b < MTB; ++b) acc[r][b] = v4i{0, 0, 0, 0};

  // ---- the walk along k with the first NI items of every bin of the tile
  auto walk = [&](auto ni) __attribute__((always_inline)) {
    constexpr int NI = decltype(ni)::value;
    asm volatile("; %0 items" ::"i"(NI));   // keeps the walks apart: what they request first would be requested before the branch between them
    constexpr int AHEAD = (DP - 1) * (NI * WN + XC);   // loads in flight behind those of the next stage
    Codes<BITS, SK> w0[NI], w1[NI], w2[DP > 1 ? NI : 1];
    request(w0, xs0);
    if constexpr (DP > 1) request(w1, xs1);
    window_sums();
    side();
    wait_for(std::integral_constant<int, AHEAD>{});
    // One stage: its codes and activations have arrived (every wave waits for its own at the end of the stage before)
    // and `far` and `free_slot`, multiplied in the stage before, take the stage that is requested now.
    auto stage = [&](Codes<BITS, SK>(&now)[NI], const v4i* slot, Codes<BITS, SK>(&far)[NI], v4i* free_slot, bool multiply, bool ask) __attribute__((always_inline)) {
      asm volatile("s_barrier" ::: "memory");    // everyone's have arrived, and the slot of the stage before is free
      if (DP == 1 && ask) request(far, free_slot);
      __builtin_amdgcn_sched_barrier(0);
      if (multiply) {
        // Software pipeline of the SK 64-k steps: a wave issues in order, so everything that is not an MFMA has to sit in
        // the shadow of one.  The fragments of step j+1 are requested before step j's MFMAs start (two register
        // sets), and the codes of item r+1 are widened between the MFMAs of item r (two register sets).
        const v4i* xs = slot + grp * (MTB * SK * FRAG) + lane;
        v4i xf[XF][MTB];
        v4i wf[2];
#pragma unroll
        for (int b = 0; b < MTB; ++b) xf[0][b] = xs[b * SK * FRAG];
        wf[0] = widen<BITS, SK>(now[0], 0);
#pragma unroll
        for (int j = 0; j < SK; ++j) {
          if (XF == 2 && j + 1 < SK) {
#pragma unroll
            for (int b = 0; b < MTB; ++b) xf[(j + 1) % XF][b] = xs[(b * SK + j + 1) * FRAG];
          }
#pragma unroll
          for (int r = 0; r < NI; ++r) {
            const int n = j * NI + r;   // item-steps so far: the register set of this one's codes
            if (DP > 1 && ask) {        // its share of the loads that are requested now
              constexpr int TOT = NI * WN + XC, STEPS = SK * NI;
#pragma unroll
              for (int i = n * TOT / STEPS; i < (n + 1) * TOT / STEPS; ++i) ask_part(far, free_slot, i);
              if (n == STEPS - 1) ask_next();
              __builtin_amdgcn_sched_barrier(0);
            }
            if (r + 1 < NI) wf[(n + 1) & 1] = widen<BITS, SK>(now[r + 1], j);
            else if (j + 1 < SK) wf[(n + 1) & 1] = widen<BITS, SK>(now[0], j + 1);
#pragma unroll
            for (int b = 0; b < MTB; ++b)
              acc[r][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[n & 1], xf[j % XF][b], acc[r][b], 0, 0, 0);
            if (BITS != 8) {
              // one MFMA, then some of the unpack instructions, and so on
#pragma unroll
              for (int b = 0; b < MTB; ++b) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 8 / MTB, 0);
              }
            }
            __builtin_amdgcn_sched_barrier(0);   // keep the items apart: bounds live registers
          }
          if (XF == 1 && j + 1 < SK) {
#pragma unroll
            for (int b = 0; b < MTB; ++b) xf[0][b] = xs[(b * SK + j + 1) * FRAG];
          }
        }
      }
      if (DP == 1 || ask) wait_for(std::integral_constant<int, AHEAD>{});
      else wait_for(std::integral_constant<int, 0>{});
    };
    // Two (three) stages a round, so that the slots and register sets keep their roles.  One stage in flight: behind an odd number of stages
    // the second half multiplies nothing.
    if constexpr (DP == 1) {
      for (int s = 0; s < n_stage; s += 2) {
        stage(w0, xs0, w1, xs1, active, s + 1 < n_stage);
        stage(w1, xs1, w0, xs0, active && s + 1 < n_stage, s + 2 < n_stage);
      }
    } else {
      // Two in flight: every stage multiplies, also of a wave without items (codes of the all-zero position) and of a group behind its
      // part (codes out of range, zeros), and the loop has one exit.  With a path that requests a stage and multiplies nothing, or one out of the middle,
      // the compiler takes the registers that loads are writing to for others and makes a stage wait for all of them first (cycles: see above).
      int s = 0;
      for (; s + 3 <= n_max; s += 3) {
        stage(w0, xs0, w2, xs2, true, true);
        stage(w1, xs1, w0, xs0, true, true);
        stage(w2, xs2, w1, xs1, true, true);
      }
      if (s < n_max) stage(w0, xs0, w2, xs2, true, false);
      if (s + 1 < n_max) stage(w1, xs1, w0, xs0, true, false);
      wait_for(std::integral_constant<int, 0>{});   // the slots are written to the end
    }
  };
  // (64 tokens of the ternary convolution: a second loop would spill; chain layers: see launch_gemm_bins)
  constexpr bool THREE = !(CONV && SK * MTB == 16) && MODE != MODE_CHAIN && MODE != MODE_RELU;
  if (tile_items == 0) { window_sums(); side(); }
  else if (THREE && tile_items == 3 && p.three) walk(std::integral_constant<int, THREE ? 3 : 4>{});
  else walk(std::integral_constant<int, 4>{});

  // ---- the groups' sums meet: in step i a group hands the token blocks of the i-th group behind it over
  v4i own[4][MB];
  if constexpr (G == 1) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int b = 0; b < MB; ++b) own[r][b] = acc[r][b];
  } else {
    // one token block after the other, through 16 KiB of each of two slots
    static_assert(G == 2 && SLOT >= 16 * FRAG, "exchange");
    v4i* mine = (grp == 0 ? xs0 : xs1) + wave * (4 * FRAG) + lane;
    const v4i* other = (grp == 0 ? xs1 : xs0) + wave * (4 * FRAG) + lane;
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      __syncthreads();   // the slots have been read
#pragma unroll
      for (int r = 0; r < 4; ++r) mine[r * FRAG] = grp == 0 ? acc[r][MB + b] : acc[r][b];
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) own[r][b] = (grp == 0 ? acc[r][b] : acc[r][MB + b]) + other[r * FRAG];
    }
  }

  // ---- epilogue: orders folded in ascending k, one output row block after the other.  A lane holds 4 channels of one
  // token per 16-token block, 64 contiguous bytes of a token per 16 lanes.
  int lane_e = lane;
  asm volatile("" : "+v"(lane_e));   // keeps the epilogue's addresses out of the loop's live range
  const int tl = lane_e & 15, g = lane_e >> 4;
  int rs[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) rs[b] = OFF ? lds.rs[wid][b * 16 + tl] : 0;
  // the slots as they are now, read while the orders are folded
  const bool two_sided = p.amax_neg != nullptr;
  float mx = 0.f, mn = 0.f;
  const uint32_t seen = p.amax_out != nullptr ? slot_seen(&p.amax_out[m]) : 0u;
  const uint32_t seen_neg = two_sided ? slot_seen(&p.amax_neg[m]) : 0u;
  const bool with_bias = p.bias != nullptr && (m == 0 || !p.apart || p.bias_mstride != 0);
  float* ym = p.y + (size_t)(p.apart ? m : 0) * p.T * p.out + 4 * g;
  const int n_res = (MODE == MODE_CHAIN && p.res != nullptr) ? (p.apart ? (m < p.res_members ? 1 : 0) : p.res_members) : 0;
  const float* resm = MODE == MODE_CHAIN ? p.res + (size_t)(p.apart ? m : 0) * p.res_mstride + 4 * g : nullptr;
  // the skip tensor of a row block, requested a row block ahead (two sets of registers: with all four a workgroup less fits), or
  // with it where four workgroups cover it
  constexpr int RQ = MINW == 4 ? 1 : 2;
  constexpr bool READS = MODE == MODE_CHAIN || MODE == MODE_SUM;
  float4 rq[READS ? RQ : 1][READS ? MB : 1];
  auto skip = [&](int r) __attribute__((always_inline)) {
    if constexpr (MODE == MODE_CHAIN) {
      if (n_res > 0 && ((ends >> r) & 1)) {
#pragma unroll
        for (int b = 0; b < MB; ++b)
          rq[r & (RQ - 1)][b] = *reinterpret_cast<const float4*>(resm + (size_t)min(tg + b * 16 + tl, p.T - 1) * p.out + rb[r] * 16);
      }
    }
    if constexpr (MODE == MODE_SUM) {   // what the members before have left, with the row block's first item
      if (rb[r] >= 0 && (r == 0 || ((ends >> (r - 1)) & 1))) {
#pragma unroll
        for (int b = 0; b < MB; ++b)
          rq[r & (RQ - 1)][b] = *reinterpret_cast<const float4*>(ym + (size_t)min(tg + b * 16 + tl, p.T - 1) * p.out + rb[r] * 16);
      }
    }
  };
  if (RQ == 2) skip(0);
  float v[MB][4], gate[MODE == MODE_GATED ? MB : 1][4];
#pragma unroll
  for (int b = 0; b < MB; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) v[b][i] = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (RQ == 1) skip(r);
    else if (r < 3) skip(r + 1);
    if constexpr (MODE == MODE_SUM) {
      if (rb[r] >= 0 && (r == 0 || ((ends >> (r - 1)) & 1))) {
#pragma unroll
        for (int b = 0; b < MB; ++b) {
          const float4 y0 = rq[r & (RQ - 1)][b];
          v[b][0] = y0.x; v[b][1] = y0.y; v[b][2] = y0.z; v[b][3] = y0.w;
        }
      }
    }
    // (a row block that a later member of a sum pruned keeps what is there, also where the member's scale is infinite)
    if (MODE != MODE_SUM || ((ends >> (4 + r)) & 1)) {
      const v4f sc = *reinterpret_cast<const v4f*>(&lds.scl[wid][r * 16 + g * 4]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float s = p.fold_sx ? sc[i] * sx : sc[i];
#pragma unroll
        for (int b = 0; b < MB; ++b) v[b][i] = fmaf(s, (float)(own[r][b][i] - OFF * rs[b]), v[b][i]);
      }
    }
    if (!((ends >> r) & 1)) continue;
    v4f bb = v4f{0.f, 0.f, 0.f, 0.f};
    if (with_bias) bb = *reinterpret_cast<const v4f*>(&lds.bias[wid][r * 16 + g * 4]);
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) v[b][i] = p.fold_sx ? v[b][i] + bb[i] : fmaf(sx, v[b][i], bb[i]);   // same rounding as the other contraction kernels
    if (MODE == MODE_GATED && !((ups >> r) & 1)) {
#pragma unroll
      for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) { gate[b][i] = v[b][i]; v[b][i] = 0.f; }
      continue;
    }
#pragma unroll
    for (int b = 0; b < MB; ++b) {
      const int t = tg + b * 16 + tl;
      if (MODE == MODE_CHAIN) {
        float4 rs4 = n_res > 0 ? rq[r & (RQ - 1)][b] : make_float4(0.f, 0.f, 0.f, 0.f);
        for (int mm = 1; mm < n_res; ++mm) {   // a sum over several members, each with a skip tensor of its own
          const float4 x = *reinterpret_cast<const float4*>(resm + (size_t)mm * p.res_mstride + (size_t)min(t, p.T - 1) * p.out + rb[r] * 16);
          rs4.x += x.x; rs4.y += x.y; rs4.z += x.z; rs4.w += x.w;
        }
        const float rr[4] = {rs4.x, rs4.y, rs4.z, rs4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (p.res_pre_act) v[b][i] += rr[i];
          if (p.act == PIPE_ACT_RELU) v[b][i] = fmaxf(v[b][i], 0.f);
          else if (p.act == PIPE_ACT_GELU) v[b][i] = gelu_erf(v[b][i]);
          if (!p.res_pre_act) v[b][i] += rr[i];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (MODE == MODE_RELU) v[b][i] = fmaxf(v[b][i], 0.f);
        if (MODE == MODE_GELU) v[b][i] = gelu_erf(v[b][i]);
        if (MODE == MODE_GATED) v[b][i] = gate[b][i] / (1.f + expf(-gate[b][i])) * v[b][i];
      }
      if (t < p.T) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          mx = fmaxf(mx, two_sided ? v[b][i] : fabsf(v[b][i]));
          if (two_sided) mn = fmaxf(mn, -v[b][i]);
        }
        *reinterpret_cast<float4*>(ym + (size_t)t * p.out + rb[r] * 16) = make_float4(v[b][0], v[b][1], v[b][2], v[b][3]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) v[b][i] = 0.f;
    }
  }
  if (p.amax_out != nullptr) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) slot_raise(&p.amax_out[m], seen, mx);
    if (two_sided) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) mn = fmaxf(mn, __shfl_xor(mn, o, 64));
      if (lane == 0) slot_raise(&p.amax_neg[m], seen_neg, mn);
    }
  }
}

#define PIPE_BINS_ARGS p.bins, p.codes, p.order.n_ct, p.order.n_tt, p.order.strip, p.order.toks, p.dead_ct, p.dead_gap, p.nks, p

template <int BITS, int MTB, int MINW, int G = 1, int DP = G>
int launch_cfg(BinsParams& p, int live_ct, int n_ct, hipEvent_t ev0, hipEvent_t ev1, hipStream_t st) {
  const int n_tt = ceil_div(p.T, 16 * MTB);
  p.order = tile_order(n_ct, n_tt, false);
  const dim3 grid((unsigned)p.order.blocks());
  const int act = p.cq8 != nullptr ? 0 : p.act;
  if (p.cq8 != nullptr && (p.res != nullptr || p.act != 0)) return PIPE_EINVAL;   // implicit-GEMM convolution: plain epilogue
  // Workgroups per compute unit, three or four: four cover each other's epilogues and first loads better (a round of four takes
  // 1.30 of one of three, not 1.33), but end in larger rounds.  So four where as many or fewer places are filled: 11008 x 4096 ternary, 4096
  // tokens (4864 tiles) 197 -> 191 us, 700 tokens 46.2 -> 44.4, 3300 165 -> 162; gate||up 22016 x 4096 4 bit, 2048 tokens 398 -> 372;
  // but 3072 x 768 4 bit with GELU, 4096 tokens (1536 tiles, two full rounds of three) 30 -> 32.  Chain layers
  // without a skip tensor have a mode of their own, the others request theirs a row block at a time: eight 2048 x 2048 ternary layers, two members
  // of 4 orders, 4096 tokens 682 -> 658 us, six 4-bit ones of two members of 2 orders, 2500 tokens 444 -> 423.  Convolutions hold too much for four (they would spill).
  const bool chain = p.res != nullptr || act == PIPE_ACT_RELU;
  if constexpr (MTB == 4 && MINW == 3 && DP == 1) {
    const int64_t tiles = (int64_t)live_ct * n_tt, cus = pipe_resident_workgroups();
    const bool four = (tiles + 4 * cus - 1) / (4 * cus) * 4 <= (tiles + 3 * cus - 1) / (3 * cus) * 3;
    if (four && p.cq8 == nullptr) return launch_cfg<BITS, MTB, 4>(p, live_ct, n_ct, ev0, ev1, st);
  }
  if constexpr (MTB == 4 && MINW == 4 && DP == 1) {
    if (p.cq8 != nullptr) return PIPE_EINVAL;
    if (chain && p.res == nullptr) {
      PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_RELU, false, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
      PIPE_HIP(hipGetLastError());
      return PIPE_OK;
    }
    if (chain) {
      PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_CHAIN, false, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
      PIPE_HIP(hipGetLastError());
      return PIPE_OK;
    }
  } else {
    if (p.cq8 != nullptr) {
      PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_PLAIN, true, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
      PIPE_HIP(hipGetLastError());
      return PIPE_OK;
    }
    if (chain) {
      PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_CHAIN, false, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
      PIPE_HIP(hipGetLastError());
      return PIPE_OK;
    }
  }
  if (p.later) {
    PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_SUM, false, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
  } else if (act == PIPE_ACT_GELU) {
    PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_GELU, false, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
  } else if (act == PIPE_ACT_SILU_GATED) {
    PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_GATED, false, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
  } else {
    PIPE_LAUNCH((gemm_bins_kernel<BITS, MTB, MINW, MODE_PLAIN, false, G, DP>), grid, dim3(256 * G), st, ev0, ev1, PIPE_BINS_ARGS);
  }
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

// The tiles' height, groups and loads ahead, by how many there are
int launch_tiles(BinsParams& p, int bits, int live, int n_ct, hipEvent_t ev0, hipEvent_t ev1, hipStream_t st) {
  // Token-tile height: 64 tokens amortize the unpacking of the codes best (the 4096-token layer above: 203, 245 and 317 us
  // with 64, 32 and 16), and a second tile on a compute unit costs less than twice one; so the tallest that still gives
  // three quarters of the 256 compute units a tile (256 tokens of that layer, 304 tiles of 64: 29.4, 27.2 and 29.1 us; 129
  // tokens: 22 us each).  Around the line of 192 tiles the choice is within 7 % of the best height for the 3 x 3 convolution 256 x 256 4 bit,
  // K = 3 (147 tiles of 64: 17.8 against 17.5 us; 196: 18.1 and 18.0) and for layers of 3072 x 768, 1024 x 1024 and 4096 x 4096 at 2, 4
  // and 8 bits; far below it 16 tokens lose to 32 by up to a quarter at 8 bits (128 x 128 convolution of 4704 pixels, K = 2: 14.0 and 11.0 us).
  int mtb = g_tiled_mtb, groups = 1, ahead = 1;
  const int64_t cus = pipe_resident_workgroups();
  auto tiles = [&](int tokens) { return (int64_t)n_ct * ceil_div(p.T, tokens); };
  // tiles of this height that the fullest of the 8 XCDs is dealt; whether each has a compute unit for itself
  auto fullest = [&](int tokens) {
    const TileOrder o = tile_order(n_ct, ceil_div(p.T, tokens), false);
    const int64_t chunks = (o.n_tt + o.toks - 1) / o.toks, rest = n_ct % o.strip;   // of a strip; column tiles of the last one
    return ((n_ct / o.strip * chunks + 7) / 8 * o.strip + (rest > 0 ? (chunks + 7) / 8 * rest : 0)) * o.toks;
  };
  auto alone = [&](int tokens) { return fullest(tokens) * 8 <= cus; };
  if (mtb != 1 && mtb != 2 && mtb != 4) {
    mtb = tiles(64) >= 192 ? 4 : (tiles(32) >= 192 ? 2 : 1);
    // What a tile that is alone on its compute unit spends beside its multiplies nothing else covers, so there its loads are asked for two stages ahead
    // and between the multiplies, and the lowest height is taken that still leaves every tile alone: on the fullest XCD as well (768 x 3072
    // 8 bit, K = 2, 2600 tokens, 246 tiles of which one XCD's 32 units get 36: 42.5 us against 39.8 one stage ahead).  Calls, us, as here and
    // with two groups of 32 or 64 tokens or as above:
    //   16 tokens: 768 x 3072 4 bit, K = 3, 150 tokens 16.0 / 18.3, ternary, 250 tokens 15.9 / 17.9, 8 bit, K = 2, 600 tokens 22.1 / 23.6; convolution of
    //   256 x 14 x 14, 5 images, 4 bit 17.6 / 19.3, 8 bit 18.5 / 22.4; of ternary ones a stage's few loads are better in one go (17.5; so 18.1);
    //   8 bits, 32 or 64 tokens (two groups hold a compute unit each and share its path to the L1, which 8-bit codes fill): 4096 x 4096, 200 tokens
    //   24.1 / 27.4, 500 tokens 28.7 / 30.7; 768 x 3072, 1000 tokens 24.4 / 26.8; convolution of 512 x 7 x 7, 32 images 27.3 / 32.4.
    // 8 bits, at most two low tiles a unit where the last high one would be half empty: 11008 x 4096, 160 tokens 33.2 / 35.0 (three: 190 tokens 46.5 / 36.0;
    // none saved: 3072 x 768, K = 2, half kept, 700 tokens 21.1 / 19.8).
    // Two groups of waves along k, 2 and 4 bits, where the walk is long enough (24 64-k steps) for the second prologue and the exchange: 4096 x 11008 4 bit,
    // K = 4, 140 tokens 32.5 / 37.2 with one group, 300 tokens 44.1 / 45.2; 4096 x 4096, 130 tokens 19.3 / 20.3; convolution of
    // 256 x 14 x 14, 32 images 25.0 / 26.2; 3x3 of 512 x 7 x 7, 20 images, ternary 24.2 / 26.7; long ternary walks also with two
    // low tiles a unit where the high ones would not be alone: 4096 x 11008, 350 tokens 59.8 / 63.0 (300 tokens, alone 47.3 / 44.6).  Shorter 4-bit walks, 32 tokens, one group, ahead: 3072 x 768,
    // 300 tokens, affine codes 14.4 / 15.0, 2048 x 1024, 250 tokens 13.0 / 13.8; ternary ones and convolutions gain nothing.
    // Tiles of 64 tokens that the chip holds two of a unit also ask two stages ahead: 11008 x 4096 ternary, 333
    // tokens (456 tiles) 33.7 / 37.4, 4096 x 11008 4 bit, 420 tokens 63.3 / 69.7, gate||up 11008 x 2048, 216 tokens (480 tiles) a whole MLP 65.8 / 70.6;
    // at 4 bits not where an XCD's units are dealt all of the two (1536 x 2048, 1700 tokens 34.1 / 32.2; 4096 x 4096, 700 tokens 46.0 / 44.2), nor
    // ternary convolutions of shorter walks (128 rows of 64 x 56 x 56, 8 images 25.9 / 24.3; 72 steps, 512 x 7 x 7, 40 images 30.7 / 32.5), nor 8 bits (4096 x 4096, 600 tokens 38.8 / 36.5).
    // Chain layers of 16 to 23 steps gain by it only while a unit holds one tile: what follows the walk there (skip tensor, ReLU, maxima) is covered by
    // the four workgroups of the loads one stage ahead (two 1024 x 1024 layers and a head, 4 bit, K = 4, 1700 tokens, 432 tiles 133.9 / 114.1,
    // 1100 tokens, 288 tiles 107.6 / 101.6; half the groups kept, 1112 tokens, 216 tiles 108.6 / 106.6; 1280 wide, 240 tiles 98.2 / 107.0).
    const bool conv = p.cq8 != nullptr, chain = p.res != nullptr || p.act == PIPE_ACT_RELU;
    if (p.nks >= (bits == 8 ? 8 : 16) && alone(16)) { mtb = 1; ahead = bits == 2 && conv ? 1 : 2; }
    else if (bits == 8) {
      if (p.nks >= 8 && (alone(32) || alone(64))) { mtb = alone(32) ? 2 : 4; ahead = 2; }
      else if (p.nks >= 8 && tiles(32) < 2 * tiles(64) && fullest(32) * 8 <= 2 * cus) mtb = 2;
    }
    else if (p.nks >= 24 && (alone(32) || (bits == 2 && !conv && p.nks >= 64 && tiles(32) <= 2 * cus && !alone(64)))) { mtb = 2; groups = 2; }
    else if (p.nks >= 24 && bits == 4 && alone(64)) { mtb = 4; groups = 2; }
    else if (p.nks >= 12 && p.nks < 24 && bits == 4 && !conv && alone(32)) { mtb = 2; ahead = 2; }
    else if ((p.nks >= 24 || (p.nks >= 16 && tiles(64) >= 192 && !(chain && tiles(64) > cus))) && !(bits == 2 && conv && p.nks < 64) &&
             (bits == 2 ? tiles(64) <= 2 * cus : fullest(64) * 64 <= 15 * cus)) { mtb = 4; ahead = 2; }
  }
  const int sk = bits == 2 || mtb == 1 || (groups == 2 && mtb == 2) ? 4 : 2;   // as in the kernel
  p.one_tap = p.cq8 != nullptr && p.cC % (sk * 64) == 0;
  if (groups == 2) {
    switch (bits * 8 + mtb) {
      case 4 * 8 + 4: return launch_cfg<4, 4, 2, 2>(p, live, n_ct, ev0, ev1, st);
      case 4 * 8 + 2: return launch_cfg<4, 2, 2, 2>(p, live, n_ct, ev0, ev1, st);
      case 2 * 8 + 2: return launch_cfg<2, 2, 2, 2>(p, live, n_ct, ev0, ev1, st);
      default: return PIPE_EINVAL;
    }
  }
  if (ahead == 2) {
    switch (bits * 8 + mtb) {
      case 8 * 8 + 4: return launch_cfg<8, 4, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      case 8 * 8 + 2: return launch_cfg<8, 2, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      case 8 * 8 + 1: return launch_cfg<8, 1, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      case 4 * 8 + 4: return launch_cfg<4, 4, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      case 4 * 8 + 2: return launch_cfg<4, 2, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      case 4 * 8 + 1: return launch_cfg<4, 1, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      case 2 * 8 + 4: return launch_cfg<2, 4, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      case 2 * 8 + 1: return launch_cfg<2, 1, 2, 1, 2>(p, live, n_ct, ev0, ev1, st);
      default: return PIPE_EINVAL;
    }
  }
  switch (bits * 8 + mtb) {
    case 8 * 8 + 4: return launch_cfg<8, 4, 2>(p, live, n_ct, ev0, ev1, st);
    case 8 * 8 + 2: return launch_cfg<8, 2, 2>(p, live, n_ct, ev0, ev1, st);
    case 8 * 8 + 1: return launch_cfg<8, 1, 2>(p, live, n_ct, ev0, ev1, st);
    case 4 * 8 + 4: return launch_cfg<4, 4, 3>(p, live, n_ct, ev0, ev1, st);
    case 4 * 8 + 2: return launch_cfg<4, 2, 4>(p, live, n_ct, ev0, ev1, st);
    case 4 * 8 + 1: return launch_cfg<4, 1, 3>(p, live, n_ct, ev0, ev1, st);
    case 2 * 8 + 4: return launch_cfg<2, 4, 3>(p, live, n_ct, ev0, ev1, st);
    case 2 * 8 + 2: return launch_cfg<2, 2, 4>(p, live, n_ct, ev0, ev1, st);
    case 2 * 8 + 1: return launch_cfg<2, 1, 4>(p, live, n_ct, ev0, ev1, st);
    default: return PIPE_EINVAL;
  }
}

}  // namespace

// Members whose outputs stay apart each have their own bins; members that share one input and are summed are one set of
// orders.  A sum over members with inputs of their own (but see pipe_sum_apply), a member with more orders than a bin holds, a gate||up pair that
// may need more than a bin (3 orders and more), and the integer export run pass by pass (pipe_gemm.hip).
bool pipe_bins_apply(const GemmArgs& a) {
  if (a.acc_out != nullptr) return false;
  const bool joined = a.M == 1 || a.reduce;
  if (joined) {
    if (a.M > 1 && (a.qx_mstride != 0 || a.sx_mstride != 0)) return false;
    if (a.act == PIPE_ACT_SILU_GATED) return a.M == 1 && a.e->K <= 2;
    return a.e->K <= 4;
  }
  for (int m = 0; m < a.M; ++m)
    if (a.member_hi[m] - a.member_lo[m] + 1 > (a.act == PIPE_ACT_SILU_GATED ? 2 : 4)) return false;
  return true;
}

int launch_gemm_bins(const GemmArgs& a, hipStream_t st) {
  const pipe_expansion* e = a.e;
  if (a.T <= 0) return PIPE_OK;
  if (a.T_pad % TOK_TILE != 0 || a.T_pad < a.T) return PIPE_ESHAPE;
  if (a.conv_q8 != nullptr && (a.conv_C % 64 != 0 || (a.M > 1 && a.qx_mstride != 0))) return PIPE_ESHAPE;
  if (a.res != nullptr && (a.act == PIPE_ACT_SILU_GATED || a.res_members < 1 || a.res_members > a.M)) return PIPE_EINVAL;
  if (a.act == PIPE_ACT_SILU_GATED && a.reduce) return PIPE_EINVAL;
  int rc = PIPE_OK;
  const TileBins* tb = pipe_get_bins(e, a, &rc);
  if (tb == nullptr) return rc;
  BinsParams p;
  p.qx = a.qx; p.qx_mstride = a.qx_mstride; p.rowsum = a.rowsum; p.rowsum_mstride = a.rowsum_mstride;
  p.s_x = a.s_x; p.sx_mstride = a.sx_mstride;
  p.codes = e->codes_dev; p.scales = e->scales_all_dev; p.bins = tb->bins_dev;
  p.bias = a.bias; p.bias_mstride = a.bias_mstride; p.y = a.y; p.amax_out = a.amax_out; p.amax_neg = a.amax_neg;
  p.zero_after = a.zero_after; p.zero_n = a.zero_n; p.zero_big = a.zero_big; p.zero_big_n = a.zero_big_n;
  // The shorter walk of tiles with 3 items pays wherever they are the rule, and for plain and gate||up layers also next to tiles of
  // 4 (4096 x 4096 4 bit, K = 4, half the groups kept, 4096 tokens: 174.7 -> 161 us a call; gate||up 22016 x 4096, 2048 tokens, the
  // MLP 665 -> 641).  GELU layers lose by the mixture (768 x 3072 and back, K = 3, half the groups kept, 4096 tokens 81.5 -> 82.6;
  // all kept 104.8 -> 97.4).  The chains' layers walk with 4: with 3 for tiles of 3 they gain or lose by how the rounds fall (eight 2048 x 2048
  // ternary layers, two members of 4 orders, 1000, 2000, 3000 and 4096 tokens 302 -> 284, 412 -> 435, 532 -> 535 and 654 -> 653 us; one member of 4
  // orders, 4000 tokens 403 -> 424, 4 bit, 1500 tokens 273 -> 249).
  p.three = a.act != PIPE_ACT_GELU || tb->n_four * 8 <= tb->n_three;
  p.later = 0; p.dead_ct = tb->n_ct; p.dead_gap = 0;
  p.T = a.T; p.T_pad = a.T_pad; p.out = e->out; p.nks = e->nks;
  p.apart = !a.reduce; p.fold_sx = a.reduce && a.M > 1; p.act = a.act;
  p.res = a.res; p.res_mstride = a.res_mstride; p.res_members = a.res_members; p.res_pre_act = a.res_pre_act;
  p.hidden = 0;
  if (a.act == PIPE_ACT_SILU_GATED) { p.hidden = e->out / 2; p.out = e->out / 2; }
  p.cq8 = a.conv_q8; p.ccsum = a.conv_csum; p.cbytes = a.conv_q8 != nullptr ? (unsigned)((int64_t)a.T / (a.conv_Ho * a.conv_Wo) * a.conv_C * a.conv_H * a.conv_W) : 0u;
  p.cC = a.conv_C; p.cH = a.conv_H; p.cW = a.conv_W; p.ckh = a.conv_kh; p.ckw = a.conv_kw; p.cstride = a.conv_stride; p.cpad = a.conv_pad;
  p.cHo = a.conv_Ho; p.cWo = a.conv_Wo;
  return launch_tiles(p, e->bits, tb->n_four + tb->n_three, tb->n_ct, a.ev_start, a.ev_stop, st);
}

// The sum over two members with inputs of their own (the second layer of an MLP, the last of a chain), one launch of the single-pass kernel
// per member: the first leaves its part in y, the second starts from it, so every output is summed as pass by pass, in
// ascending order, to the same bits.  y is written, read and written again (it fits the last level cache), which long walks are worth:
// see pipe_sum_apply.
int launch_gemm_sum(const GemmArgs& a, hipStream_t st) {
  GemmArgs apart = a;
  apart.reduce = 0;
  int rc = PIPE_OK;
  const TileBins* tb = pipe_get_bins(a.e, apart, &rc);
  if (tb == nullptr) return rc;
  const pipe_expansion* e = a.e;
  BinsParams p{};
  p.qx = a.qx; p.qx_mstride = a.qx_mstride; p.rowsum = a.rowsum; p.rowsum_mstride = a.rowsum_mstride;
  p.s_x = a.s_x; p.sx_mstride = a.sx_mstride;
  p.codes = e->codes_dev; p.scales = e->scales_all_dev; p.y = a.y;
  p.T = a.T; p.T_pad = a.T_pad; p.out = e->out; p.nks = e->nks;
  p.fold_sx = 1; p.three = 1;
  int n_dead = 0, dead0 = 0, live0 = 0;
  for (int m = 0; m < a.M; ++m) n_dead += tb->dead_ct[m];
  for (int m = 0; m < a.M; dead0 += tb->dead_ct[m], live0 += tb->live_ct[m], ++m) {
    const bool last = m == a.M - 1;
    p.later = m > 0;
    if (last) {
      p.bias = a.bias;
      p.zero_after = a.zero_after; p.zero_n = a.zero_n; p.zero_big = a.zero_big; p.zero_big_n = a.zero_big_n;
    }
    // column tiles of row blocks that this member pruned: only for the first value of y, and for the bias
    const int dead = m == 0 || (last && (a.bias != nullptr || tb->live_ct[m] == 0)) ? tb->dead_ct[m] : 0;
    p.bins = tb->bins_dev + 4 * (size_t)(dead > 0 ? dead0 : n_dead + live0);
    p.dead_ct = dead;
    p.dead_gap = dead > 0 ? n_dead + live0 - dead0 - dead : 0;
    const int n_ct = dead + tb->live_ct[m];
    if (n_ct == 0) continue;
    // timed as one: the first launch records the begin, the last the end
    const hipEvent_t ev0 = m == 0 ? a.ev_start : nullptr, ev1 = last ? a.ev_stop : nullptr;
    rc = launch_tiles(p, e->bits, tb->live_ct[m], n_ct, ev0, ev1, st);
    if (rc != PIPE_OK) return rc;
  }
  return PIPE_OK;
}

// Against the pass-by-pass kernel, which multiplies a member's orders one walk after the other in tiles that run the most passes of their row
// blocks (whole MLP calls, us): 4096-11008-4096 gated 4 bit, members of 2 orders, 300 tokens 218 -> 166, 500 268 -> 203, 1000 374 -> 338, 2048 630 -> 621;
// ternary, 1500 tokens 419 -> 358; 768-3072-768 GELU, 2500 tokens 113 -> 94, 4096 140 -> 128.  A member of a single order has a launch's
// fixed parts for half the work: from 192 tiles of 64 tokens on it gains (K = 3 in 2 and 1, 1500 tokens, 192 tiles 538 -> 444), with 128 and 44 it
// loses (1024-4096-1024, 4096 tokens 156.6 -> 159.5; 2048-5504-2048 gated, 652 tokens 103.5 -> 106.2).  Walks of 8 to 32 64-k steps (the last layer
// of a chain) are within 0.5 % either way and stay one launch; more than two members would read and write y once more each.
bool pipe_sum_apply(const GemmArgs& a) {
  if (a.acc_out != nullptr || a.M != 2 || !a.reduce || (a.qx_mstride == 0 && a.sx_mstride == 0) || a.e->nks < 48) return false;
  if (a.act != PIPE_ACT_NONE || a.res != nullptr || a.amax_out != nullptr || a.conv_q8 != nullptr || a.bias_mstride != 0) return false;
  if (a.T <= 0 || a.T_pad % TOK_TILE != 0 || a.T_pad < a.T) return false;   // (launch_gemm_tiled reports it)
  for (int m = 0; m < a.M; ++m) {
    const int orders = a.member_hi[m] - a.member_lo[m] + 1;
    if (orders > 4) return false;
    if (orders == 1 && (int64_t)ceil_div(a.e->orders[a.member_lo[m]].n_kept * a.e->rbpg, 16) * ceil_div(a.T, 64) < 192) return false;
  }
  return true;
}
