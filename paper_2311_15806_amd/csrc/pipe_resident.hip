// Resident kernel for decode-sized batches (T <= 16): ONE launch walks a whole chain of expanded
// layers (App. B "Ensemble of more Layers", Sec. 3.2: a member is the whole network; App. B,
// Eq. (define_dre) per layer), so the packed codes of layer l+1 stream from HBM while layer l's
// results are still being exchanged, and no launch boundary separates the layers.
//
// One workgroup per compute unit, 12 waves:
//   waves 0-7  ("workers") stream packed codes and multiply.  A wave owns the 1-KiB code tiles
//              w, w+8, ... of every item (stored row block) of its workgroup's units and keeps RD
//              rounds of 4 tiles in flight in registers, across unit and LAYER boundaries: the
//              codes do not depend on the activations, so the first rounds of the next layer are
//              requested before the grid-wide exchange that makes its input codes available.
//              Exact int32 partial tiles are added up in LDS; token code sums (for the offset-binary
//              codes) are added up by v_dot4 beside the first sub-unit.
//   waves 8-11 ("epilogue") turn the integer tiles into fp32 outputs with the arithmetic and order of
//              the per-layer kernels (bit-identical results), and run the exchange between layers:
//              every workgroup quantizes the outputs it produced itself (network input: a slice of x).
// Exchange between layers, two grid-wide steps, no read-modify-write atomics and no cache-wide
// fences (a release or acquire fence at device scope costs 10-30 us on this chip, measured):
//   A  max|.|: each workgroup publishes {epoch, max} as one 64-bit device-scope store per tensor and
//      reads everybody's, so all derive the same scale max/q_max (skipped for a given static scale);
//   B  codes:  each workgroup writes its own outputs' codes with device-scope (write-through) stores,
//      waits for their completion, publishes its epoch in its flag word and polls the others' flags.
//   Everything one workgroup writes for another goes through device-scope stores; the consumers'
//   bulk reads of the codes are ordinary loads from a buffer that no cache can hold stale (each
//   layer has its own, first read in this launch after the flags were seen).
// What bounds a layer (8 ternary layers of 4096 <-> 11008, 16 tokens; 132.5 us a call before, 104 now): 3.5 us from the last workgroup's outputs
// to the codes of the next layer, 2 us for the first fragments of them, then rounds of about 0.7 us: 64 KiB of codes and fragments through
// a compute unit's 64 bytes a cycle, and the instructions of a wave in order; 1.2 us of epilogue.  Hence the layers' arguments in LDS (they lie in
// host memory: every new line of them cost a wave microseconds), scalar pointers that step through the tiles, waits that leave the
// rounds behind in flight, scales and bias fetched by the waves that do not poll, and codes written a row block per wave.
// Every wait is bounded: after `spin_limit` polls a workgroup records the failure in a status word,
// stops waiting for the rest of the launch and runs to its end, so the grid always drains.
#include "pipe_internal.h"

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <type_traits>

int g_decode_resident = 1;
int g_resident_spin_limit = 1 << 19;
unsigned long long* g_resident_trace = nullptr;

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int RES_WORKERS = 8;
constexpr int RES_EPI = 4;
constexpr int RES_THREADS = (RES_WORKERS + RES_EPI) * 64;
// Dynamic LDS of the epilogue waves (a compute unit holds one workgroup)
constexpr int RES_STASH = 48;            // 1-KiB slots of fp32 outputs a workgroup keeps in LDS between a layer and the next exchange
constexpr int RES_SIDE = 32;             // units whose row scales and bias are fetched into LDS before the layer begins
constexpr int RES_COLS = 768;            // output row blocks of a workgroup and layer
constexpr int RES_PAD_LDS = (RES_STASH + RES_SIDE + 2 + 8) * 1024 + RES_COLS * 4;
static_assert(PIPE_RES_DESC_INTS / 48 * 8 <= RES_COLS, "a unit has at most 8 output row blocks and at least 48 descriptor words");

// A unit's epilogue descriptor: numbers of items (stored row blocks) and outputs (output row blocks), then per item its position, per output
// its row block, per item its output's row block, and four items a word (order | output << 4).  The items lie output by output, in
// ascending order.
enum { UE_ITEMS = 0, UE_OUTS = 1, UE_POS = 2, UE_ORB = 10, UE_IRB = 18, UE_KO = 26, UE_N = 32 };
constexpr int UE_NO_ORDER = 15;   // of an item that is not there

struct ResLayer {
  const uint8_t* codes;     // stored row blocks of the layer, schedule order
  const float* scales;      // 16 row scales per position
  const int32_t* subs;      // [n_units * nsub] ResSub
  const int32_t* epi;       // [n_units * UE_N]
  const float* bias;        // or nullptr
  float* out;               // hidden layer: [M, T, out_w]; last layer: [T, out_w] (members summed)
  const float* res;         // skip tensor or nullptr
  long long res_mstride;
  uint8_t* qin;             // codes entering the layer: [xm][nks][1 KiB] (fragment layout, one 16-token block)
  int n_units, nsub, n_tiles, nks;
  int out_w;                // width of a row of `out` (gated layer: hidden width)
  int in, in_pad;
  int xm;                   // distinct activation tensors entering the layer: 1 (first layer) or M
  int act, res_members, res_pre_act, gated, reduce, res_device;
  float s_in[2];            // > 0: given scales of the tensors entering the layer (no exchange of maxima then)
};

struct ResParams {
  ResLayer layer[PIPE_RES_MAX_LAYERS];
  int L, T, M, G;
  int member_lo[PIPE_RES_MAX_M], member_hi[PIPE_RES_MAX_M];
  int member_of[4];
  const float* x;           // network input [T, in0]
  float s_static;           // > 0: given scale of the network input
  float act_qmax;
  int n_rep;                // copies of flags and amax_tag
  uint32_t* flags;          // [n_rep][G] epoch each workgroup reached
  unsigned long long* amax_tag;   // [n_rep][G][2] {epoch, bit pattern of the local max}
  uint32_t* gen;            // epoch the previous launch on this scratch ended with
  uint32_t* status;         // != 0: a wait ran into the spin limit
  int spin_limit;
  unsigned long long* trace;   // profiling: [G][L][8] timestamps (100 MHz) of the phases of every layer, or nullptr
};

// A layer's words in LDS: the arguments, then this workgroup's number of units and where their descriptors begin.  (The arguments lie in
// host memory by default: a wave that reaches a layer's first word would wait microseconds for it, and then for the next one.)
constexpr int RES_ARGS = sizeof(ResLayer) / 4, RES_NU = RES_ARGS, RES_AT = RES_ARGS + 1, RES_WORDS = RES_ARGS + 2;
static_assert(sizeof(ResLayer) % 4 == 0 && RES_WORDS <= 64, "a lane holds a word");

// a pointer that went through integers, known to be global again (else: flat accesses, which count as LDS operations too)
template <class T>
__device__ __forceinline__ T* global_ptr(T* q) {
  typedef __attribute__((address_space(1))) T* gptr;
  return (T*)(gptr)(unsigned long long)q;
}

static_assert(sizeof(ResParams) <= 3584, "kernel arguments are limited to 4 KiB");

template <int BITS>
__device__ __forceinline__ void unpack_step_r(const v4i& wi, int j, v4i& o) {
  const uint4 w = make_uint4((uint32_t)wi[0], (uint32_t)wi[1], (uint32_t)wi[2], (uint32_t)wi[3]);
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

// wave-uniform loads of the schedule tables (written once by the host): scalar loads
template <class T>
__device__ __forceinline__ T cload_r(const void* base, size_t idx) {
  typedef const __attribute__((address_space(4))) T* cptr;
  return ((cptr)(unsigned long long)base)[idx];
}

__device__ __forceinline__ void st_dev_u32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_dev_u32(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// XM: activation tensors a unit's items can read (1, or one per member: 2).  RD: rounds of four code
// tiles a worker wave keeps in flight.
template <int BITS, int XM, int RD>
__global__ __launch_bounds__(RES_THREADS, 1) void chain_resident_kernel(const ResParams p) {
  constexpr int OFF = BITS == 8 ? 0 : (BITS == 4 ? 8 : 1);
  constexpr int KSUP = 512 / BITS;
  constexpr int STEPS = KSUP / 64;
  __shared__ int tile[2][PIPE_RES_MAX_ITEMS + 2][256];
  __shared__ float s_wmax[RES_EPI][2];
  __shared__ float s_scale[2];   // scales of the codes entering the current layer
  __shared__ int s_fail;
  __shared__ unsigned long long s_ts[PIPE_RES_MAX_LAYERS][8];
  __shared__ uint32_t s_seen;   // the last epoch one of the polling waves has seen every workgroup reach
  // this workgroup's unit descriptors of all layers, copied once (a cold scalar load per unit on the
  // workers' path costs more than the unit's arithmetic): per layer, per local unit, its sub-units
  // (16 ints each) and then its epilogue descriptor (32 ints)
  __shared__ alignas(16) int s_desc[PIPE_RES_DESC_INTS];
  __shared__ int s_par[PIPE_RES_MAX_LAYERS * RES_WORDS];
  extern __shared__ int pad_lds[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = blockIdx.x, G = p.G;
  for (int i = threadIdx.x; i < 2 * (PIPE_RES_MAX_ITEMS + 2) * 256; i += RES_THREADS) (&tile[0][0][0])[i] = 0;
  if (threadIdx.x == 0) { s_fail = 0; s_scale[0] = 0.f; s_scale[1] = 0.f; }
  if (threadIdx.x < PIPE_RES_MAX_LAYERS * 8) (&s_ts[0][0])[threadIdx.x] = 0ull;
  for (int i = threadIdx.x; i < p.L * RES_ARGS; i += RES_THREADS)
    s_par[i / RES_ARGS * RES_WORDS + i % RES_ARGS] = reinterpret_cast<const int*>(p.layer)[i];
  __syncthreads();
  // units of every layer and where their descriptors begin: lane l, layer l
  int n_desc = 0, my_at = 0;
  {
    const int* w = &s_par[min(lane, p.L - 1) * RES_WORDS];
    const int n = w[offsetof(ResLayer, n_units) / 4], words = w[offsetof(ResLayer, nsub) / 4] * 16 + UE_N;
    const int nu = lane < p.L && n > wg ? (n - wg + G - 1) / G : 0;
    int sum = nu * words;
#pragma unroll
    for (int o = 1; o < PIPE_RES_MAX_LAYERS; o <<= 1) {
      const int v = __shfl_up(sum, o, 64);
      if (lane >= o) sum += v;
    }
    n_desc = __builtin_amdgcn_readlane(sum, PIPE_RES_MAX_LAYERS - 1);   // the host has checked that all layers fit
    my_at = sum - nu * words;
    if (wave == 0 && lane < p.L) {
      s_par[lane * RES_WORDS + RES_NU] = nu;
      s_par[lane * RES_WORDS + RES_AT] = my_at;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n_desc; i += RES_THREADS) {   // all layers' words travel together
    int l = 0;
    for (int j = 1; j < p.L; ++j) l += i >= __builtin_amdgcn_readlane(my_at, j);
    const int* w = &s_par[l * RES_WORDS];
    const int sub = w[offsetof(ResLayer, nsub) / 4] * 16, k = i - w[RES_AT], u = k / (sub + UE_N), at = k - u * (sub + UE_N);
    const size_t unit = (size_t)(wg + u * G);
    const int part = at < sub ? (int)offsetof(ResLayer, subs) / 4 : (int)offsetof(ResLayer, epi) / 4;
    const int32_t* src = global_ptr(reinterpret_cast<const int32_t*>((unsigned long long)(unsigned)w[part] | (unsigned long long)(unsigned)w[part + 1] << 32));
    s_desc[i] = at < sub ? src[unit * sub + at] : src[unit * UE_N + (at - sub)];
  }
  __syncthreads();
  // layer l, in scalar registers
  struct Words { int w[RES_ARGS]; };
  struct Layer : ResLayer { int nu, at, stride; };
  auto layer_of = [&](int l) __attribute__((always_inline)) {
    const int v = s_par[l * RES_WORDS + min(lane, RES_WORDS - 1)];
    Words w;
#pragma unroll
    for (int i = 0; i < RES_ARGS; ++i) w.w[i] = __builtin_amdgcn_readlane(v, i);
    Layer y;
    static_cast<ResLayer&>(y) = __builtin_bit_cast(ResLayer, w);
    y.codes = global_ptr(y.codes); y.scales = global_ptr(y.scales); y.bias = global_ptr(y.bias); y.out = global_ptr(y.out);
    y.res = global_ptr(y.res); y.qin = global_ptr(y.qin);
    y.nu = __builtin_amdgcn_readlane(v, RES_NU); y.at = __builtin_amdgcn_readlane(v, RES_AT); y.stride = y.nsub * 16 + UE_N;
    return y;
  };
  auto dword_at = [&](const int* d, int i) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(d[i]); };
  // profiling: slot 0 exchange begins, 1 maxima known, 2 codes stored, 3 all flags seen, 4 last unit's epilogue done
  // (first epilogue wave); 7 worker wave 0 has multiplied its last round and passed the unit's barrier
  // (kept in LDS and written out when the kernel ends: a store in the middle would be waited for by the next load)
  auto stamp = [&](int l, int slot) __attribute__((always_inline)) {
    if (p.trace != nullptr && lane == 0) s_ts[l][slot] = wall_clock64();
  };

  if (wave < RES_WORKERS) {
    // ============================================================== workers
    // The loads of a step are unconditional and their number fixed (a step without real work loads
    // a valid address and drops the result), so the waits for them are exact counts: RD - 1 rounds of
    // codes (across layer boundaries) and a round of fragments stay in flight while a round is multiplied.
    constexpr int NXL = XM * STEPS;        // fragment loads of a round
    constexpr int XR = 2;                  // rounds of fragments in flight (four: 2 to 4 % slower, more loads that no one uses at the ends)
    const bool xlive = (lane & 15) < p.T;
    // (lanes of tokens beyond the batch: out of the resource's range, zeros)
    const unsigned xl = xlive ? lane * 16 : 0x80000000u;
    v4i acc[4];
    int csum[XM];   // this lane's share of its token's code sum
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int m = 0; m < XM; ++m) csum[m] = 0;
    // a ring of RD rounds of codes (round q of a layer lives in slot q % RD; every layer's rounds are
    // padded to a multiple of RD, so the mapping is static) and two rounds of activation fragments
    v4i wreg[RD][4], xreg[XR][NXL];
#pragma unroll
    for (int s = 0; s < RD; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r) wreg[s][r] = v4i{0, 0, 0, 0};

    // rounds of this wave in layer l: units x sub-units x tiles; a wave beyond the layer's tiles
    // still walks one empty round per sub-unit (it takes part in the unit's barrier)
    auto ru_of = [&](int nt) { return nt > wave ? (nt - wave + RES_WORKERS - 1) / RES_WORKERS : 0; };

    // ---- issue cursor: the next round whose codes have not been requested (runs ahead, across layers).  A wave issues its
    // instructions one after the other, so what a round costs beside its loads and multiplies is kept to a few scalar additions: four
    // scalar pointers that step through a sub-unit's tiles, set from the descriptor when one ends.
    int il = 0, iq = 0, iu = 0, ig = 0;               // layer, round in layer, local unit, sub-unit
    int ileft = 0;                                    // rounds left in the sub-unit
    const uint8_t* ip[4];
    const uint8_t* i_codes = nullptr;                 // the cursor's layer
    int i_ntiles = 1, i_ru = 0, i_nsub = 1, i_nu = 0, i_at = 0, i_stride = 48;
    auto issue_desc = [&]() __attribute__((always_inline)) {
      const v4i d = *reinterpret_cast<const v4i*>(&s_desc[i_at + iu * i_stride + ig * 16]);
      // items a sub-unit does not have repeat its first one (a cache hit; the product is dropped)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        ip[r] = i_codes + ((size_t)(unsigned)__builtin_amdgcn_readfirstlane(d[r]) * i_ntiles + (i_ru > 0 ? wave : 0)) * 1024;
      ileft = max(i_ru, 1);
    };
    auto issue_seek = [&]() __attribute__((always_inline)) {   // skip layers without rounds, fetch the descriptor
      Layer y = layer_of(min(il, p.L - 1));
      while (il < p.L && y.nu == 0) { ++il; y = layer_of(min(il, p.L - 1)); }
      i_codes = y.codes; i_ntiles = y.n_tiles; i_ru = ru_of(y.n_tiles); i_nsub = y.nsub; i_nu = y.nu; i_at = y.at; i_stride = y.stride;
      if (il < p.L) {
        issue_desc();
      } else {   // nothing left: the last rounds' loads take any valid address
#pragma unroll
        for (int r = 0; r < 4; ++r) ip[r] = i_codes;
      }
    };
    issue_seek();
    // Four code loads: the cursor's round, which moves on if `real`; else nobody uses the data.
    auto issue_codes = [&](v4i (&w)[4], bool real) __attribute__((always_inline)) {
      unsigned off = lane * 16;
      asm volatile("" : "+v"(off));   // a 32-bit offset next to the loads: they take the scalar base + offset form
#pragma unroll
      for (int r = 0; r < 4; ++r) w[r] = *reinterpret_cast<const v4i*>(ip[r] + off);
      __builtin_amdgcn_sched_barrier(0);
      if (real) {
        ++iq;
#pragma unroll
        for (int r = 0; r < 4; ++r) ip[r] += RES_WORKERS * 1024;
        if (--ileft == 0) {
          if (++ig >= i_nsub) { ig = 0; ++iu; }
          if (iu >= i_nu) { ++il; iq = 0; iu = 0; issue_seek(); }
          else issue_desc();
        }
      }
    };

    int buf = 0;
    const int mof = p.member_of[0] | p.member_of[1] << 1 | p.member_of[2] << 2 | p.member_of[3] << 3;
    for (int l = 0; l < p.L; ++l) {
      const Layer ly = layer_of(l);
      // rounds of this wave in the layer: units x sub-units x tiles; a wave beyond the layer's tiles
      // still walks one empty round per sub-unit (it takes part in the unit's barrier)
      const int ru = ru_of(ly.n_tiles), ru_eff = max(ru, 1);
      const int rounds = ly.nu * ly.nsub * ru_eff;
      const int rounds_pad = (rounds + RD - 1) / RD * RD;
      // codes of the first rounds, unless the previous layer's last steps requested them already
      if (il == l && iq == 0) {
#pragma unroll
        for (int s = 0; s < RD; ++s)
          if (il == l && iq == s) issue_codes(wreg[s], true);
      }
      // the codes entering this layer are being produced: four workgroup barriers of the exchange
      __syncthreads();
      __syncthreads();
      __syncthreads();
      __syncthreads();
      const int l_nks = ly.nks, l_xm = ly.xm, l_nsub = ly.nsub, l_stride = ly.stride;
      const __amdgpu_buffer_rsrc_t l_x = __builtin_amdgcn_make_buffer_rsrc(ly.qin, 0, (unsigned)(l_xm * l_nks * 1024), 0x00020000);
      constexpr int XSTEP = STEPS * 1024;
      const int x_0 = ru > 0 ? wave * XSTEP : 0, x_m1 = l_xm > 1 ? l_nks * 1024 : 0;
      int x_at = x_0, xleft = ru_eff;   // fragments of the next round that have not been requested, rounds of the sub-unit from there on
      auto issue_x = [&](v4i (&x)[NXL], bool real) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < XM; ++m)
#pragma unroll
          for (int j = 0; j < STEPS; ++j)
            x[m * STEPS + j] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(l_x, xl + j * 1024, x_at + (m > 0 ? x_m1 : 0), 0);
        __builtin_amdgcn_sched_barrier(0);   // rounds in the order they are used
        if (real) {
          x_at += RES_WORKERS * XSTEP;
          if (--xleft == 0) { x_at = x_0; xleft = ru_eff; }
        }
      };
      // ---- consume cursor
      int cat = ly.at, cg = 0, cleft = ru_eff, cn = 0, cslot0 = 0, clast = 0, csel = 0;   // csel: bit r: item r reads the second tensor
      auto cons_desc = [&]() __attribute__((always_inline)) {
        const v4i e = *reinterpret_cast<const v4i*>(&s_desc[cat + cg * 16 + 8]);
        cn = __builtin_amdgcn_readfirstlane(e[0]); cslot0 = __builtin_amdgcn_readfirstlane(e[1]); clast = __builtin_amdgcn_readfirstlane(e[2]);
        if (XM == 2 && l_xm == 2) {
          const v4i k = *reinterpret_cast<const v4i*>(&s_desc[cat + cg * 16 + 4]);
          csel = 0;
#pragma unroll
          for (int r = 0; r < 4; ++r) csel |= ((mof >> (__builtin_amdgcn_readfirstlane(k[r]) & 3)) & 1) << r;
        }
      };
      if (rounds > 0) cons_desc();

      auto step = [&](auto slot, int q) __attribute__((always_inline)) {
          constexpr int s = decltype(slot)::value;
          // 1. multiply round q
          if (q < rounds) {
            if (ru > 0) {
              v4i (&w)[4] = wreg[s];
#pragma unroll
              for (int j = 0; j < STEPS; ++j) {
                v4i x[XM];
#pragma unroll
                for (int m = 0; m < XM; ++m) x[m] = xreg[s % XR][m * STEPS + j];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  v4i xf = x[0];
                  if (XM == 2) {
                    const bool pick1 = (csel >> r) & 1;
#pragma unroll
                    for (int i = 0; i < 4; ++i) xf[i] = pick1 ? x[XM - 1][i] : xf[i];
                  }
                  v4i wf;
                  unpack_step_r<BITS>(w[r], j, wf);
                  acc[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf, xf, acc[r], 0, 0, 0);
                }
                if (OFF != 0 && cg == 0) {
                  // token code sums (a multiply with a row block of ones would take 7 more registers)
#pragma unroll
                  for (int m = 0; m < XM; ++m)
#pragma unroll
                    for (int i = 0; i < 4; ++i) csum[m] = __builtin_amdgcn_sdot4(x[m][i], 0x01010101, csum[m], false);
                }
              }
            }
          }
          // A round that is not multiplied takes its data all the same: registers that no one reads on some path are reused there while
          // their loads are in flight, and every round then waits for all loads.
#pragma unroll
          for (int r = 0; r < 4; ++r) asm volatile("" ::"v"(wreg[s][r]));
#pragma unroll
          for (int i = 0; i < NXL; ++i) asm volatile("" ::"v"(xreg[s % XR][i]));
          // 2. fragments of round q + XR into the set just read; codes of round q + RD into the slot just read
          //    (once this layer's are all requested: round s of the next layer).  Always NXL + 4 loads.
          issue_x(xreg[s % XR], q + XR < rounds);
          issue_codes(wreg[s], il < p.L && (il == l ? iq == q + RD : iq == s));
          // 3. end of a sub-unit: this wave's share of its integer tiles joins the others' in LDS
          if (q < rounds) {
            if (--cleft == 0) {
              if (ru > 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  if (r < cn) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) atomicAdd(&tile[buf][cslot0 + r][c * 64 + lane], acc[r][c]);
                  }
                  acc[r] = v4i{0, 0, 0, 0};
                }
              }
              if (clast) {
                if (OFF != 0 && ru > 0) {
#pragma unroll
                  for (int m = 0; m < XM; ++m) {
                    atomicAdd(&tile[buf][PIPE_RES_MAX_ITEMS + m][lane & 15], csum[m]);
                    csum[m] = 0;
                  }
                }
                __syncthreads();   // the unit's tiles are complete: the epilogue waves take them
                buf ^= 1;
              }
              cleft = ru_eff;
              if (++cg >= l_nsub) { cg = 0; cat += l_stride; }
              if (q + 1 < rounds) cons_desc();
              else if (wave == 0) stamp(l, 7);
            }
          }
      };
      // The first two rounds stand before the loop, so that where it begins the same loads are in flight on both ways there: the waits in it
      // are then exact (else every fourth round waited for all that had been requested).
      if (rounds_pad > 0) {
        typedef std::integral_constant<int, 0> S0;
        typedef std::integral_constant<int, 1> S1;
        typedef std::integral_constant<int, RD == 4 ? 2 : 0> S2;
        typedef std::integral_constant<int, RD == 4 ? 3 : 1> S3;
        static_assert(XR == 2 && (RD == 2 || RD == 4), "rounds before the loop");
        issue_x(xreg[0], 0 < rounds);
        issue_x(xreg[1], 1 < rounds);
        step(S0{}, 0);
        step(S1{}, 1);
        if constexpr (RD == 4) {
          for (int q = 2;; q += 4) {
            step(S2{}, q);
            step(S3{}, q + 1);
            if (q + 2 >= rounds_pad) break;
            step(S0{}, q + 2);
            step(S1{}, q + 3);
          }
        } else {
          for (int q = 2; q < rounds_pad; q += 2) {
            step(S0{}, q);
            step(S1{}, q + 1);
          }
        }
      }
    }
  } else {
    // ============================================================== epilogue waves
    const int e = threadIdx.x - RES_WORKERS * 64;   // 0..255
    const int ewave = e >> 6;
    const int t = e >> 4, ch = e & 15;
    const int fidx = (ch & 3) * 64 + (ch >> 2) * 16 + t;   // (c * 64 + lane of the workers: their additions meet no bank twice)
    const bool tok = t < p.T;
    // Every epilogue wave tracks the epoch; the first one polls and tells the others through LDS and
    // the workgroup barrier that follows.
    uint32_t epoch = ld_dev_u32(p.gen);
    const uint32_t epoch0 = epoch;
    if (e == 0) s_seen = epoch;
    int buf = 0;
    const float qmax = p.act_qmax;
    // what this thread produced in the current layer: its max|.| per member, and the values themselves
    // (LDS, as far as it reaches; the rest is read back from the layer's output)
    float* stash = reinterpret_cast<float*>(pad_lds);
    float* side = stash + RES_STASH * 256;        // per unit: row scales [8][16], bias of its output row blocks [8][16]
    float* sums = side + (RES_SIDE + 2) * 256;          // a unit's finished sums, this thread's only
    int* s_col = pad_lds + (RES_STASH + RES_SIDE + 2 + 8) * 256;   // output row blocks of the layer before, in the order of their stash slots
    float mx_out[2] = {0.f, 0.f};
    int nout_prev = 0, n_apart_prev = 1;   // ... how many, and tensors each
    auto seen = [&]() __attribute__((always_inline)) {
      return (int)(__hip_atomic_load(&s_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - epoch) >= 0 || s_fail != 0;
    };

    // The flags and tags are kept n_rep times, and workgroup w polls copy w % n_rep (that of its XCD): 256 polling workgroups
    // crowd one copy's memory channels.  A poll's loads travel together.  Eight ternary layers of 4096 <-> 11008, 16 tokens:
    // 153 us with one copy and a load after the other, 147 with the loads together, 138, 134 and 132 with 2, 4 and 8 copies.
    const int n_rep = p.n_rep, rep = wg % n_rep;
    // one grid-wide step: publish this workgroup's epoch, wait until every workgroup has reached it
    auto grid_wait = [&]() __attribute__((always_inline)) {
      if (ewave != 0) return;   // one polling wave per workgroup: more of them only crowd the flags' memory channel (measured)
      if (lane < n_rep) st_dev_u32(&p.flags[lane * G + wg], epoch);
      const uint32_t* flags = p.flags + rep * G;
      bool ok = seen();
      for (int it = 0; it < p.spin_limit && !ok; ++it) {
        bool mine = true;
        for (int w0 = 0; w0 < G; w0 += 256) {   // four loads in flight: a poll is one trip to memory
          uint32_t f[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) f[i] = ld_dev_u32(&flags[min(w0 + i * 64 + lane, G - 1)]);
#pragma unroll
          for (int i = 0; i < 4; ++i) mine &= (int)(f[i] - epoch) >= 0;
        }
        ok = __all(mine);
        if (ok && lane == 0) __hip_atomic_store(&s_seen, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        ok = ok || seen();
      }
      if (!ok && lane == 0) { s_fail = 1; st_dev_u32(p.status, 1u); }
    };

    float* out_prev = nullptr;   // of the layer before
    int outw_prev = 0;
    for (int l = 0; l < p.L; ++l) {
      const Layer ly = layer_of(l);
      const int n_in = ly.xm;   // tensors to quantize for this layer
      const float st0 = l == 0 ? p.s_static : ly.s_in[0], st1 = l == 0 ? p.s_static : ly.s_in[1];
      const bool dynamic = !(st0 > 0.f);
      // ---------------- exchange, step A: max|.| of the tensor(s) entering layer l
      if (wave == RES_WORKERS) stamp(l, 0);
      float mx[2] = {0.f, 0.f};
      if (dynamic) {
        if (l == 0) {
          const int n4 = (p.T * ly.in) >> 2;
          const float4* x4 = reinterpret_cast<const float4*>(p.x);
          for (int i = wg * 256 + e; i < n4; i += G * 256) {
            const float4 v = x4[i];
            mx[0] = fmaxf(mx[0], fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
          }
        } else {
          // the outputs this workgroup produced in layer l-1
          mx[0] = mx_out[0]; mx[1] = mx_out[1];
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) mx[m] = fmaxf(mx[m], __shfl_xor(mx[m], o, 64));
          if (lane == 0) s_wmax[ewave][m] = mx[m];
        }
      }
      if (nout_prev * n_apart_prev > RES_STASH) __builtin_amdgcn_s_waitcnt(0x0F70);   // values that are read back from memory have arrived there
      __syncthreads();   // P1
      if (dynamic) {
        ++epoch;
        if (ewave == 0) {
          const int m = lane & (n_in - 1), r = lane >> (n_in - 1);   // n_in is 1 or 2
          if (r < n_rep) {
            float v = s_wmax[0][m];
#pragma unroll
            for (int w = 1; w < RES_EPI; ++w) v = fmaxf(v, s_wmax[w][m]);
            __hip_atomic_store(&p.amax_tag[(r * G + wg) * 2 + m], ((unsigned long long)epoch << 32) | __float_as_uint(v), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          }
        }
        const unsigned long long* tags = p.amax_tag + rep * G * 2;
        bool ok = ewave != 0 || seen();   // one polling wave per workgroup
        for (int it = 0; it < p.spin_limit && !ok; ++it) {
          bool mine = true;
          float g0 = 0.f, g1 = 0.f;
          for (int w0 = 0; w0 < G; w0 += 256) {
            unsigned long long t0[4], t1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const unsigned long long* at = &tags[min(w0 + i * 64 + lane, G - 1) * 2];
              t0[i] = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              t1[i] = n_in == 2 ? __hip_atomic_load(at + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (unsigned long long)epoch << 32;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              mine &= (uint32_t)(t0[i] >> 32) == epoch && (uint32_t)(t1[i] >> 32) == epoch;
              g0 = fmaxf(g0, __uint_as_float((uint32_t)t0[i]));
              g1 = fmaxf(g1, __uint_as_float((uint32_t)t1[i]));
            }
          }
          ok = __all(mine);
          if (ok) {
            // every workgroup's maximum of this epoch: the scales (any wave that gets here writes the same values)
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) { g0 = fmaxf(g0, __shfl_xor(g0, o, 64)); g1 = fmaxf(g1, __shfl_xor(g1, o, 64)); }
            if (lane == 0) {
              s_scale[0] = __fdiv_rn(g0, qmax); s_scale[1] = __fdiv_rn(g1, qmax);
              __hip_atomic_store(&s_seen, epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
          }
          ok = ok || seen();
        }
        if (!ok && lane == 0) { s_fail = 1; s_scale[0] = 0.f; s_scale[1] = 0.f; st_dev_u32(p.status, 2u); }
      } else if (e == 0) {
        s_scale[0] = st0; s_scale[1] = st1;
      }
      __syncthreads();   // P2
      if (wave == RES_WORKERS) stamp(l, 1);
      // ---------------- exchange, step B: every workgroup writes the codes of what it produced
      {
        const float s0 = s_scale[0], s1 = s_scale[1];
        auto q1 = [&](float v, float s) __attribute__((always_inline)) {
          const float q = fminf(fmaxf(rintf(__fdiv_rn(v, s)), -qmax), qmax);
          return s > 0.f ? (int)q : 0;
        };
        uint32_t* qw = reinterpret_cast<uint32_t*>(ly.qin);
        if (l == 0) {
          const int in = ly.in, q4 = in >> 2, n4 = p.T * q4;
          const float4* x4 = reinterpret_cast<const float4*>(p.x);
          for (int i = wg * 256 + e; i < n4; i += G * 256) {
            const float4 v = x4[i];
            const int tq = i / q4, k = (i - tq * q4) * 4;
            const uint32_t c = (uint32_t)(uint8_t)q1(v.x, s0) | ((uint32_t)(uint8_t)q1(v.y, s0) << 8) | ((uint32_t)(uint8_t)q1(v.z, s0) << 16) |
                               ((uint32_t)(uint8_t)q1(v.w, s0) << 24);
            st_dev_u32(&qw[(((k >> 6) * 64 + ((k >> 4) & 3) * 16 + tq) * 16 + (k & 15)) >> 2], c);
          }
        } else {
          // a wave takes an output row block, a lane four neighbouring channels of a token, which are four neighbouring bytes of a fragment
          const int tq = lane >> 2, c4 = (lane & 3) * 4;
          for (int j = ewave; j < nout_prev; j += RES_EPI) {
            const int col = __builtin_amdgcn_readfirstlane(s_col[j]) * 16 + c4;
#pragma unroll
            for (int m = 0; m < 2; ++m)
              if (m < n_in) {
                const int si = j * n_in + m;
                float4 v;
                if (si < RES_STASH) {
                  v = *reinterpret_cast<const float4*>(&stash[si * 256 + tq * 16 + c4]);
                } else {
                  const uint32_t* o = reinterpret_cast<const uint32_t*>(out_prev + ((size_t)m * p.T + min(tq, p.T - 1)) * outw_prev + col);
                  v = make_float4(__uint_as_float(ld_dev_u32(o)), __uint_as_float(ld_dev_u32(o + 1)), __uint_as_float(ld_dev_u32(o + 2)),
                                  __uint_as_float(ld_dev_u32(o + 3)));
                }
                const float sm = m == 0 ? s0 : s1;
                const uint32_t w = (uint32_t)(uint8_t)q1(v.x, sm) | ((uint32_t)(uint8_t)q1(v.y, sm) << 8) | ((uint32_t)(uint8_t)q1(v.z, sm) << 16) |
                                   ((uint32_t)(uint8_t)q1(v.w, sm) << 24);
                if (tq < p.T) st_dev_u32(&qw[((size_t)m * ly.nks * 1024 + (size_t)(((col >> 6) * 64 + ((col >> 4) & 3) * 16 + tq) * 16 + (col & 15))) >> 2], w);
              }
          }
        }
        // codes beyond in_features are zero: the first workgroup writes them
        if (wg == 0) {
          const int pad4 = (ly.in_pad - ly.in) >> 2;
          for (int i = e; i < p.T * pad4 * n_in; i += 256) {
            const int m = i / (p.T * pad4), r = i - m * (p.T * pad4);
            const int tq = r / pad4, k = ly.in + (r - tq * pad4) * 4;
            st_dev_u32(&qw[((size_t)m * ly.nks * 1024 + (size_t)(((k >> 6) * 64 + ((k >> 4) & 3) * 16 + tq) * 16 + (k & 15))) >> 2], 0u);
          }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's device-scope stores have completed
      }
      __syncthreads();   // P3
      if (wave == RES_WORKERS) stamp(l, 2);
      ++epoch;
      grid_wait();
      // row scales and bias of a unit: value i of 128
      auto fetch_side = [&](const int* d, int slot, int i) __attribute__((always_inline)) {
        const int it = i >> 4, c = i & 15;
        // bias: of the items' rows, or of the gate and the up rows (a gate||up unit's second and third row block)
        const float sc = it < d[UE_ITEMS] ? ly.scales[(size_t)d[UE_POS + it] * 16 + c] : 0.f;
        const float bb = ly.bias != nullptr && it < (ly.gated ? 3 : d[UE_ITEMS]) ? ly.bias[d[(ly.gated ? UE_ORB : UE_IRB) + it] * 16 + c] : 0.f;
        side[slot * 256 + i] = sc;
        side[slot * 256 + 128 + i] = bb;
      };
      if (ewave != 0) {
        // the waves that do not poll fetch what the layer's epilogues need (a poll would come back behind these cold loads)
        const int n = min(ly.nu, RES_SIDE) * 128;
        for (int i = e - 64; i < n; i += RES_EPI * 64 - 64) fetch_side(&s_desc[ly.at + (i >> 7) * ly.stride + ly.nsub * 16], i >> 7, i & 127);
      }
      if (wave == RES_WORKERS) stamp(l, 3);
      __syncthreads();   // P4: the workers may read the codes entering layer l

      // ---------------- the layer's units
      const float sx0 = s_scale[0], sx1 = s_scale[1];
      const int nu = ly.nu;
      const bool last = l == p.L - 1;
      // the layer's description in registers (ly comes from LDS)
      const int e_reduce = ly.reduce, e_xm = ly.xm, e_act = ly.act, e_pre = ly.res_pre_act, e_gated = ly.gated, e_outw = ly.out_w;
      const int e_resm = ly.res_members, e_resdev = ly.res_device, e_nsub = ly.nsub, e_stride = ly.stride, e_at = ly.at, e_M = p.M, e_T = p.T;
      const long long e_resms = ly.res_mstride;
      const float* e_bias = ly.bias;
      const float* e_res = ly.res;
      float* e_out = ly.out;
      const int e_klo0 = p.member_lo[0], e_khi0 = p.member_hi[0], e_klo1 = p.member_lo[1], e_khi1 = p.member_hi[1];
      const bool fold_sx = e_reduce && e_M > 1;
      const int n_apart = e_reduce ? 1 : e_M;
      mx_out[0] = 0.f; mx_out[1] = 0.f;
      nout_prev = 0; n_apart_prev = n_apart;
      for (int u = 0; u < nu; ++u) {
        const int* d = &s_desc[e_at + u * e_stride + e_nsub * 16];
        const int n_items = dword_at(d, UE_ITEMS), n_out = e_gated ? 1 : dword_at(d, UE_OUTS), first = nout_prev;
        // per item 4 bits: its member, 2: the last of its sum, 4: in use; and the sums without an item (bit 2 * output + member)
        int ctl = 0, empty = 0, out4 = 0, up = 0;   // out4: the items' outputs; up: items of the up block
        {
          const int ko0 = dword_at(d, UE_KO), ko1 = dword_at(d, UE_KO + 1);
          int next = -1;
          for (int o = 0; o < n_out; ++o) empty |= (n_apart == 2 ? 3 : 1) << (2 * o);
#pragma unroll
          for (int i = PIPE_RES_MAX_ITEMS - 1; i >= 0; --i) {
            if (i >= n_items) continue;
            const int ko = (i < 4 ? ko0 : ko1) >> (8 * (i & 3)) & 255, k = ko & 15, o = ko >> 4;
            const int m = k >= e_klo0 && k <= e_khi0 ? 0 : (e_M > 1 && k >= e_klo1 && k <= e_khi1 ? 1 : -1);
            if (m < 0) continue;
            const int g = fold_sx ? 2 * o : 2 * o + m;
            ctl |= (4 | (g != next ? 2 : 0) | m) << (4 * i);
            out4 |= o << (4 * i);
            next = g;
            empty &= ~(1 << g);
          }
          up = out4;
        }
        // skip tensors: what output o of member m (or the member sum) adds.  Requested before the unit's barrier, like everything
        // that comes from memory: a wait for a load also waits for the stores before it, and a device-scope (write-through) store
        // takes more than a microsecond to complete.
        float rsv[PIPE_RES_MAX_ITEMS][2];
        if (e_res != nullptr) {
#pragma unroll
          for (int o = 0; o < PIPE_RES_MAX_ITEMS; ++o) {
            rsv[o][0] = 0.f; rsv[o][1] = 0.f;
            if (o >= n_out) continue;
            const int col = dword_at(d, UE_ORB + o) * 16 + ch;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
              if (m >= n_apart) continue;
              // the members summed into this output each add their own skip tensor (members kept apart:
              // member m adds its own if it has one)
              const int n_res = e_reduce ? e_resm : (m < e_resm ? 1 : 0);
              const float* rp = e_res + (size_t)(e_reduce ? 0 : m) * e_resms + (size_t)min(t, e_T - 1) * e_outw + col;
              float rsum = 0.f;
              for (int mm = 0; mm < n_res; ++mm) {
                // a tensor an earlier layer of this launch produced is read with device scope
                const float* rq = rp + (size_t)mm * e_resms;
                rsum += e_resdev ? __uint_as_float(ld_dev_u32(reinterpret_cast<const uint32_t*>(rq))) : *rq;
              }
              rsv[o][m] = rsum;
            }
          }
        }
        // (units beyond the side array: two more slots in turn, so that one is never written before everyone has read it)
        const int slot = u < RES_SIDE ? u : RES_SIDE + (u & 1);
        if (u >= RES_SIDE && e < 128) fetch_side(d, slot, e);
        const float* scl = side + slot * 256 + ch;
        int irb[PIPE_RES_MAX_ITEMS];
#pragma unroll
        for (int i = 0; i < PIPE_RES_MAX_ITEMS; ++i) irb[i] = dword_at(d, UE_IRB + i);
        auto bias_at = [&](int i) __attribute__((always_inline)) { return scl[128 + i * 16]; };   // of item i (gate||up: row block i)
        float scv[PIPE_RES_MAX_ITEMS];
        __syncthreads();   // the workers have added up this unit's tiles
        if (wave == RES_WORKERS && u == 0) stamp(l, 5);
        int a_it[PIPE_RES_MAX_ITEMS];
#pragma unroll
        for (int i = 0; i < PIPE_RES_MAX_ITEMS; ++i) {
          if (i >= 4 && n_items <= 4) { a_it[i] = 0; scv[i] = 0.f; continue; }
          a_it[i] = tile[buf][i][fidx];   // (slots of items that the unit does not have are zero)
          tile[buf][i][fidx] = 0;
          scv[i] = scl[i * 16];
        }
        int rs[2] = {0, 0};
        if (OFF != 0) {
#pragma unroll
          for (int m = 0; m < XM; ++m) {   // (all who read a token's are in one wave)
            rs[m] = tile[buf][PIPE_RES_MAX_ITEMS + m][t];
            if (ch == 0) tile[buf][PIPE_RES_MAX_ITEMS + m][t] = 0;
          }
        }
        buf ^= 1;
        // ---- stores: the last layer's result plainly, a hidden tensor with device scope (other workgroups'
        // skips read it), into the stash (quantized in the next exchange), and its max
        auto put = [&](int o, int m, int rb, float v) __attribute__((always_inline)) {
          if (tok) {
            float* dst = e_out + ((size_t)m * e_T + t) * e_outw + rb * 16 + ch;
            if (last) {
              *dst = v;
            } else {
              st_dev_u32(reinterpret_cast<uint32_t*>(dst), __float_as_uint(v));
              const int si = (first + o) * n_apart + m;
              if (si < RES_STASH) stash[si * 256 + e] = v;
              if (m == 0) mx_out[0] = fmaxf(mx_out[0], fabsf(v)); else mx_out[1] = fmaxf(mx_out[1], fabsf(v));
            }
          }
        };
        if (e_gated) {
          // items with slot 0 are the gate block's orders, slot 1 the up block's; h = SiLU(gate) * up per member
          float gs[2] = {0.f, 0.f}, us[2] = {0.f, 0.f};
#pragma unroll
          for (int i = 0; i < PIPE_RES_MAX_ITEMS; ++i) {
            const int c = ctl >> (4 * i);
            if (!(c & 4)) continue;
            const float a = (float)(a_it[i] - OFF * rs[0]);
            if (((up >> (4 * i)) & 1) == 0) {
              if (c & 1) gs[1] = fmaf(scv[i], a, gs[1]); else gs[0] = fmaf(scv[i], a, gs[0]);
            } else {
              if (c & 1) us[1] = fmaf(scv[i], a, us[1]); else us[0] = fmaf(scv[i], a, us[0]);
            }
          }
          const float bg = bias_at(1), bu = bias_at(2);
          const int rb = dword_at(d, UE_ORB);
#pragma nounroll
          for (int m = 0; m < e_M; ++m) {
            const float vg = fmaf(sx0, m == 0 ? gs[0] : gs[1], m == 0 ? bg : 0.f), vu = fmaf(sx0, m == 0 ? us[0] : us[1], m == 0 ? bu : 0.f);
            put(0, m, rb, vg / (1.f + expf(-vg)) * vu);
          }
        } else {
          // v: a sum's fp32 value (same rounding as the per-layer kernels)
          auto act_put = [&](int o, int m, int rb, float v, float rsum, auto gelu) __attribute__((always_inline)) {
            if (e_pre) v += rsum;
            if (decltype(gelu)::value) v = gelu_erf(v);
            else if (e_act == PIPE_ACT_RELU) v = fmaxf(v, 0.f);
            if (!e_pre) v += rsum;
            put(o, m, rb, v);
          };
          auto skip_of = [&](int o, int m) __attribute__((always_inline)) {
            float rsum = 0.f;
            if (e_res != nullptr) {
#pragma unroll
              for (int i = 0; i < PIPE_RES_MAX_ITEMS; ++i)
                if (i == o) rsum = m == 0 ? rsv[i][0] : rsv[i][1];
            }
            return rsum;
          };
          int n_sum = 0;
          unsigned om = 0;   // GELU: 4 bits per sum: output | member << 3
          float yacc = 0.f;
#pragma unroll
          for (int i = 0; i < PIPE_RES_MAX_ITEMS; ++i) {
            const int c = ctl >> (4 * i);
            if (!(c & 4)) continue;
            const int st_m = e_xm == 1 ? 0 : c & 1;
            const float sx = st_m == 0 ? sx0 : sx1;
            const float a = (float)(a_it[i] - OFF * (st_m == 0 ? rs[0] : rs[1]));
            yacc = fmaf(fold_sx ? scv[i] * sx : scv[i], a, yacc);
            if (!(c & 2)) continue;
            const int o = out4 >> (4 * i) & 7, m = e_reduce ? 0 : c & 1;
            const float bm = (m == 0 || fold_sx) && e_bias != nullptr ? bias_at(i) : 0.f;
            const float v = fold_sx ? yacc + bm : fmaf(sx, yacc, bm);
            if (e_act == PIPE_ACT_GELU) {   // one copy of it, below: eight are code that comes from memory (an epilogue of 1.2 us took 2.7)
              sums[n_sum * 256 + e] = v;
              om |= (unsigned)(o | m << 3) << (4 * n_sum);
              ++n_sum;
            } else {
              act_put(o, m, irb[i], v, skip_of(o, m), std::false_type{});
            }
            yacc = 0.f;
          }
          // GELU, and the sums that no order of their member adds to
#pragma nounroll
          for (int f = 0; f < n_sum || empty != 0; ++f) {
            int o, m;
            float v;
            if (f < n_sum) {
              o = (om >> (4 * f)) & 7; m = (om >> (4 * f + 3)) & 1;
              v = sums[f * 256 + e];
            } else {
              o = __builtin_ctz(empty) >> 1; m = __builtin_ctz(empty) & 1;
              empty &= empty - 1;
              const float bm = (m == 0 || fold_sx) && e_bias != nullptr ? e_bias[dword_at(d, UE_ORB + o) * 16 + ch] : 0.f;
              v = fold_sx ? bm : fmaf(e_xm == 1 || m == 0 ? sx0 : sx1, 0.f, bm);
            }
            const int rb = dword_at(d, UE_ORB + o);
            if (e_act == PIPE_ACT_GELU) act_put(o, m, rb, v, skip_of(o, m), std::true_type{});
            else act_put(o, m, rb, v, skip_of(o, m), std::false_type{});
          }
        }
        if (e < n_out) s_col[first + e] = d[UE_ORB + e];
        nout_prev = first + n_out;
        if (wave == RES_WORKERS && u == 0) stamp(l, 6);
      }
      out_prev = e_out; outw_prev = e_outw;
      if (wave == RES_WORKERS) stamp(l, 4);
    }
    if (wg == 0 && e == 0 && epoch != epoch0) st_dev_u32(p.gen, epoch);
  }
  if (p.trace != nullptr) {
    __syncthreads();
    if ((int)threadIdx.x < p.L * 8) p.trace[(size_t)wg * p.L * 8 + threadIdx.x] = (&s_ts[0][0])[threadIdx.x];
  }
}

template <int BITS, int XM>
int launch_res(const ResParams& p, hipEvent_t ev0, hipEvent_t ev1, hipStream_t st) {
  constexpr int RD = (XM == 2 && BITS == 2) ? 2 : 4;   // rounds of code registers; two tensors of ternary fragments leave room for two
  static bool attr_set = false;
  if (!attr_set) {
    PIPE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&chain_resident_kernel<BITS, XM, RD>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, RES_PAD_LDS));
    attr_set = true;
  }
  if (pipe_dry_run()) return PIPE_OK;
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL((chain_resident_kernel<BITS, XM, RD>), dim3((unsigned)p.G), dim3(RES_THREADS), RES_PAD_LDS, st, ev0, ev1, 0, p);
  else
    hipLaunchKernelGGL((chain_resident_kernel<BITS, XM, RD>), dim3((unsigned)p.G), dim3(RES_THREADS), RES_PAD_LDS, st, p);
  PIPE_HIP(hipGetLastError());
  return PIPE_OK;
}

}  // namespace

// ------------------------------------------------------------------ host side
// Work units of the resident kernel for one expansion.  kind 0: groups of output row blocks with all
// their orders, at most 4 items each, when there are at least as many groups as workgroups, else one unit per
// output row block; kind 1: a gate||up layer as (gate block, up block) pairs, two sub-units of at most 4 items.
int pipe_resident_tables(const pipe_expansion* ce, int kind, int G, ResidentTables* out) {
  pipe_expansion* e = const_cast<pipe_expansion*>(ce);
  ResidentTables& t = e->res_tables[kind];
  if (t.subs_dev != nullptr && t.G == G) { *out = t; return PIPE_OK; }
  if (pipe_capturing()) return PIPE_ENOTREADY;
  if (e->bin_cap != 4 || e->K > 4) return PIPE_ESHAPE;
  // kind 0: units of at most 4 items and 4 output row blocks, formed here from the row blocks' stored orders:
  // row blocks with the most orders first, those with equal sets of orders next to each other, each into the
  // most recent of the last 64 units that still has room.  (The bins of the weight-streaming kernel fix where
  // the codes lie in memory and are packed for the fewest unused positions; units need no neighbours in
  // memory, and this grouping measured 6 % faster on an 8-layer stack than units taken from those bins: its
  // units hold row blocks of like weight, so fewer units carry several outputs through the epilogue.)
  struct RbItems { uint32_t mask; int pop; int rb; };
  struct UnitBin { int n_out, out_rb[4]; };
  std::vector<UnitBin> bins;
  std::vector<RbItems> rbs;
  if (kind == 0) {
    rbs.resize(e->n_rb);
    for (int rb = 0; rb < e->n_rb; ++rb) {
      uint32_t mask = 0;
      for (int kk = 0; kk < e->K; ++kk)
        if (e->pos_of[(size_t)kk * e->n_rb + rb] >= 0) mask |= 1u << kk;
      rbs[rb] = RbItems{mask, __builtin_popcount(mask), rb};
    }
    std::stable_sort(rbs.begin(), rbs.end(), [](const RbItems& a, const RbItems& b) {
      if (a.pop != b.pop) return a.pop > b.pop;
      if (a.mask != b.mask) return a.mask < b.mask;
      return a.rb < b.rb;
    });
    std::vector<int> room;
    for (const RbItems& it : rbs) {
      int which = -1;
      for (int j = (int)bins.size() - 1; j >= 0 && j >= (int)bins.size() - 64; --j)
        if (room[j] >= it.pop) { which = j; break; }
      if (which < 0) {
        bins.push_back(UnitBin{});
        room.push_back(4);
        which = (int)bins.size() - 1;
      }
      UnitBin& bn = bins[which];
      bn.out_rb[bn.n_out++] = it.rb;
      room[which] -= it.pop;
    }
  }
  const int n_bins = (int)bins.size();
  std::vector<int32_t> subs, epi;
  int n_units = 0, nsub = 1;
  auto push_sub = [&](const int* pos, const int* k, int n, int slot0, int last) {
    int32_t s[16] = {0};
    for (int r = 0; r < 4; ++r) { s[r] = pos[r < n ? r : 0]; s[4 + r] = r < n ? k[r] : 0; }
    s[8] = n; s[9] = slot0; s[10] = last;
    subs.insert(subs.end(), s, s + 16);
  };
  auto push_epi = [&](int n_items, int n_out, const int* k, const int* slot, const int* pos, const int* orb, int n_orb) {
    int32_t s[UE_N] = {0};
    s[UE_ITEMS] = n_items; s[UE_OUTS] = n_out;
    for (int i = 0; i < n_items; ++i) {
      s[UE_POS + i] = pos[i];
      s[UE_IRB + i] = orb[slot[i]];
      s[UE_KO + i / 4] |= (k[i] | slot[i] << 4) << (8 * (i & 3));
    }
    for (int o = 0; o < n_orb; ++o) s[UE_ORB + o] = orb[o];
    epi.insert(epi.end(), s, s + UE_N);
  };
  if (kind == 0) {
    const bool by_bin = n_bins >= G;   // (one unit per output row block whenever bins deal unevenly measured slower: the per-unit barrier and epilogue cost more than the imbalance)
    struct U { int n; int pos[PIPE_RES_MAX_ITEMS], k[PIPE_RES_MAX_ITEMS], slot[PIPE_RES_MAX_ITEMS], orb[PIPE_RES_MAX_ITEMS], n_out; };
    auto add = [&](U& u, int rb) {
      u.orb[u.n_out] = rb;
      for (int kk = 0; kk < e->K; ++kk) {
        const int32_t q = e->pos_of[(size_t)kk * e->n_rb + rb];
        if (q < 0) continue;
        u.pos[u.n] = q; u.k[u.n] = kk; u.slot[u.n] = u.n_out;
        ++u.n;
      }
      ++u.n_out;
    };
    std::vector<U> us;
    // Between one and two bins a workgroup: one unit of up to 8 items each, dealt by weight, as two sub-units with one epilogue (the workgroups
    // with a second unit of 4 kept the others waiting for 5 us of an 11008 x 4096 ternary layer, 16 tokens, 301 bins).
    if (n_bins > G && n_bins <= 2 * G) {
      us.assign(G, U{});
      bool fits = true;
      int most = 0;
      for (const RbItems& it : rbs) {   // (most orders first)
        U& u = *std::min_element(us.begin(), us.end(), [](const U& a, const U& b) { return a.n < b.n; });
        if (u.n + it.pop > PIPE_RES_MAX_ITEMS || u.n_out == PIPE_RES_MAX_ITEMS) { fits = false; break; }
        add(u, it.rb);
        most = std::max(most, u.n);
      }
      if (fits) nsub = most > 4 ? 2 : 1;
      else us.clear();
    }
    if (us.empty()) {
      for (int b = 0; b < n_bins; ++b) {
        const UnitBin& bn = bins[b];
        if (by_bin) us.push_back(U{});
        for (int o = 0; o < bn.n_out; ++o) {
          if (!by_bin) us.push_back(U{});
          add(us.back(), bn.out_rb[o]);
        }
      }
    }
    std::stable_sort(us.begin(), us.end(), [](const U& a, const U& b) { return a.n > b.n; });
    for (const U& u : us) {
      push_sub(u.pos, u.k, std::min(u.n, 4), 0, nsub == 1);
      if (nsub == 2) push_sub(u.pos + 4 * (u.n > 4), u.k + 4 * (u.n > 4), std::max(u.n - 4, 0), 4, 1);
      push_epi(u.n, u.n_out, u.k, u.slot, u.pos, u.orb, u.n_out);
    }
    n_units = (int)us.size();
  } else {
    if (e->n_rb % 2 != 0) return PIPE_ESHAPE;
    nsub = 2;
    const int half = e->n_rb / 2;
    struct P { int rb; int n; };
    std::vector<P> ps;
    auto items_of = [&](int rb, int* pos, int* k) {
      int n = 0;
      for (int kk = 0; kk < e->K; ++kk) {
        const int32_t q = e->pos_of[(size_t)kk * e->n_rb + rb];
        if (q >= 0) { pos[n] = q; k[n] = kk; ++n; }
      }
      return n;
    };
    for (int rb = 0; rb < half; ++rb) {
      int pos[4], k[4];
      ps.push_back(P{rb, items_of(rb, pos, k) + items_of(rb + half, pos, k)});
    }
    std::stable_sort(ps.begin(), ps.end(), [](const P& a, const P& b) { return a.n > b.n; });
    for (const P& pr : ps) {
      int pg[4], kg[4], pu[4], ku[4];
      const int ng = items_of(pr.rb, pg, kg), nu = items_of(pr.rb + half, pu, ku);
      push_sub(pg, kg, ng, 0, 0);
      push_sub(pu, ku, nu, 4, 1);
      // the epilogue indexes the LDS tiles: gate items at 0.., up items at 4..; items the blocks do not have: an order that no member holds
      int kk[8], ss[8] = {0, 0, 0, 0, 1, 1, 1, 1}, pp[8] = {0};
      for (int i = 0; i < 4; ++i) { kk[i] = i < ng ? kg[i] : UE_NO_ORDER; pp[i] = i < ng ? pg[i] : 0; }
      for (int i = 0; i < 4; ++i) { kk[4 + i] = i < nu ? ku[i] : UE_NO_ORDER; pp[4 + i] = i < nu ? pu[i] : 0; }
      const int orb[3] = {pr.rb, pr.rb, pr.rb + half};   // the output, the bias of the gate and of the up rows
      push_epi(8, 1, kk, ss, pp, orb, 3);
    }
    n_units = (int)ps.size();
  }
  int32_t *sd = nullptr, *ed = nullptr;
  PIPE_HIP(hipMalloc(&sd, subs.size() * 4));
  if (!pipe_hip_ok(hipMalloc(&ed, epi.size() * 4), "hipMalloc(units)")) { (void)hipFree(sd); return PIPE_ENOMEM; }
  if (!pipe_hip_ok(hipMemcpy(sd, subs.data(), subs.size() * 4, hipMemcpyHostToDevice), "hipMemcpy(units)") ||
      !pipe_hip_ok(hipMemcpy(ed, epi.data(), epi.size() * 4, hipMemcpyHostToDevice), "hipMemcpy(units)")) {
    (void)hipFree(sd); (void)hipFree(ed);
    return PIPE_EDEVICE;
  }
  if (t.subs_dev) (void)hipFree(t.subs_dev);
  if (t.epi_dev) (void)hipFree(t.epi_dev);
  t.subs_dev = sd; t.epi_dev = ed; t.n_units = n_units; t.nsub = nsub; t.G = G;
  *out = t;
  return PIPE_OK;
}

int pipe_resident_workgroups() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 64;
    cus = std::min(n, PIPE_RES_MAX_G);
  }
  return cus;
}

int launch_resident_chain(const ResidentArgs& a, hipStream_t st) {
  if (a.L < 1 || a.L > PIPE_RES_MAX_LAYERS || a.T < 1 || a.T > PIPE_RES_MAX_T || a.M < 1 || a.M > PIPE_RES_MAX_M) return PIPE_ESHAPE;
  ResParams p;
  std::memset(&p, 0, sizeof(p));
  p.L = a.L; p.T = a.T; p.M = a.M; p.G = a.G;
  for (int m = 0; m < a.M; ++m) {
    p.member_lo[m] = a.member_lo[m]; p.member_hi[m] = a.member_hi[m];
    for (int k = a.member_lo[m]; k <= a.member_hi[m] && k < 4; ++k) p.member_of[k] = m;
  }
  p.x = a.x; p.s_static = a.s_static; p.act_qmax = g_act_qmax_host;
  p.n_rep = std::max(1, std::min(8, PIPE_RES_FLAGS / a.G));
  p.flags = a.flags; p.amax_tag = a.amax_tag; p.gen = a.gen; p.status = a.status;
  p.spin_limit = g_resident_spin_limit;
  p.trace = g_resident_trace;
  const int bits = a.layers[0].e->bits;
  for (int l = 0; l < a.L; ++l) {
    const ResidentLayerArgs& la = a.layers[l];
    const pipe_expansion* e = la.e;
    if (e->bits != bits || e->bin_cap != 4) return PIPE_ESHAPE;
    ResLayer& ly = p.layer[l];
    ly.codes = e->codes_dev; ly.scales = e->scales_all_dev;
    ly.subs = la.tables.subs_dev; ly.epi = la.tables.epi_dev;
    ly.n_units = la.tables.n_units; ly.nsub = la.tables.nsub;
    ly.bias = la.bias; ly.out = la.out; ly.res = la.res; ly.res_mstride = la.res_mstride;
    ly.qin = la.qin;
    ly.n_tiles = e->in_pad / (512 / e->bits); ly.nks = e->nks;
    ly.out_w = la.gated ? e->out / 2 : e->out;
    ly.in = e->in; ly.in_pad = e->in_pad;
    ly.xm = l == 0 ? 1 : a.M;
    ly.act = la.act; ly.res_members = la.res_members; ly.res_pre_act = la.res_pre_act; ly.gated = la.gated;
    ly.reduce = l == a.L - 1 ? 1 : 0;
    ly.res_device = la.res_device;
    ly.s_in[0] = la.s_in[0]; ly.s_in[1] = la.s_in[1];
  }
  // the descriptors of the busiest workgroup (the first) have to fit their LDS copy
  int desc_ints = 0;
  for (int l = 0; l < a.L; ++l) desc_ints += ceil_div(p.layer[l].n_units, p.G) * (p.layer[l].nsub * 16 + 32);
  if (desc_ints > PIPE_RES_DESC_INTS) return PIPE_ESHAPE;
  if (a.M == 1) {
    switch (bits) {
      case 8: return launch_res<8, 1>(p, a.ev_start, a.ev_stop, st);
      case 4: return launch_res<4, 1>(p, a.ev_start, a.ev_stop, st);
      default: return launch_res<2, 1>(p, a.ev_start, a.ev_stop, st);
    }
  }
  switch (bits) {
    case 8: return launch_res<8, 2>(p, a.ev_start, a.ev_stop, st);
    case 4: return launch_res<4, 2>(p, a.ev_start, a.ev_stop, st);
    default: return launch_res<2, 2>(p, a.ev_start, a.ev_stop, st);
  }
}
