// Device helpers shared by the two tiled contraction kernels (pipe_gemm.hip, pipe_gemm_bins.hip).
#pragma once
#include "pipe_internal.h"

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// One 64-k step of packed codes as int8 MFMA operand: 8-bit codes are the operand, a 4-bit step is two dwords (lo, hi),
// a ternary one a single dword (lo).
__device__ __forceinline__ v4i widen4(uint32_t lo, uint32_t hi) {
  return v4i{(int)(lo & 0x0F0F0F0Fu), (int)((lo >> 4) & 0x0F0F0F0Fu), (int)(hi & 0x0F0F0F0Fu), (int)((hi >> 4) & 0x0F0F0F0Fu)};
}
__device__ __forceinline__ v4i widen2(uint32_t a) {
  return v4i{(int)(a & 0x03030303u), (int)((a >> 2) & 0x03030303u), (int)((a >> 4) & 0x03030303u), (int)((a >> 6) & 0x03030303u)};
}

// A load known to hit global memory.  Pointers rebuilt from integers are "generic" to the
// compiler, which would emit FLAT loads: those also count as LDS operations (every wait on the
// LDS fragment reads would then wait for the weight prefetch as well) and are ordered against
// the LDS-direct loads.
__device__ __forceinline__ v4u gload16(const void* p) {
  typedef const __attribute__((address_space(1))) v4u* gptr;
  return *(gptr)(unsigned long long)p;
}

// Loads of schedule tables at wave-uniform addresses through the constant address space: the
// compiler then uses scalar loads (the tables are written once, by the host, when the expansion
// is built; no kernel ever stores to them), which cost no vector registers and no vector wait.
template <class T>
__device__ __forceinline__ T cload(const T* base, size_t idx) {
  typedef const __attribute__((address_space(4))) T* cptr;
  return ((cptr)(unsigned long long)base)[idx];
}

// Which tile a workgroup computes.  Blocks i, i + 8, ... of a launch run on one XCD (one L2): chunks of `strip` column tiles
// x `toks` token tiles, column by column, are dealt to the 8 XCDs in turn, strip after strip (heaviest column tiles first).
struct TileOrder {
  int n_ct, n_tt, strip, toks;
  __host__ __device__ int chunks() const { return (n_ct + strip - 1) / strip * ((n_tt + toks - 1) / toks); }
  __host__ __device__ int blocks() const { return (chunks() + 7) / 8 * 8 * strip * toks; }
  __device__ __forceinline__ bool tile(int block, int* ct, int* tt) const {
    const int size = strip * toks, xcd = block & 7, j = block >> 3;
    const int c = j / size * 8 + xcd, local = j - j / size * size;
    const int per_strip = (n_tt + toks - 1) / toks, s = c / per_strip;
    const int col = local / toks;
    *ct = s * strip + col;
    *tt = (c - s * per_strip) * toks + local - col * toks;
    return *ct < n_ct && *tt < n_tt;
  }
};

// Few token tiles and many column tiles: a chunk is a column tile with all its token tiles (its codes are read by one
// XCD, the few activations by all: 333 tokens of the 11008 x 4096 ternary layer 29.8 us, 33.1 us dealt tile by tile).
// Otherwise strips of 8 column tiles and one token tile of a strip per chunk, so that neither the XCDs nor the rounds differ by
// more than 8 tiles (super-tiles of 8 x 8 per XCD: 49.8 against 29.8 us at 333 tokens, 212 against 203 at 4096; strips of
// 1, 4 and 16: 204, 205 and 209 us).
// by_weight (tiles of one strip cost differently: pass by pass): from 32 token tiles on, 8 x 8 tiles per chunk, or 16 x 4
// where that deals every XCD a share of every strip, so that an XCD starts its heaviest tiles first (eight 2048 x 2048 ternary
// layers of 8 orders, 3603 tokens: 68.4 against 72.7 us a layer).
static inline TileOrder tile_order(int n_ct, int n_tt, bool by_weight) {
  TileOrder o;
  o.n_ct = n_ct;
  o.n_tt = n_tt;
  if (by_weight && n_tt >= 32) {
    const bool tall = (n_tt + 7) / 8 % 8 != 0 && (n_tt + 3) / 4 % 8 == 0;
    o.strip = tall ? 16 : 8;
    o.toks = tall ? 4 : 8;
  } else if (n_tt <= 16 && n_ct >= 16) {
    o.strip = 1;
    o.toks = n_tt;
  } else {
    o.strip = n_ct < 8 ? n_ct : 8;
    o.toks = 1;
  }
  return o;
}
