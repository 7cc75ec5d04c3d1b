// Pieces that the tiled gather kernels share: operand padding, the work split, the row table of a panel
// of offsets and the order in which its channels are read.
#pragma once

#include "common.hpp"
#include "lds_dma.hpp"

namespace ssconv {

constexpr int kTileThreads = 512;            // 8 wavefronts, two per SIMD
constexpr int kTileMaxK = 128;
constexpr int kTileLds = 160 * 1024;
constexpr int kTileWG = 256;                 // one workgroup per compute unit
constexpr int kTileMisc = 1024 + kTileMaxK * 5 + 16;  // junk block, offset flags, offset list, count
constexpr uint32_t kAbsentRow32 = 0x80000000u;        // row offset past any operand: the DMA writes zeros
constexpr int kRawBufferWord3 = 0x00020000;           // buffer descriptor word 3 for gfx9-family raw loads

__host__ __device__ __forceinline__ int pad8(int c) { return (c + 7) & ~7; }
__host__ __device__ __forceinline__ int pad16(int c) { return (c + 15) & ~15; }
__host__ __device__ __forceinline__ int pad32(int c) { return (c + 31) & ~31; }
// channels of a packed kappa row: whole 8-channel groups, and whole chunks of 32 where the last one is
// padded (a rest of 24)
__host__ __device__ __forceinline__ int pad_k(int c) { return pad8(c) % 32 == 24 ? pad8(c) + 8 : pad8(c); }
inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Rows row0 .. in mt x nt tiles; workgroup i takes the units [i * units / G, (i + 1) * units / G) of the
// (tile, offset) sequence (units = mt * nt * K), so that every workgroup has the same number of offsets
// whatever the tile count.
struct TilePlan {
  int G, mt, nt, panel;  // panel: offsets whose tables fit the LDS at a time
  int64_t row0, units;
};
inline bool whole_tiles(const TilePlan& p, int K) { return p.units % ((int64_t)p.G * K) == 0; }

// Time that cutting nt tiles over G workgroups costs beyond the pieces' traffic, in us: a launch, and a piece after
// the other in the fix-up (300 rows, 5x5x5, 16 -> 16: five tiles of 51 pieces made the bf16 layer 36 us, with 64
// workgroups 20; the generic kernel 24).  G is tried in halves from one per compute unit down.
constexpr int kCutChoices = 4;
inline double cut_us(int G, int64_t nt) { return 8.0 + 0.22 * G / (double)nt; }

// Workgroup i -> slot such that each XCD (i % 8) runs a contiguous range of slots.
__device__ __forceinline__ int xcd_slot(int i, int n) {
  const int x = i & 7, j = i >> 3, q = n >> 3, r = n & 7;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
}

// The workgroup that holds unit u.
__device__ __forceinline__ int64_t unit_owner(const TilePlan& p, int64_t u) {
  int64_t i = u * p.G / p.units;
  while ((i + 1) * p.units / p.G <= u) ++i;
  while (i * p.units / p.G > u) --i;
  return i;
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane at byte offset off of the buffer described by rsrc into LDS at byte
// lds + 16 * lane (buffer_load_dwordx4 with the LDS bit; an offset past the end of the buffer
// writes zeros).  One wait state separates the M0 write from the DMA.
__device__ __forceinline__ void dma16_tile(__amdgpu_buffer_rsrc_t rsrc, uint32_t off, uint32_t lds) {
  const uint32_t l = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(l), "v"(off), "s"(rsrc)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// The rows (byte offsets, kAbsentRow32: no neighbour) of tile rows p0 .. p0 + BM - 1 at offsets s0 .. s0 + ns
// - 1 into rows[ns + 1][BM] (the last row: all absent), and the ordered list act of the offsets that occur
// at all; returns their number.  Begins and ends with a barrier.
template <int BM>
__device__ __forceinline__ int load_panel(const int32_t* __restrict__ nbr, int64_t n_pos, int64_t p0, int s0, int ns,
                                          uint32_t row_bytes, uint32_t* rows, uint32_t* bmask, uint8_t* act,
                                          int* n_act_p) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // opaque: the address arithmetic below must not live through the chunk loop
  const int lane = tid & 63;
  __syncthreads();  // the previous panel (or tile) is done with the table and the stages
  for (int s = tid; s < ns; s += kTileThreads) bmask[s] = 0u;
  if (tid < BM) rows[ns * BM + tid] = kAbsentRow32;
  __syncthreads();
  {
    constexpr int STEP = kTileThreads / BM;  // offsets read side by side, 8 requests in flight per thread
    const int r = tid % BM;
    const int64_t p = p0 + r;
    const bool in = p < n_pos;
    for (int j0 = tid / BM; j0 < ns; j0 += 8 * STEP) {
      int v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        v[j] = in && j0 + STEP * j < ns ? nbr[(int64_t)(s0 + j0 + STEP * j) * n_pos + p] : -1;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j0 + STEP * j < ns) {
          rows[(j0 + STEP * j) * BM + r] = v[j] >= 0 ? (uint32_t)v[j] * row_bytes : kAbsentRow32;
          if (v[j] >= 0) bmask[j0 + STEP * j] = 1u;
        }
    }
  }
  __syncthreads();
  if (tid < 64) {
    int base = 0;
    for (int j0 = 0; j0 < ns; j0 += 64) {
      const int j = j0 + lane;
      const bool a = j < ns && bmask[j] != 0;
      const uint64_t b = __ballot(a);
      if (a) act[base + __popcll(b & ((1ull << lane) - 1ull))] = (uint8_t)j;
      base += __popcll(b);
    }
    if (lane == 0) n_act_p[0] = base;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(n_act_p[0]);
}

// Order of the chunks of n_act offsets of cap channels (a multiple of 8): the `full` whole 32-channel
// chunks of each offset, then, where a rest of 8 or 16 is left, one chunk with the rests of the last
// `quad` (4 or 2) offsets, lane group g reading its share.  Whole chunks start at multiples of 64 bytes
// of the row: chunks that straddle two such pieces cost the texture path a second access per row.
struct ChunkOrder {
  int full, rest, quad;
  __host__ __device__ __forceinline__ explicit ChunkOrder(int cap)
      : full(cap / 32), rest(cap % 32), quad(rest ? 32 / rest : 1) {}
  __host__ __device__ __forceinline__ int chunks(int n_act) const {
    return n_act * full + (rest ? (n_act + quad - 1) / quad : 0);
  }
  // offset slot and first channel of lane group g in chunk c (slot >= n_act: nothing)
  __device__ __forceinline__ void at(int c, int g, int n_act, int* slot, int* ch) const {
    const int per = quad * full + (rest ? 1 : 0), grp = c / per, i = c - grp * per, base = grp * quad;
    const int m = base + quad < n_act ? quad : n_act - base;
    if (i < m * full) {
      *slot = base + i / full;
      *ch = 32 * (i % full) + 8 * g;
    } else {
      *slot = base + 8 * g / rest;
      *ch = 32 * full + 8 * g % rest;
    }
  }
};

// What the chunk loop reads instead of working positions out: entry [c][g] of chunk c and lane group g =
// {byte offset of the offset's row table | channel / 8 << 18, byte offset of the kappa group}; chunks past
// the last are absent rows.  (Positions kept in registers and advanced by branches took 350 instructions a
// chunk of 28 MFMAs, which bound the bf16 kernel.)
// A lane group past the channels (c8: the channels in whole groups of 8; a rest of 24 is padded) or past the
// last offset takes absent rows too: rows read in place go on with the next row there, and an infinity or NaN
// of that row is not undone by kappa's zeros.  Its kappa is the padding, or a group of an offset that the tile
// holds anyway.
constexpr int kChunkAhead = 8;  // absent entries past the last chunk
__device__ __forceinline__ void chunk_table(const ChunkOrder& o, int n_act, int nchunk, const uint8_t* act, int absent,
                                            int bm4, int s0, int c8, int cg, uint32_t group_bytes, uint2* tab) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  for (int i = tid; i < 4 * (nchunk + kChunkAhead); i += kTileThreads) {
    const int c = i >> 2, g = i & 3;
    uint2 e = make_uint2((uint32_t)(absent * bm4), 0u);
    if (c < nchunk) {
      int slot, ch;
      o.at(c, g, n_act, &slot, &ch);
      const int j = act[slot < n_act ? slot : n_act - 1];
      if (slot < n_act && ch < c8) e.x = (uint32_t)(j * bm4) | (uint32_t)(ch >> 3) << 18;
      e.y = (uint32_t)((s0 + j) * cg + (ch >> 3)) * group_bytes;
    }
    tab[i] = e;
  }
  __syncthreads();
}

// Offsets per panel whose row table (BM rows each, and one of absent rows) and chunk table fit `room` bytes of
// LDS, and the bytes they take.
inline int panel_offsets(int room, int BM, int cap, int K) {
  const int per = BM * 4 + 32 * (cap / 32 + 1), fixed = BM * 4 + 32 * kChunkAhead;
  const int n = (room - fixed) / per;
  return n < 0 ? 0 : n < K ? n : K;
}
inline size_t panel_bytes(int panel, int BM, int cap) {
  return (size_t)(panel + 1) * BM * 4 + 32 * ((size_t)panel * (cap / 32 + 1) + kChunkAhead);
}

}  // namespace ssconv
