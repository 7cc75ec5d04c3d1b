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
  int G, mt, nt;
  int64_t row0, units;
};
inline bool whole_tiles(const TilePlan& p, int K) { return p.units % ((int64_t)p.G * K) == 0; }

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
// - 1 into rows[ns][BM], and the ordered list act of the offsets that occur at all; returns their number.
// Begins and ends with a barrier.
template <int BM>
__device__ __forceinline__ int load_panel(const int32_t* __restrict__ nbr, int64_t n_pos, int64_t p0, int s0, int ns,
                                          uint32_t row_bytes, uint32_t* rows, uint32_t* bmask, uint8_t* act,
                                          int* n_act_p) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // opaque: the address arithmetic below must not live through the chunk loop
  const int lane = tid & 63;
  __syncthreads();  // the previous panel (or tile) is done with the table and the stages
  for (int s = tid; s < ns; s += kTileThreads) bmask[s] = 0u;
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
  int full, rest, quad, g_slot, g_ch;
  __device__ __forceinline__ ChunkOrder(int cap, int g)
      : full(cap / 32), rest(cap % 32), quad(rest ? 32 / rest : 1), g_slot(rest ? 8 * g / rest : 0),
        g_ch(rest ? 32 * full + 8 * g % rest : 0) {}
  __device__ __forceinline__ int chunks(int n_act) const { return n_act * full + (rest ? (n_act + quad - 1) / quad : 0); }
};
// Where the next chunk to fetch is: whole chunk f of offset slot (slot < end of its group), else the rests
// of the group that starts at base.
struct ChunkWalk {
  int base = 0, slot = 0, f = 0;
  // start(o, n_act, refresh): refresh(slot, channel) for this lane group of the first chunk
  template <typename R>
  __device__ __forceinline__ void seek(const ChunkOrder& o, int n_act, int g, R&& refresh) {
    const int end = base + o.quad < n_act ? base + o.quad : n_act;
    if (o.full == 0) slot = end;
    if (slot < end)
      refresh(slot, 8 * g);
    else if (o.rest)
      refresh(base + o.g_slot, o.g_ch);
  }
  // next chunk: step() within an offset, refresh() otherwise
  template <typename S, typename R>
  __device__ __forceinline__ void advance(const ChunkOrder& o, int n_act, int g, S&& step, R&& refresh) {
    const int end = base + o.quad < n_act ? base + o.quad : n_act;
    if (slot < end) {
      if (++f < o.full) {
        step();
        return;
      }
      f = 0;
      ++slot;
      if (slot == end && !o.rest) base = end;
    } else {
      base = slot = end;
      f = 0;
    }
    seek(o, n_act, g, refresh);
  }
};

}  // namespace ssconv
