// bf16 output-stationary gather -> MFMA GEMM (Sec. 3.2.3, Alg. 1 feature update):
//
//   out[x] = sum_s kappa(s) in[nbr[s][x]]   for the 64 MR output rows x of a tile
//
// The reduction runs over the offsets present in the tile and their input channels, in chunks of 32
// (one v_mfma_f32_16x16x32_bf16 step each): an offset's whole chunks first, then the rests of 8 or 16
// channels of four or two offsets in one chunk (a rest of 24 is padded).
//
// Layout and data movement (gfx950), chosen from measurement:
//   * eight wavefronts, two per SIMD: row group wm = w % 4 (MR 16-row blocks) x column group wn = w / 4
//     (ceil(NB/2) or floor(NB/2) 16-column blocks); the two wavefronts of a SIMD cover
//     complementary column groups, so with an odd block count the SIMD still does exactly the
//     tile's MFMA work, and one wavefront issues MFMAs while the other is stalled on issue;
//   * both operands reach LDS by DMA (16 bytes per lane, written at M0 + 16 * lane): gathered
//     rows with buffer DMA on 32-bit row offsets (an absent neighbour gets an offset past the
//     end of the buffer, which the hardware fills with zeros), kappa from a packed copy
//     Bp[K][k / 8][cb16][8] so that a 16-column block of one chunk is four contiguous 256-byte
//     runs; no operand is loaded into registers asynchronously;
//   * four LDS stages: iteration c waits for its own DMAs of chunk c+1, publishes them with one
//     barrier, then runs the MFMAs of chunk c with the LDS fragment reads of chunk c+1 and the
//     DMAs of chunk c+3 spread between the column blocks (issuing them in a burst stalls
//     the wavefront for the texture path's whole backlog);
//   * rows whose channels are not a multiple of 8 are copied once, padded with zeros to a multiple
//     of 32 (64-byte pieces), so that every channel count takes this path;
//   * offsets are taken in panels whose row table fits the LDS, so that every kernel size does;
//   * tiles are mapped XCD-contiguously (workgroups are dispatched round-robin over the 8 XCDs;
//     neighbouring tiles gather the same input rows and share that XCD's L2).
#include <algorithm>

#include "gather_mfma.hpp"
#include "gather_tile.hpp"
#include "norm.hpp"

namespace ssconv {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kD = 4;  // pipeline depth: LDS stages (gathered rows + kappa of one chunk)

template <int NB, int MR>
struct GB {
  static constexpr int BM = 64 * MR, BN = 16 * NB;
  static constexpr int WN0 = (NB + 1) / 2, WN1 = NB - WN0;  // column blocks of the two column groups
  static constexpr int ABYTES = 4 * MR * 1024;              // gathered rows of one chunk (16-row blocks)
  static constexpr int STAGE = ABYTES + NB * 1024;          // + kappa blocks
  static constexpr int LA = (4 * MR + 7) / 8, LB = (NB + 7) / 8, L = LA + LB;  // DMAs per wavefront per chunk
  static constexpr int NRB = MR == 4 ? 2 : 1;               // row blocks a wavefront fetches
  static constexpr int PITCH = WN0 * 32 + 16;               // bytes per staged output row in the epilogue
  static constexpr int ROOM = kTileLds - kD * STAGE - kTileMisc;  // for the tables of a panel of offsets
};

// The wavefronts of column group wn (WNX blocks from block noff of the tile on).  Each group has its own
// copy of the tile loop: merged behind the chunk loop, the groups' accumulators cost 20 copies a chunk or
// spills.  The barriers are the same in both.
template <int NB, int MR, int WNX>
__device__ __forceinline__ void gather_bf16_body(const uint16_t* __restrict__ src, int64_t src_bytes,
                                                 int row_bytes, int ca, const uint16_t* __restrict__ Bp, int cb,
                                                 const int32_t* __restrict__ nbr, int64_t n_pos, int K, const TilePlan& plan,
                                                 float* __restrict__ part, uint16_t* __restrict__ out, int noff) {
  using G = GB<NB, MR>;
  constexpr int BM = G::BM, L = G::L, LA = G::LA, NRB = G::NRB;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* stages = smem;                                           // kD * STAGE bytes
  char* junk = smem + kD * G::STAGE;                             // 1 KB sink
  uint32_t* bmask = reinterpret_cast<uint32_t*>(junk + 1024);    // [kTileMaxK]
  uint8_t* act = reinterpret_cast<uint8_t*>(bmask + kTileMaxK);  // [kTileMaxK]
  int* n_act_p = reinterpret_cast<int*>(act + kTileMaxK);        // [4]
  uint32_t* rows = reinterpret_cast<uint32_t*>(n_act_p + 4);     // [panel + 1][BM] byte offsets of gathered rows
  uint2* const tab = reinterpret_cast<uint2*>(rows + (plan.panel + 1) * BM);  // chunk table

  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront index, scalar
  const int wm = w & 3;  // row group
  const int wg = xcd_slot(blockIdx.x, plan.G);
  const int64_t u_beg = wg * plan.units / plan.G, u_end = (wg + 1) * plan.units / plan.G;
  const int cap = pad_k(ca), cg = cap / 8, cbp = pad16(cb);
  const uint32_t stage0 = lds_addr(stages), junk_a = lds_addr(junk);
  const ChunkOrder order(cap);
  // DMA duty per chunk: row blocks w, w + 8 and kappa blocks w, w + 8; a wavefront without one fetches an
  // absent row into the junk block, so that all have the same number in flight
  const uint32_t* const my_rows = rows + 16 * (MR == 1 ? wm : w) + r16;
  uint32_t bmask_w[G::LB];
#pragma unroll
  for (int j = 0; j < G::LB; ++j) bmask_w[j] = w + 8 * j < NB ? ~0u : 0u;

  // Gathered rows are fetched with buffer DMA (32-bit offsets; an offset past the end of src
  // writes zeros, which covers absent neighbours).
  const __amdgpu_buffer_rsrc_t src_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(src), (short)0, (int)src_bytes, kRawBufferWord3);

  for (int64_t u = u_beg; u < u_end;) {
    const int64_t t = u / K;
    const int sa = (int)(u - t * K), sb = (int)(u_end - t * K < K ? u_end - t * K : K);
    const int64_t p0 = plan.row0 + (t / plan.nt) * BM;
    const int n0 = (int)(t % plan.nt) * G::BN;

    f4 acc[MR][WNX];
#pragma unroll
    for (int mb = 0; mb < MR; ++mb)
#pragma unroll
      for (int nb = 0; nb < WNX; ++nb) acc[mb][nb] = f4{0.f, 0.f, 0.f, 0.f};

    const int npan = (sb - sa + plan.panel - 1) / plan.panel;  // panels of near-equal numbers of offsets
    for (int pn = 0; pn < npan; ++pn) {
      const int s0 = sa + (sb - sa) * pn / npan, ns = sa + (sb - sa) * (pn + 1) / npan - s0;
      const int n_act = load_panel<BM>(nbr, n_pos, p0, s0, ns, (uint32_t)row_bytes, rows, bmask, act, n_act_p);
      const int nchunk = order.chunks(n_act);
      if (nchunk == 0) continue;
      chunk_table(order, n_act, nchunk, act, ns, BM * 4, s0, pad8(ca), cg, (uint32_t)cbp * 16u, tab);

      // position of the chunk being fetched (rows, kappa) and the table entry of the one after it
      uint32_t arow[NRB], bpos;
      uint2 ent = tab[g];
      const uint2* next = tab + g;
      const uint32_t col = (uint32_t)(n0 + r16) * 16u;
      auto advance = [&]() {
#pragma unroll
        for (int q = 0; q < NRB; ++q)
          arow[q] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(my_rows + 128 * q) + (ent.x & 0x3ffffu)) +
                    (ent.x >> 18) * 16u;
        bpos = ent.y + col;
        next += 4;
        ent = *next;
      };
      // DMA q of this wavefront for the chunk going into the stage at LDS address sbase
      auto dma = [&](int q, uint32_t sbase) {
        if (q < LA) {
          dma16_tile(src_rsrc, MR == 1 && w >= 4 ? kAbsentRow32 : arow[NRB == 2 ? q & 1 : 0],
                     MR == 1 && w >= 4 ? junk_a : sbase + (w + 8 * q) * 1024);
        } else {
          const int j = q - LA;
          dma16_off(Bp, (bpos + (uint32_t)(w + 8 * j) * 256u) & bmask_w[j],
                    w + 8 * j < NB ? sbase + G::ABYTES + (w + 8 * j) * 1024 : junk_a);
        }
      };
      advance();
      wait_vm<0>();  // the waits below count this panel's DMAs alone
#pragma unroll
      for (int c = 0; c < kD - 1; ++c) {
#pragma unroll
        for (int q = 0; q < L; ++q) dma(q, stage0 + c * G::STAGE);
        advance();
      }

#define SSB_FRAG(da_, db_, u_, sb_)                                                                 \
  do {                                                                                              \
    if ((u_) < MR)                                                                                  \
      da_[(u_) % MR] = *reinterpret_cast<const uint4*>((sb_) + (MR * wm + (u_)) * 1024 + 16 * lane); \
    else                                                                                            \
      db_[(u_) - MR] = *reinterpret_cast<const uint4*>((sb_) + G::ABYTES + (noff + (u_) - MR) * 1024 + 16 * lane); \
  } while (0)

  // Iteration c (stage k = c % kD): wait for this wavefront's DMA of chunk c+1, publish it with a
  // barrier (which also retires every LDS read of the stage refilled next: it was consumed by the
  // MFMAs two chunks ago), then the MFMAs of chunk c with the fragment reads of chunk c+1 and the DMAs of
  // chunk c+kD-1 spread between the column blocks, so that the texture path drains while the matrix
  // cores run.  Past the last chunk the fetches are of absent rows: no conditions in the loop.
#define SSB_BODY(k_, AC, BC, AN, BN_)                                                               \
  {                                                                                                 \
    if (c + (k_) >= nchunk) break;                                                                  \
    wait_vm<(kD - 3) * L>();                                                                        \
    asm volatile("s_barrier" ::: "memory");                                                         \
    const uint32_t si_ = stage0 + ((k_) + kD - 1) % kD * G::STAGE;                                  \
    const char* sbr_ = stages + (((k_) + 1) % kD) * G::STAGE;                                       \
    constexpr int NR = MR + WNX, RPB = (NR + WNX - 1) / WNX, DPB = (L + WNX - 1) / WNX;             \
    __builtin_amdgcn_sched_barrier(0);                                                              \
    _Pragma("unroll") for (int nb = 0; nb < WNX; ++nb) {                                            \
      _Pragma("unroll") for (int mb = 0; mb < MR; ++mb)                                             \
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, AC[mb]),   \
                                                              __builtin_bit_cast(bf16x8, BC[nb]), acc[mb][nb], 0, 0, 0); \
      __builtin_amdgcn_sched_barrier(0);                                                            \
      _Pragma("unroll") for (int u = RPB * nb; u < (RPB * nb + RPB < NR ? RPB * nb + RPB : NR); ++u) \
        SSB_FRAG(AN, BN_, u, sbr_);                                                                 \
      _Pragma("unroll") for (int q = DPB * nb; q < (DPB * nb + DPB < L ? DPB * nb + DPB : L); ++q)  \
        dma(q, si_);                                                                                \
      if (nb == (L + DPB - 1) / DPB - 1) advance();                                                 \
      __builtin_amdgcn_sched_barrier(0);                                                            \
    }                                                                                               \
  }

      static_assert(kD == 4, "the unrolled chunk loop is written for four stages");
      uint4 fa0[MR], fb0[WNX], fa1[MR], fb1[WNX];
      wait_vm<2 * L>();
      asm volatile("s_barrier" ::: "memory");
#pragma unroll
      for (int u = 0; u < MR + WNX; ++u) SSB_FRAG(fa0, fb0, u, stages);
      for (int c = 0;; c += kD) {  // four chunks per trip; the first body past the last chunk leaves the loop
        SSB_BODY(0, fa0, fb0, fa1, fb1)
        SSB_BODY(1, fa1, fb1, fa0, fb0)
        SSB_BODY(2, fa0, fb0, fa1, fb1)
        SSB_BODY(3, fa1, fb1, fa0, fb0)
      }
      wait_vm<0>();  // the fetches past the end land before the stages are used again
#undef SSB_BODY
#undef SSB_FRAG
    }

    int el = lane;
    asm volatile("" : "+v"(el));  // opaque: the address arithmetic below must not live through the chunk loop
    const int eg = el >> 4, er = el & 15;
    const int c0 = 16 * noff;
    if (sa == 0 && sb == K) {
      // Whole tile: each wavefront stages its rows, up to 32 at a time, as bf16 in LDS (row pitch padded
      // so the 2-byte writes of the four row groups fall in distinct banks) and writes them back as
      // 16-byte pieces of its column range of the output rows.
      constexpr int RP = MR < 2 ? 1 : 2;  // row blocks staged at a time
      static_assert(kTileThreads / 64 * 16 * RP * G::PITCH <= kD * G::STAGE, "epilogue staging must fit the stage area");
      __syncthreads();  // every wavefront is done with the stage area
      char* const ep = stages + w * 16 * RP * G::PITCH;
      const bool vec = (cb & 7) == 0;
#pragma unroll
      for (int part_ = 0; part_ < MR / RP; ++part_) {
#pragma unroll
        for (int m2 = 0; m2 < RP; ++m2)
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int nb = 0; nb < WNX; ++nb)
              *reinterpret_cast<uint16_t*>(ep + (16 * m2 + 4 * eg + i) * G::PITCH + (16 * nb + er) * 2) =
                  f32_to_bf16_rne(acc[RP * part_ + m2][nb][i]);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        constexpr int pieces = 2 * WNX;  // 16-byte pieces per staged row
        for (int e = el; e < 16 * RP * pieces; e += 64) {
          const int r = e / pieces, q = e - r * pieces;
          const int64_t p = p0 + 16 * MR * wm + 16 * RP * part_ + r;
          const int col = n0 + c0 + 8 * q;
          if (p >= n_pos || col >= cb) continue;
          uint16_t* dst = out + p * cb + col;
          const char* srcp = ep + r * G::PITCH + q * 16;
          if (vec) {
            *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(srcp);
          } else {
            const int n = cb - col < 8 ? cb - col : 8;
            for (int j = 0; j < n; ++j) dst[j] = reinterpret_cast<const uint16_t*>(srcp)[j];
          }
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    } else {
      float* dst = part + (int64_t)(2 * wg + (u == u_beg ? 0 : 1)) * BM * G::BN;
#pragma unroll
      for (int mb = 0; mb < MR; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int nb = 0; nb < WNX; ++nb)
            dst[(16 * (wm * MR + mb) + 4 * eg + i) * G::BN + c0 + 16 * nb + er] = acc[mb][nb][i];
    }
    u = t * K + sb;
  }
}

// Pieces of tiles that more than one workgroup holds go to part (fp32, slot 2 i: the first tile of
// workgroup i, 2 i + 1: its last) and are added in order by bf16_fixup; whole tiles go to out.
template <int NB, int MR>
__global__ __launch_bounds__(kTileThreads) void gather_bf16_kernel(const uint16_t* __restrict__ src, int64_t src_bytes,
                                                                   int row_bytes, int ca,
                                                                   const uint16_t* __restrict__ Bp, int cb,
                                                                   const int32_t* __restrict__ nbr, int64_t n_pos, int K,
                                                                   TilePlan plan, float* __restrict__ part,
                                                                   uint16_t* __restrict__ out) {
  using G = GB<NB, MR>;
  const int wn = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);  // SIMD w % 4 hosts both column groups
  if (wn == 0)
    gather_bf16_body<NB, MR, G::WN0>(src, src_bytes, row_bytes, ca, Bp, cb, nbr, n_pos, K, plan, part, out, 0);
  else
    gather_bf16_body<NB, MR, G::WN1>(src, src_bytes, row_bytes, ca, Bp, cb, nbr, n_pos, K, plan, part, out, G::WN0);
}

// Adds the pieces of the tiles that more than one workgroup held, in workgroup order.  A block takes
// 1024 consecutive values of one tile.
__global__ __launch_bounds__(256) void bf16_fixup(const float* __restrict__ part, TilePlan plan, int K, int BM, int BN,
                                                  int cb, int64_t n_pos, uint16_t* __restrict__ out) {
  const int64_t t = blockIdx.x;
  const int64_t i0 = unit_owner(plan, t * K), i1 = unit_owner(plan, t * K + K - 1);
  if (i0 == i1) return;
  const int e = (blockIdx.y * 256 + threadIdx.x) * 4, r = e / BN, c = e - r * BN;
  const int64_t p = plan.row0 + (t / plan.nt) * BM + r;
  const int col = (int)(t % plan.nt) * BN + c;
  if (r >= BM || p >= n_pos || col >= cb) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t i = i0; i <= i1; ++i) {
    const int64_t slot = 2 * i + (i * plan.units / plan.G / K == t ? 0 : 1);
    const float4 x = *reinterpret_cast<const float4*>(part + slot * BM * BN + e);
    v[0] += x.x, v[1] += x.y, v[2] += x.z, v[3] += x.w;
  }
  uint16_t* o = out + p * cb + col;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (col + k < cb) o[k] = f32_to_bf16_rne(v[k]);
}

// Thread i copies 8 channels of one row of [n][ca] to [n][pad32(ca)], zeros past ca.
__device__ __forceinline__ void pad_row(const uint16_t* __restrict__ src, int64_t n, int ca, int64_t i,
                                        uint16_t* __restrict__ Ap) {
  const int per = pad32(ca) / 8;
  if (i >= n * per) return;
  const int64_t r = i / per;
  const int k0 = (int)(i - r * per) * 8;
  uint16_t e[8];
  uint4 v;
#pragma unroll
  for (int j = 0; j < 8; ++j) e[j] = k0 + j < ca ? src[r * ca + k0 + j] : (uint16_t)0;
  __builtin_memcpy(&v, e, 16);
  *reinterpret_cast<uint4*>(Ap + i * 8) = v;
}

// Rows of two sources in one launch.
__global__ __launch_bounds__(256) void pad_rows_kernel(const uint16_t* __restrict__ x, int64_t nx, int cx, unsigned x_blocks,
                                                       uint16_t* __restrict__ xp, const uint16_t* __restrict__ y, int64_t ny,
                                                       int cy, uint16_t* __restrict__ yp) {
  if (blockIdx.x < x_blocks)
    pad_row(x, nx, cx, (int64_t)blockIdx.x * 256 + threadIdx.x, xp);
  else
    pad_row(y, ny, cy, (int64_t)(blockIdx.x - x_blocks) * 256 + threadIdx.x, yp);
}

// One launch for both operands.  Blocks below row_blocks pad the rows (row_blocks = 0: they are read in
// place).  The others: Bp[s][k / 8][n][k % 8] (pad_k(ca) / 8 groups of pad16(cb) columns, zeros past the
// ends) from kappa given as Bt[s'][n][k] (transposed = 0) or as W[s'][k][n] (transposed = 1), s' = s or
// K-1-s (mirror), a thread per 16 bytes.
__global__ __launch_bounds__(256) void pack_operands(const uint16_t* __restrict__ src, int64_t n_src, int ca,
                                                     unsigned row_blocks, const uint16_t* __restrict__ W, int K, int cb,
                                                     int transposed, int mirror, uint16_t* __restrict__ Ap,
                                                     uint16_t* __restrict__ Bp) {
  if (blockIdx.x < row_blocks) {
    pad_row(src, n_src, ca, (int64_t)blockIdx.x * 256 + threadIdx.x, Ap);
    return;
  }
  uint16_t e[8];
  uint4 v;
  const int cg = pad_k(ca) / 8, cbp = pad16(cb);
  const int64_t i = (int64_t)(blockIdx.x - row_blocks) * 256 + threadIdx.x;
  if (i >= (int64_t)K * cg * cbp) return;
  const int n = (int)(i % cbp), kg = (int)((i / cbp) % cg), k0 = 8 * kg;
  const int64_t s = i / ((int64_t)cbp * cg), sw = mirror ? K - 1 - s : s;
  if (!transposed && (ca & 7) == 0 && n < cb && k0 < ca) {
    v = *reinterpret_cast<const uint4*>(W + (sw * cb + n) * ca + k0);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      e[j] = n < cb && k0 + j < ca ? W[transposed ? (sw * ca + k0 + j) * cb + n : (sw * cb + n) * ca + k0 + j]
                                   : (uint16_t)0;
    __builtin_memcpy(&v, e, 16);
  }
  *reinterpret_cast<uint4*>(Bp + i * 8) = v;
}

// The launches of a call: plan[0], and plan[1] for the rows a last round of tall tiles would leave most
// compute units idle on (n = 1: none).
struct Bf16Shape {
  int nb, n, mr[2];
  TilePlan plan[2];
};

size_t ap_bytes(int64_t n_src, int ca) { return ca % 8 == 0 ? 0 : align256((size_t)n_src * pad32(ca) * 2); }
// (the column blocks of the last tile past cb16 read on past the end: up to 4 KB)
size_t bp_bytes(int ca, int cb, int K) { return align256((size_t)K * pad_k(ca) * pad16(cb) * 2 + 4096); }
size_t part_bytes(const TilePlan& p, int mr, int nb, int K) {
  return whole_tiles(p, K) ? 0 : align256((size_t)2 * p.G * 64 * mr * 16 * nb * 4);
}
size_t shape_bytes(const Bf16Shape& s, int64_t n_src, int ca, int cb, int K) {
  size_t part = 0;
  for (int i = 0; i < s.n; ++i) part = std::max(part, part_bytes(s.plan[i], s.mr[i], s.nb, K));
  return ap_bytes(n_src, ca) + bp_bytes(ca, cb, K) + part;
}

// A 32-channel chunk of an MR x NB tile takes about 0.15 + 0.012 MR NB us (measured 0.77 at 4 x 13).
double chunk_us(int mr, int nb) { return 0.15 + 0.012 * mr * nb; }

// The cheapest of whole and cut tiles of each height for rows row0 .. n_pos - 1 (a cut costs the pieces'
// traffic and one more launch); plans whose pieces fit `room` bytes come first.
TilePlan best_plan(int64_t row0, int64_t n_pos, int nt, int nb, int K, double chunks, size_t room, int* mr, double* cost) {
  TilePlan best{}, p;
  bool best_fits = false;
  for (int i = 0; i < 3 * (1 + kCutChoices); ++i) {
    const int m = 4 >> (i / (1 + kCutChoices)), cut = i % (1 + kCutChoices);
    p.row0 = row0;
    p.mt = (int)cdiv(n_pos - row0, 64 * m);
    p.nt = nt;
    const int64_t tiles = (int64_t)p.mt * nt;
    p.units = tiles * K;
    double c = chunks * chunk_us(m, nb);
    if (cut) {
      p.G = (int)std::min<int64_t>(kTileWG >> (cut - 1), p.units);
      c = c * tiles / p.G + cut_us(p.G, tiles) + (double)part_bytes(p, m, nb, K) / 4e6;
    } else {
      p.G = (int)tiles;
      c *= cdiv(tiles, kTileWG);
    }
    const bool fits = part_bytes(p, m, nb, K) <= room;
    if (i == 0 || (fits && !best_fits) || (fits == best_fits && c < *cost))
      best = p, best_fits = fits, *cost = c, *mr = m;
  }
  return best;
}

// Column blocks per tile: the instantiated width that covers cb in the fewest, most even tiles.
int bf16_nb(int cb) {
  const int blocks = (cb + 15) / 16, tiles = (blocks + 13) / 14, per = (blocks + tiles - 1) / tiles;
  return per <= 2 ? 2 : per <= 4 ? 4 : per <= 7 ? 7 : per <= 8 ? 8 : per <= 13 ? 13 : 14;
}

Bf16Shape bf16_shape(int64_t n_src, int ca, int cb, int64_t n_pos, int K) {
  Bf16Shape s, two;
  s.nb = two.nb = bf16_nb(cb);
  const int nt = (int)cdiv(cb, 16 * s.nb);
  const double chunks = pad_k(ca) / 32.0 * K;
  const size_t used = ap_bytes(n_src, ca) + bp_bytes(ca, cb, K);
  const size_t room = used < SSCONV_NOALLOC_SCRATCH_BYTES ? SSCONV_NOALLOC_SCRATCH_BYTES - used : 0;
  double cost, tail;
  s.n = 1;
  s.plan[0] = best_plan(0, n_pos, nt, s.nb, K, chunks, room, &s.mr[0], &cost);
  // full rounds of 256-row tiles, then the other rows by a plan of their own (about 6 us for the launch)
  const int64_t rounds = n_pos / 256 * nt / kTileWG, mt = rounds * kTileWG / nt;
  if (mt == 0 || mt * 256 >= n_pos) return s;
  two.n = 2;
  two.mr[0] = 4;
  two.plan[0] = {(int)(mt * nt), (int)mt, nt, 0, 0, mt * nt * K};
  two.plan[1] = best_plan(mt * 256, n_pos, nt, s.nb, K, chunks, room, &two.mr[1], &tail);
  return rounds * chunks * chunk_us(4, s.nb) + tail + 6.0 < cost ? two : s;
}

template <int NB, int MR>
int launch_bf16(TilePlan plan, const void* src, int64_t src_bytes, int row_bytes, int ca, const void* Bp, int cb,
                const int32_t* nbr, int64_t n_pos, int K, float* part, void* out, hipStream_t st) {
  using G = GB<NB, MR>;
  plan.panel = panel_offsets(G::ROOM, G::BM, pad_k(ca), K);
  const size_t smem = (size_t)(kTileLds - G::ROOM) + panel_bytes(plan.panel, G::BM, pad_k(ca));
  auto kern = gather_bf16_kernel<NB, MR>;
  SSC_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  kern<<<plan.G, kTileThreads, smem, st>>>((const uint16_t*)src, src_bytes, row_bytes, ca, (const uint16_t*)Bp, cb, nbr,
                                           n_pos, K, plan, part, (uint16_t*)out);
  if (!whole_tiles(plan, K)) {
    const int BM = 64 * MR, BN = 16 * NB;
    bf16_fixup<<<dim3((unsigned)(plan.mt * plan.nt), cdiv(BM * BN, 1024)), 256, 0, st>>>(part, plan, K, BM, BN, cb, n_pos,
                                                                                         (uint16_t*)out);
  }
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

}  // namespace

int pad_rows_bf16(const uint16_t* x, int64_t nx, int cx, uint16_t* xp, const uint16_t* y, int64_t ny, int cy, uint16_t* yp,
                  hipStream_t st) {
  const unsigned xb = cdiv(nx * (pad32(cx) / 8), 256), yb = cdiv(ny * (pad32(cy) / 8), 256);
  if (xb + yb == 0) return SSCONV_OK;
  pad_rows_kernel<<<xb + yb, 256, 0, st>>>(x, nx, cx, xb, xp, y, ny, cy, yp);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

bool gather_bf16_supported(int64_t n_src, int ca, int cb, int K) {
  // 32-bit byte offsets: every gathered row and every packed kappa entry below 2^31
  // and a panel of at least two offsets
  return ca >= 1 && ca <= 8192 && cb >= 1 && K >= 1 && K <= kTileMaxK && n_src >= 0 &&
         n_src * (ca % 8 == 0 ? ca : pad32(ca)) * 2 < ((int64_t)1 << 31) && bp_bytes(ca, cb, K) < ((size_t)1 << 31);
}

size_t gather_bf16_bytes(int64_t n_src, int ca, int cb, int64_t n_pos, int K) {
  return shape_bytes(bf16_shape(n_src, ca, cb, n_pos, K), n_src, ca, cb, K);
}

int gather_bf16(const void* src, int64_t n_src, int ca, const void* W, bool transposed, bool mirror, int cb,
                const int32_t* nbr, int64_t n_pos, int K, void* out, hipStream_t st, CallScratch* sc,
                const uint16_t* padded) {
  if (n_pos == 0) return SSCONV_OK;
  const Bf16Shape s = bf16_shape(n_src, ca, cb, n_pos, K);
  char* ws = nullptr;
  const bool pad = ca % 8 != 0 && !padded;
  const size_t ap = pad ? ap_bytes(n_src, ca) : 0;
  SSC_TRY(scratch_take(sc, (void**)&ws, shape_bytes(s, n_src, ca, cb, K) - ap_bytes(n_src, ca) + ap, st));
  uint16_t* Ap = (uint16_t*)ws;
  uint16_t* Bp = (uint16_t*)(ws + ap);
  float* part = (float*)(ws + ap + bp_bytes(ca, cb, K));
  const unsigned row_blocks = pad ? cdiv(n_src * (pad32(ca) / 8), 256) : 0;
  const unsigned b_blocks = cdiv((int64_t)K * (pad_k(ca) / 8) * pad16(cb), 256);
  pack_operands<<<row_blocks + b_blocks, 256, 0, st>>>((const uint16_t*)src, n_src, ca, row_blocks, (const uint16_t*)W, K,
                                                       cb, transposed ? 1 : 0, mirror ? 1 : 0, Ap, Bp);
  int rc = hipGetLastError() == hipSuccess ? SSCONV_OK : fail(SSCONV_E_HIP, "operand packing launch failed");
  const void* A = padded ? (const void*)padded : pad ? (const void*)Ap : src;
  const int row_bytes = 2 * (padded || pad ? pad32(ca) : ca);
  for (int i = 0; i < s.n && rc == SSCONV_OK; ++i) {
#define SSB_GO(NB_, MR_) \
  rc = launch_bf16<NB_, MR_>(s.plan[i], A, n_src * row_bytes, row_bytes, ca, Bp, cb, nbr, n_pos, K, part, out, st)
#define SSB_NB(NB_)                      \
  if (s.mr[i] == 4) SSB_GO(NB_, 4);      \
  else if (s.mr[i] == 2) SSB_GO(NB_, 2); \
  else SSB_GO(NB_, 1);                   \
  break
    switch (s.nb) {
      case 2: SSB_NB(2);
      case 4: SSB_NB(4);
      case 7: SSB_NB(7);
      case 8: SSB_NB(8);
      case 13: SSB_NB(13);
      default: SSB_NB(14);
    }
#undef SSB_NB
#undef SSB_GO
  }
  scratch_give(sc, ws, st);
  return rc;
}

}  // namespace ssconv
