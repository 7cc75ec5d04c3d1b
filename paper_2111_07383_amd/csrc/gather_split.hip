// fp32 output-stationary gather -> MFMA GEMM on the bf16 matrix cores (Sec. 3.2.3, Alg. 1):
//
//   out[x] = sum_s kappa(s) in[nbr[s][x]]
//
// Every fp32 value is the sum of three bf16 values (a0 = bf16(a), a1 = bf16(a - a0), a2 = the rest:
// 24 bits, exact), so a product of two is six bf16 products -- a2 b0, a1 b1, a0 b2, a1 b0, a0 b1 and
// a0 b0, summed in fp32 -- and three dropped ones below 2^-26 of it.  Six bf16 products cost 0.375 of
// one fp32 MFMA product's matrix-core time.  The five small terms of a chunk are summed by
// themselves and join the large sum once, so that the latter is rounded twice a chunk instead of six
// times: errors against fp64 came out 0.3 - 0.8 of those of v_mfma_f32_16x16x4f32 on every layer tried.
// The scheme is that of Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial intelligence datatype
// for higher-precision computations" (2019).  For what three parts cannot carry see split_guard.hpp.
//
// Bound: the matrix cores (63% busy) and the texture path that feeds the LDS (63 KB of DMA per
// 256 x 112 x 32 chunk, 2.0 GB of a launch from past the L2 at 5 TB/s).  Two workgroup-wide stages of 69 KB fill
// the LDS; tall tiles because LDS reads per product fall with the tile (256 rows: 93 bytes a clock of 128).
// Measured on a 36 555-site 5x5x5 layer, 104 -> 104: 1100 us (fp32 MFMA, 286 tiles on 256 compute units) -> 445,
// 411 of them this kernel.  On the way: chunks that straddle two 64-byte parts 544 us against 496 aligned; DMAs
// issued in one burst 568 against 534 spread out; kappa and rows always from L2 (a probe) 510 against 544, so
// memory is not what bounds it.
#include <algorithm>

#include "conv.hpp"
#include "gather_split.hpp"
#include "gather_tile.hpp"

namespace ssconv {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Split rows: [row][ceil(ca / 32)][3 parts][32 channels] bf16, zero past ca; 192 bytes per 32 channels.
__host__ __device__ __forceinline__ int chunks32(int ca) { return (ca + 31) / 32; }
// The parts of x; returns whether they are not all of it (an infinity or NaN leaves NaN behind).
__device__ __forceinline__ bool split3(float x, uint16_t* p) {
  p[0] = f32_to_bf16_rne(x);
  const float r1 = x - bf16_to_f32(p[0]);
  p[1] = f32_to_bf16_rne(r1);
  const float r2 = r1 - bf16_to_f32(p[1]);
  p[2] = f32_to_bf16_rne(r2);
  return !(r2 == bf16_to_f32(p[2]));
}

__device__ __forceinline__ void store_parts(const uint16_t (*e)[3], uint16_t* dst, int64_t step) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    uint16_t t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = e[j][p];
    uint4 v;
    __builtin_memcpy(&v, t, 16);
    *reinterpret_cast<uint4*>(dst + p * step) = v;
  }
}

// Thread i splits 8 channels of one row.
__device__ __forceinline__ void split_row(const float* __restrict__ src, int64_t n, int ca, int64_t i,
                                          uint16_t* __restrict__ A3, int* __restrict__ flag) {
  const int cc = chunks32(ca), per = 4 * cc;
  if (i >= n * per) return;
  const int64_t r = i / per;
  const int q = (int)(i - r * per), c0 = 8 * q;
  const float* s = src + r * ca + c0;
  float v[8];
  uint16_t e[8][3];
  if ((ca & 3) == 0 && c0 + 8 <= ca) {
    const float4 a = *reinterpret_cast<const float4*>(s), b = *reinterpret_cast<const float4*>(s + 4);
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = c0 + j < ca ? s[j] : 0.f;
  }
  bool lost = false;
#pragma unroll
  for (int j = 0; j < 8; ++j) lost |= split3(v[j], e[j]);
  if (lost) *flag = 1;
  store_parts(e, A3 + (r * cc + (q >> 2)) * 96 + 8 * (q & 3), 32);
}

// Rows of two sources in one launch.
__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ x, int64_t nx, int cx, unsigned x_blocks,
                                                         uint16_t* __restrict__ x3, int* __restrict__ x_flag,
                                                         const float* __restrict__ y, int64_t ny, int cy,
                                                         uint16_t* __restrict__ y3, int* __restrict__ y_flag) {
  if (blockIdx.x < x_blocks)
    split_row(x, nx, cx, (int64_t)blockIdx.x * 256 + threadIdx.x, x3, x_flag);
  else
    split_row(y, ny, cy, (int64_t)(blockIdx.x - x_blocks) * 256 + threadIdx.x, y3, y_flag);
}

// Both operands in one launch: blocks below row_blocks split the gathered rows, the others kappa into
// B3[s][pad_k(ca) / 8][3 parts][cb16][8] (zeros past the end), a thread one 8-channel run of one column, and
// where Bt is given into Bt[s][n][k] in fp32.
__global__ __launch_bounds__(256) void split_operands(const float* __restrict__ src, int64_t n_src, int ca,
                                                      unsigned row_blocks, SplitKernel B, int K, int cb,
                                                      uint16_t* __restrict__ A3, uint16_t* __restrict__ B3,
                                                      int* __restrict__ rows_flag, int* __restrict__ kappa_flag,
                                                      float* __restrict__ Bt) {
  if (blockIdx.x < row_blocks) {
    split_row(src, n_src, ca, (int64_t)blockIdx.x * 256 + threadIdx.x, A3, rows_flag);
    return;
  }
  uint16_t e[8][3];
  const int cg = pad_k(ca) / 8, cbp = pad16(cb);
  const int64_t i = (int64_t)(blockIdx.x - row_blocks) * 256 + threadIdx.x;
  if (i >= (int64_t)K * cg * cbp) return;
  const int n = (int)(i % cbp);
  const int64_t sc = i / cbp;
  const int k0 = (int)(sc % cg) * 8;
  const int64_t s = sc / cg, sw = B.mirror ? K - 1 - s : s;
  bool lost = false;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float x = 0.f;
    if (n < cb && k0 + j < ca) x = B.transposed ? B.W[(sw * ca + k0 + j) * cb + n] : B.W[(sw * cb + n) * ca + k0 + j];
    lost |= split3(x, e[j]);
    if (Bt && n < cb && k0 + j < ca) Bt[(s * cb + n) * ca + k0 + j] = x;
  }
  if (lost) *kappa_flag = 1;
  store_parts(e, B3 + (sc * 3 * cbp + n) * 8, (int64_t)cbp * 8);
}

// Tile of BM = 64 MR output rows x 16 NB columns.  Row group wm = w % 4 (MR 16-row blocks), column
// group wn = w / 4 (ceil or floor of NB / 2 blocks); the two wavefronts of a SIMD have one of each.
template <int NB, int MR>
struct GS {
  static constexpr int BM = 64 * MR, BN = 16 * NB;
  static constexpr int WN0 = (NB + 1) / 2, WN1 = NB - WN0;
  static constexpr int ABYTES = 4 * MR * 3 * 1024;           // gathered rows of one 32-channel chunk
  static constexpr int STAGE = ABYTES + NB * 3 * 1024;       // + kappa
  static constexpr int S = MR == 4 ? 2 : 3;                  // LDS stages
  static constexpr int LA = (12 * MR + 7) / 8, LB = (3 * NB + 7) / 8, L = LA + LB;  // DMAs per wavefront per chunk
  static constexpr int NRB = MR == 4 ? 2 : 1;                // row blocks a wavefront fetches
  static constexpr int ROOM = kTileLds - S * STAGE - kTileMisc;  // for the tables of a panel of offsets
};

// A tile's first
// piece (mostly the whole tile) is written to out; a workgroup that starts inside a tile leaves that piece
// in part, slot i, and split_fixup adds the pieces in order.
template <int NB, int MR>
__global__ __launch_bounds__(kTileThreads) void gather_split_kernel(const uint16_t* __restrict__ A3, int64_t a_bytes, int ca,
                                                           const uint16_t* __restrict__ B3, int cb,
                                                           const int32_t* __restrict__ nbr, int64_t n_pos, int K,
                                                           TilePlan plan, float* __restrict__ part,
                                                           const int* __restrict__ rows_flag, SplitFlags flags,
                                                           float* __restrict__ out) {
  if (*rows_flag | *flags.kappa()) return;  // set before this kernel: the plain one computes it all
  using G = GS<NB, MR>;
  constexpr int BM = G::BM, S = G::S, NRB = G::NRB;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* stages = smem;
  char* junk = smem + S * G::STAGE;
  uint32_t* bmask = reinterpret_cast<uint32_t*>(junk + 1024);   // [kTileMaxK]
  uint8_t* act = reinterpret_cast<uint8_t*>(bmask + kTileMaxK);     // [kTileMaxK]
  int* n_act_p = reinterpret_cast<int*>(act + kTileMaxK);           // [4]
  uint32_t* rows = reinterpret_cast<uint32_t*>(n_act_p + 4);    // [panel + 1][BM] byte offsets of gathered rows
  uint2* const tab = reinterpret_cast<uint2*>(rows + (plan.panel + 1) * BM);  // chunk table

  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w & 3, wn = w >> 2;
  const int wg = xcd_slot(blockIdx.x, plan.G);
  const int64_t u_beg = wg * plan.units / plan.G, u_end = (wg + 1) * plan.units / plan.G;
  const int cc = chunks32(ca), cap = pad_k(ca), cg = cap / 8, cbp = pad16(cb);
  const uint32_t row_bytes = (uint32_t)cc * 192u;
  const uint32_t stage0 = lds_addr(stages), junk_a = lds_addr(junk);
  const __amdgpu_buffer_rsrc_t a_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(A3), (short)0, (int)a_bytes, kRawBufferWord3);
  const ChunkOrder order(cap);
  const uint32_t* const my_rows = rows + 16 * (MR == 1 ? wm : w) + r16;
  uint32_t boff[G::LB];  // kappa block e = w + 8 j: part e % 3 of column block e / 3
#pragma unroll
  for (int j = 0; j < G::LB; ++j) boff[j] = (uint32_t)((w + 8 * j) % 3 * cbp + (w + 8 * j) / 3 * 16) * 16u;

  for (int64_t u = u_beg; u < u_end;) {
    const int64_t t = u / K;
    const int sa = (int)(u - t * K), sb = (int)(u_end - t * K < K ? u_end - t * K : K);
    const int64_t p0 = plan.row0 + (t / plan.nt) * BM;
    const int n0 = (int)(t % plan.nt) * G::BN;

    f4 acc[MR][G::WN0];
#pragma unroll
    for (int mb = 0; mb < MR; ++mb)
#pragma unroll
      for (int nb = 0; nb < G::WN0; ++nb) acc[mb][nb] = f4{0.f, 0.f, 0.f, 0.f};

    // panels of near-equal numbers of offsets whose row table fits the LDS
    const int npan = (sb - sa + plan.panel - 1) / plan.panel;
    for (int pn = 0; pn < npan; ++pn) {
      const int s0 = sa + (sb - sa) * pn / npan, ns = sa + (sb - sa) * (pn + 1) / npan - s0;
      const int n_act = load_panel<BM>(nbr, n_pos, p0, s0, ns, row_bytes, rows, bmask, act, n_act_p);
      const int nchunk = order.chunks(n_act);
      if (nchunk == 0) continue;
      chunk_table(order, n_act, nchunk, act, ns, BM * 4, s0, pad8(ca), cg, (uint32_t)cbp * 48u, tab);

      // position of the chunk being fetched (rows, kappa) and the table entry of the one after it
      uint32_t arow[NRB], bbase;
      uint2 ent = tab[g];
      const uint2* next = tab + g;
      const uint32_t colb = (uint32_t)(n0 + r16) * 16u;
      auto advance = [&]() {
        const uint32_t c8 = ent.x >> 18;  // channel / 8: its chunk of 192 bytes, 16 bytes within each part
#pragma unroll
        for (int q = 0; q < NRB; ++q)
          arow[q] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(my_rows + 128 * q) + (ent.x & 0x3ffffu)) +
                    (c8 >> 2) * 192u + (c8 & 3u) * 16u;
        bbase = ent.y + colb;
        next += 4;
        ent = *next;
      };
      // DMA q of this wavefront for the chunk going into stage k: q < LA a row block's part, else a
      // part of a kappa block
      auto dma = [&](int q, uint32_t sbase) {
        if (q < G::LA) {
          // row block w + 8 (q % 2) part q / 2 of 16 blocks; block w part q of 8; block w % 4 part w / 4 + 2 q of 4
          const uint32_t row = arow[MR == 4 ? q & 1 : 0];
          if constexpr (MR == 4)
            dma16_tile(a_rsrc, row + (q >> 1) * 64u, sbase + w * 3072 + (q & 1) * 24576 + (q >> 1) * 1024);
          else if constexpr (MR == 2)
            dma16_tile(a_rsrc, row + q * 64u, sbase + w * 3072 + q * 1024);
          else if (q == 0 || w < 4)
            dma16_tile(a_rsrc, row + (wn + 2 * q) * 64u, sbase + wm * 3072 + (wn + 2 * q) * 1024);
          else
            dma16_tile(a_rsrc, kAbsentRow32, junk_a);
        } else {
          const int j = q - G::LA;
          if (8 * j + 8 <= 3 * NB || w < 3 * NB - 8 * j)
            dma16_off(B3, bbase + boff[j], sbase + G::ABYTES + (w + 8 * j) * 1024);
          else if (S > 2)
            dma16_tile(a_rsrc, kAbsentRow32, junk_a);
        }
      };
      advance();
      wait_vm<0>();  // the waits below count this panel's DMAs alone
      for (int c = 0; c < S - 1; ++c) {
#pragma unroll
        for (int q = 0; q < G::L; ++q) dma(q, stage0 + c * G::STAGE);
        advance();
      }

      // iteration c: this wavefront's DMAs of chunk c have landed, one barrier publishes them (and
      //    retires the reads of the stage refilled next); the fragments are read one step ahead of the
      //    MFMAs that use them, the DMAs of chunk c + S - 1 go out between the first steps (past the last
      //    chunk: of absent rows, so that the loop has no conditions)
#define SSG_RDA(d_, mb_)                                                                            \
  _Pragma("unroll") for (int p = 0; p < 3; ++p)                                                     \
    d_[p] = *reinterpret_cast<const uint4*>(sb_ + ((wm * MR + (mb_)) * 3 + p) * 1024 + 16 * lane)
#define SSG_RDB(nb_)                                                                                \
  _Pragma("unroll") for (int p = 0; p < 3; ++p)                                                     \
    fb[nb_][p] = *reinterpret_cast<const uint4*>(sb_ + G::ABYTES + ((NOFF + (nb_)) * 3 + p) * 1024 + 16 * lane)
#define SSG_LOOP(WNX_, NOFF_)                                                                       \
  {                                                                                                 \
    constexpr int WNX = WNX_;                                                                       \
    const int NOFF = NOFF_;                                                                         \
    constexpr int NP = WNX < 2 ? 1 : WNX / 2;   /* steps per row block: two columns, the last three if odd */ \
    constexpr int NS = 2 * MR * NP;             /* places for DMAs: two per step */                 \
    int k_ = 0, ki_ = S - 1;                                                                        \
    for (int c = 0; c < nchunk; ++c) {                                                              \
      wait_vm<(S - 2) * G::L>();                                                                    \
      asm volatile("s_barrier" ::: "memory");                                                       \
      const char* sb_ = stages + k_ * G::STAGE;                                                     \
      const uint32_t si_ = stage0 + ki_ * G::STAGE;                                                 \
      uint4 fa[2][3], fb[WNX][3];                                                                   \
      constexpr int W0 = NP == 1 ? WNX : 2;                                                         \
      f4 low_[2][WNX - 2 * NP + 2];                                                                 \
      /* in the order the products need them: the first may start after two reads */                \
      _Pragma("unroll") for (int p = 0; p < 3; ++p) {                                               \
        fa[0][2 - p] = *reinterpret_cast<const uint4*>(sb_ + (wm * MR * 3 + 2 - p) * 1024 + 16 * lane); \
        _Pragma("unroll") for (int h = 0; h < W0; ++h)                                              \
          fb[h][p] = *reinterpret_cast<const uint4*>(sb_ + G::ABYTES + ((NOFF + h) * 3 + p) * 1024 + 16 * lane); \
      }                                                                                             \
      __builtin_amdgcn_sched_barrier(0);                                                            \
      _Pragma("unroll") for (int mb = 0; mb < MR; ++mb) {                                           \
        _Pragma("unroll") for (int np = 0; np < NP; ++np) {                                         \
          const int n1 = np == NP - 1 ? WNX : 2 * np + 2;                                           \
          if (mb == 0 && np + 1 < NP) {                                                             \
            _Pragma("unroll") for (int nb = n1; nb < (np + 2 == NP ? WNX : n1 + 2); ++nb) { SSG_RDB(nb % WNX); } \
          }                                                                                         \
          if (np == NP - 1 && mb + 1 < MR) { SSG_RDA(fa[(mb + 1) & 1], mb + 1); }                   \
          _Pragma("unroll") for (int th = 0; th < 2; ++th) {                                        \
            const int place = (mb * NP + np) * 2 + th;                                              \
            _Pragma("unroll") for (int q = place * G::L / NS; q < (place + 1) * G::L / NS; ++q)     \
              dma(q, si_);                                                                          \
            /* the step before: its small terms, long done, join the sum */                         \
            if (th == 1 && mb * NP + np > 0) {                                                      \
              const int pmb = np > 0 ? mb : mb - 1, pnp = np > 0 ? np - 1 : NP - 1;                 \
              _Pragma("unroll") for (int nb = 2 * pnp; nb < (pnp == NP - 1 ? WNX : 2 * pnp + 2); ++nb) \
                acc[pmb][nb] += low_[(pmb * NP + pnp) & 1][nb - 2 * pnp];                           \
            }                                                                                       \
            __builtin_amdgcn_sched_barrier(0);                                                      \
            _Pragma("unroll") for (int term = 3 * th; term < 3 * th + 3; ++term) {                  \
              constexpr int qa_[6] = {2, 1, 0, 1, 0, 0}, qb_[6] = {0, 1, 2, 0, 1, 0};               \
              _Pragma("unroll") for (int nb = 2 * np; nb < n1; ++nb) {                              \
                f4& lo = low_[(mb * NP + np) & 1][nb - 2 * np];                                     \
                if (term == 0) lo = f4{0.f, 0.f, 0.f, 0.f};                                         \
                f4& to = term == 5 ? acc[mb][nb] : lo;                                              \
                to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(                                       \
                    __builtin_bit_cast(bf16x8, fa[mb & 1][qa_[term]]),                              \
                    __builtin_bit_cast(bf16x8, fb[nb][qb_[term]]), to, 0, 0, 0);                    \
              }                                                                                     \
            }                                                                                       \
            __builtin_amdgcn_sched_barrier(0);                                                      \
          }                                                                                         \
        }                                                                                           \
      }                                                                                             \
      advance();                                                                                    \
      _Pragma("unroll") for (int nb = 2 * NP - 2; nb < WNX; ++nb)                                   \
        acc[MR - 1][nb] += low_[(MR * NP - 1) & 1][nb - 2 * NP + 2];                                \
      k_ = k_ + 1 == S ? 0 : k_ + 1;                                                                \
      ki_ = ki_ + 1 == S ? 0 : ki_ + 1;                                                             \
    }                                                                                               \
  }
      if constexpr (G::WN0 == G::WN1) {
        SSG_LOOP(G::WN0, wn * G::WN0)
      } else {
        if (wn == 0) SSG_LOOP(G::WN0, 0) else SSG_LOOP(G::WN1, G::WN0)
      }
      wait_vm<0>();  // the fetches past the end land before the stages are used again
#undef SSG_LOOP
#undef SSG_RDA
#undef SSG_RDB
    }

    // the tile, or this workgroup's share of it
    // (the lane index again, opaque: its address arithmetic would otherwise be hoisted out of the tile
    // loop and hold some 60 registers through the chunk loop)
    int el = lane;
    asm volatile("" : "+v"(el));
    const int g = el >> 4, r16 = el & 15;
    const int nbc = wn == 0 ? G::WN0 : G::WN1;
    const int c0 = 16 * G::WN0 * wn;
    if (sa == 0) {  // whole, or its first piece: straight to out
      bool past = false;
#pragma unroll
      for (int mb = 0; mb < MR; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t p = p0 + 16 * (wm * MR + mb) + 4 * g + i;
          if (p >= n_pos) continue;
#pragma unroll
          for (int nb = 0; nb < G::WN0; ++nb) {
            const int col = n0 + c0 + 16 * nb + r16;
            if (nb < nbc && col < cb) {
              out[p * cb + col] = acc[mb][nb][i];
              past |= past_range(acc[mb][nb][i]);
            }
          }
        }
      if (past) *flags.gathered() = 1;
    } else {
      float* dst = part + (int64_t)wg * BM * G::BN;
#pragma unroll
      for (int mb = 0; mb < MR; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * (wm * MR + mb) + 4 * g + i;
#pragma unroll
          for (int nb = 0; nb < G::WN0; ++nb)
            if (nb < nbc) dst[row * G::BN + c0 + 16 * nb + r16] = acc[mb][nb][i];
        }
    }
    u = t * K + sb;
  }
}

// Adds the pieces of the tiles that more than one workgroup held, in workgroup order.  A block takes
// 1024 consecutive values of one tile.
__global__ __launch_bounds__(256) void split_fixup(const float* __restrict__ part, TilePlan plan, int K, int BM,
                                                   int BN, int cb, int64_t n_pos, SplitFlags flags,
                                                   float* __restrict__ out) {
  const int64_t t = blockIdx.x;
  const int64_t i0 = unit_owner(plan, t * K), i1 = unit_owner(plan, t * K + K - 1);
  if (i0 == i1) return;
  const int e = (blockIdx.y * 256 + threadIdx.x) * 4, r = e / BN, c = e - r * BN;
  const int64_t p = plan.row0 + (t / plan.nt) * BM + r;
  const int col = (int)(t % plan.nt) * BN + c;
  if (r >= BM || p >= n_pos || col >= cb) return;
  float* o = out + p * cb + col;
  float v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = col + k < cb ? o[k] : 0.f;
  for (int64_t i = i0 + 1; i <= i1; ++i) {
    const float4 x = *reinterpret_cast<const float4*>(part + i * BM * BN + e);
    v[0] += x.x, v[1] += x.y, v[2] += x.z, v[3] += x.w;
  }
  if (past_range(v[0]) || past_range(v[1]) || past_range(v[2]) || past_range(v[3])) *flags.gathered() = 1;
  if ((cb & 3) == 0) {
    *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (col + k < cb) o[k] = v[k];
  }
}

struct SplitShape {
  int nb, mr;
  TilePlan plan;
  double us;  // of the gather and the pieces
};

size_t a3_bytes(int64_t n_src, int ca) { return align256((size_t)n_src * chunks32(ca) * 192); }
// (the column blocks of the last tile past cb16 read on past the end: up to 2 KB)
size_t b3_bytes(int ca, int cb, int K) { return align256((size_t)K * pad_k(ca) * pad16(cb) * 6 + 2048); }
size_t part_bytes(const SplitShape& s, int K) {
  return whole_tiles(s.plan, K) ? 0 : (size_t)s.plan.G * 64 * s.mr * 16 * s.nb * 4;
}
size_t shape_bytes(const SplitShape& s, int64_t n_src, int ca, int cb, int K) {
  return a3_bytes(n_src, ca) + b3_bytes(ca, cb, K) + part_bytes(s, K);
}

// Tile height and share of the workgroups.  A 32-channel chunk of an MR x NB tile takes about
// 0.3 + 0.0625 MR NB us (measured: 2.07 us at 4 x 7; the constant part is the barrier and the first
// fragment reads, which is why tall tiles win where there are rows enough).  Either every workgroup
// holds whole tiles, in rounds of one per compute unit, or the (tile, offset) sequence is cut evenly
// over the compute units, or over fewer workgroups, which costs the pieces' traffic and one more launch
// (cut_us).  A gradient's plan that is larger than the fixed region has to be a twentieth cheaper: closer than
// that whole tiles are sooner done (60k sites, 3x3x3, 128 -> 128: modelled 248 and 245, measured 265 and 292).
SplitShape split_shape(int64_t n_src, int ca, int cb, int64_t n_pos, int K, SplitPlans plans) {
  const int blocks = (cb + 15) / 16, tiles = (blocks + 7) / 8, per = (blocks + tiles - 1) / tiles;
  SplitShape best{}, s{};
  s.nb = per <= 2 ? 2 : per <= 4 ? 4 : per;
  s.plan.nt = (int)cdiv(cb, 16 * s.nb);
  s.plan.row0 = 0;
  const double chunks = pad_k(ca) / 32.0 * K;
  bool best_fits = false;
  double best_us = 0;
  for (int i = 0; i < 3 * (1 + kCutChoices); ++i) {
    s.mr = 4 >> (i / (1 + kCutChoices));
    s.plan.mt = (int)cdiv(n_pos, 64 * s.mr);
    const int64_t nt = (int64_t)s.plan.mt * s.plan.nt;
    s.plan.units = nt * K;
    const int cut = i % (1 + kCutChoices);
    s.us = chunks * (0.3 + 0.0625 * s.mr * s.nb);
    if (cut) {
      s.plan.G = (int)std::min<int64_t>(kTileWG >> (cut - 1), s.plan.units);
      s.us = s.us * nt / s.plan.G + cut_us(s.plan.G, nt) + (double)part_bytes(s, K) / 4e6;
    } else {
      s.plan.G = (int)std::min<int64_t>(nt, INT32_MAX);
      s.us *= cdiv(nt, kTileWG);
    }
    const bool fits = shape_bytes(s, n_src, ca, cb, K) + SplitFlags::kBytes <= SSCONV_NOALLOC_SCRATCH_BYTES;
    const double us = s.us * (fits ? 1.0 : 1.05);
    if (i == 0 || (plans == SplitPlans::kForward && fits != best_fits ? fits : us < best_us))
      best = s, best_fits = fits, best_us = us;
  }
  return best;
}

template <int NB, int MR>
int launch(const SplitShape& sh, const uint16_t* A3, int64_t a_bytes, int ca, const uint16_t* B3, int cb,
           const int32_t* nbr, int64_t n_pos, int K, float* part, const int* rows_flag, const SplitFlags& flags,
           float* out, hipStream_t st) {
  auto kern = gather_split_kernel<NB, MR>;
  using G = GS<NB, MR>;
  TilePlan plan = sh.plan;
  plan.panel = panel_offsets(G::ROOM, G::BM, pad_k(ca), K);
  const size_t smem = (size_t)(kTileLds - G::ROOM) + panel_bytes(plan.panel, G::BM, pad_k(ca));
  SSC_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  kern<<<plan.G, kTileThreads, smem, st>>>(A3, a_bytes, ca, B3, cb, nbr, n_pos, K, plan, part, rows_flag, flags, out);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

}  // namespace

bool gather_split_supported(int64_t n_src, int ca, int cb, int K) {
  return ca >= 1 && ca <= 4096 && cb >= 1 && K >= 1 && K <= kTileMaxK && n_src >= 1 && a3_bytes(n_src, ca) < ((size_t)1 << 31) &&
         b3_bytes(ca, cb, K) < ((size_t)1 << 31);
}

__global__ void clear_words(int* __restrict__ w) { w[threadIdx.x] = 0; }

int clear_split_flags(const SplitFlags& f, hipStream_t st) {
  clear_words<<<1, SplitFlags::kBytes / 4, 0, st>>>(f.w);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

size_t gather_split_bytes(int64_t n_src, int ca, int cb, int64_t n_pos, int K, SplitPlans plans) {
  return shape_bytes(split_shape(n_src, ca, cb, n_pos, K, plans), n_src, ca, cb, K);
}

// Fitted to 350 measured layers within a tenth: launches (the guard's among them), the rows read and written as
// parts, kappa, the gather, the row tables of the tiles past one round.
double gather_split_us(int64_t n_src, int ca, int cb, int64_t n_pos, int K) {
  const double rounds = (double)cdiv(n_pos, 256) * cdiv(cb, 128) / kTileWG;
  const double gather = split_shape(n_src, ca, cb, n_pos, K, SplitPlans::kGradient).us;
  return 13.5 + 0.5e-6 * n_src * (4.0 * ca + split_row_bytes(ca)) +
         1e-6 * K * (4.0 * ca * cb + 6.0 * pad_k(ca) * pad16(cb)) + gather +
         0.1 * K * std::max(0.0, rounds - 1.0);
}

int64_t split_row_bytes(int ca) { return (int64_t)chunks32(ca) * 192; }

int split_rows(const float* x, int64_t nx, int cx, uint16_t* x3, int* x_flag, const float* y, int64_t ny, int cy,
               uint16_t* y3, int* y_flag, hipStream_t st) {
  const unsigned xb = cdiv(nx * 4 * chunks32(cx), 256), yb = cdiv(ny * 4 * chunks32(cy), 256);
  if (xb + yb == 0) return SSCONV_OK;
  split_rows_kernel<<<xb + yb, 256, 0, st>>>(x, nx, cx, xb, x3, x_flag, y, ny, cy, y3, y_flag);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

int gather_split(const float* src, int64_t n_src, int ca, const SplitKernel& B, int cb, const int32_t* nbr,
                 int64_t n_pos, int K, float* out, const SplitFlags& flags, int* rows_flag, hipStream_t st, CallScratch* sc,
                 SplitPlans plans, const uint16_t* rows3, float* Bt) {
  if (n_pos == 0) return SSCONV_OK;
  const SplitShape s = split_shape(n_src, ca, cb, n_pos, K, plans);
  char* ws = nullptr;
  const size_t a3 = rows3 ? 0 : a3_bytes(n_src, ca);
  SSC_TRY(scratch_take(sc, (void**)&ws, a3 + b3_bytes(ca, cb, K) + part_bytes(s, K), st));
  uint16_t* const split = (uint16_t*)ws;
  const uint16_t* A3 = rows3 ? rows3 : split;
  uint16_t* B3 = (uint16_t*)(ws + a3);
  float* part = (float*)(ws + a3 + b3_bytes(ca, cb, K));
  const unsigned row_blocks = rows3 ? 0 : cdiv(n_src * 4 * chunks32(ca), 256);
  const unsigned b_blocks = cdiv((int64_t)K * (pad_k(ca) / 8) * pad16(cb), 256);
  split_operands<<<row_blocks + b_blocks, 256, 0, st>>>(src, n_src, ca, row_blocks, B, K, cb, split, B3,
                                                        rows_flag, flags.kappa(), Bt);
  int rc = hipGetLastError() == hipSuccess ? SSCONV_OK : fail(SSCONV_E_HIP, "operand split launch failed");
  const int64_t ab = (int64_t)n_src * chunks32(ca) * 192;
#define SSG_GO(NB_, MR_) rc = launch<NB_, MR_>(s, A3, ab, ca, B3, cb, nbr, n_pos, K, part, rows_flag, flags, out, st)
#define SSG_NB(NB_)                                                   \
  case NB_:                                                           \
    if (s.mr == 4) SSG_GO(NB_, 4);                                    \
    else if (s.mr == 2) SSG_GO(NB_, 2);                               \
    else SSG_GO(NB_, 1);                                              \
    break;
  if (rc == SSCONV_OK) {
    switch (s.nb) {
      SSG_NB(2) SSG_NB(4) SSG_NB(5) SSG_NB(6) SSG_NB(7)
      default:
        if (s.mr == 4) SSG_GO(8, 4);
        else if (s.mr == 2) SSG_GO(8, 2);
        else SSG_GO(8, 1);
    }
  }
#undef SSG_NB
#undef SSG_GO
  if (rc == SSCONV_OK && !whole_tiles(s.plan, K)) {
    const int BM = 64 * s.mr, BN = 16 * s.nb;
    dim3 grid((unsigned)(s.plan.mt * s.plan.nt), cdiv(BM * BN, 1024));
    split_fixup<<<grid, 256, 0, st>>>(part, s.plan, K, BM, BN, cb, n_pos, flags, out);
    if (hipGetLastError() != hipSuccess) rc = fail(SSCONV_E_HIP, "split fix-up launch failed");
  }
  scratch_give(sc, ws, st);
  return rc;
}

}  // namespace ssconv
