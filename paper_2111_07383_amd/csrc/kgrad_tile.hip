// Gradient of the kernel tensor (the adjoint of Alg. 1's feature update) on the bf16 matrix cores:
//
//   dkappa(s)[o][i] = sum_{(x, y) in R_s} grad_out[x][o] * feats[y][i]
//
// a GEMM per offset whose reduction runs over the compact pair list R_s.  The pair lists of all offsets
// are cut into work units of about equal length; each workgroup computes one (32 WM x 32 WN) tile of one
// offset over one unit and writes its own fp32 partial, and the partials of an offset are summed in a fixed
// order afterwards (deterministic, no atomics).
//
// P = 1: bf16 rows, one v_mfma_f32_16x16x32_bf16 per 16x16 block and 32 pairs.  P = 3: fp32 rows as three
// bf16 parts (24 bits, exact); six products, the five small ones in sums of their own, so that the large
// sum is rounded once per 32 pairs (v_mfma_f32_16x16x4f32: eight times, at 2.7 times the matrix-core cost).
//
// The operand of v_mfma_f32_16x16x32_bf16 is 8 consecutive PAIRS of one channel per lane, the transpose of
// the row layout.  A chunk of 32 pairs is staged in LDS in quads: 32 channels of one part of the 32 rows,
// 64 bytes a row, 2 KB, granule (16 bytes) p of row r at position p ^ 2 ((r / 8) % 2), so that the lanes a
// transpose read serves together hit distinct banks; one 1 KB DMA (buffer_load ... lds) fills a quad for
// 16 rows.  Operands are read with ds_read_b64_tr_b16: within a 16-lane group, output lane i / slot j
// receives element i%4 of the 8 bytes addressed by source lane 4j + i/4, so source lane L pointing at row
// (base + L/4), channel (c0 + 4*(L%4)) delivers pairs base..base+3 of channel c0 + i; two reads form one
// operand.
//
// Four wavefronts (2 x 2, one per SIMD).  Iteration c waits for the DMAs of chunk c+1, publishes them with
// one barrier, then runs the MFMAs of chunk c with the transpose reads of chunk c+1 and the DMAs of chunk
// c+S-1 spread between the rows of blocks.  One wavefront per SIMD has to issue everything under its own
// MFMAs, so the loop has no conditions: past the unit's end the rows are absent (zeros).
#include <algorithm>

#include "gather_tile.hpp"
#include "kgrad_tile.hpp"

namespace ssconv {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s4 __attribute__((ext_vector_type(4)));

constexpr int kPairBlock = 512;  // pair indices staged per block, double-buffered

template <int P, int WM, int WN>
struct KT {
  static constexpr int S = P == 1 ? 4 : 3;              // LDS stages
  static constexpr int Q = P * (WM + WN);               // quads per stage: grad_out's, then feats'
  static constexpr int STAGE = 2048 * Q;
  static constexpr int L = Q / 2;                       // DMAs per wavefront per chunk: half of every other quad
  static constexpr int SMEM = S * STAGE + 2 * kPairBlock * 8;
  static_assert(Q % 2 == 0, "the four wavefronts take two half quads each in turn");
  static_assert(SMEM <= kTileLds, "stages and pair blocks must fit the LDS");
};

__device__ __forceinline__ s4 tr_read(uint32_t lds) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4*)(uintptr_t)lds);
}

template <int P, int WM, int WN>
__global__ __launch_bounds__(256) void kgrad_tile_kernel(KgradRows G, int cout, KgradRows F, int cin,
                                                         const int2* __restrict__ pairs,
                                                         const int64_t* __restrict__ pair_off, KgradUnits units,
                                                         KgradOrder order, int mtiles, int ntiles, SplitFlags flags,
                                                         float* __restrict__ part) {
  if (P == 3 && (*flags.grad_out() | *flags.feats())) return;  // set before this kernel
  using C = KT<P, WM, WN>;
  constexpr int S = C::S, L = C::L;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* pblk = smem + S * C::STAGE;  // [2][kPairBlock] int2
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 1, wn = w & 1;

  // launch slot -> slice j of R_s, in the order of the rows (an XCD runs all offsets of a stretch of rows
  // together, which its L2 then holds), and tile
  const int tile = blockIdx.x % (mtiles * ntiles);
  const int slot = xcd_slot(blockIdx.x / (mtiles * ntiles), units.nunits);
  const int u = order.unit[slot];
  int s = 0;
  for (int b = 64; b > 0; b >>= 1)
    if (s + b < units.K && units.uoff[s + b] <= u) s += b;
  const int j = u - units.uoff[s], ns = units.uoff[s + 1] - units.uoff[s];
  const int m0 = tile / ntiles * 32 * WM, n0 = tile % ntiles * 32 * WN;
  const int64_t off = pair_off[s], cnt = pair_off[s + 1] - off;
  const int64_t beg = off + cnt * j / ns, end = off + cnt * (j + 1) / ns;
  const int npairs = (int)(end - beg);
  const int nchunk = (npairs + 31) / 32;

  const __amdgpu_buffer_rsrc_t g_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(G.p), (short)0, (int)G.bytes, kRawBufferWord3);
  const __amdgpu_buffer_rsrc_t f_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(F.p), (short)0, (int)F.bytes, kRawBufferWord3);
  // the unit's pair list as a byte buffer (past its end: zeros, masked below)
  const __amdgpu_buffer_rsrc_t p_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int2*>(pairs + beg), (short)0, npairs * 8, kRawBufferWord3);
  const uint32_t stage0 = lds_addr(smem), pblk_a = lds_addr(pblk);

  // DMA q of this wavefront fills rows 16 (w % 2) .. + 15 of quad h L + q, h = w / 2 (neighbouring quads of a
  // row share cache lines), so a lane keeps one pair row for the whole chunk: row 16 (w % 2) + l / 4,
  // granule (l % 4) ^ the quad's swizzle
  const int h = w >> 1, q0 = h * L;
  const int prow = 16 * (w & 1) + (lane >> 2);
  const uint32_t granule = 16u * (uint32_t)((lane & 3) ^ (((prow >> 3) & 1) << 1));
  const uint32_t g_stat = (uint32_t)m0 * 2u * P + granule + 64u * (uint32_t)q0;
  const uint32_t f_stat = (uint32_t)n0 * 2u * P + granule + 64u * (uint32_t)(q0 - P * WM);  // quads count on from grad_out's
  const int nqg = ((cout - m0 + 31) / 32) * P, nqf = P * WM + ((cin - n0 + 31) / 32) * P;  // quads that hold channels

  // pair block b (slice pairs [b, b + 1) * kPairBlock) into buffer b % 2: 1 KB per wavefront
  auto load_pairs = [&](int b) {
    dma16_tile(p_rsrc, (uint32_t)(b * kPairBlock * 8 + w * 1024 + 16 * lane),
               pblk_a + (b & 1) * kPairBlock * 8 + w * 1024);
  };
  // byte offsets of this lane's rows in chunk c (kAbsentRow32 past the unit's end)
  uint32_t grow, frow;
  auto rows_of = [&](int c) {
    const int2 v = *reinterpret_cast<const int2*>(
        pblk + ((c / (kPairBlock / 32)) & 1) * (kPairBlock * 8) + (c % (kPairBlock / 32)) * 256 + prow * 8);
    const bool in = prow < npairs - c * 32;
    grow = in ? (uint32_t)v.x * (uint32_t)G.stride + g_stat : kAbsentRow32;
    frow = in ? (uint32_t)v.y * (uint32_t)F.stride + f_stat : kAbsentRow32;
  };
  const __amdgpu_buffer_rsrc_t x_rsrc = h ? f_rsrc : g_rsrc;
  auto dma = [&](int q, uint32_t sbase) {
    const int qd = q0 + q;
    const uint32_t lds = sbase + qd * 2048 + (w & 1) * 1024;
    if (L + q < P * WM)  // grad_out's in both halves
      dma16_tile(g_rsrc, qd < nqg ? grow + q * 64u : kAbsentRow32, lds);
    else if (q >= P * WM)  // feats' in both
      dma16_tile(f_rsrc, qd < nqf ? frow + q * 64u : kAbsentRow32, lds);
    else
      dma16_tile(x_rsrc, qd < (h ? nqf : nqg) ? (h ? frow : grow) + q * 64u : kAbsentRow32, lds);
  };

  // operands via transpose reads: rows R = 8g + 4h + L/4, channel 16 b + 4 (L % 4) of MFMA block b, i.e. quad
  // b / 2, position 2 ((b % 2) ^ (g % 2)) + (L % 4) / 2, byte 8 ((L % 4) % 2)
  const uint32_t rd_lane = (uint32_t)((8 * g + (r16 >> 2)) * 64 + ((r16 & 3) >> 1) * 16 + (r16 & 1) * 8);
  const uint32_t gx = (uint32_t)(g & 1) * 32u;
  auto frag = [&](uint32_t sbase, int quad0, int b, int p) {
    const uint32_t a = sbase + rd_lane + (uint32_t)(quad0 + (b >> 1) * P + p) * 2048u + ((((uint32_t)b & 1u) * 32u) ^ gx);
    const s4 lo = tr_read(a), hi = tr_read(a + 256u);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // zeros the compiler cannot fold, each an expression of its own: with one shared zero the register
  // allocator merges the accumulators and then copies them apart on every path into the chunk loop
  f4 acc[WM][WN], low[P == 3 ? WM : 1][P == 3 ? WN : 1];
  {
    const float z = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane(npairs < 0 ? 1 : 0));
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int k = 0; k < WN; ++k) {
        const float zi = z * (float)(i * WN + k + 1), zl = z * (float)(i * WN + k + 1 + WM * WN);
        acc[i][k] = f4{zi, zi, zi, zi};
        if constexpr (P == 3) low[i][k] = f4{zl, zl, zl, zl};
      }
  }

  constexpr int NR = (WM + WN) * P;  // fragments of a wavefront's blocks
#define SSK_FRAG(AF, BF, u_, sb_)                                                                   \
  do {                                                                                              \
    if ((u_) < WM * P)                                                                              \
      AF[(u_) / P][(u_) % P] = frag(sb_, 0, wm * WM + (u_) / P, (u_) % P);                          \
    else                                                                                            \
      BF[((u_) - WM * P) / P][((u_) - WM * P) % P] = frag(sb_, P * WM, wn * WN + ((u_) - WM * P) / P, ((u_) - WM * P) % P); \
  } while (0)

  // The barrier of iteration c needs no LDS fence: the transpose reads of a chunk are consumed by its
  // MFMAs before the next barrier, and its stage is refilled only after that.
#define SSK_BODY(c_, k_, AC, BC, AN, BN)                                                            \
  {                                                                                                 \
    const int cc_ = (c_);                                                                           \
    wait_vm<(S - 3) * L>();                                                                         \
    asm volatile("s_barrier" ::: "memory");                                                         \
    const int ci_ = cc_ + S - 1; /* chunk whose rows are issued now */                              \
    if (ci_ % (kPairBlock / 32) == 0 && ci_ / (kPairBlock / 32) + 1 < nblk)                         \
      load_pairs(ci_ / (kPairBlock / 32) + 1);                                                      \
    const uint32_t si_ = stage0 + ((k_) + S - 1) % S * C::STAGE, sr_ = stage0 + ((k_) + 1) % S * C::STAGE; \
    rows_of(ci_);                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                              \
    _Pragma("unroll") for (int i = 0; i < WM; ++i) {                                                \
      if constexpr (P == 1) {                                                                       \
        _Pragma("unroll") for (int n = 0; n < WN; ++n)                                              \
          acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(AC[i][0], BC[n][0], acc[i][n], 0, 0, 0); \
      } else {                                                                                      \
        constexpr int qa[6] = {2, 1, 0, 1, 0, 0}, qb[6] = {0, 1, 2, 0, 1, 0};                       \
        _Pragma("unroll") for (int t = 0; t < 6; ++t) {                                             \
          _Pragma("unroll") for (int n = 0; n < WN; ++n) {                                          \
            f4& to = t == 5 ? acc[i][n] : low[P == 3 ? i : 0][P == 3 ? n : 0];                      \
            to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(AC[i][P == 1 ? 0 : qa[t]], BC[n][P == 1 ? 0 : qb[t]], to, 0, 0, 0); \
          }                                                                                         \
          if (t == 2) {                                                                             \
            __builtin_amdgcn_sched_barrier(0);                                                      \
            _Pragma("unroll") for (int u2 = i * NR / WM; u2 < (2 * i + 1) * NR / (2 * WM); ++u2) SSK_FRAG(AN, BN, u2, sr_); \
            _Pragma("unroll") for (int q = i * L / WM; q < (2 * i + 1) * L / (2 * WM); ++q) dma(q, si_); \
            __builtin_amdgcn_sched_barrier(0);                                                      \
          }                                                                                         \
        }                                                                                           \
      }                                                                                             \
      __builtin_amdgcn_sched_barrier(0);                                                            \
      _Pragma("unroll") for (int u2 = P == 1 ? i * NR / WM : (2 * i + 1) * NR / (2 * WM); u2 < (i + 1) * NR / WM; ++u2) \
        SSK_FRAG(AN, BN, u2, sr_);                                                                  \
      _Pragma("unroll") for (int q = P == 1 ? i * L / WM : (2 * i + 1) * L / (2 * WM); q < (i + 1) * L / WM; ++q) dma(q, si_); \
      __builtin_amdgcn_sched_barrier(0);                                                            \
    }                                                                                               \
  }

  const int nblk = (npairs + kPairBlock - 1) / kPairBlock;
  if (nchunk > 0) {
    load_pairs(0);
    if (nblk > 1) load_pairs(1);
    wait_vm<0>();
    __syncthreads();
#pragma unroll
    for (int c = 0; c < S - 1; ++c) {
      rows_of(c);
#pragma unroll
      for (int q = 0; q < L; ++q) dma(q, stage0 + c * C::STAGE);
    }
    bf16x8 a0[WM][P], b0[WN][P], a1[WM][P], b1[WN][P];
    wait_vm<(S - 2) * L>();
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int u2 = 0; u2 < NR; ++u2) SSK_FRAG(a0, b0, u2, stage0);
    // the stage index and the fragment sets repeat every lcm(S, 2) chunks (guards, not breaks: with breaks the
    // accumulators are copied on every path out of the loop)
    for (int c = 0; c < nchunk; c += S == 4 ? 4 : 6) {
      SSK_BODY(c, 0, a0, b0, a1, b1)
      if (c + 1 < nchunk) SSK_BODY(c + 1, 1, a1, b1, a0, b0)
      if (c + 2 < nchunk) SSK_BODY(c + 2, 2, a0, b0, a1, b1)
      if (c + 3 < nchunk) SSK_BODY(c + 3, 3 % S, a1, b1, a0, b0)
      if constexpr (S == 3) {
        if (c + 4 < nchunk) SSK_BODY(c + 4, 1, a0, b0, a1, b1)
        if (c + 5 < nchunk) SSK_BODY(c + 5, 2, a1, b1, a0, b0)
      }
    }
    wait_vm<0>();  // the fetches past the end land before the LDS is given back
  }
#undef SSK_BODY
#undef SSK_FRAG

  float* dst = part + (int64_t)u * cout * cin;
  bool past = false;
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + (wm * WM + i) * 16 + 4 * g + e;
      if (m >= cout) continue;
#pragma unroll
      for (int n = 0; n < WN; ++n) {
        const int col = n0 + (wn * WN + n) * 16 + r16;
        if (col >= cin) continue;
        const float v = P == 3 ? low[P == 3 ? i : 0][P == 3 ? n : 0][e] + acc[i][n][e] : acc[i][n][e];
        dst[(int64_t)m * cin + col] = v;
        past |= past_range(v);
      }
    }
  if (P == 3 && past) *flags.kgrad() = 1;
}

template <int P, int WM, int WN>
int launch(const KgradRows& G, const KgradRows& F, int cin, int cout, const ssconv_rulebook* rb, const KgradTile& t,
           const KgradUnits& units, const KgradOrder& order, const SplitFlags& flags, float* part, hipStream_t st) {
  auto kern = kgrad_tile_kernel<P, WM, WN>;
  constexpr int smem = KT<P, WM, WN>::SMEM;
  SSC_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem));
  kern<<<(unsigned)(units.nunits * t.mtiles * t.ntiles), 256, smem, st>>>(
      G, cout, F, cin, reinterpret_cast<const int2*>(rb->pairs), rb->pair_off_dev, units, order, t.mtiles, t.ntiles, flags,
      part);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

}  // namespace

// The tile with the least matrix work on padded channels and transpose reads (about 0.35 of a block's MFMA
// each).  Units have at least 256 pairs, below which the partials outweigh the rows.
// bf16: about equal pieces of the lists, so that one long list (isolated sites: nearly all pairs are those of
// the centre) is spread over the chip: 40k isolated sites, 3x3x3, 208 -> 208, as many slices of every list 150
// us, equal pieces 80.  As many units as workgroups are on the chip at a time (their LDS), at most 512;
// on 7x7 tiles, of which a compute unit holds one, two rounds where the rows take longer than
// the further partials (200k sites, 5.4M pairs, 208 -> 208: 9 slices of every list 463 us and 18 to add the
// partials up, 18 slices 446 and 24; 80k sites, 1.4M pairs: 218 us with 18 slices in all, 170 with 256 units).
// Split rows: four rounds, since their gathers miss the L2 more (an XCD runs all offsets of a stretch of rows
// together: 36k sites, 5x5x5, 104 -> 104, as many slices of every list: 2 slices 780 us, 4 661, 8 596, 12 617;
// in equal pieces the training step of that layer 1634 -> 1594).
KgradTile kgrad_tile(const ssconv_rulebook* rb, int parts, int cin, int cout) {
  static const int shapes[][2] = {{2, 2}, {2, 4}, {4, 2}, {4, 4}, {7, 7}};
  KgradTile best{};
  double best_cost = 0.0;
  for (int i = 0; i < (parts == 1 ? 5 : 4); ++i) {
    KgradTile t;
    t.wm = shapes[i][0];
    t.wn = shapes[i][1];
    t.mtiles = (cout + 32 * t.wm - 1) / (32 * t.wm);
    t.ntiles = (cin + 32 * t.wn - 1) / (32 * t.wn);
    const double cost = (double)t.mtiles * t.ntiles * (t.wm * t.wn + 0.35 * (t.wm + t.wn));
    if (i == 0 || cost < best_cost) best = t, best_cost = cost;
  }
  const int tiles = best.mtiles * best.ntiles;
  const int64_t by_pairs = rb->n_pairs / 256;
  const int64_t most = parts == 3 ? 1024 : best.wm < 7 || rb->n_pairs >= 4000000 ? 512 : 256;
  best.units = (int)std::max<int64_t>(1, std::min<int64_t>(most / tiles, by_pairs));
  return best;
}

int kgrad_tiles(const KgradRows& G, const KgradRows& F, int parts, int cin, int cout, const ssconv_rulebook* rb,
                const KgradTile& t, const KgradUnits& units, const KgradOrder& order, const SplitFlags& flags,
                float* part, hipStream_t st) {
  if (units.nunits == 0) return SSCONV_OK;
#define SSK_GO(P_, M_, N_) return launch<P_, M_, N_>(G, F, cin, cout, rb, t, units, order, flags, part, st)
  if (parts == 1) {
    if (t.wm == 7) SSK_GO(1, 7, 7);
    if (t.wm == 4 && t.wn == 4) SSK_GO(1, 4, 4);
    if (t.wm == 4) SSK_GO(1, 4, 2);
    if (t.wn == 4) SSK_GO(1, 2, 4);
    SSK_GO(1, 2, 2);
  }
  if (t.wm == 4 && t.wn == 4) SSK_GO(3, 4, 4);
  if (t.wm == 4) SSK_GO(3, 4, 2);
  if (t.wn == 4) SSK_GO(3, 2, 4);
  SSK_GO(3, 2, 2);
#undef SSK_GO
}

}  // namespace ssconv
