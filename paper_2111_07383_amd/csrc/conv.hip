// Sparse steerable convolution on matrix cores (Sec. 3.2.3, the feature update of Alg. 1) and its adjoint.
//
// gather_gemm: output-stationary implicit GEMM.  A workgroup owns BM = 64 output
// rows x BN = 16*WNB output channels and accumulates, in MFMA accumulators,
//     out[x] = sum_s sum_{y = nbr[s][x]} kappa(s) feats[y]
// over the offsets present in its rows (an offset with no neighbour in the
// tile is skipped entirely; missing rows of a present offset are zero-filled).
// Feature rows are gathered with 16-byte loads into LDS tiles of 32 channels;
// kappa(s) is staged transposed so both MFMA operands are read as contiguous
// 8-element runs.  Each output element is written exactly once: no atomics.
// The feature gradient is the same kernel on (grad_out, kappa^T, transposed
// neighbour map).
//
// dw_gemm: dkappa(s) = sum_{(x,y) in R_s} grad_out[x] feats[y]^T, a gather-gather
// GEMM over the compact pair list of each offset, split along the pairs into
// fixed chunks whose partial sums are reduced in a fixed order (deterministic).
//
// MFMA: fp32 uses v_mfma_f32_16x16x4f32 (eight K-steps per 32-channel chunk,
// lane group g = lane/16 taking channels 8g..8g+7), bf16 uses the gfx950
// v_mfma_f32_16x16x32_bf16 (one step per chunk).  Any assignment of channels
// to K-steps is valid as long as both operands use the same one.
#include <algorithm>
#include <cmath>

#include "conv.hpp"
#include "norm.hpp"
#include "gather_mfma.hpp"
#include "gather_split.hpp"
#include "gather_tile.hpp"
#include "kgrad_mfma.hpp"

namespace ssconv {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kNT = 256;
constexpr int BM = 64;
constexpr int BK = 32;

template <typename T>
struct Cfg {
  static constexpr int VE = 16 / (int)sizeof(T);     // elements per 16-byte vector
  static constexpr int VPR = BK / VE;                // vectors per 32-element row chunk
  static constexpr int ROW = BK + VE;                // padded LDS row (elements): +16 bytes
};

template <typename T>
__device__ __forceinline__ uint4 load_vec(const T* __restrict__ p, int avail, bool vec_ok) {
  if (vec_ok && avail >= Cfg<T>::VE) return *reinterpret_cast<const uint4*>(p);
  T tmp[Cfg<T>::VE];
#pragma unroll
  for (int e = 0; e < Cfg<T>::VE; ++e) tmp[e] = e < avail ? p[e] : T(0);
  uint4 r;
  __builtin_memcpy(&r, tmp, 16);
  return r;
}

// One 32-element K chunk: acc += A_frag x B_frag for a 16x16 block.
__device__ __forceinline__ void mma_chunk(f4& acc, const float* a, const float* b) {
  const uint4 a0 = *reinterpret_cast<const uint4*>(a), a1 = *reinterpret_cast<const uint4*>(a + 4);
  const uint4 b0 = *reinterpret_cast<const uint4*>(b), b1 = *reinterpret_cast<const uint4*>(b + 4);
  const float av[8] = {__uint_as_float(a0.x), __uint_as_float(a0.y), __uint_as_float(a0.z), __uint_as_float(a0.w),
                       __uint_as_float(a1.x), __uint_as_float(a1.y), __uint_as_float(a1.z), __uint_as_float(a1.w)};
  const float bv[8] = {__uint_as_float(b0.x), __uint_as_float(b0.y), __uint_as_float(b0.z), __uint_as_float(b0.w),
                       __uint_as_float(b1.x), __uint_as_float(b1.y), __uint_as_float(b1.z), __uint_as_float(b1.w)};
#pragma unroll
  for (int t = 0; t < 8; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t], bv[t], acc, 0, 0, 0);
}

__device__ __forceinline__ void mma_chunk(f4& acc, const uint16_t* a, const uint16_t* b) {
  const uint4 ar = *reinterpret_cast<const uint4*>(a), br = *reinterpret_cast<const uint4*>(b);
  bf16x8 av, bv;
  __builtin_memcpy(&av, &ar, 16);
  __builtin_memcpy(&bv, &br, 16);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// output-stationary gather GEMM (forward and feature gradient)
// ---------------------------------------------------------------------------
template <typename T, int WNB>
__global__ __launch_bounds__(kNT) void gather_gemm(const T* __restrict__ src, int ca, const T* __restrict__ Bt,
                                                   int cb, const int32_t* __restrict__ nbr, int64_t n_rows, int K,
                                                   T* __restrict__ out, OnlyIf only) {
  if (idle(only)) return;
  using C = Cfg<T>;
  constexpr int BN = 16 * WNB;
  constexpr int AV = BM * C::VPR / kNT;                 // A vectors per thread (2 f32 / 1 bf16)
  constexpr int BV = (BN * C::VPR + kNT - 1) / kNT;     // B vectors per thread (upper bound)
  __shared__ __attribute__((aligned(16))) T As[BM * C::ROW];
  __shared__ __attribute__((aligned(16))) T Bs[BN * C::ROW];
  __shared__ uint32_t smask[4];

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, r16 = lane & 15;
  const int64_t p0 = (int64_t)blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;
  const bool vec_ok = (ca % C::VE) == 0;

  if (tid < 4) smask[tid] = 0;
  __syncthreads();
  for (int s = w; s < K; s += 4) {
    const int64_t p = p0 + lane;
    const int idx = p < n_rows ? nbr[(int64_t)s * n_rows + p] : -1;
    const uint64_t any = __ballot(idx >= 0);
    if (lane == 0 && any) atomicOr(&smask[s >> 5], 1u << (s & 31));
  }
  __syncthreads();
  const uint32_t mk[4] = {smask[0], smask[1], smask[2], smask[3]};

  f4 acc[WNB];
#pragma unroll
  for (int nb = 0; nb < WNB; ++nb) acc[nb] = f4{0.f, 0.f, 0.f, 0.f};

  for (int s = 0; s < K; ++s) {
    if (!((mk[s >> 5] >> (s & 31)) & 1u)) continue;
    int aidx[AV];
#pragma unroll
    for (int j = 0; j < AV; ++j) {
      const int r = (tid + kNT * j) / C::VPR;
      const int64_t p = p0 + r;
      aidx[j] = p < n_rows ? nbr[(int64_t)s * n_rows + p] : -1;
    }
    const T* Bs_s = Bt + (int64_t)s * cb * ca;
    for (int k0 = 0; k0 < ca; k0 += BK) {
      uint4 av[AV], bv[BV];
#pragma unroll
      for (int j = 0; j < AV; ++j) {
        const int v = tid + kNT * j, cv = v % C::VPR, col = k0 + cv * C::VE;
        av[j] = (aidx[j] >= 0 && col < ca) ? load_vec(src + (int64_t)aidx[j] * ca + col, ca - col, vec_ok)
                                          : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < BV; ++j) {
        const int v = tid + kNT * j, n = v / C::VPR, cv = v % C::VPR, col = k0 + cv * C::VE;
        bv[j] = (v < BN * C::VPR && n0 + n < cb && col < ca)
                    ? load_vec(Bs_s + (int64_t)(n0 + n) * ca + col, ca - col, vec_ok)
                    : make_uint4(0, 0, 0, 0);
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < AV; ++j) {
        const int v = tid + kNT * j, r = v / C::VPR, cv = v % C::VPR;
        *reinterpret_cast<uint4*>(&As[r * C::ROW + cv * C::VE]) = av[j];
      }
#pragma unroll
      for (int j = 0; j < BV; ++j) {
        const int v = tid + kNT * j, n = v / C::VPR, cv = v % C::VPR;
        if (v < BN * C::VPR) *reinterpret_cast<uint4*>(&Bs[n * C::ROW + cv * C::VE]) = bv[j];
      }
      __syncthreads();
      const T* a = &As[(16 * w + r16) * C::ROW + 8 * g];
#pragma unroll
      for (int nb = 0; nb < WNB; ++nb) mma_chunk(acc[nb], a, &Bs[(16 * nb + r16) * C::ROW + 8 * g]);
    }
  }

#pragma unroll
  for (int nb = 0; nb < WNB; ++nb) {
    const int col = n0 + 16 * nb + r16;
    if (col >= cb) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = p0 + 16 * w + 4 * g + i;
      if (row < n_rows) out[row * cb + col] = DT<T>::from_f(acc[nb][i]);
    }
  }
}

// ---------------------------------------------------------------------------
// dkappa partials: gather-gather GEMM over the pair list of one offset
// ---------------------------------------------------------------------------
template <typename T, int WNB>
__global__ __launch_bounds__(kNT) void dw_gemm(const T* __restrict__ G, int cout, const T* __restrict__ F, int cin,
                                               const int32_t* __restrict__ pairs,
                                               const int64_t* __restrict__ pair_off, int K, int ntn, int nsplit,
                                               float* __restrict__ part) {
  using C = Cfg<T>;
  constexpr int BN = 16 * WNB;
  constexpr int VA = BM / C::VE;   // vectors per gathered grad row segment (64 channels)
  constexpr int VB = BN / C::VE;   // vectors per gathered feature row segment
  __shared__ __attribute__((aligned(16))) T At[BM * C::ROW];   // [m = out channel][k = pair]
  __shared__ __attribute__((aligned(16))) T Bs[BN * C::ROW];   // [n = in channel][k = pair]
  __shared__ int2 sp[BK];

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, r16 = lane & 15;
  const int mt = blockIdx.x / ntn, nt = blockIdx.x % ntn;
  const int split = blockIdx.y, s = blockIdx.z;
  const int m0 = mt * BM, n0 = nt * BN;
  const int64_t off = pair_off[s], cnt = pair_off[s + 1] - off;
  const int64_t beg = off + cnt * split / nsplit, end = off + cnt * (split + 1) / nsplit;
  const bool vec_a = (cout % C::VE) == 0, vec_b = (cin % C::VE) == 0;

  f4 acc[WNB];
#pragma unroll
  for (int nb = 0; nb < WNB; ++nb) acc[nb] = f4{0.f, 0.f, 0.f, 0.f};

  for (int64_t kb = beg; kb < end; kb += BK) {
    __syncthreads();
    if (tid < BK) sp[tid] = (kb + tid < end) ? reinterpret_cast<const int2*>(pairs)[kb + tid] : make_int2(-1, -1);
    __syncthreads();
    // A: BK pairs x 64 out channels, stored transposed
    for (int v = tid; v < BK * VA; v += kNT) {
      const int k = v / VA, cv = v % VA, col = m0 + cv * C::VE;
      const int o = sp[k].x;
      uint4 x = (o >= 0 && col < cout) ? load_vec(G + (int64_t)o * cout + col, cout - col, vec_a) : make_uint4(0, 0, 0, 0);
      T e[C::VE];
      __builtin_memcpy(e, &x, 16);
#pragma unroll
      for (int q = 0; q < C::VE; ++q) At[(cv * C::VE + q) * C::ROW + k] = e[q];
    }
    for (int v = tid; v < BK * VB; v += kNT) {
      const int k = v / VB, cv = v % VB, col = n0 + cv * C::VE;
      const int i = sp[k].y;
      uint4 x = (i >= 0 && col < cin) ? load_vec(F + (int64_t)i * cin + col, cin - col, vec_b) : make_uint4(0, 0, 0, 0);
      T e[C::VE];
      __builtin_memcpy(e, &x, 16);
#pragma unroll
      for (int q = 0; q < C::VE; ++q) Bs[(cv * C::VE + q) * C::ROW + k] = e[q];
    }
    __syncthreads();
    const T* a = &At[(16 * w + r16) * C::ROW + 8 * g];
#pragma unroll
    for (int nb = 0; nb < WNB; ++nb) mma_chunk(acc[nb], a, &Bs[(16 * nb + r16) * C::ROW + 8 * g]);
  }

  float* dst = part + ((int64_t)split * K + s) * cout * cin;
#pragma unroll
  for (int nb = 0; nb < WNB; ++nb) {
    const int col = n0 + 16 * nb + r16;
    if (col >= cin) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = m0 + 16 * w + 4 * g + i;
      if (row < cout) dst[(int64_t)row * cin + col] = acc[nb][i];
    }
  }
}

// dW (field-pair-blocked, dw_block_pos) = sum of the splits' [K][cout][cin] partials, in split order.
__global__ void reduce_splits(const float* __restrict__ part, int nsplit, int64_t n, FieldTab fout, FieldTab fin,
                              int K, int cin, int cout, float* __restrict__ dst) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  float acc = 0.f;
  for (int j = 0; j < nsplit; ++j) acc += part[(int64_t)j * n + e];
  const int64_t plane = (int64_t)cin * cout;
  const int s = (int)(e / plane), r = (int)(e - s * plane), o = r / cin, i = r - o * cin;
  dst[dw_block_pos(fout, fin, K, cin, s, o, i)] = acc;
}

template <typename T>
__global__ void transpose_kernel(const T* __restrict__ W, int K, int rows, int cols, int mirror, T* __restrict__ Wt) {
  // W [K][rows][cols] -> Wt [K][cols][rows], offsets reversed (Wt[s] = W[K-1-s]^T) when mirror
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t per = (int64_t)rows * cols;
  if (i >= per * K) return;
  const int64_t s = i / per, r = i % per;
  const int c = (int)(r / rows), rr = (int)(r % rows);
  Wt[i] = W[(mirror ? K - 1 - s : s) * per + (int64_t)rr * cols + c];
}

__global__ void fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void invert_nbr(const int32_t* __restrict__ nbr, int64_t n_out, int K, int64_t n_in,
                           int32_t* __restrict__ nbrT) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int s = blockIdx.y;
  if (p >= n_out) return;
  const int i = nbr[(int64_t)s * n_out + p];
  if (i >= 0) nbrT[(int64_t)s * n_in + i] = (int32_t)p;
}

template <typename T, int WNB>
void launch_gg(const void* src, int ca, const void* Bt, int cb, const int32_t* nbr, int64_t n_rows, int K, void* out,
               hipStream_t st, const OnlyIf& only) {
  dim3 grid(cdiv(n_rows, BM), cdiv(cb, 16 * WNB));
  gather_gemm<T, WNB><<<grid, kNT, 0, st>>>((const T*)src, ca, (const T*)Bt, cb, nbr, n_rows, K, (T*)out, only);
}

// Picks the N-tile width (in 16-column blocks) for cb output channels.
int pick_wnb(int cb) {
  const int blocks = (cb + 15) / 16;
  if (blocks <= 8) return blocks;
  // split wide outputs into near-equal tiles of at most 8 blocks
  const int tiles = (blocks + 7) / 8;
  return (blocks + tiles - 1) / tiles;
}

template <typename T>
int dispatch_gg(const void* src, int64_t n_src, int ca, const void* Bt, int cb, const int32_t* nbr, int64_t n_rows, int K,
                void* out, hipStream_t st, CallScratch* sc = nullptr, NormSink* sink = nullptr,
                const OnlyIf& only = OnlyIf()) {
  const ssconv_dtype dt = sizeof(T) == 4 ? SSCONV_F32 : SSCONV_BF16;
  if (gather_mfma_supported(dt, ca, cb, K))
    return gather_mfma(src, n_src, dt, ca, Bt, cb, nbr, nullptr, n_rows, K, out, st, sc, sink, only);
  switch (pick_wnb(cb)) {
    case 1: launch_gg<T, 1>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
    case 2: launch_gg<T, 2>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
    case 3: launch_gg<T, 3>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
    case 4: launch_gg<T, 4>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
    case 5: launch_gg<T, 5>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
    case 6: launch_gg<T, 6>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
    case 7: launch_gg<T, 7>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
    default: launch_gg<T, 8>(src, ca, Bt, cb, nbr, n_rows, K, out, st, only); break;
  }
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

// Offsets that a tile of `rows` destination rows holds, were the pairs spread evenly (every site is its own
// neighbour in a submanifold layer).
double active_offsets(const ssconv_rulebook* rb, int64_t n_dst, int rows) {
  const int own = rb->submanifold ? 1 : 0;
  if (rb->K <= own || n_dst <= 0) return own;
  const double share = ((double)rb->n_pairs - own * n_dst) / ((double)n_dst * (rb->K - own));
  return own + (rb->K - own) * (1.0 - std::pow(1.0 - std::min(1.0, std::max(0.0, share)), rows));
}

// Time of the feature gradient by dispatch_gg in fp32, us.  gather_gemm walks the offsets in steps of 32 channels:
// bound by a step's latency, or by the work of the workgroups that share a compute unit.
double plain_us(const ssconv_rulebook* rb, int ca, int cb, int64_t n_dst) {
  if (gather_mfma_supported(SSCONV_F32, ca, cb, rb->K))
    return gather_mfma_us(ca, cb, n_dst, rb->K, active_offsets(rb, n_dst, kMfmaRows));
  const int wnb = pick_wnb(cb);
  const double tiles = (double)cdiv(n_dst, BM) * cdiv(cb, 16 * wnb);
  return 5.0 + active_offsets(rb, n_dst, BM) * cdiv(ca, BK) * std::max(0.9 + 0.14 * wnb, tiles / 256 * (0.5 + 0.13 * wnb));
}

template <typename T, int WNB>
void launch_dw(const void* G, int cout, const void* F, int cin, const int32_t* pairs, const int64_t* pair_off, int K,
               int nsplit, float* part, hipStream_t st) {
  const int ntm = (int)cdiv(cout, BM), ntn = (int)cdiv(cin, 16 * WNB);
  dim3 grid(ntm * ntn, nsplit, K);
  dw_gemm<T, WNB><<<grid, kNT, 0, st>>>((const T*)G, cout, (const T*)F, cin, pairs, pair_off, K, ntn, nsplit, part);
}

template <typename T>
int dispatch_dw(const void* G, int cout, const void* F, int cin, const int32_t* pairs, const int64_t* pair_off, int K,
                int nsplit, float* part, hipStream_t st) {
  switch (pick_wnb(cin)) {
    case 1: launch_dw<T, 1>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
    case 2: launch_dw<T, 2>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
    case 3: launch_dw<T, 3>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
    case 4: launch_dw<T, 4>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
    case 5: launch_dw<T, 5>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
    case 6: launch_dw<T, 6>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
    case 7: launch_dw<T, 7>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
    default: launch_dw<T, 8>(G, cout, F, cin, pairs, pair_off, K, nsplit, part, st); break;
  }
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

}  // namespace

// The bf16 pipeline kernel.  With a fixed scratch region a call whose operands do not fit takes the
// kernels that need none, except where packed kappa alone was always the limit (channels in multiples of
// 8, at most 27 offsets): there the region's error stands.
static bool use_bf16_kernel(const CallScratch* sc, ssconv_dtype dt, int64_t n_src, int ca, int cb, int64_t n_pos, int K) {
  if (dt != SSCONV_BF16 || debug_gather_variant() == 5 || !gather_bf16_supported(n_src, ca, cb, K)) return false;
  if (!(sc && sc->fixed()) || gather_bf16_bytes(n_src, ca, cb, n_pos, K) <= sc->left()) return true;
  return ca % 8 == 0 && K <= 27 && (size_t)K * ca * cb * 2 > sc->left();
}

// fp32 on the bf16 matrix cores; the overrides that pick an fp32 MFMA variant keep that kernel, and a
// fixed scratch region too small for the split operands does.
static bool use_split(const CallScratch* sc, int64_t n_src, int ca, int cb, int64_t n_pos, int K) {
  const int64_t v = debug_gather_variant();
  if (v == 1 || v == 2 || v == 3 || v == 8 || !gather_split_supported(n_src, ca, cb, K)) return false;
  return !(sc && sc->fixed()) ||
         SplitFlags::kBytes + gather_split_bytes(n_src, ca, cb, n_pos, K, SplitPlans::kForward) <= sc->left();
}

// Forwards below 2^35 multiply-adds (of n_out x K, not of pairs) keep the kernels that they have always had and
// with them their bits, which a ReLU or a gate behind them may turn on.  That is a choice and no matter of
// precision: above the line the same holds, the split kernel's errors are the smaller ones, and small calls would
// gain as well (2.5k sites, 3x3x3, 104 -> 128: 52 -> 35 us).  Above it calls take half a millisecond and more and
// the gain counts (36k sites, 5x5x5, 104 -> 104, 49 G: 1100 -> 445 us; 5.2M sites, 3x3x3, 16 -> 16: 3590 -> 2110;
// 700k, 32 -> 64: 1850 -> 570).  The pair path is compared with the fp32 matrix cores on both sides of the line.
static bool split_forward(const ssconv_rulebook* rb, int cin, int cout) {
  return debug_gather_variant() == 13 || (double)rb->n_out * rb->K * cin * cout >= 34359738368.0;
}

// Records the timing-hook events (ssconv_debug_set option 4) around one kernel launch.
struct KernelTimer {
  hipEvent_t start = nullptr, stop = nullptr;
  hipStream_t st;
  bool on;
  explicit KernelTimer(hipStream_t s) : st(s), on(debug_timing_events(&start, &stop)) {
    if (on) (void)hipEventRecord(start, st);
  }
  ~KernelTimer() {
    if (on) (void)hipEventRecord(stop, st);
  }
};

int conv_forward(const void* feats, ssconv_dtype dt, int cin, const ssconv_rulebook* rb, const void* W, int cout,
                 void* out, hipStream_t st, CallScratch* sc, NormSink* sink) {
  if (rb->n_out == 0) return SSCONV_OK;
  // the pair-list path needs its Y buffer; with a fixed scratch region too small for it the
  // output-stationary kernel runs instead (same sums, another order of the fp32 additions)
  const bool pair_fits = !(sc && sc->fixed()) || pair_path_bytes(rb, cin, cout, rb->n_out) <= sc->left();
  if (dt == SSCONV_F32 && pair_fits && pair_path_wins(rb, dt, cin, cout, rb->n_out)) {
    void* ws = nullptr;
    SSC_TRY(scratch_take(sc, &ws, pair_path_bytes(rb, cin, cout, rb->n_out), st));
    int rc;
    {
      KernelTimer timer(st);
      rc = pair_gemm(feats, cin, W, cout, rb, 1, out, rb->n_out, ws, st, sink);
    }
    scratch_give(sc, ws, st);
    return rc;
  }
  if (dt == SSCONV_F32 && split_forward(rb, cin, cout) && use_split(sc, rb->n_in, cin, cout, rb->n_out, rb->K)) {
    SplitFlags flags;
    SSC_TRY(scratch_take(sc, (void**)&flags.w, SplitFlags::kBytes, st));
    int rc = clear_split_flags(flags, st);
    if (rc == SSCONV_OK) {
      KernelTimer timer(st);
      rc = gather_split((const float*)feats, rb->n_in, cin, {(const float*)W, 0, 0}, cout, rb->nbr, rb->n_out, rb->K,
                        (float*)out, flags, flags.feats(), st, sc, SplitPlans::kForward);
      if (rc == SSCONV_OK)
        rc = dispatch_gg<float>(feats, rb->n_in, cin, W, cout, rb->nbr, rb->n_out, rb->K, out, st, nullptr, nullptr,
                                {flags.feats(), flags.kappa(), flags.gathered()});
    }
    scratch_give(sc, flags.w, st);
    return rc;
  }
  if (dt == SSCONV_F32) {
    KernelTimer timer(st);
    return dispatch_gg<float>(feats, rb->n_in, cin, W, cout, rb->nbr, rb->n_out, rb->K, out, st, sc, sink);
  }
  if (use_bf16_kernel(sc, dt, rb->n_in, cin, cout, rb->n_out, rb->K)) {
    KernelTimer timer(st);
    return gather_bf16(feats, rb->n_in, cin, W, false, false, cout, rb->nbr, rb->n_out, rb->K, out, st, sc);
  }
  KernelTimer timer(st);
  return dispatch_gg<uint16_t>(feats, rb->n_in, cin, W, cout, rb->nbr, rb->n_out, rb->K, out, st, sc, sink);
}

// The convolution with the Norm of its output (Sec. 3.3, Eq. 11).  The kernel that writes y also
// leaves its per-channel sums (the fp32 output-stationary kernel per row tile, the pair-list and
// offset-split reduces per row block), so the Norm needs no pass of its own over y before the
// elementwise one; the other paths (the bf16 and split gathers, the generic fallback kernel, an input
// set without rows) leave none and the separate statistics pass runs instead.
int conv_forward_norm(const void* feats, ssconv_dtype dt, int cin, const ssconv_rulebook* rb, const void* W, int cout,
                      const FieldTab& f, double eps, void* y, void* z, hipStream_t st) {
  const int64_t n = rb->n_out;
  if (n == 0) return SSCONV_OK;
  NormSink sink;
  sink.C = cout;
  int rc;
  if (rb->n_in == 0) {
    rc = hipMemsetAsync(y, 0, (size_t)n * cout * dtype_bytes(dt), st) == hipSuccess
             ? SSCONV_OK
             : fail(SSCONV_E_HIP, "clearing the output failed");
  } else {
    rc = conv_forward(feats, dt, cin, rb, W, cout, y, st, nullptr, &sink);
  }
  if (rc == SSCONV_OK && sink.nblk == 0) {
    const NormStatsPlan p = norm_stats_plan(dt, y, n, cout);
    rc = norm_sink_take(&sink, p.nblk, st);
    if (rc == SSCONV_OK) rc = norm_forward_sums(dt, y, n, p, sink.ws, st);
  }
  if (rc == SSCONV_OK) rc = norm_forward_finish(f, dt, y, n, eps, sink.nblk, sink.ws, z, st);
  if (sink.ws) dev_free(sink.ws, st);
  return rc;
}

int dw_nsplit(const ssconv_rulebook* rb) {
  int64_t mx = 0;
  for (int s = 0; s < rb->K; ++s) mx = std::max(mx, rb->pair_off[s + 1] - rb->pair_off[s]);
  int64_t ns = mx / 2048;
  if (ns < 1) ns = 1;
  if (ns > 16) ns = 16;
  return (int)ns;
}

// Bytes of a row as the tile kernel gradient reads it, and of the copy it takes where it cannot be read in place.
static int64_t kgrad_row_bytes(ssconv_dtype dt, int c) {
  return dt == SSCONV_F32 ? split_row_bytes(c) : 2 * (int64_t)(c % 8 == 0 ? c : pad32(c));
}
static size_t kgrad_copy_bytes(ssconv_dtype dt, int64_t n, int c) {
  return dt == SSCONV_BF16 && c % 8 == 0 ? 0 : align256((size_t)n * kgrad_row_bytes(dt, c));
}

// fp32: the tile kernel on split rows against the ring kernel on the fp32 matrix cores, by their times in us
// fitted to measured layers.  Both write and read back the partials.  The ring kernel runs its tasks one or two to
// a SIMD (25 + 4.1 B ps a pair and tile of B blocks of 16 x 16, more where some SIMDs have two tasks and others
// one; a task of few pairs takes 0.15 + 0.018 B us per four of them).  The tile kernel splits the rows first, with
// three launches more, and takes 45 to 170 ps a pair and tile, half as much again where the offsets have fewer
// than four units each and their rows no longer meet in an L2; its launches are 12 us, and 8 more of the host's,
// which is what small calls wait for.  Coefficient gradients, ring and tile kernel, us:
//   80k sites, 3x3x3 (1.4M pairs): 16 -> 16 62 and 98, 71 -> 45 189 and 204, 104 -> 104 324 and 298
//   80k sites, 5x5x5 (4.2M): 24 -> 24 172 and 223, 60 -> 120 674 and 520, 104 -> 104 973 and 790
//   5k sites, 3x3x3 (79k): 16 -> 16 26 and 31, 71 -> 45 58 and 44, 208 -> 208 179 and 149
// (the tenth in favour of the ring kernel is what the fit is good for).  Where each row is gathered a few times
// only the split alone is too much (60 -> 120 channels, 99k pairs of 79k rows: 22 us and 15 for the split against 36
// on the ring kernel; 17k of 1.9k: 9 and 4 against 20).
static bool split_kgrad_wins(const ssconv_rulebook* rb, int cin, int cout) {
  if (rb->n_pairs < 6 * (rb->n_in + rb->n_out)) return false;
  const KgradPlan r = kgrad_plan(rb, SSCONV_F32, cin, cout);
  const KgradTile t = kgrad_tile(rb, 3, cin, cout);
  const double pairs = (double)rb->n_pairs, partial = 8.0 * cin * cout / 4.5e6;
  const double r_units = std::max(rb->K, kgrad_f32_units_want(rb, cin, cout)), t_units = std::max(rb->K, t.units);
  const double r_tiles = r.mtiles * r.ntiles, t_tiles = t.mtiles * t.ntiles, B = r.wmb * r.wnb;
  // sums of more pairs than these in one accumulator lose to the tile kernel's, which are rounded once per 32 pairs
  // (60k sites, 5x5x5, 208 -> 208, 8400 pairs a unit: error 1.7e-6 of the result against 0.9e-6, 4138 and 4150 us)
  if (B > kKgradFoldBlocks && pairs > kKgradRingPairs * r_units) return true;
  const double tasks = r_units * r_tiles, uneven = tasks > 1024 ? std::ceil(tasks / 1024) * 1024 / tasks : 1.0;
  const double ring = std::max(pairs / r_units / 4 * (0.15 + 0.018 * B), pairs * r_tiles * (25 + 4.1 * B) * 1e-6 * uneven) +
                      r_units * partial;
  const double rows = rb->n_in * (4.0 * cin + kgrad_row_bytes(SSCONV_F32, cin)) +
                      rb->n_out * (4.0 * cout + kgrad_row_bytes(SSCONV_F32, cout));
  const double ps = (t.wm * t.wn == 4 ? 45 : t.wm * t.wn == 8 ? 110 : 170) * (t_units < 4 * rb->K ? 1.5 : 1.0);
  const double tile = 20 + rows / 4.5e6 + pairs * t_tiles * ps * 1e-6 + t_units * partial;
  return tile < 0.9 * ring;
}

// The kernel gradient on the bf16 matrix cores: every row offset below 2^31.  Overrides 6 and 12 keep the
// other bf16 kernels (12 where it has the channels in columns), 7 the fp32 one that loads rows into registers.
static bool use_kgrad_tiles(const ssconv_rulebook* rb, ssconv_dtype dt, int cin, int cout) {
  const int64_t v = debug_gather_variant();
  if (dt == SSCONV_F32 && v != 13 && !split_kgrad_wins(rb, cin, cout)) return false;
  if (dt == SSCONV_F32 ? v == 7 : v == 6 || (v == 12 && kgrad_supported(dt, cin, cout))) return false;
  // padding bf16 rows is a launch: not where the generic kernel is done sooner, whose time grows with the longest
  // list (3x3x3: 979 pairs, 48 in the longest list, 71 -> 45: 17.5 us against 21.8, 60 -> 120: 18.7 against 22.2;
  // 360 pairs, all but 60 in one list: 34 against 22 and 28 against 23; 17k and 625, 4 -> 8: 29 against 22)
  if (dt == SSCONV_BF16 && v != 13 && !(cin % 8 == 0 && cout % 8 == 0)) {
    int64_t longest = 0;
    for (int s = 0; s < rb->K; ++s) longest = std::max(longest, rb->pair_off[s + 1] - rb->pair_off[s]);
    if (longest * (cin + cout + 46) < 18000) return false;
  }
  return rb->K <= kKgradMaxK && rb->n_in > 0 && rb->n_out > 0 &&
         rb->n_in * kgrad_row_bytes(dt, cin) < ((int64_t)1 << 31) && rb->n_out * kgrad_row_bytes(dt, cout) < ((int64_t)1 << 31);
}

// The other kernels over work units.
static bool use_kgrad_units(const ssconv_rulebook* rb, ssconv_dtype dt, int cin, int cout) {
  if (dt == SSCONV_F32) return kgrad_f32_units_ok(rb, cin, cout);
  return debug_gather_variant() != 6 && kgrad_supported(dt, cin, cout) && rb->K <= kKgradMaxK &&
         (int64_t)rb->n_in * cin * 2 < ((int64_t)1 << 31) && (int64_t)rb->n_out * cout * 2 < ((int64_t)1 << 31);
}

// Work units of the kernel gradient: slices of about equal length, on the tile kernel (and the bf16 one in
// columns, override 12) launched in the order of the rows, on the fp32 ring kernel enough wavefront tasks for one round of
// the wavefront slots.
static KgradUnits plan_units(const ssconv_rulebook* rb, ssconv_dtype dt, int cin, int cout, bool tiles) {
  if (dt == SSCONV_F32 && !tiles)
    return kgrad_units(rb, kgrad_f32_units_want(rb, cin, cout), kKgradMaxUnitsF32);
  return kgrad_units(rb, kgrad_tile(rb, dt == SSCONV_F32 ? 3 : 1, cin, cout).units, kKgradMaxUnits);
}

int bwd_rows(const void* feats, const void* grad_out, ssconv_dtype dt, int cin, int cout, const ssconv_rulebook* rb,
             char* ws, const BwdLayout& L, BwdRows* r, hipStream_t st) {
  if (!L.tiles) return SSCONV_OK;
  const size_t gb = kgrad_copy_bytes(dt, rb->n_out, cout), fb = kgrad_copy_bytes(dt, rb->n_in, cin);
  uint16_t* gc = gb ? (uint16_t*)(ws + L.rows) : nullptr;
  uint16_t* fc = fb ? (uint16_t*)(ws + L.rows + gb) : nullptr;
  const int64_t ng = gc ? rb->n_out : 0, nf = fc ? rb->n_in : 0;
  int rc;
  const SplitFlags flags{(int*)(ws + L.flags)};
  if (dt == SSCONV_F32)
    rc = split_rows((const float*)grad_out, ng, cout, gc, flags.grad_out(), (const float*)feats, nf, cin, fc,
                    flags.feats(), st);
  else
    rc = pad_rows_bf16((const uint16_t*)grad_out, ng, cout, gc, (const uint16_t*)feats, nf, cin, fc, st);
  const int64_t gs = kgrad_row_bytes(dt, cout), fs = kgrad_row_bytes(dt, cin);
  r->parts = dt == SSCONV_F32 ? 3 : 1;
  r->grad_out = {gc ? gc : grad_out, rb->n_out * gs, (int)gs};
  r->feats = {fc ? fc : feats, rb->n_in * fs, (int)fs};
  r->grad_out_copy = gc;
  return rc;
}

// The kernel of the fp32 feature gradient, by the times that the three are measured to take (the split one from a
// tenth on; 5 us against it and 8 against the pair path for two and four launches more, which take the host's time
// where it is what small calls wait for).  Feature gradients on the fp32 matrix cores, as pairs and split, us:
//   300 sites, 3x3x3: 4 -> 8 channels 11, 18, 15; 32 -> 64 19, 21, 25; 120 -> 60 115, 23, 29; 208 -> 208 85, 39, 43
//   5k sites, 3x3x3, stride 2: 60 -> 120 46, 28, 41; 71 -> 45 92, -, 37
//   20k sites, 3x3x3: 32 -> 64 52, 51, 50; 104 -> 104 161, 158, 89
//   80k sites, 3x3x3: 16 -> 16 44, 67, 55; 5x5x5: 104 -> 104 2210, 1735, 885; 208 -> 208, 20k sites 2121, 1286, 1354
// (-: no pair path).  Generated output sets build the inverse map for all but the pair path.
static auto feats_path(const ssconv_rulebook* rb, int cin, int cout) {
  const int64_t v = debug_gather_variant();
  const bool split = use_split(nullptr, rb->n_out, cout, cin, rb->n_in, rb->K);
  const bool pair = (v == 0 || v == 9 || v == 11 || v == 12) && pair_path_supported(rb, SSCONV_F32, cout, cin);
  if (v == 13) return split ? BwdLayout::kSplit : BwdLayout::kPlain;
  if (v == 9 && pair) return BwdLayout::kPair;
  const double inverse = rb->submanifold ? 0.0 : 4.0 + 0.4e-6 * rb->K * (8.0 * rb->n_in + 4.0 * rb->n_out);
  const double t_plain = plain_us(rb, cout, cin, rb->n_in) + inverse;
  const double t_split = 5.0 + 1.1 * gather_split_us(rb->n_out, cout, cin, rb->n_in, rb->K) + inverse;
  const double t_pair = 8.0 + pair_path_us(rb, cout, cin, rb->n_in);
  if (pair && t_pair < t_plain && (!split || t_pair < t_split)) return BwdLayout::kPair;
  return split && t_split < t_plain ? BwdLayout::kSplit : BwdLayout::kPlain;
}

BwdLayout bwd_layout(const ssconv_rulebook* rb, ssconv_dtype dt, int cin, int cout) {
  BwdLayout L;
  const size_t K = rb->K, sz = dtype_bytes(dt);
  size_t nparts;  // fp32 partial tiles of cout x cin
  L.tiles = use_kgrad_tiles(rb, dt, cin, cout);
  if (L.tiles || use_kgrad_units(rb, dt, cin, cout)) {
    L.units = plan_units(rb, dt, cin, cout, L.tiles);
    nparts = (size_t)L.units.nunits;
  } else {
    L.nsplit = kgrad_supported(dt, cin, cout) ? kgrad_plan(rb, dt, cin, cout).nsplit : dw_nsplit(rb);
    nparts = (size_t)L.nsplit * K;
  }
  size_t o = 0;
  if (rb->n_in > 0 && rb->n_out > 0) {
    if (dt == SSCONV_F32)
      L.feats = feats_path(rb, cin, cout);
    else if (use_bf16_kernel(nullptr, dt, rb->n_out, cout, cin, rb->n_in, rb->K))
      L.feats = BwdLayout::kBf16;
  }
  L.nbrT = o;  // inverse neighbour map: only generated output sets on the gather kernels need one
  if (!rb->submanifold && !L.pair_feats()) o += align256(K * (size_t)rb->n_in * 4);
  L.pair = o;
  if (L.pair_feats()) o += align256(pair_path_bytes(rb, cout, cin, rb->n_in));
  // rows copied for the kernel gradient and behind them the scratch of the feature gradient, which then needs
  // no copy of grad_out of its own
  const size_t gb = L.tiles ? kgrad_copy_bytes(dt, rb->n_out, cout) : 0;
  const size_t fb = L.tiles ? kgrad_copy_bytes(dt, rb->n_in, cin) : 0;
  const size_t scratch = L.feats == BwdLayout::kSplit  ? gather_split_bytes(rb->n_out, cout, cin, rb->n_in, rb->K,
                                                                            SplitPlans::kGradient)
                         : L.feats == BwdLayout::kBf16 ? gather_bf16_bytes(rb->n_out, cout, cin, rb->n_in, rb->K)
                                                       : 0;
  L.rows = o;
  L.gather = o + gb + fb;
  o += std::max(gb, align256(scratch)) + fb;
  L.Wt = o;
  if (L.feats != BwdLayout::kBf16) o += align256(K * (size_t)cin * cout * sz);
  L.split_rows = L.tiles && dt == SSCONV_F32;
  L.flags = o;
  if (L.split_rows || L.feats == BwdLayout::kSplit) o += SplitFlags::kBytes;
  L.part = o;
  o += align256(nparts * cin * cout * 4);
  L.dW = o;
  o += align256(K * (size_t)cin * cout * 4);
  L.total = o;
  return L;
}

// The feature gradient is the gather GEMM over the transposed neighbour map with kappa^T.  For a
// submanifold layer the transposed map is the map itself with the offsets reversed (y = x - d(s)
// holds exactly when x = y - d(K-1-s), d(K-1-s) = -d(s), on the same site set), so it runs on the
// forward map with kappa^T stored in reversed offset order and no inverse map is built.
int conv_backward_feats(const void* grad_out, ssconv_dtype dt, int cin, int cout, const ssconv_rulebook* rb,
                        const void* W, void* grad_feats, char* ws, const BwdLayout& L, const BwdRows& rows,
                        hipStream_t st) {
  if (rb->n_in == 0) return SSCONV_OK;
  if (L.pair_feats()) {
    // kappa^T in the same offset order: the pairs of R_s are walked with their roles swapped
    const int64_t nw = (int64_t)rb->K * cin * cout;
    transpose_kernel<float><<<cdiv(nw, 256), 256, 0, st>>>((const float*)W, rb->K, cout, cin, false,
                                                            (float*)(ws + L.Wt));
    SSC_HIP(hipGetLastError());
    KernelTimer timer(st);
    return pair_gemm(grad_out, cout, ws + L.Wt, cin, rb, 0, grad_feats, rb->n_in, ws + L.pair, st);
  }
  const bool mirror = rb->submanifold != 0;
  const int32_t* nbrT = rb->nbr;
  void* Wt = ws + L.Wt;
  const int K = rb->K;
  if (!mirror) {
    int32_t* inv = (int32_t*)(ws + L.nbrT);
    const int64_t nT = (int64_t)K * rb->n_in;
    fill_i32<<<cdiv(nT, 256), 256, 0, st>>>(inv, nT, -1);
    if (rb->n_out > 0) {
      dim3 gi(cdiv(rb->n_out, 256), K);
      invert_nbr<<<gi, 256, 0, st>>>(rb->nbr, rb->n_out, K, rb->n_in, inv);
    }
    nbrT = inv;
  }
  const int64_t nw = (int64_t)K * cin * cout;
  CallScratch sc;
  sc.base = ws + (rows.parts ? L.gather : L.rows);
  sc.cap = ws + L.Wt - sc.base;
  if (L.feats == BwdLayout::kSplit) {
    const SplitFlags flags{(int*)(ws + L.flags)};
    const OnlyIf only{flags.grad_out(), flags.kappa(), flags.gathered()};
    KernelTimer timer(st);
    SSC_TRY(gather_split((const float*)grad_out, rb->n_out, cout, {(const float*)W, 1, mirror ? 1 : 0}, cin, nbrT,
                         rb->n_in, K, (float*)grad_feats, flags, flags.grad_out(), st, &sc, SplitPlans::kGradient,
                         rows.grad_out_copy, (float*)Wt));
    return dispatch_gg<float>(grad_out, rb->n_out, cout, Wt, cin, nbrT, rb->n_in, K, grad_feats, st, nullptr, nullptr,
                              only);
  }
  if (dt == SSCONV_F32) {
    transpose_kernel<float><<<cdiv(nw, 256), 256, 0, st>>>((const float*)W, K, cout, cin, mirror, (float*)Wt);
    SSC_HIP(hipGetLastError());
    KernelTimer timer(st);
    return dispatch_gg<float>(grad_out, rb->n_out, cout, Wt, cin, nbrT, rb->n_in, K, grad_feats, st);
  }
  if (L.feats == BwdLayout::kBf16) {
    KernelTimer timer(st);
    return gather_bf16(grad_out, rb->n_out, cout, W, true, mirror, cin, nbrT, rb->n_in, K, grad_feats, st, &sc,
                       rows.grad_out_copy);
  }
  transpose_kernel<uint16_t><<<cdiv(nw, 256), 256, 0, st>>>((const uint16_t*)W, K, cout, cin, mirror, (uint16_t*)Wt);
  SSC_HIP(hipGetLastError());
  KernelTimer timer(st);
  return dispatch_gg<uint16_t>(grad_out, rb->n_out, cout, Wt, cin, nbrT, rb->n_in, K, grad_feats, st);
}

int conv_backward_dw(const void* feats, const void* grad_out, ssconv_dtype dt, int cin, int cout,
                     const ssconv_rulebook* rb, const FieldTab& fout, const FieldTab& fin, char* ws,
                     const BwdLayout& L, const BwdRows& rows, float** dW_out, hipStream_t st, hipStream_t* tail) {
  float* part = (float*)(ws + L.part);
  float* dW = (float*)(ws + L.dW);
  *dW_out = dW;
  if (tail) *tail = st;
  const int K = rb->K;
  const int64_t n = (int64_t)K * cin * cout;
  if (L.units.nunits > 0) {
    const KgradUnits& units = L.units;
    if (rows.parts) {
      const SplitFlags flags{rows.parts == 3 ? (int*)(ws + L.flags) : nullptr};
      SSC_TRY(kgrad_tiles(rows.grad_out, rows.feats, rows.parts, cin, cout, rb, kgrad_tile(rb, rows.parts, cin, cout),
                          units, kgrad_order(units), flags, part, st));
      if (rows.parts == 3)  // the same units on the fp32 matrix cores
        SSC_TRY(kgrad_f32(grad_out, feats, cin, cout, rb, units, part, st,
                          {flags.grad_out(), flags.feats(), flags.kgrad()}));
    } else if (dt == SSCONV_F32)
      SSC_TRY(kgrad_f32(grad_out, feats, cin, cout, rb, units, part, st));
    else
      SSC_TRY(kgrad_bf16(grad_out, rb->n_out, feats, rb->n_in, cin, cout, rb, units, kgrad_order(units), part, st));
    hipStream_t rst = st;
    if (tail) {
      SSC_TRY(aux_fork(st, &rst));
      *tail = rst;
    }
    return reduce_units(part, units, cin, cout, fout, fin, dW, rst);
  }
  if (kgrad_supported(dt, cin, cout))
    SSC_TRY(kgrad_partials(grad_out, feats, dt, cin, cout, rb, kgrad_plan(rb, dt, cin, cout), part, st));
  else if (dt == SSCONV_F32)
    SSC_TRY(dispatch_dw<float>(grad_out, cout, feats, cin, rb->pairs, rb->pair_off_dev, K, L.nsplit, part, st));
  else
    SSC_TRY(dispatch_dw<uint16_t>(grad_out, cout, feats, cin, rb->pairs, rb->pair_off_dev, K, L.nsplit, part, st));
  reduce_splits<<<cdiv(n, 256), 256, 0, st>>>(part, L.nsplit, n, fout, fin, K, cin, cout, dW);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

}  // namespace ssconv
