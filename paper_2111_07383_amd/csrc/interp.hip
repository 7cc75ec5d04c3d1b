// Tensor-to-Point: trilinear interpolation of a sparse tensor at points, and its adjoint (Sec. 4.1
// interpolates point-wise features from the sparse backbone maps).
//
// The features live at the cell centres origin + (x + 1/2) voxel of the active sites and are zero
// elsewhere; a point is the trilinear blend of the 8 site centres around it.  With
// u = (p - origin) / voxel - 1/2 (fp32, rounded to nearest in that order: floor(u) decides which
// sites are read), x0 = floor(u), w = u - x0, corner x0 + c (c in {0,1}^3, index 4 cx + 2 cy + cz)
// has weight prod_a (c_a ? w_a : 1 - w_a).  Corners are found in the rule book's coordinate hash;
// corners outside the grid or inactive contribute nothing, and points never read sites of
// another batch entry.  The backward pass is the exact adjoint, deterministic: the (point,
// corner) entries of every site are bucketed (integer-atomic counts, whose returned values are the
// entries' slots in their buckets, a scan, a plain scatter), each bucket is sorted by entry index,
// and every site adds weight * grad over its bucket in that order.
#include <algorithm>
#include <cmath>

#include "hash.hpp"
#include "bucket_sort.hpp"
#include "gather_tile.hpp"
#include "scan.hpp"

namespace ssconv {
namespace {

// Entry e = 8 * point + corner: its site row (or -1) and weight, one thread each, so that eight
// times as many hash probes are in flight and the stores are whole lines (a thread per point that
// did its eight corners in turn: 22 us for 151k points, now 12.5).  COUNT: also counts the
// entries of every site and gives each its slot among them (any order: the buckets are sorted).
// Counting is bound by the atomics on memory, about 37 per ns; points that neighbour each other
// share sites, so a workgroup counts in LDS first, in a table keyed by the site (256 entries never
// fill 512 slots), and adds each site's count once (23 + 31 us in two passes, 42 in one, 25 so).
constexpr int kCountSlots = 512;

template <bool COUNT>
__global__ __launch_bounds__(256) void interp_corners_kernel(const float* __restrict__ pts,
                                                             const int32_t* __restrict__ batch, int64_t ne, float ox,
                                                             float oy, float oz, float voxel, int g0, int g1, int g2,
                                                             int bmax, const uint64_t* __restrict__ slots,
                                                             uint64_t mask, int32_t* __restrict__ rows,
                                                             float* __restrict__ wts, int32_t* __restrict__ cnt,
                                                             int32_t* __restrict__ slot) {
  __shared__ int s_site[COUNT ? kCountSlots : 1], s_num[COUNT ? kCountSlots : 1];
  if constexpr (COUNT) {
    for (int t = threadIdx.x; t < kCountSlots; t += 256) s_site[t] = -1, s_num[t] = 0;
    __syncthreads();
  }
  const int64_t e = (int64_t)xcd_slot(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  const int64_t i = min(e, ne - 1) >> 3;  // ne is a multiple of 8: the last point
  const int k = (int)e & 7;
  const float o[3] = {ox, oy, oz};
  const int g[3] = {g0, g1, g2};
  float w = 1.f;
  int x[3];
  bool ok = e < ne;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float u = __fsub_rn(__fdiv_rn(__fsub_rn(pts[3 * i + a], o[a]), voxel), 0.5f);
    ok = ok && isfinite(u) && fabsf(u) < 1e9f;
    const float f = floorf(u), wa = __fsub_rn(u, f);  // exact: u - floor(u)
    const int ca = (k >> (2 - a)) & 1;
    x[a] = (ok ? (int)f : 0) + ca;
    ok = ok && x[a] >= 0 && x[a] < g[a];
    const float v = ca ? wa : 1.f - wa;
    w = a == 0 ? v : w * v;
  }
  const int b = batch ? batch[i] : 0;
  ok = ok && b >= 0 && b <= bmax;  // larger b would wrap the 32-bit key onto other sites
  const int r = ok ? hash_find(slots, mask, site_key(b, x[0], x[1], x[2], g0, g1, g2)) : -1;
  if (e < ne) {
    rows[e] = r;
    wts[e] = w;
  }
  if constexpr (COUNT) {
    int h = 0, mine = 0;
    if (r >= 0) {
      h = (int)(mix32((uint32_t)r) & (kCountSlots - 1));
      for (;;) {
        const int was = atomicCAS(&s_site[h], -1, r);
        if (was == -1 || was == r) break;
        h = (h + 1) & (kCountSlots - 1);
      }
      mine = atomicAdd(&s_num[h], 1);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kCountSlots; t += 256)
      if (s_site[t] >= 0) s_num[t] = atomicAdd(&cnt[s_site[t]], s_num[t]);
    __syncthreads();
    if (r >= 0) slot[e] = s_num[h] + mine;
  }
}

// The row and first channel of this thread's V channels: threads take (row, channel group) in
// order, and the workgroups of one XCD a contiguous range of rows, so that the rows which
// neighbouring points or sites share stay in that XCD's L2.
template <int V>
__device__ __forceinline__ bool row_group(int64_t m, int C, int64_t* row, int* c) {
  const uint32_t nv = (uint32_t)(C / V);
  const int64_t e0 = (int64_t)xcd_slot(blockIdx.x, gridDim.x) * 256, i0 = e0 / nv;  // the same in all lanes
  const uint32_t off = (uint32_t)(e0 - i0 * nv) + threadIdx.x, q = off / nv;
  *row = i0 + q;
  *c = (int)(off - q * nv) * V;
  return *row < m;
}

template <int V>
struct Chans {
  float v[V];
};
template <int V>
__device__ __forceinline__ Chans<V> load_chans(const float* __restrict__ p) {
  Chans<V> r;
  if constexpr (V == 4) {
    const float4 f = *reinterpret_cast<const float4*>(p);
    r.v[0] = f.x, r.v[1] = f.y, r.v[2] = f.z, r.v[3] = f.w;
  } else {
    r.v[0] = p[0];
  }
  return r;
}
template <int V>
__device__ __forceinline__ void store_chans(float* __restrict__ p, const float (&s)[V]) {
  if constexpr (V == 4)
    *reinterpret_cast<float4*>(p) = make_float4(s[0], s[1], s[2], s[3]);
  else
    p[0] = s[0];
}

// out[i][c..c+V) = sum over the corners, in corner order, of weight * feats[row][c..c+V)
// (V = 4 with 16-byte accesses when C % 4 == 0).  Bound by the L2: all eight rows are loaded
// before the first is used (an absent corner loads row 0 and leaves the sum alone), and the rows
// stay in one XCD (104 channels, 151k points: 56 -> 32 us).
template <int V>
__global__ __launch_bounds__(256) void interp_fwd_kernel(const float* __restrict__ feats, int C,
                                                         const int32_t* __restrict__ rows,
                                                         const float* __restrict__ wts, int64_t m,
                                                         float* __restrict__ out) {
  int64_t i;
  int c;
  if (!row_group<V>(m, C, &i, &c)) return;
  int r[8];
  float w[8];
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // the tables start on 256 bytes
    const int4 rv = reinterpret_cast<const int4*>(rows)[i * 2 + h];
    const float4 wv = reinterpret_cast<const float4*>(wts)[i * 2 + h];
    r[4 * h] = rv.x, r[4 * h + 1] = rv.y, r[4 * h + 2] = rv.z, r[4 * h + 3] = rv.w;
    w[4 * h] = wv.x, w[4 * h + 1] = wv.y, w[4 * h + 2] = wv.z, w[4 * h + 3] = wv.w;
  }
  Chans<V> f[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) f[k] = load_chans<V>(feats + (int64_t)max(r[k], 0) * C + c);
  float s[V];
#pragma unroll
  for (int v = 0; v < V; ++v) s[v] = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int v = 0; v < V; ++v) s[v] = r[k] >= 0 ? fmaf(w[k], f[k].v[v], s[v]) : s[v];
  store_chans<V>(out + i * C + c, s);
}

// Bucket fill: entry e = 8 * point + corner goes to slot slot[e] of its site's bucket (the order
// inside a bucket is that of the atomics, sorted afterwards).
__global__ void interp_fill_kernel(const int32_t* __restrict__ rows, int64_t ne, const int64_t* __restrict__ start,
                                   const int32_t* __restrict__ slot, int32_t* __restrict__ ent) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne) return;
  const int32_t r = rows[e];
  if (r >= 0) ent[start[r] + slot[e]] = (int32_t)e;
}

// grad_feats[r][c..c+V) = sum over the sorted bucket of weight * grad[point][c..c+V); every site
// row written (V = 4 with 16-byte accesses when C % 4 == 0).  kBwdAhead entries are loaded before
// the first is used (past the bucket's end its last entry again, which leaves the sum alone): a
// bucket is a chain of entry -> weight and gradient otherwise, ~32 entries long (104 channels, 38k sites: 61 -> 38 us).
constexpr int kBwdAhead = 8;

template <int V>
__global__ __launch_bounds__(256) void interp_bwd_kernel(const float* __restrict__ grad, int C,
                                                         const float* __restrict__ wts,
                                                         const int64_t* __restrict__ start,
                                                         const int32_t* __restrict__ cnt,
                                                         const int32_t* __restrict__ ent, int64_t n,
                                                         float* __restrict__ gf) {
  int64_t r;
  int c;
  if (!row_group<V>(n, C, &r, &c)) return;
  const int32_t* a = ent + start[r];
  const int mcount = cnt[r];
  float s[V];
#pragma unroll
  for (int v = 0; v < V; ++v) s[v] = 0.f;
  for (int j = 0; j < mcount; j += kBwdAhead) {
    int32_t en[kBwdAhead];
    float w[kBwdAhead];
    Chans<V> g[kBwdAhead];
#pragma unroll
    for (int q = 0; q < kBwdAhead; ++q) en[q] = a[min(j + q, mcount - 1)];
#pragma unroll
    for (int q = 0; q < kBwdAhead; ++q) {
      w[q] = wts[en[q]];
      g[q] = load_chans<V>(grad + (int64_t)(en[q] >> 3) * C + c);
    }
#pragma unroll
    for (int q = 0; q < kBwdAhead; ++q)
#pragma unroll
      for (int v = 0; v < V; ++v) s[v] = j + q < mcount ? fmaf(w[q], g[q].v[v], s[v]) : s[v];
  }
  store_chans<V>(gf + r * C + c, s);
}

int interp_args(ssconv_rulebook_t rb, int C, const float* points, int64_t m, const float* origin, float voxel) {
  if (!rb) return fail(SSCONV_E_INVALID, "NULL rule book");
  SSC_TRY(rulebook_settle(rb));
  if (C < 1) return fail(SSCONV_E_INVALID, "channels must be positive");
  if (m < 0 || m > 0x0fffffffll) return fail(SSCONV_E_INVALID, "m must be in [0, 2^28)");
  if (!origin || !(voxel > 0.f) || !std::isfinite(voxel)) return fail(SSCONV_E_INVALID, "bad origin / voxel");
  for (int a = 0; a < 3; ++a)
    if (!std::isfinite(origin[a])) return fail(SSCONV_E_INVALID, "origin must be finite");
  if (m > 0 && !points) return fail(SSCONV_E_INVALID, "NULL points");
  return SSCONV_OK;
}

// Fills the corner table: rows [m*8] int32 (site row or -1) and weights [m*8] fp32; with cnt also
// the entries per site and every entry's slot among them.
void launch_corners(ssconv_rulebook_t rb, const float* points, const int32_t* batch, int64_t m, const float* origin,
                    float voxel, int32_t* rows, float* wts, int32_t* cnt, int32_t* slot, hipStream_t st) {
  // the largest batch index whose keys fit 32 bits (key ~0 is reserved), as in the rule book
  const int64_t cells = (int64_t)rb->grid[0] * rb->grid[1] * rb->grid[2];
  const int bmax = (int)std::min<int64_t>(0xFFFFFFFFll / cells - 1, 0x7fffffff);
  auto* kernel = cnt ? interp_corners_kernel<true> : interp_corners_kernel<false>;
  kernel<<<cdiv(m * 8, 256), 256, 0, st>>>(points, batch, m * 8, origin[0], origin[1], origin[2], voxel, rb->grid[0],
                                           rb->grid[1], rb->grid[2], bmax, rb->hash_in, (uint64_t)(rb->cap_in - 1),
                                           rows, wts, cnt, slot);
}

}  // namespace
}  // namespace ssconv

using namespace ssconv;

extern "C" int ssconv_interpolate(ssconv_rulebook_t rb, const float* feats, int channels, const float* points,
                                  const int32_t* batch, int64_t m, const float* origin, float voxel, float* out,
                                  hipStream_t stream) {
  SSC_TRY(interp_args(rb, channels, points, m, origin, voxel));
  if (m == 0) return SSCONV_OK;
  if (!out || (rb->n_in > 0 && !feats)) return fail(SSCONV_E_INVALID, "NULL feature buffer");
  if (rb->n_in == 0) {
    SSC_HIP(hipMemsetAsync(out, 0, (size_t)m * channels * 4, stream));
    return SSCONV_OK;
  }
  char* ws = nullptr;
  const size_t o_w = ((size_t)m * 32 + 255) & ~(size_t)255;
  SSC_TRY(dev_alloc((void**)&ws, o_w + (size_t)m * 32, stream));
  int32_t* rows = (int32_t*)ws;
  float* wts = (float*)(ws + o_w);
  launch_corners(rb, points, batch, m, origin, voxel, rows, wts, nullptr, nullptr, stream);
  if (channels % 4 == 0 && aligned16(feats) && aligned16(out))
    interp_fwd_kernel<4><<<cdiv(m * channels / 4, 256), 256, 0, stream>>>(feats, channels, rows, wts, m, out);
  else
    interp_fwd_kernel<1><<<cdiv(m * channels, 256), 256, 0, stream>>>(feats, channels, rows, wts, m, out);
  int rc = SSCONV_OK;
  if (hipGetLastError() != hipSuccess) rc = fail(SSCONV_E_HIP, "interpolation launch failed");
  dev_free(ws, stream);
  return rc;
}

extern "C" int ssconv_interpolate_backward(ssconv_rulebook_t rb, const float* grad, int channels, const float* points,
                                           const int32_t* batch, int64_t m, const float* origin, float voxel,
                                           float* grad_feats, hipStream_t stream) {
  SSC_TRY(interp_args(rb, channels, points, m, origin, voxel));
  const int64_t n = rb->n_in;
  if (n == 0) return SSCONV_OK;
  if (!grad_feats || (m > 0 && !grad)) return fail(SSCONV_E_INVALID, "NULL gradient buffer");
  if (m == 0) {
    SSC_HIP(hipMemsetAsync(grad_feats, 0, (size_t)n * channels * 4, stream));
    return SSCONV_OK;
  }
  const int64_t ne = m * 8;
  auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
  const size_t o_w = up(ne * 4), o_cnt = o_w + up(ne * 4), o_big = o_cnt + up(n * 4);  // cnt, big: one fill
  const size_t o_fill = o_big + up((n + 1) * 4), o_start = o_fill + up(ne * 4);
  const size_t o_ent = o_start + up(n * 8), o_tmp = o_ent + up(ne * 4);
  const size_t total = o_tmp + up((size_t)(scan_tmp_elems(n) + 1) * 8);
  char* ws = nullptr;
  SSC_TRY(dev_alloc((void**)&ws, total, stream));
  int32_t* rows = (int32_t*)ws;
  float* wts = (float*)(ws + o_w);
  int32_t* cnt = (int32_t*)(ws + o_cnt);
  int32_t* slot = (int32_t*)(ws + o_fill);  // each entry's slot in its site's bucket
  int64_t* start = (int64_t*)(ws + o_start);
  int32_t* ent = (int32_t*)(ws + o_ent);
  int64_t* tmp = (int64_t*)(ws + o_tmp);
  int32_t* big = (int32_t*)(ws + o_big);
  auto run = [&]() -> int {
    SSC_HIP(hipMemsetAsync(cnt, 0, o_big - o_cnt + 256, stream));
    launch_corners(rb, points, batch, m, origin, voxel, rows, wts, cnt, slot, stream);
    SSC_TRY(exclusive_scan(cnt, n, start, tmp + scan_tmp_elems(n), tmp, stream));
    interp_fill_kernel<<<cdiv(ne, 256), 256, 0, stream>>>(rows, ne, start, slot, ent);
    SSC_TRY(sort_buckets(nullptr, n, n, start, cnt, ent, big, false, stream));
    if (channels % 4 == 0 && aligned16(grad) && aligned16(grad_feats))
      interp_bwd_kernel<4><<<cdiv(n * channels / 4, 256), 256, 0, stream>>>(grad, channels, wts, start, cnt, ent, n,
                                                                            grad_feats);
    else
      interp_bwd_kernel<1><<<cdiv(n * channels, 256), 256, 0, stream>>>(grad, channels, wts, start, cnt, ent, n,
                                                                        grad_feats);
    SSC_HIP(hipGetLastError());
    return SSCONV_OK;
  };
  const int rc = run();
  dev_free(ws, stream);
  return rc;
}
