// Feature-Steering of a sparse tensor by a rigid motion (r, t) (Sec. 4.1): every field of order l
// is rotated by its Wigner-D matrix D^l(r) (the block-diagonal rho(r) of Eq. 5, applied as a
// matrix product), every site is taken to the centre of its cell, origin + (x + 1/2) voxel, moved
// to r p + t, and the moved points are re-voxelised with the features of sites that land in one
// cell averaged (the voxelisation of voxel.hip).  The centre and the moved point are computed in
// fp32 with every product and sum rounded to nearest in a fixed order, because they decide the
// integer cells.
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace ssconv {

void wigner_d(int l, const double* r, double* D);

namespace {

constexpr int kDFloats = 1 + 9 + 25 + 49 + 81;  // D^0 .. D^4, row-major, concatenated

struct SteerArgs {
  FieldTab f;
  float D[kDFloats];
  float r[9], t[3], origin[3], voxel;
};

__host__ __device__ constexpr int d_offset(int l) { return l == 0 ? 0 : l == 1 ? 1 : l == 2 ? 10 : l == 3 ? 35 : 84; }

// Site i's moved cell centre and its batch index.
__device__ __forceinline__ void move_site(const SteerArgs& a, const int32_t* __restrict__ coords, int64_t i,
                                          float* __restrict__ pts, int32_t* __restrict__ batch) {
  const int4 c = reinterpret_cast<const int4*>(coords)[i];
  const float p[3] = {__fadd_rn(__fmul_rn(__fadd_rn((float)c.y, 0.5f), a.voxel), a.origin[0]),
                      __fadd_rn(__fmul_rn(__fadd_rn((float)c.z, 0.5f), a.voxel), a.origin[1]),
                      __fadd_rn(__fmul_rn(__fadd_rn((float)c.w, 0.5f), a.voxel), a.origin[2])};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float s = __fadd_rn(__fadd_rn(__fmul_rn(a.r[3 * k], p[0]), __fmul_rn(a.r[3 * k + 1], p[1])),
                              __fmul_rn(a.r[3 * k + 2], p[2]));
    pts[3 * i + k] = __fadd_rn(s, a.t[k]);
  }
  batch[i] = c.x;
}

__device__ __forceinline__ int field_entry(const FieldTab& t, int field) {
  int e = 0;
  while (e + 1 < t.n && field >= t.f0[e + 1]) ++e;
  return e;
}

// y = D x for one field of d components (x and y may be the same).
template <int d>
__device__ __forceinline__ void rotate_field(const float* D, const float* x, float* y) {
  float v[d];
#pragma unroll
  for (int k = 0; k < d; ++k) v[k] = x[k];
#pragma unroll
  for (int r = 0; r < d; ++r) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < d; ++k) s = fmaf(D[r * d + k], v[k], s);
    y[r] = s;
  }
}
__device__ __forceinline__ void rotate_any(int l, const float* D, const float* x, float* y) {
  D += d_offset(l);
  switch (l) {
    case 0: return rotate_field<1>(D, x, y);
    case 1: return rotate_field<3>(D, x, y);
    case 2: return rotate_field<5>(D, x, y);
    case 3: return rotate_field<7>(D, x, y);
    default: return rotate_field<9>(D, x, y);
  }
}

// Whole rows through LDS: both directions of memory in 16-byte pieces, the fields (one thread each)
// rotated in place, the matrices in LDS too; the workgroup also moves its sites.  Bandwidth-bound:
// a thread per field that addressed memory itself stepped 3 or 5 elements per lane and kept its
// components in private memory (38k sites of 104 channels: 24 + 4 us in two launches, now 22 in one).
constexpr int kSteerNT = 256;
constexpr int kSteerLds = 32 << 10;  // five workgroups of a compute unit
constexpr int kSteerRows = 4;        // rows of a workgroup are a multiple of this (4 floats = 16 bytes)

inline int64_t steer_head_bytes(const FieldTab& t) { return (kDFloats * 4 + 4 + t.f0[t.n] * 8 + 15) / 16 * 16; }

// Rows of a workgroup, 0 when even the smallest number needs more LDS than kSteerLds; few rows are
// spread over two workgroups per compute unit.
inline int steer_rows(const FieldTab& t, int64_t n) {
  const int64_t row = (int64_t)t.ch0[t.n] * 4 * kSteerRows, room = kSteerLds - steer_head_bytes(t);
  const int64_t fit = room < row || row == 0 ? 0 : room / row, want = (n + 512 * kSteerRows - 1) / (512 * kSteerRows);
  return (int)std::min<int64_t>(std::min(fit, want), kSteerNT / kSteerRows) * kSteerRows;
}

__global__ __launch_bounds__(kSteerNT) void steer_rows_kernel(SteerArgs a, const int32_t* __restrict__ coords,
                                                              const float* __restrict__ f, int64_t n, int rows,
                                                              float* __restrict__ pts, int32_t* __restrict__ batch,
                                                              float* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int nf = a.f.f0[a.f.n], C = a.f.ch0[a.f.n], tid = threadIdx.x;
  float* D = reinterpret_cast<float*>(lds);
  int2* tab = reinterpret_cast<int2*>(lds + kDFloats * 4 + 4);  // (first channel, order) of each field
  float* xs = reinterpret_cast<float*>(lds + (kDFloats * 4 + 4 + nf * 8 + 15) / 16 * 16);
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  const int m = (int)(n - r0 < rows ? n - r0 : rows), cnt = m * C;
  const float* src = f + r0 * C;
  float* dst = out + r0 * C;
  for (int i = tid; i < cnt / 4; i += kSteerNT) reinterpret_cast<float4*>(xs)[i] = reinterpret_cast<const float4*>(src)[i];
  for (int i = cnt / 4 * 4 + tid; i < cnt; i += kSteerNT) xs[i] = src[i];
  if (tid < kDFloats) D[tid] = a.D[tid];
  for (int q = tid; q < nf; q += kSteerNT) {
    const int e = field_entry(a.f, q), l = a.f.l[e];
    tab[q] = make_int2(a.f.ch0[e] + (q - a.f.f0[e]) * (2 * l + 1), l);
  }
  if (tid < m) move_site(a, coords, r0 + tid, pts, batch);
  __syncthreads();
  for (uint32_t i = tid; i < (uint32_t)(m * nf); i += kSteerNT) {
    const uint32_t row = i / (uint32_t)nf;
    const int2 t = tab[i - row * nf];
    float* x = xs + row * C + t.x;
    rotate_any(t.y, D, x, x);
  }
  __syncthreads();
  for (int i = tid; i < cnt / 4; i += kSteerNT) reinterpret_cast<float4*>(dst)[i] = reinterpret_cast<const float4*>(xs)[i];
  for (int i = cnt / 4 * 4 + tid; i < cnt; i += kSteerNT) dst[i] = xs[i];
}

// Rows too wide for LDS, and features off a 16-byte boundary: a thread per site, and one per
// (site, field).
__global__ void steer_points_kernel(SteerArgs a, const int32_t* __restrict__ coords, int64_t n,
                                    float* __restrict__ pts, int32_t* __restrict__ batch) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) move_site(a, coords, i, pts, batch);
}

__global__ void steer_rotate_kernel(SteerArgs a, const float* __restrict__ f, int64_t n, float* __restrict__ out) {
  const int n_fields = a.f.f0[a.f.n], C = a.f.ch0[a.f.n];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * n_fields) return;
  const int64_t row = i / n_fields;
  const int field = (int)(i - row * n_fields), e = field_entry(a.f, field), l = a.f.l[e];
  const int64_t at = row * C + a.f.ch0[e] + (field - a.f.f0[e]) * (2 * l + 1);
  rotate_any(l, a.D, f + at, out + at);
}

}  // namespace
}  // namespace ssconv

using namespace ssconv;

extern "C" int ssconv_steer(const int32_t* coords, const float* feats, int64_t n, const ssconv_fields* fields,
                            const double* rot, const double* trans, const float* origin, float voxel,
                            const int32_t* grid, int nbatch, int32_t* coords_out, float* feats_out,
                            int32_t* site_row, int64_t* n_sites, hipStream_t stream) {
  if (!rot || !trans || !origin || !grid || !n_sites) return fail(SSCONV_E_INVALID, "NULL host argument");
  *n_sites = 0;
  SteerArgs a;
  SSC_TRY(make_fieldtab(fields, &a.f));
  const int C = a.f.ch0[a.f.n];
  // r must be a proper rotation (orthonormal, det +1)
  double dev = 0.0;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double s = 0.0;
      for (int k = 0; k < 3; ++k) s += rot[3 * i + k] * rot[3 * j + k];
      dev = std::max(dev, std::fabs(s - (i == j ? 1.0 : 0.0)));
    }
  const double det = rot[0] * (rot[4] * rot[8] - rot[5] * rot[7]) - rot[1] * (rot[3] * rot[8] - rot[5] * rot[6]) +
                     rot[2] * (rot[3] * rot[7] - rot[4] * rot[6]);
  if (!(dev < 1e-6) || !(std::fabs(det - 1.0) < 1e-6)) return fail(SSCONV_E_INVALID, "rot is not a rotation");
  for (int k = 0; k < 3; ++k)
    if (!std::isfinite(trans[k])) return fail(SSCONV_E_INVALID, "trans must be finite");
  if (n < 0 || n > 0x7fffffffll) return fail(SSCONV_E_INVALID, "n must be in [0, 2^31)");
  if (n > 0 && (!coords || !feats || !aligned16(coords))) return fail(SSCONV_E_INVALID, "bad coords / feats");
  for (int l = 0; l <= SSCONV_MAX_L; ++l) {
    // matrices of absent orders stay zero and unread
    if (std::find(a.f.l, a.f.l + a.f.n, l) == a.f.l + a.f.n) {
      std::fill(a.D + d_offset(l), a.D + d_offset(l) + (2 * l + 1) * (2 * l + 1), 0.f);
      continue;
    }
    double D[81];
    wigner_d(l, rot, D);
    for (int k = 0; k < (2 * l + 1) * (2 * l + 1); ++k) a.D[d_offset(l) + k] = (float)D[k];
  }
  for (int k = 0; k < 9; ++k) a.r[k] = (float)rot[k];
  for (int k = 0; k < 3; ++k) {
    a.t[k] = (float)trans[k];
    a.origin[k] = origin[k];
  }
  a.voxel = voxel;
  if (n == 0) return ssconv_voxelize(nullptr, nullptr, nullptr, 0, C, origin, voxel, grid, nbatch, coords_out,
                                     feats_out, site_row, n_sites, stream);
  char* ws = nullptr;
  const size_t o_pts = 0, o_b = (n * 12 + 255) & ~(size_t)255, o_f = o_b + ((n * 4 + 255) & ~(size_t)255);
  SSC_TRY(dev_alloc((void**)&ws, o_f + (size_t)n * C * 4 + 256, stream));
  float* pts = (float*)(ws + o_pts);
  int32_t* bat = (int32_t*)(ws + o_b);
  float* rf = (float*)(ws + o_f);
  const int64_t work = n * a.f.f0[a.f.n];
  const int rows = aligned16(feats) ? steer_rows(a.f, n) : 0;
  if (rows) {
    steer_rows_kernel<<<cdiv(n, rows), kSteerNT, steer_head_bytes(a.f) + (int64_t)rows * C * 4, stream>>>(
        a, coords, feats, n, rows, pts, bat, rf);
  } else {
    steer_points_kernel<<<cdiv(n, 256), 256, 0, stream>>>(a, coords, n, pts, bat);
    if (work > 0) steer_rotate_kernel<<<cdiv(work, 256), 256, 0, stream>>>(a, feats, n, rf);
  }
  int rc = SSCONV_OK;
  if (hipGetLastError() != hipSuccess) rc = fail(SSCONV_E_HIP, "steering launch failed");
  if (rc == SSCONV_OK)
    rc = ssconv_voxelize(pts, bat, rf, n, C, origin, voxel, grid, nbatch, coords_out, feats_out, site_row, n_sites,
                         stream);
  dev_free(ws, stream);
  return rc;
}
