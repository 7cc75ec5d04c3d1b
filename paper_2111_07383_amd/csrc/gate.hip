// Gated nonlinearity (Sec. 3.3, Eq. 12): ReLU on scalar fields, Sigmoid(gate) * f on
// fields of order l > 0, the gate being an extra scalar channel of the producing
// convolution (one per l > 0 field, appended after the fields in field order).
// Elementwise and bandwidth-bound.  One thread per (site, field) addressing memory itself reaches
// a fifth of the memory's rate: a field of order 2 makes a lane step over 5 elements, so a wave
// touches every cache line several times in pieces of 2 or 4 bytes.  The kernels below take whole
// rows through LDS instead, in 16-byte pieces in both directions, and only the arithmetic is by
// (site, field); the results are the same bits.  Measured: 208 + 48 bf16 channels on eight objects
// of a 64^3 grid 22 -> 17 us; 120 + 24 fp32 channels on 32 sparse objects 20 -> 11 us forward and
// 20 -> 14 us backward (what is left is launch, one round trip to memory and the division by field).
#include "common.hpp"

namespace ssconv {
namespace {

struct GateTab {
  FieldTab f;
  int gate0[SSCONV_MAX_ENTRIES];  // gate index of the first field of each entry (l > 0 entries)
  int C, G, n_fields;
};

__device__ __forceinline__ int find_entry(const FieldTab& t, int field) {
  int e = 0;
  while (e + 1 < t.n && field >= t.f0[e + 1]) ++e;
  return e;
}

__device__ __forceinline__ float sigmoidf(float x) { return 1.f / (1.f + __expf(-x)); }

template <typename T>
__global__ void gate_fwd_kernel(GateTab t, const T* __restrict__ x, int64_t n, T* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * t.n_fields) return;
  const int64_t row = i / t.n_fields;
  const int field = (int)(i % t.n_fields);
  const int e = find_entry(t.f, field), l = t.f.l[e], d = 2 * l + 1;
  const int c0 = t.f.ch0[e] + (field - t.f.f0[e]) * d;
  const T* xr = x + row * (t.C + t.G);
  T* yr = y + row * t.C;
  if (l == 0) {
    const float v = DT<T>::to_f(xr[c0]);
    yr[c0] = DT<T>::from_f(v > 0.f ? v : 0.f);
  } else {
    const float sg = sigmoidf(DT<T>::to_f(xr[t.C + t.gate0[e] + field - t.f.f0[e]]));
    for (int c = 0; c < d; ++c) yr[c0 + c] = DT<T>::from_f(sg * DT<T>::to_f(xr[c0 + c]));
  }
}

template <typename T>
__global__ void gate_bwd_kernel(GateTab t, const T* __restrict__ x, const T* __restrict__ dy, int64_t n,
                                T* __restrict__ dx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * t.n_fields) return;
  const int64_t row = i / t.n_fields;
  const int field = (int)(i % t.n_fields);
  const int e = find_entry(t.f, field), l = t.f.l[e], d = 2 * l + 1;
  const int c0 = t.f.ch0[e] + (field - t.f.f0[e]) * d;
  const T* xr = x + row * (t.C + t.G);
  const T* dyr = dy + row * t.C;
  T* dxr = dx + row * (t.C + t.G);
  if (l == 0) {
    const float v = DT<T>::to_f(xr[c0]);
    dxr[c0] = DT<T>::from_f(v > 0.f ? DT<T>::to_f(dyr[c0]) : 0.f);
  } else {
    const int gc = t.C + t.gate0[e] + field - t.f.f0[e];
    const float sg = sigmoidf(DT<T>::to_f(xr[gc]));
    float dot = 0.f;
    for (int c = 0; c < d; ++c) {
      const float g = DT<T>::to_f(dyr[c0 + c]);
      dot = fmaf(g, DT<T>::to_f(xr[c0 + c]), dot);
      dxr[c0 + c] = DT<T>::from_f(g * sg);
    }
    dxr[gc] = DT<T>::from_f(dot * sg * (1.f - sg));
  }
}

// Staged rows.  A workgroup's rows are one contiguous range of x, dy and the result, a multiple of
// 8 rows, so every range starts 16-byte aligned when the arrays do.
constexpr int kGateNT = 256;
constexpr int kGateLds = 32 << 10;  // five workgroups of a compute unit
constexpr int kGateRows = 8;        // rows of a workgroup are a multiple of this (8 bf16 = 16 bytes)

// Bytes of the tables and of the rows of one workgroup (x and, behind it, y or dy).
inline int64_t gate_tab_bytes(const GateTab& t) { return (t.n_fields * 8 + 15) / 16 * 16; }
inline int64_t gate_row_bytes(const GateTab& t, int64_t es) { return (2 * t.C + t.G) * es; }

// Rows of a workgroup, 0 when even the smallest number needs more LDS than kGateLds or the rows are too few: staging
// is two more round trips and barriers, and a workgroup of 8 wide rows has many fields for its 256 threads.  Few rows
// are spread over at least two workgroups per compute unit where there are enough.  By field and staged, forward, us:
//   fp32: 28 fields, 40k rows 10.6 and 9.0, 3k rows 4.1 and 3.8; 80 fields, 40k rows 28 and 19, 100 rows 4.0 and 4.8
//   bf16: 28 fields, 40k rows 10.1 and 12.1, 300k rows 61 and 44; 280 fields, 3k rows 7.5 and 10.5, 100 rows 4.1 and
//   9.5, 40k rows 73 and 46
//   scalars alone, which are addressed in order anyway: 5, 300k rows 5.6 and 6.3; 64, 40k rows 7.8 and 7.7, 300k 46
//   and 32
// Override 13 stages any number.
inline int gate_rows(const GateTab& t, int64_t es, int64_t n) {
  const int64_t line = t.G == 0 ? 4000000 : es == 4 ? 1000000 : 2000000;
  if (n * t.n_fields < line && debug_gather_variant() != 13) return 0;
  const int64_t fit = (kGateLds - gate_tab_bytes(t)) / (gate_row_bytes(t, es) * kGateRows);
  if (kGateLds < gate_tab_bytes(t) || fit < 1) return 0;
  const int64_t want = (n + 512 * kGateRows - 1) / (512 * kGateRows);
  return (int)(fit < want ? fit : want) * kGateRows;
}

// tab[f] = (first channel, components | gate channel << 8) of field f.
__device__ __forceinline__ void gate_fields_table(const GateTab& t, int2* tab) {
  for (int f = threadIdx.x; f < t.n_fields; f += kGateNT) {
    const int e = find_entry(t.f, f), d = 2 * t.f.l[e] + 1;
    tab[f] = make_int2(t.f.ch0[e] + (f - t.f.f0[e]) * d, d | (t.C + t.gate0[e] + f - t.f.f0[e]) << 8);
  }
}

// cnt elements between LDS and memory, both 16-byte aligned.
template <typename T>
__device__ __forceinline__ void copy_elems(T* __restrict__ dst, const T* __restrict__ src, int cnt) {
  constexpr int V = 16 / sizeof(T);
  const int nv = cnt / V;
  for (int i = threadIdx.x; i < nv; i += kGateNT) reinterpret_cast<int4*>(dst)[i] = reinterpret_cast<const int4*>(src)[i];
  for (int i = nv * V + threadIdx.x; i < cnt; i += kGateNT) dst[i] = src[i];
}

template <typename T>
__global__ __launch_bounds__(kGateNT) void gate_fwd_rows(GateTab t, const T* __restrict__ x, int64_t n, int rows,
                                                         T* __restrict__ y) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  int2* tab = reinterpret_cast<int2*>(lds);
  T* ys = reinterpret_cast<T*>(lds + (t.n_fields * 8 + 15) / 16 * 16);
  T* xs = ys + rows * t.C;
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  const int m = (int)(n - r0 < rows ? n - r0 : rows), S = t.C + t.G;
  copy_elems(xs, x + r0 * S, m * S);
  gate_fields_table(t, tab);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < (uint32_t)(m * t.n_fields); i += kGateNT) {
    const uint32_t row = i / (uint32_t)t.n_fields;
    const int2 f = tab[i - row * t.n_fields];
    const int d = f.y & 255;
    const T* xr = xs + row * S;
    T* yr = ys + row * t.C + f.x;
    if (d == 1) {
      const float v = DT<T>::to_f(xr[f.x]);
      yr[0] = DT<T>::from_f(v > 0.f ? v : 0.f);
    } else {
      const float sg = sigmoidf(DT<T>::to_f(xr[f.y >> 8]));
      for (int c = 0; c < d; ++c) yr[c] = DT<T>::from_f(sg * DT<T>::to_f(xr[f.x + c]));
    }
  }
  __syncthreads();
  copy_elems(y + r0 * t.C, ys, m * t.C);
}

// The gradient takes x's place in LDS: a field owns its components and its gate.
template <typename T>
__global__ __launch_bounds__(kGateNT) void gate_bwd_rows(GateTab t, const T* __restrict__ x, const T* __restrict__ dy,
                                                         int64_t n, int rows, T* __restrict__ dx) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  int2* tab = reinterpret_cast<int2*>(lds);
  T* dys = reinterpret_cast<T*>(lds + (t.n_fields * 8 + 15) / 16 * 16);
  T* xs = dys + rows * t.C;
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  const int m = (int)(n - r0 < rows ? n - r0 : rows), S = t.C + t.G;
  copy_elems(xs, x + r0 * S, m * S);
  copy_elems(dys, dy + r0 * t.C, m * t.C);
  gate_fields_table(t, tab);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < (uint32_t)(m * t.n_fields); i += kGateNT) {
    const uint32_t row = i / (uint32_t)t.n_fields;
    const int2 f = tab[i - row * t.n_fields];
    const int d = f.y & 255;
    T* xr = xs + row * S;
    const T* gr = dys + row * t.C + f.x;
    if (d == 1) {
      const float v = DT<T>::to_f(xr[f.x]);
      xr[f.x] = DT<T>::from_f(v > 0.f ? DT<T>::to_f(gr[0]) : 0.f);
    } else {
      const float sg = sigmoidf(DT<T>::to_f(xr[f.y >> 8]));
      float dot = 0.f;
      for (int c = 0; c < d; ++c) {
        const float g = DT<T>::to_f(gr[c]);
        dot = fmaf(g, DT<T>::to_f(xr[f.x + c]), dot);
        xr[f.x + c] = DT<T>::from_f(g * sg);
      }
      xr[f.y >> 8] = DT<T>::from_f(dot * sg * (1.f - sg));
    }
  }
  __syncthreads();
  copy_elems(dx + r0 * S, xs, m * S);
}

// The staged kernels take rows that fit LDS and arrays on 16-byte boundaries (a view may start
// anywhere); the others stay with the kernels that address memory by field.
template <typename T>
int launch_fwd(const GateTab& t, const T* x, int64_t n, T* y, hipStream_t st) {
  const int rows = gate_rows(t, sizeof(T), n);
  if (rows && (((uintptr_t)x | (uintptr_t)y) & 15) == 0)
    gate_fwd_rows<T><<<cdiv(n, rows), kGateNT, gate_tab_bytes(t) + rows * gate_row_bytes(t, sizeof(T)), st>>>(t, x, n,
                                                                                                          rows, y);
  else
    gate_fwd_kernel<T><<<cdiv(n * t.n_fields, 256), 256, 0, st>>>(t, x, n, y);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

template <typename T>
int launch_bwd(const GateTab& t, const T* x, const T* dy, int64_t n, T* dx, hipStream_t st) {
  const int rows = gate_rows(t, sizeof(T), n);
  if (rows && (((uintptr_t)x | (uintptr_t)dy | (uintptr_t)dx) & 15) == 0)
    gate_bwd_rows<T><<<cdiv(n, rows), kGateNT, gate_tab_bytes(t) + rows * gate_row_bytes(t, sizeof(T)), st>>>(
        t, x, dy, n, rows, dx);
  else
    gate_bwd_kernel<T><<<cdiv(n * t.n_fields, 256), 256, 0, st>>>(t, x, dy, n, dx);
  SSC_HIP(hipGetLastError());
  return SSCONV_OK;
}

int make_gatetab(const ssconv_fields* f, GateTab* t) {
  SSC_TRY(make_fieldtab(f, &t->f));
  t->C = t->f.ch0[t->f.n];
  t->n_fields = t->f.f0[t->f.n];
  int g = 0;
  for (int e = 0; e < t->f.n; ++e) {
    t->gate0[e] = g;
    if (t->f.l[e] > 0) g += t->f.mult[e];
  }
  t->G = g;
  return SSCONV_OK;
}

}  // namespace
}  // namespace ssconv

using namespace ssconv;

extern "C" int ssconv_gate_forward(const ssconv_fields* fields, const void* x, ssconv_dtype dtype, int64_t n, void* y,
                                   hipStream_t stream) {
  if (dtype != SSCONV_F32 && dtype != SSCONV_BF16) return fail(SSCONV_E_DTYPE, "unsupported dtype");
  if (n < 0 || (n > 0 && (!x || !y))) return fail(SSCONV_E_INVALID, "bad arguments");
  GateTab t;
  SSC_TRY(make_gatetab(fields, &t));
  if (n * t.n_fields == 0) return SSCONV_OK;
  if (dtype == SSCONV_F32) return launch_fwd<float>(t, (const float*)x, n, (float*)y, stream);
  return launch_fwd<uint16_t>(t, (const uint16_t*)x, n, (uint16_t*)y, stream);
}

extern "C" int ssconv_gate_backward(const ssconv_fields* fields, const void* x, const void* dy, ssconv_dtype dtype,
                                    int64_t n, void* dx, hipStream_t stream) {
  if (dtype != SSCONV_F32 && dtype != SSCONV_BF16) return fail(SSCONV_E_DTYPE, "unsupported dtype");
  if (n < 0 || (n > 0 && (!x || !dy || !dx))) return fail(SSCONV_E_INVALID, "bad arguments");
  GateTab t;
  SSC_TRY(make_gatetab(fields, &t));
  if (n * t.n_fields == 0) return SSCONV_OK;
  if (dtype == SSCONV_F32)
    return launch_bwd<float>(t, (const float*)x, (const float*)dy, n, (float*)dx, stream);
  return launch_bwd<uint16_t>(t, (const uint16_t*)x, (const uint16_t*)dy, n, (uint16_t*)dx, stream);
}
