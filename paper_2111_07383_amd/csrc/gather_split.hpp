// fp32 output-stationary gather GEMM on the bf16 matrix cores (three bf16 parts per value).
#pragma once

#include "common.hpp"
#include "split_guard.hpp"

namespace ssconv {

// kappa as the kernels see it: B[s][n][k] = W[s][n][k], or W[s'][k][n] when transposed, s' = s or
// K-1-s (mirror); W fp32.
struct SplitKernel {
  const float* W;
  int transposed, mirror;
};

// True when the shape is handled (32-bit byte offsets into the split operands).
bool gather_split_supported(int64_t n_src, int ca, int cb, int K);
// Which plans come first.  Forwards: those whose scratch fits the fixed region of the allocation-free entry point,
// so that both entry points give the same bits.  Gradients have the workspace that their plan asks for, and the
// cheapest plan (104 -> 104 channels, 5x5x5, us, within the region and without: 38k sites 533 and 480, 50k 721 and
// 637, 70k 1131 and 830; 3x3x3, 70k: 302 and 252).
enum class SplitPlans { kForward, kGradient };

// Scratch of a call (the split operands and the partial tiles).
size_t gather_split_bytes(int64_t n_src, int ca, int cb, int64_t n_pos, int K, SplitPlans plans);
// Time of a gradient's call in us.
double gather_split_us(int64_t n_src, int ca, int cb, int64_t n_pos, int K);
// out[p][:] = sum_s B[s] (cb x ca) . src[nbr[s][p]] for p < n_pos; src [n_src, ca], out [n_pos, cb].
// rows3 (optional): the rows of src already split.  rows_flag (one of flags) is that of src's rows; where
// one of the words is set afterwards, out is not valid.  Bt (optional): receives B[s][n][k] in fp32, which the
// plain kernel then reads.
int gather_split(const float* src, int64_t n_src, int ca, const SplitKernel& B, int cb, const int32_t* nbr,
                 int64_t n_pos, int K, float* out, const SplitFlags& flags, int* rows_flag, hipStream_t st, CallScratch* sc,
                 SplitPlans plans, const uint16_t* rows3 = nullptr, float* Bt = nullptr);

// Split rows [n][ceil(c / 32)][3 parts][32 channels] of two sources (either may have no rows).
int64_t split_row_bytes(int c);
int split_rows(const float* x, int64_t nx, int cx, uint16_t* x3, int* x_flag, const float* y, int64_t ny, int cy,
               uint16_t* y3, int* y_flag, hipStream_t st);

}  // namespace ssconv
