// Output-stationary gather -> MFMA GEMM over flattened (offset, channel) chunks.
#pragma once

#include "common.hpp"
#include "split_guard.hpp"

namespace ssconv {

struct NormSink;

// True when gather_mfma handles the shape (ca a multiple of 8, at most 128 offsets).
bool gather_mfma_supported(ssconv_dtype dt, int ca, int cb, int K);

// Its time in us (fp32); active: the offsets that occur in a tile of kMfmaRows rows.
constexpr int kMfmaRows = 128;
double gather_mfma_us(int ca, int cb, int64_t n_pos, int K, double active);

// out[order ? order[p] : p][:] = sum_s Bt[s] (cb x ca) . src[nbr[s][p]] for p < n_pos.
// src [*, ca], Bt [K][cb][ca] and out [*, cb] in dt; nbr [K][n_pos] (-1 = absent).
// Offset splits (fp32 partials added in split order) take their partials from sc (nullptr: the
// device memory cache); with a fixed scratch region the split count is lowered until they fit.
// sink (optional): the kernel that writes out also leaves the Norm statistics of out there (norm.hpp).
// only: condition of the launch (one launch then, no splits).
int gather_mfma(const void* src, int64_t n_src, ssconv_dtype dt, int ca, const void* Bt, int cb, const int32_t* nbr,
                const int32_t* order, int64_t n_pos, int K, void* out, hipStream_t st, CallScratch* sc = nullptr,
                NormSink* sink = nullptr, const OnlyIf& only = OnlyIf());

// bf16 pipeline kernel (gather_bf16.hip): any channel counts whose operands stay below 2 GB.
bool gather_bf16_supported(int64_t n_src, int ca, int cb, int K);
// Scratch of a call (padded rows, packed kappa, pieces of tiles).
size_t gather_bf16_bytes(int64_t n_src, int ca, int cb, int64_t n_pos, int K);
// out[p][:] = sum_s B[s] (cb x ca) . src[nbr[s][p]] for p < n_pos; B[s][n][k] = W[s'][n][k], or
// W[s'][k][n] when transposed, s' = s or K-1-s (mirror); src holds n_src rows; padded
// (optional, channels not in multiples of 8): its rows padded by pad_rows_bf16.
int gather_bf16(const void* src, int64_t n_src, int ca, const void* W, bool transposed, bool mirror, int cb,
                const int32_t* nbr, int64_t n_pos, int K, void* out, hipStream_t st, CallScratch* sc,
                const uint16_t* padded = nullptr);

// Rows [n][c] -> [n][c rounded up to 32], zeros past c, of two sources (either may have no rows).
int pad_rows_bf16(const uint16_t* x, int64_t nx, int cx, uint16_t* xp, const uint16_t* y, int64_t ny, int cy, uint16_t* yp,
                  hipStream_t st);

}  // namespace ssconv
