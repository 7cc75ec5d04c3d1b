// Kernel gradient on the bf16 matrix cores: bf16 rows, or fp32 rows as three bf16 parts.
#pragma once

#include "kgrad_mfma.hpp"
#include "split_guard.hpp"

namespace ssconv {

// Gathered rows as the kernels read them: row r at byte r * stride, channel c of a bf16 row at 2 c, the
// parts p of channels 32 j .. 32 j + 31 of a split row at 192 j + 64 p; zeros past the channels.
struct KgradRows {
  const void* p = nullptr;
  int64_t bytes = 0;
  int stride = 0;
};

// Tile of a workgroup in 32-channel steps (out, in), tiles covering the channels, work units wanted.
struct KgradTile {
  int wm, wn, mtiles, ntiles, units;
};
KgradTile kgrad_tile(const ssconv_rulebook* rb, int parts, int cin, int cout);

// part[u][o][i] (fp32) = sum over unit u's slice of R_s of grad_out[x][o] feats[y][i].  flags (split rows): where a
// word of the rows or of the sums is set afterwards, part is not valid.
int kgrad_tiles(const KgradRows& grad_out, const KgradRows& feats, int parts, int cin, int cout,
                const ssconv_rulebook* rb, const KgradTile& t, const KgradUnits& units, const KgradOrder& order,
                const SplitFlags& flags, float* part, hipStream_t st);

}  // namespace ssconv
