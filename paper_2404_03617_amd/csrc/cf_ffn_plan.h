// cf_ffn_plan.h -- host arithmetic of the two-launch wide block (cf_ffn.h), in
// plain C++ so that a test can walk through it without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace cf {
namespace ffn {

// shares of a chunk: one where two would not leave room for two slots
constexpr int shares(int C) { return C == 512 ? 1 : 2; }
constexpr int chunk(int C) { return 32 * shares(C); }  // hidden channels per step

// Chunks per group when at most g groups share them, and the groups that then
// have any (12 chunks over 8 groups: 6 of two).  The launch and the reduction
// that adds the partials must agree on the count, so every count is one that
// filled_groups returns.
constexpr int group_chunks(int chunks, int g) { return (chunks + g - 1) / g; }
constexpr int filled_groups(int chunks, int g) {
    return g < 1 ? 1 : (chunks + group_chunks(chunks, g) - 1) / group_chunks(chunks, g);
}

// The groups out of `want` whose partials, `one` bytes each, fit `bytes`.
constexpr int fitting_groups(int chunks, int want, size_t one, size_t bytes) {
    return filled_groups(chunks, (size_t)want * one <= bytes ? want : (int)(bytes / one));
}

// Threads of the depth-wise launch over rows of W pixels: one for 8 channels of
// up to four (or seven, when that makes fewer strips) neighbouring pixels, in
// workgroups of 256.  A launch holds fewer than 2^32: images of one or two
// columns reach that at 64 and 128 GiB.
constexpr uint64_t dw_threads(int64_t rows, int W, int C) {
    return ((uint64_t)rows * ((W + 3) / 4) * (C / 8) + 255) / 256 * 256;
}
constexpr bool dw_launchable(int64_t rows, int W, int C) { return dw_threads(rows, W, C) < (uint64_t)1 << 32; }

}  // namespace ffn
}  // namespace cf
