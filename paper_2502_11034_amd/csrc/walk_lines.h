// When the update kernel walks the tensors of a list in whole 128-byte lines (kernels.hip).  Plain C++, without HIP.
#ifndef ADAGC_WALK_LINES_H
#define ADAGC_WALK_LINES_H

#include <cstdint>

#include "adagc.h"

namespace adagc {

// The least list (elements) for which whole lines pay, and the least launch (workgroups) where the caller limits it
// (adagc_config::grid_blocks) below a workgroup for each work item; 0 elements: never.  The kernel that walks lines spends more
// instructions, and reads and writes up to 37 elements of a tensor one by one: with few workgroups it is bound by those, and in a small
// list by the chain of accesses of its first and last tiles.  Time per step without / with, equal tensors of 16501 to 1048577
// elements end to end, by size of the list in 2^20 elements:
//                      1.5         3           4           6           12          32
//   AdamW, copy        .98 - .99   1.02 - 1.03 1.02 - 1.06 1.07 - 1.08 1.11        1.12 - 1.14
//   AdamW, bf16        .96 - .98   .96 - 1.00  .99 - 1.01  1.03 - 1.04 1.06 - 1.07 1.09 - 1.10
//   AdamW, f32         .97         .97 - 1.00  .99 - 1.01  1.02 - 1.04 1.06        1.09 - 1.10
//   Lion, bf16 + copy  .94 - 1.01  .97 - 1.01  .99 - 1.00  .97 - 1.00  1.01 - 1.02
// and lists of 9, 30 and 64 M elements by workgroups (AdamW then with 4 vectors in flight and items of 4096 elements):
//                      160         256         320         640
//   AdamW, copy        .97 - 1.07  1.06 - 1.24 1.08 - 1.18 1.07 - 1.20
//   AdamW, bf16        .90 - .92   .98 - 1.01  1.00 - 1.10 1.06 - 1.11
//   AdamW, f32         .83 - .84   .95 - 1.03  1.02 - 1.12 .98 - 1.08
//   Lion, bf16 + copy  .82 - .84   .85 - .89   .91 - .99   1.07 - 1.17
// (Lion at 8: 1.00 - 1.02, with 512 workgroups .93 - 1.04.  Fewer, larger work items, adagc_config::update_split 1 or 2: 1.01 - 1.13 at
// the size where the line lies and twice that.)
struct LineLimits {
    int64_t elems, workgroups;
};
constexpr LineLimits line_limits(int optimizer, bool bf16_grads, bool copy)
{
    if (optimizer == ADAGC_OPT_LION && bf16_grads && copy) return {(int64_t)8 << 20, 640};
    if (optimizer != ADAGC_OPT_ADAMW) return {0, 0};
    if (copy) return {(int64_t)3 << 20, 256};
    return {(int64_t)(bf16_grads ? 4 : 6) << 20, 320};
}

// The numbers of vectors in flight (adagc_config::unroll) that there is a kernel with whole lines for: those the library chooses
// itself.  us per step, 1500 ragged tensors (391 M elements) end to end, AdamW with unroll = 4, without / with: f32 2299 / 2066, with the copy
// 2579 / 2236, bf16 and the copy 2292 / 1966.
constexpr bool lines_with_unroll(int optimizer, int unroll) { return unroll == 2 || (optimizer == ADAGC_OPT_ADAMW && unroll == 4); }

// Whether a step's update kernel walks whole lines: the list and the launch (workgroups for so many work items) are large enough, most
// of the elements (off_lines of elems) belong to tensors that start off a line, and those are long enough.  us per step, packed end
// to end, without / with; mean elements per tensor:
//   AdamW, f32 gradients          330 000: 356 / 331   91 000: 199 / 187   22 000: 237 / 227   5800: 140 / 142   3200: 108 / 113
//   AdamW, bf16 and the copy               382 / 329            218 / 191           254 / 226         152 / 142         117 / 113
//   Lion, bf16 and the copy                243 / 234            142 / 136           168 / 163         103 / 103          81 / 84
//   Lion, f32 gradients                    238 / 255            136 / 143           164 / 171         102 / 103          79 / 80
// (Lion without the copy writes two arrays and reads three: the loads' overlap is worth more than the lines.)
// The mean is a coarse measure for AdamW with f32 gradients and no copy, which gains least: of lists with means of 16 500 to 26 000 those
// of equal or log-uniform sizes gain 2 to 5 %, those of log-normal sizes (few short tensors) lose 1 to 2 (196 / 201 us).
inline bool walk_lines(int optimizer, bool bf16_grads, bool copy, int64_t n_tensors, int64_t elems, int64_t off_lines, int64_t workgroups,
                       int64_t items)
{
    const LineLimits least = line_limits(optimizer, bf16_grads, copy);
    return least.elems && elems >= least.elems && (workgroups >= items || workgroups >= least.workgroups) && 2 * off_lines > elems &&
           elems >= 16384 * n_tensors;
}

}  // namespace adagc
#endif
