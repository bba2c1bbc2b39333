// The launcher's choice between the LayerNorm kernels, in plain C++ (no HIP header: the CPU tests compile this file alone).
#pragma once

#include <cstdint>

namespace nm {

constexpr int kRowThreads = 256;

// layernorm_row_kernel: a wavefront per row and no loop over rows, so its grid grows with them.  HIP refuses a launch of 2^32
// work-items and more: from 2^26 - 3 rows on (64 GiB of 256 columns) the kernel that walks the rows takes the call.
constexpr int64_t layernorm_row_blocks(int64_t rows) { return (rows - 1) / (kRowThreads / 64) + 1; }
constexpr bool layernorm_row_takes(int64_t rows, int cols, int nseg)
{
    return rows >= 1 && cols % 256 == 0 && cols <= 1024 && nseg <= 256 && layernorm_row_blocks(rows) < (1LL << 32) / kRowThreads;
}

// Rows of 16-byte loads: the row kernel, or layernorm_pwl_kernel with the vectors requested with the first row (held in registers:
// a third to three quarters more of them) or behind the look-up.  plain: one table, no segment output.  us, row kernel | with
// the row | behind the look-up, int8 results, int8 and fp32:
//   4096 x 256   2.82 | 2.90 | 2.85    3.35 | 3.41 | 3.38      8195 x 256    3.76 | 3.58 | 3.59    4.92 | 4.71 | 4.77
// 131075 x 256   30.9 | 25.3 | 28.2    62.4 | 48.1 | 52.2      8195 x 512    4.79 | 4.64 | 4.47    7.09 | 7.14 | 7.53
//  16384 x 512   8.33 | 8.37 | 9.19    12.5 | 12.6 | 14.2      8195 x 768    5.93 | 6.33 | 6.09    9.52 | 9.97 | 10.3
//   1027 x 384          2.85 | 2.85           2.97 | 3.02      8195 x 384           5.15 | 4.86           6.99 | 6.64
//  24000 x 384          10.0 | 10.9           13.8 | 14.7      6000 x 640           5.45 | 4.86           7.63 | 7.07
//  14000 x 640          10.3 | 11.1           14.0 | 15.9      5000 x 896           6.34 | 5.41           8.99 | 7.95
//  10000 x 896          10.6 | 10.2           14.7 | 15.1     10000 x 1000         10.9 | 11.1           15.6 | 16.2
//  12000 x 896          12.1 | 12.8           16.6 | 17.4      8195 x 1000          9.19 | 9.54           12.9 | 13.8
// and on both sides of the lines, the first two pairs with fp32 results:
//   5993 x 832  9.51 | 8.82     9616 x 432  7.96 | 7.69     6258 x  960  7.67 | 7.32
//   6685 x 896  11.0 | 11.7    10039 x 476  8.48 | 8.78     7460 x 1000  8.93 | 9.33    12358 x 724  10.3 | 11.0
// A wavefront of the row kernel reads table and vectors for one row, which of 256 columns are more than the row.  Requested
// with the row the vectors arrive earlier, and rows beyond the 4096 workgroups find them there; in between fewer wavefronts
// fit a CU: from about one row for each of them to the second round of the others.
enum LayerNormForm { LN_ROW, LN_AHEAD, LN_LATE };
constexpr LayerNormForm layernorm_form(int64_t rows, int cols, int nseg, bool plain, bool f32)
{
    if (plain && layernorm_row_takes(rows, cols, nseg)) {
        if (cols == 256) return rows <= 5000 ? LN_ROW : LN_AHEAD;
        return cols == 512 && !f32 && rows > 5000 && rows <= 14000 ? LN_LATE : LN_ROW;
    }
    if (cols <= 256 || cols > 1024) return LN_AHEAD;
    const int64_t most = f32 ? (cols > 512 ? 6144 : cols > 384 ? 9728 : 12000) : cols > 896 ? 6656 : cols > 768 ? 11000 : cols > 512 ? 12288 : 16384;
    return rows >= (f32 ? 4096 : 1250) && rows <= most ? LN_LATE : LN_AHEAD;
}

}  // namespace nm
