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

}  // namespace nm
