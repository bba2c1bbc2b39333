// The tile kernel for products whose K is a multiple of 16 but not of 128 (layers of an odd number of heads of 64, most of all), in a
// translation unit of its own.  The streaming kernel, which had them, fetches 64-byte slices at half the rate and leaves its k-loop to the
// compiler.  us a layer of F = 4 H, before -> after (neighbouring widths): width 704, 16 x 100 tokens 63.0 -> 47.4 (768: 44.6), 32 x 128
// 81.4 -> 64.6 (62.3), 8 x 512 90.8 -> 74.1 (72.9); width 960, 32 x 128 112 -> 86; width 448, 32 x 300 106 -> 89.
#include "nm_gemm_tile.h"

namespace nm {

int32_t launch_tile_end(int cfg, GemmParams& p, int epi, size_t table_bytes, hipStream_t s) { return launch_tile_config<true>(cfg, p, epi, table_bytes, s); }

}  // namespace nm
