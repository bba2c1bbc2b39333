// The tile kernel for int8 results through a table that slots do not take (of more than 256 segments, most of all), in kernels and a translation
// unit of their own: as a third form in the other tables' kernels, with the entries beyond one per thread requested behind the k-loop, it was
// slower, and so were they (code in front of what runs arrives with it; requested in front as here, the entries cost them 0.1 us more).
// us, that -> this: 1000 x 2304 x 768 with 1000 segments 7.77 -> 7.47, with 2048 8.22 -> 7.76, 2048 x 1024 x 1024 with 512 6.46 -> 6.28,
// 1500 x 2048 x 512 with 4096 8.48 -> 8.05; with 64, in slots, 847 x 3072 x 768 7.43 -> 7.30, 2500 x 3072 x 768 11.1 -> 10.9.
#include "nm_gemm_tile.h"

namespace nm {

int32_t launch_tile_long(int cfg, GemmParams& p, size_t table_bytes, hipStream_t s)
{
    return p.K % 128 ? launch_tile_config<true, true>(cfg, p, EPI_Q_LONG, table_bytes, s) : launch_tile_config<false, true>(cfg, p, EPI_Q_LONG, table_bytes, s);
}

}  // namespace nm
