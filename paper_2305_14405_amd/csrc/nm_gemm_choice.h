// Choices that the GEMM launchers make on the host, in plain C++ (no HIP header: the CPU tests compile this file alone).
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdlib>
#include <cstring>

namespace nm {

// Debug switch NM_GEMM_CFG (tuning aid): the kernel, and the configuration of it, that a product takes wherever it meets that
// configuration's requirements; anywhere else, and where the value is not one of these, the rules decide.
//   big|wide|split|small|mid3|mid2|oldbig   streaming kernel (big: the tile kernel's 256x192 where that one takes the product,
//                                           which has replaced the streaming kernel's, oldbig)
//   direct<0-6>  unaligned<0-3>  tile<0-9>  small-tile, register-staged and tile kernel
//   relu<2,5-11>                            tile kernel with the epilogues of convolutions
enum ForcedKind { FORCED_NONE, FORCED_STREAM, FORCED_DIRECT, FORCED_UNALIGNED, FORCED_RELU, FORCED_TILE };
enum { STREAM_BIG, STREAM_WIDE, STREAM_SPLIT, STREAM_SMALL, STREAM_MID3, STREAM_MID2, STREAM_OLDBIG };
struct ForcedCfg {
    ForcedKind kind = FORCED_NONE;
    int number = -1;
};

inline ForcedCfg parse_forced_cfg(const char* e)
{
    static const char* const stream[] = {"big", "wide", "split", "small", "mid3", "mid2", "oldbig"};
    static const struct { const char* name; ForcedKind kind; unsigned numbers; } numbered[] = {
        {"direct", FORCED_DIRECT, 0x7f}, {"unaligned", FORCED_UNALIGNED, 0xf}, {"tile", FORCED_TILE, 0x3ff}, {"relu", FORCED_RELU, 0xfe4}};
    ForcedCfg f;
    if (!e) return f;
    for (int i = 0; i < 7; ++i)
        if (!std::strcmp(e, stream[i])) f.kind = FORCED_STREAM, f.number = i;
    for (const auto& n : numbered) {
        const size_t len = std::strlen(n.name);
        if (std::strncmp(e, n.name, len)) continue;
        const char* const digits = e + len;   // one or two, nothing in front of or behind them
        const size_t count = std::strspn(digits, "0123456789");
        if (count < 1 || count > 2 || digits[count]) continue;
        const int number = std::atoi(digits);
        if (number < 32 && (n.numbers >> number & 1)) f.kind = n.kind, f.number = number;
    }
    return f;
}

// Requirements of a configuration beyond those of its kernel.  k128: K (of a gathered row: Cin) is a multiple of 128; split_ok:
// and the table leaves room for a ring of three such slices; kunit: K or Cin, a multiple of 64 (9 and 10 have slices of 64 bytes).
constexpr bool stream_takes(int c, bool conv, bool k128, bool split_ok)
{
    return c == STREAM_BIG || c == STREAM_OLDBIG ? !conv && k128 : c == STREAM_SPLIT || c == STREAM_SMALL ? split_ok : true;
}
constexpr bool relu_takes(int c, int kunit) { return c == 9 || c == 10 || kunit % 128 == 0; }

// Operands of the tile kernel's epilogues for convolutions: rows of W with K bytes each (not [K,N]), 32-bit offsets from both
// bases; gathered rows whose taps are bits of a word and whose offsets stay positive with the padding's, plain ones aligned to 16
// bytes.  kunit: K, or Cin of gathered rows; a_bytes: of the image or of M rows.
struct ReluOperands {
    bool gathered, w_is_kn, w_aligned, both_aligned, resid;
    int kunit, taps;
    long long a_bytes, w_bytes;
};
constexpr bool relu_operands(const ReluOperands& o)
{
    return !o.w_is_kn && o.w_aligned && o.w_bytes < (1LL << 32) && o.kunit % 64 == 0 &&
           (o.gathered ? !o.resid && o.taps <= 32 && o.a_bytes < (1LL << 31) - (1 << 24) : o.both_aligned && o.a_bytes < (1LL << 32));
}

// Which tile of the tile kernel: the one whose predicted time is smallest.  A configuration takes
//   start + rounds * slice * K / 128 + rounds' * epilogue   us,
// rounds being its tiles over its places on the 256 CUs (up to three workgroups share one).  Up to 256 tiles behind the
// full rounds have a CU each and are charged the fraction `alone` of a round (`alone_epi` of an epilogue),
// up to 512 where three share a CU `paired`.  A ring of two stages only pays where workgroups do share (from
// `least` tiles on; it is also the one for K = 384): alone on a CU it waits for its operands, 23 instead of 17 us at
// 4096 x 768 x 3072 with 128x128.  The last entry is 128x128 with two wavefronts to a sub-tile, each taking half of a slice's
// k-steps: two on every SIMD where one workgroup has a CU, for the fp32 epilogue (4096 x 768 x 3072 18.4 -> 16.4 us, 2560 x
// 1024 x 4096 20.9 -> 18.3, 4096 x 768 x 768 10.6 -> 9.4); the shorter int8 ones do not repay the exchange (1500 x 2304 x 768
// 6.6, 7.0).  The constants are least-squares fits to 180 measured shapes: M from 64 to
// 16384, the four products of a layer of width 512, 768 and 1024.  Over those the chosen tile is 1.2 % slower than
// the best of the first nine (12 % at worst); full rounds weighted by one number per tile, over four of them,
// were 7 % (54 %) slower from M = 2048 on.  On 106 shapes outside the fit (widths 384, 640, 896, 1152, 1280 and 1536, FFNs
// of 4 H and 2 H + 128, M drawn up to 16384) it is 1.6 % slower than the best, at a tenth of them 6 % or more, at the
// two worst 38 % (1683 x 4608 x 1536) and 11 %.  Examples, us, 256x256 | 256x192 | 256x128 | 128x192 with three and two stages |
// 128x128 likewise | 64x128 likewise:
//   16384 x 1024 x 4096, fp32:   64 | 87 | 72 | 84 | 79 | 89 | 77
//   12000 x 3072 x  768, table:  52 | 51 | 58 | 59 | 43 | 58 | 47
//    4096 x  768 x 3072, fp32:   34 | 29 | 21 | 19 | 23 | 17 | 21 | 18 | 19
//    2048 x  768 x 3072, fp32:   33 | 26 | 20 | 17 | 17 | 15 | 15 | 10 | 11
// An epilogue's constant of 0 says that the configuration is not built for it: fp32 results take 128x128 with three stages in the
// last entry's form alone, int8 ones in the first.  allowed: a bit per configuration.
struct TileConfig {
    int bm, bn, stages, places, least;
    double alone, paired, alone_epi, start, slice, f32, q, table;
};
constexpr TileConfig kTileConfigs[] = {
    {256, 256, 2, 256, 0, 1, 1, 1, -1.88, 1.15, 11.73, 7.67, 11.42}, {256, 192, 2, 256, 0, 1, 1, 1, -2.43, 0.89, 10.88, 7.70, 9.41},
    {256, 128, 3, 256, 0, 1, 1, 1, -0.71, 0.68, 8.25, 4.37, 6.47},   {128, 192, 3, 256, 0, 1, 1, 1, 0.08, 0.54, 7.35, 4.55, 5.87},
    {128, 192, 2, 512, 257, 0.65, 1, 0.65, 0.94, 1.10, 9.88, 5.25, 6.32}, {128, 128, 3, 256, 0, 1, 1, 1, 0.21, 0.44, 0, 2.75, 3.90},
    {128, 128, 2, 512, 257, 0.65, 1, 0.65, 0.48, 0.87, 8.91, 2.98, 4.47}, {64, 128, 3, 512, 0, 0.45, 1, 0.8, 1.19, 0.52, 3.52, 2.23, 3.00},
    {64, 128, 2, 768, 513, 0.5, 0.7, 0.5, 1.27, 0.80, 5.53, 2.23, 3.44}, {128, 128, 3, 256, 0, 1, 1, 1, 0.21, 0.385, 6.7, 0, 0}};

// Whether the tile kernel's configuration c is built for such results (fp32 or int8) and takes a contraction of K bytes: its
// k-loop is a first slice, the steady state and the last slices, so it needs one slice more than its ring has stages.
constexpr bool tile_takes(int c, int K, bool f32)
{
    return c >= 0 && c < (int)(sizeof(kTileConfigs) / sizeof(kTileConfigs[0])) && (K + 127) / 128 >= kTileConfigs[c].stages + 1 &&
           (f32 ? kTileConfigs[c].f32 : kTileConfigs[c].q) != 0;
}

inline int choose_tile(int M, int N, int K, bool f32, bool table, unsigned allowed = ~0u)
{
    int best = -1;
    const int nk = (K + 127) / 128;
    double best_us = 0.0;
    for (int c = 0; c < (int)(sizeof(kTileConfigs) / sizeof(kTileConfigs[0])); ++c) {
        const auto& t = kTileConfigs[c];
        const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn), rest = tiles % t.places;
        if (!(allowed >> c & 1) || !tile_takes(c, K, f32) || (tiles < t.least && nk > 3)) continue;
        const bool alone = rest <= t.places - 256 && rest <= 256, paired = rest <= t.places - 256;
        const double full = (double)(tiles / t.places);
        const double rounds = full + (rest == 0 ? 0.0 : alone ? t.alone : paired ? t.paired : 1.0);
        const double epilogues = full + (rest == 0 ? 0.0 : alone ? t.alone_epi : paired ? t.paired : 1.0);
        const double us = t.start + rounds * t.slice * nk + epilogues * (f32 ? t.f32 : table ? t.table : t.q);
        if (best < 0 || us < best_us) best_us = us, best = c;
    }
    return best;
}

// Which of the tile kernel's configurations with the epilogues for convolutions: 128-byte slices and the cost model's tile where K (a
// gathered row's Cin, kunit) is a multiple of 128 and long enough for a ring; 64-byte ones of 128x128 tiles (9), three in flight,
// otherwise; of 128x64 (10) for at most 64 columns; 11 is 5 with two wavefronts to a sub-tile.
inline int choose_relu(int M, int N, int K, int kunit)
{
    if (N <= 64) return 10;
    if (kunit % 128 != 0 || K < 384) return 9;
    const int c = choose_tile(M, N, K, false, false, 0x1e4);
    return c == 5 && K >= 1536 ? 11 : c;   // 12544 x 256 x 2304 (3x3) 12.8 -> 12.0; 12544 x 256 x 1024 7.0 with 5, 7.6
}

// Outputs from which the larger tiles take an aligned product and the small-tile kernel no longer does.  tile_ok: those of the tile
// kernel with the epilogues of an encoder layer.
constexpr long long direct_below(bool tile_ok, int N, int K) { return tile_ok ? 1050000 : K <= 256 || N <= 64 ? 1700000 : 1000000; }

// Which tile, aligned operands: the one whose predicted time is smallest,
//   start + L * (tile + slice * slices) + R * (round + chain * c) + wave * c   us,
// c being the slices of a wavefront, L the workgroups of the CU that has most and R the rounds it takes for them (as many
// workgroups share a CU as LDS and its 32 wavefronts allow).  The constants are least-squares fits to 285 measured
// products (16 to 1500 rows, the four products of layers of width 384 to 1024, convolutions of a residual CNN as products;
// rms 5 to 9 %).  Over those the chosen tile is 0.8 % slower than the best of nine (11 % at worst), the rule by the
// number of tiles before it 3.0 %.  us, 16x32 | 32x32 | 32x64 with four wavefronts, with eight | 48x64 | 64x64:
//   128 x 768 x 3072   3.9 | 3.9 | 5.9 | 5.2 | 5.8 | 6.9      847 x  768 x 3072  11.4 | 10.1 | 10.5 | 12.0 | 8.4 | 9.2
//   512 x 1024 x 4096   10 | 8.9 | 9.8 | 7.7 | 8.4 | 9.4     1024 x 1024 x 1024   6.6 |  6.5 |  6.0 |  7.2 | 7.9 | 5.9
// Rows gathered from an image cost other things (addresses and tap masks in every slice), and with those constants long filters
// took 1.1 to 1.6 times as long as the rule by the number of tiles: they have their own, and 32x32 tiles with eight wavefronts.
// Fitted to 1120 convolutions (filters of 1 to 7, 64 to 1024 channels, 16 to 14000 positions, 510 of them a residual CNN's at images
// of 32 to 224; rms 6 to 7 %) by what the choice costs: over 500 others the chosen tile is 0.03 % slower than the best of seven (3 % at
// worst; a least-squares fit of the times alone 0.8 and 16 %).  us, by the other constants -> by these: 1575 x 128 x 25088
// (7x7) 26.8 -> 17.0, 972 x 200 x 12800 (5x5) 15.5 -> 10.8, 972 x 200 x 9216 (3x3) 11.9 -> 9.3; by the fit of the times -> by these:
// 3136 x 64 x 576 (3x3) 3.7 -> 3.4, 6075 x 64 x 576 4.3 -> 4.0, 576 x 512 x 256 (1x1, stride 2) 3.7 -> 3.3, 144 x 2048 x 1024 4.6 -> 4.0.
struct DirectCost {
    double start, tile, round, slice, chain, wave;
};
struct DirectTile {
    int bm, bn, kw, depth;
    DirectCost plain, gathered;   // a start of 0: not built
};
constexpr DirectTile kDirectTiles[] = {
    {16, 32, 8, 3, {1.92, 0.14, 0.33, 0.055, 0.36, -0.37}, {1.603, 0.494, 0.399, 0.044, 0.211, -0.072}},
    {32, 32, 4, 2, {1.92, 0.08, 0.45, 0.102, 0.14, -0.25}, {0.909, 0.152, 1.452, 0.044, 0.243, 0.11}},
    {32, 64, 4, 1, {1.38, 0.30, 0.93, 0.134, -0.16, 0.29}, {1.141, 0.121, 1.799, 0.091, 0.246, 0.119}},
    {32, 64, 8, 1, {1.92, 0.43, 0.43, 0.125, 0.69, -0.74}, {1.244, 0.89, 0.89, 0.07, 0.528, -0.286}},
    {48, 64, 4, 2, {1.67, 0.43, 0.97, 0.116, 0.44, -0.31}, {0.8, 0.6, 2.057, 0.116, 0.034, 0.241}},
    {64, 64, 4, 2, {1.38, 0.63, 1.45, 0.132, 0.41, -0.20}, {2.079, 0.057, 2.323, 0, 0.909, -0.077}},
    {32, 32, 8, 2, {0, 0, 0, 0, 0, 0}, {1.379, 0.575, 0.843, 0.05, 0.334, -0.13}}};
constexpr int kDirectTileCount = sizeof(kDirectTiles) / sizeof(kDirectTiles[0]);

// LDS of configuration c at most: the wavefronts' rings, and the table.
inline size_t direct_lds(int c, int K, size_t table_bytes)
{
    const DirectTile& t = kDirectTiles[c];
    const int chain = ((K + 127) / 128 + t.kw - 1) / t.kw;
    return (size_t)t.kw * (chain < t.depth ? chain : t.depth) * (t.bm + t.bn) * 128 + table_bytes;
}
constexpr const DirectCost& direct_cost(int c, bool gathered) { return gathered ? kDirectTiles[c].gathered : kDirectTiles[c].plain; }
// Whether configuration c exists for such rows and its rings and the table fit LDS (16x32 tiles and a table of 4096 segments do not).
inline bool direct_takes(int c, int K, size_t table_bytes, bool gathered)
{
    return c >= 0 && c < kDirectTileCount && direct_cost(c, gathered).start > 0 && direct_lds(c, K, table_bytes) <= 160 * 1024;
}

inline long direct_tiles(int c, int M, int N) { return (long)((M + kDirectTiles[c].bm - 1) / kDirectTiles[c].bm) * ((N + kDirectTiles[c].bn - 1) / kDirectTiles[c].bn); }
// slices: of a tile, on average
inline double direct_us(int c, long tiles, int K, double slices, size_t table_bytes, bool gathered)
{
    const DirectTile& t = kDirectTiles[c];
    const DirectCost& u = direct_cost(c, gathered);
    const int chain = ((K + 127) / 128 + t.kw - 1) / t.kw;
    const size_t lds = direct_lds(c, K, table_bytes);
    const long L = (tiles + 255) / 256, fit = (long)(160 * 1024 / (lds + 1024)), cap = 32 / t.kw, share = fit < 1 ? 1 : fit < cap ? fit : cap;
    const long R = (L + share - 1) / share;
    return u.start + L * (u.tile + u.slice * slices) + R * (u.round + u.chain * chain) + u.wave * chain;
}

inline int choose_direct(int M, int N, int K, int batches, size_t table_bytes, bool gathered)
{
    // Many products of a short contraction (attention scores; the fit has none): 32x32 tiles, 16x32 where those are few.  us, 16x32 |
    // 32x32 | 32x64 with four wavefronts: 270 of 58 x 58 x 64 10.0 | 8.5 | 13.1, 384 of 40 x 40 x 64 11.0 | 8.6 | 12.0, 2 of
    // 16 x 16 x 16 2.8 | 2.9 | 3.3; from 640 on the fit holds again (270 of 58 x 58 x 640 14.0 | 17.2 | 22.7).
    if (batches > 1 && K <= 512) return (long)((M + 31) / 32) * ((N + 31) / 32) * batches <= 128 ? 0 : 1;
    int best = 2;
    double best_us = 0.0;
    bool any = false;
    for (int c = 0; c < kDirectTileCount; ++c) {
        if (!direct_takes(c, K, table_bytes, gathered)) continue;
        const double us = direct_us(c, direct_tiles(c, M, N) * batches, K, (K + 127) / 128, table_bytes, gathered);
        if (!any || us < best_us) best_us = us, best = c, any = true;
    }
    return best;
}

// Two gathered products as one launch: the tile for both, or -1 where two launches are predicted to take less.  The cost is that of all
// tiles with the longer contraction's chain and the tiles' mean number of slices.
inline int choose_direct_pair(const int (&M)[2], const int (&N)[2], const int (&K)[2])
{
    double apart = 0.0;
    for (int i = 0; i < 2; ++i) {
        const int c = choose_direct(M[i], N[i], K[i], 1, 0, true);
        apart += direct_us(c, direct_tiles(c, M[i], N[i]), K[i], (K[i] + 127) / 128, 0, true);
    }
    int best = -1;
    for (int c = 0; c < kDirectTileCount; ++c) {
        const int k = K[0] > K[1] ? K[0] : K[1];
        if (!direct_takes(c, k, 0, true)) continue;
        const long t0 = direct_tiles(c, M[0], N[0]), t1 = direct_tiles(c, M[1], N[1]);
        const double us = direct_us(c, t0 + t1, k, (double)(t0 * ((K[0] + 127) / 128) + t1 * ((K[1] + 127) / 128)) / (t0 + t1), 0, true);
        if (us < apart) apart = us, best = c;
    }
    return best;
}

// Whether the register-staged tiles take a product whose operands cannot go to LDS directly in whole slices (align: of their rows and
// chunks, 1, 4 or 16 bytes; at 16, K is no multiple of 64) or the small-tile kernel does: the sign of a fit to the logarithm of their
// times' ratio.  The small tiles hold longer where operands are aligned to 16 bytes (the others cost them shifts), where a slice or
// two are all the contraction (nothing repays the larger tiles' prologue) and with fp32 results or several; shorter where result
// rows are not, since the register-staged kernel aligns its stores, and where few columns leave tiles half empty.  Fitted
// to 1229 products aligned to 16 and 771 others of 0.4 to 4.5 million outputs and K up to 4096 (with nothing below or beyond: the
// fit is not asked there), results and options drawn; over 725 and 475 others the kernel chosen is 0.7 and 0.5 % slower than the
// faster one, 38 and 22 % at worst (a line by alignment and K alone: 1.6 and 1.2 %, 41 and 51 %; at 0.8 million outputs: 4.7 and
// 1.1 %, 67 and 28 %).  us, small tiles | register-staged, int8 results:
//   16 bytes:  1016 x 896 x 144 4.3 | 5.9    784 x 1312 x 480 5.6 | 7.3   3064 x 722 x 624 14.4 | 9.9   1054 x 1488 x 2800 18.3 | 14.6
//   less:      700 x 700 x 1001 6.5 | 8.2   1000 x 999 x 999 11.2 | 9.9   8000 x 100 x 777 11.4 | 8.5
//   fp32 too:  11704 x 199 x 16 12.1 | 8.8   4420 x 438 x 80 10.8 | 8.1   (less) 8195 x 107 x 51 9.6 | 6.9
inline bool staged_faster(int align, int M, int N, int K, bool q, bool f32, bool table, bool resid)
{
    static constexpr struct { double one, outputs, k, f32, q, ragged, ragged_f32, ragged_q, table, resid, narrow; } kLog[2] = {
        {-0.17, 0.40, 0.20, -0.08, -0.08, 0.11, 0.03, 0.07, -0.08, -0.05, 0.09}, {0.04, 0.46, 0.07, -0.06, -0.06, 0.04, 0.09, -0.01, 0, 0, 0.09}};
    const auto& t = kLog[align < 16];
    const double outputs = (double)M * N * 1e-6;
    if (outputs < 0.4) return false;
    const bool ragged = N % 16 != 0;
    return t.one + t.outputs * std::log(outputs < 4.5 ? outputs : 4.5) + t.k * std::log(1 + (K < 4096 ? K : 4096) / 900.0) + (f32 ? t.f32 : 0) + (q ? t.q : 0) +
               (ragged ? t.ragged + (f32 ? t.ragged_f32 : 0) + (q ? t.ragged_q : 0) : 0) + (table ? t.table : 0) + (resid ? t.resid : 0) +
               t.narrow * (N > 64 ? 64.0 / N : 1) > 0;
}

// Which tile of the register-staged kernel: the one whose predicted time is smallest,  start + L * (slice * slices + epilogue) +
// latency * slices  us, L being the workgroups of the CU that has most.  The constants are least-squares fits to 40 to 76 measured
// shapes each (M and N from 10 to 16384, K from 16 to 4096, rms 10 to 15 %); over the 55 of them with 0.8 million outputs and more
// the tile chosen is 1.6 % slower than the best (23 % at worst).  The smallest tiles where a CU would get more than two of them
// are left out: there the fit flatters them (1951 x 2393 x 35 15.4 us, 128x64 12.5).
inline int choose_unaligned(int M, int N, int K, bool q, bool f32, bool table, bool resid)
{
    static constexpr struct { int bm, bn; double start, slice, latency, q, f32, table, resid; } kTiles[] = {
        {256, 128, 1.0, 1.70, -0.62, 5.8, 6.1, 1.9, 2.8}, {128, 128, 2.4, 0.91, -0.18, 3.2, 3.0, 0.9, 0.2},
        {128, 64, 2.8, 0.44, 0.19, 1.3, 1.8, 0.5, 0.3},   {64, 64, 3.7, 0.26, 0.21, 0.55, 1.0, 0.3, 0.4}};
    int cfg = 0;
    double best = 0.0;
    for (int c = 0; c < 4; ++c) {
        const auto& t = kTiles[c];
        const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        if (c == 3 && tiles > 512) continue;
        const double L = (double)((tiles + 255) / 256), nk = (K + 127) / 128;
        const double us = t.start + t.latency * nk + L * (t.slice * nk + (q ? t.q : 0.0) + (f32 ? t.f32 : 0.0) + (table ? t.table : 0.0) + (resid ? t.resid : 0.0));
        if (c == 0 || us < best) best = us, cfg = c;
    }
    return cfg;
}

// LDS of nm_gemm_ln.hip: a slice of W rows per 128 bytes of K, the A image (whole pieces of 256 columns) and the product's table, for which K beyond
// 896 and 128 columns leave 2048 segments' room.
constexpr size_t ln_gemm_lds(int tile, int K, size_t table_bytes)
{
    return (size_t)((K + 127) / 128) * (32 << tile) * 128 + (size_t)((K + 255) / 256) * 2 * 16 * 128 + table_bytes;
}

// Whether a product makes the LayerNorm in front of it, and with which tile of nm_gemm_ln.hip (16x32, 16x64, 16x128), or -1: as two
// kernels.  The narrowest tile whose workgroups a single round of the 256 CUs holds: a wider one repeats less of the LayerNorm but
// leaves CUs idle, and a second round costs more than the launch it saves.  us of GPU time, one kernel less two, 16x32 | 16x64 |
// 16x128 with the workgroups of each, weights from memory:
//    64 x 1152 x  384   144 -1.3 |  72 -1.3 |  36 -1.0       128 x 2304 x 768   576      | 288 +1.5 | 144 -0.6
//    64 x 2560 x  640   320 +1.1 | 160 -1.4 |  80 -1.1       128 x 4096 x 1024 1024      | 512 +2.3 | 256 -0.2
//   200 x 2560 x  640            | 520 +3.1 | 260 +1.6       256 x 2048 x 512            | 512 +0.4 | 256 -0.4
//   200 x 3072 x  768                       | 312 +2.4       384 x 1152 x 384                       | 216 -0.9
// Launches of their own are 3.1 us of host time each as well, which is what narrow layers of few rows wait for: nine layers of
// width 384 over 64 tokens 25.5 us a layer, 4.8 less by either product.  Where the table does not fit LDS beside the operands: two kernels.
inline int ln_gemm_tile(int M, int N, int K, size_t table_bytes)
{
    const long rows = (M + 15) / 16;
    for (int t = 0; t < 3; ++t)
        if (rows * ((N + (32 << t) - 1) / (32 << t)) <= 256) return ln_gemm_lds(t, K, table_bytes) <= 160 * 1024 ? t : -1;
    return -1;
}

// Whether the QKV projection and attention of a layer are one kernel (nm_qkv_attention.hip), by workgroups (128 tokens of whole sequences and a head)
// and by how much of their rows is tokens.  Up to 256 workgroups, each alone on a CU: eight wavefronts, which the contraction has
// slices enough for; beyond, four in a ring of two stages, two workgroups to a CU.  Workgroups x share of rows below 90 leave the chip to
// kernels of smaller tiles, padded rows cost what tokens do.  us a layer, this less the two kernels; width, workgroups, share:
//   eight:  768  48 1.00 +0.6 |  768 120 0.86 -0.5 |  768 132 0.60 +0.2 |  768 192 1.00 -2.4 | 1024  64 1.00 +0.4 | 1024 176 0.60 -1.5
//           512  80 1.00 +0.7 |  512 128 1.00 -1.6 |  768 156 0.70 -0.7 |  896  70 0.78 +1.4 | 1024 240 0.25 +2.2 | 1024 128 1.00 -1.0
//   four:   768 384 1.00 -2.6 |  768 768 0.62 +2.0 |  768 768 0.75 -2.4 |  768 768 0.70 -0.7 | 1024 768 0.60 +3.5 | 1024 2048 1.00 -18
//           768 264 1.00 -0.2 | 1024 512 0.75 -3.4 |  512 400 0.78 -3.5 |  384 600 0.52 +3.0 |  384 360 0.55 -0.7 |  384  96 1.00 -1.1
enum { QKV_ATTENTION_NONE, QKV_ATTENTION_FOUR, QKV_ATTENTION_EIGHT };
inline int qkv_attention_form(int B, int S, int heads, int K)
{
    if (S > 128 || K <= 256) return QKV_ATTENTION_NONE;
    const int seqs = S <= 64 ? 2 : 1;
    const long groups = ((long)B + seqs - 1) / seqs * heads;
    const double share = seqs * S / 128.0;
    if (groups > 256) return share >= 0.75 ? QKV_ATTENTION_FOUR : QKV_ATTENTION_NONE;
    if (share < 0.6 || groups * share < 90) return QKV_ATTENTION_NONE;
    return K > 384 ? QKV_ATTENTION_EIGHT : QKV_ATTENTION_FOUR;
}

// Rows per workgroup with which steps 5 to 9 of a layer (and step 1 of the next) are one kernel over blocks of rows (nm_block.hip), 0: the separate
// kernels.  One workgroup runs on a CU, so up to 4096 rows 16 per workgroup are one round of the chip and cost what 64 rows cost;
// beyond, 32 rows halve the rounds.  The cost of a round grows with the weights (65 bytes per ns), that of the separate kernels with the rows and,
// little by little, with F: they cross at as many rows as 2.4 H^2 + 2 H F has thousands, earlier never below 0.37 million, later beyond 1.3.  Over 864
// layers of stacks (H of 128 to 512, F of H to 8 H, 32 to 4096 rows) the choice is 0.05 % slower than the better one and 6 % at worst (by the
// weights' number alone 0.9 and 23 %).  us a layer, heads of 64, this kernel | separate ones:
//   H = 128  F 1024   128 rows 16.2 | 18.2   4096 18.1 | 33.1      H = 320  F  640   512 22.2 | 20.5    768 22.5 | 22.8   4096 26.7 | 37.2
//   H = 192  F  384   128 15.8 | 16.8         768 16.1 | 18.8              F 1280  1024 29.7 | 28.5   1536 30.0 | 31.8   4096 32.9 | 40.1
//            F  768   384 18.2 | 18.0         768 18.4 | 21.0      H = 384  F  768   768 25.0 | 25.0   1024 25.2 | 27.1   4096 29.5 | 38.8
//   H = 256  F  512   256 17.4 | 17.1         768 17.9 | 19.9              F 1536  1024 32.8 | 30.2   1536 33.2 | 33.8   4096 36.4 | 39.3
//            F 1024   512 20.7 | 19.3         768 20.9 | 21.3      H = 512  F 1024  2048 36.7 | 33.5   4096 40.7 | 37.2
//   beyond 4096 rows (32 to a workgroup), F = 4 H: H = 256 8192 32.4 | 47.5, 12288 52.3 | 64.0; 320 12288 69.0 | 69.8; 384 6144 64.7 | 51.6
inline int block_rows_faster(int M, int H, int F)
{
    const double h = H, weights = 4 * h * h + 2 * h * F, size = 2.4 * h * h + 2 * h * F;
    if (M > 4096) return M <= 24576 && weights <= 1.25e6 ? 32 : 0;
    const double rows = size < 0.37e6 ? 0.0 : 1e-3 * size + (size > 1.3e6 ? 1.5e-3 * (size - 1.3e6) : 0.0);
    return weights <= 2e6 && M >= rows ? 16 : 0;
}

// Two 1x1 convolutions as one kernel (nm_conv_chain.hip): K to N1 channels with a shortcut, and those to N2, at M positions.
constexpr int chain_waves(int K) { return K == 64 ? 4 : 8; }   // of a workgroup
// LDS: both filters, scale and bias of both products' columns, a word per wavefront.
constexpr size_t conv_chain_lds(int K, int N1, int N2) { return (size_t)N1 * (K + N2) + 8 * (size_t)(N1 + N2) + 32; }
constexpr bool conv_chain_built(int K, int N1, int N2)
{
    return (K == 64 || (K == 128 && N2 == 128)) && (N2 == 64 || N2 == 128) && N1 % 256 == 0 && conv_chain_lds(K, N1, N2) <= 148 * 1024;
}
// Workgroups that a CU holds: by LDS, and by registers (12 or 8 wavefronts).
constexpr int conv_chain_share(int K, int N1, int N2)
{
    const int fit = (int)(160 * 1024 / conv_chain_lds(K, N1, N2)), most = K != 64 ? 1 : N2 == 64 ? 3 : 2;
    return fit < most ? fit : most;
}
// Whether the one kernel is predicted to take less than two: a chain of 32 positions through all N1 channels per wavefront, as often as a
// SIMD (at K = 128, its two wavefronts) has to, and the bytes of the one; a latency and the bytes of the two, which small tiles keep
// from falling further.  Fitted to 160 measured triples of M from 300 to 262144 (rms 6 % and 9 %); over them the choice is 0.3 % slower than the better
// one and 7 % at worst.  us, two kernels | one:
//    64 ->  256 ->  64:  3136 7.7 | 7.8     12544 11.2 |  8.3    36000 11.8 | 12.6   100352 24.0 | 20.7   200704 36.7 | 29.7
//    64 ->  256 -> 128:  3136 8.1 | 8.6     12544 12.6 |  9.4    36000 13.6 | 14.0   100352 27.6 | 23.8   200704 42.2 | 34.8
//   128 ->  512 -> 128: 12544 11.6 | 18.9   36000 20.7 | 20.2    50176 25.1 | 21.1    75000 34.8 | 36.4   131072 51.1 | 42.4
//    64 -> 1024 ->  64: 12544 15.3 | 21.4   32000 26.3 | 23.0    36000 29.7 | 34.0    65536 40.9 | 34.9   200704 135  | 127
// Two-segment tables that are no ReLU (relu: relu_codes holds for both) take a vector instruction or two more per code, and in the one kernel a
// loop without a ring: constants of their own, fitted to 87 and 204 such pairs (rms 3 to 5 % and 8 %).  Over the 126 that the others' constants
// chain the choice is 1.3 % slower than the better one and never by more than 2.5 % slower than two kernels (all of them chained: 5 and 34 %);
// 64 -> 512 -> 64 and wider gain nothing.  us, two kernels | one:
//    64 ->  256 ->  64:  5000 9.0 | 10.4    12544 12.0 | 10.9    36000 14.2 | 16.5   100352 28.2 | 26.5   200704 45.2 | 42.0
//    64 ->  256 -> 128:  5000 9.5 | 11.1    16000 11.0 | 11.9    45000 17.2 | 17.8    65536 22.5 | 19.6   131072 36.7 | 32.2
//   128 ->  512 -> 128: 50176 30.2 | 29.2   58000 33.9 | 30.6    65536 36.6 | 31.7   115000 57.4 | 55.2
//    64 ->  768 ->  64: 26000 23.5 | 26.5   58000 38.5 | 46.1   200704 130  | 156
inline bool conv_chain_faster(int M, int K, int N1, int N2, bool relu)
{
    const double m = M * 1e-6, bytes = m * (K + 2.0 * N1 + N2);
    const long blocks = ((long)M + 31) / 32;
    const double turns = (double)(K == 64 ? (blocks + 1023) / 1024 : (blocks + 2047) / 2048) * N1 / 256;
    if (!relu) {
        if (N2 == 64 && N1 != 256) return false;
        const double apart = 7.5 + 0.225 * (bytes + m * N1), least = m * N1 > 3.0 ? 11.5 : 0.0;
        const double one = K != 64 ? 8.02 + 6.49 * turns + 0.127 * bytes : N2 == 64 ? 6.76 + 3.26 * turns + 0.121 * bytes : 6.79 + 3.8 * turns + 0.12 * bytes;
        return one < (apart > least ? apart : least);
    }
    const double apart = 6.0 + 0.2 * (bytes + m * N1), least = m * N1 > 1.2 ? 10.0 : 0.0;
    const double one = K != 64 ? 6.55 + 5.34 * turns + 0.097 * bytes : N2 == 64 ? 5.04 + 3.03 * turns + 0.05 * bytes : 5.31 + 3.45 * turns + 0.061 * bytes;
    return one < (apart > least ? apart : least);
}

// 3x3 convolutions of 64 channels (nm_conv_taps.hip), or the small-tile and the tile kernel: up to here the filter, which every workgroup
// loads whole, costs more than the image read nine times.  us, those | this, ReLU: 3136 positions 3.7 | 4.4, 6272 4.1 | 4.5, 9000 5.0 | 4.8, 10000
// 5.1 | 4.8, 12544 5.2 | 4.8, 25088 8.1 | 5.2, 50176 7.4 | 6.3, 200704 17.3 | 13.9; another table 10000 5.1 | 5.1, 16000 5.3 | 5.3, 20000 6.1 | 5.4; without
// one, which takes the other table's code here, 9000 4.9 | 5.1, 12000 5.0 | 5.2, 16000 5.2 | 5.3, 18000 6.0 | 5.4, 200704 17.7 | 15.2.
constexpr int kTapsWaves = 8;   // of a workgroup
constexpr bool conv_taps_faster(int M, bool table) { return M >= (table ? 8192 : 16384); }

// Tile rows per group of the tile order.  Workgroup i runs on XCD i % 8, and the kernels hand XCD x the
// x-th eighth of the tile sequence, which walks groups of group_m tile rows column by column.  An
// eighth of r x c tiles reads r * BM rows of A and c * BN rows of W through that XCD's L2: pick the r that makes this
// sum smallest, counting the rows and columns that an eighth straddles where r x c tiles are not exactly one.  (Operand
// stream of 128x128 tiles of 4096 x 768 x 3072 alone: 20.5 TB/s with 4 x 6 tiles to an XCD, 11.5 with 24 x 1.)
// It is host work of every launch: of the r whose groups an eighth holds whole, r = 1 reads fewest rows, and r beyond the
// best sum's rows cannot be better.  Every r up to an eighth of the tiles took 1.7 us at 1568 x 2 tiles and 25 at 12544 x 4;
// these few take less than 0.02 (a launch takes 3.1).
inline int xcd_group_rows(int tiles_m, int tiles_n, int BM, int BN)
{
    const int ntiles = tiles_m * tiles_n, share = (ntiles + 7) / 8, whole = share / tiles_n;
    int best = 1;
    long best_cost = -1;
    for (int r = 1; r <= tiles_m && r <= share; r = r == 1 && whole > 1 ? whole + 1 : r + 1) {
        if (best_cost >= 0 && (long)r * BM + BN >= best_cost) break;
        long rows, cols;
        if (r <= whole) {   // whole groups (r = 1)
            rows = share % tiles_n == 0 ? whole : whole + 2;
            cols = tiles_n;
        } else {
            const bool exact = ntiles % 8 == 0 && share % r == 0 && tiles_n % (share / r) == 0 && tiles_m % r == 0;
            rows = exact ? r : r + r / 2;
            cols = exact ? share / r : share / r + 1;
        }
        if (rows > tiles_m) rows = tiles_m;
        if (cols > tiles_n) cols = tiles_n;
        const long cost = rows * BM + cols * BN;
        if (best_cost < 0 || cost < best_cost) best_cost = cost, best = r;
    }
    return best;
}

}  // namespace nm
