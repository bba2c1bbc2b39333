// The host-side choices of the launchers (csrc/nm_gemm_choice.h, csrc/nm_rows_choice.h), compiled alone by
// tests/test_gemm_choice.py with -fsanitize=address,undefined.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>

#include "nm_gemm_choice.h"
#include "nm_rows_choice.h"

using namespace nm;

#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED %s (line %d)\n", #cond, __LINE__); return 1; } } while (0)

static bool is(const char* value, ForcedKind kind, int number)
{
    const ForcedCfg f = parse_forced_cfg(value);
    return f.kind == kind && f.number == number;
}

static int forced_values()
{
    static const char* const stream[] = {"big", "wide", "split", "small", "mid3", "mid2", "oldbig"};
    for (int i = 0; i < 7; ++i) EXPECT(is(stream[i], FORCED_STREAM, i));
    char name[32];
    for (int i = 0; i < 100; ++i) {
        struct { const char* name; ForcedKind kind; bool known; } kinds[] = {
            {"direct", FORCED_DIRECT, i <= 6}, {"unaligned", FORCED_UNALIGNED, i <= 3}, {"tile", FORCED_TILE, i <= 9},
            {"relu", FORCED_RELU, i == 2 || (i >= 5 && i <= 11)}};
        for (const auto& k : kinds) {
            std::snprintf(name, sizeof(name), "%s%d", k.name, i);
            EXPECT(k.known ? is(name, k.kind, i) : is(name, FORCED_NONE, -1));
        }
    }
    EXPECT(is(nullptr, FORCED_NONE, -1));
    for (const char* v : {"", "tile", "tile-1", "tile+1", "tile 1", "tile1x", "tile001", "tile99999999999", "bigger", "mid", "direct", "relu2 ", "Tile1"})
        EXPECT(is(v, FORCED_NONE, -1));
    return 0;
}

// What the kernels assume of a configuration, with the ring depths and slice widths of their instantiations.
static int requirements()
{
    static const int stages[10] = {2, 2, 3, 3, 2, 3, 2, 3, 2, 3};
    EXPECT(sizeof(kTileConfigs) / sizeof(kTileConfigs[0]) == 10);
    for (int c = 0; c < 10; ++c) {
        EXPECT(kTileConfigs[c].stages == stages[c]);
        for (int slices = 1; slices <= 8; ++slices) {   // 5: int8 alone, 9: fp32 alone
            EXPECT(tile_takes(c, 128 * slices, false) == (slices >= stages[c] + 1 && c != 9));
            EXPECT(tile_takes(c, 128 * slices, true) == (slices >= stages[c] + 1 && c != 5));
        }
    }
    for (int f32 = 0; f32 < 2; ++f32) EXPECT(!tile_takes(-1, 4096, f32) && !tile_takes(10, 4096, f32) && !tile_takes(49, 4096, f32));
    for (int K = 384; K <= 8192; K += 128)
        for (int M : {1, 77, 847, 1005, 1205, 4096, 16384})
            for (int N : {16, 400, 768, 1744, 4096})
                for (int f32 = 0; f32 < 2; ++f32)
                    for (unsigned allowed : {~0u, 0x1e4u}) {
                        const int c = choose_tile(M, N, K, f32 != 0, false, allowed);
                        EXPECT(c >= 0 && (allowed >> c & 1) && tile_takes(c, K, f32 != 0));
                    }
    for (int c = 0; c < 12; ++c) {   // a contraction of 64 (2 n + 1) bytes has no whole slices of 128
        EXPECT(relu_takes(c, 128) && relu_takes(c, 1024));
        EXPECT(relu_takes(c, 64) == (c == 9 || c == 10) && relu_takes(c, 192) == (c == 9 || c == 10));
    }
    const ReluOperands plain = {false, false, true, true, false, 512, 0, 1 << 20, 1 << 20}, conv = {true, false, true, true, false, 128, 9, 1 << 20, 1 << 20};
    for (ReluOperands o : {plain, conv}) {
        EXPECT(relu_operands(o));
        auto without = [&o](auto change) { ReluOperands q = o; change(q); return relu_operands(q); };
        EXPECT(!without([](ReluOperands& q) { q.w_is_kn = true; }));   // V in nm_attn_context: rows of W are not contiguous in k
        EXPECT(!without([](ReluOperands& q) { q.w_aligned = q.both_aligned = false; }));
        EXPECT(!without([](ReluOperands& q) { q.kunit = 96; }) && without([](ReluOperands& q) { q.kunit = 192; }));
        EXPECT(!without([](ReluOperands& q) { q.w_bytes = 1LL << 32; }) && !without([](ReluOperands& q) { q.a_bytes = 1LL << 32; }));
        EXPECT(without([](ReluOperands& q) { q.resid = true; }) == !o.gathered && without([](ReluOperands& q) { q.both_aligned = false; }) == o.gathered);
        EXPECT(without([](ReluOperands& q) { q.taps = 33; }) == !o.gathered && without([](ReluOperands& q) { q.a_bytes = (1LL << 31) - (1 << 24); }) == !o.gathered);
    }
    for (int c = 0; c < 7; ++c) {
        const bool big = c == STREAM_BIG || c == STREAM_OLDBIG, split = c == STREAM_SPLIT || c == STREAM_SMALL;
        EXPECT(stream_takes(c, false, true, true) && stream_takes(c, true, true, true) == !big);
        EXPECT(stream_takes(c, false, false, false) == (!big && !split) && stream_takes(c, false, true, false) == !split);
    }
    for (int K : {16, 128, 200, 1024, 3072, 65536})
        for (size_t table : {size_t(0), size_t(16), size_t(16384), size_t(16392), size_t(32768)}) {
            for (int gathered = 0; gathered < 2; ++gathered) {
                for (int c = 0; c < 6; ++c) EXPECT(direct_takes(c, K, table, gathered) == (direct_lds(c, K, table) <= 160 * 1024));
                EXPECT(direct_takes(0, K, table, gathered) == (K < 3072 || table <= 16384));   // 24 slices in rings of three
                EXPECT(direct_takes(6, K, table, gathered) == (gathered && (K <= 1024 || table <= 32768)));
                for (int M : {1, 100, 1500}) EXPECT(direct_takes(choose_direct(M, 512, K, 1, table, gathered), K, table, gathered));
            }
        }
    EXPECT(!direct_takes(-1, 128, 0, true) && !direct_takes(7, 128, 0, true));
    for (int cin : {256, 512, 1024})   // long filters over few positions: eight wavefronts to a 32x32 tile
        for (int k : {5, 7}) EXPECT(choose_direct(1575, 128, k * k * cin, 1, 0, true) == 6 && choose_direct(972, 200, k * k * cin, 1, 0, true) == 6);
    // short filters of a residual CNN, each with the fastest tile (us 3.3, 4.0, 4.0 and 3.4; with those of a fit of the times alone 3.7, 4.6, 4.3 and 3.7)
    EXPECT(choose_direct(576, 512, 256, 1, 0, true) == 1 && choose_direct(144, 2048, 1024, 1, 0, true) == 3);
    EXPECT(choose_direct(6075, 64, 576, 1, 0, true) == 3 && choose_direct(3136, 64, 576, 1, 0, true) == 6);
    const int gathered[][4] = {{392, 64, 576, 0}, {840, 208, 256, 1}, {2520, 400, 256, 2}, {4048, 72, 576, 3}, {3599, 136, 576, 4},   // tests/test_gpu_conv.py
                               {3870, 400, 256, 5}, {899, 136, 4800, 6}, {840, 136, 3136, 6}};
    for (const auto& g : gathered)   // without a table and with a ReLU's two segments
        for (size_t table : {size_t(0), size_t(16)})
            EXPECT(g[0] * g[1] < direct_below(false, g[1], g[2]) && choose_direct(g[0], g[1], g[2], 1, table, true) == g[3]);
    for (int K : {16, 64, 80, 256, 512}) {   // attention scores: many small products
        EXPECT(choose_direct(58, 58, K, 270, 0, false) == 1 && choose_direct(40, 40, K, 384, 0, false) == 1 && choose_direct(10, 10, K, 168, 0, false) == 1);
        EXPECT(choose_direct(16, 16, K, 8, 0, false) == 0 && choose_direct(500, 500, K, 4, 0, false) == 1);
    }
    return 0;
}

// Products on both sides of the line between the small-tile and the register-staged kernel, each with the faster one.
static int staged_line()
{
    const struct { int M, N, K, align; bool staged; } products[] = {
        {1016, 896, 144, 16, false}, {667, 2112, 272, 16, false}, {784, 1312, 480, 16, false}, {198, 4192, 992, 16, false}, {565, 1440, 480, 16, false},
        {149, 5680, 16, 16, false}, {23492, 105, 16, 16, true}, {3064, 722, 624, 16, true}, {1054, 1488, 2800, 16, true}, {2048, 768, 1008, 16, true}, {783, 676, 416, 16, false},
        {122, 8192, 11, 1, false}, {1220, 900, 40, 4, true}, {700, 700, 1001, 1, false}, {8000, 100, 777, 1, true},
        {1000, 999, 999, 1, true}, {4096, 1001, 1000, 4, true}};
    for (const auto& p : products) EXPECT(staged_faster(p.align, p.M, p.N, p.K, true, false, false, false) == p.staged);
    // which results, and whether their rows are aligned, count too
    EXPECT(staged_faster(16, 8020, 202, 16, true, true, false, false) && staged_faster(16, 5322, 191, 1040, true, false, false, false));
    EXPECT(staged_faster(1, 8195, 107, 51, true, true, false, false) && !staged_faster(16, 737, 3168, 80, true, true, false, true));
    for (int align : {1, 4, 16})
        for (int options = 0; options < 4; ++options) {   // beyond what was measured
            EXPECT(!staged_faster(align, 630, 630, 65536, true, false, options & 1, options & 2));
            EXPECT(staged_faster(align, 16384, 16384, 65536, true, true, options & 1, options & 2));
        }
    return 0;
}

// Every r in turn.
static int group_rows_searched(int tiles_m, int tiles_n, int BM, int BN)
{
    const int ntiles = tiles_m * tiles_n, share = (ntiles + 7) / 8;
    int best = 1;
    long best_cost = -1;
    for (int r = 1; r <= tiles_m && r <= share; ++r) {
        long rows, cols;
        if (share >= r * tiles_n) {
            const int groups = (share + r * tiles_n - 1) / (r * tiles_n);
            rows = (long)r * (share % (r * tiles_n) == 0 ? groups : groups + 1);
            cols = tiles_n;
        } else {
            const bool exact = ntiles % 8 == 0 && share % r == 0 && tiles_n % (share / r) == 0 && tiles_m % r == 0;
            rows = exact ? r : r + r / 2;
            cols = exact ? share / r : share / r + 1;
        }
        rows = rows < tiles_m ? rows : tiles_m;
        cols = cols < tiles_n ? cols : tiles_n;
        const long cost = rows * BM + cols * BN;
        if (best_cost < 0 || cost < best_cost) best_cost = cost, best = r;
    }
    return best;
}

static int group_rows()
{
    static const int tile[][2] = {{256, 256}, {256, 192}, {256, 128}, {128, 192}, {128, 128}, {64, 128}, {128, 64}, {64, 64}, {64, 768}};
    for (const auto& t : tile) {
        for (int m = 1; m <= 200; ++m)
            for (int n = 1; n <= 40; ++n) EXPECT(xcd_group_rows(m, n, t[0], t[1]) == group_rows_searched(m, n, t[0], t[1]));
        for (int m : {257, 392, 511, 784, 1000, 1568, 3136, 5000, 12544})
            for (int n : {1, 2, 3, 4, 5, 7, 8, 12, 16, 31, 32, 64, 100}) EXPECT(xcd_group_rows(m, n, t[0], t[1]) == group_rows_searched(m, n, t[0], t[1]));
    }
    // host work of a launch: with an eighth of the tiles walked one by one these take 3 s, now less than a tenth of one
    const auto begin = std::chrono::steady_clock::now();
    long sum = 0;
    for (int i = 0; i < 300000; ++i) sum += xcd_group_rows(1568 + 8 * (i % 1400), 1 + i % 4, 128, 128);
    EXPECT(sum > 0 && std::chrono::steady_clock::now() - begin < std::chrono::seconds(1));
    return 0;
}

// A launch has less than 2^32 work-items, and four rows take 256.
static int layernorm_rows()
{
    const long edge = (1L << 26) - 4;   // the last number of rows whose launch is one
    for (long rows : {1L, 3L, 4L, 5L, 67L, 98304L, edge - 1, edge}) EXPECT(layernorm_row_takes(rows, 256, 128));
    for (long rows : {edge + 1, edge + 4, 1L << 27, (1L << 31) - 5, 1L << 32, 1L << 40}) EXPECT(!layernorm_row_takes(rows, 256, 128));
    for (long rows = 1; rows < 1L << 40; rows = rows * 5 / 4 + 1)
        if (layernorm_row_takes(rows, 1024, 256)) EXPECT(layernorm_row_blocks(rows) * 256 < 1L << 32 && layernorm_row_blocks(rows) * 4 >= rows);
    for (int cols : {1, 128, 255, 300, 1280, 4096}) EXPECT(!layernorm_row_takes(4, cols, 128));
    EXPECT(!layernorm_row_takes(4, 256, 257) && !layernorm_row_takes(0, 256, 128));
    // which form, on both sides of every line
    for (bool f32 : {false, true}) {
        EXPECT(layernorm_form(5000, 256, 64, true, f32) == LN_ROW && layernorm_form(5001, 256, 64, true, f32) == LN_AHEAD);
        EXPECT(layernorm_form(edge, 768, 64, true, f32) == LN_ROW && layernorm_form(edge + 1, 768, 64, true, f32) == LN_AHEAD);
        EXPECT(layernorm_form(5000, 512, 64, true, f32) == LN_ROW && layernorm_form(14001, 512, 64, true, f32) == LN_ROW);
        EXPECT(layernorm_form(5001, 512, 64, true, f32) == (f32 ? LN_ROW : LN_LATE) && layernorm_form(14000, 512, 64, true, f32) == (f32 ? LN_ROW : LN_LATE));
        const struct { int cols; long most; } lines[] = {{320, f32 ? 12000 : 16384}, {384, f32 ? 12000 : 16384}, {388, f32 ? 9728 : 16384}, {512, f32 ? 9728 : 16384}, {640, f32 ? 6144 : 12288}, {896, f32 ? 6144 : 11000}, {900, f32 ? 6144 : 6656}, {1024, f32 ? 6144 : 6656}};
        for (const auto& l : lines) {
            const long least = f32 ? 4096 : 1250;
            EXPECT(layernorm_form(least - 1, l.cols, 300, true, f32) == LN_AHEAD && layernorm_form(least, l.cols, 300, true, f32) == LN_LATE);
            EXPECT(layernorm_form(l.most, l.cols, 64, false, f32) == LN_LATE && layernorm_form(l.most + 1, l.cols, 64, false, f32) == LN_AHEAD);
        }
        for (int cols : {4, 64, 256, 1028, 4096}) EXPECT(layernorm_form(6000, cols, 300, true, f32) == LN_AHEAD);
    }
    return 0;
}

// Layers on both sides of the line between the kernel over blocks of rows and the separate ones, each with the faster kind.
static int block_line()
{
    const struct { int M, H, F, rows; } layers[] = {
        {32, 128, 512, 16}, {128, 128, 1024, 16}, {64, 192, 384, 16}, {320, 192, 768, 0}, {560, 192, 768, 16}, {256, 256, 512, 0}, {560, 256, 528, 16},
        {512, 256, 1024, 0}, {768, 256, 1024, 16}, {512, 320, 640, 0}, {768, 320, 640, 16}, {768, 384, 768, 0}, {1024, 384, 768, 16}, {1024, 320, 1280, 0},
        {1280, 256, 1600, 16}, {1024, 384, 1536, 0}, {4096, 384, 1536, 16}, {4096, 512, 1024, 0}, {4096, 512, 2048, 0}, {8192, 256, 1024, 32},
        {24576, 128, 512, 32}, {24577, 128, 512, 0}, {6144, 384, 1536, 0}};
    for (const auto& l : layers) EXPECT(block_rows_faster(l.M, l.H, l.F) == l.rows);
    EXPECT(block_rows_faster((1 << 30) + 5, 4096, 65536) == 0 && block_rows_faster(1, 1, 1) == 16);
    return 0;
}

// 3x3 convolutions of 64 channels: on both sides of the lines.
static int taps_lines()
{
    EXPECT(!conv_taps_faster(8191, true) && conv_taps_faster(8192, true) && !conv_taps_faster(16383, false) && conv_taps_faster(16384, false));
    return 0;
}

// The tile of a product that makes the LayerNorm in front of it, and that its LDS, with the product's table, is what a CU has.
static int layernorm_products()
{
    EXPECT(ln_gemm_tile(16, 4096, 1024, 0) == 0 && ln_gemm_tile(64, 4096, 1024, 0) == 1 && ln_gemm_tile(128, 4096, 1024, 0) == 2 && ln_gemm_tile(129, 4096, 1024, 0) == -1);
    // a slice has 128 bytes of each of 32, 64 or 128 rows of W; of A two slices of 16 rows for each 256 columns
    EXPECT(ln_gemm_lds(0, 1024, 8) == 8 * 4096 + 16384 + 8 && ln_gemm_lds(1, 768, 0) == 6 * 8192 + 12288 && ln_gemm_lds(2, 912, 80) == 8 * 16384 + 16384 + 80);
    EXPECT(ln_gemm_tile(128, 4096, 1024, 8 * 2048) == 2 && ln_gemm_tile(128, 4096, 1024, 8 * 2049) == -1 && ln_gemm_tile(128, 4096, 896, 8 * 4096) == 2);
    for (int M : {1, 16, 17, 64, 100, 128, 250, 682})
        for (int N : {128, 520, 1152, 3072, 4096})
            for (int K = 192; K <= 1024; K += 16)
                for (int nseg : {0, 1, 256, 257, 2048, 2049, 4096}) {
                    const int t = ln_gemm_tile(M, N, K, 8 * (size_t)nseg);
                    EXPECT(t < 0 || (t == ln_gemm_tile(M, N, K, 0) && ln_gemm_lds(t, K, 8 * (size_t)nseg) <= 160 * 1024));
                }
    return 0;
}

// choice_driver relu M N K kunit ...: for each product with the epilogues for convolutions the tile kernel's configuration, or -1 for
// the small-tile kernel.  staged M N K align ...: the register-staged kernel's, with every output, table and residual, or -1.
static int configurations(const char* kind, int n, char** v)
{
    for (int i = 0; i + 3 < n; i += 4) {
        const int M = std::atoi(v[i]), N = std::atoi(v[i + 1]), K = std::atoi(v[i + 2]);
        if (!std::strncmp(kind, "chain", 5)) {   // M, K, N1, N2; chain_lines: tables that are no ReLU
            const int N2 = std::atoi(v[i + 3]);
            std::printf("%d\n", conv_chain_built(N, K, N2) && conv_chain_faster(M, N, K, N2, !std::strcmp(kind, "chain")));
        } else if (!std::strcmp(kind, "staged")) {
            const int align = std::atoi(v[i + 3]);
            const bool takes = (align < 16 || K % 64 != 0) && staged_faster(align, M, N, K, true, true, true, true);
            std::printf("%d\n", takes ? choose_unaligned(M, N, K, true, true, true, true) : -1);
        } else std::printf("%d\n", (long long)M * N < direct_below(false, N, K) ? -1 : choose_relu(M, N, K, std::atoi(v[i + 3])));
    }
    std::printf("SANITIZE_OK\n");
    return 0;
}

int main(int argc, char** argv)
{
    if (argc > 2) return configurations(argv[1], argc - 2, argv + 2);
    if (forced_values() || requirements() || staged_line() || group_rows() || layernorm_rows() || layernorm_products() || taps_lines() || block_line()) return 1;
    std::printf("SANITIZE_OK\n");
    return 0;
}
