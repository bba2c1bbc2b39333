// LayerNorm-PWL and the product behind it in one kernel, for few rows: the product's A operand is given as the fp32 rows in
// front of the LayerNorm, and every workgroup normalises the rows of its tile itself (paper Section 3.2 for the function, Section
// 3.1 for the product; arithmetic and order are those of the separate kernels, so results are bit-identical).
//
// As a kernel of its own the LayerNorm of 128 rows is mostly a launch (2.1 us, of which an empty one is 1.6, and 3.1 of host time) in
// front of a product that takes 4.  Here eight wavefronts of a workgroup normalise BM / 8 rows each, a row at a time as in
// layernorm_row_kernel, and write the codes as the A image of all slices to LDS, while eight others wait for the tile's weights: a
// slice (128 bytes of K, which is at most 1024) of BN rows each, which they multiply then and whose partial tiles meet in LDS.  What
// bounds it is latency: the rows' trip from memory, two reductions, and code that arrives as it is first run (by counter, 128 rows of 768 columns,
// vector instructions issue in 29 % of the cycles, LDS is busy in 7 %, the matrix cores in 2 %).  (With the weights
// requested by the wavefronts that normalise, the counter that tells them of gamma's and beta's arrival made them wait for the weights
// too: 12 layers of width 768 over 128 tokens 310 us instead of 287, weights not in the caches; the kernels apart 305.)  Every column
// tile repeats the work, so the kernel is for products of few rows (ln_gemm_tile, with what it measured); of 32 rows a
// workgroup took 1 to 2 us more than the separate kernels wherever it was tried.
#include "nm_gemm_choice.h"
#include "nm_gemm_common.h"

namespace nm {

struct LnGemmParams {
    const float* x;
    const float* gamma;
    const float* beta;
    const float2* ln_kb;
    const int8_t* W;
    const float* bias;
    int8_t* ln_out;
    int8_t* out_q;
    int M, N, K, ldw, ldo, tiles_m, tiles_n;
    FastDiv div_tiles_m;
    float alpha, out_inv_scale;
    int split_cols;
    float inv3[3];
    float ln_lo, ln_hi, ln_inv_w;
    int ln_nseg, ln_clamp;
    float ln_eps, ln_inv_L, ln_inv_scale;
    const float2* kb;
    float lo, inv_w;
    int nseg;
};

// kC: 1 KB pieces of an fp32 row (K rounded up to 256 columns); kEpi: EPI_Q or EPI_Q_TABLE.
template <int BM, int BN, int kC, int kEpi>
__global__ __launch_bounds__(1024) void gemm_ln_kernel(LnGemmParams p)
{
    constexpr int KW = 8, NT = 64 * KW, R = BM / KW;   // wavefronts and threads of each kind, rows a wavefront normalises
    constexpr int TM = BM / 16, TN = BN / 16, NI = BN / 8;
    constexpr int SLICE = BN * 128;                    // W rows of a slice
    constexpr int G4 = BN / 4, NGRP = BM * G4, GPT = (NGRP + NT - 1) / NT;   // groups of four outputs, ... per thread
    static_assert(NT % G4 == 0 && (NGRP % NT == 0 || NGRP < NT), "groups split evenly");
    static_assert(BM * BN * 4 <= SLICE, "a partial tile fits a slice");
    constexpr auto pslot = [](int row, int slot) { return slot ^ (BN >= 64 ? row & 15 : (row >> 1) & 7); };   // spread over the banks
    constexpr bool kTable = kEpi == EPI_Q_TABLE;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];   // [slices][W rows of 128 bytes], [slices][BM rows of 128 bytes], table

    // all arguments in one step
    asm volatile("" : : "s"(p.x), "s"(p.gamma), "s"(p.beta), "s"(p.ln_kb), "s"(p.W), "s"(p.bias), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.ldw), "s"(p.ldo),
                 "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.div_tiles_m.magic), "s"(p.div_tiles_m.shift), "s"(p.ln_nseg), "s"(p.alpha), "s"(p.out_inv_scale),
                 "s"(p.ln_out), "s"(p.out_q));
    asm volatile("" : : "s"(p.ln_lo), "s"(p.ln_hi), "s"(p.ln_inv_w), "s"(p.ln_clamp), "s"(p.ln_eps), "s"(p.ln_inv_L), "s"(p.ln_inv_scale), "s"(p.split_cols));
    if (kTable) asm volatile("" : : "s"(p.kb), "s"(p.nseg), "s"(p.lo), "s"(p.inv_w));

    const int lane = threadIdx.x & 63, wave16 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wave16 & (KW - 1);
    const bool rows_wave = wave16 < KW;
    // an XCD gets a contiguous eighth of the tiles, rows of tiles innermost
    const int ntiles = p.tiles_m * p.tiles_n, share = (ntiles + 7) >> 3;
    const int id = (blockIdx.x % 8) * share + blockIdx.x / 8;
    if (id >= ntiles) return;
    const int tile_n = (int)quotient((unsigned)id, p.div_tiles_m);
    const int m0 = (id - tile_n * p.tiles_m) * BM, n0 = tile_n * BN;
    const int K = p.K, nk = (K + 127) >> 7;
    int8_t* const s_a = smem + nk * SLICE;
    float2* const s_kb = reinterpret_cast<float2*>(s_a + 2 * kC * BM * 128);

    if (rows_wave) {
        // ---- the rows: accumulator i of the normative sums is lane i ---------------------------------------------------
        v4f x[R][kC], ga[kC], be[kC];
        float2 tab[4];
        const bool last_live = 256 * (kC - 1) + 4 * lane < K;   // (the last piece of a row may be a part of one)
        const int last_col = min(256 * (kC - 1) + 4 * lane, K - 4);
        const auto row_of = [&](int r) { return p.x + (long)min(m0 + wave * R + r, p.M - 1) * K; };   // past the edge: the last one, never stored
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < kC; ++c) x[r][c] = *reinterpret_cast<const v4f*>(row_of(r) + (c < kC - 1 ? 256 * c + 4 * lane : last_col));
#pragma unroll
        for (int c = 0; c < 4; ++c) tab[c] = p.ln_kb[min(lane + 64 * c, p.ln_nseg - 1)];
#pragma unroll
        for (int c = 0; c < kC; ++c) ga[c] = *reinterpret_cast<const v4f*>(p.gamma + (c < kC - 1 ? 256 * c + 4 * lane : last_col));
#pragma unroll
        for (int c = 0; c < kC; ++c) be[c] = *reinterpret_cast<const v4f*>(p.beta + (c < kC - 1 ? 256 * c + 4 * lane : last_col));
        __builtin_amdgcn_sched_barrier(0);
        // (The loop stays rolled: a kernel starts with an empty instruction cache, and the code of two rows at a time took longer
        // to arrive than a row takes.)
#pragma unroll 1
        for (int r = 0; r < R; ++r) {
            v4f d[kC];
            float part = 0.0f;
#pragma unroll
            for (int c = 0; c < kC; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    d[c][q] = c == kC - 1 && !last_live ? 0.0f : x[0][c][q];   // (an accumulator is never -0: adding 0 leaves it as it is)
                    part = part + d[c][q];
                }
#pragma unroll
            for (int t = 1; t < R; ++t)
#pragma unroll
                for (int c = 0; c < kC; ++c) x[t - 1][c] = x[t][c];
            const float mu = group_sum<64>(part) * p.ln_inv_L;
            part = 0.0f;
#pragma unroll
            for (int c = 0; c < kC; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    d[c][q] = c == kC - 1 && !last_live ? 0.0f : d[c][q] - mu;
                    part = __builtin_fmaf(d[c][q], d[c][q], part);
                }
            float u = group_sum<64>(part) * p.ln_inv_L + p.ln_eps;
            const float uc = __builtin_amdgcn_fmed3f(u, p.ln_lo, p.ln_hi);
            u = p.ln_clamp ? uc : u;
            const int seg = __builtin_amdgcn_readfirstlane(seg_index(u, p.ln_lo, p.ln_inv_w, p.ln_nseg));
            float2 e = tab[0];
#pragma unroll
            for (int c = 1; c < 4; ++c) e = seg >> 6 == c ? tab[c] : e;
            e.x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e.x), seg & 63));
            e.y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e.y), seg & 63));
            const float scale = __builtin_fmaf(e.x, u, e.y);
            const int row = wave * R + r;
            // slice 2 c + lane / 32, chunk lane / 4 % 8 of the row, spread as the fragments are read
            int8_t* const to = s_a + ((lane >> 5) * BM + row) * 128 + ((((lane >> 2) & 7) ^ ((row >> 1) & 7)) << 4) + 4 * (lane & 3);
            unsigned w[kC];
#pragma unroll
            for (int c = 0; c < kC; ++c) {
                int q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = requant(__builtin_fmaf(d[c][i] * scale, ga[c][i], be[c][i]), p.ln_inv_scale);
                w[c] = pack4(q[0], q[1], q[2], q[3]);
                if (c == kC - 1 && !last_live) w[c] = 0;   // beyond K the A image is zero, whatever the W slice has there
                *reinterpret_cast<unsigned*>(to + 2 * c * BM * 128) = w[c];
            }
            if (tile_n == 0 && p.ln_out && m0 + row < p.M) {
                int8_t* const out = p.ln_out + (long)(m0 + row) * K + 4 * lane;
#pragma unroll
                for (int c = 0; c < kC; ++c)
                    if (c < kC - 1 || last_live) *reinterpret_cast<unsigned*>(out + 256 * c) = w[c];
            }
        }
        __syncthreads();
        __syncthreads();
        return;
    }

    // ---- the product's wavefronts: a slice each ---------------------------------------------------------------------------
    const int tid = threadIdx.x - NT;
    const int c4 = tid % G4, row0 = tid / G4, nb = n0 + 4 * c4;
    int8_t* const mine = smem + wave * SLICE;
    if (wave < nk) {
        const int lrow = lane >> 3, chunk0 = (lane & 7) ^ (lane >> 4);   // row and chunk of the lane in even pieces; the others: chunk ^ 4
        const unsigned ring = (unsigned)(uintptr_t)mine;
        const unsigned left = (unsigned)(K - 128 * wave - 16);   // the row's last chunk from here: chunks beyond are that one again
        const unsigned ldw = (unsigned)p.ldw, w_row0 = (unsigned)(n0 + lrow) * ldw, w_last = (unsigned)(p.N - 1) * ldw;
#pragma unroll
        for (int b = 0; b < NI; ++b)
            dma16s(p.W + 128 * wave, min(w_row0 + 8u * b * ldw, w_last) + min(16u * (unsigned)(chunk0 ^ ((b & 1) << 2)), left), ring + 1024 * b);
    }
    v4f bias_r = {0.0f, 0.0f, 0.0f, 0.0f};
    if (p.bias) bias_r = *reinterpret_cast<const v4f_a4*>(p.bias + min(nb, p.N - 4));
    if (kTable)
        for (int e = tid; e < p.nseg; e += NT) s_kb[e] = p.kb[e];
    wait_vmcnt<0>();
    __syncthreads();

    const int fr = lane & 15, fq = lane >> 4;
    v4i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4i{0, 0, 0, 0};
    if (wave < nk) {
        const int8_t* const sa = s_a + wave * BM * 128;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int fo = fr * 128 + (((4 * ks + fq) ^ ((fr >> 1) & 7)) << 4);
            v4i fa[TM], fw[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[j] = *reinterpret_cast<const v4i*>(mine + 2048 * j + fo);
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const v4i*>(sa + 2048 * i + fo);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[j], fa[i], acc[i][j], 0, 0, 0);
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");   // its W slice has been read: the partial tile lies over it
    if (wave < nk) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                *reinterpret_cast<v4i*>(mine + (16 * i + fr) * (BN * 4) + 16 * pslot(16 * i + fr, 4 * j + fq)) = acc[i][j];
    }
    __syncthreads();
    if (NGRP < NT && row0 >= BM) return;
    if (nb >= p.N) return;

    v4f inv = {p.out_inv_scale, p.out_inv_scale, p.out_inv_scale, p.out_inv_scale};
    if (!kTable && p.split_cols > 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) inv[e] = nb + e >= 2 * p.split_cols ? p.inv3[2] : nb + e >= p.split_cols ? p.inv3[1] : p.inv3[0];
    }
    v4i a[GPT];
    v4f y[GPT];
#pragma unroll
    for (int t = 0; t < GPT; ++t) {
        const int row = row0 + t * (NT / G4);
        const int8_t* at = smem + row * (BN * 4) + 16 * pslot(row, c4);
        a[t] = *reinterpret_cast<const v4i*>(at);
#pragma unroll
        for (int w = 1; w < KW; ++w)
            if (w < nk) a[t] += *reinterpret_cast<const v4i*>(at + w * SLICE);
    }
#pragma unroll
    for (int t = 0; t < GPT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float v = __builtin_fmaf((float)a[t][e], p.alpha, bias_r[e]);
            if (kTable) {
                const float u = __builtin_amdgcn_fmed3f((v - p.lo) * p.inv_w, 0.0f, (float)(p.nseg - 1));
                const float2 kb = s_kb[(int)u];
                v = __builtin_fmaf(kb.x, v, kb.y);
            }
            y[t][e] = v;
        }
#pragma unroll
    for (int t = 0; t < GPT; ++t) {
        const int m = m0 + row0 + t * (NT / G4);
        if (m < p.M)
            *reinterpret_cast<unsigned*>(p.out_q + (long)m * p.ldo + nb) =
                pack4(requant(y[t][0], inv[0]), requant(y[t][1], inv[1]), requant(y[t][2], inv[2]), requant(y[t][3], inv[3]));
    }
}

template <int BM, int BN, int kC, int kEpi>
static int32_t launch_ln(LnGemmParams& p, hipStream_t s)
{
    auto kern = gemm_ln_kernel<BM, BN, kC, kEpi>;
    static_assert(BM == 16 && (BN == 32 || BN == 64 || BN == 128), "tiles of ln_gemm_lds");
    const size_t shmem = ln_gemm_lds(BN / 64, p.K, kEpi == EPI_Q_TABLE ? sizeof(float2) * (size_t)p.nseg : 0);
    static std::once_flag once;  // one attribute call per instantiation
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(gemm_ln_kernel)");
    });
    if (once_rc) return once_rc;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    p.div_tiles_m = fast_div(p.tiles_m);
    queue_kernel(kern, dim3((p.tiles_m * p.tiles_n + 7) / 8 * 8), dim3(1024), shmem, s, p);
    return check_hip(hipGetLastError(), "LayerNorm + gemm launch");
}
template <int BM, int BN>
static int32_t launch_ln_tile(LnGemmParams& p, bool table, hipStream_t s)
{
    switch ((p.K + 255) / 256) {
    case 1: return table ? launch_ln<BM, BN, 1, EPI_Q_TABLE>(p, s) : launch_ln<BM, BN, 1, EPI_Q>(p, s);
    case 2: return table ? launch_ln<BM, BN, 2, EPI_Q_TABLE>(p, s) : launch_ln<BM, BN, 2, EPI_Q>(p, s);
    case 3: return table ? launch_ln<BM, BN, 3, EPI_Q_TABLE>(p, s) : launch_ln<BM, BN, 3, EPI_Q>(p, s);
    default: return table ? launch_ln<BM, BN, 4, EPI_Q_TABLE>(p, s) : launch_ln<BM, BN, 4, EPI_Q>(p, s);
    }
}

// Whether the kernel takes the LayerNorm n and the product g behind it: whole chunks of at most 1024 columns, rows that follow one
// another, 16-byte rows of x and W, int8 results in whole groups of four, one table of at most 256 segments for the rows (it lies in
// registers).
bool ln_gemm_takes(const LnRows& n, const GemmArgs& g)
{
    return !gemm_switched() && g.K % 16 == 0 && g.K >= 192 && g.K <= 1024 && aligned(n.x, 16) && aligned(n.gamma, 16) && aligned(n.beta, 16) && n.table.nseg <= 256 &&
           (!n.out_q || aligned(n.out_q, 4)) && g.N % 4 == 0 && aligned(g.W, 16) && g.ldw % 16 == 0 && (int64_t)g.N * g.ldw < (1LL << 31) &&
           (!g.bias || aligned(g.bias, 4)) && g.out_q && aligned(g.out_q, 4) && g.ldo % 4 == 0 && g.ldo < (1LL << 31) && !g.out_f32 && !g.out_acc &&
           !g.alpha_vec && !g.resid && !g.out_inv_scale_vec && !g.dbg_seg && !g.conv && !g.w_is_kn && g.outer_count * g.inner_count == 1 &&
           !(g.has_table && (g.table.clamp_input || g.split_cols > 0));
}

int32_t launch_ln_gemm(const LnRows& n, const GemmArgs& g, int tile, hipStream_t s)
{
    LnGemmParams p{};
    p.x = n.x; p.gamma = n.gamma; p.beta = n.beta; p.ln_kb = n.table.kb; p.W = g.W; p.bias = g.bias; p.ln_out = n.out_q; p.out_q = g.out_q;
    p.M = g.M; p.N = g.N; p.K = g.K; p.ldw = (int)g.ldw; p.ldo = (int)g.ldo;
    p.alpha = g.alpha; p.out_inv_scale = g.out_inv_scale; p.split_cols = g.split_cols;
    for (int i = 0; i < 3; ++i) p.inv3[i] = g.inv3[i];
    p.ln_lo = n.table.lo; p.ln_hi = n.table.hi; p.ln_inv_w = n.table.inv_w; p.ln_nseg = n.table.nseg; p.ln_clamp = n.table.clamp_input;
    p.ln_eps = n.eps; p.ln_inv_L = (float)(1.0 / (double)g.K); p.ln_inv_scale = n.inv_scale;
    p.kb = g.table.kb; p.lo = g.table.lo; p.inv_w = g.table.inv_w; p.nseg = g.has_table ? g.table.nseg : 0;
    switch (tile) {
    case 0: return launch_ln_tile<16, 32>(p, g.has_table != 0, s);
    case 1: return launch_ln_tile<16, 64>(p, g.has_table != 0, s);
    default: return launch_ln_tile<16, 128>(p, g.has_table != 0, s);
    }
}

}  // namespace nm
