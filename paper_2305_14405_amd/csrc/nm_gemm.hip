// int8 x int8 -> int32 GEMM on the gfx950 matrix cores with the fused epilogue
// (dequantise, bias, residual, PWL table lookup from LDS, requantise), plus the two attention
// products, which are the same kernel launched over (batch, head) with strided operands.
//
// Paper basis: Section 3.1 (fully connected layers, attention and residual additions are matrix
// multiplications / additions) and Section 3.2 (the nonlinearity after a linear operator is the
// element-wise PWL calculation y = k[s]*x + b[s]).  The paper blocks its matrices for a systolic
// array with a three-level buffer hierarchy; here the blocking is for CDNA4: a workgroup of four or
// eight wavefronts owns a BM x BN tile of the output, the k-loop streams 64- or 128-byte slices of
// both operands through a ring of LDS stages, and each wavefront issues 32x32x32 int8 MFMAs on its
// WM x WN sub-tile with int32 accumulators that never leave registers until the epilogue.
// Here: gemm_stream_kernel (aligned operands, K a multiple of 64: operands go global -> LDS
// directly; also gathers the rows of a convolution's patch matrix on the fly) in several tile
// configurations, and gemm_pwl_kernel (any shape and alignment, W as [N,K] or [K,N], operands through
// registers); large plain products take the tile kernel (nm_gemm_tile.h), small outputs the small-tile
// kernel (nm_gemm_direct.hip), and unaligned operands that one or the register-staged tile kernel
// (nm_gemm_unaligned.hip).  launch_gemm chooses.
//
// Operand roles: the MFMA's first operand supplies the rows of its 32x32 result and the second
// the columns.  W rows (output columns n) go first and A rows (output rows m) second, so a lane
// ends up with one output row m and, per group of four accumulator registers, four consecutive
// output columns n: four int8 results pack into one 32-bit store and bias / per-column scales
// are read as four consecutive floats.
//
// Both operands are K-contiguous, which is what the int8 MFMA wants: a lane feeds 16 consecutive
// k of one row.  The same k of A and W always meet in the same (lane group, byte) slot, and int32
// addition is exact, so results do not depend on tiling, on the k order or on any split of K.
#include <cstdlib>

#include "nm_gemm_common.h"
#include "nm_gemm_tile.h"

namespace nm {

// Debug switch: NM_GEMM_GENERIC=1 in the environment sends every shape to the generic kernel.
static bool force_generic()
{
    static const bool v = [] { const char* e = getenv("NM_GEMM_GENERIC"); return e && e[0] == '1'; }();
    return v;
}
// Debug switch NM_GEMM_CFG (tuning aid), read once per process.
static ForcedCfg forced_cfg()
{
    static const ForcedCfg v = parse_forced_cfg(getenv("NM_GEMM_CFG"));
    return v;
}

bool gemm_switched() { return force_generic() || forced_cfg().kind != FORCED_NONE; }

// 16 bytes of a row-major int8 matrix at (row, k .. k+15); zeros outside [0,nrows) x [0,K).
template <bool kAligned>
__device__ __forceinline__ v4i load_chunk(const int8_t* __restrict__ X, long ld, int row, int nrows,
                                          int k, int K)
{
    v4i v = {0, 0, 0, 0};
    if (row < nrows) {
        const int8_t* p = X + (long)row * ld + k;
        if (kAligned) {
            if (k < K) v = *reinterpret_cast<const v4i*>(p);
        } else {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                unsigned word = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (k + 4 * w + b < K) word |= (unsigned)(uint8_t)p[4 * w + b] << (8 * b);
                v[w] = (int)word;
            }
        }
    }
    return v;
}

// ---------------------------------------------------------------------------------------------
// Generic kernel: any shape and alignment, W as [N, K] or [K, N].  Operands go global -> registers
// -> LDS (two stages); out-of-range rows and the k tail are zero-filled.
// ---------------------------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, bool kAligned, bool kWKN>
__global__ __launch_bounds__(kGemmThreads) void gemm_pwl_kernel(GemmParams p)
{
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int WAVES_N = BN / WN;
    static_assert((BM / WM) * (BN / WN) == kGemmThreads / 64, "four wavefronts per workgroup");
    constexpr int LA = BM / 64, LW = BN / 64;  // 16-byte chunks per thread and stage

    __shared__ __attribute__((aligned(16))) int8_t sA[2][BM * kBK];
    __shared__ __attribute__((aligned(16))) int8_t sW[2][BN * kBK];
    extern __shared__ float2 s_kb[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wave_m = (wave / WAVES_N) * WM;
    const int wave_n = (wave % WAVES_N) * WN;

    const int tile_m = blockIdx.x % p.tiles_m;
    const int tile_n = blockIdx.x / p.tiles_m;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int outer = blockIdx.y / p.inner_count;
    const int inner = blockIdx.y % p.inner_count;
    const int8_t* __restrict__ A = p.A + outer * p.a_outer + inner * p.a_inner;
    const int8_t* __restrict__ W = p.W + outer * p.w_outer + inner * p.w_inner;
    const long obase = outer * p.o_outer + inner * p.o_inner;

    if (p.has_table) { if (p.table.cellmap) stage_table_two_level(s_kb, p.table); else stage_table(s_kb, p.table); }

    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    v4i ra[LA], rw[LW];
    const int ld_row = tid >> 2, ld_chunk = tid & 3;

    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < LA; ++i)
            ra[i] = load_chunk<kAligned>(A, p.lda, m0 + ld_row + 64 * i, p.M, k0 + 16 * ld_chunk, p.K);
        if (!kWKN) {
#pragma unroll
            for (int i = 0; i < LW; ++i)
                rw[i] = load_chunk<kAligned>(W, p.ldw, n0 + ld_row + 64 * i, p.N, k0 + 16 * ld_chunk, p.K);
        } else {
            // W is [K, N]: this thread takes k-row kk and 16 consecutive n
#pragma unroll
            for (int i = 0; i < LW; ++i) {
                const int idx = tid + kGemmThreads * i;  // 0 .. 64 * BN/16 - 1
                const int kk = idx / (BN / 16), nc = idx % (BN / 16);
                rw[i] = load_chunk<kAligned>(W, p.ldw, k0 + kk, p.K, n0 + 16 * nc, p.N);
            }
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < LA; ++i)
            *reinterpret_cast<v4i*>(&sA[buf][lds_off(ld_row + 64 * i, ld_chunk)]) = ra[i];
        if (!kWKN) {
#pragma unroll
            for (int i = 0; i < LW; ++i)
                *reinterpret_cast<v4i*>(&sW[buf][lds_off(ld_row + 64 * i, ld_chunk)]) = rw[i];
        } else {
#pragma unroll
            for (int i = 0; i < LW; ++i) {
                const int idx = tid + kGemmThreads * i;
                const int kk = idx / (BN / 16), nc = idx % (BN / 16);
#pragma unroll
                for (int b = 0; b < 16; ++b) {
                    const int n = 16 * nc + b;
                    sW[buf][lds_off(n, kk >> 4) + (kk & 15)] = (int8_t)((unsigned)rw[i][b >> 2] >> (8 * (b & 3)));
                }
            }
        }
    };

    const int nk = (p.K + kBK - 1) / kBK;
    fetch(0);
    stash(0);
    __syncthreads();

    const int frag_row = lane & 31, frag_half = lane >> 5;
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) fetch((kt + 1) * kBK);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            v4i fa[TM], fw[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[i] = *reinterpret_cast<const v4i*>(&sA[cur][lds_off(wave_m + 32 * i + frag_row, 2 * ks + frag_half)]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fw[j] = *reinterpret_cast<const v4i*>(&sW[cur][lds_off(wave_n + 32 * j + frag_row, 2 * ks + frag_half)]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[j], fa[i], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) stash(cur ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int nb = n0 + wave_n + 32 * j + 8 * g + 4 * frag_half;
            if (nb >= p.N) continue;
            const bool vec = p.vec_out && nb + 3 < p.N;
            Col4 c;
            load_cols<EPI_GENERIC>(p, nb, c);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int m = m0 + wave_m + 32 * i + frag_row;
                if (m >= p.M) continue;
                const long rowoff = obase + (long)m * p.ldo;
                int a4[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) a4[e] = acc[i][j][4 * g + e];
                int r4[4] = {0, 0, 0, 0};
                if (p.resid) load_resid4(p, rowoff, nb, vec, r4);
                Epi4 o;
                epi_math<EPI_GENERIC>(p, s_kb, a4, c, r4, o);
                epi_store<EPI_GENERIC>(p, rowoff, nb, a4, o, vec, false);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Streaming kernel: K a multiple of 64 (of BK), 16-byte aligned rows, W as [N, K].  Operands go global -> LDS directly (global_load_lds_dwordx4: a wavefront
// instruction moves 64 x 16 bytes into 1 KB of consecutive LDS, no registers in between) through
// a ring of kStages stages; a wavefront waits with an explicit vmcnt for the stage it is about to
// use while the loads of the later stages stay in flight.  The LDS image of a stage is
// (BM + BN) rows of BK bytes: 1 KB of consecutive rows per wavefront instruction, with the chunk
// swizzle applied on the global side (with 64-byte rows lane p of an instruction fetches row p/4,
// logical chunk (p%4) ^ swz(row)).  Rows past the matrix edge are clamped to the last row: they only feed
// accumulators that are never stored.
// Workgroups are numbered so that the eight XCDs (workgroup id mod 8) each own a compact block of
// output tiles: the A rows and W rows a block needs fit that XCD's L2.
// int8 output goes through a per-wavefront LDS patch so that rows leave as 16-byte stores.
// ---------------------------------------------------------------------------------------------
// LDS offset of (row, 16-byte chunk) for rows of BK bytes.  BK = 64: four chunks, the swizzle of
// the generic kernel.  BK = 128: eight chunks, 16 consecutive rows spread over all chunk positions
// of two adjacent rows' worth of banks.
// KSPLIT = 2 doubles the wavefronts of a workgroup without shrinking the wavefront tile: two
// wavefronts share each WM x WN sub-tile and take alternate 32-byte k-steps of every k-slice (so
// the LDS read traffic and the operand traffic stay those of the KSPLIT = 1 kernel, while each
// SIMD has two wavefronts whose LDS waits and MFMAs overlap).  After the main loop the two swap
// halves of their int32 partial accumulators through LDS (integer addition is exact in any
// order) and each finishes half of the sub-tile's rows, which also halves the epilogue per
// wavefront.  Used where the grid has fewer workgroups than CUs times two (N = 768 GEMMs).
//
// kConv: the A operand is gathered from an NHWC image (convolution as a matrix product, paper
// Section 3.1).  A k-slice never straddles a filter tap (Cin % BK == 0), so for the slice of tap
// (i, j) and channels c0.. a lane's 16 bytes are x[b, ho*stride - pad + i, wo*stride - pad + j,
// c0 + 16*chunk ..] or, in the padding, 16 bytes of the zero line; only the per-lane source
// address of the direct global -> LDS load changes, the rest of the kernel is the same.
// Wavefronts per SIMD the register allocation should leave room for: as many workgroups per CU as
// the operand ring lets LDS hold (small rings exist so that several workgroups overlap), at most 3.
constexpr int stream_waves_per_simd(int ring_bytes, int waves)
{
    const int wgs = ring_bytes <= 49152 ? 3 : ring_bytes <= 73728 ? 2 : 1;
    const int w = wgs * waves / 4;
    return w < 1 ? 1 : w > 3 ? 3 : w;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int KSPLIT, int BK, int kStages, int kEpi, bool kConv = false>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * KSPLIT,
                             stream_waves_per_simd(kStages * (BM + BN) * BK, WAVES_M * WAVES_N * KSPLIT))
void gemm_stream_kernel(GemmParams p)
{
    constexpr int NWT = WAVES_M * WAVES_N;       // wavefront tiles per workgroup
    constexpr int NW = NWT * KSPLIT;             // wavefronts per workgroup
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int TMF = TM / KSPLIT;             // 32-row blocks a wavefront finishes
    constexpr int ROWS = BM + BN;
    constexpr int CPR = BK / 16;                 // 16-byte chunks per LDS row
    constexpr int RPI = 64 / CPR;                // rows moved by one wavefront instruction (1 KB)
    constexpr int NBLK = ROWS / RPI;             // 1 KB blocks per stage
    constexpr int LB = (NBLK + NW - 1) / NW;     // blocks per wavefront (some have LB - 1)
    constexpr int STAGE_BYTES = ROWS * BK;
    constexpr int SW = WN + 16;                  // row stride of the int8 output patch
    constexpr int KS = BK / 32;                  // MFMA k-steps per k-slice
    constexpr int KSW = KS / KSPLIT;             // ... per wavefront
    static_assert(BK == 64 || BK == 128, "k-slice of 64 or 128 bytes");
    static_assert(KSPLIT == 1 || KSPLIT == 2, "one or two wavefronts per sub-tile");
    static_assert(TM % KSPLIT == 0 && KS % KSPLIT == 0, "halves split evenly");
    static_assert(BM % 32 == 0 && BN % 32 == 0 && ROWS % RPI == 0, "tile shape");
    static_assert(WM * SW * NWT <= kStages * STAGE_BYTES, "output patch fits the operand ring");
    static_assert(KSPLIT == 1 || NW * TMF * TN * 4096 <= kStages * STAGE_BYTES, "exchange fits the ring");
    static_assert(kStages >= 2 && kStages <= 4, "ring depth");

    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    float* s_cols = reinterpret_cast<float*>(smem + kStages * STAGE_BYTES);  // scale | bias | inv, BN each
    float2* s_kb = reinterpret_cast<float2*>(s_cols + 3 * BN);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_t = wave % NWT;               // which sub-tile
    const int kg = wave / NWT;                   // which half of the k-steps (0 when KSPLIT == 1)
    const int wave_m = (wave_t / WAVES_N) * WM;
    const int wave_n = (wave_t % WAVES_N) * WN;

    // every argument of the prologue in one step (left alone, the compiler fetches them in eight dependent ones)
    asm volatile("" : : "s"(p.A), "s"(p.W), "s"(p.bias), "s"(p.alpha_vec), "s"(p.resid), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.lda), "s"(p.ldw),
                 "s"(p.ldo), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.alpha), "s"(p.out_inv_scale), "s"(p.has_table), "s"(p.batched),
                 "s"(p.r16), "s"(p.split_cols), "s"(p.table.kb), "s"(p.table.nseg), "s"(p.table.cellmap), "s"(p.div_group.magic),
                 "s"(p.div_group.shift));
    if (kConv)
        asm volatile("" : : "s"(p.cH), "s"(p.cW), "s"(p.cCin), "s"(p.cKw), "s"(p.cStride), "s"(p.cPad), "s"(p.cWo), "s"(p.cHo), "s"(p.div_wo.magic),
                     "s"(p.div_wo.shift), "s"(p.div_ho.magic), "s"(p.div_ho.shift));
    // XCD-aware tile order: ids that share (id mod 8) are renumbered to be consecutive, then
    // consecutive ids fill groups of 8 tile rows column by column
    int id = blockIdx.x;
    const int ntiles = p.tiles_m * p.tiles_n;
    if (ntiles % 8 == 0) id = (id % 8) * (ntiles / 8) + id / 8;
    constexpr int GM = 8;
    const int group = (int)quotient((unsigned)id, p.div_group);   // by GM * tiles_n
    const int first_m = group * GM;
    const int gm = min(GM, p.tiles_m - first_m);
    const int in_group = id - group * GM * p.tiles_n;
    const int tile_n = gm == GM ? in_group / GM : in_group / gm;
    const int tile_m = first_m + in_group - tile_n * gm;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int8_t* __restrict__ A = p.A;
    const int8_t* __restrict__ W = p.W;
    long obase = 0;
    if (p.batched) {
        const int outer = blockIdx.y / p.inner_count, inner = blockIdx.y % p.inner_count;
        A += outer * p.a_outer + inner * p.a_inner;
        W += outer * p.w_outer + inner * p.w_inner;
        obase = outer * p.o_outer + inner * p.o_inner;
    }

    // per-lane source pointers of this wavefront's blocks (k = 0)
    const int8_t* src[LB];
    int conv_h[LB], conv_w[LB];  // kConv, A rows: top-left input coordinate of the lane's output position
    const bool has_last = wave + (LB - 1) * NW < NBLK;  // wave-uniform
#pragma unroll
    for (int b = 0; b < LB; ++b) {
        int blk = wave + b * NW;
        if (blk >= NBLK) blk = wave;  // unused slot
        const int r = blk * RPI + lane / CPR;
        const int chunk = (lane % CPR) ^ swz_bk<BK>(r);
        conv_h[b] = 0; conv_w[b] = 0;
        if (r < BM) {
            const int m = min(m0 + r, p.M - 1);
            if (kConv) {
                const int t = (int)quotient((unsigned)m, p.div_wo), wo = m - t * p.cWo;
                const int bi = (int)quotient((unsigned)t, p.div_ho), ho = t - bi * p.cHo;
                conv_h[b] = ho * p.cStride - p.cPad;
                conv_w[b] = wo * p.cStride - p.cPad;
                src[b] = A + (long)bi * p.cH * p.cW * p.cCin + 16 * chunk;  // image base + chunk
            } else {
                src[b] = A + (long)m * p.lda + 16 * chunk;
            }
        } else {
            src[b] = W + (long)min(n0 + r - BM, p.N - 1) * p.ldw + 16 * chunk;
        }
    }
    const unsigned lds_base = (unsigned)(uintptr_t)smem;
    // Issue the loads of k-slice kt into ring slot `stage`; with parts > 1 only the blocks b with
    // b % parts == part, so that the issue slots can be spread between the MFMAs of the main loop
    // (a wavefront issues in order: a burst of LB loads would stall its MFMA stream).
    // kConv: slices are issued in increasing kt, so the tap (ti, tj) and the channel offset tc of
    // the slice being issued are kept as running (wave-uniform) counters.
    int ti = 0, tj = 0, tc = 0;
    const int8_t* zero_src = g_zero_line + 16 * (lane % CPR);
    auto issue = [&](int kt, int stage, int part, int parts) {
        const unsigned dst = lds_base + stage * STAGE_BYTES + wave * 1024;
#pragma unroll
        for (int b = 0; b < LB; ++b)
            if (b % parts == part && (b < LB - 1 || has_last)) {
                const int blk = wave + b * NW;
                if (kConv && blk * RPI < BM) {  // wave-uniform: an A block
                    // offsets inside one image fit 32 bits (checked on the host): cheap integer
                    // arithmetic and one select instead of 64-bit multiplies under a branch
                    const int hi = conv_h[b] + ti, wi = conv_w[b] + tj;
                    const bool inside = (unsigned)hi < (unsigned)p.cH && (unsigned)wi < (unsigned)p.cW;
                    const int off = (hi * p.cW + wi) * p.cCin + tc;
                    const int8_t* g = inside ? src[b] + off : zero_src;
                    dma16(g, dst + b * NW * 1024);
                } else {
                    dma16(src[b] + (long)kt * BK, dst + b * NW * 1024);
                }
            }
        if (kConv && part == parts - 1) {  // the slice is complete: advance to the next one
            tc += BK;
            if (tc == p.cCin) { tc = 0; if (++tj == p.cKw) { tj = 0; ++ti; } }
        }
    };

    const int nk = p.K / BK;
#pragma unroll
    for (int st = 0; st < kStages - 1; ++st)
        if (st < nk) issue(st, st, 0, 1);

    // Behind the first slices, what only the epilogue reads; it stays in registers until the products are done.  (In
    // front of them, each waited for on its way to LDS, the table and the columns' vectors kept the first slice from
    // being requested for two memory round trips.)
    // The specialised residual epilogues read the int8 residual rows this wavefront will finish with 16-byte
    // row loads; after the main loop they pass through the (then free) LDS patch to the lanes that need them.
    // Every lane makes every load (rows and columns past the edge: the last ones), so that their number is known
    // to the waits of the main loop.
    constexpr bool kResid8 = kEpi == EPI_F32_RESID || kEpi == EPI_Q_TABLE_RESID;
    constexpr int RCPR = WN / 16;                 // 16-byte chunks per residual row of the sub-tile
    constexpr int RCH = 32 * TMF * RCPR;          // chunks of the rows this wavefront finishes
    constexpr int RL = RCH / 64;
    static_assert(RCH % 64 == 0, "chunks split evenly");
    v4i rpre[RL];
    const bool resid_rows = kResid8 && p.r16;     // uniform
    if (resid_rows) {
#pragma unroll
        for (int t = 0; t < RL; ++t) {
            const int c = lane + 64 * t;
            const int mr = min(m0 + wave_m + 32 * (kg * TMF) + c / RCPR, p.M - 1), n = min(n0 + wave_n + 16 * (c % RCPR), p.N - 16);
            rpre[t] = *reinterpret_cast<const v4i*>(p.resid + obase + (long)mr * p.ldo + n);
        }
    }
    static_assert(BN <= 64 * NW, "a column per thread");
    float col_scale = p.alpha, col_bias = 0.0f, col_inv = p.out_inv_scale;
    if (kEpi != EPI_ACC) {
        const int n = min(n0 + min(tid, BN - 1), p.N - 1);
        if (p.bias) col_bias = p.bias[n];
        if (p.alpha_vec) col_scale = p.alpha_vec[n];
        if (kEpi == EPI_GENERIC && p.out_inv_scale_vec) col_inv = p.out_inv_scale_vec[n];
        else if (p.split_cols > 0) col_inv = n >= 2 * p.split_cols ? p.inv3[2] : (n >= p.split_cols ? p.inv3[1] : p.inv3[0]);
    }
    float2 kb_reg = make_float2(0.0f, 0.0f);   // one table entry (and word of a cell map) per thread; a larger table is staged late
    unsigned map_reg = 0;
    if (p.has_table) {
        if (p.table.cellmap) {
            kb_reg = p.table.ckb[min(tid, p.table.nkb - 1)];
            map_reg = reinterpret_cast<const unsigned*>(p.table.cellmap)[min(tid, (p.table.nseg + 3) / 4 - 1)];
        } else {
            kb_reg = p.table.kb[min(tid, p.table.nseg - 1)];
        }
    }

    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    const int frag_row = lane & 31, frag_half = lane >> 5;
    // LDS offsets of this lane's fragments inside a stage, per k-step this wavefront owns
    int offA[KSW][TM], offW[KSW][TN];
#pragma unroll
    for (int kk = 0; kk < KSW; ++kk) {
        const int ks = KSPLIT == 1 ? kk : kg + KSPLIT * kk;
#pragma unroll
        for (int i = 0; i < TM; ++i) offA[kk][i] = lds_off_bk<BK>(wave_m + 32 * i + frag_row, 2 * ks + frag_half);
#pragma unroll
        for (int j = 0; j < TN; ++j) offW[kk][j] = BM * BK + lds_off_bk<BK>(wave_n + 32 * j + frag_row, 2 * ks + frag_half);
    }
    int stage = 0;
    for (int kt = 0; kt < nk; ++kt) {
        // The loads of stage kt are older than those of the stages issued after it: wait until only
        // the younger ones are in flight.  `young` = number of younger stages already issued.
        const int young = min(kStages - 2, nk - 1 - kt);
        if (kResid8 && resid_rows && kt < kStages - 1) {   // the residual's loads are younger still
            if (young <= 0) wait_vmcnt<RL>();
            else if (young == 1) { if (has_last) wait_vmcnt<LB + RL>(); else wait_vmcnt<LB - 1 + RL>(); }
            else { if (has_last) wait_vmcnt<2 * LB + RL>(); else wait_vmcnt<2 * (LB - 1) + RL>(); }
        } else if (young <= 0) wait_vmcnt<0>();
        else if (young == 1) { if (has_last) wait_vmcnt<LB>(); else wait_vmcnt<LB - 1>(); }
        else { if (has_last) wait_vmcnt<2 * LB>(); else wait_vmcnt<2 * (LB - 1)>(); }
        __syncthreads();  // stage kt has landed for every wavefront; stage kt - 1 is free again
        int nxt = stage + kStages - 1;
        if (nxt >= kStages) nxt -= kStages;
        const bool more = kt + kStages - 1 < nk;
        const int8_t* st = smem + stage * STAGE_BYTES;
#pragma unroll
        for (int kk = 0; kk < KSW; ++kk) {
            v4i fa[TM], fw[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const v4i*>(st + offA[kk][i]);
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[j] = *reinterpret_cast<const v4i*>(st + offW[kk][j]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[j], fa[i], acc[i][j], 0, 0, 0);
            if (more) issue(kt + kStages - 1, nxt, kk, KSW);  // in the shadow of the MFMAs just issued
        }
        stage = stage + 1 == kStages ? 0 : stage + 1;
    }

    if (kEpi != EPI_ACC && tid < BN) {
        s_cols[tid] = col_scale;
        s_cols[BN + tid] = col_bias;
        s_cols[2 * BN + tid] = col_inv;
    }
    if (p.has_table) {
        if (p.table.cellmap) {
            unsigned* map = reinterpret_cast<unsigned*>(s_kb + p.table.nkb);
            const int nw = (p.table.nseg + 3) / 4;
            if (tid < p.table.nkb) s_kb[tid] = kb_reg;
            if (tid < nw) map[tid] = map_reg;
            for (int e = tid + 64 * NW; e < p.table.nkb; e += 64 * NW) s_kb[e] = p.table.ckb[e];
            for (int e = tid + 64 * NW; e < nw; e += 64 * NW) map[e] = reinterpret_cast<const unsigned*>(p.table.cellmap)[e];
        } else {
            if (tid < p.table.nseg) s_kb[tid] = kb_reg;
            for (int e = tid + 64 * NW; e < p.table.nseg; e += 64 * NW) s_kb[e] = p.table.kb[e];
        }
    }

    // ---- combine the two k-halves (KSPLIT == 2): swap accumulator halves through LDS ----------
    v16i fin[TMF][TN];
    __syncthreads();  // every wavefront is done with the ring
    if (KSPLIT == 2) {
        int* xch = reinterpret_cast<int*>(smem);
        const int mine = (wave_t * 2 + kg) * (TMF * TN * 1024), other = (wave_t * 2 + (1 - kg)) * (TMF * TN * 1024);
#pragma unroll
        for (int i = 0; i < TMF; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)  // give away the row blocks the partner finishes
                    xch[mine + ((i * TN + j) * 16 + v) * 64 + lane] = kg == 0 ? acc[TMF + i][j][v] : acc[i][j][v];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TMF; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    fin[i][j][v] = (kg == 0 ? acc[i][j][v] : acc[TMF + i][j][v]) + xch[other + ((i * TN + j) * 16 + v) * 64 + lane];
        __syncthreads();  // the exchange area is about to become the output patch
    } else {
#pragma unroll
        for (int i = 0; i < TMF; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) fin[i][j] = acc[i][j];
    }
    const int row_blk0 = kg * TMF;  // first 32-row block of the sub-tile this wavefront finishes

    // ---- epilogue ------------------------------------------------------------------------------
    const bool patch_q = (kEpi == EPI_GENERIC || kEpi == EPI_Q || kEpi == EPI_Q_TABLE || kEpi == EPI_Q_TABLE_RESID) &&
                         p.out_q != nullptr && p.q16;  // uniform: int8 rows leave through LDS
    int8_t* patch = smem + wave_t * (WM * SW);
    // the specialised residual epilogue fetches all of the lane's residual words up front
    unsigned resw[TMF][TN][4];
    if (resid_rows) {
#pragma unroll
        for (int t = 0; t < RL; ++t) {
            const int c = lane + 64 * t;
            if (c < RCH) *reinterpret_cast<v4i*>(patch + (32 * row_blk0 + c / RCPR) * SW + 16 * (c % RCPR)) = rpre[t];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int i = 0; i < TMF; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    resw[i][j][g] = *reinterpret_cast<const unsigned*>(
                        patch + (32 * (row_blk0 + i) + frag_row) * SW + 32 * j + 8 * g + 4 * frag_half);
        // the patch is reused for the output rows: every lane's reads come first
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else if (kEpi == EPI_F32_RESID || kEpi == EPI_Q_TABLE_RESID) {
#pragma unroll
        for (int i = 0; i < TMF; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int m = m0 + wave_m + 32 * (row_blk0 + i) + frag_row;
                    const int nb = n0 + wave_n + 32 * j + 8 * g + 4 * frag_half;
                    resw[i][j][g] = 0;
                    if (m < p.M && nb + 3 < p.N)
                        resw[i][j][g] = *reinterpret_cast<const unsigned*>(p.resid + obase + (long)m * p.ldo + nb);
                }
    }
    // Row blocks outermost: as soon as a block of 32 rows is finished its int8 rows are read back
    // from the patch and stored, so the stores of one block overlap the arithmetic of the next
    // (the patch rows of a block are written and read by the same wavefront: no workgroup barrier).
    // The body exists twice: for a tile that lies wholly inside the output (and vector-aligned
    // outputs) every bounds test is a compile-time constant, which leaves straight-line code whose
    // table look-ups the scheduler can batch; edge tiles take the guarded copy.
    // Full tiles through a table of two segments compare instead of gathering; where that table is a ReLU
    // (and the columns' scales and biases cannot make a sum infinite), clamping the code at 0 is all of it:
    // 4.75 vector instructions per element less of the 19 the residual epilogue issued (ResNet-50, 64 images:
    // the 1x1 convolutions with shortcut 35 -> 30, 23 -> 21 and 17 -> 15 us, all of it 1.127 -> 1.051 ms).
    auto finish_rows = [&](auto full_c, auto form_c) {
        constexpr bool kFullTile = decltype(full_c)::value;
        constexpr bool kTwoSeg = decltype(form_c)::value == FORM_TWO_SEGMENTS, kRelu = decltype(form_c)::value == FORM_RELU;
#pragma unroll
        for (int i = 0; i < TMF; ++i) {
            const int prow = 32 * (row_blk0 + i) + frag_row;  // row inside the sub-tile
            const int m = m0 + wave_m + prow;
            const long rowoff = obase + (long)m * p.ldo;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int cl = wave_n + 32 * j + 8 * g + 4 * frag_half;  // column inside the tile
                    const int nb = n0 + cl;
                    if (!kFullTile && (nb >= p.N || m >= p.M)) continue;
                    const bool vec = kFullTile || (p.vec_out && nb + 3 < p.N);
                    Col4 c;
                    {
                        const v4f sc = *reinterpret_cast<const v4f*>(s_cols + cl);
                        const v4f bi = *reinterpret_cast<const v4f*>(s_cols + BN + cl);
                        v4f iv = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                        if (!kRelu) iv = *reinterpret_cast<const v4f*>(s_cols + 2 * BN + cl);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { c.scale[e] = sc[e]; c.bias[e] = bi[e]; c.inv[e] = iv[e]; }
                    }
                    int a4[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) a4[e] = fin[i][j][4 * g + e];
                    int r4[4] = {0, 0, 0, 0};
                    if (kEpi == EPI_F32_RESID || kEpi == EPI_Q_TABLE_RESID) {
                        if (kFullTile || nb + 3 < p.N) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) r4[e] = (int)(int8_t)(resw[i][j][g] >> (8 * e));
                        } else {
                            load_resid4(p, rowoff, nb, false, r4);
                        }
                    } else if (kEpi == EPI_GENERIC && p.resid) {
                        load_resid4(p, rowoff, nb, vec, r4);
                    }
                    if (kRelu) {
                        unsigned w = 0;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float v = __builtin_fmaf((float)a4[e], c.scale[e], c.bias[e]);
                            if (kEpi == EPI_Q_TABLE_RESID) v = __builtin_fmaf((float)r4[e], p.resid_scale, v);
                            w = relu_requant(v, p.out_inv_scale, e, w);
                        }
                        *reinterpret_cast<unsigned*>(patch + prow * SW + 32 * j + 8 * g + 4 * frag_half) = w;
                        continue;
                    }
                    Epi4 o;
                    epi_math<kEpi, kTwoSeg>(p, s_kb, a4, c, r4, o);
                    epi_store<kEpi>(p, rowoff, nb, a4, o, vec, patch_q);
                    if (patch_q)
                        *reinterpret_cast<unsigned*>(patch + prow * SW + 32 * j + 8 * g + 4 * frag_half) =
                            pack4(o.q[0], o.q[1], o.q[2], o.q[3]);
                }
            }
            if (patch_q) {
                // same wavefront wrote these 32 patch rows: order its LDS writes before its reads
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                constexpr int PCPR = WN / 16;  // 16-byte chunks per patch row
                for (int c = lane; c < 32 * PCPR; c += 64) {
                    const int row = 32 * (row_blk0 + i) + c / PCPR, cc = c % PCPR;
                    const int mr = m0 + wave_m + row, n = n0 + wave_n + 16 * cc;
                    if (kFullTile || (mr < p.M && n < p.N)) {
                        const v4i v = *reinterpret_cast<const v4i*>(patch + row * SW + 16 * cc);
                        int8_t* dst = p.out_q + obase + (long)mr * p.ldo + n;
                        if (kFullTile || n + 15 < p.N) {
                            *reinterpret_cast<v4i*>(dst) = v;
                        } else {
                            for (int b = 0; b < 16 && n + b < p.N; ++b)
                                dst[b] = (int8_t)((unsigned)v[b >> 2] >> (8 * (b & 3)));
                        }
                    }
                }
            }
        }
    };
    using Any = std::integral_constant<int, FORM_ANY>;
    if (m0 + BM <= p.M && n0 + BN <= p.N && p.vec_out) {
        if constexpr (kEpi == EPI_Q_TABLE || kEpi == EPI_Q_TABLE_RESID) {
            bool relu = p.relu && patch_q;
            if (relu) {
                for (int c = lane; c < WN; c += 64) relu = relu && relu_finite(s_cols[wave_n + c], s_cols[BN + wave_n + c]);
                relu = __all(relu);
            }
            if (relu) finish_rows(std::true_type{}, std::integral_constant<int, FORM_RELU>{});
            else if (p.table.two_seg) finish_rows(std::true_type{}, std::integral_constant<int, FORM_TWO_SEGMENTS>{});
            else finish_rows(std::true_type{}, Any{});
        } else {
            finish_rows(std::true_type{}, Any{});
        }
    } else {
        finish_rows(std::false_type{}, Any{});
    }
}

template <int BM, int BN, int WM, int WN>
static void launch_cfg(const GemmParams& p, bool al, bool wkn, dim3 grid, size_t shmem, hipStream_t s)
{
    if (al && !wkn) queue_kernel(gemm_pwl_kernel<BM, BN, WM, WN, true, false>, grid, dim3(kGemmThreads), shmem, s, p);
    else if (!al && !wkn) queue_kernel(gemm_pwl_kernel<BM, BN, WM, WN, false, false>, grid, dim3(kGemmThreads), shmem, s, p);
    else if (al && wkn) queue_kernel(gemm_pwl_kernel<BM, BN, WM, WN, true, true>, grid, dim3(kGemmThreads), shmem, s, p);
    else queue_kernel(gemm_pwl_kernel<BM, BN, WM, WN, false, true>, grid, dim3(kGemmThreads), shmem, s, p);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int KSPLIT, int BK, int kStages, int kEpi, bool kConv = false>
static int32_t launch_stream_epi(GemmParams& p, int batches, size_t table_bytes, hipStream_t s)
{
    auto kern = gemm_stream_kernel<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, kEpi, kConv>;
    const size_t shmem = (size_t)kStages * (BM + BN) * BK + 3 * BN * sizeof(float) + table_bytes;
    static std::once_flag once;  // one attribute call per instantiation
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(gemm_stream_kernel)");
    });
    if (once_rc) return once_rc;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    p.batched = batches > 1;
    p.div_group = fast_div(8 * p.tiles_n);
    if (kConv) p.div_wo = fast_div(p.cWo), p.div_ho = fast_div(p.cHo);
    queue_kernel(kern, dim3(p.tiles_m * p.tiles_n, batches), dim3(64 * WAVES_M * WAVES_N * KSPLIT), shmem, s, p);
    return NM_OK;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int KSPLIT, int BK, int kStages>
static int32_t launch_stream(GemmParams& p, int epi, int batches, size_t table_bytes, hipStream_t s)
{
    switch (epi) {
    case EPI_Q: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_Q>(p, batches, table_bytes, s);
    case EPI_Q_TABLE: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_Q_TABLE>(p, batches, table_bytes, s);
    case EPI_F32_RESID: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_F32_RESID>(p, batches, table_bytes, s);
    case EPI_Q_TABLE_RESID: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_Q_TABLE_RESID>(p, batches, table_bytes, s);
    case EPI_ACC: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_ACC>(p, batches, table_bytes, s);
    default: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_GENERIC>(p, batches, table_bytes, s);
    }
}

// Convolutions use three epilogues (everything else falls to the generic one).
template <int BM, int BN, int WAVES_M, int WAVES_N, int KSPLIT, int BK, int kStages>
static int32_t launch_stream_conv(GemmParams& p, int epi, size_t table_bytes, hipStream_t s)
{
    switch (epi) {
    case EPI_Q: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_Q, true>(p, 1, table_bytes, s);
    case EPI_Q_TABLE: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_Q_TABLE, true>(p, 1, table_bytes, s);
    case EPI_Q_TABLE_RESID: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_Q_TABLE_RESID, true>(p, 1, table_bytes, s);
    default: return launch_stream_epi<BM, BN, WAVES_M, WAVES_N, KSPLIT, BK, kStages, EPI_GENERIC, true>(p, 1, table_bytes, s);
    }
}

// The LayerNorm-folding kernel: workgroups of 64 rows x all N columns (eight wavefronts, each all 64
// rows of N / 8 columns), 64-byte k-slices so that two ring stages of 64 + N rows fit LDS.
bool gemm_folds_layernorm(const GemmArgs& g)
{
    if (force_generic() || g.conv || g.w_is_kn || g.outer_count * g.inner_count != 1) return false;
    if (g.N != 768 && g.N != 1024) return false;
    if (g.K % 64 != 0 || g.K / 64 < 3 || g.alpha_vec || g.has_table || !g.resid || !g.ln_gamma || !g.ln_beta) return false;
    if (!(g.ln_out_q || g.ln_out_f32)) return false;
    const bool al = aligned(g.A, 16) && g.lda % 16 == 0 && aligned(g.W, 16) && g.ldw % 16 == 0 && aligned(g.resid, 16) &&
                    g.ldo == g.N && aligned(g.ln_gamma, 16) && aligned(g.ln_beta, 16) &&
                    (!g.ln_out_q || aligned(g.ln_out_q, 16)) && (!g.ln_out_f32 || aligned(g.ln_out_f32, 16)) &&
                    (!g.bias || aligned(g.bias, 4));
    return al && (int64_t)g.M * g.lda < (1LL << 32) && (int64_t)g.N * g.ldw < (1LL << 32);
}

// 16-byte loads need every row start and every batch offset on a 16-byte boundary
static bool rows_aligned(const void* base, long ld, long outer, long inner) { return aligned(base, 16) && ld % 16 == 0 && outer % 16 == 0 && inner % 16 == 0; }

// table: g's, or its expanded form
static void fill_params(const GemmArgs& g, const DevTable& table, GemmParams& p)
{
    p.M = g.M; p.N = g.N; p.K = g.K;
    p.A = g.A; p.lda = g.lda; p.W = g.W; p.ldw = g.ldw;
    p.inner_count = g.inner_count;
    p.a_outer = g.a_outer; p.a_inner = g.a_inner; p.w_outer = g.w_outer; p.w_inner = g.w_inner;
    p.o_outer = g.o_outer; p.o_inner = g.o_inner;
    p.bias = g.bias; p.alpha_vec = g.alpha_vec; p.alpha = g.alpha;
    p.resid = g.resid; p.resid_scale = g.resid_scale;
    p.has_table = g.has_table; p.table = table;
    p.out_inv_scale = g.out_inv_scale; p.out_inv_scale_vec = g.out_inv_scale_vec;
    p.split_cols = g.split_cols;
    p.relu = g.has_table && g.split_cols == 0 && !g.out_inv_scale_vec && relu_codes(table, g.out_inv_scale, g.resid ? g.resid_scale : 0.0f);
    for (int i = 0; i < 3; ++i) p.inv3[i] = g.inv3[i];
    p.ldo = g.ldo;
    p.cH = g.cH; p.cW = g.cW; p.cCin = g.cCin; p.cKw = g.cKw; p.cStride = g.cStride; p.cPad = g.cPad;
    p.cHo = g.cHo; p.cWo = g.cWo;
    p.out_q = g.out_q; p.out_f32 = g.out_f32; p.out_acc = g.out_acc; p.dbg_seg = g.dbg_seg;

    p.vec_out = g.ldo % 4 == 0 && g.o_outer % 4 == 0 && g.o_inner % 4 == 0 &&
                (!g.out_q || aligned(g.out_q, 4)) && (!g.out_f32 || aligned(g.out_f32, 16)) &&
                (!g.out_acc || aligned(g.out_acc, 16)) && (!g.dbg_seg || aligned(g.dbg_seg, 8)) &&
                (!g.resid || aligned(g.resid, 4));
    p.r16 = g.resid && aligned(g.resid, 16) && g.ldo % 16 == 0 && g.o_outer % 16 == 0 && g.o_inner % 16 == 0 && g.N % 16 == 0;
    p.q16 = g.out_q && aligned(g.out_q, 16) && g.ldo % 16 == 0 && g.o_outer % 16 == 0 && g.o_inner % 16 == 0;
    p.vec_cols = (!g.bias || aligned(g.bias, 16)) && (!g.alpha_vec || aligned(g.alpha_vec, 16)) &&
                 (!g.out_inv_scale_vec || aligned(g.out_inv_scale_vec, 16));
}

// Bytes of A that a gathered or plain product reads.
static int64_t operand_extent(const GemmArgs& g)
{
    return g.conv ? (int64_t)(g.M / (g.cHo * g.cWo)) * g.cH * g.cW * g.cCin : (int64_t)(g.M - 1) * g.lda + g.K;
}

int32_t launch_conv_pair(const GemmArgs& a, const GemmArgs& b, hipStream_t stream, bool* done)
{
    *done = false;
    const GemmArgs* const g[2] = {&a, &b};
    GemmParams p[2] = {};
    for (int i = 0; i < 2; ++i) {
        const GemmArgs& c = *g[i];
        fill_params(c, c.table, p[i]);
        if (gemm_switched() || !rows_aligned(c.A, 0, 0, 0) || !rows_aligned(c.W, c.ldw, 0, 0) || c.cCin % 64 != 0 ||
            c.K % (c.cCin * c.cKw) != 0 || operand_extent(c) >= (1LL << 31) || (int64_t)(c.N - 1) * c.ldw + c.K >= (1LL << 31) ||
            (int64_t)c.M * c.N >= direct_below(false, c.N, c.K) || !direct_pair_takes(p[i]))
            return NM_OK;
    }
    const int cfg = choose_direct_pair({a.M, b.M}, {a.N, b.N}, {a.K, b.K});
    if (cfg < 0) return NM_OK;
    *done = true;
    return launch_direct_pair(p, cfg, stream);
}

int32_t launch_gemm(const GemmArgs& g, hipStream_t stream)
{
    if (g.M == 0) return NM_OK;
    if (g.ln) {
        if (!gemm_folds_layernorm(g)) return fail(NM_ERR_UNSUPPORTED, "gemm: this shape does not fold the LayerNorm");
        GemmLnParams q{};
        q.M = g.M; q.N = g.N; q.K = g.K; q.A = g.A; q.lda = g.lda; q.W = g.W; q.ldw = g.ldw; q.inner_count = 1;
        q.bias = g.bias; q.alpha = g.alpha; q.resid = g.resid; q.resid_scale = g.resid_scale; q.ldo = g.ldo;
        q.ln_gamma = g.ln_gamma; q.ln_beta = g.ln_beta; q.ln_eps = g.ln_eps; q.ln_inv_scale = g.ln_inv_scale;
        q.ln_table = g.ln_table; q.ln_out_q = g.ln_out_q; q.ln_out_f32 = g.ln_out_f32;
        int32_t rc = g.N == 768 ? launch_tile_epi<64, 768, 1, 8, 2, EPI_F32_RESID_LN, 64>(q, 0, stream)
                                : launch_tile_epi<64, 1024, 1, 8, 2, EPI_F32_RESID_LN, 64>(q, 0, stream);
        if (rc) return rc;
        return check_hip(hipGetLastError(), "gemm + LayerNorm launch");
    }
    // A merged table kept in two levels is looked up in its expanded form where the results are int8 codes alone: one look-up
    // instead of two, and the fixed epilogues (4096 x 3072 x 768: 16.9 us in two levels in the tile kernel, 15.6 expanded).
    const bool only_q = g.out_q && !g.out_f32 && !g.out_acc;
    DevTable table = g.table;
    if (only_q && !g.resid && !g.out_inv_scale_vec && !g.dbg_seg && !table.clamp_input) table.cellmap = nullptr;
    GemmParams p{};
    fill_params(g, table, p);
    const bool a_al = rows_aligned(g.A, g.lda, g.a_outer, g.a_inner), w_al = rows_aligned(g.W, g.ldw, g.w_outer, g.w_inner);
    const bool al = a_al && w_al && g.K % 16 == 0 && (!g.w_is_kn || g.N % 16 == 0);

    // LDS bytes of the table: {k, b} per segment, or for the two-level form of a merged table one
    // {k, b} per merged segment plus a byte per primary cell
    const size_t table_bytes = !g.has_table ? 0
                             : table.cellmap ? two_level_bytes(table) : sizeof(float2) * (size_t)table.nseg;
    const int batches = g.outer_count * g.inner_count;
    if (batches > 65535) return fail(NM_ERR_UNSUPPORTED, "gemm: more than 65535 batched problems");
    int32_t rc = NM_OK;
    int epi = EPI_GENERIC;
    if (!g.out_inv_scale_vec && !g.dbg_seg && !(g.has_table && table.cellmap)) {
        // EPI_Q_TABLE is compiled without the input clamp; a table with that flag takes the generic epilogue
        if (only_q && !g.resid) epi = !g.has_table ? EPI_Q : g.table.clamp_input ? EPI_GENERIC : EPI_Q_TABLE;
        else if (g.out_f32 && !g.out_q && !g.out_acc && g.resid && !g.has_table && p.vec_out) epi = EPI_F32_RESID;
        else if (only_q && g.resid && g.has_table && !g.table.clamp_input && p.vec_out) epi = EPI_Q_TABLE_RESID;
        else if (g.out_acc && !g.out_q && !g.out_f32) epi = EPI_ACC;
    }
    // Tile configuration, from same-process timings of every configuration on the shapes of the
    // workloads.  NARROW (256x64) for outputs of at most 64 columns.  Wide outputs (N >= 1536): BIG
    // (256x192, two 128-byte stages, one workgroup per CU) when its tiles fill whole rounds of the
    // 256 CUs to at least 90 %, WIDE (256x128 with 128x64 wavefront tiles, 48 KB ring) when those come six or more to a CU.
    // Otherwise by the number of 128x128 tiles: three or more per CU -> MID2 (two 64-byte stages,
    // 32 KB: four workgroups share a CU and one's epilogue overlaps another's loads); 1.25 to 3 per
    // CU -> MID3 (three stages), or SMALL (64x128, two wavefronts per sub-tile on alternate
    // k-steps, 128-byte slices) for long contractions; fewer -> SPLIT (128x128, same scheme), or
    // SMALL when even those would leave more than a third of the CUs idle.
    const bool k128 = g.K % 128 == 0 && (!g.conv || g.cCin % 128 == 0);  // 128-byte k-slices fetch ~1.5x faster
    const long big_tiles = (long)((g.M + 255) / 256) * ((g.N + 191) / 192) * batches;
    const long mid_tiles = (long)((g.M + 127) / 128) * ((g.N + 127) / 128) * batches;
    const long wide_tiles = (long)((g.M + 255) / 256) * ((g.N + 127) / 128) * batches;
    const bool split_ok = k128 && table_bytes <= 32768;
    // share of CU slots the BIG tiles use over their rounds (one workgroup per CU; a single partly
    // filled round counts as full: there is nothing better to do with the idle CUs)
    const double big_fill = big_tiles <= 256 ? 1.0 : (double)big_tiles / (double)((big_tiles + 255) / 256 * 256);
    enum { CFG_BIG, CFG_WIDE, CFG_SPLIT, CFG_SMALL, CFG_MID3, CFG_MID2, CFG_NARROW } cfg;
    if (g.N <= 64) cfg = CFG_NARROW;
    else if (g.N >= 1536 && g.K > 256 && wide_tiles >= 1536) cfg = CFG_WIDE;
    else if (!g.conv && k128 && g.N >= 1536 && big_tiles >= 192 && big_fill >= 0.9) cfg = CFG_BIG;
    else if (mid_tiles >= 768) cfg = CFG_MID2;
    else if (mid_tiles >= 320) cfg = (split_ok && g.K >= 2048) ? CFG_SMALL : CFG_MID3;
    else if (split_ok) cfg = (mid_tiles < 160 && g.M > 64) ? CFG_SMALL : CFG_SPLIT;
    else cfg = CFG_MID3;
    // a gathered A operand is read 16 bytes at a time by every kernel that takes one (the caller has
    // checked Cin % 64 == 0, 16-byte aligned image and weights)
    if (g.conv && (!w_al || !aligned(g.A, 16) || g.cCin % 64 != 0 || g.K % (g.cCin * g.cKw) != 0))
        return fail(NM_ERR_UNSUPPORTED, "conv gemm: operands not aligned for the gathered loader");
    const bool rows_ok = al && !g.conv && !g.w_is_kn && !force_generic(), stream_ok = rows_ok && g.K % 64 == 0;
    // The tile kernel: plain matrix products with the encoder layer's epilogues
    const bool tile_epi = (epi == EPI_Q || epi == EPI_Q_TABLE) ? p.q16 != 0
                        : epi == EPI_F32_RESID ? (p.r16 != 0 && aligned(g.out_f32, 16) && g.ldo % 4 == 0) : false;
    const bool tile_ok = rows_ok && tile_epi && batches == 1 && g.K > 256 && !g.alpha_vec &&
                         g.N % 16 == 0 && g.split_cols % 4 == 0 && (int64_t)g.M * g.lda < (1LL << 32) &&
                         (int64_t)g.N * g.ldw < (1LL << 32) && table_bytes <= 40 * 1024;
    // The small-tile kernel takes any shape and alignment whose operands are addressable with 31 bits.  It is
    // chosen when the output is too small for the larger tiles to occupy the chip, and for unaligned operands
    // that the register-staged tiles do not take.
    // Against the tile kernel the line is 1.05 million outputs, 256 tiles of 64x64: up to there one round of its tiles holds
    // the output, beyond it a second one begins.  Tiles over this kernel, us, products of layers of width 384 to 1024:
    //    512 x 2048 x  512  4.64 | 4.17     1200 x 768 x 3072  11.1 | 10.2    1024 x 1024 x 4096  13.0 | 10.8
    //    700 x 1536 x  512  3.98 | 4.40     1400 x 768 x 3072  11.2 | 14.8    1200 x 1024 x 4096  13.7 | 16.5
    //   1024 x 1152 x  384  3.77 | 4.25     2500 x 384 x  384  4.69 | 4.47    3300 x  384 x  384  4.90 | 5.19
    // The largest losses on this side are 300 x 3072 x 1024 (4.9 | 5.3) and 1500 x 640 x 640 (5.1 | 5.2).  The streaming
    // kernel's tiles need about a million outputs, more when the contraction is short and a large tile is mostly
    // prologue and epilogue.
    const int64_t a_extent = operand_extent(g);
    const bool direct_ok = !force_generic() && !g.w_is_kn && a_extent < (1LL << 31) && (int64_t)(g.N - 1) * g.ldw + g.K < (1LL << 31);
    const int direct_align = !(aligned(g.A, 4) && g.lda % 4 == 0 && g.a_outer % 4 == 0 && g.a_inner % 4 == 0 && aligned(g.W, 4) &&
                               g.ldw % 4 == 0 && g.w_outer % 4 == 0 && g.w_inner % 4 == 0) ? 1 : al ? 16 : 4;
    const int64_t outputs = (int64_t)g.M * g.N * batches;
    // Register-staged tiles, for operands that cannot go to LDS directly in whole slices (staged_faster)
    const bool unaligned_ok = direct_ok && !g.conv && batches == 1 && g.N >= 4;
    const bool staged = unaligned_ok && !tile_ok && (direct_align < 16 || g.K % 64 != 0);
    // The tile kernel's epilogues for convolutions (int8, per-column scales, no table or one of two segments, an int8
    // residual; the rows gathered or not).  us, streaming kernel -> these: 200704 x 64 x 576 (3x3) 21.7 -> 17.0, 200704 x 64 x 256 17.9 ->
    // 13.3, 50176 x 512 x 128 with residual 18.4 -> 15.4, 12544 x 1024 x 256 with residual 12.8 -> 11.8, 200704 x 256 x 64
    // 22.6 -> 19.6, with residual 26.3 -> 25.6; with 128-byte slices in launch_tile_relu.
    const bool relu_epi = (epi == EPI_Q ? g.conv || g.alpha_vec : (epi == EPI_Q_TABLE || epi == EPI_Q_TABLE_RESID) && g.table.two_seg) &&
                          p.q16 && g.N % 16 == 0 && batches == 1 && g.split_cols == 0 && (!g.resid || p.r16) && !force_generic();
    const int kunit = g.conv ? g.cCin : g.K;
    const bool relu_ok = relu_epi && relu_operands({g.conv != 0, g.w_is_kn != 0, w_al, al, g.resid != nullptr, kunit, g.conv ? g.K / g.cCin : 0,
                                                    g.conv ? a_extent : (int64_t)g.M * g.lda, (int64_t)g.N * g.ldw});
    // the debug switch's configuration, if this product meets its requirements
    ForcedCfg forced = forced_cfg();
    const bool holds = forced.kind == FORCED_STREAM ? g.N > 64 && (g.conv || stream_ok) && stream_takes(forced.number, g.conv != 0, k128, split_ok)
                     : forced.kind == FORCED_DIRECT ? direct_ok && direct_takes(forced.number, g.K, table_bytes, g.conv != 0)
                     : forced.kind == FORCED_UNALIGNED ? unaligned_ok
                     : forced.kind == FORCED_RELU ? relu_ok && relu_takes(forced.number, kunit)
                     : forced.kind == FORCED_TILE ? tile_ok && tile_takes(forced.number, g.K, epi == EPI_F32_RESID) : false;
    if (!holds) forced = ForcedCfg();
    const bool free_choice = forced.kind == FORCED_NONE;
    if (forced.kind == FORCED_UNALIGNED || (free_choice && staged && staged_faster(direct_align, g.M, g.N, g.K, g.out_q != nullptr, g.out_f32 || g.out_acc, g.has_table != 0, g.resid != nullptr))) {
        rc = launch_unaligned(p, direct_align, table_bytes, forced.number, stream);
        if (rc) return rc;
        return check_hip(hipGetLastError(), "gemm launch");
    }
    if (forced.kind == FORCED_DIRECT || (free_choice && direct_ok && (staged || direct_align < 16 || outputs < direct_below(tile_ok, g.N, g.K)))) {
        rc = launch_direct(p, direct_align, g.conv != 0, batches, table_bytes, forced.number, stream);
        if (rc) return rc;
        return check_hip(hipGetLastError(), "gemm launch");
    }
    if (forced.kind == FORCED_RELU || (free_choice && relu_ok)) {
        p.taps_w = g.cKw;
        if (g.conv) p.div_wo = fast_div(g.cWo), p.div_ho = fast_div(g.cHo);
        switch (free_choice ? choose_relu(g.M, g.N, g.K, kunit) : forced.number) {
        case 2: rc = launch_tile_relu<256, 128, 4, 2, 3>(p, g.conv != 0, stream); break;
        case 5: rc = launch_tile_relu<128, 128, 2, 2, 3>(p, g.conv != 0, stream); break;
        case 6: rc = launch_tile_relu<128, 128, 2, 2, 2>(p, g.conv != 0, stream); break;
        case 7: rc = launch_tile_relu<64, 128, 2, 2, 3>(p, g.conv != 0, stream); break;
        case 8: rc = launch_tile_relu<64, 128, 2, 2, 2>(p, g.conv != 0, stream); break;
        case 11: rc = launch_tile_relu<128, 128, 2, 2, 3, 128, 2>(p, g.conv != 0, stream); break;
        case 9: rc = launch_tile_relu<128, 128, 2, 2, 3, 64>(p, g.conv != 0, stream); break;
        default: rc = launch_tile_relu<128, 64, 4, 1, 3, 64>(p, g.conv != 0, stream); break;
        }
        if (rc) return rc;
        return check_hip(hipGetLastError(), "gemm launch");
    }
    if (forced.kind == FORCED_STREAM) {
        static constexpr decltype(cfg) kStream[] = {CFG_BIG, CFG_WIDE, CFG_SPLIT, CFG_SMALL, CFG_MID3, CFG_MID2, CFG_BIG};
        cfg = kStream[forced.number];
    }
    if (g.conv) {
        // gathered A operand: one problem, no batching
        if (cfg == CFG_NARROW) rc = launch_stream_conv<256, 64, 4, 1, 1, 64, 2>(p, epi, table_bytes, stream);
        else if (cfg == CFG_WIDE) rc = launch_stream_conv<256, 128, 2, 2, 1, 64, 2>(p, epi, table_bytes, stream);
        else if (cfg == CFG_MID2) rc = launch_stream_conv<128, 128, 2, 2, 1, 64, 2>(p, epi, table_bytes, stream);
        else if (cfg == CFG_SPLIT) rc = launch_stream_conv<128, 128, 2, 2, 2, 128, 3>(p, epi, table_bytes, stream);
        else if (cfg == CFG_SMALL) rc = launch_stream_conv<64, 128, 1, 2, 2, 128, 3>(p, epi, table_bytes, stream);
        else rc = launch_stream_conv<128, 128, 2, 2, 1, 64, 3>(p, epi, table_bytes, stream);
        if (rc) return rc;
        return check_hip(hipGetLastError(), "conv gemm launch");
    }
    int tile_cfg = -1;
    if (tile_ok) {
        if (free_choice) tile_cfg = choose_tile(g.M, g.N, g.K, epi == EPI_F32_RESID, g.has_table != 0);
        else if (forced.kind == FORCED_TILE) tile_cfg = forced.number;
        else if (forced.number == STREAM_BIG) tile_cfg = 1;
    }
    if (tile_cfg >= 0 && epi == EPI_Q_TABLE && !table.slots) {
        rc = launch_tile_long(tile_cfg, p, table_bytes, stream);
    } else if (tile_cfg >= 0) {
        // (no bytes for the table: slots are part of the kernel's own LDS)
        rc = g.K % 128 ? launch_tile_end(tile_cfg, p, epi, 0, stream) : launch_tile_config<false>(tile_cfg, p, epi, 0, stream);
    } else if (stream_ok && cfg == CFG_WIDE) {
        rc = launch_stream<256, 128, 2, 2, 1, 64, 2>(p, epi, batches, table_bytes, stream);
    } else if (stream_ok && cfg == CFG_BIG) {
        rc = launch_stream<256, 192, 4, 2, 1, 128, 2>(p, epi, batches, table_bytes, stream);
    } else if (stream_ok && cfg == CFG_MID2) {
        rc = launch_stream<128, 128, 2, 2, 1, 64, 2>(p, epi, batches, table_bytes, stream);
    } else if (stream_ok && cfg == CFG_SMALL) {
        rc = launch_stream<64, 128, 1, 2, 2, 128, 3>(p, epi, batches, table_bytes, stream);
    } else if (stream_ok && cfg == CFG_SPLIT) {
        rc = launch_stream<128, 128, 2, 2, 2, 128, 3>(p, epi, batches, table_bytes, stream);
    } else if (stream_ok && cfg == CFG_MID3) {
        rc = launch_stream<128, 128, 2, 2, 1, 64, 3>(p, epi, batches, table_bytes, stream);
    } else if (stream_ok && g.N > 32 && g.M >= 1024) {
        // narrow outputs with many rows (the 64-channel convolutions of a residual CNN)
        rc = launch_stream<256, 64, 4, 1, 1, 64, 2>(p, epi, batches, table_bytes, stream);
    } else if (g.N <= 64) {
        p.tiles_m = (g.M + 127) / 128; p.tiles_n = (g.N + 63) / 64;
        launch_cfg<128, 64, 32, 64>(p, al, g.w_is_kn, dim3(p.tiles_m * p.tiles_n, batches), table_bytes, stream);
    } else {
        p.tiles_m = (g.M + 127) / 128; p.tiles_n = (g.N + 127) / 128;
        launch_cfg<128, 128, 64, 64>(p, al, g.w_is_kn, dim3(p.tiles_m * p.tiles_n, batches), table_bytes, stream);
    }
    if (rc) return rc;
    return check_hip(hipGetLastError(), "gemm launch");
}

}  // namespace nm

using namespace nm;

extern "C" {

int32_t nm_gemm_pwl(const nm_gemm_desc* d, void* stream)
{
    if (!d) return fail(NM_ERR_INVALID_ARG, "nm_gemm_pwl: desc is NULL");
    if (d->M < 1 || d->N < 1 || d->K < 1) return fail(NM_ERR_INVALID_ARG, "nm_gemm_pwl: M, N, K must be >= 1");
    if (!d->A || !d->W) return fail(NM_ERR_INVALID_ARG, "nm_gemm_pwl: A or W is NULL");
    if (!d->out_q && !d->out_f32 && !d->out_acc) return fail(NM_ERR_INVALID_ARG, "nm_gemm_pwl: no output");
    if (d->K > 65536) return fail(NM_ERR_UNSUPPORTED, "nm_gemm_pwl: K %d > 65536", d->K);
    if ((int64_t)d->M * d->N >= (1LL << 31)) return fail(NM_ERR_UNSUPPORTED, "nm_gemm_pwl: M*N >= 2^31");
    if (d->split_cols < 0 || (d->split_cols > 0 && d->out_inv_scale_vec))
        return fail(NM_ERR_INVALID_ARG, "nm_gemm_pwl: split_cols must be >= 0 and excludes out_inv_scale_vec");
    GemmArgs g;
    g.M = d->M; g.N = d->N; g.K = d->K;
    g.A = d->A; g.lda = d->K; g.W = d->W; g.ldw = d->K;
    g.bias = d->bias; g.alpha_vec = d->alpha_vec; g.alpha = d->alpha;
    g.resid = d->resid; g.resid_scale = d->resid_scale;
    if (d->table_idx >= 0) {
        int32_t rc = get_dev_table(d->tables, d->table_idx, &g.table, "nm_gemm_pwl", true);
        if (rc) return rc;
        g.has_table = 1;
    }
    g.out_inv_scale = d->out_inv_scale; g.out_inv_scale_vec = d->out_inv_scale_vec;
    g.split_cols = d->split_cols;
    for (int i = 0; i < 3; ++i) g.inv3[i] = d->out_inv_scale3[i];
    g.ldo = d->N;
    g.out_q = d->out_q; g.out_f32 = d->out_f32; g.out_acc = d->out_acc; g.dbg_seg = d->dbg_seg;
    return launch_gemm(g, (hipStream_t)stream);
}

static int32_t check_attn(const char* what, const void* a, const void* b, const void* c, int32_t B,
                          int32_t S, int32_t H, int32_t heads)
{
    if (!a || !b || !c) return fail(NM_ERR_INVALID_ARG, "%s: NULL pointer", what);
    if (B < 1 || S < 1 || H < 1 || heads < 1) return fail(NM_ERR_INVALID_ARG, "%s: dimensions must be >= 1", what);
    if (H % heads != 0) return fail(NM_ERR_INVALID_ARG, "%s: H %d not divisible by heads %d", what, H, heads);
    if (S > 4096) return fail(NM_ERR_UNSUPPORTED, "%s: S %d > 4096", what, S);
    if ((int64_t)B * heads > 65535) return fail(NM_ERR_UNSUPPORTED, "%s: B * heads > 65535", what);
    if ((int64_t)B * S * 3 * H >= (1LL << 31)) return fail(NM_ERR_UNSUPPORTED, "%s: B*S*3H >= 2^31", what);
    return NM_OK;
}

int32_t nm_attn_scores(const int8_t* qkv, int32_t B, int32_t S, int32_t H, int32_t heads,
                       int32_t* scores, void* stream)
{
    int32_t rc = check_attn("nm_attn_scores", qkv, qkv, scores, B, S, H, heads);
    if (rc) return rc;
    const int d = H / heads;
    GemmArgs g;
    g.M = S; g.N = S; g.K = d;
    g.A = qkv; g.lda = 3L * H; g.W = qkv + H; g.ldw = 3L * H;
    g.outer_count = B; g.inner_count = heads;
    g.a_outer = (long)S * 3 * H; g.a_inner = d;
    g.w_outer = (long)S * 3 * H; g.w_inner = d;
    g.o_outer = (long)heads * S * S; g.o_inner = (long)S * S;
    g.ldo = S;
    g.out_acc = scores;
    return launch_gemm(g, (hipStream_t)stream);
}

int32_t nm_attn_context(const int8_t* p, const int8_t* qkv, int32_t B, int32_t S, int32_t H,
                        int32_t heads, float alpha, float out_inv_scale, int8_t* ctx, void* stream)
{
    int32_t rc = check_attn("nm_attn_context", p, qkv, ctx, B, S, H, heads);
    if (rc) return rc;
    const int d = H / heads;
    GemmArgs g;
    g.M = S; g.N = d; g.K = S;
    g.A = p; g.lda = S;
    g.W = qkv + 2L * H; g.ldw = 3L * H; g.w_is_kn = 1;  // V is [S, d] per head: k = j runs over rows
    g.outer_count = B; g.inner_count = heads;
    g.a_outer = (long)heads * S * S; g.a_inner = (long)S * S;
    g.w_outer = (long)S * 3 * H; g.w_inner = d;
    g.o_outer = (long)S * H; g.o_inner = d;
    g.ldo = H;
    g.alpha = alpha; g.out_inv_scale = out_inv_scale;
    g.out_q = ctx;
    return launch_gemm(g, (hipStream_t)stream);
}

}  // extern "C"
