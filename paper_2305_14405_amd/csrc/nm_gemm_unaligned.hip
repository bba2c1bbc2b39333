// The register-staged tile int8 GEMM kernel: matrix products whose operand rows are not 16-byte aligned (a
// contraction of 1000 or 1001 bytes), or aligned ones of a K that is no multiple of 64, whose output is large enough for
// tiles (staged_faster; paper Section 3.1; the epilogue is that of every other GEMM kernel here).
//
// Such rows cannot go global -> LDS directly.  They pass through registers: buffer loads of 16 bytes (words past the end of the
// buffer read as zero), shifted to the row's own start when they are written to LDS, two slices of 128 bytes in LDS and
// D more on their way.  A slice costs a workgroup 0.62 us (128x128 tiles, 4096 x 1000 x 1024 .. 4096): LDS carries each
// operand byte once in and three times out, 1024 of the 1300 clocks.  The partly filled slice comes first, so that
// the loop has no special case.
// The epilogue was the larger half before its options became loops of their own and its stores aligned: 4096 x 1000 x
// 128 through a table 13.2 -> 6.6 us, 4096 x 1001 x 128 20.9 -> 7.3, with fp32 results 15.0 -> 7.7.
// Against the small-tile kernel, which took these shapes (gemm_direct_kernel, tiles of at most 32x64), us: 4096x1001x1000
// through a table 29.1 -> 12.6, 2766x491x1334 19.4 -> 15.1, 10932x1375x163 58 -> 23, 13810x1350x2686 251 -> 111,
// 16384x4000x4095 1135 -> 440; 2048x768x1008 (aligned) 18.9 -> 8.9.
#include "nm_gemm_common.h"

namespace nm {

constexpr int unaligned_front_bytes(int bm, int bn, int nw, int wn)
{
    const int slices = 2 * (bm + bn) * 128, patches = nw * 32 * (wn + 4) * 4;
    return slices > patches ? slices : patches;
}

// kAl: 4 or 1, bytes every operand row is aligned to.  D: slices on their way to registers.
template <int BM, int BN, int WAVES_M, int WAVES_N, int D, int kAl>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 2) void gemm_unaligned_kernel(GemmParams p)
{
    constexpr int NW = WAVES_M * WAVES_N, NT = 64 * NW;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 32, TN = WN / 32;
    constexpr int SLICE = (BM + BN) * 128;           // 128 bytes of k of every row
    constexpr int NI = (BM + BN) / 8 / NW;           // 1 KB pieces (8 rows) per wavefront; the first NA are A rows
    constexpr int NA = BM / 8 / NW;
    constexpr int PW = WN + 4;                       // row stride of a wavefront's patch of 32 rows, in words
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "pieces split evenly");
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];   // two slices, or the patches | scale, bias, inverse scale per column | table
    float* s_cols = reinterpret_cast<float*>(smem + unaligned_front_bytes(BM, BN, NW, WN));
    float2* s_kb = reinterpret_cast<float2*>(s_cols + 3 * BN);

    asm volatile("" : : "s"(p.A), "s"(p.W), "s"(p.bias), "s"(p.alpha_vec), "s"(p.resid), "s"(p.table.kb), "s"(p.M), "s"(p.N), "s"(p.K),
                 "s"(p.lda), "s"(p.ldw), "s"(p.ldo), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.has_table), "s"(p.group_m));

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = (wave / WAVES_N) * WM, wave_n = (wave % WAVES_N) * WN;

    // Workgroup i runs on XCD i % 8: an XCD gets a contiguous eighth of the tile sequence, which walks groups of
    // group_m tile rows column by column.
    const int ntiles = p.tiles_m * p.tiles_n, share = (ntiles + 7) >> 3;
    const int id = (blockIdx.x % 8) * share + blockIdx.x / 8;
    if (id >= ntiles) return;
    const int group = id / (p.group_m * p.tiles_n), first_m = group * p.group_m, gm = min(p.group_m, p.tiles_m - first_m);
    const int in_group = id - first_m * p.tiles_n;
    const int m0 = (first_m + in_group % gm) * BM, n0 = (in_group / gm) * BN;

    // source of the lane's 16 bytes in every piece: row l / 8 of the piece, chunk l % 8 (swizzled as lds_off_bk
    // reads it); rows past the edge are clamped to the last one (they only feed outputs that are never stored)
    const int lrow = lane >> 3, chunk0 = (lane & 7) ^ (lane >> 4) ^ ((wave & 1) << 2);
    static_assert(NW % 2 == 0, "a wavefront's pieces are all even or all odd");
    const unsigned sha = kAl == 1 ? (unsigned)((uintptr_t)p.A & 3) : 0u, shw = kAl == 1 ? (unsigned)((uintptr_t)p.W & 3) : 0u;
    const unsigned lda = (unsigned)p.lda, ldw = (unsigned)p.ldw;
    const unsigned a_last = (unsigned)(p.M - 1) * lda, w_last = (unsigned)(p.N - 1) * ldw;
    const rsrc_t ra = make_rsrc(p.A - sha, (a_last + (unsigned)p.K + sha + 3) & ~3u);
    const rsrc_t rw = make_rsrc(p.W - shw, (w_last + (unsigned)p.K + shw + 3) & ~3u);
    unsigned voff[NI];
#pragma unroll
    for (int b = 0; b < NI; ++b) {
        if (b < NA) voff[b] = (unsigned)min(m0 + 8 * (wave + b * NW) + lrow, p.M - 1) * lda + 16u * chunk0 + sha;
        else voff[b] = (unsigned)min(n0 + 8 * (wave + (b - NA) * NW) + lrow, p.N - 1) * ldw + 16u * chunk0 + shw;
    }
    // Slice 0 is the partly filled one (when there is one): bytes [K - K % 128, K) of every row, zeros behind them; the
    // others follow in order.
    const int nk = (p.K + 127) >> 7, part = p.K & 127;
    // (kAl == 1: five words around the 16 bytes, shifted when they go to LDS, so that nothing waits for them before that)
    v4i reg[D][NI];
    unsigned regx[D][NI];
    auto fetch = [&](int set, int kt) {
        const unsigned k0 = 128u * (unsigned)(part ? kt - 1 : kt);
#pragma unroll
        for (int b = 0; b < NI; ++b) {
            const unsigned at = (kAl == 4 ? voff[b] : voff[b] & ~3u) + k0;
            reg[set][b] = buf16(b < NA ? ra : rw, at);
            if (kAl == 1) regx[set][b] = buf4(b < NA ? ra : rw, at + 16);
        }
    };
    auto put = [&](int buf, int b, v4i v) { *reinterpret_cast<v4i*>(smem + buf * SLICE + (wave + b * NW) * 1024 + 16 * lane) = v; };
    auto stash = [&](int set, int buf) {
#pragma unroll
        for (int b = 0; b < NI; ++b) {
            v4i v = reg[set][b];
            if (kAl == 1) {
                const unsigned sh = voff[b] & 3u;
#pragma unroll
                for (int t = 0; t < 3; ++t) v[t] = (int)__builtin_amdgcn_alignbyte((unsigned)v[t + 1], (unsigned)v[t], sh);
                v[3] = (int)__builtin_amdgcn_alignbyte(regx[set][b], (unsigned)v[3], sh);
            }
            put(buf, b, v);
        }
    };
    v4i first[NI];
    if (part) {
        const unsigned k0 = (unsigned)(p.K - part);
        const int left = part - 16 * chunk0;
#pragma unroll
        for (int b = 0; b < NI; ++b) first[b] = load_tail<kAl>(b < NA ? ra : rw, voff[b] + k0, left);
    } else {
        fetch(0, 0);
    }
#pragma unroll
    for (int d = 1; d < D; ++d)
        if (d < nk) fetch(d, d);
    // per-column vectors and the table, behind the first slice's loads
    for (int t = tid; t < BN; t += NT) {
        const int n = min(n0 + t, p.N - 1);
        s_cols[t] = p.alpha_vec ? p.alpha_vec[n] : p.alpha;
        s_cols[BN + t] = p.bias ? p.bias[n] : 0.0f;
        s_cols[2 * BN + t] = p.out_inv_scale_vec ? p.out_inv_scale_vec[n]
                           : p.split_cols > 0 ? (n >= 2 * p.split_cols ? p.inv3[2] : n >= p.split_cols ? p.inv3[1] : p.inv3[0]) : p.out_inv_scale;
    }
    if (p.has_table) { if (p.table.cellmap) stage_table_two_level(s_kb, p.table); else stage_table(s_kb, p.table); }

    v16i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
    const int frag_row = lane & 31, frag_half = lane >> 5;
    int offA[4], offW[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        offA[ks] = lds_off_bk<128>(wave_m + frag_row, 2 * ks + frag_half);
        offW[ks] = BM * 128 + lds_off_bk<128>(wave_n + frag_row, 2 * ks + frag_half);
    }
    if (part) {
#pragma unroll
        for (int b = 0; b < NI; ++b) put(0, b, first[b]);
    } else {
        stash(0, 0);
    }
    if (D < nk) fetch(0, D);
    __syncthreads();
    // Slice kt is in LDS, the D behind it on their way to registers: the next one goes to the other half of LDS under
    // this slice's matrix instructions, and its registers are requested again behind that.
    auto slice = [&](int kt, int set) {   // set: of slice kt + 1
        const int8_t* st = smem + (kt & 1) * SLICE;
        v4i fa[2][TM], fw[2][TN];
        auto frags = [&](int ks) {
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[ks & 1][j] = *reinterpret_cast<const v4i*>(st + offW[ks] + j * 32 * 128);
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[ks & 1][i] = *reinterpret_cast<const v4i*>(st + offA[ks] + i * 32 * 128);
        };
        frags(0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) frags(ks + 1);
            if (ks == 2 && kt + 1 < nk) {
                stash(set, (kt + 1) & 1);
                if (kt + 1 + D < nk) fetch(set, kt + 1 + D);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[ks & 1][j], fa[ks & 1][i], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    };
    for (int kt = 0; kt < nk; kt += D) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (kt + d < nk) slice(kt + d, (d + 1) % D);
    }

    // Epilogue, 32 rows at a time: the accumulators pass through a patch of the wavefront's own, so that a lane
    // finishes four neighbouring columns of rows and a row leaves in consecutive lanes, whatever its alignment.
    constexpr int LPR = WN / 4, RPP = 64 / LPR, NP = 32 / RPP;   // lanes per row, rows per pass, passes
    static_assert(LPR == 16, "a row is a DPP row");
    int* const patch = reinterpret_cast<int*>(smem) + wave * 32 * PW;
    const int prow = lane / LPR, pl = lane % LPR, pcol = 4 * pl;
    const int nb = n0 + wave_n + pcol;
    const int cols = p.N - nb, ncl = min(nb, p.N - 4);    // (N >= 4: host)
    const v4f sc = *reinterpret_cast<const v4f*>(s_cols + wave_n + pcol), bi = *reinterpret_cast<const v4f*>(s_cols + BN + wave_n + pcol),
              iv = *reinterpret_cast<const v4f*>(s_cols + 2 * BN + wave_n + pcol);
    const float scale[4] = {sc[0], sc[1], sc[2], sc[3]}, bias[4] = {bi[0], bi[1], bi[2], bi[3]};
    const int shr = 8 * min(nb - ncl, 3);   // the last lane of a row reads the last four codes; whole groups: no shift
    // Rows whose alignment is that of their elements (!p.vec_out, or columns not in whole fours): a store whose address is
    // not a multiple of its size is split by the hardware (4096 x 1002 codes took 6 us longer than 4096 x 1000), so words
    // leave one element per lane, and codes as the aligned words of a row and single bytes at its ends.
    const bool whole = p.vec_out && (p.N & 3) == 0;
    const int L = min(p.N - (n0 + wave_n), WN);   // columns of this piece
    auto fence = [] {   // the wavefront reads what it wrote, or writes what it has read
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // the patch's words to rows m_first .. of out
    auto store_words = [&](int* out, int m_first) {
        int* const dst = out + (long)m_first * p.ldo + n0 + wave_n + lane;
        int v[32];
#pragma unroll
        for (int r = 0; r < 32; ++r) v[r] = patch[r * PW + lane];
#pragma unroll
        for (int r = 0; r < 32; ++r)
            if (m_first + r < p.M && lane < L) dst[(long)r * p.ldo] = v[r];
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int mb = m0 + wave_m + 32 * i + prow;
        if (mb - prow >= p.M || n0 + wave_n >= p.N) break;   // wave-uniform
        unsigned res[NP];
        if (p.resid) {
#pragma unroll
            for (int t = 0; t < NP; ++t) res[t] = *reinterpret_cast<const u32_a1*>(p.resid + (long)min(mb + t * RPP, p.M - 1) * p.ldo + ncl) >> shr;
        }
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<v4i*>(patch + frag_row * PW + 32 * j + 8 * g + 4 * frag_half) =
                    v4i{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        fence();
        v4i a[NP];
        float y[NP][4];
        int seg[NP][4];
#pragma unroll
        for (int t = 0; t < NP; ++t) a[t] = *reinterpret_cast<const v4i*>(patch + (prow + t * RPP) * PW + pcol);
        if (p.out_acc) {
            if (whole) {
#pragma unroll
                for (int t = 0; t < NP; ++t)
                    if (mb + t * RPP < p.M && cols > 0) *reinterpret_cast<v4i*>(p.out_acc + (long)(mb + t * RPP) * p.ldo + nb) = a[t];
            } else {
                store_words(p.out_acc, mb - prow);
            }
        }
        epi_values<NP>(p, s_kb, a, scale, bias, res, y, seg);
        if (p.dbg_seg && p.has_table) {
#pragma unroll
            for (int t = 0; t < NP; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (mb + t * RPP < p.M && nb + e < p.N) p.dbg_seg[(long)(mb + t * RPP) * p.ldo + nb + e] = (uint16_t)seg[t][e];
        }
        if (p.out_f32) {
            if (whole) {
#pragma unroll
                for (int t = 0; t < NP; ++t)
                    if (mb + t * RPP < p.M && cols > 0)
                        *reinterpret_cast<v4f*>(p.out_f32 + (long)(mb + t * RPP) * p.ldo + nb) = v4f{y[t][0], y[t][1], y[t][2], y[t][3]};
            } else {
                fence();
#pragma unroll
                for (int t = 0; t < NP; ++t)
                    *reinterpret_cast<v4f*>(patch + (prow + t * RPP) * PW + pcol) = v4f{y[t][0], y[t][1], y[t][2], y[t][3]};
                fence();
                store_words(reinterpret_cast<int*>(p.out_f32), mb - prow);
            }
        }
        if (p.out_q) {
            unsigned w[NP];
#pragma unroll
            for (int t = 0; t < NP; ++t)
                w[t] = pack4(requant(y[t][0], iv[0]), requant(y[t][1], iv[1]), requant(y[t][2], iv[2]), requant(y[t][3], iv[3]));
            if (whole) {
#pragma unroll
                for (int t = 0; t < NP; ++t)
                    if (mb + t * RPP < p.M && cols > 0) *reinterpret_cast<unsigned*>(p.out_q + (long)(mb + t * RPP) * p.ldo + nb) = w[t];
            } else {
                fence();
#pragma unroll
                for (int t = 0; t < NP; ++t) {
                    // the aligned word that ends inside the lane's columns: its front comes from the lane before
                    int8_t* const dst = p.out_q + (long)(mb + t * RPP) * p.ldo + nb;
                    const int sh = (int)((uintptr_t)dst & 3);
                    const unsigned prev = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w[t], 0x111, 0xf, 0xf, false);   // lane - 1
                    const unsigned word = sh ? __builtin_amdgcn_alignbyte(w[t], prev, 4 - sh) : w[t];
                    if (mb + t * RPP < p.M && (pcol > 0 || sh == 0) && 3 - sh < cols) *reinterpret_cast<unsigned*>(dst - sh) = word;
                    patch[(prow + t * RPP) * PW + pcol / 4] = (int)w[t];
                }
                fence();
                // both ends of the 32 rows, one per lane: the columns in front of the first aligned word and behind the last one
                const int r = lane >> 1, m = mb - prow + r;
                int8_t* const dst = p.out_q + (long)m * p.ldo + n0 + wave_n;
                const int sh = (int)((uintptr_t)dst & 3), head = min(sh ? 4 - sh : 0, L), tail = max(((L + sh) & ~3) - sh, head);
                const int from = lane & 1 ? tail : 0, to = lane & 1 ? L : head;
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    if (m < p.M && from + b < to) dst[from + b] = reinterpret_cast<const int8_t*>(patch + r * PW)[from + b];
            }
        }
        fence();
    }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int D, int kAl>
static int32_t launch_unaligned_t(GemmParams& p, size_t table_bytes, hipStream_t s)
{
    auto kern = gemm_unaligned_kernel<BM, BN, WAVES_M, WAVES_N, D, kAl>;
    const size_t shmem = unaligned_front_bytes(BM, BN, WAVES_M * WAVES_N, BN / WAVES_N) + 3 * BN * sizeof(float) + table_bytes;
    static std::once_flag once;  // one attribute call per instantiation
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(gemm_unaligned_kernel)");
    });
    if (once_rc) return once_rc;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    p.group_m = xcd_group_rows(p.tiles_m, p.tiles_n, BM, BN);
    queue_kernel(kern, dim3((p.tiles_m * p.tiles_n + 7) / 8 * 8), dim3(64 * WAVES_M * WAVES_N), shmem, s, p);
    return NM_OK;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int D>
static int32_t launch_unaligned_a(GemmParams& p, int align, size_t table_bytes, hipStream_t s)
{
    return align >= 4 ? launch_unaligned_t<BM, BN, WAVES_M, WAVES_N, D, 4>(p, table_bytes, s)
                      : launch_unaligned_t<BM, BN, WAVES_M, WAVES_N, D, 1>(p, table_bytes, s);
}

int32_t launch_unaligned(GemmParams& p, int align, size_t table_bytes, int forced, hipStream_t s)
{
    const int cfg = forced >= 0 ? forced : choose_unaligned(p.M, p.N, p.K, p.out_q != nullptr, p.out_f32 || p.out_acc, p.has_table != 0, p.resid != nullptr);
    switch (cfg) {
    case 0: return launch_unaligned_a<256, 128, 4, 2, 2>(p, align, table_bytes, s);
    case 1: return launch_unaligned_a<128, 128, 4, 2, 2>(p, align, table_bytes, s);
    case 2: return launch_unaligned_a<128, 64, 4, 1, 2>(p, align, table_bytes, s);
    default: return launch_unaligned_a<64, 64, 2, 1, 2>(p, align, table_bytes, s);
    }
}

}  // namespace nm
