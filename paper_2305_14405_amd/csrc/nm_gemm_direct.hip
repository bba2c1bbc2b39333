// The small-tile int8 GEMM kernel: matrix products whose output has too few large tiles to occupy
// the chip, and operands of any alignment (paper Section 3.1: fully connected layers and convolutions
// as matrix products; the epilogue is that of every other GEMM kernel here).
//
// What bounds such a product is latency, not a rate: with the LDS-ring kernels 128 x 768 x 3072 is 12
// workgroups that each wait 24 times for a k-slice, and their prologue and epilogue are as long as
// the loop.  Here a workgroup owns a small tile (16 x 32 .. 64 x 64 outputs) and its four or eight
// wavefronts divide K between them.  Each streams its own slices (128 bytes of every A and W row of the
// tile) through an LDS ring of its own, so the loop has no workgroup barrier and most of what a CU needs is
// in flight at once: rows of 128 bytes keep the loads at the full 64 bytes per clock and CU (loading
// fragments straight into registers, 16 rows of 64 bytes per instruction, reached 8).  The wavefronts'
// int32 partial tiles meet in LDS (exact in any order) and every thread finishes groups of four
// neighbouring outputs; the epilogue's vectors, residual and table are requested behind the first slices and
// not waited for until then, and all kernel arguments are fetched in one step (together 0.4 .. 1.5 us of
// a launch).  Measured, us before -> after, weights from HBM: 128x768x3072 13.9 -> 5.3, 128x3072x768 8.6 ->
// 5.0, 64x128x128 6.4 -> 2.9 (an empty launch is 1.6), 847x768x3072 15.0 -> 10.9, 3x3 convolution of
// 512 channels at 7x7 28.9 -> 6.7.
//
// Operands that are not 16-byte aligned come through registers and buffer descriptors: words past the end
// of the buffer read as zero, bytes past K are cleared.
#include "nm_gemm_common.h"

namespace nm {

// Arguments of the fixed epilogues: what they use, under the names GemmParams has for it.  (The host pays 0.9 us more for a
// launch with the 560 bytes of GemmParams than for one with 160.)
struct DirectTable {
    const float2* kb;
    float lo, inv_w;
    int nseg;
    float k0, b0, k1, b1, tau;
};
struct DirectParams {
    const int8_t* A;
    const int8_t* W;
    const float* bias;
    const float* alpha_vec;
    const int8_t* resid;
    int8_t* out_q;
    float* out_f32;
    int M, N, K, lda, ldw, ldo, tiles_m, tiles_n;
    FastDiv div_tiles_m;
    float alpha, resid_scale, out_inv_scale;
    int split_cols;
    float inv3[3];
    DirectTable table;
};
struct DirectConvParams : DirectParams {
    int cH, cW, cCin, cKw, cStride, cPad, cHo, cWo;
    FastDiv div_wo, div_ho, div_cin, div_kw;
};
template <bool kConv, int kEpi>
using DirectArgs = std::conditional_t<kEpi == EPI_GENERIC, GemmParams, std::conditional_t<kConv, DirectConvParams, DirectParams>>;

static void direct_args(GemmParams& q, const GemmParams& p) { q = p; }
static void direct_args(DirectParams& q, const GemmParams& p)
{
    q.A = p.A; q.W = p.W; q.bias = p.bias; q.alpha_vec = p.alpha_vec; q.resid = p.resid; q.out_q = p.out_q; q.out_f32 = p.out_f32;
    q.M = p.M; q.N = p.N; q.K = p.K; q.lda = (int)p.lda; q.ldw = (int)p.ldw; q.ldo = (int)p.ldo; q.tiles_m = p.tiles_m; q.tiles_n = p.tiles_n;
    q.div_tiles_m = p.div_tiles_m; q.alpha = p.alpha; q.resid_scale = p.resid_scale; q.out_inv_scale = p.out_inv_scale;
    q.split_cols = p.split_cols;
    for (int i = 0; i < 3; ++i) q.inv3[i] = p.inv3[i];
    const DevTable& t = p.table;
    q.table = {t.kb, t.lo, t.inv_w, t.nseg, t.k0, t.b0, t.k1, t.b1, t.tau};
}
static void direct_args(DirectConvParams& q, const GemmParams& p)
{
    direct_args(static_cast<DirectParams&>(q), p);
    q.cH = p.cH; q.cW = p.cW; q.cCin = p.cCin; q.cKw = p.cKw; q.cStride = p.cStride; q.cPad = p.cPad; q.cHo = p.cHo; q.cWo = p.cWo;
    q.div_wo = p.div_wo; q.div_ho = p.div_ho; q.div_cin = p.div_cin; q.div_kw = p.div_kw;
}

// KW wavefronts divide K in slices of 128 bytes; a wavefront has up to D slices in flight.
// kAl: 16: operands go global -> LDS directly; 4, 1: alignment of the rows in bytes, through registers.
// kEpi, kForm: EPI_GENERIC, or one of the fixed epilogues for a single problem whose columns come in whole fours and, unless
// gathered, with K a multiple of 16 (lean_epilogue; kEnd: not of 128, the last slice is partly filled).  Every kernel starts with an empty instruction cache and runs
// most of this code once: stamps at 128 x 3072 x 768 put 1300 to 2700 clocks on the 190 instructions in front of the first
// load and 1400 on the epilogue, of 7000 in all.  The fixed forms are a third of the code on the way, and divisions are by
// host-made reciprocals: 12 base layers over 1 x 128 tokens 360 -> 340 us, ResNet-50 on one image 245 -> 211.
// The arguments by value: by reference the compiler loads some of them once more, one by one, where they are chosen among (four images of 28 x 28, 128 to
// 128 channels 3x3 without a table 4.7 us by reference, 4.5; two convolutions in one launch 5.4 | 5.1, 6.9 | 6.4).  Aligned rows with the
// generic epilogue alone are better off with fewer held (16 x 2304 x 768 with both results 3.6 us by value, 3.5).
template <bool kConv, int kEpi, int kAl>
using DirectArgsIn = std::conditional_t<kEpi == EPI_GENERIC && !kConv && kAl == 16, const DirectArgs<kConv, kEpi>&, const DirectArgs<kConv, kEpi>>;
template <int BM, int BN, int KW, int D, int kAl, bool kConv, int kEpi, int kForm, bool kEnd>
__device__ __forceinline__ void direct_tile(DirectArgsIn<kConv, kEpi, kAl> p, const unsigned block)
{
    constexpr int TM = BM / 16, TN = BN / 16, NT = 64 * KW;
    constexpr int NA = BM / 8, NI = (BM + BN) / 8;   // 1 KB pieces (8 rows) of a slice; the first NA are A rows
    constexpr int SLICE = (BM + BN) * 128;
    constexpr int G4 = BN / 4, NGRP = BM * G4;       // groups of four outputs
    constexpr int GPT = (NGRP + NT - 1) / NT;        // ... per thread
    static_assert(NT % G4 == 0, "a thread's groups share their columns");
    static_assert(NGRP % NT == 0 || NGRP < NT, "groups split evenly");
    static_assert(BM * BN * 4 <= SLICE, "a wavefront's partial tile fits one slice");
    // 16-byte column slot of a partial tile's row, spread over the banks
    constexpr auto pslot = [](int row, int slot) { return slot ^ (BN == 64 ? row & 15 : BN == 32 ? (row >> 1) & 7 : (row >> 2) & 3); };
    static_assert(!kConv || kAl == 16, "gathered operand: aligned");
    constexpr bool kLean = kEpi != EPI_GENERIC;
    static_assert(!kLean || kAl == 16, "fixed epilogues: aligned");
    constexpr bool kResid = kEpi == EPI_F32_RESID || kEpi == EPI_Q_TABLE_RESID, kTable = kEpi == EPI_Q_TABLE || kEpi == EPI_Q_TABLE_RESID;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];   // [wavefronts with slices][slots][BM + BN rows of 128 bytes]

    // One wait for the kernel arguments the whole kernel uses (left alone, the compiler fetches them in
    // half a dozen dependent steps, each a memory round trip).
    asm volatile("" : : "s"(p.A), "s"(p.W), "s"(p.bias), "s"(p.alpha_vec), "s"(p.resid), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.lda), "s"(p.ldw),
                 "s"(p.ldo), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.alpha), "s"(p.out_q), "s"(p.out_f32), "s"(p.div_tiles_m.magic),
                 "s"(p.div_tiles_m.shift), "s"(p.out_inv_scale), "s"(p.resid_scale));
    if constexpr (!kLean)
        asm volatile("" : : "s"(p.has_table), "s"(p.vec_out), "s"(p.batched), "s"(p.table.kb), "s"(p.table.nseg), "s"(p.table.cellmap));
    if (kTable && kForm == FORM_ANY) asm volatile("" : : "s"(p.table.kb), "s"(p.table.nseg), "s"(p.table.lo), "s"(p.table.inv_w));
    if (kTable && kForm == FORM_TWO_SEGMENTS)
        asm volatile("" : : "s"(p.table.k0), "s"(p.table.b0), "s"(p.table.k1), "s"(p.table.b1), "s"(p.table.tau));
    if constexpr (kConv)
        asm volatile("" : : "s"(p.cH), "s"(p.cW), "s"(p.cCin), "s"(p.cKw), "s"(p.cStride), "s"(p.cPad), "s"(p.cWo), "s"(p.cHo), "s"(p.div_wo.magic),
                     "s"(p.div_wo.shift), "s"(p.div_ho.magic), "s"(p.div_ho.shift));

    // only as many rings and slots as this K needs (short contractions: several workgroups per CU)
    const int nk = (p.K + 127) >> 7;
    const int rings = kLean ? KW : min(KW, nk), slots = min(D, (nk + KW - 1) / KW);
    const int ring_bytes = slots * SLICE;
    float2* s_kb = reinterpret_cast<float2*>(smem + rings * ring_bytes);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fq = lane >> 4;

    // Workgroup i runs on XCD i % 8: an XCD gets a contiguous eighth of the tiles, rows of tiles
    // innermost, so that a panel of W is fetched into one L2.
    const int ntiles = p.tiles_m * p.tiles_n, share = (ntiles + 7) >> 3;
    const int id = (int)((block % 8) * share + block / 8);
    if (id >= ntiles) return;
    const int tile_n = (int)quotient((unsigned)id, p.div_tiles_m);
    const int m0 = (id - tile_n * p.tiles_m) * BM, n0 = tile_n * BN;
    const int8_t* A = p.A;
    const int8_t* W = p.W;
    long obase = 0;
    if constexpr (!kLean) {
        if (p.batched) {
            const int outer = blockIdx.y / p.inner_count, inner = blockIdx.y % p.inner_count;
            A += outer * p.a_outer + inner * p.a_inner;
            W += outer * p.w_outer + inner * p.w_inner;
            obase = outer * p.o_outer + inner * p.o_inner;
        }
    }

    // source of the lane's 16 bytes in every piece: row l / 8 of the piece, chunk l % 8 (swizzled);
    // rows past the edge are clamped to the last one (they only feed outputs that are never stored)
    const int lrow = lane >> 3;
    const int chunk0 = (lane & 7) ^ (lane >> 4);     // pieces 0, 2, ..; the others: chunk ^ 4
    unsigned voff[NI];
    int ch[kConv ? NA : 1], cw[kConv ? NA : 1];
    const unsigned sha = kAl == 1 ? (unsigned)((uintptr_t)A & 3) : 0u, shw = kAl == 1 ? (unsigned)((uintptr_t)W & 3) : 0u;
    const unsigned lda = (unsigned)p.lda, ldw = (unsigned)p.ldw;
    const unsigned a_row0 = (unsigned)(m0 + lrow) * lda, a_last = (unsigned)(p.M - 1) * lda;
    const unsigned w_row0 = (unsigned)(n0 + lrow) * ldw, w_last = (unsigned)(p.N - 1) * ldw;
#pragma unroll
    for (int b = 0; b < NI; ++b) {
        const unsigned co = 16u * (unsigned)(chunk0 ^ ((b & 1) << 2));
        if (b < NA) {
            if constexpr (kConv) {
                const int m = min(m0 + 8 * b + lrow, p.M - 1);
                const int t = (int)quotient((unsigned)m, p.div_wo), wo = m - t * p.cWo, bi = (int)quotient((unsigned)t, p.div_ho), ho = t - bi * p.cHo;
                ch[b] = ho * p.cStride - p.cPad;
                cw[b] = wo * p.cStride - p.cPad;
                voff[b] = (unsigned)(bi * p.cH * p.cW * p.cCin) + (co & 63u);
            } else {
                voff[b] = min(a_row0 + 8u * b * lda, a_last) + co + sha;
            }
        } else {
            voff[b] = min(w_row0 + 8u * (b - NA) * ldw, w_last) + co + shw;
        }
    }
    const unsigned ring = (unsigned)(uintptr_t)smem + wave * ring_bytes;
    int8_t* const ring_p = smem + wave * ring_bytes;

    // this wavefront's slices
    const int per = nk / KW, rem = nk % KW;
    const int s0 = wave * per + min(wave, rem), cnt = per + (wave < rem ? 1 : 0);
    const bool ragged = kLean && !kConv ? kEnd : (p.K & 127) != 0;   // the last slice is partly filled
    const int8_t* zero_src = g_zero_line + 16 * (lane & 7);

    // ---- aligned operands: slice t of this wavefront goes straight to its ring slot ----
    int ti = 0, tj = 0, tc = 0;   // kConv: tap and channel of the next half slice to load
    if constexpr (kConv) {
        const int tap = (int)quotient((unsigned)s0 * 128u, p.div_cin);
        tc = s0 * 128 - tap * p.cCin;
        ti = (int)quotient((unsigned)tap, p.div_kw);
        tj = tap - ti * p.cKw;
    }
    auto issue = [&](int t, int slot) {
        const int k0 = 128 * (s0 + t);
        const unsigned dst = ring + slot * SLICE;
        const bool part = ragged && k0 + 128 > p.K;  // wave-uniform
        if constexpr (kConv) {
            int h2[2], w2[2], c2[2];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                h2[hf] = ti; w2[hf] = tj; c2[hf] = tc;
                tc += 64;
                if (tc == p.cCin) { tc = 0; if (++tj == p.cKw) { tj = 0; ++ti; } }
            }
            // past the last tap the row is outside every image
            if (part) h2[1] = 1 << 28;
#pragma unroll
            for (int b = 0; b < NA; ++b) {
                const bool up = ((chunk0 ^ ((b & 1) << 2)) & 4) != 0;
                const int hi = ch[b] + (up ? h2[1] : h2[0]), wi = cw[b] + (up ? w2[1] : w2[0]);
                const bool in = (unsigned)hi < (unsigned)p.cH && (unsigned)wi < (unsigned)p.cW;
                const unsigned off = voff[b] + (unsigned)((hi * p.cW + wi) * p.cCin + (up ? c2[1] : c2[0]));
                dma16(in ? A + off : zero_src, dst + 1024 * b);
            }
        }
        if (part) {
#pragma unroll
            for (int b = kConv ? NA : 0; b < NI; ++b)
                dma16(k0 + 16 * (chunk0 ^ ((b & 1) << 2)) < p.K ? (b < NA ? A : W) + k0 + voff[b] : zero_src, dst + 1024 * b);
        } else {
#pragma unroll
            for (int b = kConv ? NA : 0; b < NI; ++b) dma16s((b < NA ? A : W) + k0, voff[b], dst + 1024 * b);
        }
    };

    v4i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4i{0, 0, 0, 0};
    // fragment addresses: row fr of a 16-row block, chunk 4 * ks + fq
    const int fsw = (fr >> 1) & 7;
    auto compute = [&](const int8_t* st) {
        v4i fa[2][TM], fw[2][TN];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int fo = fr * 128 + (((4 * ks + fq) ^ fsw) << 4);
#pragma unroll
            for (int j = 0; j < TN; ++j) fw[ks][j] = *reinterpret_cast<const v4i*>(st + BM * 128 + 2048 * j + fo);
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[ks][i] = *reinterpret_cast<const v4i*>(st + 2048 * i + fo);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    };

    // What the epilogue needs, behind the first slices: the waits for these count younger slices only, so a
    // slice that is waited for brings along some of it, which is needed as soon as the products are done.
    const int c4 = tid % G4, row0 = tid / G4;
    const int nb = n0 + 4 * c4;
    const bool n4 = kLean || (p.N & 3) == 0;   // a group of four columns is all in or all out
    v4f bias_r = {0.0f, 0.0f, 0.0f, 0.0f}, scale_r = {p.alpha, p.alpha, p.alpha, p.alpha};
    unsigned res_r[GPT];
    float2 kb_reg = make_float2(0.0f, 0.0f);   // one table entry (and word of a cell map) per thread; a larger table is staged late
    unsigned map_reg = 0;
    bool two_level = false, one_level = kTable && kForm == FORM_ANY;
    if constexpr (!kLean) {
        two_level = p.has_table && p.table.cellmap;
        one_level = p.has_table && !two_level;
    }
    auto request_epilogue = [&] {
        if (n4) {
            const int ncl = min(nb, p.N - 4);
            if (p.bias) bias_r = *reinterpret_cast<const v4f_a4*>(p.bias + ncl);
            if (p.alpha_vec) scale_r = *reinterpret_cast<const v4f_a4*>(p.alpha_vec + ncl);
            if (kLean ? kResid : p.resid != nullptr) {
#pragma unroll
                for (int t = 0; t < GPT; ++t)
                    res_r[t] = *reinterpret_cast<const u32_a1*>(p.resid + obase + (long)min(m0 + row0 + t * (NT / G4), p.M - 1) * p.ldo + ncl);
            }
        }
        if (one_level) kb_reg = p.table.kb[min(tid, p.table.nseg - 1)];
        if constexpr (!kLean) {
            if (two_level) {
                kb_reg = p.table.ckb[min(tid, p.table.nkb - 1)];
                map_reg = reinterpret_cast<const unsigned*>(p.table.cellmap)[min(tid, (p.table.nseg + 3) / 4 - 1)];
            }
        }
    };

    if (kAl == 16) {
#pragma unroll 1
        for (int d = 0; d < min(D, cnt); ++d) issue(d, d);
        request_epilogue();
        int slot = 0;
        for (int t = 0; t < cnt; ++t) {
            const int young = min(D - 1, cnt - 1 - t);   // younger slices in flight (wave-uniform)
            if (D >= 4 && young >= 3) wait_vmcnt<3 * NI>();
            else if (D >= 3 && young == 2) wait_vmcnt<2 * NI>();
            else if (D >= 2 && young == 1) wait_vmcnt<NI>();
            else wait_vmcnt<0>();
            compute(ring_p + slot * SLICE);
            if (t + D < cnt) {
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");   // the slot's fragments have been read
                issue(t + D, slot);
            }
            slot = slot + 1 == slots ? 0 : slot + 1;
        }
    } else {
        // ---- any alignment: through registers, the next slice requested before this one is used ----
        const rsrc_t ra = make_rsrc(A - sha, (a_last + (unsigned)p.K + sha + 3) & ~3u);
        const rsrc_t rw = make_rsrc(W - shw, (w_last + (unsigned)p.K + shw + 3) & ~3u);
        v4i reg[NI];
        auto fetch = [&](int t) {
            const unsigned k0 = 128u * (unsigned)(s0 + t);
            if (ragged && (int)k0 + 128 > p.K) {
#pragma unroll
                for (int b = 0; b < NI; ++b)
                    reg[b] = load_tail<kAl>(b < NA ? ra : rw, voff[b] + k0, p.K - (int)k0 - 16 * (chunk0 ^ ((b & 1) << 2)));
            } else {
#pragma unroll
                for (int b = 0; b < NI; ++b) reg[b] = load_unit<kAl>(b < NA ? ra : rw, voff[b] + k0);
            }
        };
        if (cnt > 0) fetch(0);
        request_epilogue();
        for (int t = 0; t < cnt; ++t) {
#pragma unroll
            for (int b = 0; b < NI; ++b) *reinterpret_cast<v4i*>(ring_p + 1024 * b + 16 * lane) = reg[b];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (t + 1 < cnt) fetch(t + 1);
            compute(ring_p);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }

    // Partial tiles meet in LDS, each in its wavefront's own ring (whose fragments have all been read).
    // Lane (fr, fq) holds row 16i + fr, columns 16j + 4fq .. +3.
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    if (kLean || cnt > 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                *reinterpret_cast<v4i*>(ring_p + (16 * i + fr) * (BN * 4) + 16 * pslot(16 * i + fr, 4 * j + fq)) = acc[i][j];
    }
    if (one_level) {
        if (tid < p.table.nseg) s_kb[tid] = kb_reg;
        for (int e = tid + NT; e < p.table.nseg; e += NT) s_kb[e] = p.table.kb[e];
    }
    if constexpr (!kLean) {
        if (two_level) {
            unsigned* map = reinterpret_cast<unsigned*>(s_kb + p.table.nkb);
            const int nw = (p.table.nseg + 3) / 4;
            if (tid < p.table.nkb) s_kb[tid] = kb_reg;
            if (tid < nw) map[tid] = map_reg;
            for (int e = tid + NT; e < p.table.nkb; e += NT) s_kb[e] = p.table.ckb[e];
            for (int e = tid + NT; e < nw; e += NT) map[e] = reinterpret_cast<const unsigned*>(p.table.cellmap)[e];
        }
    }
    __syncthreads();
    if (NGRP < NT && row0 >= BM) return;
    if (nb >= p.N) return;
    auto partial_sum = [&](int row) {
        const int8_t* at = smem + row * (BN * 4) + 16 * pslot(row, c4);
        v4i s = *reinterpret_cast<const v4i*>(at);
#pragma unroll
        for (int w = 1; w < KW; ++w)
            if (kLean || w < rings) s += *reinterpret_cast<const v4i*>(at + w * ring_bytes);
        return s;
    };
    if constexpr (kLean) {
        const long at0 = (long)(m0 + row0) * (long)p.ldo + nb;
        const int left = p.M - (m0 + row0);
        v4f inv = {p.out_inv_scale, p.out_inv_scale, p.out_inv_scale, p.out_inv_scale};
        if (kEpi == EPI_Q && p.split_cols > 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) inv[e] = nb + e >= 2 * p.split_cols ? p.inv3[2] : nb + e >= p.split_cols ? p.inv3[1] : p.inv3[0];
        }
        v4i a[GPT];
        v4f y[GPT];
#pragma unroll
        for (int t = 0; t < GPT; ++t) a[t] = partial_sum(row0 + t * (NT / G4));
#pragma unroll
        for (int t = 0; t < GPT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = __builtin_fmaf((float)a[t][e], scale_r[e], bias_r[e]);
                if (kResid) v = __builtin_fmaf((float)(int)(int8_t)(res_r[t] >> (8 * e)), p.resid_scale, v);
                if (kTable && kForm == FORM_TWO_SEGMENTS) v = pwl_eval_two_segments(v, p.table);
                int seg;
                if (kTable && kForm == FORM_ANY) v = pwl_eval_noclamp(v, p.table, s_kb, seg);
                y[t][e] = v;
            }
#pragma unroll
        for (int t = 0; t < GPT; ++t)
            if (t * (NT / G4) < left) {
                const long at = at0 + (long)(t * (NT / G4)) * p.ldo;
                if (kEpi == EPI_F32_RESID) *reinterpret_cast<v4f*>(p.out_f32 + at) = y[t];
                else *reinterpret_cast<unsigned*>(p.out_q + at) =
                         pack4(requant(y[t][0], inv[0]), requant(y[t][1], inv[1]), requant(y[t][2], inv[2]), requant(y[t][3], inv[3]));
            }
    } else if (n4 && p.vec_out) {
        v4f inv = {p.out_inv_scale, p.out_inv_scale, p.out_inv_scale, p.out_inv_scale};
        if (p.out_inv_scale_vec) {
            inv = *reinterpret_cast<const v4f_a4*>(p.out_inv_scale_vec + nb);
        } else if (p.split_cols > 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) inv[e] = nb + e >= 2 * p.split_cols ? p.inv3[2] : nb + e >= p.split_cols ? p.inv3[1] : p.inv3[0];
        }
        v4i a[GPT];
        float y[GPT][4];
        int seg[GPT][4];
        const float scale[4] = {scale_r[0], scale_r[1], scale_r[2], scale_r[3]}, bias[4] = {bias_r[0], bias_r[1], bias_r[2], bias_r[3]};
#pragma unroll
        for (int t = 0; t < GPT; ++t) a[t] = partial_sum(row0 + t * (NT / G4));
        epi_values<GPT>(p, s_kb, a, scale, bias, res_r, y, seg);
        const long at0 = obase + (long)(m0 + row0) * p.ldo + nb;
        const int left = p.M - (m0 + row0);
        auto each = [&](auto store) {
#pragma unroll
            for (int t = 0; t < GPT; ++t)
                if (t * (NT / G4) < left) store(at0 + (long)(t * (NT / G4)) * p.ldo, t);
        };
        if (p.out_q)
            each([&](long at, int t) {
                *reinterpret_cast<unsigned*>(p.out_q + at) = pack4(requant(y[t][0], inv[0]), requant(y[t][1], inv[1]), requant(y[t][2], inv[2]), requant(y[t][3], inv[3]));
            });
        if (p.out_f32) each([&](long at, int t) { *reinterpret_cast<v4f*>(p.out_f32 + at) = v4f{y[t][0], y[t][1], y[t][2], y[t][3]}; });
        if (p.out_acc) each([&](long at, int t) { *reinterpret_cast<v4i*>(p.out_acc + at) = a[t]; });
        if (p.dbg_seg && p.has_table)
            each([&](long at, int t) {
                *reinterpret_cast<uint2*>(p.dbg_seg + at) = make_uint2((unsigned)seg[t][0] | ((unsigned)seg[t][1] << 16), (unsigned)seg[t][2] | ((unsigned)seg[t][3] << 16));
            });
    } else {
        Col4 c;
        load_cols<EPI_GENERIC>(p, nb, c);
#pragma unroll 1
        for (int t = 0; t < GPT; ++t) {
            const int row = row0 + t * (NT / G4), m = m0 + row;
            if (m >= p.M) break;
            const v4i a = partial_sum(row);
            int a4[4] = {a[0], a[1], a[2], a[3]}, r4[4] = {0, 0, 0, 0};
            if (p.resid) load_resid4(p, obase + (long)m * p.ldo, nb, false, r4);
            Epi4 o;
            epi_math<EPI_GENERIC>(p, s_kb, a4, c, r4, o);
            epi_store<EPI_GENERIC>(p, obase + (long)m * p.ldo, nb, a4, o, false, false);
        }
    }
}

template <int BM, int BN, int KW, int D, int kAl, bool kConv, int kEpi, int kForm, bool kEnd>
__global__ __launch_bounds__(64 * KW) void gemm_direct_kernel(DirectArgs<kConv, kEpi> p)
{
    direct_tile<BM, BN, KW, D, kAl, kConv, kEpi, kForm, kEnd>(p, blockIdx.x);
}

// Two convolutions that do not depend on one another (the 3x3 one of a residual block and the projection of its shortcut): the workgroups of
// the second behind the first's.  At small batches either is half a launch.  us, two launches -> one, four such pairs: ResNet-50 on one image of 224 x 224
// 196 -> 188, a network of one block a stage 79 -> 71, on three images of 160 x 160 83 -> 75.
struct DirectPair {
    DirectConvParams p[2];
    unsigned first;   // workgroups of the first, a multiple of 8
};
template <int BM, int BN, int KW, int D>
__global__ __launch_bounds__(64 * KW) void gemm_direct_pair_kernel(DirectPair q)
{
    const bool second = blockIdx.x >= q.first;
    direct_tile<BM, BN, KW, D, 16, true, EPI_Q_TABLE, FORM_TWO_SEGMENTS, false>(second ? q.p[1] : q.p[0], second ? blockIdx.x - q.first : blockIdx.x);
}

template <int BM, int BN, int KW, int D, int kAl, bool kConv, int kEpi = EPI_GENERIC, int kForm = FORM_ANY, bool kEnd = false>
static int32_t launch_direct_t(GemmParams& p, int batches, size_t table_bytes, hipStream_t s)
{
    auto kern = gemm_direct_kernel<BM, BN, KW, D, kAl, kConv, kEpi, kForm, kEnd>;
    const int nk = (p.K + 127) / 128, need = (nk + KW - 1) / KW;
    const size_t shmem = (size_t)(nk < KW && kEpi == EPI_GENERIC ? nk : KW) * (need < D ? need : D) * (BM + BN) * 128 + table_bytes;
    static std::once_flag once;  // one attribute call per instantiation
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(gemm_direct_kernel)");
    });
    if (once_rc) return once_rc;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    p.batched = batches > 1;
    p.div_tiles_m = fast_div(p.tiles_m);
    if (kConv) p.div_wo = fast_div(p.cWo), p.div_ho = fast_div(p.cHo), p.div_cin = fast_div(p.cCin), p.div_kw = fast_div(p.cKw);
    const int grid = (p.tiles_m * p.tiles_n + 7) / 8 * 8;   // the kernel's eighths are (tiles + 7) / 8 each
    DirectArgs<kConv, kEpi> args;
    direct_args(args, p);
    queue_kernel(kern, dim3(grid, batches), dim3(64 * KW), shmem, s, args);
    return NM_OK;
}

// The fixed epilogue that computes what p asks for (and nothing else), or EPI_GENERIC.
static int lean_epilogue(const GemmParams& p, bool conv, int batches)
{
    if (batches != 1 || p.N % 4 != 0 || !p.vec_out || p.ldo >= (1LL << 31) || (!conv && p.K % 16 != 0)) return EPI_GENERIC;
    if (p.dbg_seg || p.out_acc || p.out_inv_scale_vec || (p.out_q != nullptr) == (p.out_f32 != nullptr)) return EPI_GENERIC;
    if (p.has_table && (p.table.cellmap || p.table.clamp_input || p.split_cols > 0)) return EPI_GENERIC;
    if (p.out_f32) return p.resid && !p.has_table ? EPI_F32_RESID : EPI_GENERIC;
    if (p.resid) return p.has_table && p.table.two_seg ? EPI_Q_TABLE_RESID : EPI_GENERIC;
    return p.has_table ? EPI_Q_TABLE : EPI_Q;
}

template <int BM, int BN, int KW, int D>
static int32_t launch_direct_conv(GemmParams& p, int batches, size_t table_bytes, hipStream_t s)
{
    const int epi = lean_epilogue(p, true, batches);
    if (epi == EPI_Q) return launch_direct_t<BM, BN, KW, D, 16, true, EPI_Q>(p, batches, 0, s);
    if (epi == EPI_Q_TABLE && p.table.two_seg) return launch_direct_t<BM, BN, KW, D, 16, true, EPI_Q_TABLE, FORM_TWO_SEGMENTS>(p, batches, 0, s);
    return launch_direct_t<BM, BN, KW, D, 16, true>(p, batches, table_bytes, s);
}

template <int BM, int BN, int KW, int D>
static int32_t launch_direct_aligned(GemmParams& p, bool conv, int batches, size_t table_bytes, hipStream_t s)
{
    if (conv) return launch_direct_conv<BM, BN, KW, D>(p, batches, table_bytes, s);
    const int epi = lean_epilogue(p, false, batches);
    const bool two = p.has_table && p.table.two_seg;
    if (p.K % 128 != 0) {
        if (epi == EPI_Q) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_Q, FORM_ANY, true>(p, batches, 0, s);
        if (epi == EPI_F32_RESID) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_F32_RESID, FORM_ANY, true>(p, batches, 0, s);
        if (epi == EPI_Q_TABLE) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_Q_TABLE, FORM_ANY, true>(p, batches, table_bytes, s);
        return launch_direct_t<BM, BN, KW, D, 16, false>(p, batches, table_bytes, s);
    }
    if (epi == EPI_Q) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_Q>(p, batches, 0, s);
    if (epi == EPI_F32_RESID) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_F32_RESID>(p, batches, 0, s);
    if (epi == EPI_Q_TABLE_RESID) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_Q_TABLE_RESID, FORM_TWO_SEGMENTS>(p, batches, 0, s);
    if (epi == EPI_Q_TABLE && two) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_Q_TABLE, FORM_TWO_SEGMENTS>(p, batches, 0, s);
    if (epi == EPI_Q_TABLE) return launch_direct_t<BM, BN, KW, D, 16, false, EPI_Q_TABLE>(p, batches, table_bytes, s);
    return launch_direct_t<BM, BN, KW, D, 16, false>(p, batches, table_bytes, s);
}

template <int BM, int BN, int KW>
static int32_t launch_direct_unaligned(GemmParams& p, int align, int batches, size_t table_bytes, hipStream_t s)
{
    if (align >= 4) return launch_direct_t<BM, BN, KW, 1, 4, false>(p, batches, table_bytes, s);
    return launch_direct_t<BM, BN, KW, 1, 1, false>(p, batches, table_bytes, s);
}

// forced: a configuration that direct_takes, or -1 for the rule.  Operands aligned to 4 or 1 bytes pass through registers, a slice at a time: the
// smallest tile whose workgroups still fit the chip about once, beyond that the one that reads its operands least often.
int32_t launch_direct(GemmParams& p, int align, bool conv, int batches, size_t table_bytes, int forced, hipStream_t s)
{
    if (align < 16) {
        const long t32 = (long)((p.M + 31) / 32) * ((p.N + 31) / 32) * batches;
        const long wide_from = p.K >= 576 ? 640 : p.K >= 512 ? 1100 : 1L << 40;
        if (t32 <= 128) return launch_direct_unaligned<16, 32, 8>(p, align, batches, table_bytes, s);
        if (t32 <= 256 && p.K >= 2048) return launch_direct_unaligned<32, 32, 8>(p, align, batches, table_bytes, s);
        if (t32 <= wide_from) return launch_direct_unaligned<32, 32, 4>(p, align, batches, table_bytes, s);
        return launch_direct_unaligned<32, 64, 4>(p, align, batches, table_bytes, s);
    }
    switch (forced >= 0 ? forced : choose_direct(p.M, p.N, p.K, batches, table_bytes, conv)) {
    case 0: return launch_direct_aligned<16, 32, 8, 3>(p, conv, batches, table_bytes, s);
    case 1: return launch_direct_aligned<32, 32, 4, 2>(p, conv, batches, table_bytes, s);
    case 2: return launch_direct_aligned<32, 64, 4, 1>(p, conv, batches, table_bytes, s);
    case 3: return launch_direct_aligned<32, 64, 8, 1>(p, conv, batches, table_bytes, s);
    case 4: return launch_direct_aligned<48, 64, 4, 2>(p, conv, batches, table_bytes, s);
    case 6: return launch_direct_conv<32, 32, 8, 2>(p, batches, table_bytes, s);
    default: return launch_direct_aligned<64, 64, 4, 2>(p, conv, batches, table_bytes, s);
    }
}

template <int BM, int BN, int KW, int D>
static int32_t launch_pair(GemmParams (&p)[2], hipStream_t s)
{
    auto kern = gemm_direct_pair_kernel<BM, BN, KW, D>;
    static std::once_flag once;  // one attribute call per instantiation
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(gemm_direct_pair_kernel)");
    });
    if (once_rc) return once_rc;
    DirectPair q;
    size_t shmem = 0;
    unsigned grid[2];
    for (int i = 0; i < 2; ++i) {
        const int need = ((p[i].K + 127) / 128 + KW - 1) / KW;
        const size_t lds = (size_t)KW * (need < D ? need : D) * (BM + BN) * 128;
        shmem = shmem > lds ? shmem : lds;
        p[i].tiles_m = (p[i].M + BM - 1) / BM;
        p[i].tiles_n = (p[i].N + BN - 1) / BN;
        p[i].batched = 0;
        p[i].div_tiles_m = fast_div(p[i].tiles_m);
        p[i].div_wo = fast_div(p[i].cWo), p[i].div_ho = fast_div(p[i].cHo), p[i].div_cin = fast_div(p[i].cCin), p[i].div_kw = fast_div(p[i].cKw);
        grid[i] = (unsigned)(p[i].tiles_m * p[i].tiles_n + 7) / 8 * 8;
        direct_args(q.p[i], p[i]);
        if (!p[i].has_table) q.p[i].table.k0 = q.p[i].table.k1 = 1.0f, q.p[i].table.b0 = q.p[i].table.b1 = q.p[i].table.tau = 0.0f;   // x itself
    }
    q.first = grid[0];
    queue_kernel(kern, dim3(grid[0] + grid[1]), dim3(64 * KW), shmem, s, q);
    return check_hip(hipGetLastError(), "gemm pair launch");
}

bool direct_pair_takes(const GemmParams& p)
{
    const int epi = lean_epilogue(p, true, 1);
    return epi == EPI_Q || (epi == EPI_Q_TABLE && p.table.two_seg);
}

int32_t launch_direct_pair(GemmParams (&p)[2], int cfg, hipStream_t s)
{
    switch (cfg) {
    case 0: return launch_pair<16, 32, 8, 3>(p, s);
    case 1: return launch_pair<32, 32, 4, 2>(p, s);
    case 2: return launch_pair<32, 64, 4, 1>(p, s);
    case 3: return launch_pair<32, 64, 8, 1>(p, s);
    case 4: return launch_pair<48, 64, 4, 2>(p, s);
    case 6: return launch_pair<32, 32, 8, 2>(p, s);
    default: return launch_pair<64, 64, 4, 2>(p, s);
    }
}

}  // namespace nm
