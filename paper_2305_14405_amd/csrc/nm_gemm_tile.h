// The large-tile int8 GEMM kernel (paper Section 3.1: fully connected layers as matrix products;
// Section 3.2: the nonlinearity behind one is the PWL calculation y = k[s]*x + b[s]).
#pragma once

#include "nm_attention.h"
#include "nm_gemm_common.h"

namespace nm {

// ---------------------------------------------------------------------------------------------
// Tile kernel: the large-tile path for the plain matrix products of the encoder layer (aligned
// operands, K a multiple of 16 and more than 256, scalar alpha, int8 output with or without the table, or fp32
// output with the int8 residual).  Same LDS image and MFMA operand roles as the streaming kernel;
// what differs is how the instruction stream is laid out:
//  * the k-loop is software-pipelined by hand and its issue order is pinned with scheduling
//    barriers: one matrix instruction, then at most one LDS fragment read (for the NEXT k-step, into
//    the other of two fragment register sets) and one global -> LDS load in its shadow.  A wavefront
//    therefore never waits for a fragment it has just asked for, and the one barrier per k-slice
//    sits in the middle of a k-step whose fragments are already in registers;
//  * a k-slice's ring slot is refilled right after that barrier (all of its fragments have been
//    read by then), addresses are one scalar base per operand plus a 32-bit lane offset;
//  * first slice, steady state and the last slices are straight-line code around one loop, so the
//    accumulators stay in the same registers throughout;
//  * the per-column vectors and the table are fetched when the kernel starts but written to LDS
//    after the k-loop (nothing in front of the first operand slice waits for them);
//  * the epilogue works on groups of four columns; the table look-up of a group is issued three
//    groups before its result is used, and int8 rows leave through an LDS patch as 16-byte stores.
// Two wavefronts on every SIMD: the fp32 epilogue issues almost twice as fast that way as with one (measured:
// a single wavefront cannot issue dependent-free vector instructions back to back at the SIMD's full
// rate).  The large tiles do it with eight wavefronts, the small ones with four and, in a ring of two
// stages, two workgroups per CU: one's prologue and epilogue then run under the other's matrix work
// (16384 x 4096 x 1024 with table, 128x192 tiles: 122 us with one workgroup and three stages, 89 with two).
//
// What bounds it.  256x256 tiles at 16384 x 1024 x 4096: 64 us, of which 10 are the 64 MB of fp32 results and about
// 5 launch and prologue; the k-loop runs at the rate the card's power allows (all operands zero: 54 us
// with the same instructions; operand rows that all lie in L2: no change).  256x128 tiles there: 72 us, because
// a slice then needs 47 bytes per matrix clock and CU through the direct loads, which deliver about 40 (256x256: 32).
// With short K the epilogue is the larger part: 10 vector instructions per element with the table, 6 without.
// ---------------------------------------------------------------------------------------------
// LDS that the epilogue lays over the ring: the wavefronts' int8 row patches, or the residual tile and the
// wavefronts' fp32 row patches, then the bias and the table.
// In front of the int8 patches of EPI_Q_TABLE lie the table's slots, so that a slot's offset is its address.
constexpr int tile_front_bytes(int bm, int bn, int nw, int wm, int wn, int epi)
{
    return epi == EPI_ATTENTION ? (int)kSlotBytes + kQkvRecip * 8 + 3 * bm * 64 + nw * kCtxPatch
         : epi == EPI_Q_TABLE ? (int)kSlotBytes + nw * wm * (wn + 16)
         : epi == EPI_Q_RELU_RESID ? bm * (bn + 16)
         : epi == EPI_F32_RESID_LN ? bm * (bn + 16) + (bm * 64 + 2 * bm) * 4
         : epi == EPI_F32_RESID ? bm * (bn + 16) + nw * 32 * (wn + 4) * 4 : nw * wm * (wn + 16);
}

template <int kEpi>
using TileParams = std::conditional_t<kEpi == EPI_F32_RESID_LN, GemmLnParams, std::conditional_t<kEpi == EPI_ATTENTION, QkvAttnParams, GemmParams>>;

// kEnd: K is a multiple of 16 but not of 128.  The last slice is then the last 128 bytes of K, whose first chunks the slice in front has had
// already: of A they are cleared in registers (around other matrix instructions for this slice the compiler moves accumulators
// between register classes and spills, whole slices or not: 256x256 tiles 400 registers).
template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int kEpi, int BK = 128, bool kConv = false, int KSPLIT = 1, bool kEnd = false>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * KSPLIT, 2) void gemm_tile_kernel(TileParams<kEpi> p)
{
    constexpr int NWT = WAVES_M * WAVES_N;   // wavefront tiles
    constexpr int NW = NWT * KSPLIT;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int EM = WM / KSPLIT, ETM = TM / KSPLIT;   // rows, 32-row blocks a wavefront finishes
    constexpr int ROWS = BM + BN;
    constexpr int CPR = BK / 16;
    constexpr int RPI = 64 / CPR;
    constexpr int NBLK = ROWS / RPI;         // 1 KB blocks of a k-slice
    constexpr int LB = (NBLK + NW - 1) / NW; // ... per wavefront: when they do not split evenly the last
                                             // ones are fetched twice into spare LDS behind the stage
    constexpr int ABLK = BM / RPI;           // blocks that hold A rows
    constexpr bool kEven = NBLK % NW == 0 && ABLK % NW == 0;
    constexpr int LBA = ABLK / NW;           // A blocks per wavefront (even split)
    constexpr int STAGE_BYTES = LB * NW * 1024;
    constexpr int KS = BK / 32 / KSPLIT;     // k-steps of a slice that are the wavefront's
    constexpr int NR = TM + TN;              // fragments per k-step
    constexpr int NMF = TM * TN;             // matrix instructions per k-step
    constexpr int HALF = NMF - NR >= 1 ? NMF - NR : 1;  // ... of the last k-step in front of the slice barrier
    constexpr int POST = NMF - HALF;                    // issue slots behind it
    constexpr int RPS = (NR + POST - 1) / POST;         // fragment reads per slot there
    constexpr int RPS2 = (NR + NMF - 1) / NMF;          // ... and in the other k-steps
    constexpr int DPS = (LB + POST + NMF - 1) / (POST + NMF);  // refill loads per slot (those slots and the next k-step's)
    static_assert(ROWS % RPI == 0 && BM % RPI == 0, "whole blocks");
    static_assert(TN >= 2 && KS % 2 == 0 && TM % KSPLIT == 0, "wavefront tile");
    constexpr bool kSlots = kEpi == EPI_Q_TABLE, kTable = kSlots || kEpi == EPI_Q_LONG;
    constexpr bool kRelu = kEpi == EPI_Q_RELU || kEpi == EPI_Q_RELU_RESID;   // per-column scales, two segments
    static_assert(kEpi == EPI_Q || kTable || kRelu || kEpi == EPI_F32_RESID || kEpi == EPI_F32_RESID_LN || kEpi == EPI_ATTENTION,
                  "epilogues of the tile kernel");
    static_assert(!kConv || kEven, "gathered rows: a wavefront's A blocks are the same for every slice");
    static_assert(kEpi != EPI_F32_RESID_LN || WAVES_M == 1, "row statistics: a wavefront holds all rows of its columns");
    constexpr bool kResid = kEpi == EPI_F32_RESID || kEpi == EPI_F32_RESID_LN || kEpi == EPI_Q_RELU_RESID;

    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    float* s_bias = reinterpret_cast<float*>(smem + tile_front_bytes(BM, BN, NW, EM, WN, kEpi));
    float2* s_kb = reinterpret_cast<float2*>(s_bias + BN);
    float* s_scale = s_bias + BN;   // kRelu (which has no table in LDS)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KSPLIT == 1 ? 0 : wave / NWT, wave_t = KSPLIT == 1 ? wave : wave % NWT;   // half of the k-steps, sub-tile
    const int wave_m = (wave_t / WAVES_N) * WM;
    const int wave_n = (wave_t % WAVES_N) * WN;

    // the arguments of everything in front of the first loads, in one step
    asm volatile("" : : "s"(p.A), "s"(p.W), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.lda), "s"(p.ldw), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.group_m),
                 "s"(p.div_group.magic), "s"(p.div_group.shift), "s"(p.div_gm.magic), "s"(p.div_gm.shift), "s"(p.bias));
    // Workgroup i runs on XCD i % 8: an XCD gets a contiguous eighth of the tile sequence, which walks groups of
    // group_m tile rows column by column (xcd_group_rows).
    const int ntiles = p.tiles_m * p.tiles_n, share = (ntiles + 7) >> 3;
    const int id = (blockIdx.x & 7) * share + (blockIdx.x >> 3);
    if (id >= ntiles) return;
    const int GM = p.group_m, group = (int)quotient((unsigned)id, p.div_group);   // by GM * tiles_n
    const int first_m = group * GM, gm = min(GM, p.tiles_m - first_m);
    const int in_group = id - first_m * p.tiles_n;
    const int tile_n = gm == GM ? (int)quotient((unsigned)in_group, p.div_gm) : in_group / gm;
    const int tile_m = first_m + in_group - tile_n * gm;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    // per-lane byte offsets of this wavefront's blocks (rows past the edge are clamped: they only
    // feed accumulators that are never stored); M * K and N * K fit 32 bits (host)
    // kConv: row r of A is an output position; ctap[b] has a bit for every filter tap whose input position lies inside the
    // image, voff[b] is the (possibly negative) offset of the tap (0, 0).
    unsigned voff[LB];
    unsigned ctap[kConv ? LBA : 1];
    if constexpr (kConv)
        asm volatile("" : : "s"(p.cH), "s"(p.cW), "s"(p.cCin), "s"(p.taps_w), "s"(p.cStride), "s"(p.cPad), "s"(p.cWo), "s"(p.cHo),
                     "s"(p.div_wo.magic), "s"(p.div_wo.shift), "s"(p.div_ho.magic), "s"(p.div_ho.shift));
#pragma unroll
    for (int b = 0; b < LB; ++b) {
        const int blk = wave + b * NW;
        const int r = blk * RPI + lane / CPR;
        const int chunk = (lane % CPR) ^ swz_bk<BK>(r);
        const bool is_a = kEven ? b < LBA : blk < ABLK;  // wave-uniform
        if constexpr (kEpi == EPI_ATTENTION) {
            // row r: token r % keys of the workgroup's sequence r / keys; column c: of Q, K or V (c / 64) of head tile_n
            static_assert(BM == 128 && BN == 192, "a head's Q, K and V");
            const int seq = min((tile_m << (7 - p.keys_log2)) + (r >> p.keys_log2), p.B - 1), token = min(r & ((1 << p.keys_log2) - 1), p.at.S - 1);
            const int c = r - BM;
            voff[b] = (is_a ? (unsigned)(seq * p.at.S + token) * (unsigned)p.lda : (unsigned)((c >> 6) * p.at.H + tile_n * 64 + (c & 63)) * (unsigned)p.ldw) + 16u * chunk;
        } else if (kConv && b < LBA) {
            if constexpr (kConv) {
                const int m = min(m0 + r, p.M - 1), q = (int)quotient((unsigned)m, p.div_wo), bi = (int)quotient((unsigned)q, p.div_ho);
                const int h0 = (q - bi * p.cHo) * p.cStride - p.cPad, w0 = (m - q * p.cWo) * p.cStride - p.cPad;
                voff[b] = (unsigned)(((bi * p.cH + h0) * p.cW + w0) * p.cCin + 16 * chunk);
                // taps of a row that lie inside, then the rows
                unsigned cols = 0;
                for (int j = 0; j < p.taps_w; ++j) cols |= (unsigned)(w0 + j) < (unsigned)p.cW ? 1u << j : 0u;
                const int rows = p.K / (p.cCin * p.taps_w);
                unsigned in = 0;
                for (int i = 0; i < rows; ++i) in |= (unsigned)(h0 + i) < (unsigned)p.cH ? cols << (i * p.taps_w) : 0u;
                ctap[b] = in;
            }
        } else if (is_a) voff[b] = (unsigned)min(m0 + r, p.M - 1) * (unsigned)p.lda + 16u * chunk;
        else voff[b] = (unsigned)min(n0 + r - BM, p.N - 1) * (unsigned)p.ldw + 16u * chunk;
    }
    const unsigned lds_base = (unsigned)(uintptr_t)smem;
    const int8_t* __restrict__ gA = p.A;
    const int8_t* __restrict__ gW = p.W;
    // kConv: tap and offset of the slice whose A blocks are requested next (slices are requested in order)
    unsigned tap_bit = 1;
    int tap_off = 0, tap_col = 0, tap_c = 0;
    const int8_t* const zero_src = g_zero_line + 16 * (lane % CPR);
    auto issue1 = [&](int kt, int slot, int b) {
        const unsigned dst = lds_base + slot * STAGE_BYTES + (wave + b * NW) * 1024;
        if constexpr (kConv) {
            if (b < LBA) {
                dma16((ctap[b] & tap_bit) ? gA + (int)(voff[b] + (unsigned)tap_off) : zero_src, dst);
                if (b == LBA - 1) {
                    tap_off += BK;
                    tap_c += BK;
                    if (tap_c == p.cCin) {   // the next tap's offset is that of this one's end, but for the image's row
                        tap_c = 0;
                        tap_bit <<= 1;
                        if (++tap_col == p.taps_w) { tap_col = 0; tap_off += (p.cW - p.taps_w) * p.cCin; }
                    }
                }
                return;
            }
        }
        const bool is_a = kEven ? b < LBA : wave + b * NW < ABLK;
        dma16s((is_a ? gA : gW) + (kEnd ? min((long)kt * BK, (long)p.K - BK) : (long)kt * BK), voff[b], dst);
    };
    const int nk = kEnd ? (p.K + BK - 1) / BK : p.K / BK;  // >= STAGES + 1 (host; any with kShort)
    const int first_chunk = kEnd ? nk * CPR - p.K / 16 : 0;   // that counts in the last slice
    static_assert(!kEnd || (!kRelu && !kConv && BK == 128), "whole slices");
    constexpr bool kShort = kRelu;
#pragma unroll
    for (int st = 0; st < STAGES; ++st) {
        if (kShort && st >= nk) break;
#pragma unroll
        for (int b = 0; b < LB; ++b) issue1(st, st, b);
    }

    // epilogue parameters: fetched now, parked in registers until the k-loop is over
    constexpr int BPT = (BN + 64 * NW - 1) / (64 * NW);
    float bias_reg[BPT], scale_reg[kRelu ? BPT : 1];
#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        const int c = tid + t * 64 * NW;
        if constexpr (kEpi == EPI_ATTENTION) bias_reg[t] = (p.bias && c < BN) ? p.bias[(c >> 6) * p.at.H + tile_n * 64 + (c & 63)] : 0.0f;
        else bias_reg[t] = (p.bias && c < BN && n0 + c < p.N) ? p.bias[n0 + c] : 0.0f;
        if (kRelu) scale_reg[t] = (p.alpha_vec && c < BN && n0 + c < p.N) ? p.alpha_vec[n0 + c] : p.alpha;
    }
    static_assert(!kSlots || 64 * NW >= kSlotSegments, "a slot per thread");
    constexpr int KPT = kSlots ? 1 : 4;   // table entries per thread held in registers (more are staged late)
    float2 kb_reg[KPT];
    if (kTable) {
#pragma unroll
        for (int t = 0; t < KPT; ++t) kb_reg[t] = p.table.kb[min(tid + t * 64 * NW, p.table.nseg - 1)];
    }

    AttnTables<EXP_SLOTS, kEpi == EPI_ATTENTION ? 64 * NW : kSlotSegments> attn_tabs;
    if constexpr (kEpi == EPI_ATTENTION) attn_tabs.request(p.at);

    // the int8 residual tile (fp32 epilogue) as 16-byte row pieces
    constexpr int CPRW = BN / 16;
    constexpr int RPT = (BM * CPRW + 64 * NW - 1) / (64 * NW);
    v4i res_reg[RPT];
    if (kResid) {
#pragma unroll
        for (int t = 0; t < RPT; ++t) {
            const int c = tid + t * 64 * NW, row = c / CPRW, cc = c % CPRW;
            const int mr = m0 + row, n = n0 + 16 * cc;
            res_reg[t] = v4i{0, 0, 0, 0};
            if (c < BM * CPRW && mr < p.M && n < p.N) res_reg[t] = *reinterpret_cast<const v4i*>(p.resid + (long)mr * p.ldo + n);
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
    int offA[KS], offW[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int ra = wave_m + frag_row, rw = wave_n + frag_row;
        offA[ks] = lds_off_bk<BK>(ra, 2 * (kg * KS + ks) + frag_half);
        offW[ks] = BM * BK + lds_off_bk<BK>(rw, 2 * (kg * KS + ks) + frag_half);
    }
    v4i fa[2][TM], fw[2][TN];
    // fragment t of a k-step, in the order the matrix instructions of that k-step need them
    auto ldfrag1 = [&](int buf, int slot, int ks, int t) {
        const int8_t* st = smem + slot * STAGE_BYTES;
        if (t == 0) fw[buf][0] = *reinterpret_cast<const v4i*>(st + offW[ks]);
        else if (t == 1) fa[buf][0] = *reinterpret_cast<const v4i*>(st + offA[ks]);
        else if (t < 1 + TN) fw[buf][t - 1] = *reinterpret_cast<const v4i*>(st + offW[ks] + (t - 1) * 32 * BK);
        else fa[buf][t - TN] = *reinterpret_cast<const v4i*>(st + offA[ks] + (t - TN) * 32 * BK);
    };

    // k-slice 0 has landed (the younger slices of the prologue stay in flight)
    if (kShort && nk == 1) wait_vmcnt<0>();
    else if (kShort && STAGES > 2 && nk == 2) wait_vmcnt<LB>();
    else wait_vmcnt<(STAGES - 1) * LB>();
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NR; ++t) ldfrag1(0, 0, 0, t);

    int slot = 0, pslot = 0;
    // One k-slice.  MORE: slice kt + STAGES exists and refills this slice's slot (first blocks);
    // MOREP: the rest of the refill begun during the previous slice; YOUNG: slices younger than
    // kt + 1 in flight when kt + 1 is awaited (-1: there is no slice kt + 1).
    auto slice = [&](auto more_c, auto morep_c, auto young_c, int kt) {
        constexpr bool MORE = decltype(more_c)::value, MOREP = decltype(morep_c)::value;
        constexpr int YOUNG = decltype(young_c)::value;
        const int nslot = slot + 1 == STAGES ? 0 : slot + 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int cur = ks & 1;
#pragma unroll
            for (int t = 0; t < NMF; ++t) {
                const int i = t / TN, j = t % TN;
                if (kEnd && YOUNG < 0 && t == 0) {
                    const bool counts = 2 * (kg * KS + ks) + frag_half >= first_chunk;
#pragma unroll
                    for (int r = 0; r < TM; ++r)
#pragma unroll
                        for (int e = 0; e < 4; ++e) fa[cur][r][e] = counts ? fa[cur][r][e] : 0;
                }
                if (ks == KS - 1 && t == HALF && YOUNG >= 0) {
                    // every wavefront has read all of slice kt (its last fragments were requested
                    // during the previous k-step); slice kt + 1 has landed for this wavefront
                    wait_vmcnt<(YOUNG > 0 ? YOUNG : 0) * LB>();
                    __syncthreads();
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[cur][j], fa[cur][i], acc[i][j], 0, 0, 0);
                if (ks < KS - 1) {
#pragma unroll
                    for (int r = t * RPS2; r < (t + 1) * RPS2; ++r)
                        if (r < NR) ldfrag1(cur ^ 1, slot, ks + 1, r);
                    if (MOREP && ks == 0) {
#pragma unroll
                        for (int d = (POST + t) * DPS; d < (POST + t + 1) * DPS; ++d)
                            if (d < LB) issue1(kt - 1 + STAGES, pslot, d);
                    }
                } else if (t >= HALF) {
                    const int u = t - HALF;
                    if (YOUNG >= 0) {
#pragma unroll
                        for (int r = u * RPS; r < (u + 1) * RPS; ++r)
                            if (r < NR) ldfrag1(cur ^ 1, nslot, 0, r);
                    }
                    if (MORE) {
#pragma unroll
                        for (int d = u * DPS; d < (u + 1) * DPS; ++d)
                            if (d < LB) issue1(kt + STAGES, slot, d);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        pslot = slot;
        slot = nslot;
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    auto tail = [&](auto self, auto r_c) -> void {
        constexpr int R = decltype(r_c)::value;  // slices after this one
        slice(F_{}, F_{}, std::integral_constant<int, R - 1>{}, nk - 1 - R);
        if constexpr (R > 0) self(self, std::integral_constant<int, R - 1>{});
    };
    if (kShort && nk == 1) {
        tail(tail, std::integral_constant<int, 0>{});
    } else if (kShort && nk == 2) {
        tail(tail, std::integral_constant<int, 1>{});
    } else if (kShort && STAGES > 2 && nk == 3) {
        tail(tail, std::integral_constant<int, (STAGES > 2 ? 2 : 1)>{});
    } else {
        slice(T_{}, F_{}, std::integral_constant<int, STAGES - 2>{}, 0);
        for (int kt = 1; kt < nk - STAGES; ++kt) slice(T_{}, T_{}, std::integral_constant<int, STAGES - 2>{}, kt);
        slice(F_{}, T_{}, std::integral_constant<int, STAGES - 2>{}, nk - STAGES);
        tail(tail, std::integral_constant<int, STAGES - 2>{});
    }
    __syncthreads();  // every wavefront is done with the ring

    // KSPLIT == 2: the two wavefronts of a sub-tile swap halves of their sums through LDS (exact in any order) and each
    // finishes half of its rows
    v16i half_sum[KSPLIT == 2 ? ETM : 1][TN];
    if constexpr (KSPLIT == 2) {
        static_assert(NW * ETM * TN * 4096 <= STAGES * STAGE_BYTES, "exchange fits the ring");
        v4i* const mine = reinterpret_cast<v4i*>(smem) + (wave_t * 2 + kg) * (ETM * TN * 256) + lane;
        const v4i* const other = reinterpret_cast<const v4i*>(smem) + (wave_t * 2 + 1 - kg) * (ETM * TN * 256) + lane;
#pragma unroll
        for (int i = 0; i < ETM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {   // give away the row blocks the partner finishes
                    v4i o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = kg == 0 ? acc[ETM + i][j][4 * v + e] : acc[i][j][4 * v + e];
                    mine[((i * TN + j) * 4 + v) * 64] = o;
                }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ETM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const v4i o = other[((i * TN + j) * 4 + v) * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) half_sum[i][j][4 * v + e] = (kg == 0 ? acc[i][j][4 * v + e] : acc[ETM + i][j][4 * v + e]) + o[e];
                }
        __syncthreads();
    }
    auto sum = [&](int i, int j) -> v16i& {
        if constexpr (KSPLIT == 2) return half_sum[i][j];
        else return acc[i][j];
    };
    const int erow = wave_m + kg * EM;   // first row of the tile that this wavefront finishes

#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        const int c = tid + t * 64 * NW;
        if (c < BN) s_bias[c] = bias_reg[t];
        if (kRelu && c < BN) s_scale[c] = scale_reg[t];
    }
    if constexpr (kSlots) {
        write_slots(reinterpret_cast<float2*>(smem), kb_reg[0], tid);
    } else if constexpr (kTable) {
#pragma unroll
        for (int t = 0; t < KPT; ++t)
            if (tid + t * 64 * NW < p.table.nseg) s_kb[tid + t * 64 * NW] = kb_reg[t];
        for (int e = tid + KPT * 64 * NW; e < p.table.nseg; e += 64 * NW) s_kb[e] = p.table.kb[e];
    }
    if constexpr (kEpi == EPI_ATTENTION) attn_tabs.write(p.at, reinterpret_cast<float2*>(smem), reinterpret_cast<float2*>(smem + kSlotBytes));
    constexpr int RW = BN + 16;  // row stride of the residual image
    int8_t* s_res = smem;        // in the ring, which is free now
    if (kResid) {
#pragma unroll
        for (int t = 0; t < RPT; ++t) {
            const int c = tid + t * 64 * NW, row = c / CPRW, cc = c % CPRW;
            if (c < BM * CPRW) *reinterpret_cast<v4i*>(s_res + row * RW + 16 * cc) = res_reg[t];
        }
    }
    __syncthreads();

    // ---- epilogue -----------------------------------------------------------------------------
    // uniform factors in vector registers: with a scalar operand an instruction issues at half the rate
    const float alpha = in_vgpr(p.alpha);
    const bool full = m0 + BM <= p.M && n0 + BN <= p.N;
    v4f bi[TN][4];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) bi[j][g] = *reinterpret_cast<const v4f*>(s_bias + wave_n + 32 * j + 8 * g + 4 * frag_half);
    constexpr int NG = ETM * TN * 4;  // groups of four columns per lane
    if constexpr (kTable || kEpi == EPI_Q) {
        constexpr int SW = WN + 16;
        constexpr int kAt = kSlots ? (int)kSlotBytes : 0;
        static_assert(kAt + NW * EM * SW <= STAGES * STAGE_BYTES, "patch fits the ring");
        int8_t* patch = smem + kAt + wave * (EM * SW);
        // inverse output scale of a group (the QKV projection has one per column third)
        const float inv_all = in_vgpr(p.out_inv_scale);
        float inv_g[TN][4];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + wave_n + 32 * j + 8 * g + 4 * frag_half;
                inv_g[j][g] = p.split_cols > 0 ? (n >= 2 * p.split_cols ? p.inv3[2] : n >= p.split_cols ? p.inv3[1] : p.inv3[0])
                                               : inv_all;
            }
        constexpr int DEPTH = 3;
        float x[DEPTH + 1][4];
        float2 kb[DEPTH + 1][4];
        // group index -> (i, j, g), i innermost: consecutive groups use different accumulators
        // kPow2: the segment's position by one fma (the same bits: DevTable) instead of two steps.  In slots (nm_device.h): of an element's
        // eleven instructions nine issued at half the rate (scalar operands, clamp, conversions, shift), now two and a half of ten.  us,
        // before -> after: 4096 x 3072 x 768 16.3 -> 16.1, 8192 x 3072 x 768 29.3 -> 28.9, 16384 x 4096 x 1024 85.8 -> 85.0, with 100 segments
        // 87.4 -> 85.0 (the card's power limits that one); a base stack over 16 x 512 tokens 0.4 % less, a large one over 32 x 512 1 %.
        auto finish = [&](auto pow2_c) {
        constexpr bool kPow2 = decltype(pow2_c)::value;
        constexpr float kPart = kSlots ? 1.0f / kSlotSegments : 1.0f;
        const float tlo = in_vgpr(p.table.lo), tiw = in_vgpr(p.table.inv_w * kPart), tu0 = in_vgpr(p.table.u0 * kPart);
        const float steps = in_vgpr(8.0f * kSlotSegments), tmax = (float)(p.table.nseg - 1);
        auto stage_a = [&](int G) {
            const int i = G % ETM, jg = G / ETM, j = jg / 4, g = jg % 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = __builtin_fmaf((float)sum(i, j)[4 * g + e], alpha, bi[j][g][e]);
                x[G % (DEPTH + 1)][e] = v;
                if (!kTable) continue;
                if (kSlots) {
                    const float u = kPow2 ? fma_clamp01(v, tiw, tu0) : mul_clamp01(v - tlo, tiw);
                    kb[G % (DEPTH + 1)][e] = slot_line(slot_offset(u, steps));
                } else {  // clamp in float, floor
                    const float u = __builtin_amdgcn_fmed3f(kPow2 ? __builtin_fmaf(v, tiw, tu0) : (v - tlo) * tiw, 0.0f, tmax);
                    kb[G % (DEPTH + 1)][e] = s_kb[(int)u];
                }
            }
        };
        auto stage_b = [&](int G) {
            const int i = G % ETM, jg = G / ETM, j = jg / 4, g = jg % 4;
            int q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = x[G % (DEPTH + 1)][e];
                if (kTable) v = __builtin_fmaf(kb[G % (DEPTH + 1)][e].x, v, kb[G % (DEPTH + 1)][e].y);
                q[e] = requant(v, inv_g[j][g]);
            }
            *reinterpret_cast<unsigned*>(patch + (32 * i + frag_row) * SW + 32 * j + 8 * g + 4 * frag_half) =
                pack4(q[0], q[1], q[2], q[3]);
        };
#pragma unroll
        for (int G = 0; G < NG + DEPTH; ++G) {
            if (G < NG) stage_a(G);
            __builtin_amdgcn_sched_barrier(0);
            if (G >= DEPTH) stage_b(G - DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
        };
        if (kTable && (kSlots ? p.table.slots == SLOTS_POW2 : p.table.pow2)) finish(std::true_type{}); else finish(std::false_type{});
        // the wavefront reads back the rows it wrote: order its LDS writes before its reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        constexpr int PCPR = WN / 16;
        constexpr int NCH = EM * PCPR / 64;  // 16-byte chunks per lane
        static_assert(EM * PCPR % 64 == 0, "chunks split evenly");
        v4i rows[NCH];
#pragma unroll
        for (int t = 0; t < NCH; ++t) {
            const int c = lane + 64 * t, row = c / PCPR, cc = c % PCPR;
            rows[t] = *reinterpret_cast<const v4i*>(patch + row * SW + 16 * cc);
        }
#pragma unroll
        for (int t = 0; t < NCH; ++t) {
            const int c = lane + 64 * t, row = c / PCPR, cc = c % PCPR;
            const int mr = m0 + erow + row, n = n0 + wave_n + 16 * cc;
            if (full || (mr < p.M && n < p.N)) *reinterpret_cast<v4i*>(p.out_q + (long)mr * p.ldo + n) = rows[t];
        }
    } else if constexpr (kEpi == EPI_ATTENTION) {
        // The codes become the images that attention reads (nm_attention.h; Q's is K's), then every wavefront takes 16 queries, or twice.
        static_assert(TN == 3 && NW * ETM == 8, "wavefront tiles of 64 x 96");
        int8_t* const images = smem + kSlotBytes + kQkvRecip * 8;
        const float2* const s_recip = reinterpret_cast<const float2*>(smem + kSlotBytes);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int t = wave_n / 32 + j, third = t >> 1;   // block of 32 columns
            const float inv = in_vgpr(third == 0 ? p.inv3[0] : third == 1 ? p.inv3[1] : p.inv3[2]);
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int i = 0; i < ETM; ++i) {
                    int q[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) q[e] = requant(__builtin_fmaf((float)sum(i, j)[4 * g + e], alpha, bi[j][g][e]), inv);
                    const int row = erow + 32 * i + frag_row, chunk = 2 * (t & 1) + (g >> 1);
                    const int turn = ((row >> 2) & 3) ^ (third == 2 ? (row >> 4) & 3 : 0);
                    *reinterpret_cast<unsigned*>(images + third * (BM * 64) + row * 64 + ((chunk ^ turn) << 4) + 8 * (g & 1) + 4 * frag_half) =
                        pack4(q[0], q[1], q[2], q[3]);
                }
        }
        __syncthreads();
        auto attend = [&](auto ng_c, auto full_c, auto mode_c) {
            constexpr int NG = decltype(ng_c)::value, kMode = decltype(mode_c)::value;
            const AttnConsts<kMode> consts(p.at);
#pragma unroll 1
            for (int t = 0; t < 8 / NW; ++t) {
                const int row0 = 16 * (8 / NW * wave + t), first = row0 & ~(64 * NG - 1), q0 = row0 - first;   // first row of the sequence
                const int seq = (tile_m << (NG == 1 ? 1 : 0)) + (NG == 1 ? row0 >> 6 : 0);
                if (seq >= p.B || q0 >= p.at.S) continue;
                const v4i qf = *reinterpret_cast<const v4i*>(images + attn_koff(row0 + (lane & 15), lane >> 4));
                attn_queries<1, NG, decltype(full_c)::value, kMode, true>(p.at, consts, qf, nullptr, images + BM * 64 + first * 64, images + 2 * BM * 64 + first * 64,
                                                                         images + 3 * BM * 64, smem, s_recip, lane, wave, p.at.S, 0, seq, tile_n, q0);
            }
        };
        auto by_mode = [&](auto ng_c, auto full_c) {
            if (p.pow2) attend(ng_c, full_c, std::integral_constant<int, EXP_SLOTS_POW2>{});
            else attend(ng_c, full_c, std::integral_constant<int, EXP_SLOTS>{});
        };
        if (p.keys_log2 == 6) {
            if (p.at.S == 64) by_mode(std::integral_constant<int, 1>{}, std::true_type{});
            else by_mode(std::integral_constant<int, 1>{}, std::false_type{});
        } else {
            if (p.at.S == 128) by_mode(std::integral_constant<int, 2>{}, std::true_type{});
            else by_mode(std::integral_constant<int, 2>{}, std::false_type{});
        }
    } else if constexpr (kRelu) {
        // Codes go to an image of the tile's rows (over the residual's, word by word, where there is one) and leave as
        // 16-byte stores.  Where the table is a ReLU and the columns' numbers cannot make a sum infinite, clamping the
        // code at 0 is all of it; any other table of two segments is a compare.
        constexpr int SW = kResid ? RW : WN + 16;
        int8_t* patch = kResid ? s_res + erow * RW + wave_n : smem + wave * (EM * SW);
        const float rs = p.resid_scale, inv = p.out_inv_scale;
        const bool plain = !p.has_table;
        bool relu = p.relu;
        if (relu) {
            for (int c = lane; c < WN; c += 64) relu = relu && relu_finite(s_scale[wave_n + c], s_bias[wave_n + c]);
            relu = __all(relu);
        }
        auto finish = [&](auto clamp_c, auto table_c) {
            constexpr bool kClamp = decltype(clamp_c)::value, kLines = decltype(table_c)::value;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int cl = 32 * j + 8 * g + 4 * frag_half;
                    const v4f sc = *reinterpret_cast<const v4f*>(s_scale + wave_n + cl);
                    unsigned rw[ETM];
                    if (kResid) {
#pragma unroll
                        for (int i = 0; i < ETM; ++i) rw[i] = *reinterpret_cast<const unsigned*>(patch + (32 * i + frag_row) * SW + cl);
                    }
#pragma unroll
                    for (int i = 0; i < ETM; ++i) {
                        unsigned w = 0;
                        int q[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float v = __builtin_fmaf((float)sum(i, j)[4 * g + e], sc[e], bi[j][g][e]);
                            if (kResid) v = __builtin_fmaf((float)(int)(int8_t)(rw[i] >> (8 * e)), rs, v);
                            if (kClamp) w = relu_requant(v, inv, e, w);
                            else q[e] = requant(kLines ? pwl_eval_two_segments(v, p.table) : v, inv);
                        }
                        if (!kClamp) w = pack4(q[0], q[1], q[2], q[3]);
                        *reinterpret_cast<unsigned*>(patch + (32 * i + frag_row) * SW + cl) = w;
                    }
                }
        };
        if (relu) finish(std::true_type{}, std::false_type{});
        else if (plain) finish(std::false_type{}, std::false_type{});
        else finish(std::false_type{}, std::true_type{});
        // the wavefront reads back the rows it wrote
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        constexpr int PCPR = WN / 16, NCH = EM * PCPR / 64;
        static_assert(EM * PCPR % 64 == 0, "chunks split evenly");
#pragma unroll
        for (int t = 0; t < NCH; ++t) {
            const int c = lane + 64 * t, row = c / PCPR, cc = c % PCPR;
            const v4i o = *reinterpret_cast<const v4i*>(patch + row * SW + 16 * cc);
            const int mr = m0 + erow + row, n = n0 + wave_n + 16 * cc;
            if (full || (mr < p.M && n < p.N)) *reinterpret_cast<v4i*>(p.out_q + (long)mr * p.ldo + n) = o;
        }
    } else if constexpr (kEpi == EPI_F32_RESID) {
        // Rows leave through an LDS patch of 32 rows per wavefront, 16 or 24 lanes per row.  Stored straight
        // from the accumulators (32 bytes of each of 32 rows per instruction) the 64 MB of a 16384 x 1024
        // result took 15 us behind the matrix work (kernel with K = 1024: 36 us); whole lines take 10 (30).
        constexpr int PW = WN + 4, LPR = WN / 4, NST = 32 * LPR / 64;
        static_assert(32 * LPR % 64 == 0, "pieces split evenly");
        float* patch = reinterpret_cast<float*>(smem + BM * RW) + wave * 32 * PW;
        const float rs = in_vgpr(p.resid_scale);
#pragma unroll
        for (int i = 0; i < ETM; ++i) {
#pragma unroll
            for (int jg = 0; jg < 4 * TN; ++jg) {
                const int j = jg / 4, g = jg % 4;
                const int cl = 32 * j + 8 * g + 4 * frag_half;
                const unsigned rw = *reinterpret_cast<const unsigned*>(s_res + (erow + 32 * i + frag_row) * RW + wave_n + cl);
                v4f y;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = __builtin_fmaf((float)sum(i, j)[4 * g + e], alpha, bi[j][g][e]);
                    y[e] = __builtin_fmaf((float)(int)(int8_t)(rw >> (8 * e)), rs, v);
                }
                *reinterpret_cast<v4f*>(patch + frag_row * PW + cl) = y;
            }
            // the wavefront reads back the rows it wrote, and writes the next ones after that
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int t = 0; t < NST; ++t) {
                const int c = lane + 64 * t, row = c / LPR, cc = c % LPR;
                const v4f y = *reinterpret_cast<const v4f*>(patch + row * PW + 4 * cc);
                const int m = m0 + erow + 32 * i + row, n = n0 + wave_n + 4 * cc;
                if (full || (m < p.M && n < p.N)) *reinterpret_cast<v4f*>(p.out_f32 + (long)m * p.ldo + n) = y;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    } else {
        // ---- fp32 result + residual, then LayerNorm-PWL over the row (the tile covers whole rows:
        // BN == N, n0 == 0, and every wavefront holds all BM rows of its WN columns).  Row sums keep
        // the normative order: column group G (four consecutive columns) belongs to accumulator
        // G % 64, an accumulator adds its groups in increasing G and each group's elements in
        // increasing column, starting from +0; the 64 accumulators of a row are then combined by the
        // butterfly 32, 16, 8, 4, 2, 1.  Groups 64 apart live in different wavefronts, so the
        // accumulators pass through LDS: round s adds the groups G with G / 64 == s.
        static_assert(BM <= 64 && BN % 256 == 0 && WN % 4 == 0, "row block shape");
        constexpr int NS = (BN / 4 + 63) / 64;         // rounds
        float* s_part = reinterpret_cast<float*>(smem + BM * RW);  // [BM][64] accumulators, behind the residual image
        float* s_stat = s_part + BM * 64;                           // [BM] mean, then [BM] scale
        static_assert(BM * RW + (BM * 64 + 2 * BM) * 4 <= STAGES * STAGE_BYTES, "statistics fit the ring");
        const float rs = p.resid_scale;
        const float inv_L = (float)(1.0 / (double)BN);
        // the fp32 values of the lane (they replace the accumulators)
        float xv[TM][TN][16];
#pragma unroll
        for (int G = 0; G < NG; ++G) {
            const int i = G % TM, jg = G / TM, j = jg / 4, g = jg % 4;
            const int row = 32 * i + frag_row, cl = wave_n + 32 * j + 8 * g + 4 * frag_half;
            const unsigned rw = *reinterpret_cast<const unsigned*>(s_res + row * RW + cl);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = __builtin_fmaf((float)acc[i][j][4 * g + e], alpha, bi[j][g][e]);
                xv[i][j][4 * g + e] = __builtin_fmaf((float)(int)(int8_t)(rw >> (8 * e)), rs, v);
            }
        }
        // one pass over the row: SQ == false sums x, SQ == true sums fma(d, d, .)
        auto row_pass = [&](auto sq_c) {
            constexpr bool SQ = decltype(sq_c)::value;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int G = (wave_n + 32 * j + 8 * g + 4 * frag_half) >> 2;  // column group in the row
                        if ((G >> 6) != s) continue;                                 // wave-uniform (G and G ^ 1 share a round)
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            float* slot = s_part + (32 * i + frag_row) * 64 + (G & 63);
                            float a = s == 0 ? 0.0f : *slot;
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                a = SQ ? __builtin_fmaf(xv[i][j][4 * g + e], xv[i][j][4 * g + e], a) : a + xv[i][j][4 * g + e];
                            *slot = a;
                        }
                    }
                __syncthreads();
            }
            // butterfly over the 64 accumulators of each row: lane = accumulator
            for (int row = wave; row < BM; row += NW) {
                float v = s_part[row * 64 + lane];
#pragma unroll
                for (int mask = 32; mask >= 1; mask >>= 1) v = v + __shfl_xor(v, mask, 64);
                if (lane == 0) s_stat[row] = v * inv_L;
            }
            __syncthreads();
        };
        row_pass(std::false_type{});
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const float mu = s_stat[32 * i + frag_row];
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) xv[i][j][v] = xv[i][j][v] - mu;
        }
        __syncthreads();  // every lane has read its means before the variances overwrite them
        row_pass(std::true_type{});
        // scale of a row: r = PWL_rsqrt(var + eps), one look-up per row
        if (tid < BM) {
            int sr;
            const float u = s_stat[tid] + p.ln_eps;
            s_stat[BM + tid] = pwl_eval(u, p.ln_table, p.ln_table.kb, sr);
        }
        __syncthreads();
        // y = fma(d * r, gamma, beta); int8 rows leave through an LDS image as 16-byte stores
        int8_t* s_out = smem;  // [BM][RW], over the residual image (its last reader was the first loop above)
        const float inv = p.ln_inv_scale;
#pragma unroll
        for (int G = 0; G < NG; ++G) {
            const int i = G % TM, jg = G / TM, j = jg / 4, g = jg % 4;
            const int row = 32 * i + frag_row, cl = wave_n + 32 * j + 8 * g + 4 * frag_half;
            const float r = s_stat[BM + row];
            const v4f ga = *reinterpret_cast<const v4f*>(p.ln_gamma + cl);
            const v4f be = *reinterpret_cast<const v4f*>(p.ln_beta + cl);
            v4f y;
            int q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                y[e] = __builtin_fmaf(xv[i][j][4 * g + e] * r, ga[e], be[e]);
                q[e] = requant(y[e], inv);
            }
            if (p.ln_out_q) *reinterpret_cast<unsigned*>(s_out + row * RW + cl) = pack4(q[0], q[1], q[2], q[3]);
            if (p.ln_out_f32 && m0 + row < p.M) *reinterpret_cast<v4f*>(p.ln_out_f32 + (long)(m0 + row) * BN + cl) = y;
        }
        if (p.ln_out_q) {
            __syncthreads();
            for (int c = tid; c < BM * CPRW; c += 64 * NW) {
                const int row = c / CPRW, cc = c % CPRW;
                if (m0 + row < p.M)
                    *reinterpret_cast<v4i*>(p.ln_out_q + (long)(m0 + row) * BN + 16 * cc) =
                        *reinterpret_cast<const v4i*>(s_out + row * RW + 16 * cc);
            }
        }
    }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int kEpi, int BK = 128, bool kConv = false, int KSPLIT = 1, bool kEnd = false, typename Params>
static int32_t launch_tile_epi(Params& p, size_t table_bytes, hipStream_t s)
{
    auto kern = gemm_tile_kernel<BM, BN, WAVES_M, WAVES_N, STAGES, kEpi, BK, kConv, KSPLIT, kEnd>;
    constexpr int NW = WAVES_M * WAVES_N * KSPLIT, NBLK = (BM + BN) * BK / 1024;
    constexpr int kRing = STAGES * ((NBLK + NW - 1) / NW * NW) * 1024;
    constexpr int kFront = tile_front_bytes(BM, BN, NW, BM / WAVES_M / KSPLIT, BN / WAVES_N, kEpi);
    static_assert(kFront % 16 == 0 && kFront + BN * 4 <= 160 * 1024 && kRing <= 160 * 1024, "LDS");
    const size_t epilogue = kFront + BN * sizeof(float) + table_bytes, shmem = epilogue > kRing ? epilogue : (size_t)kRing;   // (table_bytes: of EPI_Q_LONG's table)
    static std::once_flag once;  // one attribute call per instantiation
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(gemm_tile_kernel)");
    });
    if (once_rc) return once_rc;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    p.group_m = xcd_group_rows(p.tiles_m, p.tiles_n, BM, BN);
    p.div_group = fast_div(p.group_m * p.tiles_n);
    p.div_gm = fast_div(p.group_m);
    queue_kernel(kern, dim3((p.tiles_m * p.tiles_n + 7) / 8 * 8), dim3(64 * NW), shmem, s, p);
    return NM_OK;
}

// The epilogues a configuration is built for (kTileConfigs).
enum TileOutputs { OUT_ANY, OUT_INT8, OUT_F32 };
template <bool kEnd, bool kLong, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, TileOutputs kOut = OUT_ANY, int KSPLIT = 1>
static int32_t launch_tile(GemmParams& p, int epi, size_t table_bytes, hipStream_t s)
{
    if constexpr (kOut != OUT_F32 && kLong) {
        return launch_tile_epi<BM, BN, WAVES_M, WAVES_N, STAGES, EPI_Q_LONG, 128, false, KSPLIT, kEnd>(p, table_bytes, s);
    } else if constexpr (kOut != OUT_F32) {
        if (epi == EPI_Q) return launch_tile_epi<BM, BN, WAVES_M, WAVES_N, STAGES, EPI_Q, 128, false, KSPLIT, kEnd>(p, table_bytes, s);
        if (epi == EPI_Q_TABLE) return launch_tile_epi<BM, BN, WAVES_M, WAVES_N, STAGES, EPI_Q_TABLE, 128, false, KSPLIT, kEnd>(p, table_bytes, s);
    }
    if constexpr (kOut != OUT_INT8 && !kLong) {
        if (epi == EPI_F32_RESID) return launch_tile_epi<BM, BN, WAVES_M, WAVES_N, STAGES, EPI_F32_RESID, 128, false, KSPLIT, kEnd>(p, table_bytes, s);
    }
    return fail(NM_ERR_UNSUPPORTED, "gemm: tile configuration not built for this epilogue");
}
// Configuration cfg of kTileConfigs.  kLong: with EPI_Q_LONG, which the others are built without.
template <bool kEnd, bool kLong = false>
static int32_t launch_tile_config(int cfg, GemmParams& p, int epi, size_t table_bytes, hipStream_t s)
{
    switch (cfg) {
    case 0: return launch_tile<kEnd, kLong, 256, 256, 2, 4, 2>(p, epi, table_bytes, s);
    case 1: return launch_tile<kEnd, kLong, 256, 192, 4, 2, 2>(p, epi, table_bytes, s);
    case 2: return launch_tile<kEnd, kLong, 256, 128, 4, 2, 3>(p, epi, table_bytes, s);
    case 3: return launch_tile<kEnd, kLong, 128, 192, 2, 2, 3>(p, epi, table_bytes, s);
    case 4: return launch_tile<kEnd, kLong, 128, 192, 2, 2, 2>(p, epi, table_bytes, s);
    case 5: return launch_tile<kEnd, kLong, 128, 128, 2, 2, 3, OUT_INT8>(p, epi, table_bytes, s);
    case 6: return launch_tile<kEnd, kLong, 128, 128, 2, 2, 2>(p, epi, table_bytes, s);
    case 7: return launch_tile<kEnd, kLong, 64, 128, 2, 2, 3>(p, epi, table_bytes, s);
    case 8: return launch_tile<kEnd, kLong, 64, 128, 2, 2, 2>(p, epi, table_bytes, s);
    default: return launch_tile<kEnd, kLong, 128, 128, 2, 2, 3, OUT_F32, 2>(p, epi, table_bytes, s);
    }
}

// Convolutions, as products or with gathered rows.  us, streaming kernel -> this one with 128-byte slices: 12544 x 256 x 2304
// (3x3) 16.4 -> 12.0, 3136 x 512 x 4608 (3x3) 22.3 -> 14.2, 50176 x 128 x 1152 (3x3) 15.8 -> 11.9, 3136 x 2048 x 512 with
// residual 14.1 -> 8.4, 12544 x 256 x 1024 9.3 -> 6.9, 3136 x 2048 x 1024 (stride 2) 15.9 -> 11.1.
template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int BK = 128, int KSPLIT = 1>
static int32_t launch_tile_relu(GemmParams& p, bool conv, hipStream_t s)
{
    constexpr size_t cols = BN * sizeof(float);   // the scales, where other epilogues have their table
    if (conv) return launch_tile_epi<BM, BN, WAVES_M, WAVES_N, STAGES, EPI_Q_RELU, BK, true, KSPLIT>(p, cols, s);
    if (p.resid) return launch_tile_epi<BM, BN, WAVES_M, WAVES_N, STAGES, EPI_Q_RELU_RESID, BK, false, KSPLIT>(p, cols, s);
    return launch_tile_epi<BM, BN, WAVES_M, WAVES_N, STAGES, EPI_Q_RELU, BK, false, KSPLIT>(p, cols, s);
}

}  // namespace nm
