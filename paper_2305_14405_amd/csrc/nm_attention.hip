// Fused attention for gfx950: scores = Q K^T, softmax-PWL, context = P V in one kernel, per
// (batch, head, block of queries).  The int32 scores and the int8 probabilities never leave
// registers (they are written out only when the caller asks for them).
//
// Paper basis: Section 3.1 (attention is a linear operation mapped to matrix products) and
// Section 3.2 (exp and 1/x as PWL tables); the arithmetic is exactly that of the three separate
// entry points (nm_attn_scores, nm_softmax_pwl, nm_attn_context), including the normative order
// of the row sum, so the results are bit-identical to the unfused path.
//
// Layout: a wavefront owns 16 queries and uses the 16x16x64 integer MFMA (one instruction covers
// the whole head dimension).  K rows feed the row operand and Q rows the column operand, so lane
// (m, hq) (m = lane % 16 = query, hq = lane / 16) ends with the scores of query m for the keys
// 16*blk + 4*hq + e (blk = key block, e = 0..3): groups of four consecutive keys, which are the
// 4-element groups of the normative row sum (accumulator index (4*blk + hq) % 64).  The butterfly
// over accumulators is then: in-register adds over blk (masks 32, 16, 8, 4) and two cross-lane
// adds (lane ^ 32 for mask 2, lane ^ 16 for mask 1).
// The int8 probabilities are packed in place, four per register, and four such registers ARE the
// operand of the second product: the contraction index of an integer MFMA may be permuted freely
// as long as both operands use the same permutation.  V stays row-major in LDS ([key][64 bytes],
// copied like K); its operand fragments (one head column per lane, 16 keys) come out of the
// transposing LDS read of gfx950 (ds_read_b64_tr_b8: within 16 lanes, lane j receives byte j % 8
// of the eight rows addressed by lanes j / 8, j / 8 + 2, ...), with the row addresses chosen so
// that the keys arrive in the order the probabilities have in the lanes.
//
// What bounds it: vector instructions (by counter 14.1 per score at 32 x 512 tokens and 16 heads, 10.5 of them in the loops over
// the scores), the matrix instructions, which the SIMD issues in their stead (16 clocks each, an eighth of the time), and
// what is not hidden of loads and look-ups: without K's and V's loads the kernel takes 91 % of its time, without the
// look-ups 91 %, without V's reads 92 %.  The instructions beyond the loops' are paid once per 16 queries and up to 256
// keys: addresses, table staging, the exchange between wavefronts, the context's codes.  The loops' steps
// have the same values as the normative ones:
//  * the score accumulators start at the bits of the float 1.5 * 2^23, so an accumulator read as a float
//    is 1.5 * 2^23 + score exactly (|score| <= 2^20) and the difference of two is the exact difference
//    of the scores: no conversion; and their integer order is the order of the scores;
//  * the table lies in slots (nm_device.h) and everything uniform in vector registers, so that all steps but the maximum and the
//    final conversion are of the kind that issues at twice the rate;
//  * where inv_w is a power of two, (t - lo) * inv_w is one fma: scaling by it commutes with rounding;
//  * a row whose codes provably lie in [0, 127] (bounds of the exp table over every reachable t, times
//    the row's reciprocal: rounding is monotone) is requantised by v_cvt_pk_u8_f32, which rounds to
//    nearest even, saturates and packs; other rows take the clamping form.
#include <climits>
#include <cmath>
#include <mutex>

#include "nm_attention.h"

namespace nm {

// Workgroups are dealt to the eight XCDs round-robin.  Renumbered so that an XCD receives consecutive
// (head, query block) pairs: the query blocks of a head share its K and V, and neighbouring heads
// share 128-byte lines (a head's rows are 64-byte halves), so these fetches then meet in one L2
// instead of going to memory once per XCD.
__device__ __forceinline__ int attn_block_id(int total)
{
    return (int)(blockIdx.x & 7) * ((total + 7) >> 3) + (int)(blockIdx.x >> 3);
}

// A wavefront holds at most 256 keys of its 16 queries (64 score registers), so that four wavefronts fit
// a SIMD and one workgroup's K / V loads run under another's arithmetic.  Beyond 256 keys kParts = 2 or 4 wavefronts
// share 16 queries: part h takes every kParts-th 16-key block from block h on, i.e. (its bits 2, or 2 and 3, being h) whole
// accumulators of the row sum with all their elements, and the parts have equally many blocks, but for one, whatever S is.
// They exchange their row maxima, their sums at the butterfly's steps with masks 8 and 4, and their partial contexts
// (exact integers, each part finishing its share of the head's columns) through the K image, which is free by then.
// NG: groups of four such blocks per part.  kFull: S == 64 * kParts * NG and head size 64, so that nothing is masked or clamped.
// kHead64: head size 64 (else 16, 32 or 48: Q is zero in the chunks beyond the head's, and the column blocks beyond it are left out).
// us per launch, one behind the other, before -> after the division by blocks, the slots and the look-ups requested ahead, 12 heads
// of 64: 16 x 512 tokens 28.8 -> 26.6 (16 heads, 32 x 512: 69 -> 64), 16 x 384 20.6 -> 18.4, 8 x 300 8.7 -> 8.9, 16 x 256 8.8 ->
// 8.5, 32 x 128 6.2 -> 6.0, 11 x 77 4.6 -> 4.3, 4 x 640 20.7 -> 16.9, 8 x 1024 81 -> 54.
template <int kParts, int NG, bool kFull, int kMode, bool kHead64>
__global__ __launch_bounds__(256 * kParts) __attribute__((amdgpu_waves_per_eu(4))) void attention_pwl_kernel(AttnParams p)
{
    static_assert(!kFull || kHead64, "nothing clamped");
    constexpr int kWaves = 4 * kParts, kAttnThreads = 64 * kWaves;
    constexpr int kQueries = 64;              // queries per workgroup
    constexpr int SK = 64 * kParts * NG;      // padded key count
    // With up to 1024 keys one workgroup fills a CU: V is requested behind K and arrives under the scores and the softmax.
    constexpr bool kLateV = kParts >= 2;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    // tables (the exp table's at 0, so that a slot's offset is its address), then K and V images, context patches
    int8_t* const s_tile = smem + p.off_tile;
    int8_t* sK = s_tile;
    int8_t* sV = s_tile + SK * 64;
    int8_t* sO = s_tile + 2 * SK * 64;
    // the kernel arguments everything in front of the loads needs, in one step
    asm volatile("" : : "s"(p.qkv), "s"(p.S), "s"(p.H), "s"(p.heads), "s"(p.qblocks), "s"(p.total), "s"(p.t_exp.kb), "s"(p.t_recip.kb),
                 "s"(p.t_exp.nseg), "s"(p.t_recip.nseg), "s"(p.div_qblocks.magic), "s"(p.div_qblocks.shift), "s"(p.div_heads.magic),
                 "s"(p.div_heads.shift), "s"(p.alpha_scores), "s"(p.inv_s_p), "s"(p.alpha_ctx), "s"(p.inv_s_ctx), "s"(p.t_exp.lo),
                 "s"(p.t_exp.inv_w), "s"(p.t_exp.u0), "s"(p.t_recip.lo), "s"(p.t_recip.hi), "s"(p.t_recip.inv_w),
                 "s"(p.t_recip.clamp_input), "s"(p.e_lo), "s"(p.e_hi), "s"(p.ctx), "s"(p.ctx_vec16), "s"(p.nch), "s"(p.off_tile));
    if (kMode == EXP_ANY) asm volatile("" : : "s"(p.scores_out), "s"(p.p_out), "s"(p.t_exp.hi), "s"(p.t_exp.clamp_input));
    float2* s_kb_recip = reinterpret_cast<float2*>(smem + attn_exp_bytes(kMode, p.t_exp.nseg));

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, hq = lane >> 4;
    const int id = attn_block_id(p.total);
    if (id >= p.total) return;
    const int by = (int)quotient((unsigned)id, p.div_qblocks), bx = id - by * p.qblocks;
    const int b = (int)quotient((unsigned)by, p.div_heads), head = by - b * p.heads;
    const int S = kFull ? SK : p.S, H = p.H, nch = kHead64 ? 4 : p.nch;
    const int ld = 3 * H;
    const int8_t* base = p.qkv + (long)b * S * ld + head * (16 * nch);

    AttnTables<kMode, kAttnThreads> tabs;
    tabs.request(p);
    // K and V -> LDS, row-major, by direct global -> LDS loads (16 rows of 64 bytes per wavefront
    // instruction; the chunk rotation is applied to the source address).  Rows past S repeat the last
    // one: their keys are masked.  Chunks beyond the head's meet zeros of Q and unused columns: any valid address will do.
    const auto load = [&](int third, const int8_t* image, int rotation) {
        const unsigned lds = (unsigned)(uintptr_t)image;
        const int c = (lane & 3) ^ hq ^ rotation, row = lane >> 2;
        const int at = third * H + 16 * (kHead64 || c < nch ? c : 0), voff = row * ld + at;
        const int nb16 = kFull ? SK / 16 : (S + 15) >> 4;
        for (int blk16 = wave; blk16 < nb16; blk16 += kWaves) {
            int v = voff;
            if (!kFull && 16 * blk16 + 16 > S) v = min(row, S - 1 - 16 * blk16) * ld + at;
            dma16s(base + (long)(16 * blk16 * ld), (unsigned)v, lds + 1024 * blk16);
        }
    };
    const int v_rotation = (wave / kParts) & 3;   // (a wavefront's blocks are kWaves apart)
    load(1, sK, 0);
    if (!kLateV) load(2, sV, v_rotation);
    // this lane's query row, straight from global memory into the MFMA operand registers
    const int q0 = bx * kQueries + wave / kParts * 16, m = q0 + fr;
    v4i qf = {0, 0, 0, 0};
    if (kHead64 || hq < nch) qf = *reinterpret_cast<const v4i*>(base + (long)(kFull ? m : min(m, S - 1)) * ld + 16 * hq);
    tabs.write(p, reinterpret_cast<float2*>(smem), s_kb_recip);
    const AttnConsts<kMode> consts(p);
    wait_vmcnt<0>();   // this wavefront's loads have landed (the barrier covers the others')
    __syncthreads();
    if (!kFull && kParts == 1 && q0 >= S) return;
    if (kLateV) {
        asm volatile("" : : "v"(qf));   // (the compiler's wait for Q, which would count the loads of V)
        load(2, sV, v_rotation);
    }

    attn_queries<kParts, NG, kFull, kMode, kHead64>(p, consts, qf, s_tile, sK, sV, sO, smem, s_kb_recip, lane, wave, S, by, b, head, q0);
}

// Sequences beyond 1024 keys: the scores are computed three times, for the row maximum, for the sum and for the
// probabilities (matrix work is cheap, and no score or probability goes to memory).  K, and V in the last pass, come
// through LDS in chunks of 256 keys, the next chunk loading while one is used.  A workgroup is four wavefronts of 16
// queries.  Up to 1024 keys the kernel above is the faster one: 4 x 520 tokens, 12 heads of 64, 17.8 us here, 15.1 there; 2 x
// 1000, 8 heads, 23.6 and 10.8; and heads of 32 at any length: 32 x 128 tokens, 8 heads, 6.5 and 4.9.
constexpr int kLongThreads = 256, kLongKeys = 256;
constexpr size_t kLongLds = 4 * (size_t)kLongKeys * 64 + (kLongThreads / 64) * (size_t)kCtxPatch;

template <int kMode>
__global__ __launch_bounds__(kLongThreads) __attribute__((amdgpu_waves_per_eu(2))) void attention_long_kernel(AttnParams p)
{
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];   // tables, K, K, V, V chunks of 16 KB, context patches
    int8_t* const s_tile = smem + p.off_tile;
    int8_t* sO = s_tile + 4 * kLongKeys * 64;
    asm volatile("" : : "s"(p.qkv), "s"(p.S), "s"(p.H), "s"(p.heads), "s"(p.qblocks), "s"(p.total), "s"(p.t_exp.kb), "s"(p.t_recip.kb),
                 "s"(p.t_exp.nseg), "s"(p.t_recip.nseg), "s"(p.nch), "s"(p.scores_out), "s"(p.p_out), "s"(p.div_qblocks.magic),
                 "s"(p.div_qblocks.shift), "s"(p.div_heads.magic), "s"(p.div_heads.shift), "s"(p.off_tile));
    float2* s_kb_recip = reinterpret_cast<float2*>(smem + attn_exp_bytes(kMode, p.t_exp.nseg));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, hq = lane >> 4;
    const int id = attn_block_id(p.total);
    if (id >= p.total) return;
    const int by = (int)quotient((unsigned)id, p.div_qblocks), bx = id - by * p.qblocks;
    const int b = (int)quotient((unsigned)by, p.div_heads), head = by - b * p.heads;
    const int S = p.S, H = p.H, ld = 3 * H, nch = p.nch;
    const int8_t* base = p.qkv + (long)b * S * ld + head * (16 * nch);

    AttnTables<kMode, kLongThreads> tabs;
    tabs.request(p);
    const int nchunks = (S + kLongKeys - 1) / kLongKeys, steps = 3 * nchunks;
    const unsigned lds0 = (unsigned)(uintptr_t)s_tile;
    // chunks of a row beyond the head's are never used (Q is zero there): any valid address will do
    auto chunk_at = [&](int c) { return 16 * (c < nch ? c : 0); };
    auto issue = [&](int pass, int c, int buf) {
        const int nb16 = min(16, (S - kLongKeys * c + 15) >> 4);
        for (int blk = wave; blk < nb16; blk += kLongThreads / 64) {
            const int r = min(kLongKeys * c + 16 * blk + (lane >> 2), S - 1);
            const unsigned at = (unsigned)(r * ld + H);
            dma16s(base, at + chunk_at((lane & 3) ^ hq), lds0 + buf * 16384 + 1024 * blk);
            if (pass == 2) dma16s(base, at + H + chunk_at((lane & 3) ^ hq ^ (blk & 3)), lds0 + 32768 + buf * 16384 + 1024 * blk);
        }
    };
    issue(0, 0, 0);
    const int q0 = bx * (kLongThreads / 4) + wave * 16, m = q0 + fr;
    v4i qf = {0, 0, 0, 0};
    if (hq < nch) qf = *reinterpret_cast<const v4i*>(base + (long)min(m, S - 1) * ld + 16 * hq);
    tabs.write(p, reinterpret_cast<float2*>(smem), s_kb_recip);
    const AttnConsts<kMode> consts(p);

    const bool ragged = (S & 63) != 0, vec4 = (S & 3) == 0;
    const long row_ss = ((long)by * S + m) * S;
    const VFragments<1> vfrag(lane);
    int mi = INT_MIN;
    float part[16], fm = 0.0f, r = 0.0f;
    v4i a2[4];
#pragma unroll
    for (int q = 0; q < 16; ++q) part[q] = 0.0f;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) a2[cb] = v4i{0, 0, 0, 0};

    int step = 0;
    auto run_pass = [&](auto pass_c, auto small_c) {
        constexpr int kPass = decltype(pass_c)::value;
        constexpr bool kSmall = decltype(small_c)::value;
        for (int c = 0; c < nchunks; ++c, ++step) {
            wait_vmcnt<0>();
            __syncthreads();   // chunk of this step has landed; everybody is done with the other buffer
            if (step + 1 < steps) {
                const bool wrap = c + 1 == nchunks;
                issue(wrap ? kPass + 1 : kPass, wrap ? 0 : c + 1, (step + 1) & 1);
            }
            const int8_t* sK = s_tile + (step & 1) * 16384;
            const int8_t* sV = s_tile + 32768 + (step & 1) * 16384;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int k0 = kLongKeys * c + 64 * g;   // first key of the group
                if (k0 >= S) break;
                v4i acc[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4i kf = *reinterpret_cast<const v4i*>(&sK[attn_koff(64 * g + 16 * q + fr, hq)]);
                    acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf, qf, v4i{kScoreBias, kScoreBias, kScoreBias, kScoreBias}, 0, 0, 0);
                }
                auto body = [&](auto mask_c) {
                    constexpr bool kMask = decltype(mask_c)::value;
                    const auto key_ok = [&](int q, int e) { return !kMask || k0 + 16 * q + 4 * hq + e < S; };
                    if (kPass == 0) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (key_ok(q, e)) mi = max(mi, acc[q][e]);
                        return;
                    }
                    // eight look-ups at a time: left alone, the compiler takes them one by one or in batches as it happens
                    // to number the registers (4 x 640 tokens 24.2 us and 22.0)
                    v4i pf;
                    float x[4][4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        // (a score of a row that was not loaded may be above the maximum, and its index beyond the padded table)
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[q][e] = attn_exp<kMode>(attn_padded(kMode) && kMask && !key_ok(q, e) ? INT_MIN : acc[q][e], fm, p, consts, smem);
                        if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (kMask && !key_ok(q, e)) x[q][e] = 0.0f;
                        if (kPass == 1) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) part[4 * g + q] = part[4 * g + q] + x[q][e];
                        } else {
                            pf[q] = (int)attn_pack(x[q], r, consts.inv_p, kSmall);
                            // (0 also where r or inv_s_p is not finite: see attention_pwl_kernel)
                            if (kMask && !kSmall) pf[q] = (int)attn_keep((unsigned)pf[q], S - k0 - 16 * q - 4 * hq);
                        }
                    }
                    if (kPass != 2) return;
                    if (kMode == EXP_ANY && (p.scores_out || p.p_out) && m < S) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int key = k0 + 16 * q + 4 * hq;
                            if (p.scores_out) {
                                if (vec4 && key < S) *reinterpret_cast<v4i*>(p.scores_out + row_ss + key) = acc[q] - kScoreBias;
                                else
#pragma unroll
                                    for (int e = 0; e < 4; ++e)
                                        if (key + e < S) p.scores_out[row_ss + key + e] = acc[q][e] - kScoreBias;
                            }
                            if (p.p_out) {
                                if (vec4 && key < S) *reinterpret_cast<unsigned*>(p.p_out + row_ss + key) = (unsigned)pf[q];
                                else
#pragma unroll
                                    for (int e = 0; e < 4; ++e)
                                        if (key + e < S) p.p_out[row_ss + key + e] = (int8_t)((unsigned)pf[q] >> (8 * e));
                            }
                        }
                    }
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb)   // (column blocks beyond the head's are computed and never stored)
                        a2[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vfrag.read(sV + 4096 * g, cb), pf, a2[cb], 0, 0, 0);
                };
                if (ragged && k0 + 64 > S) body(std::true_type{}); else body(std::false_type{});
            }
        }
    };
    run_pass(std::integral_constant<int, 0>{}, std::false_type{});
    fm = __int_as_float(row_max(mi));
    run_pass(std::integral_constant<int, 1>{}, std::false_type{});
#pragma unroll
    for (int mask = 8; mask >= 1; mask >>= 1)
#pragma unroll
        for (int q = 0; q < mask; ++q) part[q] = part[q] + part[q + mask];
    int segr;
    r = pwl_eval(row_add(part[0]), p.t_recip, s_kb_recip, segr);
    // The two forms of the last pass are two copies of its barriers, so the choice is the workgroup's: a wavefront
    // whose rows would allow the packing conversion takes the clamping form beside one whose rows do not.  (The
    // patches are not in use yet, and the last pass begins with a barrier.)
    int* s_small = reinterpret_cast<int*>(sO);
    const bool wave_small = attn_small(r, p);
    if (lane == 0) s_small[wave] = wave_small;
    __syncthreads();
    const bool small = __all(s_small[lane & (kLongThreads / 64 - 1)]);
    if (small) run_pass(std::integral_constant<int, 2>{}, std::true_type{});
    else run_pass(std::integral_constant<int, 2>{}, std::false_type{});
    attn_store_ctx(p, a2, sO + wave * kCtxPatch, lane, (long)b * S, q0, head, nch);
}

template <typename Kern>
static int32_t launch_attn_kernel(Kern kern, std::once_flag& once, int32_t& once_rc, AttnParams& p, int threads, size_t shmem, hipStream_t st)
{
    std::call_once(once, [&] {   // one attribute call per instantiation
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(attention kernel)");
    });
    if (once_rc) return once_rc;
    p.div_qblocks = fast_div(p.qblocks);
    p.div_heads = fast_div(p.heads);
    queue_kernel(kern, dim3((p.total + 7) / 8 * 8), dim3(threads), shmem, st, p);
    return NM_OK;
}

template <int kParts, int NG, bool kFull, int kMode, bool kHead64>
static int32_t launch_short(AttnParams& p, size_t tables, hipStream_t st)
{
    static std::once_flag once;
    static int32_t once_rc = NM_OK;
    return launch_attn_kernel(attention_pwl_kernel<kParts, NG, kFull, kMode, kHead64>, once, once_rc, p, 256 * kParts,
                              attn_lds_bytes(kParts, NG) + tables, st);
}
template <int kMode>
static size_t table_bytes(AttnParams& p)
{
    const size_t tables = (attn_exp_bytes(kMode, p.t_exp.nseg) + sizeof(float2) * (size_t)p.t_recip.nseg + 255) & ~(size_t)255;
    p.off_tile = (int)tables;
    return tables;
}
template <int kMode>
static int32_t launch_long(AttnParams& p, hipStream_t st)
{
    static std::once_flag once;
    static int32_t once_rc = NM_OK;
    return launch_attn_kernel(attention_long_kernel<kMode>, once, once_rc, p, kLongThreads, kLongLds + table_bytes<kMode>(p), st);
}

template <int kParts, int NG, int kMode>
static int32_t launch_groups(AttnParams& p, size_t tables, hipStream_t st)
{
    if (p.nch != 4) return launch_short<kParts, NG, false, kMode, false>(p, tables, st);
    // (EXP_ANY too: masked stores of the optional outputs are four times as many; 32 x 128 tokens, 12 heads 20.5 us masked, 12.9, 16 x 256 39.5 and 20.7)
    if (p.S == 64 * kParts * NG) return launch_short<kParts, NG, true, kMode, true>(p, tables, st);
    return launch_short<kParts, NG, false, kMode, true>(p, tables, st);
}

// kLongMode: of the kernel for long sequences.
template <int kMode, int kLongMode = kMode>
static int32_t launch_mode(AttnParams& p, hipStream_t st)
{
    const size_t tables = table_bytes<kMode>(p);
    const int parts = attn_parts(p.S), ng = (p.S + 64 * parts - 1) / (64 * parts);
    if (p.S > 1024 || attn_lds_bytes(parts, ng) + tables > 160 * 1024) return launch_long<kLongMode>(p, st);
    if (parts == 1) {
        if (ng == 1) return launch_groups<1, 1, kMode>(p, tables, st);
        if (ng == 2) return launch_groups<1, 2, kMode>(p, tables, st);
        if (ng == 3) return launch_groups<1, 3, kMode>(p, tables, st);
        return launch_groups<1, 4, kMode>(p, tables, st);
    }
    if (parts == 2) return ng == 3 ? launch_groups<2, 3, kMode>(p, tables, st) : launch_groups<2, 4, kMode>(p, tables, st);
    return ng == 3 ? launch_groups<4, 3, kMode>(p, tables, st) : launch_groups<4, 4, kMode>(p, tables, st);
}

bool fused_attention_covers(int S, int H, int heads)
{
    const int d = H / heads;
    return d <= kHeadDim && d % 16 == 0 && S <= 4096;
}

int32_t attn_params(const AttnArgs& a, const char* what, AttnParams* out, AttnExp* e)
{
    AttnParams& p = *out;
    DevTable t_exp, t_recip;
    int32_t rc = get_dev_table(a.tables, a.exp_idx, &t_exp, what);
    if (rc) return rc;
    if ((rc = get_dev_table(a.tables, a.recip_idx, &t_recip, what))) return rc;
    auto pick = [](const DevTable& t) { return AttnTable{t.kb, t.lo, t.hi, t.inv_w, t.u0, t.nseg, t.clamp_input}; };
    p.t_exp = pick(t_exp);
    p.t_recip = pick(t_recip);
    p.qkv = a.qkv; p.S = a.S; p.H = a.H; p.heads = a.heads;
    p.nch = a.H / a.heads / 16;
    p.alpha_scores = a.alpha_scores; p.inv_s_p = a.inv_s_p; p.alpha_ctx = a.alpha_ctx; p.inv_s_ctx = a.inv_s_ctx;
    p.ctx = a.ctx; p.scores_out = a.scores_out; p.p_out = a.p_out;
    p.ctx_vec16 = aligned(a.ctx, 16) ? 1 : 0;
    // |score difference| <= 2 * 64 * 128^2
    const double reach = 2097152.0 * std::fabs((double)a.alpha_scores);
    double vmin, vmax;
    table_value_bounds(a.tables, a.exp_idx, a.alpha_scores >= 0 ? -reach : 0.0, a.alpha_scores >= 0 ? 0.0 : reach, &vmin, &vmax);
    p.e_lo = (float)vmin; p.e_hi = (float)vmax;
    // index of t = 0 by the kernels' own arithmetic
    const float from_lo = 0.0f - t_exp.lo, at_0 = from_lo * t_exp.inv_w;
    e->slots = a.alpha_scores >= 0.0f ? t_exp.slots : SLOTS_NONE;
    e->padded = a.alpha_scores >= 0.0f && !t_exp.clamp_input && at_0 < (float)(t_exp.nseg + 1);
    e->pow2 = t_exp.pow2;
    return NM_OK;
}

int32_t launch_attention(const AttnArgs& a, const char* what, hipStream_t st)
{
    AttnParams p{};
    AttnExp e;
    int32_t rc = attn_params(a, what, &p, &e);
    if (rc) return rc;
    static_assert(kLongThreads / 4 == 64, "queries per workgroup");
    p.qblocks = (p.S + 63) / 64;
    p.total = p.qblocks * a.B * a.heads;
    if (p.scores_out || p.p_out || (e.slots == SLOTS_NONE && !e.padded)) rc = launch_mode<EXP_ANY>(p, st);
    else if (e.slots == SLOTS_POW2) rc = launch_mode<EXP_SLOTS_POW2>(p, st);
    else if (e.slots == SLOTS_ANY) rc = launch_mode<EXP_SLOTS>(p, st);
    else rc = e.pow2 ? launch_mode<EXP_PADDED, EXP_PADDED_POW2>(p, st) : launch_mode<EXP_PADDED>(p, st);
    if (rc) return rc;
    return check_hip(hipGetLastError(), "attention launch");
}

}  // namespace nm

using namespace nm;

extern "C" int32_t nm_attention_pwl(const int8_t* qkv, int32_t B, int32_t S, int32_t H, int32_t heads,
                                    float alpha_scores, const nm_tables* tables, int32_t exp_idx,
                                    int32_t recip_idx, float inv_s_p, float alpha_ctx, float inv_s_ctx,
                                    int8_t* ctx, int32_t* scores_out, int8_t* p_out, void* stream)
{
    if (!qkv || !ctx) return fail(NM_ERR_INVALID_ARG, "nm_attention_pwl: NULL pointer");
    if (B < 1 || S < 1 || H < 1 || heads < 1) return fail(NM_ERR_INVALID_ARG, "nm_attention_pwl: dimensions must be >= 1");
    if (!(alpha_scores == alpha_scores) || __builtin_isinf(alpha_scores))
        return fail(NM_ERR_INVALID_ARG, "nm_attention_pwl: alpha_scores must be finite");
    if (H % heads != 0) return fail(NM_ERR_INVALID_ARG, "nm_attention_pwl: H %d not divisible by heads %d", H, heads);
    DevTable t;
    int32_t rc = get_dev_table(tables, exp_idx, &t, "nm_attention_pwl(exp)");
    if (rc) return rc;
    rc = get_dev_table(tables, recip_idx, &t, "nm_attention_pwl(recip)");
    if (rc) return rc;
    if (H / heads != kHeadDim) return fail(NM_ERR_UNSUPPORTED, "nm_attention_pwl: head size %d (only 64 is fused)", H / heads);
    if (S > 512) return fail(NM_ERR_UNSUPPORTED, "nm_attention_pwl: S %d > 512 (use the three separate calls)", S);
    if ((int64_t)B * heads > 65535) return fail(NM_ERR_UNSUPPORTED, "nm_attention_pwl: B * heads > 65535");
    if ((int64_t)B * S * 3 * H >= (1LL << 31)) return fail(NM_ERR_UNSUPPORTED, "nm_attention_pwl: B*S*3H >= 2^31");
    if (!aligned(qkv, 16) || H % 16 != 0 || !aligned(ctx, 4) || H % 4 != 0 || (scores_out && !aligned(scores_out, 16)) ||
        (p_out && !aligned(p_out, 4)))
        return fail(NM_ERR_UNSUPPORTED, "nm_attention_pwl: pointers / H not aligned for the fused kernel");
    return launch_attention({qkv, B, S, H, heads, alpha_scores, inv_s_p, alpha_ctx, inv_s_ctx, tables, exp_idx, recip_idx, ctx,
                             scores_out, p_out}, "nm_attention_pwl", (hipStream_t)stream);
}
