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
// What bounds it: vector instructions (matrix work is a tenth).  By counter 16.0 per score at 32 x 512 tokens and
// 16 heads, issued in 91 % of the cycles, and 18.5 at 32 x 128 and 12 heads (18.9 in 67 %, and 24.5, before the
// steps below).  Ten and a half of them, and the table's LDS read, are the loops over the scores (18 before); the
// rest is paid once per 16 queries and up to 256 keys: addresses of the loads and of the transposing reads,
// accumulator start values, table staging, the exchange between wavefronts, the context's codes.  The loops' steps
// have the same values as the normative ones:
//  * the score accumulators start at the bits of the float 1.5 * 2^23, so an accumulator read as a float
//    is 1.5 * 2^23 + score exactly (|score| <= 2^20) and the difference of two is the exact difference
//    of the scores: no conversion; and their integer order is the order of the scores;
//  * t = difference * alpha <= 0, so the segment index needs no upper clamp when the table is
//    extended by a copy of its last entry (the index of t = 0 is at most nseg), and the hardware's
//    unsigned conversion saturates below at 0;
//  * where inv_w is a power of two, (t - lo) * inv_w is one fma: scaling by it commutes with rounding;
//  * a row whose codes provably lie in [0, 127] (bounds of the exp table over every reachable t, times
//    the row's reciprocal: rounding is monotone) is requantised by v_cvt_pk_u8_f32, which rounds to
//    nearest even, saturates and packs; other rows take the clamping form.
#include <climits>
#include <cmath>
#include <mutex>

#include "nm_device.h"

namespace nm {

struct AttnTable {   // what the kernels use of a DevTable, under its names
    const float2* kb;
    float lo, hi, inv_w, u0;
    int nseg, clamp_input;
};

struct AttnParams {
    const int8_t* qkv;
    int8_t* ctx;
    int S, H, heads, qblocks, total;   // total: workgroups that have work
    int nch;                           // 16-byte chunks of a head's row (head size / 16)
    float alpha_scores, inv_s_p, alpha_ctx, inv_s_ctx;
    float e_lo, e_hi;                  // bounds of the exp table's value over every reachable input
    int ctx_vec16;                     // ctx is 16-byte aligned: context rows leave as 16-byte stores
    FastDiv div_qblocks, div_heads;
    AttnTable t_exp, t_recip;
    int32_t* scores_out;               // optional [B, heads, S, S]
    int8_t* p_out;                     // optional [B, heads, S, S]
};

// How the exp table's segment is found: any table and scale (this form also writes the optional
// outputs); a table whose index at t = 0 is at most nseg, with alpha >= 0 and no input clamp; the same
// with inv_w a power of two.
enum { EXP_ANY = 0, EXP_PADDED = 1, EXP_PADDED_POW2 = 2 };

// Wavefronts per workgroup of 64 queries: one per 16 queries, two beyond 256 keys.
constexpr int attn_waves(int nkb) { return nkb >= 8 ? 8 : 4; }
constexpr int kHeadDim = 64;
constexpr int kScoreBias = 0x4B400000;   // bits of 1.5 * 2^23: the accumulators' start value

// K image: 64-byte rows, the four 16-byte chunks of a row rotated by (row / 4) % 4 so that the 16
// lanes of an operand read (16 consecutive rows, one chunk) cover all banks.
__device__ __forceinline__ int attn_koff(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 2) & 3)) << 4); }
// V image: the same, with the rotation also depending on (row / 16) % 4, because one transposing
// read touches rows 16 apart.

constexpr int kCtxPatch = 16 * 80;   // per wavefront: 16 context rows of 64 bytes, 80 apart
constexpr size_t attn_lds_bytes(int nkb) { return 2 * (size_t)nkb * 64 * 64 + (size_t)attn_waves(nkb) * kCtxPatch; }

typedef int v2i_t __attribute__((ext_vector_type(2)));

// Over the four lanes (m, 0..3) of a query: lane ^ 32, then lane ^ 16.
template <typename Op>
__device__ __forceinline__ int query_reduce(int v, Op op) { return butterfly_step<16>(butterfly_step<32>(v, op), op); }
__device__ __forceinline__ int row_max(int v) { return query_reduce(v, MaxI32{}); }
__device__ __forceinline__ float row_add(float v) { return __int_as_float(query_reduce(__float_as_int(v), AddF32{})); }

// PWL exp of one score; acc and row maximum as biased accumulators.
template <int kMode>
__device__ __forceinline__ float attn_exp(int acc, float fmax_, const AttnParams& p, float clo, float chi, const float2* s_kb)
{
    const float t = (__int_as_float(acc) - fmax_) * p.alpha_scores;
    if (kMode == EXP_ANY) return pwl_eval_bounded(t, clo, chi, p.t_exp, s_kb);
    float u;
    if (kMode == EXP_PADDED_POW2) u = __builtin_fmaf(t, p.t_exp.inv_w, p.t_exp.u0);
    else u = (t - p.t_exp.lo) * p.t_exp.inv_w;
    const float2 e = s_kb[cvt_u32_sat(u)];
    return __builtin_fmaf(e.x, t, e.y);
}

// Four probabilities as int8 codes; small: all codes of the row are known to lie in [0, 127].
__device__ __forceinline__ unsigned attn_pack(const float (&x)[4], float r, float inv, bool small)
{
    if (small) {
        unsigned w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) w = __builtin_amdgcn_cvt_pk_u8_f32((x[e] * r) * inv, e, w);
        return w;
    }
    return pack4(requant(x[0] * r, inv), requant(x[1] * r, inv), requant(x[2] * r, inv), requant(x[3] * r, inv));
}
// The first n (any integer) of a word's four bytes; zeros behind them.
__device__ __forceinline__ unsigned attn_keep(unsigned w, int n)
{
    return w & (unsigned)(0xffffffffull >> (8 * (4 - min(max(n, 0), 4))));
}
// Whether every row of the wavefront is of that kind: r >= 0 and the bounds of e times r times inv are.
__device__ __forceinline__ bool attn_small(float r, const AttnParams& p)
{
    const bool ok = r >= 0.0f && p.inv_s_p >= 0.0f && (p.e_hi * r) * p.inv_s_p <= 127.0f && (p.e_lo * r) * p.inv_s_p >= -0.5f;
    return __all(ok);
}

// The exp table with its last entry twice, then the reciprocal table, requested into registers
// (before the operand loads, which are younger) and written to LDS.
struct AttnTables {
    float2 te, tr;
    __device__ __forceinline__ void request(const AttnParams& p)
    {
        te = p.t_exp.kb[min((int)threadIdx.x, p.t_exp.nseg - 1)];
        tr = p.t_recip.kb[min((int)threadIdx.x, p.t_recip.nseg - 1)];
    }
    template <int kThreads>
    __device__ __forceinline__ void write(const AttnParams& p, float2* s_exp, float2* s_recip) const
    {
        const int ne = p.t_exp.nseg, nr = p.t_recip.nseg, tid = threadIdx.x;
        if (tid <= ne) s_exp[tid] = te;
        if (tid < nr) s_recip[tid] = tr;
        for (int i = tid + kThreads; i <= ne; i += kThreads) s_exp[i] = p.t_exp.kb[min(i, ne - 1)];
        for (int i = tid + kThreads; i < nr; i += kThreads) s_recip[i] = p.t_recip.kb[i];
    }
};

// Context accumulators of a wavefront -> int8 rows, through a per-wavefront LDS patch so that every lane
// stores 16 consecutive bytes.  Lane (m, hq) holds head columns 16*cb + 4*hq + e of query m.
__device__ __forceinline__ void attn_store_ctx(const AttnParams& p, const v4i (&a2)[4], int8_t* patch, int lane, long row0, int q0,
                                               int head, int nch)
{
    const int fr = lane & 15, hq = lane >> 4;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
        int q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = requant(__builtin_fmaf((float)a2[cb][e], p.alpha_ctx, 0.0f), p.inv_s_ctx);
        *reinterpret_cast<unsigned*>(patch + fr * 80 + 16 * cb + 4 * hq) = pack4(q[0], q[1], q[2], q[3]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int mq = q0 + (lane >> 2), c = lane & 3;
    if (mq < p.S && c < nch) {
        const v4i o = *reinterpret_cast<const v4i*>(patch + (lane >> 2) * 80 + 16 * c);
        int8_t* dst = p.ctx + (row0 + mq) * p.H + head * (16 * nch) + 16 * c;
        if (p.ctx_vec16) {
            *reinterpret_cast<v4i*>(dst) = o;
        } else {
#pragma unroll
            for (int w = 0; w < 4; ++w) *reinterpret_cast<int*>(dst + 4 * w) = o[w];
        }
    }
}

// Operand slot s (0..15) of lane group hq must hold key 64*kb + 16*(s/4) + 4*hq + s%4 (where the
// probabilities sit).  A transposing read delivers eight rows: this lane supplies the address of
// row (lane % 16) / 2 of its group, shifted by 8 bytes for odd lanes so that lanes 8..15 of the
// group receive head columns 8..15.
struct VFragments {
    int off[2], sw[2];
    __device__ __forceinline__ VFragments(int lane)
    {
        const int fr = lane & 15, hq = lane >> 4;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int sidx = 8 * hh + (fr >> 1);
            off[hh] = (16 * (sidx >> 2) + 4 * hq + (sidx & 3)) * 64 + 8 * (fr & 1);
            sw[hh] = hq ^ (sidx >> 2);   // chunk position of column block cb: cb ^ sw
        }
    }
    __device__ __forceinline__ v4i read(const int8_t* base, int cb) const
    {
        v2i_t part[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
            part[hh] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                (__attribute__((address_space(3))) v2i_t*)(base + off[hh] + 16 * (cb ^ sw[hh])));
        return v4i{part[0][0], part[0][1], part[1][0], part[1][1]};
    }
};

// Workgroups are dealt to the eight XCDs round-robin.  Renumbered so that an XCD receives consecutive
// (head, query block) pairs: the query blocks of a head share its K and V, and neighbouring heads
// share 128-byte lines (a head's rows are 64-byte halves), so these fetches then meet in one L2
// instead of going to memory once per XCD.
__device__ __forceinline__ int attn_block_id(int total)
{
    return (int)(blockIdx.x & 7) * ((total + 7) >> 3) + (int)(blockIdx.x >> 3);
}

// NKB: padded key count / 64, head size 64.  kFull: S == 64 * NKB, so no key or query is masked.
//
// A wavefront holds at most 256 keys of its 16 queries (64 score registers), so that four wavefronts fit
// a SIMD and one workgroup's K / V loads run under another's arithmetic.  Beyond 256 keys two wavefronts
// share 16 queries (kSplit): half h takes the 64-key groups 2h, 2h + 1, 4 + 2h, 5 + 2h, i.e. the
// accumulators 32h .. 32h + 31 of the row sum with all their elements; the halves exchange their row
// maxima, their accumulators at the butterfly's first step (mask 32) and their partial contexts
// (exact integers) through the K image, which is free by then.  (With all 512 keys in one wavefront it had 128
// score registers, and two wavefronts a SIMD.)
// us per launch, one behind the other, against the kernel before these steps: 32 x 512 tokens, 16 heads 98 -> 63;
// with 12 heads 16 x 512 39 -> 25, 16 x 384 59 -> 20, 8 x 300 37 -> 8.1, 16 x 256 10 -> 8.1, 32 x 128 6.7 -> 5.6, 11 x 77 5.9 ->
// 4.4, 32 x 64 3.9 -> 3.6.  In the 24- and 12-layer stacks, beside operands that come from further away, the first two take
// 73 and 30.
template <int NKB, bool kFull, int kMode>
__global__ __launch_bounds__(64 * attn_waves(NKB)) __attribute__((amdgpu_waves_per_eu(4))) void attention_pwl_kernel(AttnParams p)
{
    constexpr bool kSplit = NKB > 4;
    constexpr int kAttnThreads = 64 * attn_waves(NKB);
    constexpr int kQueries = 64;       // queries per workgroup
    constexpr int SK = NKB * 64;       // padded key count
    constexpr int NG = kSplit ? NKB / 2 : NKB;   // 64-key groups of a wavefront
    constexpr int NACC = kSplit ? 8 : 4 * NG;    // row-sum accumulators of a lane
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    int8_t* sK = smem;
    int8_t* sV = smem + SK * 64;
    int8_t* sO = smem + 2 * SK * 64;   // context patches
    float2* s_kb = reinterpret_cast<float2*>(smem + attn_lds_bytes(NKB));
    // the kernel arguments everything in front of the loads needs, in one step
    asm volatile("" : : "s"(p.qkv), "s"(p.S), "s"(p.H), "s"(p.heads), "s"(p.qblocks), "s"(p.total), "s"(p.t_exp.kb), "s"(p.t_recip.kb),
                 "s"(p.t_exp.nseg), "s"(p.t_recip.nseg), "s"(p.div_qblocks.magic), "s"(p.div_qblocks.shift), "s"(p.div_heads.magic),
                 "s"(p.div_heads.shift), "s"(p.alpha_scores), "s"(p.inv_s_p), "s"(p.alpha_ctx), "s"(p.inv_s_ctx), "s"(p.t_exp.lo),
                 "s"(p.t_exp.inv_w), "s"(p.t_exp.u0), "s"(p.t_recip.lo), "s"(p.t_recip.hi), "s"(p.t_recip.inv_w),
                 "s"(p.t_recip.clamp_input), "s"(p.e_lo), "s"(p.e_hi), "s"(p.ctx), "s"(p.ctx_vec16));
    if (kMode == EXP_ANY) asm volatile("" : : "s"(p.scores_out), "s"(p.p_out), "s"(p.t_exp.hi), "s"(p.t_exp.clamp_input));
    float2* s_kb_recip = s_kb + p.t_exp.nseg + 1;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, hq = lane >> 4;
    const int id = attn_block_id(p.total);
    if (id >= p.total) return;
    const int by = (int)quotient((unsigned)id, p.div_qblocks), bx = id - by * p.qblocks;
    const int b = (int)quotient((unsigned)by, p.div_heads), head = by - b * p.heads;
    const int S = kFull ? SK : p.S, H = p.H;
    const int ld = 3 * H;
    const int8_t* base = p.qkv + (long)b * S * ld + head * kHeadDim;

    AttnTables tabs;
    tabs.request(p);
    // K and V -> LDS, row-major, by direct global -> LDS loads (16 rows of 64 bytes per wavefront
    // instruction; the chunk rotation is applied to the source address).  Rows past S repeat the last
    // one: their keys are masked.
    {
        const unsigned lds_k = (unsigned)(uintptr_t)sK, lds_v = (unsigned)(uintptr_t)sV;
        const int nb16 = kFull ? SK / 16 : (S + 15) >> 4;
        for (int blk16 = wave; blk16 < nb16; blk16 += kAttnThreads / 64) {
            int r = 16 * blk16 + (lane >> 2);
            if (!kFull) r = min(r, S - 1);
            const int at = r * ld + H;
            dma16s(base, (unsigned)(at + 16 * ((lane & 3) ^ hq)), lds_k + 1024 * blk16);
            dma16s(base, (unsigned)(at + H + 16 * ((lane & 3) ^ hq ^ (blk16 & 3))), lds_v + 1024 * blk16);
        }
    }
    // this lane's query row, straight from global memory into the MFMA operand registers
    const int half = kSplit ? wave & 1 : 0, qwave = kSplit ? wave >> 1 : wave;
    const int q0 = bx * kQueries + qwave * 16, m = q0 + fr;
    const v4i qf = *reinterpret_cast<const v4i*>(base + (long)(kFull ? m : min(m, S - 1)) * ld + 16 * hq);
    tabs.template write<kAttnThreads>(p, s_kb, s_kb_recip);
    wait_vmcnt<0>();   // this wavefront's loads have landed (the barrier covers the others')
    __syncthreads();
    if (!kFull && !kSplit && q0 >= S) return;

    const int ngroups = kFull ? NKB : (S + 63) >> 6;   // 64-key groups with valid keys; the last may be partial
    const bool ragged = !kFull && (S & 63) != 0;
    const auto group_of = [&](int g) { return kSplit ? (g & 1) + 2 * half + 4 * (g >> 1) : g; };   // g-th group of this wavefront
    const auto keys_left = [&](int g) { return S - 64 * group_of(g) - 4 * hq; };   // key (g, q, e) is valid if 16q + e is below it

    // ---- scores and row maximum -----------------------------------------------------------------
    int sc[16 * NG];   // biased scores, then exp values (float bits): key 16q + 4hq + e of group g is sc[16g + 4q + e]
    int mi = INT_MIN;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int gg = group_of(g);
        if (!kFull && gg >= ngroups) continue;   // (the values of an absent group are never read)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i kf = *reinterpret_cast<const v4i*>(&sK[4096 * gg + attn_koff(16 * q + fr, hq)]);
            const v4i a = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf, qf, v4i{kScoreBias, kScoreBias, kScoreBias, kScoreBias}, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) sc[16 * g + 4 * q + e] = a[e];
        }
        if (ragged && gg == ngroups - 1) {
            const int left = keys_left(g);
#pragma unroll
            for (int i = 0; i < 16; ++i) sc[16 * g + i] = 16 * (i / 4) + i % 4 < left ? sc[16 * g + i] : INT_MIN;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) mi = max(mi, sc[16 * g + i]);
        // keeps the operand reads of later groups from piling up in registers
        if (NG >= 4) __builtin_amdgcn_sched_barrier(0);
    }
    const long row_ss = ((long)by * S + m) * S;  // offset of this query's row in [B,heads,S,S]
    const bool vec4 = (S & 3) == 0;
    if (kMode == EXP_ANY && p.scores_out && (kFull || m < S)) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int key = 64 * group_of(g) + 16 * q + 4 * hq;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (kFull || key + e < S) p.scores_out[row_ss + key + e] = sc[16 * g + 4 * q + e] - kScoreBias;
            }
    }
    mi = row_max(mi);
    int* s_max = reinterpret_cast<int*>(sO);             // (the patches are not in use yet)
    int8_t* s_xch = sK;                                  // exchange area, once everybody is done with K
    if (kSplit) {
        if (lane < 16) s_max[16 * wave + lane] = mi;
        __syncthreads();
        mi = max(mi, s_max[16 * (wave ^ 1) + fr]);
    }

    // ---- softmax-PWL ----------------------------------------------------------------------------
    // Keys 256.. wrap onto the 64 accumulators of keys 0..255 (accumulator = (key / 4) % 64) and continue
    // their sums.
    float part[NACC];
    const float fm = __int_as_float(mi);
    const float clo = p.t_exp.clamp_input ? p.t_exp.lo : -__builtin_inff();
    const float chi = p.t_exp.clamp_input ? p.t_exp.hi : __builtin_inff();
#pragma unroll
    for (int q = 0; q < NACC; ++q) part[q] = 0.0f;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if (!kFull && group_of(g) >= ngroups) continue;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            sc[16 * g + i] = __float_as_int(attn_exp<kMode>(sc[16 * g + i], fm, p, clo, chi, s_kb));
            // bounds the number of table look-ups in flight (each holds three registers)
            if (NG >= 4 && i % 8 == 7) __builtin_amdgcn_sched_barrier(0);
        }
        if (ragged && group_of(g) == ngroups - 1) {
            const int left = keys_left(g);
#pragma unroll
            for (int i = 0; i < 16; ++i) sc[16 * g + i] = 16 * (i / 4) + i % 4 < left ? sc[16 * g + i] : 0;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) part[(4 * g + i / 4) % NACC] = part[(4 * g + i / 4) % NACC] + __int_as_float(sc[16 * g + i]);
        if (NG >= 4) __builtin_amdgcn_sched_barrier(0);
    }
    // butterfly over the accumulator index 4*blk + hq: masks 32, 16, 8, 4 (blk), then 2, 1 (hq)
    if (kSplit) {
#pragma unroll
        for (int i = 0; i < NACC; i += 4)
            *reinterpret_cast<v4f*>(s_xch + wave * 2048 + i * 256 + 16 * lane) = v4f{part[i], part[i + 1], part[i + 2], part[i + 3]};
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NACC; i += 4) {
            const v4f o = *reinterpret_cast<const v4f*>(s_xch + (wave ^ 1) * 2048 + i * 256 + 16 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) part[i + e] = part[i + e] + o[e];
        }
    }
#pragma unroll
    for (int mask = NACC / 2; mask >= 1; mask >>= 1)
#pragma unroll
        for (int i = 0; i < mask; ++i) part[i] = part[i] + part[i + mask];
    const float sum = row_add(part[0]);
    int segr;
    const float r = pwl_eval(sum, p.t_recip, s_kb_recip, segr);

    // ---- probabilities and context --------------------------------------------------------------
    const VFragments vfrag(lane);
    v4i a2[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) a2[cb] = v4i{0, 0, 0, 0};
    auto finish = [&](auto small_c) {
        constexpr bool kSmall = decltype(small_c)::value;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int gg = group_of(g);
            if (!kFull && gg >= ngroups) continue;
            v4i pf;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int* at = sc + 16 * g + 4 * q;
                const float x[4] = {__int_as_float(at[0]), __int_as_float(at[1]), __int_as_float(at[2]), __int_as_float(at[3])};
                pf[q] = (int)attn_pack(x, r, p.inv_s_p, kSmall);
            }
            // A masked key's code is 0 whatever r and inv_s_p are (0 times an infinity is a NaN, of code -127); what
            // the V image holds for these keys then does not count.  In the other form r and inv_s_p are finite.
            if (!kSmall && ragged && gg == ngroups - 1) {
                const int left = keys_left(g);
#pragma unroll
                for (int q = 0; q < 4; ++q) pf[q] = (int)attn_keep((unsigned)pf[q], left - 16 * q);
            }
            if (kMode == EXP_ANY && p.p_out && (kFull || m < S)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int key = 64 * gg + 16 * q + 4 * hq;
                    if (vec4 && (kFull || key < S)) {
                        *reinterpret_cast<unsigned*>(p.p_out + row_ss + key) = (unsigned)pf[q];
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (key + e < S) p.p_out[row_ss + key + e] = (int8_t)((unsigned)pf[q] >> (8 * e));
                    }
                }
            }
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                a2[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vfrag.read(sV + 4096 * gg, cb), pf, a2[cb], 0, 0, 0);
            if (NG >= 4) __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (attn_small(r, p)) finish(std::true_type{}); else finish(std::false_type{});
    if (kSplit) {
        // half 0 finishes the context; half 1 hands its partial sums over
        int8_t* x = s_xch + 16384 + qwave * 4096 + 16 * lane;
        if (half == 1) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) *reinterpret_cast<v4i*>(x + 1024 * cb) = a2[cb];
        }
        __syncthreads();
        if (half == 1) return;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) a2[cb] += *reinterpret_cast<const v4i*>(x + 1024 * cb);
    }
    attn_store_ctx(p, a2, sO + wave * kCtxPatch, lane, (long)b * S, q0, head, 4);
}

// Sequences whose scores do not fit a wavefront's registers (more than 512 keys) and head sizes 16, 32 and
// 48: the scores are computed three times, for the row maximum, for the sum and for the probabilities
// (matrix work is cheap: 22.3 vector instructions per score by counter at 4 x 640 tokens, and no score or
// probability goes to memory).  K, and V in the last pass, come through LDS in chunks of 256 keys, the
// next chunk loading while one is used.  A workgroup is four wavefronts of 16 queries.
// Four sequences of 640 tokens, 12 heads of 64: 22 us; scores, softmax and context as three kernels took 21 + 20
// + 15.
constexpr int kLongThreads = 256, kLongKeys = 256;
constexpr size_t kLongLds = 4 * (size_t)kLongKeys * 64 + (kLongThreads / 64) * (size_t)kCtxPatch;

template <int kMode>
__global__ __launch_bounds__(kLongThreads) __attribute__((amdgpu_waves_per_eu(2))) void attention_long_kernel(AttnParams p)
{
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];   // K, K, V, V chunks of 16 KB, context patches, tables
    int8_t* sO = smem + 4 * kLongKeys * 64;
    float2* s_kb = reinterpret_cast<float2*>(smem + kLongLds);
    asm volatile("" : : "s"(p.qkv), "s"(p.S), "s"(p.H), "s"(p.heads), "s"(p.qblocks), "s"(p.total), "s"(p.t_exp.kb), "s"(p.t_recip.kb),
                 "s"(p.t_exp.nseg), "s"(p.t_recip.nseg), "s"(p.nch), "s"(p.scores_out), "s"(p.p_out), "s"(p.div_qblocks.magic),
                 "s"(p.div_qblocks.shift), "s"(p.div_heads.magic), "s"(p.div_heads.shift));
    float2* s_kb_recip = s_kb + p.t_exp.nseg + 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, hq = lane >> 4;
    const int id = attn_block_id(p.total);
    if (id >= p.total) return;
    const int by = (int)quotient((unsigned)id, p.div_qblocks), bx = id - by * p.qblocks;
    const int b = (int)quotient((unsigned)by, p.div_heads), head = by - b * p.heads;
    const int S = p.S, H = p.H, ld = 3 * H, nch = p.nch;
    const int8_t* base = p.qkv + (long)b * S * ld + head * (16 * nch);

    AttnTables tabs;
    tabs.request(p);
    const int nchunks = (S + kLongKeys - 1) / kLongKeys, steps = 3 * nchunks;
    const unsigned lds0 = (unsigned)(uintptr_t)smem;
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
    tabs.write<kLongThreads>(p, s_kb, s_kb_recip);

    const bool ragged = (S & 63) != 0, vec4 = (S & 3) == 0;
    const long row_ss = ((long)by * S + m) * S;
    const float clo = p.t_exp.clamp_input ? p.t_exp.lo : -__builtin_inff();
    const float chi = p.t_exp.clamp_input ? p.t_exp.hi : __builtin_inff();
    const VFragments vfrag(lane);
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
            const int8_t* sK = smem + (step & 1) * 16384;
            const int8_t* sV = smem + 32768 + (step & 1) * 16384;
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
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[q][e] = attn_exp<kMode>(acc[q][e], fm, p, clo, chi, s_kb);
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
                            pf[q] = (int)attn_pack(x[q], r, p.inv_s_p, kSmall);
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

template <int NKB, bool kFull, int kMode>
static int32_t launch_short(AttnParams& p, size_t tables, hipStream_t st)
{
    static std::once_flag once;
    static int32_t once_rc = NM_OK;
    return launch_attn_kernel(attention_pwl_kernel<NKB, kFull, kMode>, once, once_rc, p, 64 * attn_waves(NKB), attn_lds_bytes(NKB) + tables, st);
}
template <int kMode>
static int32_t launch_long(AttnParams& p, size_t tables, hipStream_t st)
{
    static std::once_flag once;
    static int32_t once_rc = NM_OK;
    return launch_attn_kernel(attention_long_kernel<kMode>, once, once_rc, p, kLongThreads, kLongLds + tables, st);
}

template <int NKB, int kMode>
static int32_t launch_nkb(AttnParams& p, int pairs, size_t tables, hipStream_t st)
{
    p.qblocks = (p.S + 63) / 64;
    p.total = p.qblocks * pairs;
    // (from 256 keys on the masked form is the better one even where nothing is masked: its branches keep the
    // compiler from interleaving the groups until registers spill)
    if constexpr (NKB <= 2) {
        if (p.S == 64 * NKB) return launch_short<NKB, true, kMode>(p, tables, st);
    }
    return launch_short<NKB, false, kMode>(p, tables, st);
}

template <int kMode>
static int32_t launch_mode(AttnParams& p, int pairs, hipStream_t st)
{
    const size_t tables = sizeof(float2) * ((size_t)p.t_exp.nseg + 1 + (size_t)p.t_recip.nseg);
    if (p.nch != 4 || p.S > 512) {
        p.qblocks = (p.S + kLongThreads / 4 - 1) / (kLongThreads / 4);
        p.total = p.qblocks * pairs;
        return launch_long<kMode>(p, tables, st);
    }
    if (p.S <= 64) return launch_nkb<1, kMode>(p, pairs, tables, st);
    if (p.S <= 128) return launch_nkb<2, kMode>(p, pairs, tables, st);
    if (p.S <= 256) return launch_nkb<4, kMode>(p, pairs, tables, st);
    return launch_nkb<8, kMode>(p, pairs, tables, st);
}

bool fused_attention_covers(int S, int H, int heads)
{
    const int d = H / heads;
    return d <= kHeadDim && d % 16 == 0 && S <= 4096;
}

int32_t launch_attention(const AttnArgs& a, const char* what, hipStream_t st)
{
    AttnParams p{};
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
    // index of t = 0 by the kernel's own arithmetic
    const float d0 = 0.0f - p.t_exp.lo, u_at_0 = d0 * p.t_exp.inv_w;
    const bool padded = a.alpha_scores >= 0.0f && !p.t_exp.clamp_input && u_at_0 < (float)(p.t_exp.nseg + 1);
    const int pairs = a.B * a.heads;
    if (!padded || p.scores_out || p.p_out) rc = launch_mode<EXP_ANY>(p, pairs, st);
    else if (t_exp.pow2) rc = launch_mode<EXP_PADDED_POW2>(p, pairs, st);
    else rc = launch_mode<EXP_PADDED>(p, pairs, st);
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
