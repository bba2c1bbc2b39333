// The part of fused attention that its kernels share (device code): nm_attention.hip, whose comment has the layout and what bounds it,
// and nm_qkv_attention.hip.
#pragma once

#include <climits>

#include "nm_gemm_common.h"

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
    int off_tile;                      // bytes of LDS in front of the images: the tables
    int ctx_vec16;                     // ctx is 16-byte aligned: context rows leave as 16-byte stores
    FastDiv div_qblocks, div_heads;
    AttnTable t_exp, t_recip;
    int32_t* scores_out;               // optional [B, heads, S, S]
    int8_t* p_out;                     // optional [B, heads, S, S]
};

// For B sequences of S <= 2^keys_log2 tokens (64 or 128): Q, K and V of 128 >> keys_log2 of them and one head, then attention (nm_qkv_attention.hip).
// M and N of the product are 128 rows a workgroup and 192 columns a head.
struct QkvAttnParams : GemmParams {
    AttnParams at;
    int B, keys_log2, pow2;
};
constexpr int kQkvRecip = 256;   // entries of the reciprocal table at most

// How the exp table may be looked up (all false and SLOTS_NONE: as any table).
struct AttnExp {
    int slots;           // TableSlots
    bool padded, pow2;   // as EXP_PADDED; with the position by one fma
};
// Fills p and e.
int32_t attn_params(const AttnArgs& a, const char* what, AttnParams* p, AttnExp* e);

// How the exp table's segment is found.  EXP_ANY: any table and scale (this form also writes the optional outputs).  EXP_SLOTS: a table of at
// most 256 segments without input clamp, in slots, EXP_SLOTS_POW2 with inv_w a power of two.  EXP_PADDED: one that slots do not take (of more
// segments, most of all), without input clamp and with an index of at most nseg at t = 0, the largest t where alpha_scores >= 0: its last
// entry twice instead of the clamp; EXP_PADDED_POW2 (sequences beyond 1024 keys alone, where a SIMD's one wavefront pays for every
// instruction) with inv_w a power of two.  us, any | padded, 257 segments: 32 x 128 tokens, 12 heads 7.3 | 7.1, 16 x 256 10.6 | 10.1, 16 x 512 29.0 |
// 27.5; layers of 4 heads over 2 x 1200 tokens 49.2 | 46.0, over 1 x 4000 117 | 105 (512 segments 117 | 104).
enum { EXP_ANY = 0, EXP_SLOTS = 1, EXP_SLOTS_POW2 = 2, EXP_PADDED = 3, EXP_PADDED_POW2 = 4 };
constexpr bool attn_slots(int mode) { return mode == EXP_SLOTS || mode == EXP_SLOTS_POW2; }
constexpr bool attn_padded(int mode) { return mode == EXP_PADDED || mode == EXP_PADDED_POW2; }
constexpr size_t attn_exp_bytes(int mode, int nseg) { return attn_slots(mode) ? kSlotBytes : sizeof(float2) * (size_t)(nseg + (attn_padded(mode) ? 1 : 0)); }

// Wavefronts that share 16 queries (at most 256 keys each).
constexpr int attn_parts(int S) { return S <= 256 ? 1 : S <= 512 ? 2 : 4; }
constexpr int kHeadDim = 64;
constexpr int kScoreBias = 0x4B400000;   // bits of 1.5 * 2^23: the accumulators' start value

// K image: 64-byte rows, the four 16-byte chunks of a row rotated by (row / 4) % 4 so that the 16
// lanes of an operand read (16 consecutive rows, one chunk) cover all banks.
__device__ __forceinline__ int attn_koff(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 2) & 3)) << 4); }
// V image: the same, with the rotation also depending on (row / (16 kParts)) % 4, because one transposing
// read touches rows that far apart.

constexpr int kCtxPatch = 16 * 80;   // per wavefront: 16 context rows of 64 bytes, 80 apart
// K and V images of ng groups of 64 keys per part, then the context patches or, where wavefronts share queries, their row maxima
// (64 bytes each) and sums (256)
constexpr size_t attn_lds_bytes(int parts, int ng)
{
    return 2 * (size_t)(parts * ng) * 64 * 64 + 4 * (size_t)parts * (parts > 1 ? 64 + 256 : kCtxPatch);
}

typedef int v2i_t __attribute__((ext_vector_type(2)));

// Over the four lanes (m, 0..3) of a query: lane ^ 32, then lane ^ 16.
template <typename Op>
__device__ __forceinline__ int query_reduce(int v, Op op) { return butterfly_step<16>(butterfly_step<32>(v, op), op); }
__device__ __forceinline__ int row_max(int v) { return query_reduce(v, MaxI32{}); }
__device__ __forceinline__ float row_add(float v) { return __int_as_float(query_reduce(__float_as_int(v), AddF32{})); }

// What the loops over the scores use, in vector registers (nm_device.h: a scalar operand halves an instruction's rate).
template <int kMode>
struct AttnConsts {
    float alpha, inv_p, lo, inv_w, u0, steps;   // position in slots: times inv_w (and plus u0), which are 1/256 of the table's
    float clo, chi;                             // EXP_ANY: the input clamp, or infinities
    __device__ __forceinline__ AttnConsts(const AttnParams& p) : alpha(in_vgpr(p.alpha_scores)), inv_p(in_vgpr(p.inv_s_p)), lo(0.0f), u0(0.0f)
    {
        if (kMode == EXP_ANY) {
            clo = p.t_exp.clamp_input ? p.t_exp.lo : -__builtin_inff();
            chi = p.t_exp.clamp_input ? p.t_exp.hi : __builtin_inff();
        } else {
            constexpr float kPart = attn_slots(kMode) ? 1.0f / kSlotSegments : 1.0f;
            inv_w = in_vgpr(p.t_exp.inv_w * kPart);
            if (kMode == EXP_SLOTS_POW2 || kMode == EXP_PADDED_POW2) u0 = in_vgpr(p.t_exp.u0 * kPart);
            else lo = in_vgpr(p.t_exp.lo);
            steps = in_vgpr(8.0f * kSlotSegments);
        }
    }
};

// PWL exp of one score (acc and row maximum as biased accumulators) in two steps: the score's t in its place and its line
// requested, then the line's value in its place.  (Left to itself the compiler writes the value over the line's b, and every one
// keeps the register pair of its table entry: 64 of them spill.)
struct AttnLine { float k, b; };
template <int kMode>
__device__ __forceinline__ AttnLine attn_look_up(int& s, float fmax_, const AttnParams& p, const AttnConsts<kMode>& c, const int8_t* s_exp)
{
    float t = (__int_as_float(s) - fmax_) * c.alpha;
    float2 e;
    if (kMode == EXP_ANY) {
        t = __builtin_amdgcn_fmed3f(t, c.clo, c.chi);
        e = reinterpret_cast<const float2*>(s_exp)[seg_index(t, p.t_exp.lo, p.t_exp.inv_w, p.t_exp.nseg)];
    } else if (attn_padded(kMode)) {
        const float u = kMode == EXP_PADDED_POW2 ? __builtin_fmaf(t, c.inv_w, c.u0) : (t - c.lo) * c.inv_w;
        e = slot_line(cvt_u32_sat(u) * (unsigned)sizeof(float2));   // (the table is the first thing in LDS)
    } else {
        const float u = kMode == EXP_SLOTS_POW2 ? fma_clamp01(t, c.inv_w, c.u0) : mul_clamp01(t - c.lo, c.inv_w);
        e = slot_line(slot_offset(u, c.steps));   // (the slots are the first thing in LDS)
    }
    s = __float_as_int(t);
    return {e.x, e.y};
}
__device__ __forceinline__ void attn_line(int& s, const AttnLine& e)
{
    asm("v_fma_f32 %0, %1, %0, %2" : "+v"(s) : "v"(e.k), "v"(e.b));
}
template <int kMode>
__device__ __forceinline__ float attn_exp(int acc, float fmax_, const AttnParams& p, const AttnConsts<kMode>& c, const int8_t* s_exp)
{
    const AttnLine e = attn_look_up<kMode>(acc, fmax_, p, c, s_exp);
    return __builtin_fmaf(e.k, __int_as_float(acc), e.b);
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

// The exp table (in slots, or its entries) and the reciprocal table, requested into registers
// (before the operand loads, which are younger) and written to LDS.
template <int kMode, int kThreads>
struct AttnTables {
    static_assert(kThreads >= kSlotSegments, "a slot per thread");
    float2 te, tr, last;
    __device__ __forceinline__ void request(const AttnParams& p)
    {
        te = p.t_exp.kb[min((int)threadIdx.x, p.t_exp.nseg - 1)];
        tr = p.t_recip.kb[min((int)threadIdx.x, p.t_recip.nseg - 1)];
        if (attn_padded(kMode)) last = p.t_exp.kb[p.t_exp.nseg - 1];
    }
    __device__ __forceinline__ void write(const AttnParams& p, float2* s_exp, float2* s_recip) const
    {
        const int ne = p.t_exp.nseg, nr = p.t_recip.nseg, tid = threadIdx.x;
        if (!attn_slots(kMode)) {
            if (tid < ne) s_exp[tid] = te;
            for (int i = tid + kThreads; i < ne; i += kThreads) s_exp[i] = p.t_exp.kb[i];
            if (attn_padded(kMode) && tid == 0) s_exp[ne] = last;
        } else {
            write_slots(s_exp, te, tid);
        }
        if (tid < nr) s_recip[tid] = tr;
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

// Operand slot s (0..15) of lane group hq must hold key 4*hq + s%4 of the (s/4)-th of four 16-key blocks, kParts blocks apart
// (where the probabilities sit).  A transposing read delivers eight rows: this lane supplies the address of
// row (lane % 16) / 2 of its group, shifted by 8 bytes for odd lanes so that lanes 8..15 of the
// group receive head columns 8..15.
template <int kParts>
struct VFragments {
    int off[2], sw[2];
    __device__ __forceinline__ VFragments(int lane)
    {
        const int fr = lane & 15, hq = lane >> 4;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int sidx = 8 * hh + (fr >> 1);
            off[hh] = (16 * kParts * (sidx >> 2) + 4 * hq + (sidx & 3)) * 64 + 8 * (fr & 1);
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

// Attention of a wavefront's 16 queries (head columns in qf) over the keys whose K and V rows lie in the images: scores, softmax-PWL,
// context codes to memory.  Used behind both kernels' barrier; with kParts > 1 every wavefront of the workgroup takes part.
template <int kParts, int NG, bool kFull, int kMode, bool kHead64>
__device__ __forceinline__ void attn_queries(const AttnParams& p, const AttnConsts<kMode>& consts, v4i qf, int8_t* s_tile, int8_t* sK, int8_t* sV,
                                             int8_t* sO, const int8_t* s_exp, const float2* s_kb_recip, int lane, int wave, int S, int by, int b,
                                             int head, int q0)
{
    constexpr int kWaves = 4 * kParts, SK = 64 * kParts * NG;
    constexpr int NU = 4 * NG;                // 16-key blocks of a part
    constexpr int kPeriod = 16 / kParts;      // ... of each 256 keys: the row sum's accumulators of a lane
    constexpr int NACC = NU < kPeriod ? NU : kPeriod;
    constexpr int kBlock = 1024 * kParts;     // bytes of K and V from one block of a part to the next
    constexpr int kColumns = 4 / kParts;      // column blocks of the context that a wavefront finishes
    constexpr bool kLateV = kParts >= 2;
    const int fr = lane & 15, hq = lane >> 4, part_id = wave & (kParts - 1), qwave = wave / kParts, m = q0 + fr;
    const int H = p.H, nch = kHead64 ? 4 : p.nch;
    // Unit u: the part's u-th block, keys 16 (kParts u + part) + 4 hq + e.  Keys from S on lie in the last group's units alone:
    // all bits set where e + 16 kParts (u - first unit of that group) is below `left`.
    sK += 1024 * part_id;
    sV += 1024 * part_id;
    const int left = S - 16 * kParts * 4 * (NG - 1) - 16 * part_id - 4 * hq;
    const auto valid = [&](int u, int e) { return (16 * kParts * (u - 4 * (NG - 1)) + e - left) >> 31; };

    // ---- scores and row maximum -----------------------------------------------------------------
    // operands of a group one group ahead of its products, the maximum one behind
    int sc[16 * NG];   // biased scores, then t, then exp values (float bits): e of unit u is sc[4u + e]
    int mi = INT_MIN;
    v4i kf[2][4];
    const int8_t* const k_frag = sK + attn_koff(fr, hq);
    const auto load_k = [&](int g) {
#pragma unroll
        for (int q = 0; q < 4; ++q) kf[g & 1][q] = *reinterpret_cast<const v4i*>(k_frag + kBlock * (4 * g + q));
    };
    const auto group_max = [&](int g) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            int& s = sc[16 * g + i];
            if (!kFull && g == NG - 1) {
                const int ok = valid(4 * g + i / 4, i % 4);
                s = (s & ok) | (INT_MIN & ~ok);
            }
            mi = max(mi, s);
        }
    };
    load_k(0);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG) load_k(g + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i a = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf[g & 1][q], qf, v4i{kScoreBias, kScoreBias, kScoreBias, kScoreBias}, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) sc[16 * g + 4 * q + e] = a[e];
        }
        if (g > 0) group_max(g - 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    group_max(NG - 1);
    const long row_ss = ((long)by * S + m) * S;  // offset of this query's row in [B,heads,S,S]
    const bool vec4 = (S & 3) == 0;
    const auto key_of = [&](int u) { return 16 * (kParts * u + part_id) + 4 * hq; };
    if (kMode == EXP_ANY && p.scores_out && m < S) {
#pragma unroll
        for (int i = 0; i < 16 * NG; ++i)
            if (key_of(i / 4) + i % 4 < S) p.scores_out[row_ss + key_of(i / 4) + i % 4] = sc[i] - kScoreBias;
    }
    mi = row_max(mi);
    int* const s_max = reinterpret_cast<int*>(sO);
    float* const s_sum = reinterpret_cast<float*>(sO + 64 * kWaves);
    if (kParts > 1) {
        if (lane < 16) s_max[16 * wave + lane] = mi;
        __syncthreads();   // (everybody is done with K, too)
#pragma unroll
        for (int o = 1; o < kParts; ++o) mi = max(mi, s_max[16 * (wave ^ o) + fr]);
    }

    // ---- softmax-PWL ----------------------------------------------------------------------------
    // Keys 256.. wrap onto the 64 accumulators of keys 0..255 (accumulator = (key / 4) % 64) and continue
    // their sums.  The look-ups of a unit are requested kAhead units before they are used, so that a wavefront has
    // some in flight all the time (eight at a time and then waited for: 32 x 512 tokens, 16 heads 68 us, 66 so).
    float part[NACC];
    const float fm = __int_as_float(mi);
#pragma unroll
    for (int j = 0; j < NACC; ++j) part[j] = 0.0f;
    // (The forms without slots need more registers for a look-up: with three ahead EXP_ANY spilled 16 at 256 keys, 16 x 256 tokens, 12 heads, with
    // the input clamp 12.7 us, now 9.8.)
    constexpr int kAhead = attn_slots(kMode) ? 3 : 1;
    AttnLine line[kAhead + 1][4];
#pragma unroll
    for (int u = 0; u < NU + kAhead; ++u) {
        if (u < NU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) line[u % (kAhead + 1)][e] = attn_look_up<kMode>(sc[4 * u + e], fm, p, consts, s_exp);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (u >= kAhead) {
            const int d = u - kAhead;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int& s = sc[4 * d + e];
                attn_line(s, line[d % (kAhead + 1)][e]);
                if (!kFull && d >= 4 * (NG - 1)) s &= valid(d, e);
                part[d % kPeriod] = part[d % kPeriod] + __int_as_float(s);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // butterfly over the accumulator index 4 * (kParts j + part) + hq: masks 32 .. of j, then the part's, then 2 and 1 (hq)
    if (kLateV) wait_vmcnt<0>();   // V has landed (the next barrier covers the others')
#pragma unroll
    for (int mask = kPeriod / 2; mask >= 1; mask >>= 1)
#pragma unroll
        for (int j = 0; j < mask; ++j)
            if (j + mask < NACC) part[j] = part[j] + part[j + mask];   // (an absent one is +0, and no sum is -0)
    float sum = part[0];
    if (kParts > 1) {
        s_sum[64 * wave + lane] = sum;
        __syncthreads();
        sum = sum + s_sum[64 * (wave ^ (kParts / 2)) + lane];
        if (kParts == 4) sum = sum + (s_sum[64 * (wave ^ 1) + lane] + s_sum[64 * (wave ^ 3) + lane]);
    }
    sum = row_add(sum);
    int segr;
    const float r = pwl_eval(sum, p.t_recip, s_kb_recip, segr);

    // ---- probabilities and context --------------------------------------------------------------
    const VFragments<kParts> vfrag(lane);
    v4i a2[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) a2[cb] = v4i{0, 0, 0, 0};
    auto finish = [&](auto small_c) {
        constexpr bool kSmall = decltype(small_c)::value;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            v4i vf[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                if (kHead64 || cb < nch) vf[cb] = vfrag.read(sV + 4 * kBlock * g, cb);
            __builtin_amdgcn_sched_barrier(0);
            v4i pf;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int* at = sc + 16 * g + 4 * q;
                const float x[4] = {__int_as_float(at[0]), __int_as_float(at[1]), __int_as_float(at[2]), __int_as_float(at[3])};
                pf[q] = (int)attn_pack(x, r, consts.inv_p, kSmall);
            }
            // A masked key's code is 0 whatever r and inv_s_p are (0 times an infinity is a NaN, of code -127); what
            // the V image holds for these keys then does not count.  In the other form r and inv_s_p are finite.
            if (!kFull && !kSmall && g == NG - 1) {
#pragma unroll
                for (int q = 0; q < 4; ++q) pf[q] = (int)attn_keep((unsigned)pf[q], left - 16 * kParts * q);
            }
            if (kMode == EXP_ANY && p.p_out && m < S) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int key = key_of(4 * g + q);
                    if (vec4 && key < S) {
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
                if (kHead64 || cb < nch) a2[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf[cb], pf, a2[cb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (attn_small(r, p)) finish(std::true_type{}); else finish(std::false_type{});
    if constexpr (kParts == 1) {
        attn_store_ctx(p, a2, sO + wave * kCtxPatch, lane, (long)b * S, q0, head, nch);
    } else {
        // part h finishes column blocks kColumns * h .., the others hand their sums of these over
        int8_t* const x = s_tile + 16 * lane;
        const auto slot = [&](int cb, int from) {   // of part from (not the finisher) for column block cb
            return ((qwave * 4 + cb) * (kParts - 1) + from - (from > cb / kColumns ? 1 : 0)) * 1024;
        };
        static_assert(16 * (kParts - 1) * 1024 <= SK * 64, "exchange fits the K image");
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
            if (cb / kColumns != part_id) *reinterpret_cast<v4i*>(x + slot(cb, part_id)) = a2[cb];
        __syncthreads();
        v4i mine[kColumns];
#pragma unroll
        for (int c = 0; c < kColumns; ++c) {
            mine[c] = a2[c];
#pragma unroll
            for (int h = 1; h < kParts; ++h)   // (a2 is indexed by constants only: its registers have no addresses)
                if (part_id == h) mine[c] = a2[kColumns * h + c];
#pragma unroll
            for (int o = 0; o < kParts - 1; ++o)
                mine[c] += *reinterpret_cast<const v4i*>(x + ((qwave * 4 + kColumns * part_id + c) * (kParts - 1) + o) * 1024);
        }
        if (!kFull && m >= S) return;
        int8_t* dst = p.ctx + ((long)b * S + m) * H + head * (16 * nch) + 16 * kColumns * part_id + 4 * hq;
#pragma unroll
        for (int c = 0; c < kColumns; ++c) {
            if (!kHead64 && kColumns * part_id + c >= nch) break;
            int q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = requant(__builtin_fmaf((float)mine[c][e], p.alpha_ctx, 0.0f), p.inv_s_ctx);
            *reinterpret_cast<unsigned*>(dst + 16 * c) = pack4(q[0], q[1], q[2], q[3]);
        }
    }
}

}  // namespace nm
