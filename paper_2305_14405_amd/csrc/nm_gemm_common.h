// Declarations shared by the GEMM kernels of this library (device code; included by nm_gemm.hip).
#pragma once

#include <mutex>
#include <type_traits>

#include "nm_device.h"
#include "nm_gemm_choice.h"

namespace nm {

constexpr int kGemmThreads = 256;
constexpr int kBK = 64;  // bytes of k per pipeline stage

struct GemmParams {
    int M, N, K;
    int tiles_m, tiles_n;
    int group_m;  // tile rows per group of the XCD-aware tile order
    FastDiv div_group, div_gm;   // by group_m * tiles_n (streaming kernel: 8 * tiles_n) and group_m
    const int8_t* A; long lda;
    const int8_t* W; long ldw;
    int inner_count;
    long a_outer, a_inner, w_outer, w_inner, o_outer, o_inner;
    const float* bias;
    const float* alpha_vec;
    float alpha;
    const int8_t* resid;
    float resid_scale;
    int has_table;
    DevTable table;
    float out_inv_scale;
    const float* out_inv_scale_vec;
    int split_cols;
    float inv3[3];
    long ldo;
    int vec_out;
    int q16;       // int8 output rows may be written with 16-byte stores
    int r16;       // int8 residual rows may be read with 16-byte loads (and N % 16 == 0)
    int vec_cols;  // bias / per-column scale vectors may be read with 16-byte loads
    int8_t* out_q;
    float* out_f32;
    int32_t* out_acc;
    uint16_t* dbg_seg;
    // convolution in matrix form (streaming kernel with kConv): row m of A is the output position
    // (b, ho, wo), column k the (tap, channel) pair; A points to the NHWC image tensor
    int cH, cW, cCin, cKw, cStride, cPad, cHo, cWo;
    int relu;     // relu_codes holds for the table and the one output scale
    int batched;  // more than one problem (grid.y)
    int taps_w;            // tile kernel, kConv: filter columns (taps are numbered row by row, at most 32)
    FastDiv div_tiles_m, div_wo, div_ho, div_cin, div_kw;   // by tiles_m, cWo, cHo, cCin and cKw
};

struct GemmLnParams : GemmParams {
    // LayerNorm-PWL folded into the epilogue (EPI_F32_RESID_LN): y = fma(d * r, gamma, beta) with
    // r = PWL_rsqrt(var + eps); outputs its int8 code and / or fp32 value, row stride N
    const float* ln_gamma;
    const float* ln_beta;
    float ln_eps, ln_inv_scale;
    DevTable ln_table;
    int8_t* ln_out_q;
    float* ln_out_f32;
};

// The small-tile kernel (nm_gemm_direct.hip).  align: alignment of operand rows and chunks in bytes (16, 4 or
// 1); forced: tile configuration 0 .. 6, or -1 for the rule.
int32_t launch_direct(GemmParams& p, int align, bool conv, int batches, size_t table_bytes, int forced, hipStream_t s);

// Two convolutions as one launch of that kernel: whether the epilogue of p allows it, and the launch (tile configuration cfg for both).
bool direct_pair_takes(const GemmParams& p);
int32_t launch_direct_pair(GemmParams (&p)[2], int cfg, hipStream_t s);

// The tile kernel's configuration cfg for K in whole chunks of 16 bytes but not whole slices (nm_gemm_end.hip).
int32_t launch_tile_end(int cfg, GemmParams& p, int epi, size_t table_bytes, hipStream_t s);

// The same for any such K and int8 results through a table that slots do not take (nm_gemm_long.hip).
int32_t launch_tile_long(int cfg, GemmParams& p, size_t table_bytes, hipStream_t s);

// The register-staged tile kernel (nm_gemm_unaligned.hip): one problem, operands of any alignment (align: 4 or 1).
int32_t launch_unaligned(GemmParams& p, int align, size_t table_bytes, int forced, hipStream_t s);

// XOR swizzle of the 16-byte chunk index inside a 64-byte LDS row: rows that fall into the same
// bank window get different chunk positions, for both a 128-byte and a 256-byte wide LDS port.
__device__ __forceinline__ int swz(int row) { return ((row >> 1) & 3) ^ ((row >> 2) & 3); }

__device__ __forceinline__ int lds_off(int row, int chunk) { return row * kBK + ((chunk ^ swz(row)) << 4); }


// ---- operands of any alignment, through registers ------------------------------------------------
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr unsigned kOutOfRange = 0xc0000000u;  // past the end of every buffer (their extents are below 2^31)

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00027000);
}

__device__ __forceinline__ v4i buf16(rsrc_t r, unsigned off)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    return v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
}
__device__ __forceinline__ unsigned buf4(rsrc_t r, unsigned off)
{
    return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
}

// kAl: bytes every row start and every 16-byte chunk is aligned to (4: whole words, 1: any; the latter reads
// the words around the chunk and shifts).
template <int kAl>
__device__ __forceinline__ v4i load_unit(rsrc_t r, unsigned off)
{
    if (kAl == 4) return buf16(r, off);
    const unsigned base = off & ~3u, sh = off & 3u;
    const v4i w = buf16(r, base);
    const unsigned w4 = buf4(r, base + 16);
    v4i o;
    o[0] = (int)__builtin_amdgcn_alignbyte((unsigned)w[1], (unsigned)w[0], sh);
    o[1] = (int)__builtin_amdgcn_alignbyte((unsigned)w[2], (unsigned)w[1], sh);
    o[2] = (int)__builtin_amdgcn_alignbyte((unsigned)w[3], (unsigned)w[2], sh);
    o[3] = (int)__builtin_amdgcn_alignbyte(w4, (unsigned)w[3], sh);
    return o;
}
// The same for the last, partly filled k-step: word by word (each is inside the buffer or reads as
// zero), bytes at and past `left` (the number of valid ones, possibly <= 0) cleared.
template <int kAl>
__device__ __forceinline__ v4i load_tail(rsrc_t r, unsigned off, int left)
{
    const unsigned base = off & ~3u, sh = kAl == 4 ? 0u : off & 3u;
    unsigned w[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) w[t] = buf4(r, left > 0 ? base + 4 * t : kOutOfRange);
    v4i o;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const unsigned v = kAl == 4 ? w[t] : __builtin_amdgcn_alignbyte(w[t + 1], w[t], sh);
        const int nb = left - 4 * t;  // valid bytes of this word
        o[t] = nb >= 4 ? (int)v : nb <= 0 ? 0 : (int)(v & ((1u << (8 * nb)) - 1u));
    }
    return o;
}

typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32_a1 __attribute__((aligned(1)));

enum Epilogue { EPI_GENERIC = 0, EPI_Q = 1, EPI_Q_TABLE = 2, EPI_F32_RESID = 3, EPI_ACC = 4, EPI_Q_TABLE_RESID = 5, EPI_F32_RESID_LN = 6, EPI_Q_LONG = 7, EPI_Q_RELU = 8, EPI_Q_RELU_RESID = 9, EPI_ATTENTION = 10 };
// EPI_F32_RESID_LN: EPI_F32_RESID followed by LayerNorm-PWL over the row, inside the kernel: the tile
// covers whole rows (tile kernel only).
// EPI_Q_LONG: EPI_Q_TABLE with a table that slots do not take (tile kernel only, nm_gemm_long.hip; there EPI_Q_TABLE is one that they do).
// EPI_Q_RELU, EPI_Q_RELU_RESID: per-column scales, a table of two segments, without and with an int8 residual (tile
// kernel only: convolutions).
// EPI_ATTENTION: the Q, K and V of one head, which go no further than LDS, and attention behind them (tile kernel only).
// EPI_Q_TABLE_RESID: int8 residual, table (no input clamp), int8 output: the last convolution of a
// residual block (sum with the shortcut, ReLU).


template <int BK>
__device__ __forceinline__ int swz_bk(int row)
{
    return BK == 64 ? swz(row) : ((row >> 1) & 7);
}
template <int BK>
__device__ __forceinline__ int lds_off_bk(int row, int chunk)
{
    return row * BK + ((chunk ^ swz_bk<BK>(row)) << 4);
}

// ---------------------------------------------------------------------------------------------

// Epilogue shared by the kernels of any option.  A lane holds, for one output row m, four consecutive columns
// nb .. nb+3 (one group of four accumulator registers).
// ---------------------------------------------------------------------------------------------
// Epilogue specialisations: the generic one reads every option at run time; the others fix the
// set of outputs and options the encoder layer uses, which removes dead code from the unrolled
// epilogue (it is instantiated once per accumulator group).
struct Epi4 {
    float y[4];
    int q[4];
    int s[4];
};

// Per-column parameters of four consecutive columns, loaded once and reused for every row.
struct Col4 {
    float scale[4], bias[4], inv[4];
};

__device__ __forceinline__ void load4(const float* __restrict__ v, int nb, int N, bool vec, float (&out)[4])
{
    if (vec && nb + 3 < N) {
        const v4f t = *reinterpret_cast<const v4f*>(v + nb);
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = t[e];
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (nb + e < N) out[e] = v[nb + e];
    }
}

template <int kEpi>
__device__ __forceinline__ void load_cols(const GemmParams& p, int nb, Col4& c)
{
    const float alpha = p.alpha, ois = p.out_inv_scale;
#pragma unroll
    for (int e = 0; e < 4; ++e) { c.scale[e] = alpha; c.bias[e] = 0.0f; c.inv[e] = ois; }
    if (kEpi == EPI_ACC) return;
    if (p.bias) load4(p.bias, nb, p.N, p.vec_cols, c.bias);
    if (p.alpha_vec) load4(p.alpha_vec, nb, p.N, p.vec_cols, c.scale);
    if (kEpi == EPI_F32_RESID) return;
    if (kEpi == EPI_GENERIC && p.out_inv_scale_vec) {
        load4(p.out_inv_scale_vec, nb, p.N, p.vec_cols, c.inv);
    } else if (p.split_cols > 0) {
        const float i0 = p.inv3[0], i1 = p.inv3[1], i2 = p.inv3[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) c.inv[e] = nb + e >= 2 * p.split_cols ? i2 : (nb + e >= p.split_cols ? i1 : i0);
    }
}

// Residual codes of four consecutive columns of one row.
__device__ __forceinline__ void load_resid4(const GemmParams& p, long rowoff, int nb, bool vec, int (&r4)[4])
{
    if (vec) {
        const unsigned w = *reinterpret_cast<const unsigned*>(p.resid + rowoff + nb);
#pragma unroll
        for (int e = 0; e < 4; ++e) r4[e] = (int)(int8_t)(w >> (8 * e));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r4[e] = nb + e < p.N ? (int)p.resid[rowoff + nb + e] : 0;
    }
}

// How the streaming kernel's epilogue evaluates its table.
enum TableForm { FORM_ANY = 0, FORM_TWO_SEGMENTS = 1, FORM_RELU = 2 };

// The arithmetic of the epilogue for four columns of one row (no global memory access).
// kTwoSeg: the table has two segments and is evaluated with a compare (specialised table epilogues)
template <int kEpi, bool kTwoSeg = false>
__device__ __forceinline__ void epi_math(const GemmParams& p, const float2* s_kb, const int (&a4)[4],
                                         const Col4& c, const int (&r4)[4], Epi4& o)
{
    const bool use_resid = kEpi == EPI_GENERIC ? p.resid != nullptr : (kEpi == EPI_F32_RESID || kEpi == EPI_Q_TABLE_RESID);
    const bool use_table = kEpi == EPI_GENERIC ? p.has_table != 0 : (kEpi == EPI_Q_TABLE || kEpi == EPI_Q_TABLE_RESID);
    const bool need_q = kEpi == EPI_GENERIC ? p.out_q != nullptr : (kEpi == EPI_Q || kEpi == EPI_Q_TABLE || kEpi == EPI_Q_TABLE_RESID);
#pragma unroll
    for (int e = 0; e < 4; ++e) { o.y[e] = 0.0f; o.q[e] = 0; o.s[e] = 0; }
    if (kEpi == EPI_ACC) return;
    const float rs = p.resid_scale;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float v = __builtin_fmaf((float)a4[e], c.scale[e], c.bias[e]);
        if (use_resid) v = __builtin_fmaf((float)r4[e], rs, v);
        if (use_table) {
            if (kTwoSeg) v = pwl_eval_two_segments(v, p.table);
            else if (kEpi == EPI_Q_TABLE || kEpi == EPI_Q_TABLE_RESID) v = pwl_eval_noclamp(v, p.table, s_kb, o.s[e]);
            else if (p.table.cellmap) v = pwl_eval_two_level(v, p.table, s_kb, o.s[e]);  // merged table, two steps
            else v = pwl_eval(v, p.table, s_kb, o.s[e]);
        }
        o.y[e] = v;
        if (need_q) o.q[e] = requant(v, c.inv[e]);
    }
}

// The values of N groups of four columns (one row each), every option of the generic epilogue: y as the fp32 results, seg as
// dbg_seg reports them (valid where there is a table).  Each option is one test around a loop over all groups: a test
// inside splits the loop into small blocks and serialises their LDS reads (the 32 groups of a lane took 4 x as long).
template <int N>
__device__ __forceinline__ void epi_values(const GemmParams& p, const float2* s_kb, const v4i (&a)[N], const float* scale, const float* bias,
                                           const unsigned (&res)[N], float (&y)[N][4], int (&seg)[N][4])
{
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) y[t][e] = __builtin_fmaf((float)a[t][e], scale[e], bias[e]);
    if (p.resid) {
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) y[t][e] = __builtin_fmaf((float)(int)(int8_t)(res[t] >> (8 * e)), p.resid_scale, y[t][e]);
    }
    if (p.has_table) {
        const float lo = p.table.lo, hi = p.table.hi, inv_w = p.table.inv_w;
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float xc = __builtin_amdgcn_fmed3f(y[t][e], lo, hi);
                y[t][e] = p.table.clamp_input ? xc : y[t][e];
                seg[t][e] = seg_index(y[t][e], lo, inv_w, p.table.nseg);
            }
        if (p.table.cellmap) {   // merged table, two steps
            const uint8_t* map = reinterpret_cast<const uint8_t*>(s_kb + p.table.nkb);
#pragma unroll
            for (int t = 0; t < N; ++t) {
                float2 kb[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) kb[e] = s_kb[map[seg[t][e]]];
#pragma unroll
                for (int e = 0; e < 4; ++e) y[t][e] = __builtin_fmaf(kb[e].x, y[t][e], kb[e].y);
            }
        } else {
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float2 kb = s_kb[seg[t][e]];
                    y[t][e] = __builtin_fmaf(kb.x, y[t][e], kb.y);
                }
        }
    }
}

template <int kEpi>
__device__ __forceinline__ void epi_store(const GemmParams& p, long rowoff, int nb,
                                          const int (&a4)[4], const Epi4& o, bool vec, bool skip_q)
{
    const bool st_q = (kEpi == EPI_GENERIC ? p.out_q != nullptr : (kEpi == EPI_Q || kEpi == EPI_Q_TABLE || kEpi == EPI_Q_TABLE_RESID)) && !skip_q;
    const bool st_f = kEpi == EPI_GENERIC ? p.out_f32 != nullptr : kEpi == EPI_F32_RESID;
    const bool st_a = kEpi == EPI_GENERIC ? p.out_acc != nullptr : kEpi == EPI_ACC;
    const bool st_s = kEpi == EPI_GENERIC && p.dbg_seg && p.has_table;
    if (vec) {
        if (st_q) *reinterpret_cast<unsigned*>(p.out_q + rowoff + nb) = pack4(o.q[0], o.q[1], o.q[2], o.q[3]);
        if (st_f) *reinterpret_cast<v4f*>(p.out_f32 + rowoff + nb) = v4f{o.y[0], o.y[1], o.y[2], o.y[3]};
        if (st_a) *reinterpret_cast<v4i*>(p.out_acc + rowoff + nb) = v4i{a4[0], a4[1], a4[2], a4[3]};
        if (st_s)
            *reinterpret_cast<uint2*>(p.dbg_seg + rowoff + nb) =
                make_uint2((unsigned)o.s[0] | ((unsigned)o.s[1] << 16), (unsigned)o.s[2] | ((unsigned)o.s[3] << 16));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (nb + e < p.N) {
                if (st_q) p.out_q[rowoff + nb + e] = (int8_t)o.q[e];
                if (st_f) p.out_f32[rowoff + nb + e] = o.y[e];
                if (st_a) p.out_acc[rowoff + nb + e] = a4[e];
                if (st_s) p.dbg_seg[rowoff + nb + e] = (uint16_t)o.s[e];
            }
    }
}

}  // namespace nm
