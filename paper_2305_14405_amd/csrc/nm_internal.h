// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <tuple>
#include <utility>
#include <vector>

#include "nm.h"

namespace nm {

// One PWL table as the kernels see it.  kb[s] = {k, b} of segment s (device memory).
struct DevTable {
    const float2* kb;
    float lo, hi, inv_w;
    int nseg;
    int clamp_input;
    // two-level form of a merged table (NM_TABLE_COMPACT), null / 0 otherwise: cellmap[cell] is
    // the merged segment of a primary cell, ckb[segment] its {k, b}; nkb segments
    const float2* ckb;
    const uint8_t* cellmap;
    int nkb;
    // a table of two segments (without the clamp flag): its two lines and the smallest fp32 value
    // whose segment index is 1, so that a kernel may pick the line with one compare (two_seg != 0)
    int two_seg;
    float k0, b0, k1, b1, tau;
    // inv_w is a power of two: (x - lo) * inv_w == fma(x, inv_w, u0) bit for bit, u0 = -lo * inv_w exactly
    // (scaling by a power of two commutes with rounding)
    int pow2;
    float u0;
    int slots;   // TableSlots: whether the kernels may look the table up by slots
};
// nm_device.h has the look-up: tables of at most 256 segments without the clamp flag whose scaled numbers are exact; SLOTS_POW2: with
// the position by one fma.
enum TableSlots { SLOTS_NONE = 0, SLOTS_ANY = 1, SLOTS_POW2 = 2 };
constexpr int kSlotSegments = 256;

// Division by a number the host knows: exact for every n below 2^31 (Granlund and Montgomery, "Division by invariant
// integers using multiplication", 1994: a multiplier of 32 bits does for dividends of 31).
struct FastDiv {
    unsigned d, magic, shift;
};
static inline FastDiv fast_div(int d)
{
    unsigned s = 0;
    while ((1u << s) < (unsigned)d) ++s;
    // d == 1: the quotient is the number itself (magic 0)
    return {(unsigned)d, s == 0 ? 0u : (unsigned)((1ull << (31 + s)) / (unsigned)d) + 1u, s == 0 ? 0u : s - 1u};
}

// Bytes of the two-level form: {k, b} per merged segment, a byte per primary cell (padded to eight).
inline size_t two_level_bytes(const DevTable& t) { return 8 * (size_t)t.nkb + (((size_t)t.nseg + 7) & ~(size_t)7); }

// Whether the int8 code of the table's value is that of max(x, 0) for every finite x: the two lines are 0 and x,
// and between 0 and the threshold (where the float index puts it) either line's value rounds to code 0.
inline bool relu_codes(const DevTable& t, float out_inv_scale, float resid_scale)
{
    return t.two_seg && t.k0 == 0.0f && t.b0 == 0.0f && t.k1 == 1.0f && t.b1 == 0.0f && out_inv_scale > 0.0f && out_inv_scale <= 3e38f &&
           std::fabs(t.tau) * out_inv_scale < 0.49f && std::fabs(resid_scale) <= 1e30f;
}

// Bounds of a table's value (host): over its range, and the lines of its two edge segments, which
// continue outside it.
struct TableBounds {
    double vmin, vmax;              // of fma(k, x, b) over [lo, hi], widened past rounding
    double k_first, b_first, k_last, b_last;
};

struct HostTable {
    nm_table_desc desc;
    float inv_w;
    int n_distinct;
    std::vector<float> k, b;
    size_t blob_offset;  // in float2 units
    // two-level form (NM_TABLE_COMPACT): one {k, b} per merged segment and a byte per primary cell
    std::vector<float> ck, cb;
    std::vector<uint8_t> cellmap;
    size_t cblob_offset = 0;  // float2 units
    size_t map_offset = 0;    // float2 units (the map's bytes start there)
    // derived once (derive_table)
    float tau = 0.0f;         // two segments: the smallest value of segment 1
    int pow2 = 0;
    float u0 = 0.0f;
    int slots = 0;
    TableBounds bounds{};
};

int32_t launch_layernorm2(const float* in, const float* gamma, const float* beta, float eps,
                          int64_t rows, int32_t cols, const DevTable& t, const DevTable& t2, int two,
                          float out_inv_scale, int8_t* out_q, float* out_f32, uint16_t* seg, uint16_t* seg2,
                          hipStream_t stream);

}  // namespace nm

struct nm_tables {
    std::vector<nm::HostTable> tables;
    float2* d_blob = nullptr;
    int device = -1;
};

namespace nm {

// Queues a kernel; an error is what hipGetLastError returns next.  (The launch itself: the <<< >>> form first pushes and
// pops its configuration, 0.3 of the 2.8 us of host time that a launch takes.)
template <typename... P, size_t... I>
inline void queue_packed(void (*kern)(P...), dim3 grid, dim3 block, size_t shmem, hipStream_t s, std::tuple<P...>& args, std::index_sequence<I...>)
{
    void* ptrs[] = {static_cast<void*>(&std::get<I>(args))...};
    (void)hipLaunchKernel(reinterpret_cast<const void*>(kern), grid, block, ptrs, shmem, s);
}
template <typename... P, typename... A>
inline void queue_kernel(void (*kern)(P...), dim3 grid, dim3 block, size_t shmem, hipStream_t s, const A&... a)
{
    std::tuple<P...> args(static_cast<P>(a)...);
    queue_packed(kern, grid, block, shmem, s, args, std::index_sequence_for<P...>{});
}

void set_error(const char* fmt, ...);
int32_t fail(int32_t code, const char* fmt, ...);
int32_t check_hip(hipError_t e, const char* what);

// Validates idx and fills dt.  Returns NM_OK or an error (message set).
// two_level: also hand out the two-level form of a table built with NM_TABLE_COMPACT (only kernels
// that look tables up in two steps ask for it; everything else works on the expanded form).
int32_t get_dev_table(const nm_tables* t, int32_t idx, DevTable* dt, const char* what, bool two_level = false);

// Bounds of the values table idx (validated by get_dev_table before) takes for x in [xmin, xmax].
void table_value_bounds(const nm_tables* t, int32_t idx, double xmin, double xmax, double* vmin, double* vmax);

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// ---- generic (possibly batched, strided) GEMM launcher used by the public entry points --------
struct GemmArgs {
    int M = 0, N = 0, K = 0;
    const int8_t* A = nullptr; long lda = 0;
    const int8_t* W = nullptr; long ldw = 0;
    int w_is_kn = 0;  // 0: W is [N, K] (K contiguous); 1: W is [K, N] (N contiguous)
    // batching: grid.y = outer_count * inner_count problems
    int outer_count = 1, inner_count = 1;
    long a_outer = 0, a_inner = 0, w_outer = 0, w_inner = 0, o_outer = 0, o_inner = 0;
    const float* bias = nullptr;
    const float* alpha_vec = nullptr;
    float alpha = 1.0f;
    const int8_t* resid = nullptr;
    float resid_scale = 0.0f;
    int has_table = 0;
    DevTable table{};
    float out_inv_scale = 1.0f;
    const float* out_inv_scale_vec = nullptr;
    int split_cols = 0;  // > 0: out scale of column n is inv3[n / split_cols]
    float inv3[3] = {1.0f, 1.0f, 1.0f};
    long ldo = 0;  // row stride of resid and of every output
    int8_t* out_q = nullptr;
    float* out_f32 = nullptr;
    int32_t* out_acc = nullptr;
    uint16_t* dbg_seg = nullptr;
    // LayerNorm-PWL of the fp32 result, folded into the kernel when the shape allows it (else the
    // caller runs the row kernel): gamma / beta [N], rsqrt table, int8 and / or fp32 output [M, N]
    int ln = 0;
    const float* ln_gamma = nullptr;
    const float* ln_beta = nullptr;
    float ln_eps = 0.0f, ln_inv_scale = 1.0f;
    DevTable ln_table{};
    int8_t* ln_out_q = nullptr;
    float* ln_out_f32 = nullptr;
    // conv != 0: A is an NHWC image [B, cH, cW, cCin] and row m = (b, ho, wo) of the matrix is
    // gathered from it (K = kh * cKw * cCin, tap major); M = B * cHo * cWo
    int conv = 0;
    int cH = 0, cW = 0, cCin = 0, cKw = 0, cStride = 1, cPad = 0, cHo = 0, cWo = 0;
};

int32_t launch_gemm(const GemmArgs& g, hipStream_t stream);
// Two gathered products, neither of which reads or writes what the other writes, as one launch; *done = false where they are not for it.
int32_t launch_conv_pair(const GemmArgs& a, const GemmArgs& b, hipStream_t stream, bool* done);
// A 1x1 convolution (rows of K, a shortcut) and the one that reads its result (b.A == a.out_q), nothing else of which is what the other
// touches, as one launch; *done = false where they are not for it.
int32_t launch_conv_chain(const GemmArgs& a, const GemmArgs& b, hipStream_t stream, bool* done);
// A 3x3 convolution whose filter fits LDS (g.conv, operands that the gathered loader takes); *done = false where it is not for that kernel.
int32_t launch_conv_taps(const GemmArgs& g, hipStream_t stream, bool* done);
bool gemm_switched();   // one of the debug switches says which kernel products take
// True when launch_gemm would fold the LayerNorm described by g.ln_* into the GEMM kernel.
bool gemm_folds_layernorm(const GemmArgs& g);

// LayerNorm-PWL of M fp32 rows of K columns (the M and K of the product behind it), its int8 codes to out_q if given.
struct LnRows {
    const float* x = nullptr;
    const float* gamma = nullptr;
    const float* beta = nullptr;
    float eps = 0.0f, inv_scale = 1.0f;
    DevTable table{};
    int8_t* out_q = nullptr;
};
// That and a product of the codes as one kernel (g.A is not read); tile: of ln_gemm_tile.
bool ln_gemm_takes(const LnRows& n, const GemmArgs& g);
int32_t launch_ln_gemm(const LnRows& n, const GemmArgs& g, int tile, hipStream_t stream);

// The three attention steps as one kernel, for every shape fused_attention_covers accepts.
struct AttnArgs {
    const int8_t* qkv;
    int B, S, H, heads;
    float alpha_scores, inv_s_p, alpha_ctx, inv_s_ctx;
    const nm_tables* tables;
    int exp_idx, recip_idx;
    int8_t* ctx;
    int32_t* scores_out;
    int8_t* p_out;
};
bool fused_attention_covers(int S, int H, int heads);
int32_t launch_attention(const AttnArgs& a, const char* what, hipStream_t stream);
// That and the QKV projection g in front of it (a.qkv and g.out_q are not touched), where qkv_attention_takes; *done = false where the tables
// or the size are not for it.
bool qkv_attention_takes(const AttnArgs& a, const GemmArgs& g);
int32_t launch_qkv_attention(const AttnArgs& a, const GemmArgs& g, const char* what, hipStream_t stream, bool* done);

// Steps 5 to 9 of a layer (and step 1 of the next) as one kernel over blocks of rows; *done = false where it
// does not take the layer.
int32_t launch_encoder_block(const nm_layer_desc* d, const nm_layer_desc* next, const int8_t* ctx, const int8_t* x, int8_t* y_q,
                             float* y_f32, int8_t* qkv, hipStream_t stream, bool* done);

int32_t launch_softmax(const void* in, int32_t in_dtype, float alpha, int64_t rows, int32_t cols,
                       const DevTable& t_exp, const DevTable& t_recip, float out_inv_scale,
                       int8_t* out_q, float* out_f32, uint16_t* seg_exp, uint16_t* seg_recip,
                       hipStream_t stream);

int32_t launch_layernorm(const float* in, const float* gamma, const float* beta, float eps,
                         int64_t rows, int32_t cols, const DevTable& t, float out_inv_scale,
                         int8_t* out_q, float* out_f32, uint16_t* seg, hipStream_t stream);

int32_t launch_layernorm2(const float* in, const float* gamma, const float* beta, float eps,
                          int64_t rows, int32_t cols, const DevTable& t, const DevTable& t2, int two,
                          float out_inv_scale, int8_t* out_q, float* out_f32, uint16_t* seg, uint16_t* seg2,
                          hipStream_t stream);

}  // namespace nm
