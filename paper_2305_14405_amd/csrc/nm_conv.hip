// int8 convolution as a matrix product (paper Section 3.1: the matrix dimensions follow from the
// width, height and channel counts of the convolution), with the fused PWL epilogue of the GEMM,
// and the two pooling operators of a residual CNN.
//
// Three routes, chosen on the host:
//  * 1x1, stride 1, no padding: the NHWC activation tensor already IS the [B*H*W, Cin] matrix;
//  * Cin a multiple of 64 (every convolution of a ResNet-50 body): the streaming GEMM kernel
//    gathers the rows of the patch matrix straight from the image while loading its A operand
//    (no patch matrix in memory);
//  * anything else (the 3-channel stem, odd channel counts): a small kernel writes the patch
//    matrix [B*Ho*Wo, K16] (K rounded up to 64, zero filled) into the caller's workspace and the
//    GEMM runs on it.
#include <type_traits>

#include "nm_device.h"

namespace nm {

constexpr int kConvThreads = 256;

// Patch matrix: row m = (b, ho, wo), column k = (tap i, tap j, channel c), zeros in the padding
// and in the columns K .. K16-1 (K16: K rounded up to 64).  One thread writes 16 consecutive
// columns of one row.
__global__ __launch_bounds__(kConvThreads) void im2col_kernel(
    const int8_t* __restrict__ x, int H, int W, int Cin, int kw, int stride, int pad, int Ho, int Wo,
    int K, int K16, long rows, int8_t* __restrict__ out)
{
    const int chunks = K16 / 16;
    const long total = rows * chunks;
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
        const long m = idx / chunks;
        const int k0 = (int)(idx % chunks) * 16;
        const int wo = (int)(m % Wo), ho = (int)((m / Wo) % Ho);
        const long b = m / ((long)Wo * Ho);
        unsigned word[4] = {0, 0, 0, 0};
        // (tap row, tap column, channel) of column k0, then stepped along the 16 columns
        int c = k0 % Cin, tap = k0 / Cin;
        int ti = tap / kw, tj = tap % kw;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            int v = 0;
            if (k0 + e < K) {
                const int hi = ho * stride - pad + ti, wi = wo * stride - pad + tj;
                if ((unsigned)hi < (unsigned)H && (unsigned)wi < (unsigned)W)
                    v = x[((b * H + hi) * W + wi) * Cin + c];
            }
            word[e >> 2] |= (unsigned)(v & 0xff) << (8 * (e & 3));
            if (++c == Cin) { c = 0; if (++tj == kw) { tj = 0; ++ti; } }
        }
        *reinterpret_cast<v4i*>(out + m * K16 + k0) = v4i{(int)word[0], (int)word[1], (int)word[2], (int)word[3]};
    }
}

// Max pooling on int8 codes (exact, order-free); padding never takes part.  One thread per
// output position and 16 channels (C % 16 == 0, 16-byte loads).  A tap outside the image is taken from the nearest position
// inside, which lies in the same window, so all loads of a window (of a row of it where kK is 0: any size) are requested at once.  Codes are
// compared as pairs of 16-bit numbers: the word itself, whose odd bytes decide, and the word shifted by a byte for the even
// ones.  us, 64 images of 112 x 112 x 64, 3x3 with stride 2 (64 MB: 12.6 us at a copy's rate): 13.7, where one tap was waited for at a time and
// bytes compared singly 16.8; one image 2.2, was 3.9.
typedef short v2s __attribute__((ext_vector_type(2)));
template <int kK>
__global__ __launch_bounds__(kConvThreads) void maxpool16_kernel(
    const int8_t* __restrict__ x, int H, int W, int C, int k, int stride, int pad, int Ho, int Wo, FastDiv div_c, FastDiv div_wo, FastDiv div_ho,
    unsigned total, int8_t* __restrict__ y)
{
    const unsigned idx = blockIdx.x * kConvThreads + threadIdx.x;
    if (idx >= total) return;
    const unsigned m = quotient(idx, div_c), t = quotient(m, div_wo), b = quotient(t, div_ho);
    const int c = (int)(idx - m * (unsigned)(C / 16)), w0 = (int)(m - t * (unsigned)Wo) * stride - pad, h0 = (int)(t - b * (unsigned)Ho) * stride - pad;
    const int8_t* const img = x + (long)b * H * W * C + 16 * c;
    v2s odd[4], even[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) odd[q] = even[q] = v2s{-32768, -32768};
    auto take = [&](v4i w) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned u = (unsigned)w[q];   // (of a vector's element itself the cast takes the first)
            odd[q] = __builtin_elementwise_max(odd[q], __builtin_bit_cast(v2s, u));
            even[q] = __builtin_elementwise_max(even[q], __builtin_bit_cast(v2s, u << 8));
        }
    };
    const int pitch = W * C;   // (an image has less than 2^31 bytes: host)
    auto row = [&](int i) { return img + (unsigned)(min(max(h0 + i, 0), H - 1) * pitch); };
    auto tap = [&](const int8_t* r, int j) { return *reinterpret_cast<const v4i*>(r + (unsigned)(min(max(w0 + j, 0), W - 1) * C)); };
    if constexpr (kK > 0) {
        v4i w[kK * kK];
#pragma unroll
        for (int i = 0; i < kK; ++i)
#pragma unroll
            for (int j = 0; j < kK; ++j) w[i * kK + j] = tap(row(i), j);
#pragma unroll
        for (int e = 0; e < kK * kK; ++e) take(w[e]);
    } else {
        for (int i = 0; i < k; ++i) {
            const int8_t* const r = row(i);
            for (int j = 0; j < k; ++j) take(tap(r, j));
        }
    }
    v4i o;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        o[q] = (int)__builtin_amdgcn_perm(__builtin_bit_cast(unsigned, odd[q]), __builtin_bit_cast(unsigned, even[q]), 0x07030501u);
    *reinterpret_cast<v4i*>(y + 16 * (long)idx) = o;
}

// The same with four channels (C % 4 == 0) or one channel per thread.
template <bool kVec>
__global__ __launch_bounds__(kConvThreads) void maxpool_kernel(
    const int8_t* __restrict__ x, int H, int W, int C, int k, int stride, int pad, int Ho, int Wo,
    long total, int8_t* __restrict__ y)
{
    const int cg = kVec ? C / 4 : C;
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
        const int c = (int)(idx % cg);
        const long m = idx / cg;
        const int wo = (int)(m % Wo), ho = (int)((m / Wo) % Ho);
        const long b = m / ((long)Wo * Ho);
        int best[4] = {-128, -128, -128, -128};
        for (int i = 0; i < k; ++i) {
            const int hi = ho * stride - pad + i;
            if ((unsigned)hi >= (unsigned)H) continue;
            for (int j = 0; j < k; ++j) {
                const int wi = wo * stride - pad + j;
                if ((unsigned)wi >= (unsigned)W) continue;
                const long off = ((b * H + hi) * W + wi) * C;
                if (kVec) {
                    const unsigned w = *reinterpret_cast<const unsigned*>(x + off + 4 * c);
#pragma unroll
                    for (int e = 0; e < 4; ++e) best[e] = max(best[e], (int)(int8_t)(w >> (8 * e)));
                } else {
                    best[0] = max(best[0], (int)x[off + c]);
                }
            }
        }
        if (kVec) *reinterpret_cast<unsigned*>(y + m * C + 4 * c) = pack4(best[0], best[1], best[2], best[3]);
        else y[m * C + c] = (int8_t)best[0];
    }
}

// Global average pooling: exact int32 sum over the positions, one fp32 multiply, requantise.
// kVec (C a multiple of 4, 4-byte aligned tensors): a thread owns four neighbouring channels of an
// image and reads them as one word per position, eight positions in flight; otherwise one channel
// per thread, byte by byte.
template <bool kVec>
__global__ __launch_bounds__(kConvThreads) void avgpool_kernel(
    const int8_t* __restrict__ x, int B, int HW, int C, float alpha, float out_inv_scale,
    int8_t* __restrict__ out_q, float* __restrict__ out_f32)
{
    if (kVec) {
        const int C4 = C / 4;
        const long total = (long)B * C4;
        for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
            const int c4 = (int)(idx % C4);
            const long b = idx / C4;
            const int8_t* src = x + b * HW * (long)C + 4 * c4;
            int acc[4] = {0, 0, 0, 0};
            int p = 0;
            for (; p + 8 <= HW; p += 8) {
                int w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) w[u] = *reinterpret_cast<const int*>(src + (long)(p + u) * C);
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] += (int)(int8_t)(w[u] >> (8 * e));
            }
            for (; p < HW; ++p) {
                const int w = *reinterpret_cast<const int*>(src + (long)p * C);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += (int)(int8_t)(w >> (8 * e));
            }
            float v[4];
            int q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = (float)acc[e] * alpha;
                q[e] = requant(v[e], out_inv_scale);
            }
            if (out_f32) *reinterpret_cast<v4f*>(out_f32 + 4 * idx) = v4f{v[0], v[1], v[2], v[3]};
            if (out_q) *reinterpret_cast<unsigned*>(out_q + 4 * idx) = pack4(q[0], q[1], q[2], q[3]);
        }
        return;
    }
    const long total = (long)B * C;
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
        const int c = (int)(idx % C);
        const long b = idx / C;
        int acc = 0;
        for (int p = 0; p < HW; ++p) acc += (int)x[(b * HW + p) * C + c];
        const float v = (float)acc * alpha;
        if (out_f32) out_f32[idx] = v;
        if (out_q) out_q[idx] = (int8_t)requant(v, out_inv_scale);
    }
}

// ---------------------------------------------------------------------------------------------
// Direct convolution for images with at most four channels (the stem of a CNN: 7x7, stride 2,
// three channels).  A patch matrix would be 50 times the image; instead a workgroup stages the
// part of the image its 16 x 16 output positions need in LDS, one 4-byte pixel per position
// (missing channels and everything outside the image are zero), and the filter as rows of 32
// bytes per filter row (kw <= 8 pixels of 4 bytes, zero filled).  One MFMA k-step is then one
// filter row: the operand bytes of output position (ho, wo) are 32 consecutive LDS bytes starting
// at pixel (ho*stride + i, wo*stride); bytes beyond the kw-th pixel meet zero filter bytes.
// Accumulators and epilogue arithmetic are those of the matrix product (exact integers, the same
// fp32 operations), so the result is bit-identical to the other routes.
// A wavefront owns 4 rows x 16 columns of positions and all (up to 64) output channels.
// ---------------------------------------------------------------------------------------------
struct StemParams {
    const int8_t* x; const int8_t* w;   // w: the packed filter [64][kh][32] (stem_pack_filter_kernel), kPack: the filter itself
    const float* bias; const float* alpha_vec;
    float alpha, out_inv_scale;
    int has_table, relu;
    DevTable table;
    int B, H, W, Cin, Cout, kh, kw, stride, pad, Ho, Wo;
    int prow, pitch;         // staged image patch: rows, bytes per row
    int front;               // LDS in front of the column vectors: patch and filter, or the output rows over them
    int8_t* out_q;
};

// Packs the filter [Cout][kh][kw][Cin] into [64][kh][8 pixels of 4 bytes] (zero filled), once per
// call, so that every workgroup of the convolution copies it with wide loads.
__global__ __launch_bounds__(256) void stem_pack_filter_kernel(const int8_t* __restrict__ w, int Cout, int kh,
                                                               int kw, int Cin, int8_t* __restrict__ out)
{
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < 64 * kh * 8; idx += gridDim.x * blockDim.x) {
        const int j = idx % 8, i = (idx / 8) % kh, n = idx / (8 * kh);
        unsigned px = 0;
        if (n < Cout && j < kw) {
            const int8_t* src = w + (((long)n * kh + i) * kw + j) * Cin;
            for (int ch = 0; ch < Cin; ++ch) px |= (unsigned)(uint8_t)src[ch] << (8 * ch);
        }
        *reinterpret_cast<unsigned*>(out + (n * kh + i) * 32 + 4 * j) = px;
    }
}

typedef unsigned v2u __attribute__((ext_vector_type(2)));
constexpr int kStemRow = 72;   // bytes of an output position's row in LDS
__device__ __forceinline__ v4i stem_chunk(const int8_t* row)   // 16 bytes of such a row, eight-byte aligned
{
    const v2u lo = *reinterpret_cast<const v2u*>(row), hi = *reinterpret_cast<const v2u*>(row + 8);
    return v4i{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
}

// kPack: every workgroup packs the filter for itself (14 words a thread for 7 rows), which a few workgroups do in less time than a launch takes: one
// image of 224 x 224 8.0 -> 6.9 us, 16 13.7 -> 13.3.  Where they are many it is the larger part of their instructions (24: 17.1 either way).
constexpr long kStemPackers = 1024;
template <bool kPack>
__global__ __launch_bounds__(256, 4) void stem_conv_kernel(StemParams p)
{
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    int8_t* sX = smem;                                   // [prow][pitch]
    int8_t* sW = smem + p.prow * p.pitch;                // [64][kh][32]
    int8_t* sO = smem;                                   // [4 wavefronts][64 positions][kStemRow], over both once they have been read
    float* s_cols = reinterpret_cast<float*>(smem + p.front);   // scale | bias, 64 each
    float2* s_kb = reinterpret_cast<float2*>(s_cols + 128);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_w = (p.Wo + 15) / 16;
    const int ho0 = (blockIdx.x / tiles_w) * 16, wo0 = (blockIdx.x % tiles_w) * 16;
    const long b = blockIdx.y;
    const int hi0 = ho0 * p.stride - p.pad, wi0 = wo0 * p.stride - p.pad;

    // filter, already packed as [n][i][8 pixels of 4 bytes]: direct loads
    if (!kPack)
        for (int i = wave; i < 2 * p.kh; i += 4) dma16(p.w + 1024 * i + 16 * lane, (unsigned)(uintptr_t)sW + 1024 * i);
    // scale (first wavefront) and bias (second): requested here, written behind the patch
    const float* const cols = wave == 0 ? p.alpha_vec : p.bias;
    float col_value = wave == 0 ? p.alpha : 0.0f;
    if (wave < 2 && lane < p.Cout && cols) col_value = cols[lane];
    // Image patch: one dword per pixel, read as one unaligned word and shifted where that word would pass the
    // end of the tensor.  (Pixels behind the patch's last column fill the rows up to their pitch: the last
    // positions' 32-byte windows reach them, with zero filter bytes.)  A wavefront takes whole rows, a lane one column:
    // the row's address and whether it is inside are scalar work, a pixel few vector instructions.  On 64 images of
    // 224 x 224 and on one, us: pixels numbered through, one accumulator set in the other half of the register file
    // (three workgroups to a CU) 34.6 and 7.5; this with four workgroups 35.0 and 7.4 (820 vector instructions a
    // wavefront instead of 985); with the column vectors requested in front instead of waited for 31.8 and 6.7.  Vector
    // instructions issue in 64 % of the cycles; ten rows at a time instead of five need 187 registers and take 45.8.
    {
        constexpr int U = 5;
        const int npx = p.pitch >> 2, row0 = __builtin_amdgcn_readfirstlane(wave);
        const long row_bytes = (long)p.W * p.Cin;
        const int8_t* const img = p.x + b * p.H * row_bytes;
        const int8_t* const last = p.x + (long)p.B * p.H * row_bytes - 4;
        // Columns 64 .. 67 (stride 4 alone has them; a patch has at most 64 rows: host): a pixel per thread, requested in front.
        // As a second pass of the loop below they cost it as much again as the 64 columns: 8 images of 224 x 224 with 3x3
        // filters 11.1 us, now 8.7 (64 images 20.9, now 15.8).
        const int er = tid >> 2, ec = 64 + (tid & 3);
        const bool more = npx > 64;
        unsigned epx = 0, eshift = 0, emask = 0;
        if (more) {
            const int hi = hi0 + er, wi = wi0 + ec;
            const bool inside = er < p.prow && (unsigned)hi < (unsigned)p.H && (unsigned)wi < (unsigned)p.W;
            const int8_t* const a = inside ? img + hi * row_bytes + (long)wi * p.Cin : img;
            const int8_t* const from = a < last ? a : last;
            __builtin_memcpy(&epx, from, 4);
            eshift = 8 * (unsigned)(a - from);
            emask = inside ? 0xffffffffu >> (32 - 8 * p.Cin) : 0u;
        }
        const int wi = wi0 + lane;
        const bool col = (unsigned)wi < (unsigned)p.W;
        const int from_col = min(max(wi0, 0), p.W - 1);   // lanes count from here
        const unsigned off = col ? (unsigned)(wi - from_col) * (unsigned)p.Cin : 0u;
        const unsigned mask = col ? 0xffffffffu >> (32 - 8 * p.Cin) : 0u;
        for (int r0 = row0; r0 < p.prow; r0 += 4 * U) {
            unsigned px[U], shift[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int hi = hi0 + r0 + 4 * u;
                const int8_t* const a = img + ((unsigned)hi < (unsigned)p.H ? hi : 0) * row_bytes + (long)from_col * p.Cin;
                const long left = last - a;   // bytes to the last whole word; -3 at least
                const int high = (int)(left >> 32);
                const unsigned limit = high < 0 ? 0u : high > 0 ? 0x7fffffffu : (unsigned)left;
                const unsigned at = off + (high < 0 ? (unsigned)-(int)left : 0u), from = min(at, limit);
                __builtin_memcpy(&px[u], (high < 0 ? last : a) + from, 4);
                shift[u] = 8 * (at - from);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = r0 + 4 * u;
                if (r >= p.prow) break;
                const unsigned m = (unsigned)(hi0 + r) < (unsigned)p.H ? mask : 0u;
                if (lane < npx) *reinterpret_cast<unsigned*>(sX + r * p.pitch + 4 * lane) = (px[u] >> shift[u]) & m;
            }
        }
        if (more && er < p.prow && ec < npx) *reinterpret_cast<unsigned*>(sX + er * p.pitch + 4 * ec) = (epx >> eshift) & emask;
    }
    if (kPack) {
        // word j of row r = (channel, filter row) is the filter row's j-th pixel, read as one unaligned word and shifted at the tensor's end
        const int rows = p.Cout * p.kh, j = tid & 7, last = rows * p.kw * p.Cin - 4;
        const unsigned mask = j < p.kw ? 0xffffffffu >> (32 - 8 * p.Cin) : 0u;
        constexpr int U = 7;
        for (int i0 = 0; i0 < 2 * p.kh; i0 += U) {
            unsigned px[U], shift[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = min(32 * (i0 + u) + (tid >> 3), rows - 1), at = (r * p.kw + min(j, p.kw - 1)) * p.Cin, from = min(at, last);
                __builtin_memcpy(&px[u], p.w + from, 4);
                shift[u] = 8 * (unsigned)(at - from);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = 32 * (i0 + u) + (tid >> 3);
                if (i0 + u < 2 * p.kh) *reinterpret_cast<unsigned*>(sW + 32 * r + 4 * j) = r < rows ? (px[u] >> shift[u]) & mask : 0u;
            }
        }
    }
    if (wave < 2) s_cols[tid] = lane < p.Cout ? col_value : 0.0f;
    if (p.has_table && !p.table.two_seg) stage_table(s_kb, p.table);
    wait_vmcnt<0>();
    __syncthreads();

    // lane (m, half): position m of a 32-position block; block t covers wavefront rows 2t, 2t+1
    const int fr = lane & 31, half = lane >> 5;
    v16i acc[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][j][v] = 0;
    int offA[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int pr = wave * 4 + 2 * t + (fr >> 4), pc = fr & 15;   // position inside the 16 x 16 tile
        offA[t] = pr * p.stride * p.pitch + pc * p.stride * 4 + 16 * half;
    }
    for (int i = 0; i < p.kh; ++i) {
        v4i fa[2], fw[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int8_t* a = sX + offA[t] + i * p.pitch;   // 4-byte aligned
            const unsigned* a4 = reinterpret_cast<const unsigned*>(a);
            fa[t] = v4i{(int)a4[0], (int)a4[1], (int)a4[2], (int)a4[3]};
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
            fw[j] = *reinterpret_cast<const v4i*>(sW + ((32 * j + fr) * p.kh + i) * 32 + 16 * half);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[t][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[j], fa[t], acc[t][j], 0, 0, 0);
    }

    __syncthreads();   // the output rows lie over the operands
    // epilogue: lane (m, half) holds, per group g of four registers, channels 32j + 8g + 4half .. +3; the halves of two
    // groups change lanes, so that a lane writes eight consecutive channels.  Rows of 72 bytes: 32 lanes' eight bytes
    // fall on all 64 banks once.
    int8_t* patch = sO + wave * (64 * kStemRow);
    // (three times: a table of two segments is evaluated with a compare instead of index and gather, and a ReLU
    // by clamping the code)
    auto finish = [&](auto form_c) {
        constexpr bool kTwoSeg = decltype(form_c)::value == 1, kRelu = decltype(form_c)::value == 2;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4f sc[2], bi[2];
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    sc[g] = *reinterpret_cast<const v4f*>(s_cols + 32 * j + 16 * h + 8 * g + 4 * half);
                    bi[g] = *reinterpret_cast<const v4f*>(s_cols + 64 + 32 * j + 16 * h + 8 * g + 4 * half);
                }
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    unsigned w[2] = {0, 0};
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        int q[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float v = __builtin_fmaf((float)acc[t][j][8 * h + 4 * g + e], sc[g][e], bi[g][e]);
                            if (kRelu) { w[g] = relu_requant(v, p.out_inv_scale, e, w[g]); continue; }
                            if (kTwoSeg) v = pwl_eval_two_segments(v, p.table);
                            else if (p.has_table) { int sg; v = pwl_eval(v, p.table, s_kb, sg); }
                            q[e] = requant(v, p.out_inv_scale);
                        }
                        if (!kRelu) w[g] = pack4(q[0], q[1], q[2], q[3]);
                    }
                    const auto x = __builtin_amdgcn_permlane32_swap(w[0], w[1], false, false);
                    *reinterpret_cast<v2u*>(patch + (32 * t + fr) * kStemRow + 32 * j + 16 * h + 8 * half) = v2u{x[0], x[1]};
                }
            }
    };
    if (p.relu && __all(relu_finite(s_cols[lane], s_cols[64 + lane]))) finish(std::integral_constant<int, 2>{});
    else if (p.has_table && p.table.two_seg) finish(std::integral_constant<int, 1>{});
    else finish(std::integral_constant<int, 0>{});
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // 16-byte stores: position rows of Cout bytes are contiguous along wo
    const int chunks = p.Cout / 16;
    for (int c = lane; c < 64 * chunks; c += 64) {
        const int pos = c / chunks, cc = c % chunks;
        const int ho = ho0 + wave * 4 + (pos >> 4), wo = wo0 + (pos & 15);
        if (ho < p.Ho && wo < p.Wo)
            *reinterpret_cast<v4i*>(p.out_q + ((b * p.Ho + ho) * p.Wo + wo) * p.Cout + 16 * cc) =
                stem_chunk(patch + pos * kStemRow + 16 * cc);
    }
}

static int grid_for(long units)
{
    long b = (units + kConvThreads - 1) / kConvThreads;
    if (b > 256L * 32) b = 256L * 32;
    return (int)(b < 1 ? 1 : b);
}

struct ConvPlan {
    int Ho, Wo, K, K16;
    long M;
    int route;  // 0: plain matrix, 1: gathered operand, 2: patch matrix in the workspace, 3: direct (few channels)
    size_t ws_bytes;
};

static int32_t plan_conv(const nm_conv_desc* d, const char* what, ConvPlan* pl)
{
    if (!d) return fail(NM_ERR_INVALID_ARG, "%s: desc is NULL", what);
    if (d->B < 0 || d->H < 1 || d->W < 1 || d->Cin < 1 || d->Cout < 1 || d->kh < 1 || d->kw < 1 ||
        d->stride < 1 || d->pad < 0)
        return fail(NM_ERR_INVALID_ARG, "%s: bad convolution geometry", what);
    if (d->H + 2 * d->pad < d->kh || d->W + 2 * d->pad < d->kw)
        return fail(NM_ERR_INVALID_ARG, "%s: filter larger than the padded image", what);
    pl->Ho = (d->H + 2 * d->pad - d->kh) / d->stride + 1;
    pl->Wo = (d->W + 2 * d->pad - d->kw) / d->stride + 1;
    const int64_t K = (int64_t)d->kh * d->kw * d->Cin;
    const int64_t M = (int64_t)d->B * pl->Ho * pl->Wo;
    if (K > 65536) return fail(NM_ERR_UNSUPPORTED, "%s: kh*kw*Cin %lld > 65536", what, (long long)K);
    if (M * d->Cout >= (1LL << 31) || M * K >= (1LL << 40) || (int64_t)d->B * d->H * d->W * d->Cin >= (1LL << 40))
        return fail(NM_ERR_UNSUPPORTED, "%s: tensor too large", what);
    if (M >= (1LL << 31)) return fail(NM_ERR_UNSUPPORTED, "%s: more than 2^31 output positions", what);
    pl->K = (int)K;
    pl->K16 = (int)((K + 63) / 64 * 64);  // whole 64-byte k-slices: the streaming GEMM runs on the patch matrix
    pl->M = (long)M;
    const bool plain = d->kh == 1 && d->kw == 1 && d->stride == 1 && d->pad == 0;
    const bool gather = d->Cin % 64 == 0 && aligned(d->x, 16) && aligned(d->w, 16) &&
                        (int64_t)d->H * d->W * d->Cin < (1LL << 31);   // 32-bit offsets inside one image
    // direct kernel: few input channels (read as words, so at least one word in all), a filter row fits 32 bytes,
    // int8 output only
    const bool direct = !plain && d->Cin <= 4 && d->kw <= 8 && d->Cout <= 64 && d->Cout % 16 == 0 && d->out_q &&
                        !d->out_f32 && !d->dbg_acc && !d->resid && aligned(d->out_q, 16) &&
                        15 * d->stride + d->kh <= 64 && d->B <= 65535 && (int64_t)d->B * d->H * d->W * d->Cin >= 4;
    pl->route = plain ? 0 : gather ? 1 : direct ? 3 : 2;
    pl->ws_bytes = pl->route == 2 ? (size_t)M * pl->K16 + (size_t)d->Cout * pl->K16
                 : pl->route == 3 ? (size_t)64 * d->kh * 32 : 0;   // patch matrix + filter rows | packed filter
    return NM_OK;
}

// Copies the [Cout, K] filter matrix into rows of K16 bytes (zero tail) for the patch-matrix route.
__global__ __launch_bounds__(kConvThreads) void pad_rows_kernel(const int8_t* __restrict__ w, int rows, int K,
                                                                 int K16, int8_t* __restrict__ out)
{
    const long total = (long)rows * K16;
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (long)gridDim.x * blockDim.x) {
        const int k = (int)(idx % K16);
        out[idx] = k < K ? w[(idx / K16) * K + k] : (int8_t)0;
    }
}

// The product behind a convolution, without its A operand.
static int32_t conv_args(const nm_conv_desc* d, const ConvPlan& pl, GemmArgs* out)
{
    GemmArgs& g = *out;
    if (d->table_idx >= 0) {
        const int32_t rc = get_dev_table(d->tables, d->table_idx, &g.table, "nm_conv2d_pwl");
        if (rc) return rc;
        g.has_table = 1;
    }
    g.M = (int)pl.M; g.N = d->Cout; g.K = pl.K;
    g.W = d->w; g.ldw = pl.K;
    g.bias = d->bias; g.alpha_vec = d->alpha_vec; g.alpha = d->alpha;
    g.resid = d->resid; g.resid_scale = d->resid_scale;
    g.out_inv_scale = d->out_inv_scale;
    g.ldo = d->Cout;
    g.out_q = d->out_q; g.out_f32 = d->out_f32; g.out_acc = d->dbg_acc;
    return NM_OK;
}
// ... whose rows are gathered from the image.
static void gather_args(const nm_conv_desc* d, const ConvPlan& pl, GemmArgs* g)
{
    g->A = d->x; g->lda = d->Cin;
    g->conv = 1;
    g->cH = d->H; g->cW = d->W; g->cCin = d->Cin; g->cKw = d->kw; g->cStride = d->stride; g->cPad = d->pad;
    g->cHo = pl.Ho; g->cWo = pl.Wo;
}

static bool apart(const void* p, size_t n, const void* q, size_t m)
{
    const uintptr_t u = reinterpret_cast<uintptr_t>(p), v = reinterpret_cast<uintptr_t>(q);
    return !p || !q || u + n <= v || v + m <= u;
}
// Whether n bytes at `out` are apart from all that a step reads (g: its product, whose A is d->x) and writes.
static bool apart_from_step(const void* out, size_t n, const nm_conv_desc* d, const GemmArgs& g)
{
    const size_t cols = (size_t)g.N * sizeof(float), outputs = (size_t)g.M * g.N;
    return apart(out, n, d->x, (size_t)d->B * d->H * d->W * d->Cin) && apart(out, n, d->w, (size_t)g.N * g.K) && apart(out, n, d->bias, cols) &&
           apart(out, n, d->alpha_vec, cols) && apart(out, n, d->resid, outputs) && apart(out, n, d->out_q, outputs);
}

// Two steps of a network as one launch where both are small convolutions and neither touches what the other writes.
static int32_t conv_pair(const nm_conv_desc* a, const nm_conv_desc* b, hipStream_t stream, bool* done)
{
    *done = false;
    const nm_conv_desc* const d[2] = {a, b};
    GemmArgs g[2];
    for (int i = 0; i < 2; ++i) {
        ConvPlan pl;
        if (!d[i]->out_q || d[i]->out_f32 || d[i]->dbg_acc || d[i]->resid || !d[i]->x || !d[i]->w || d[i]->Cin % 64 != 0) return NM_OK;
        if (plan_conv(d[i], "nm_conv2d_pwl", &pl) || pl.route > 1 || pl.M == 0 || conv_args(d[i], pl, &g[i])) return NM_OK;   // (the step itself reports it)
        gather_args(d[i], pl, &g[i]);
    }
    for (int i = 0; i < 2; ++i)
        if (!apart_from_step(g[i].out_q, (size_t)g[i].M * g[i].N, d[1 - i], g[1 - i])) return NM_OK;
    return launch_conv_pair(g[0], g[1], stream, done);
}

// A 1x1 convolution with a shortcut and the 1x1 one that reads its result as one launch, where nothing else that either reads or writes
// is what the other writes.
static int32_t conv_chain(const nm_conv_desc* a, const nm_conv_desc* b, hipStream_t stream, bool* done)
{
    *done = false;
    if (!a->resid || b->resid || !a->out_q || b->x != a->out_q) return NM_OK;
    const nm_conv_desc* const d[2] = {a, b};
    GemmArgs g[2];
    for (int i = 0; i < 2; ++i) {
        ConvPlan pl;
        if (!d[i]->out_q || d[i]->out_f32 || d[i]->dbg_acc || !d[i]->x || !d[i]->w) return NM_OK;
        if (plan_conv(d[i], "nm_conv2d_pwl", &pl) || pl.route != 0 || pl.M == 0 || conv_args(d[i], pl, &g[i])) return NM_OK;   // (the step itself reports it)
        g[i].A = d[i]->x; g[i].lda = d[i]->Cin;
    }
    if (g[0].M != g[1].M || g[0].N != g[1].K) return NM_OK;
    const size_t n0 = (size_t)g[0].M * g[0].N, n1 = (size_t)g[1].M * g[1].N, cols0 = (size_t)g[0].N * sizeof(float), cols1 = (size_t)g[1].N * sizeof(float);
    if (!apart_from_step(g[1].out_q, n1, a, g[0]) || !apart(g[0].out_q, n0, a->x, (size_t)g[0].M * g[0].K) || !apart(g[0].out_q, n0, a->w, (size_t)g[0].N * g[0].K) ||
        !apart(g[0].out_q, n0, a->bias, cols0) || !apart(g[0].out_q, n0, a->alpha_vec, cols0) || !apart(g[0].out_q, n0, a->resid, n0) ||
        !apart(g[0].out_q, n0, b->w, (size_t)g[1].N * g[1].K) || !apart(g[0].out_q, n0, b->bias, cols1) || !apart(g[0].out_q, n0, b->alpha_vec, cols1) ||
        !apart(g[1].out_q, n1, b->w, (size_t)g[1].N * g[1].K) || !apart(g[1].out_q, n1, b->bias, cols1) || !apart(g[1].out_q, n1, b->alpha_vec, cols1))
        return NM_OK;
    return launch_conv_chain(g[0], g[1], stream, done);
}

}  // namespace nm

using namespace nm;

extern "C" {

int32_t nm_conv2d_workspace(const nm_conv_desc* d, size_t* bytes)
{
    ConvPlan pl;
    int32_t rc = plan_conv(d, "nm_conv2d_workspace", &pl);
    if (rc) return rc;
    if (!bytes) return fail(NM_ERR_INVALID_ARG, "nm_conv2d_workspace: bytes is NULL");
    *bytes = pl.ws_bytes;
    return NM_OK;
}

int32_t nm_conv2d_pwl(const nm_conv_desc* d, void* ws, size_t ws_bytes, void* stream_)
{
    ConvPlan pl;
    int32_t rc = plan_conv(d, "nm_conv2d_pwl", &pl);
    if (rc) return rc;
    if (!d->out_q && !d->out_f32 && !d->dbg_acc) return fail(NM_ERR_INVALID_ARG, "nm_conv2d_pwl: no output");
    GemmArgs g;
    if ((rc = conv_args(d, pl, &g))) return rc;
    if (pl.M == 0) return NM_OK;  // an empty batch may come with NULL pointers
    if (!d->x || !d->w) return fail(NM_ERR_INVALID_ARG, "nm_conv2d_pwl: x or w is NULL");
    hipStream_t stream = (hipStream_t)stream_;
    if (pl.route == 3) {
        if (!ws) return fail(NM_ERR_WORKSPACE, "nm_conv2d_pwl: workspace is NULL");
        if (!aligned(ws, 256)) return fail(NM_ERR_WORKSPACE, "nm_conv2d_pwl: workspace not 256-byte aligned");
        if (ws_bytes < pl.ws_bytes)
            return fail(NM_ERR_WORKSPACE, "nm_conv2d_pwl: workspace %zu bytes < %zu needed", ws_bytes, pl.ws_bytes);
        const dim3 grid(((pl.Ho + 15) / 16) * ((pl.Wo + 15) / 16), d->B);
        const bool pack = (long)grid.x * d->B <= kStemPackers;
        if (!pack)
            queue_kernel(stem_pack_filter_kernel, dim3((64 * d->kh * 8 + 255) / 256), dim3(256), 0, stream, d->w,
                         d->Cout, d->kh, d->kw, d->Cin, static_cast<int8_t*>(ws));
        StemParams sp{};
        sp.x = d->x; sp.w = pack ? d->w : static_cast<const int8_t*>(ws); sp.bias = d->bias; sp.alpha_vec = d->alpha_vec; sp.alpha = d->alpha;
        sp.out_inv_scale = d->out_inv_scale; sp.has_table = g.has_table; sp.table = g.table;
        sp.relu = g.has_table && relu_codes(g.table, d->out_inv_scale, 0.0f);
        sp.B = d->B; sp.H = d->H; sp.W = d->W; sp.Cin = d->Cin; sp.Cout = d->Cout; sp.kh = d->kh; sp.kw = d->kw;
        sp.stride = d->stride; sp.pad = d->pad; sp.Ho = pl.Ho; sp.Wo = pl.Wo;
        sp.prow = 15 * d->stride + d->kh;
        // a position's window is 32 bytes from its first pixel: the last position's reaches 8 pixels
        sp.pitch = ((15 * d->stride + 8) * 4 + 15) / 16 * 16;
        sp.out_q = d->out_q;
        const size_t operands = (size_t)sp.prow * sp.pitch + 64 * (size_t)d->kh * 32, rows = 4 * 64 * kStemRow;
        const size_t behind = 128 * sizeof(float) + (g.has_table ? sizeof(float2) * (size_t)g.table.nseg : 0);
        if (operands + rows + behind > 64 * 1024)
            return fail(NM_ERR_UNSUPPORTED, "nm_conv2d_pwl: direct route needs %zu bytes of LDS", operands + rows + behind);
        sp.front = (int)(operands > rows ? operands : rows);
        const size_t shmem = sp.front + behind;
        queue_kernel(pack ? stem_conv_kernel<true> : stem_conv_kernel<false>, grid, dim3(256), shmem, stream, sp);
        return check_hip(hipGetLastError(), "nm_conv2d_pwl direct launch");
    }
    if (pl.route == 0) {
        g.A = d->x; g.lda = d->Cin;
    } else if (pl.route == 1) {
        gather_args(d, pl, &g);
        bool done = false;
        if ((rc = launch_conv_taps(g, stream, &done)) || done) return rc;
    } else {
        if (!ws) return fail(NM_ERR_WORKSPACE, "nm_conv2d_pwl: workspace is NULL");
        if (!aligned(ws, 256)) return fail(NM_ERR_WORKSPACE, "nm_conv2d_pwl: workspace not 256-byte aligned");
        if (ws_bytes < pl.ws_bytes)
            return fail(NM_ERR_WORKSPACE, "nm_conv2d_pwl: workspace %zu bytes < %zu needed", ws_bytes, pl.ws_bytes);
        int8_t* patches = static_cast<int8_t*>(ws);
        int8_t* wpad = patches + (size_t)pl.M * pl.K16;
        queue_kernel(im2col_kernel, dim3(grid_for(pl.M * (pl.K16 / 16))), dim3(kConvThreads), 0, stream,
                           d->x, d->H, d->W, d->Cin, d->kw, d->stride, d->pad, pl.Ho, pl.Wo, pl.K, pl.K16, pl.M,
                           patches);
        queue_kernel(pad_rows_kernel, dim3(grid_for((long)d->Cout * pl.K16)), dim3(kConvThreads), 0, stream,
                           d->w, d->Cout, pl.K, pl.K16, wpad);
        if ((rc = check_hip(hipGetLastError(), "nm_conv2d_pwl patch matrix launch"))) return rc;
        g.A = patches; g.lda = pl.K16;
        g.W = wpad; g.ldw = pl.K16;
        g.K = pl.K16;
    }
    return launch_gemm(g, stream);
}

int32_t nm_maxpool_i8(const int8_t* x, int32_t B, int32_t H, int32_t W, int32_t C, int32_t k,
                      int32_t stride, int32_t pad, int8_t* y, void* stream)
{
    if (B < 0 || H < 1 || W < 1 || C < 1 || k < 1 || stride < 1 || pad < 0 || pad >= k)
        return fail(NM_ERR_INVALID_ARG, "nm_maxpool_i8: bad geometry");
    if (H + 2 * pad < k || W + 2 * pad < k) return fail(NM_ERR_INVALID_ARG, "nm_maxpool_i8: window larger than the padded image");
    const int Ho = (H + 2 * pad - k) / stride + 1, Wo = (W + 2 * pad - k) / stride + 1;
    const int64_t rows = (int64_t)B * Ho * Wo;
    if (rows * C >= (1LL << 40) || (int64_t)B * H * W * C >= (1LL << 40))
        return fail(NM_ERR_UNSUPPORTED, "nm_maxpool_i8: tensor too large");
    if (rows == 0) return NM_OK;
    if (!x || !y) return fail(NM_ERR_INVALID_ARG, "nm_maxpool_i8: NULL pointer");
    const bool vec = C % 4 == 0 && aligned(x, 4) && aligned(y, 4);
    if (C % 16 == 0 && aligned(x, 16) && aligned(y, 16) && rows * (C / 16) < (1LL << 31) && (int64_t)H * W * C < (1LL << 31)) {
        const unsigned total16 = (unsigned)(rows * (C / 16));
        queue_kernel(k == 2 ? maxpool16_kernel<2> : k == 3 ? maxpool16_kernel<3> : maxpool16_kernel<0>, dim3((total16 - 1) / kConvThreads + 1), dim3(kConvThreads), 0,
                     (hipStream_t)stream, x, H, W, C, k, stride, pad, Ho, Wo, fast_div(C / 16), fast_div(Wo), fast_div(Ho), total16, y);
        return check_hip(hipGetLastError(), "nm_maxpool_i8 launch");
    }
    const long total = rows * (vec ? C / 4 : C);
    if (vec) queue_kernel(maxpool_kernel<true>, dim3(grid_for(total)), dim3(kConvThreads), 0, (hipStream_t)stream,
                                x, H, W, C, k, stride, pad, Ho, Wo, total, y);
    else queue_kernel(maxpool_kernel<false>, dim3(grid_for(total)), dim3(kConvThreads), 0, (hipStream_t)stream,
                            x, H, W, C, k, stride, pad, Ho, Wo, total, y);
    return check_hip(hipGetLastError(), "nm_maxpool_i8 launch");
}

int32_t nm_avgpool_i8(const int8_t* x, int32_t B, int32_t HW, int32_t C, float alpha, float out_inv_scale,
                      int8_t* out_q, float* out_f32, void* stream)
{
    if (B < 0 || HW < 1 || C < 1) return fail(NM_ERR_INVALID_ARG, "nm_avgpool_i8: bad shape");
    if (HW > (1 << 23)) return fail(NM_ERR_UNSUPPORTED, "nm_avgpool_i8: more than 2^23 positions (int32 sum)");
    if (!out_q && !out_f32) return fail(NM_ERR_INVALID_ARG, "nm_avgpool_i8: no output");
    if (B == 0) return NM_OK;
    if (!x) return fail(NM_ERR_INVALID_ARG, "nm_avgpool_i8: x is NULL");
    const bool vec = C % 4 == 0 && aligned(x, 4) && (!out_q || aligned(out_q, 4)) && (!out_f32 || aligned(out_f32, 16));
    if (vec)
        queue_kernel(avgpool_kernel<true>, dim3(grid_for((long)B * (C / 4))), dim3(kConvThreads), 0,
                           (hipStream_t)stream, x, B, HW, C, alpha, out_inv_scale, out_q, out_f32);
    else
        queue_kernel(avgpool_kernel<false>, dim3(grid_for((long)B * C)), dim3(kConvThreads), 0,
                           (hipStream_t)stream, x, B, HW, C, alpha, out_inv_scale, out_q, out_f32);
    return check_hip(hipGetLastError(), "nm_avgpool_i8 launch");
}

int32_t nm_cnn_workspace(const nm_cnn_op* ops, int32_t n_ops, size_t* bytes)
{
    if (!ops || n_ops < 1) return fail(NM_ERR_INVALID_ARG, "nm_cnn_workspace: no steps");
    if (!bytes) return fail(NM_ERR_INVALID_ARG, "nm_cnn_workspace: bytes is NULL");
    size_t need = 0;
    for (int32_t i = 0; i < n_ops; ++i) {
        if (ops[i].kind == NM_OP_CONV) {
            size_t b = 0;
            int32_t rc = nm_conv2d_workspace(&ops[i].conv, &b);
            if (rc) return rc;
            if (b > need) need = b;
        } else if (ops[i].kind < NM_OP_CONV || ops[i].kind > NM_OP_GEMM) {
            return fail(NM_ERR_INVALID_ARG, "nm_cnn_workspace: step %d has unknown kind %d", i, ops[i].kind);
        }
    }
    *bytes = need;
    return NM_OK;
}

int32_t nm_cnn_run(const nm_cnn_op* ops, int32_t n_ops, void* ws, size_t ws_bytes, void* stream)
{
    if (!ops || n_ops < 1) return fail(NM_ERR_INVALID_ARG, "nm_cnn_run: no steps");
    for (int32_t i = 0; i < n_ops; ++i) {
        const nm_cnn_op& o = ops[i];
        int32_t rc;
        switch (o.kind) {
        case NM_OP_CONV: {
            bool both = false;
            if (i + 1 < n_ops && ops[i + 1].kind == NM_OP_CONV && (rc = conv_pair(&o.conv, &ops[i + 1].conv, (hipStream_t)stream, &both))) return rc;
            if (!both && i + 1 < n_ops && ops[i + 1].kind == NM_OP_CONV && (rc = conv_chain(&o.conv, &ops[i + 1].conv, (hipStream_t)stream, &both))) return rc;
            if (both) ++i;
            rc = both ? NM_OK : nm_conv2d_pwl(&o.conv, ws, ws_bytes, stream);
            break;
        }
        case NM_OP_MAXPOOL: rc = nm_maxpool_i8(o.x, o.B, o.H, o.W, o.C, o.k, o.stride, o.pad, o.y, stream); break;
        case NM_OP_AVGPOOL: rc = nm_avgpool_i8(o.x, o.B, o.H, o.C, o.alpha, o.out_inv_scale, o.y, o.y_f32, stream); break;
        case NM_OP_GEMM: rc = nm_gemm_pwl(&o.gemm, stream); break;
        default: return fail(NM_ERR_INVALID_ARG, "nm_cnn_run: step %d has unknown kind %d", i, o.kind);
        }
        if (rc) return rc;
    }
    return NM_OK;
}

}  // extern "C"
