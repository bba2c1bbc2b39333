// 3x3 convolutions of 64 channels to 64 with stride 1 and a border of 1 (paper Section 3.1: a convolution as a matrix product; Section 3.2:
// the activation as a PWL table; arithmetic is that of the tile kernel, so results are bit-identical).
//
// What bounds the tile kernel here is its operands' stream into LDS: nine times the image and, for every 128 positions, the whole filter.
// With that stride and border output position m and input pixel m are the same one, so 32 positions read three runs of 34 pixels, which
// lie in memory as they are: a wavefront has those of its block and of its next one in LDS (7 KB each; three times the image instead of
// nine), a lane's tap is an address into them, or that of zeros where the tap lies in the border.  The filter comes once per workgroup.
// Here LDS is what is waited for: 36 fragments of the filter, 18 of pixels and 16 of scales and biases for 32 positions (70 x 8 clocks, eight
// wavefronts to a CU; by counter, 200704 positions, it is busy in 47 % of the cycles, nearly half of them bank conflicts, vector instructions issue
// in 34 % and the matrix cores run in 27 %).  us, before -> after: 200704 positions (64 images of 56 x 56) 17.2 -> 14.0, 50176 7.5 -> 6.4, 25088 8.1 -> 5.1.  With the pixels
// gathered by every lane for itself, nine times the image from L1, it was 16.2: such a load, 16 bytes from each of 32 rows, takes 70 clocks.
#include <mutex>

#include "nm_device.h"
#include "nm_gemm_choice.h"

namespace nm {

constexpr int kTapRun = 34, kTapImage = 7 * 1024;   // pixels of a run; a wavefront's image of one block: 112 rows of 64 bytes, 102 of them pixels

struct TapsParams {
    int M, H, W, blocks, step;   // blocks of 32 positions, wavefronts of the grid
    FastDiv div_w, div_h;
    const int8_t *x, *w;
    const float *bias, *alpha_vec;
    float alpha, inv;
    int relu, lines;   // relu_codes holds; a table of two segments
    struct {
        float k0, b0, k1, b1, tau;
    } t;
    int8_t* y;
};

__global__ __launch_bounds__(64 * kTapsWaves, 2) void conv_taps_kernel(TapsParams p)
{
    constexpr int NW = kTapsWaves, C = 64;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fr = lane & 31, half = lane >> 5;
    float* const s_scale = reinterpret_cast<float*>(smem + 9 * C * C);
    float* const s_bias = s_scale + C;
    int* const s_relu = reinterpret_cast<int*>(s_bias + C);   // a word per wavefront, in 64 bytes
    int8_t* const s_zero = reinterpret_cast<int8_t*>(s_relu + 16);   // 64 bytes
    int8_t* const image = s_zero + 64 + wave * (2 * kTapImage);

    // A block's pixels, runs one behind the other, to image i: chunk c of row r lies at c ^ (r / 2 & 3), so that eight neighbouring rows'
    // are in different banks.  Pixels in front of the first image and behind the last are read from inside (no tap uses them).
    const auto request = [&](int blk, int i) {
#pragma unroll
        for (int n = 0; n < kTapImage / 1024; ++n) {
            const int r = 16 * n + (lane >> 2), run = min(r / kTapRun, 2), pixel = 32 * blk + (run - 1) * p.W - 1 + r - run * kTapRun;
            dma16(p.x + (long)max(0, min(pixel, p.M - 1)) * C + 16 * ((lane & 3) ^ (r >> 1 & 3)), (unsigned)(uintptr_t)image + kTapImage * i + 1024 * n);
        }
    };
    // Neighbouring blocks, which share pixels, to a workgroup; what is left of a last turn by one to every workgroup.
    const int full = p.blocks / p.step;
    const auto block_of = [&](int turn) { return turn * p.step + (turn < full ? (int)blockIdx.x * NW + wave : wave * (int)gridDim.x + (int)blockIdx.x); };
    int turn = 0, blk = block_of(0);
    request(min(blk, p.blocks - 1), 0);
    const unsigned lds = (unsigned)(uintptr_t)smem;   // the filter tap by tap, its rows in the same order
    for (int f = wave; f < 9 * C * C / 1024; f += NW) {
        const int tap = f / 4, row = 16 * (f % 4) + (lane >> 2);
        dma16(p.w + row * (9 * C) + tap * C + 16 * ((lane & 3) ^ (row >> 1 & 3)), lds + 1024 * f);
    }
    bool relu = p.relu;
    if (threadIdx.x < C) {
        s_scale[threadIdx.x] = p.alpha_vec ? p.alpha_vec[threadIdx.x] : p.alpha;
        s_bias[threadIdx.x] = p.bias ? p.bias[threadIdx.x] : 0.0f;
        relu = relu && relu_finite(s_scale[threadIdx.x], s_bias[threadIdx.x]);
    }
    if (threadIdx.x < 16) reinterpret_cast<int*>(s_zero)[threadIdx.x] = 0;
    const int own = __all(relu);
    if (lane == 0) s_relu[wave] = own;
    wait_vmcnt<0>();
    __syncthreads();
    relu = __all(s_relu[lane % NW] != 0);

    const unsigned zero = (unsigned)(s_zero - smem) + 16 * half, images = (unsigned)(image - smem);
    unsigned at[9];   // of a lane's tap in an image; k-step 1 is 32 bytes on in a row's swizzled order
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
        const int r = tap / 3 * kTapRun + tap % 3 + fr;
        at[tap] = r * C + 16 * (half ^ (r >> 1 & 3));
    }
    const unsigned wat = fr * C + 16 * (half ^ (fr >> 1 & 3));
    const float inv = in_vgpr(p.inv);
    for (; blk < p.blocks; blk = block_of(++turn)) {
        const int i = turn & 1, next = block_of(turn + 1);
        wait_vmcnt<2>();   // this block's pixels: behind their request only the two stores of the block before were queued
        request(next < p.blocks ? next : blk, i ^ 1);
        const int m = 32 * blk + fr;
        unsigned taps = 0;   // a bit for every tap inside the image
        {
            const unsigned row = min(m, p.M - 1), q = quotient(row, p.div_w), w = row - q * p.W, h = q - quotient(q, p.div_h) * p.H;
            const unsigned across = (w > 0 ? 1u : 0u) | 2u | (w + 1 < (unsigned)p.W ? 4u : 0u);
            taps = (h > 0 ? across : 0u) | across << 3 | (h + 1 < (unsigned)p.H ? across << 6 : 0u);
        }
        v16i acc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0;
        const unsigned im = images + kTapImage * i;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const unsigned a = taps >> tap & 1 ? im + at[tap] : zero;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const v4i x = *reinterpret_cast<const v4i*>(smem + (s ? a ^ 32 : a));
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i*>(smem + tap * (C * C) + t * (32 * C) + (s ? wat ^ 32 : wat)), x, acc[t], 0, 0, 0);
            }
        }
        const auto finish = [&](auto relu_c) {
            constexpr bool kRelu = decltype(relu_c)::value;
            v4i o[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                v4f sc[4], bi[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    sc[g] = *reinterpret_cast<const v4f*>(s_scale + 32 * t + 8 * g + 4 * half);
                    bi[g] = *reinterpret_cast<const v4f*>(s_bias + 32 * t + 8 * g + 4 * half);
                }
                unsigned w[4];
                int q[4][4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float v = __builtin_fmaf((float)acc[t][4 * g + e], sc[g][e], bi[g][e]);
                        if (kRelu) w[g] = relu_requant(v, inv, e, e ? w[g] : 0);
                        else q[g][e] = requant(p.lines ? pwl_eval_two_segments(v, p.t) : v, inv);
                    }
                if (!kRelu)
#pragma unroll
                    for (int g = 0; g < 4; ++g) w[g] = pack4(q[g][0], q[g][1], q[g][2], q[g][3]);
                o[t] = halves_to_row(w[0], w[1], w[2], w[3]);
            }
            if (m < p.M)
#pragma unroll
                for (int t = 0; t < 2; ++t) *reinterpret_cast<v4i*>(p.y + (long)m * C + 32 * t + 16 * half) = o[t];
        };
        if (relu) finish(std::true_type{});
        else finish(std::false_type{});
    }
    wait_vmcnt<0>();   // LDS is given back with no request under way
}

int32_t launch_conv_taps(const GemmArgs& g, hipStream_t stream, bool* done)
{
    *done = false;
    const bool lines = g.has_table && g.table.two_seg && !g.table.clamp_input && !g.table.cellmap;
    if (gemm_switched() || !g.conv || g.cCin != 64 || g.N != 64 || g.cKw != 3 || g.K != 9 * 64 || g.cStride != 1 || g.cPad != 1 || g.cHo != g.cH || g.cWo != g.cW ||
        !conv_taps_faster(g.M, g.has_table != 0) || (g.has_table && !lines) || g.resid || !g.out_q || g.out_f32 || g.out_acc || g.dbg_seg || !aligned(g.A, 16) || !aligned(g.W, 16) ||
        !aligned(g.out_q, 16) || !aligned(g.bias, 4) || !aligned(g.alpha_vec, 4))
        return NM_OK;
    static std::once_flag once;
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(conv_taps_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(conv_taps_kernel)");
    });
    if (once_rc) return once_rc;
    TapsParams p{};
    p.M = g.M; p.H = g.cH; p.W = g.cW;
    p.div_w = fast_div(g.cW); p.div_h = fast_div(g.cH);
    p.x = g.A; p.w = g.W; p.bias = g.bias; p.alpha_vec = g.alpha_vec; p.alpha = g.alpha; p.inv = g.out_inv_scale; p.y = g.out_q;
    p.lines = lines;
    p.relu = lines && relu_codes(g.table, g.out_inv_scale, 0.0f);
    p.t = {g.table.k0, g.table.b0, g.table.k1, g.table.b1, g.table.tau};
    p.blocks = (p.M + 31) / 32;
    // a workgroup to a CU, which walks the blocks: the filter comes once
    const int grid = p.blocks < 256 ? p.blocks : 256;
    p.step = grid * kTapsWaves;
    constexpr size_t shmem = 9 * 64 * 64 + 2 * 64 * sizeof(float) + 128 + kTapsWaves * 2 * kTapImage;
    static_assert(shmem <= 160 * 1024, "LDS");
    queue_kernel(conv_taps_kernel, dim3(grid), dim3(64 * kTapsWaves), shmem, stream, p);
    *done = true;
    return check_hip(hipGetLastError(), "3x3 convolution launch");
}

}  // namespace nm
