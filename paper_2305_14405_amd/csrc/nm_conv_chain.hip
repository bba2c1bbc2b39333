// Two 1x1 convolutions as one kernel: the one that widens a residual block, with the shortcut added and a two-segment table behind it,
// and the one that narrows its result for the next block (paper Section 3.1: convolutions as matrix products, Section 3.2: the
// activation as a PWL table; arithmetic and order are those of the separate kernels, so results are bit-identical).
//
// What bounds it: memory (200704 positions of 64 -> 256 -> 64 channels move 128 MB, 25 us at a copy's rate), then a wavefront's chain of
// products and vector instructions, which takes 0.5 us per 32 channels alone on a SIMD and hides behind two others (by counter vector
// instructions issue in 46 % of the cycles there, LDS is busy in 21 %, the matrix cores in 9 %).  The wide tensor is written, since the
// next shortcut needs it, but not read again.  A wavefront takes 32 positions through both products by itself: the widened 32 channels that
// a matrix instruction leaves in a lane's accumulators become, after two half swaps, the 16 bytes that the second product's operand wants
// from that lane (and that are its piece of the output row), so neither LDS nor a barrier lies between them.  LDS holds both filters whole,
// once per workgroup; the shortcut's next 256 channels are requested while the present ones are worked on.  us, two kernels -> this one:
// 200704 positions of 64 -> 256 -> 64 channels 38.1 -> 29.6, -> 128 42.7 -> 34.5, 50176 of 128 -> 512 -> 128 25.3 -> 20.5;
// conv_chain_faster has the rest.  64 positions a wavefront, which halves the reads of scales and filters, was slower (33.3), as was the
// next block's first product queued ahead (128 -> 512 -> 128 22.1) and 16 wavefronts a CU, which spill (36.4).
#include <mutex>

#include "nm_device.h"
#include "nm_gemm_choice.h"

namespace nm {

struct TwoLines {
    float k0, b0, k1, b1, tau;
};
struct ChainParams {
    int M, N1, blocks, step;   // blocks of 32 positions, wavefronts of the grid
    const int8_t *x, *w1, *w2, *resid;
    const float *bias1, *alpha_vec1, *bias2, *alpha_vec2;
    float alpha1, alpha2, resid_scale, inv1, inv2;
    int relu;                  // relu_codes holds for both
    TwoLines t1, t2;
    int8_t *y1, *y2;
};

// The other way round from halves_to_row.
__device__ __forceinline__ v4i row_to_halves(v4i r)
{
    const auto a = __builtin_amdgcn_permlane32_swap((unsigned)r[0], (unsigned)r[1], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap((unsigned)r[2], (unsigned)r[3], false, false);
    return v4i{(int)a[0], (int)b[0], (int)a[1], (int)b[1]};
}

// KS: 32-channel steps of the first product's rows; TN: blocks of 32 columns of the second's.
template <int KS, int TN>
__global__ __launch_bounds__(64 * chain_waves(32 * KS), TN == 2 ? 3 : 2) void conv_chain_kernel(ChainParams p)
{
    constexpr int NW = chain_waves(32 * KS);
    // Whole lines of 128 bytes requested and stored at a time, and a block's scales and biases at once, where registers allow: 200704
    // positions of 64 -> 256 -> 64 channels 34.7 -> 31.0 us, -> 128 38.1 -> 34.8; 128 -> 512 -> 128 (50176) 21.2 -> 23.2.
    constexpr bool kLines = KS == 2;
    constexpr int RING = 8;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fr = lane & 31, half = lane >> 5;
    const int NJ = p.N1 / 32;
    int8_t* const s_w2 = smem + NJ * KS * 1024;
    float* const s_scale1 = reinterpret_cast<float*>(s_w2 + NJ * TN * 1024);
    float* const s_bias1 = s_scale1 + p.N1;
    float* const s_scale2 = s_bias1 + p.N1;
    float* const s_bias2 = s_scale2 + 32 * TN;
    int* const s_relu = reinterpret_cast<int*>(s_bias2 + 32 * TN);   // a word per wavefront

    // Lanes past the edge compute row M - 1 again and write its bytes again: in a branch, stores would be unknown to the wait for
    // the ring's loads.
    const auto row_of = [&](int blk) { return (long)min(32 * blk + fr, p.M - 1); };
    int blk = wave * gridDim.x + blockIdx.x;   // what is left of a last turn is one block to a workgroup
    v4i x[KS], r[RING];
    const auto load_x = [&](int blk) {
#pragma unroll
        for (int s = 0; s < KS; ++s) x[s] = *reinterpret_cast<const v4i*>(p.x + row_of(blk) * (32 * KS) + 32 * s + 16 * half);
    };
    const int first = min(blk, p.blocks - 1);
    load_x(first);
#pragma unroll
    for (int j = 0; j < RING; ++j) r[j] = *reinterpret_cast<const v4i*>(p.resid + row_of(first) * p.N1 + 32 * j + 16 * half);
    const unsigned lds = (unsigned)(uintptr_t)smem;
    // Filters in slices of 128 bytes of K (the first's rows of 64 are whole ones): rows of a slice one behind the other, a load takes
    // 1 KB of whole pieces, and a chunk of 16 bytes lies where its row's number puts it, so that eight neighbouring rows' are in
    // different banks.
    constexpr int CH1 = 2 * KS;
    for (int f = wave; f < NJ * KS; f += NW) {
        const int row = (64 * f + lane) / CH1, at = lane & (CH1 - 1);
        dma16(p.w1 + row * (32 * KS) + 16 * (at ^ (KS == 2 ? row >> 1 & 3 : row & 7)), lds + 1024 * f);
    }
    for (int f = wave; f < NJ * TN; f += NW) {
        const int q = f / (4 * TN), row = f % (4 * TN) * 8 + (lane >> 3);
        dma16(p.w2 + row * p.N1 + 128 * q + 16 * ((lane & 7) ^ (row & 7)), lds + 1024 * (NJ * KS + f));
    }
    bool relu = p.relu;
    for (int c = threadIdx.x; c < p.N1; c += 64 * NW) {
        s_scale1[c] = p.alpha_vec1 ? p.alpha_vec1[c] : p.alpha1;
        s_bias1[c] = p.bias1 ? p.bias1[c] : 0.0f;
        relu = relu && relu_finite(s_scale1[c], s_bias1[c]);
    }
    for (int c = threadIdx.x; c < 32 * TN; c += 64 * NW) {
        s_scale2[c] = p.alpha_vec2 ? p.alpha_vec2[c] : p.alpha2;
        s_bias2[c] = p.bias2 ? p.bias2[c] : 0.0f;
        relu = relu && relu_finite(s_scale2[c], s_bias2[c]);
    }
    const int own = __all(relu);
    if (lane == 0) s_relu[wave] = own;
    wait_vmcnt<0>();
    __syncthreads();
    relu = __all(s_relu[lane % NW] != 0);

    // the lane's chunk of a fragment: rows fr of 32, k-step s of a slice
    const auto chunk128 = [&](int s) { return fr * 128 + 16 * ((2 * s + half) ^ (fr & 7)); };
    unsigned at1[KS], at2[4];
#pragma unroll
    for (int s = 0; s < KS; ++s) at1[s] = KS == 2 ? fr * 64 + 16 * ((2 * s + half) ^ (fr >> 1 & 3)) : chunk128(s);
#pragma unroll
    for (int s = 0; s < 4; ++s) at2[s] = chunk128(s);
    const float rs = in_vgpr(p.resid_scale), inv1 = in_vgpr(p.inv1), inv2 = in_vgpr(p.inv2);

    v16i acc2[TN];
    const auto clear = [&] {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc2[t][v] = 0;
    };
    const auto widen = [&](const int8_t* f) {
        v16i a;
#pragma unroll
        for (int v = 0; v < 16; ++v) a[v] = 0;
#pragma unroll
        for (int s = 0; s < KS; ++s) a = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i*>(f + at1[s]), x[s], a, 0, 0, 0);
        return a;
    };
    const auto narrow = [&](const int8_t* f, unsigned at, const v4i& o) {
#pragma unroll
        for (int t = 0; t < TN; ++t) acc2[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i*>(f + 4096 * t + at), o, acc2[t], 0, 0, 0);
    };
    // Scales and biases of the lane's 16 of 32 columns, and the codes of those columns, of accumulators and the shortcut's words or none, as
    // the lane's 16 bytes of the row.
    struct Columns {
        v4f scale[4], bias[4];
    };
    const auto columns = [&](const float* scale, int to_bias) {
        Columns c;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            c.scale[g] = *reinterpret_cast<const v4f*>(scale + 8 * g + 4 * half);
            c.bias[g] = *reinterpret_cast<const v4f*>(scale + to_bias + 8 * g + 4 * half);
        }
        return c;
    };
    const auto codes = [&](auto relu_c, auto resid_c, const v16i& a, const v4i& rw, const Columns& c, float inv, const TwoLines& lines) {
        constexpr bool kRelu = decltype(relu_c)::value, kResid = decltype(resid_c)::value;
        unsigned w[4];
        int q[4][4];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int g = i % 4, e = i / 4;   // (four words in turn: four chains instead of one)
            float v = __builtin_fmaf((float)a[4 * g + e], c.scale[g][e], c.bias[g][e]);
            if (kResid) v = __builtin_fmaf((float)(int)(int8_t)((unsigned)rw[g] >> (8 * e)), rs, v);
            if (kRelu) w[g] = relu_requant(v, inv, e, e ? w[g] : 0);
            else q[g][e] = requant(pwl_eval_two_segments(v, lines), inv);
        }
        if (!kRelu)
#pragma unroll
            for (int g = 0; g < 4; ++g) w[g] = pack4(q[g][0], q[g][1], q[g][2], q[g][3]);
        return halves_to_row(w[0], w[1], w[2], w[3]);
    };
    const auto finish = [&](auto relu_c, long row) {
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            const v4i o = codes(relu_c, std::false_type{}, acc2[t], v4i{}, columns(s_scale2 + 32 * t, 32 * TN), inv2, p.t2);
            *reinterpret_cast<v4i*>(p.y2 + row * (32 * TN) + 32 * t + 16 * half) = o;
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (!relu) {   // another table, or columns whose sums may be infinite: the lines themselves, without a ring
        for (; blk < p.blocks; blk += p.step) {
            const long row = row_of(blk);
            load_x(blk);
            clear();
#pragma unroll 1
            for (int j = 0; j < NJ; ++j) {
                const v4i rw = row_to_halves(*reinterpret_cast<const v4i*>(p.resid + row * p.N1 + 32 * j + 16 * half));
                const v4i o = codes(std::false_type{}, std::true_type{}, widen(smem + j * (1024 * KS)), rw, columns(s_scale1 + 32 * j, p.N1), inv1, p.t1);
                *reinterpret_cast<v4i*>(p.y1 + row * p.N1 + 32 * j + 16 * half) = o;
                narrow(s_w2 + j / 4 * (4096 * TN), chunk128(j & 3), o);
            }
            finish(std::false_type{}, row);
        }
        return;
    }
    for (; blk < p.blocks; blk += p.step) {
        const int next = blk + p.step < p.blocks ? blk + p.step : blk;
        const long row = row_of(blk);
        clear();
        for (int c0 = 0; c0 < p.N1; c0 += 32 * RING) {
            // what the ring holds next: the row's next channels, or the next row's first
            const bool more = c0 + 32 * RING < p.N1;
            const int8_t* const ahead = p.resid + row_of(more ? blk : next) * p.N1 + (more ? c0 + 32 * RING : 0) + 16 * half;
            int8_t* const out = p.y1 + row * p.N1 + c0 + 16 * half;
            const int8_t* const f1 = smem + c0 / 32 * (1024 * KS);
            const int8_t* const f2 = s_w2 + c0 / 128 * (4096 * TN);
            v4i line[4];
#pragma unroll
            for (int j = 0; j < RING; ++j) {
                const Columns c = columns(s_scale1 + c0 + 32 * j, p.N1);
                const v16i a = widen(f1 + j * (1024 * KS));
                const v4i rw = row_to_halves(r[j]);
                if (!kLines) r[j] = *reinterpret_cast<const v4i*>(ahead + 32 * j);
                else __builtin_amdgcn_sched_barrier(0);
                const v4i o = codes(std::true_type{}, std::true_type{}, a, rw, c, inv1, p.t1);
                if (!kLines) *reinterpret_cast<v4i*>(out + 32 * j) = o;
                line[j % 4] = o;
                narrow(f2 + j / 4 * (4096 * TN), at2[j % 4], o);
                if (kLines && j % 4 == 3) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) *reinterpret_cast<v4i*>(out + 32 * (j - 3 + i)) = line[i];
#pragma unroll
                    for (int i = j - 3; i <= j; ++i) r[i] = *reinterpret_cast<const v4i*>(ahead + 32 * i);
                }
                __builtin_amdgcn_sched_barrier(0);   // or the compiler keeps all blocks' operands at once, and spills
            }
        }
        load_x(next);
        finish(std::true_type{}, row);
    }
}

template <int KS, int TN>
static int32_t launch_chain_as(ChainParams& p, size_t shmem, int groups, hipStream_t s)
{
    constexpr int NW = chain_waves(32 * KS);
    auto kern = conv_chain_kernel<KS, TN>;
    static std::once_flag once;  // one attribute call per instantiation
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(conv_chain_kernel)");
    });
    if (once_rc) return once_rc;
    p.blocks = (p.M + 31) / 32;
    const int all = (p.blocks + NW - 1) / NW, grid = all < groups ? all : groups;   // (more of them, each with fewer blocks, wait for the filters: 25088 positions 8.2 -> 11.5)
    p.step = grid * NW;
    queue_kernel(kern, dim3(grid), dim3(64 * NW), shmem, s, p);
    return check_hip(hipGetLastError(), "convolution chain launch");
}

static bool lines_only(const GemmArgs& g) { return g.has_table && g.table.two_seg && !g.table.clamp_input && !g.table.cellmap; }

int32_t launch_conv_chain(const GemmArgs& a, const GemmArgs& b, hipStream_t stream, bool* done)
{
    *done = false;
    if (gemm_switched() || !conv_chain_built(a.K, a.N, b.N) || !lines_only(a) || !lines_only(b)) return NM_OK;
    const bool relu = relu_codes(a.table, a.out_inv_scale, a.resid_scale) && relu_codes(b.table, b.out_inv_scale, 0.0f);
    if (!conv_chain_faster(a.M, a.K, a.N, b.N, relu)) return NM_OK;
    const void* const rows[] = {a.A, a.W, a.resid, a.out_q, b.W, b.out_q};
    const void* const cols[] = {a.bias, a.alpha_vec, b.bias, b.alpha_vec};
    for (const void* q : rows)
        if (!q || !aligned(q, 16)) return NM_OK;
    for (const void* q : cols)
        if (!aligned(q, 4)) return NM_OK;
    ChainParams p{};
    p.M = a.M; p.N1 = a.N;
    p.x = a.A; p.w1 = a.W; p.w2 = b.W; p.resid = a.resid; p.y1 = a.out_q; p.y2 = b.out_q;
    p.bias1 = a.bias; p.alpha_vec1 = a.alpha_vec; p.bias2 = b.bias; p.alpha_vec2 = b.alpha_vec;
    p.alpha1 = a.alpha; p.alpha2 = b.alpha; p.resid_scale = a.resid_scale; p.inv1 = a.out_inv_scale; p.inv2 = b.out_inv_scale;
    p.relu = relu;
    p.t1 = {a.table.k0, a.table.b0, a.table.k1, a.table.b1, a.table.tau};
    p.t2 = {b.table.k0, b.table.b0, b.table.k1, b.table.b1, b.table.tau};
    const size_t shmem = conv_chain_lds(a.K, a.N, b.N);
    // a CU's worth of workgroups, which walk the blocks: the filters come once
    const int groups = 256 * conv_chain_share(a.K, a.N, b.N);
    *done = true;
    return b.N == 64 ? launch_chain_as<2, 2>(p, shmem, groups, stream)
         : a.K == 64 ? launch_chain_as<2, 4>(p, shmem, groups, stream) : launch_chain_as<4, 4>(p, shmem, groups, stream);
}

}  // namespace nm
