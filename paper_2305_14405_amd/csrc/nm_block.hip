// The row-local part of an encoder layer in one kernel, for narrow layers: output projection, LayerNorm-PWL,
// FFN1 + GELU-PWL, FFN2, LayerNorm-PWL and, inside a stack, the next layer's QKV projection, for a block of
// 16 or 32 rows per workgroup (paper Section 3.1 for the products, Section 3.2 for the functions; the
// arithmetic and its order are those of the separate kernels, so results are bit-identical).
//
// As separate kernels these five or six steps are bound by launches: at 64 rows of width 128 each takes
// 2.9 .. 3.3 us, of which an empty launch is 1.6 (and 3.1 us of host time), and 0.3 us of weights.  A
// workgroup that keeps its rows in LDS needs no other workgroup between attention and attention; what it
// pays is reading all weights (9 to 12 H^2 bytes) itself, so the kernel is chosen by that number
// (block_rows).  Sixteen wavefronts, each with a ring of 2 KB slots (16 weight rows x 128 bytes) of its own,
// request their slices of all products in one sequence that does not stop at the barriers between the
// products (weights do not depend on the activations).  What bounds it is the latency of one slice's round
// in a wavefront (wait, two LDS reads, two MFMAs, the next request: about 600 clocks), so wavefronts are
// what hides it: with eight of them and rings twice as deep the stream ran at 43 bytes per ns and CU, with
// sixteen at 65, of 128 that LDS-direct loads reach.  block_rows_faster has both kinds' times.
#include <mutex>

#include "nm_device.h"
#include "nm_gemm_choice.h"

namespace nm {

constexpr int kBlockWaves = 16, kBlockThreads = 64 * kBlockWaves;
constexpr int kBlockHold = 2;     // 16-column tiles of FFN2 per wavefront
constexpr int kBlockPhases = 4;   // output projection, FFN1, FFN2, QKV of the next layer

struct BlockParams {
    const int8_t* W[kBlockPhases];
    int N[kBlockPhases], K[kBlockPhases];
    int M, H, F, slots, phases;
    // byte offsets into LDS behind the rings: activations, LN1 output / context, layer output / input, vectors, tables
    int off_x, off_a1, off_a3, off_par, off_gelu, off_rsqrt;
    int par_b1, par_b2, par_bq, par_ln;       // vectors: float offsets (bo at 0; gamma1, beta1, gamma2, beta2 at par_ln)
    int par_chunks, gelu_chunks, rsqrt_chunks;  // 16-byte pieces to stage
    const int8_t* ctx;
    const int8_t* x;
    const float *bo, *b1, *b2, *bq, *gamma1, *beta1, *gamma2, *beta2;
    float alpha_o, resid1_scale, eps1, inv_ln1, alpha_1, inv_ffn1, alpha_2, resid2_scale, eps2, inv_out, alpha_q, inv_q, inv_k, inv_v, inv_L;
    DevTable t_gelu, t_rsqrt;
    int8_t* y_q;
    float* y_f32;
    int8_t* qkv;
};

// RT: 16-row tiles per workgroup.
// SLOTS: 2 KB slots of a wavefront's ring.
template <int RT, int SLOTS>
__global__ __launch_bounds__(kBlockThreads) void encoder_block_kernel(BlockParams p)
{
    constexpr int BM = 16 * RT;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    asm volatile("" : : "s"(p.H), "s"(p.F), "s"(p.M), "s"(p.ctx), "s"(p.x), "s"(p.bo), "s"(p.b1), "s"(p.b2), "s"(p.bq),
                 "s"(p.gamma1), "s"(p.beta1), "s"(p.gamma2), "s"(p.beta2), "s"(p.off_a1), "s"(p.off_a3), "s"(p.off_par), "s"(p.par_chunks));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fq = lane >> 4;
    const int H = p.H, F = p.F, m0 = blockIdx.x * BM;
    const int sH = H + 16, sF = F + 16, sX = H + 4;   // row strides: bytes, bytes, floats (an odd number of 16-byte pieces apart)
    int8_t* s_a1 = smem + p.off_a1;
    int8_t* s_a3 = smem + p.off_a3;
    int8_t* s_a2 = smem + p.off_x;                             // FFN1 output, over ...
    float* s_x = reinterpret_cast<float*>(smem + p.off_x);     // ... the fp32 rows in front of a LayerNorm
    const float* s_par = reinterpret_cast<const float*>(smem + p.off_par);
    const float2* s_gelu = reinterpret_cast<const float2*>(smem + p.off_gelu);
    const float2* s_rsqrt = reinterpret_cast<const float2*>(smem + p.off_rsqrt);
    const unsigned lds0 = (unsigned)(uintptr_t)smem;

    // ---- everything that is not a weight, by direct loads -----------------------------------------
    {
        // context rows -> a1, layer input rows -> a3; a row's padding piece is a zero
        const int hc = H / 16 + 1, rows = BM * hc;
        for (int i = wave; i * 64 < rows; i += kBlockWaves) {
            const int c = i * 64 + lane, r = c / hc, cc = c - r * hc;
            const bool in = r < BM && cc < hc - 1;
            const long at = (long)min(m0 + r, p.M - 1) * H + 16 * cc;
            dma16(in ? p.ctx + at : g_zero_line, lds0 + p.off_a1 + 1024 * i);
            dma16(in ? p.x + at : g_zero_line, lds0 + p.off_a3 + 1024 * i);
        }
        // vectors: bo | b1 | b2 | bq | gamma1 | beta1 | gamma2 | beta2 (a missing bias is zero)
        for (int i = wave; i * 64 < p.par_chunks; i += kBlockWaves) {
            const int f = (i * 64 + lane) * 4;
            const float* src;
            int at;
            if (f < p.par_b1) { src = p.bo; at = f; }
            else if (f < p.par_b2) { src = p.b1; at = f - p.par_b1; }
            else if (f < p.par_bq) { src = p.b2; at = f - p.par_b2; }
            else if (f < p.par_ln) { src = p.bq; at = f - p.par_bq; }
            else {
                at = f - p.par_ln;
                src = p.gamma1;
                if (at >= H) { at -= H; src = p.beta1; }
                if (at >= H) { at -= H; src = p.gamma2; }
                if (at >= H) { at -= H; src = p.beta2; }
                if (at >= H) src = nullptr;   // past the end
            }
            dma16(src ? (const void*)(src + at) : (const void*)g_zero_line, lds0 + p.off_par + 1024 * i);
        }
        // tables (128-byte aligned and padded in the blob)
        for (int i = wave; i * 64 < p.gelu_chunks; i += kBlockWaves) {
            const int c = i * 64 + lane;
            dma16(c < p.gelu_chunks ? (const void*)(p.t_gelu.kb + 2 * c) : (const void*)g_zero_line, lds0 + p.off_gelu + 1024 * i);
        }
        for (int i = wave; i * 64 < p.rsqrt_chunks; i += kBlockWaves) {
            const int c = i * 64 + lane;
            dma16(c < p.rsqrt_chunks ? (const void*)(p.t_rsqrt.kb + 2 * c) : (const void*)g_zero_line, lds0 + p.off_rsqrt + 1024 * i);
        }
    }

    // ---- the stream of weight slices ----------------------------------------------------------------
    // A wavefront takes the 16-column tiles wave, wave + 16, .. of every product, and of each tile the
    // 128-byte slices of K in order.
    const unsigned ring = lds0 + wave * (SLOTS * 2048);
    const int lrow = lane >> 3, chunk0 = (lane & 7) ^ (lane >> 4);   // row and chunk of the lane in piece 0; piece 1: chunk ^ 4
    int ip = -1, ileft_k = 0, ileft_t = 0, iK = 0, ink = 0, islot = 0, outstanding = 0;
    const int8_t* isrc = nullptr;   // slice to request next
    unsigned iv0 = 0, iv1 = 0;
    auto next_phase = [&] {
        int n16;
        do {
            if (++ip >= p.phases) return;
            n16 = p.N[ip] >> 4;
        } while (wave >= n16);
        iK = p.K[ip];
        ink = (iK + 127) >> 7;
        isrc = p.W[ip] + (long)wave * 16 * iK;
        ileft_k = ink;
        ileft_t = (n16 - wave + kBlockWaves - 1) / kBlockWaves;
        iv0 = (unsigned)(lrow * iK + 16 * chunk0);
        iv1 = (unsigned)((lrow + 8) * iK + 16 * (chunk0 ^ 4));
    };
    auto issue = [&] {
        if (ip >= p.phases) return;
        const unsigned dst = ring + islot;
        const int left = iK - (ink - ileft_k) * 128;
        if (left >= 128) {
            dma16s(isrc, iv0, dst);
            dma16s(isrc, iv1, dst + 1024);
        } else {   // past K: zeros
            dma16(16 * chunk0 < left ? isrc + iv0 : g_zero_line, dst);
            dma16(16 * (chunk0 ^ 4) < left ? isrc + iv1 : g_zero_line, dst + 1024);
        }
        islot = islot == (SLOTS - 1) * 2048 ? 0 : islot + 2048;
        ++outstanding;
        isrc += 128;
        if (--ileft_k == 0) {
            ileft_k = ink;
            isrc += (long)kBlockWaves * 16 * iK - 128 * ink;
            if (--ileft_t == 0) next_phase();
        }
    };
    next_phase();
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) issue();

    // wait until only `young` slices (two loads each) are in flight
    auto wait_young = [&](int young) {
        if (SLOTS > 7 && young >= 7) wait_vmcnt<14>();
        else if (SLOTS > 6 && young == 6) wait_vmcnt<12>();
        else if (SLOTS > 5 && young == 5) wait_vmcnt<10>();
        else if (SLOTS > 4 && young == 4) wait_vmcnt<8>();
        else if (SLOTS > 3 && young == 3) wait_vmcnt<6>();
        else if (young == 2) wait_vmcnt<4>();
        else if (young == 1) wait_vmcnt<2>();
        else wait_vmcnt<0>();
    };
    const int8_t* const wfrag = smem + wave * (SLOTS * 2048) + fr * 128;
    const int wo0 = (fq ^ ((fr >> 1) & 7)) << 4, wo1 = wo0 ^ 64;   // chunks fq and 4 + fq of row fr
    int cslot = 0;
    // One product: rows in LDS (stride lda) times the phase's weights; finish(tile, acc) per 16-column tile:
    // lane (fr, fq) holds row 16i + fr, columns 16 tile + 4 fq .. +3.  (Operand bytes past K belong to whatever
    // follows in LDS and meet zero weights.)
    auto product = [&](int phase, const int8_t* s_a, int lda, auto finish) {
        const int n16 = p.N[phase] >> 4, nk = (p.K[phase] + 127) >> 7;
        const int8_t* const a0 = s_a + fr * lda + 16 * fq;
        for (int tile = wave; tile < n16; tile += kBlockWaves) {
            v4i acc[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) acc[i] = v4i{0, 0, 0, 0};
            const int8_t* a = a0;
            for (int k = 0; k < nk; ++k, a += 128) {
                v4i fa[2][RT], fw[2];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int i = 0; i < RT; ++i) fa[s][i] = *reinterpret_cast<const v4i*>(a + 16 * i * lda + 64 * s);
                if (outstanding == SLOTS) wait_vmcnt<2 * (SLOTS - 1)>();   // the steady state
                else wait_young(outstanding - 1);
                fw[0] = *reinterpret_cast<const v4i*>(wfrag + cslot + wo0);
                fw[1] = *reinterpret_cast<const v4i*>(wfrag + cslot + wo1);
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[s], fa[s][i], acc[i], 0, 0, 0);
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");   // the slot has been read
                --outstanding;
                cslot = cslot == (SLOTS - 1) * 2048 ? 0 : cslot + 2048;
                issue();
            }
            finish(tile, acc);
        }
    };
    // x = fma(acc, alpha, bias) + residual (int8 rows in LDS), to the fp32 rows
    auto to_rows = [&](const float* bias, float alpha, const int8_t* s_res, float rs) {
        return [=](int tile, const v4i (&acc)[RT]) {
            const int n = 16 * tile + 4 * fq;
            const v4f b = *reinterpret_cast<const v4f*>(bias + n);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const unsigned w = *reinterpret_cast<const unsigned*>(s_res + (16 * i + fr) * sH + n);
                v4f y;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = __builtin_fmaf((float)acc[i][e], alpha, b[e]);
                    y[e] = __builtin_fmaf((float)(int)(int8_t)(w >> (8 * e)), rs, v);
                }
                *reinterpret_cast<v4f*>(s_x + (16 * i + fr) * sX + n) = y;
            }
        };
    };
    // LayerNorm-PWL of the fp32 rows, one wavefront per row: int8 rows to LDS, fp32 rows to memory on request
    auto layernorm = [&](int vec, float eps, float inv, int8_t* s_out, float* out_f32) {
        constexpr int C = 2;   // groups of four per lane (H <= 512)
        for (int r = wave; r < BM; r += kBlockWaves) {
            float x[C][4];
            float part = 0.0f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int j = 4 * (lane + 64 * c);
                const v4f a = *reinterpret_cast<const v4f*>(s_x + r * sX + min(j, H - 4));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[c][e] = a[e];
                    if (j < H) part = part + x[c][e];
                }
            }
            const float mu = group_sum<64>(part) * p.inv_L;
            float part2 = 0.0f;
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[c][e] = x[c][e] - mu;
                    if (4 * (lane + 64 * c) < H) part2 = __builtin_fmaf(x[c][e], x[c][e], part2);
                }
            const float u = group_sum<64>(part2) * p.inv_L + eps;
            int seg;
            const float s = pwl_eval(u, p.t_rsqrt, s_rsqrt, seg);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int j = 4 * (lane + 64 * c);
                if (j < H) {
                    const v4f ga = *reinterpret_cast<const v4f*>(s_par + vec + j);
                    const v4f be = *reinterpret_cast<const v4f*>(s_par + vec + H + j);
                    v4f y;
                    int q[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        y[e] = __builtin_fmaf(x[c][e] * s, ga[e], be[e]);
                        q[e] = requant(y[e], inv);
                    }
                    *reinterpret_cast<unsigned*>(s_out + r * sH + j) = pack4(q[0], q[1], q[2], q[3]);
                    if (out_f32 && m0 + r < p.M) *reinterpret_cast<v4f*>(out_f32 + (long)(m0 + r) * H + j) = y;
                }
            }
        }
    };

    // the staged rows, vectors and tables are older than the slices
    if (outstanding == SLOTS) wait_vmcnt<2 * SLOTS>();
    else wait_young(outstanding);
    __syncthreads();
    product(0, s_a1, sH, to_rows(s_par, p.alpha_o, s_a3, p.resid1_scale));
    __syncthreads();
    layernorm(p.par_ln, p.eps1, p.inv_ln1, s_a1, nullptr);
    __syncthreads();
    product(1, s_a1, sH, [&](int tile, const v4i (&acc)[RT]) {
        const int n = 16 * tile + 4 * fq;
        const v4f b = *reinterpret_cast<const v4f*>(s_par + p.par_b1 + n);
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            int q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int seg;
                const float v = pwl_eval(__builtin_fmaf((float)acc[i][e], p.alpha_1, b[e]), p.t_gelu, s_gelu, seg);
                q[e] = requant(v, p.inv_ffn1);
            }
            *reinterpret_cast<unsigned*>(s_a2 + (16 * i + fr) * sF + n) = pack4(q[0], q[1], q[2], q[3]);
        }
    });
    __syncthreads();
    {
        // the fp32 rows lie over the operand: all tiles of the product first, then the rows
        v4i hold[kBlockHold][RT];
        int cnt = 0;
        product(2, s_a2, sF, [&](int, const v4i (&acc)[RT]) {
#pragma unroll
            for (int t = 0; t < kBlockHold; ++t)
                if (t == cnt)
#pragma unroll
                    for (int i = 0; i < RT; ++i) hold[t][i] = acc[i];
            ++cnt;
        });
        __syncthreads();
        const auto put = to_rows(s_par + p.par_b2, p.alpha_2, s_a1, p.resid2_scale);
#pragma unroll
        for (int t = 0; t < kBlockHold; ++t)
            if (t < cnt) put(wave + kBlockWaves * t, hold[t]);
    }
    __syncthreads();
    layernorm(p.par_ln + 2 * H, p.eps2, p.inv_out, s_a3, p.y_f32);
    __syncthreads();
    if (p.phases > 3) {
        const int sQ = 3 * H + 16;
        product(3, s_a3, sH, [&](int tile, const v4i (&acc)[RT]) {
            const int n = 16 * tile + 4 * fq;
            const v4f b = *reinterpret_cast<const v4f*>(s_par + p.par_bq + n);
            const float inv = n >= 2 * H ? p.inv_v : n >= H ? p.inv_k : p.inv_q;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                int q[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) q[e] = requant(__builtin_fmaf((float)acc[i][e], p.alpha_q, b[e]), inv);
                *reinterpret_cast<unsigned*>(s_a2 + (16 * i + fr) * sQ + n) = pack4(q[0], q[1], q[2], q[3]);
            }
        });
        __syncthreads();
        const int qc = 3 * H / 16;
        for (int c = tid; c < BM * qc; c += kBlockThreads) {
            const int r = c / qc, cc = c - r * qc;
            if (m0 + r < p.M)
                *reinterpret_cast<v4i*>(p.qkv + (long)(m0 + r) * 3 * H + 16 * cc) = *reinterpret_cast<const v4i*>(s_a2 + r * sQ + 16 * cc);
        }
    }
    if (p.y_q) {
        const int hc = H / 16;
        for (int c = tid; c < BM * hc; c += kBlockThreads) {
            const int r = c / hc, cc = c - r * hc;
            if (m0 + r < p.M)
                *reinterpret_cast<v4i*>(p.y_q + (long)(m0 + r) * H + 16 * cc) = *reinterpret_cast<const v4i*>(s_a3 + r * sH + 16 * cc);
        }
    }
}

static size_t round_kb(size_t b) { return (b + 1023) / 1024 * 1024; }

// Fills in the LDS layout; false when it does not fit with at least two slots per wavefront.
static bool block_layout(BlockParams& p, int bm, size_t* shmem)
{
    const size_t H = p.H, F = p.F;
    size_t x = (H + 4) * 4;
    if (F + 16 > x) x = F + 16;
    if (p.phases > 3 && 3 * H + 16 > x) x = 3 * H + 16;
    const size_t rows = round_kb((size_t)bm * (H + 16));
    p.par_b1 = p.H; p.par_b2 = p.par_b1 + p.F; p.par_bq = p.par_b2 + p.H;
    p.par_ln = p.par_bq + (p.phases > 3 ? 3 * p.H : 0);
    p.par_chunks = (p.par_ln + 4 * p.H) / 4;
    p.gelu_chunks = (p.t_gelu.nseg + 1) / 2;
    p.rsqrt_chunks = (p.t_rsqrt.nseg + 1) / 2;
    const size_t fixed = round_kb((size_t)bm * x) + 2 * rows + round_kb(16 * (size_t)p.par_chunks) + round_kb(16 * (size_t)p.gelu_chunks) +
                         round_kb(16 * (size_t)p.rsqrt_chunks);
    const size_t lds = 160 * 1024, per_slot = kBlockWaves * 2048;
    if (fixed + 2 * per_slot > lds) return false;
    p.slots = fixed + 4 * per_slot <= lds ? 4 : fixed + 3 * per_slot <= lds ? 3 : 2;   // the instantiated ring depths
    size_t o = p.slots * per_slot;
    p.off_x = (int)o; o += round_kb((size_t)bm * x);
    p.off_a1 = (int)o; o += rows;
    p.off_a3 = (int)o; o += rows;
    p.off_par = (int)o; o += round_kb(16 * (size_t)p.par_chunks);
    p.off_gelu = (int)o; o += round_kb(16 * (size_t)p.gelu_chunks);
    p.off_rsqrt = (int)o; o += round_kb(16 * (size_t)p.rsqrt_chunks);
    *shmem = o;
    return true;
}

template <int RT, int SLOTS>
static int32_t launch_block_t(const BlockParams& p, size_t shmem, hipStream_t s)
{
    auto kern = encoder_block_kernel<RT, SLOTS>;
    static std::once_flag once;
    static int32_t once_rc = NM_OK;
    std::call_once(once, [&] {
        once_rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
                            "hipFuncSetAttribute(encoder_block_kernel)");
    });
    if (once_rc) return once_rc;
    queue_kernel(kern, dim3((p.M + 16 * RT - 1) / (16 * RT)), dim3(kBlockThreads), shmem, s, p);
    return check_hip(hipGetLastError(), "encoder_block launch");
}
template <int RT>
static int32_t launch_block(const BlockParams& p, size_t shmem, hipStream_t s)
{
    switch (p.slots) {
    case 4: return launch_block_t<RT, 4>(p, shmem, s);
    case 3: return launch_block_t<RT, 3>(p, shmem, s);
    default: return launch_block_t<RT, 2>(p, shmem, s);
    }
}

// Rows per workgroup for this layer, 0 when the separate kernels are the better choice (block_rows_faster) or the shape,
// alignment or LDS space rules this kernel out.
static int block_rows(BlockParams& p, size_t* shmem)
{
    const int bm = block_rows_faster(p.M, p.H, p.F);
    if (!bm || p.H % 16 || p.F % 16) return 0;
    if (p.H > 16 * kBlockWaves * kBlockHold) return 0;   // the tiles that a wavefront holds in registers
    return block_layout(p, bm, shmem) ? bm : 0;
}

static bool fill_block(const nm_layer_desc* d, const nm_layer_desc* next, BlockParams& p)
{
    p.M = d->B * d->S; p.H = d->H; p.F = d->F;
    p.phases = next ? 4 : 3;
    p.W[0] = d->Wo; p.N[0] = d->H; p.K[0] = d->H;
    p.W[1] = d->W1; p.N[1] = d->F; p.K[1] = d->H;
    p.W[2] = d->W2; p.N[2] = d->H; p.K[2] = d->F;
    p.bo = d->bo; p.b1 = d->b1; p.b2 = d->b2;
    p.gamma1 = d->gamma1; p.beta1 = d->beta1; p.gamma2 = d->gamma2; p.beta2 = d->beta2;
    if (next) {
        p.W[3] = next->Wqkv; p.N[3] = 3 * d->H; p.K[3] = d->H;
        p.bq = next->bqkv; p.alpha_q = next->alpha_qkv;
        p.inv_q = next->inv_s_q; p.inv_k = next->inv_s_k; p.inv_v = next->inv_s_v;
    }
    for (int i = 0; i < p.phases; ++i)
        if (!aligned(p.W[i], 16)) return false;
    for (const float* v : {p.bo, p.b1, p.b2, p.bq, p.gamma1, p.beta1, p.gamma2, p.beta2})
        if (!aligned(v, 16)) return false;
    p.alpha_o = d->alpha_o; p.resid1_scale = d->resid1_scale; p.eps1 = d->eps1; p.inv_ln1 = d->inv_s_ln1;
    p.alpha_1 = d->alpha_1; p.inv_ffn1 = d->inv_s_ffn1; p.alpha_2 = d->alpha_2; p.resid2_scale = d->resid2_scale;
    p.eps2 = d->eps2; p.inv_out = d->inv_s_out;
    p.inv_L = (float)(1.0 / (double)d->H);
    return true;
}

// d's steps 5 to 9 and, if next is given, next's step 1.  *done = false when the kernel does not take this
// layer (nothing has been launched then).
int32_t launch_encoder_block(const nm_layer_desc* d, const nm_layer_desc* next, const int8_t* ctx, const int8_t* x, int8_t* y_q,
                             float* y_f32, int8_t* qkv, hipStream_t stream, bool* done)
{
    *done = false;
    BlockParams p{};
    size_t shmem = 0;
    if (gemm_switched() || !aligned(ctx, 16) || !aligned(x, 16) || !aligned(y_q, 16) || !aligned(y_f32, 16) || !aligned(qkv, 16) || !fill_block(d, next, p)) return NM_OK;
    int32_t rc = get_dev_table(d->tables, d->gelu_idx, &p.t_gelu, "nm_encoder_layer(gelu)");
    if (rc) return rc;
    if ((rc = get_dev_table(d->tables, d->rsqrt_idx, &p.t_rsqrt, "nm_encoder_layer(rsqrt)"))) return rc;
    const int bm = block_rows(p, &shmem);
    if (!bm) return NM_OK;
    p.ctx = ctx; p.x = x; p.y_q = y_q; p.y_f32 = y_f32; p.qkv = qkv;
    *done = true;
    return bm == 16 ? launch_block<1>(p, shmem, stream) : launch_block<2>(p, shmem, stream);
}

}  // namespace nm
