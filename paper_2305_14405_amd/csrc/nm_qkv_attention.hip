// QKV projection and attention of a head in one kernel, for sequences of at most 128 tokens (paper Section 3.1: linear layers and
// attention as matrix products, Section 3.2: exp and 1/x as PWL tables; arithmetic and order are those of the separate kernels, so results
// are bit-identical): gemm_tile_kernel with 128 tokens (one sequence, or two of at most 64) x the 192 columns of one head's Q, K
// and V, whose codes go to LDS as the images that attention's wavefronts read; no tensor of them exists in memory.
//
// What bounds it: the operands' stream into LDS (40 KB a slice for 128 x 192 outputs, of 40 bytes per clock and CU), then
// attention's vector instructions, which the other workgroup of a CU hides where there are two (by counter, 32 x 128 tokens and 12 heads,
// vector instructions issue in 38 % of the cycles, the matrix cores run in 24 %, LDS is busy in 23 %).  As two kernels the projection's
// prologue and epilogue, a launch, and Q, K and V on their way through memory come on top.  us a layer, two kernels -> this one:
// 32 x 128 tokens of width 768 71.0 -> 68.4, 128 x 128 202 -> 191, 16 x 128 49.7 -> 47.3, 128 x 64 119 -> 114, 128 x 128 of width 1024
// 302 -> 284, 64 x 128 of width 384 64.8 -> 59.5.  qkv_attention_form has the rest.
#include "nm_gemm_tile.h"

namespace nm {

bool qkv_attention_takes(const AttnArgs& a, const GemmArgs& g)
{
    return !gemm_switched() && a.S <= 128 && a.H == 64 * a.heads && g.K % 16 == 0 && aligned(g.A, 16) && aligned(g.W, 16) && (!g.bias || aligned(g.bias, 4)) &&
           aligned(a.ctx, 4) && !a.scores_out && !a.p_out && (int64_t)g.M * g.lda < (1LL << 32) && (int64_t)g.N * g.ldw < (1LL << 32);
}

int32_t launch_qkv_attention(const AttnArgs& a, const GemmArgs& g, const char* what, hipStream_t stream, bool* done)
{
    *done = false;
    const int form = qkv_attention_form(a.B, a.S, a.heads, g.K);
    if (form == QKV_ATTENTION_NONE) return NM_OK;
    QkvAttnParams p{};
    AttnExp e;
    int32_t rc = attn_params(a, what, &p.at, &e);
    if (rc) return rc;
    if (e.slots == SLOTS_NONE || p.at.t_recip.nseg > kQkvRecip) return NM_OK;
    p.B = a.B; p.keys_log2 = a.S <= 64 ? 6 : 7; p.pow2 = e.slots == SLOTS_POW2;
    p.M = (int)(((int64_t)a.B + (128 >> p.keys_log2) - 1) >> (7 - p.keys_log2)) * 128; p.N = 192 * a.heads; p.K = g.K;
    p.A = g.A; p.lda = g.lda; p.W = g.W; p.ldw = g.ldw; p.inner_count = 1;
    p.bias = g.bias; p.alpha = g.alpha;
    for (int i = 0; i < 3; ++i) p.inv3[i] = g.inv3[i];
    const auto launch = [&](auto end_c) {
        constexpr bool kEnd = decltype(end_c)::value;
        return form == QKV_ATTENTION_EIGHT ? launch_tile_epi<128, 192, 2, 2, 3, EPI_ATTENTION, 128, false, 2, kEnd>(p, 0, stream)
                                           : launch_tile_epi<128, 192, 2, 2, 2, EPI_ATTENTION, 128, false, 1, kEnd>(p, 0, stream);
    };
    rc = g.K % 128 ? launch(std::true_type{}) : launch(std::false_type{});
    if (rc) return rc;
    *done = true;
    return check_hip(hipGetLastError(), "QKV + attention launch");
}

}  // namespace nm
