// Device-side PWL primitives (gfx950).  Compiled with -ffp-contract=off: every fused multiply-add
// is an explicit __builtin_fmaf, everything else is a separately rounded fp32 operation.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "nm_internal.h"

namespace nm {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Segment of x (paper Section 3.2: uniform segments, inputs outside the range use the edge
// segments): one subtract, one multiply, clamp in float, floor.  After the clamp u >= 0, so the
// float -> int conversion (which truncates) IS the floor.  The clamp is one median-of-three; for a
// NaN it returns the smaller bound, 0, as fmin(fmax(NaN, 0), nseg - 1) does.
__device__ __forceinline__ int seg_index(float x, float lo, float inv_w, int nseg)
{
    float u = x - lo;
    u = u * inv_w;
    u = __builtin_amdgcn_fmed3f(u, 0.0f, (float)(nseg - 1));
    return (int)u;
}

// float -> unsigned, truncating and saturating (negative and NaN -> 0).  The language leaves the conversion of a
// negative float undefined, so the instruction that does this is named.
__device__ __forceinline__ unsigned cvt_u32_sat(float x)
{
    unsigned u;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(u) : "v"(x));
    return u;
}

// y = k[s]*x + b[s] (one fma).  kb may point to LDS or to global memory.
template <typename Table>
__device__ __forceinline__ float pwl_eval(float x, const Table& t, const float2* kb, int& seg)
{
    // one median-of-three plus a select (a branch here would split the caller's unrolled loops
    // into small blocks and serialise their LDS gathers); NaN: med3 returns the smallest non-NaN
    // operand, lo, as fmin(fmax(NaN, lo), hi) does
    const float xc = __builtin_amdgcn_fmed3f(x, t.lo, t.hi);
    x = t.clamp_input ? xc : x;
    seg = seg_index(x, t.lo, t.inv_w, t.nseg);
    float2 e = kb[seg];
    return __builtin_fmaf(e.x, x, e.y);
}

// The same for a value that cannot be NaN (an int32 accumulator times finite multipliers): the
// clamp flag is folded into the bounds (clo, chi = lo, hi with the flag, -inf, +inf without), so no
// select is needed; identical results for every non-NaN x.
template <typename Table>
__device__ __forceinline__ float pwl_eval_bounded(float x, float clo, float chi, const Table& t,
                                                  const float2* kb, int& seg)
{
    x = __builtin_amdgcn_fmed3f(x, clo, chi);
    seg = seg_index(x, t.lo, t.inv_w, t.nseg);
    const float2 e = kb[seg];
    return __builtin_fmaf(e.x, x, e.y);
}
template <typename Table>
__device__ __forceinline__ float pwl_eval_bounded(float x, float clo, float chi, const Table& t,
                                                  const float2* kb)
{
    int seg;
    return pwl_eval_bounded(x, clo, chi, t, kb, seg);
}

// Without the clamp flag.
template <typename Table>
__device__ __forceinline__ float pwl_eval_noclamp(float x, const Table& t, const float2* kb, int& seg)
{
    seg = seg_index(x, t.lo, t.inv_w, t.nseg);
    const float2 e = kb[seg];
    return __builtin_fmaf(e.x, x, e.y);
}

// A table of two segments (no clamp flag): both lines, and a compare against the smallest value of
// segment 1 (found on the host with the index arithmetic itself) instead of index, gather and one
// line.  The same value as pwl_eval_noclamp for every x, NaN and infinities included.
template <typename Table>
__device__ __forceinline__ float pwl_eval_two_segments(float x, const Table& t)
{
    const float y0 = __builtin_fmaf(t.k0, x, t.b0), y1 = __builtin_fmaf(t.k1, x, t.b1);
    return x >= t.tau ? y1 : y0;
}

// ---- instructions at twice the rate -----------------------------------------------------------------
// With two or more wavefronts on a SIMD, gfx950 issues a vector instruction every 2.2 clocks, but of most kinds only one every
// 4.2: conversions, minima, maxima and medians, shifts to the left, byte permutes, three-operand integer arithmetic, and
// anything with a scalar register among its operands.  Free of that are fp32 additions, multiplications and fused
// multiply-adds (their clamp to [0, 1] and literals included), 32-bit logic, integer additions, shifts to the right and moves.
// (Measured on 256 CUs, clocks per instruction and SIMD: v_mul_f32, v_fma_f32, v_fmaak_f32, v_add_u32, v_and_b32 2.2 .. 2.5;
// v_mul_f32 with an SGPR, v_med3_f32, v_cvt_u32_f32, v_lshlrev_b32, v_lshl_add_u32, v_perm_b32, v_cvt_pk_u8_f32 4.2; both kinds in
// turn 2.2.  A single wavefront issues any of them every 5.)  A loop's time is thus 2.2 clocks an instruction or 4.2 for
// each of the slower kind, whichever is more.
//
// A uniform value in a vector register (opaque, so that no scalar register is put in its place).
__device__ __forceinline__ float in_vgpr(float x)
{
    float v;
    asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(x));
    return v;
}
// clamp(a * b + c, 0, 1) and clamp(a * b, 0, 1), rounded once in front of the clamp; a NaN becomes 0.
__device__ __forceinline__ float fma_clamp01(float a, float b, float c)
{
    float v;
    asm("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(v) : "v"(a), "v"(b), "v"(c));
    return v;
}
__device__ __forceinline__ float mul_clamp01(float a, float b)
{
    float v;
    asm("v_mul_f32 %0, %1, %2 clamp" : "=v"(v) : "v"(a), "v"(b));
    return v;
}

// A table of at most 256 segments as 512 slots of eight bytes in LDS, found by three of the faster instructions instead of four
// of the others (multiply with a scalar, clamp, convert, shift): with the position u' = u / 256 clamped to [0, 1] (the scaling is exact),
// 2048 u' + (2^23 - 0.5), rounded once, has in its low bits the integer nearest to 8 u - 0.5, which lies in
// [8 s, 8 s + 7] for every u in segment s (a tie at 8 s - 0.5 goes to the even 8 s): bits 3 .. 11 are the slot.  u below 1/16
// leaves the sum below 2^23, in the binade whose low bits then read all ones: slot 511 is segment 0 again.  Slots from nseg
// to 256 (u' = 1) hold the last segment.
constexpr int kTableSlots = 2 * kSlotSegments;
constexpr size_t kSlotBytes = kTableSlots * sizeof(float2);
__device__ __forceinline__ unsigned slot_offset(float u, float steps)   // steps: 2048 in a vector register
{
    float x;
    asm("v_fmaak_f32 %0, %1, %2, 0x4affffff" : "=v"(x) : "v"(u), "v"(steps));   // 8388607.5
    return __float_as_uint(x) & 0xff8u;
}
// The line at an offset into LDS as a whole, which the kernel's dynamic array begins (it has no other object there); added to that
// array's address, which only the linker knows to be 0, the offset would cost an instruction more.
__device__ __forceinline__ float2 slot_line(unsigned offset)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    const v2f e = *reinterpret_cast<const __attribute__((address_space(3))) v2f*>(offset);
    return make_float2(e[0], e[1]);
}
// The table into its slots, by kSlotSegments threads or more: thread i < kSlotSegments has entry min(i, nseg - 1).
__device__ __forceinline__ void write_slots(float2* s_kb, float2 entry, int i)
{
    if (i < kSlotSegments) s_kb[i] = entry;
    if (i == kSlotSegments - 1) s_kb[kSlotSegments] = entry;
    if (i == 0) s_kb[kTableSlots - 1] = entry;
}

// Symmetric int8 code: round-to-nearest-even of v * inv_scale, saturated to [-127, 127].
// Returns a word whose LOW BYTE is the code (the other bytes are not meaningful): saturate first
// (the bounds are integers and rounding is monotone, so clamp and round commute), then add
// 1.5 * 2^23: at that magnitude one ulp is 1, so the fp32 addition itself rounds to the nearest
// integer, ties to even, and the low mantissa bits are the two's-complement integer.  A NaN
// saturates to -127 (the median-of-three returns the smaller bound).
__device__ __forceinline__ int requant(float v, float inv_scale)
{
    float r = __builtin_amdgcn_fmed3f(v * inv_scale, -127.0f, 127.0f);
    return __float_as_int(r + 12582912.0f);
}

// ReLU and int8 code in one (relu_codes holds, v finite): the code of v is that of clamp(v * inv_scale, 0, 127),
// rounded, saturated and put into byte e of w by one conversion (to nearest even, as requant rounds).
__device__ __forceinline__ unsigned relu_requant(float v, float inv_scale, int e, unsigned w)
{
    return __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(v * inv_scale, 0.0f, 127.0f), e, w);
}
// Whether fma(accumulator, scale, bias) + residual stays finite whatever the accumulator (the residual's scale
// is checked by relu_codes); false for a NaN.
__device__ __forceinline__ bool relu_finite(float scale, float bias)
{
    return __builtin_fabsf(scale) <= 1e25f && __builtin_fabsf(bias) <= 1e30f;
}

// Packs the low bytes of four words into one (a in byte 0).
__device__ __forceinline__ unsigned pack4(int a, int b, int c, int d)
{
    const unsigned lo = __builtin_amdgcn_perm((unsigned)b, (unsigned)a, 0x0c0c0400u);  // a0 b0 0 0
    const unsigned hi = __builtin_amdgcn_perm((unsigned)d, (unsigned)c, 0x04000c0cu);  // 0 0 c0 d0
    return lo | hi;
}

// A row's 32 codes as a 32x32 matrix instruction leaves them (word g of a lane: columns 8 g + 4 * half, half = lane / 32) as the 16 bytes
// from column 16 * half on: the lane's piece of the row, and of the next product's operand.
__device__ __forceinline__ v4i halves_to_row(unsigned w0, unsigned w1, unsigned w2, unsigned w3)
{
    const auto a = __builtin_amdgcn_permlane32_swap(w0, w2, false, false), b = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
    return v4i{(int)a[0], (int)a[1], (int)b[0], (int)b[1]};
}
__device__ __forceinline__ unsigned quotient(unsigned n, const FastDiv& f)
{
    const unsigned q = __umulhi(n, f.magic) >> f.shift;
    return f.magic ? q : n;
}

// Copy a table's {k, b} pairs into LDS (all threads of the block take part; the caller
// synchronises before the first lookup).
__device__ __forceinline__ void stage_table(float2* dst, const DevTable& t)
{
    for (int i = threadIdx.x; i < t.nseg; i += blockDim.x) dst[i] = t.kb[i];
}

// Two-level form of a merged table (paper Algorithm 2: neighbouring primary segments with nearly
// equal slope share one line): nkb {k, b} pairs, then one byte per primary cell naming its merged
// segment.  LDS bytes: two_level_bytes (instead of 8 * nseg).
__device__ __forceinline__ void stage_table_two_level(float2* dst, const DevTable& t)
{
    for (int i = threadIdx.x; i < t.nkb; i += blockDim.x) dst[i] = t.ckb[i];
    uint8_t* map = reinterpret_cast<uint8_t*>(dst + t.nkb);
    for (int i = threadIdx.x; i < t.nseg; i += blockDim.x) map[i] = t.cellmap[i];
}

// Look-up in two steps: the primary cell of x exactly as for a uniform table (`cell` is what the
// debug outputs report), then that cell's merged segment.
__device__ __forceinline__ float pwl_eval_two_level(float x, const DevTable& t, const float2* staged, int& cell)
{
    const float xc = __builtin_amdgcn_fmed3f(x, t.lo, t.hi);
    x = t.clamp_input ? xc : x;
    cell = seg_index(x, t.lo, t.inv_w, t.nseg);
    const uint8_t* map = reinterpret_cast<const uint8_t*>(staged + t.nkb);
    const float2 e = staged[map[cell]];
    return __builtin_fmaf(e.x, x, e.y);
}

// A line of zeros in device memory: the source of operand bytes that fall into a convolution's
// padding (the direct global -> LDS loads cannot substitute a value, only an address).  One per translation unit.
static __device__ __attribute__((aligned(256))) int8_t g_zero_line[256];

// Direct global -> LDS load: every lane supplies its own global address of 16 bytes; the wavefront's
// 1 KB lands contiguously at lds_addr (wave-uniform), lane i at lds_addr + 16*i.  Asynchronous:
// completion is tracked by the vector-memory counter (wait_vmcnt), not by the LDS counter.
// The LDS address travels in M0, which is an operand of the statement (the register allocator
// knows it is written here); one wait state separates the M0 write from its use.
__device__ __forceinline__ void dma16(const void* gptr, unsigned lds_addr)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gptr), "{m0}"(lds_addr) : "memory");
}

// The same with a wave-uniform base pointer and a 32-bit per-lane byte offset (the k-loop then
// advances one scalar pointer instead of one 64-bit address per lane and load).
__device__ __forceinline__ void dma16s(const void* sbase, unsigned voff, unsigned lds_addr)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sbase), "{m0}"(lds_addr) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// One butterfly step: op(v, value of lane ^ MASK), without going through LDS.  Masks 1 and 2 are
// quad permutes, 4 and 8 compositions of the row mirrors (lane ^ 7 ^ 3, lane ^ 15 ^ 7), 16 and 32
// the gfx950 row / half swaps: swapping a register with a copy of itself leaves {even rows twice}
// in one and {odd rows twice} in the other (halves likewise), and op is commutative, so
// op(first, second) is op(v, partner) in every lane.
template <int MASK, typename Op>
__device__ __forceinline__ int butterfly_step(int v, Op op)
{
    if (MASK == 1) return op(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false));
    if (MASK == 2) return op(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false));
    if (MASK == 4) {
        const int t = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);   // lane ^ 7
        return op(v, __builtin_amdgcn_update_dpp(0, t, 0x1B, 0xf, 0xf, false));     // ... ^ 3
    }
    if (MASK == 8) {
        const int t = __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false);   // lane ^ 15
        return op(v, __builtin_amdgcn_update_dpp(0, t, 0x141, 0xf, 0xf, false));    // ... ^ 7
    }
    if (MASK == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
        return op((int)r[0], (int)r[1]);
    }
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return op((int)r[0], (int)r[1]);
}

struct AddF32 {
    __device__ __forceinline__ int operator()(int a, int b) const { return __float_as_int(__int_as_float(a) + __int_as_float(b)); }
};
struct MaxF32 {
    __device__ __forceinline__ int operator()(int a, int b) const { return __float_as_int(__builtin_fmaxf(__int_as_float(a), __int_as_float(b))); }
};
struct MaxI32 {
    __device__ __forceinline__ int operator()(int a, int b) const { return max(a, b); }
};

// Butterfly over the G lanes that own a row, partner masks G/2 ... 1 in that order.
template <int G, typename Op>
__device__ __forceinline__ int group_reduce(int v, Op op)
{
    if (G > 32) v = butterfly_step<32>(v, op);
    if (G > 16) v = butterfly_step<16>(v, op);
    if (G > 8) v = butterfly_step<8>(v, op);
    if (G > 4) v = butterfly_step<4>(v, op);
    if (G > 2) v = butterfly_step<2>(v, op);
    if (G > 1) v = butterfly_step<1>(v, op);
    return v;
}

template <int G>
__device__ __forceinline__ float group_sum(float v)
{
    return __int_as_float(group_reduce<G>(__float_as_int(v), AddF32{}));
}

}  // namespace nm
