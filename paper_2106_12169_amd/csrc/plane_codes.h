// Results of the matrix instruction -> planes of one- and two-bit codes, made in the lane that holds them.
//
// The matrix instruction gets the weights as its row operand: accumulator register r of lane (half lh, lr) is channel
// row 8 (r / 4) + 4 lh + r % 4 of a 32-channel tile and pixel lr.  A lane then holds sixteen channels of one pixel, and the
// planes of their codes are made without a lane exchange per value: t / 4 clamped to [0, 1] by the multiply-add's own clamp,
// truncated to FP4 codes 0, 0.5, 1, 1.5 (2 for t >= 4) two at a time by the converter's stochastic rounding with seed 0, whose two
// low bits are the planes.  The weight rows are dealt to the matrix rows so that nibble j of dword q in half lh is channel
// 4 j + 2 lh + q: both halves' nibbles interleave into the plane word with one lane swap.  2.5 vector instructions per value
// against about 14 with a compare and lane writes per value (finish_rows8).
#pragma once
#include "lane_util.h"

#include <cstdint>

namespace apnn {

// n / d = (n m) >> s for 0 <= n < 2^31 (round-up reciprocal)
struct Divisor {
    uint32_t m;
    int s, d;
};

inline Divisor divisor(int64_t d)
{
    Divisor r{0, 0, static_cast<int>(d)};
    int bits = 0;
    while ((int64_t(1) << bits) < d) ++bits;
    r.s = 31 + bits;                                     // n < 2^31: the error n (m d - 2^s) / 2^s stays below 1
    r.m = static_cast<uint32_t>((uint64_t(1) << r.s) / static_cast<uint64_t>(d) + 1);
    return r;
}

// Channel of a 32-channel tile for matrix row `row`, and of register r in lane half h.
__device__ __forceinline__ int code_channel_of_row(int row) { return 16 * ((row >> 3) & 1) + 4 * (row & 3) + 2 * ((row >> 2) & 1) + (row >> 4); }
__device__ __forceinline__ int code_channel(int r, int h) { return 16 * ((r >> 2) & 1) + 4 * (r & 3) + 2 * h + (r >> 3); }

// x / 4, and never zero unless x is: a sum rounds by the sign of what it loses.
__device__ __forceinline__ float quarter(float x)
{
    const float q = 0.25f * x;
    return q == 0.0f && x != 0.0f ? copysignf(__uint_as_float(1u), x) : q;
}

__device__ __forceinline__ int divide(int n, const Divisor &d)
{
    return static_cast<int>((static_cast<uint64_t>(static_cast<uint32_t>(n)) * d.m) >> d.s);
}

// a, b, c -> clamp(a b + c, 0, 1) in one instruction; NaN gives 0 (the clamp bit).  ACCUMULATOR: an operand is what a matrix
// instruction wrote.  Its first reader has to wait, and the compiler counts the wait only for instructions it sees, so there
// the instruction is left to it to make; elsewhere the statement keeps it from moving the pooling and the residual around (a pooled
// layer of 128 channels, 8 x 112 x 112: 18.4 us, 19.2 with the expression).
template <bool ACCUMULATOR> __device__ __forceinline__ float fma_clamp(float a, float b, float c)
{
    if constexpr (ACCUMULATOR) return __builtin_amdgcn_fmed3f(__fmaf_rn(a, b, c), 0.0f, 1.0f);
    float t;
    asm("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(t) : "v"(a), "v"(b), "v"(c));
    return t;
}

typedef float v2f_t __attribute__((ext_vector_type(2)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef int v4i_t __attribute__((ext_vector_type(4)));

// Byte B of d: two FP4 codes of 2 t, truncated (stochastic rounding, seed 0).  Written out because the compiler's builtin
// does not keep the other bytes of its destination.
template <int B> __device__ __forceinline__ void two_codes(uint32_t &d, v2f_t t)
{
    if constexpr (B == 0) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, 0, 0.5" : "+v"(d) : "v"(t));
    else if constexpr (B == 1) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, 0, 0.5 op_sel:[0,0,1,0]" : "+v"(d) : "v"(t));
    else if constexpr (B == 2) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, 0, 0.5 op_sel:[0,0,0,1]" : "+v"(d) : "v"(t));
    else asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, 0, 0.5 op_sel:[0,0,1,1]" : "+v"(d) : "v"(t));
}

// (mask & a) | (~mask & b)
__device__ __forceinline__ uint32_t mask_select(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }

// Eight values of a lane (results / 4 of the channels 4 j + 2 lh + q of a tile) -> eight nibbles: code k < 4 is k, everything
// above it 4.  sc, bi: the channels' constants, bi a quarter of the bias; res: the residual's codes, a nibble each.  ACCUMULATOR: the
// values are a matrix instruction's own.
template <bool ACCUMULATOR>
__device__ __forceinline__ uint32_t nibbles(const float (&v)[8], const v4f_t (&sc)[2], const v4f_t (&bi)[2], bool with_res,
                                            float res_scale, uint32_t res)
{
    uint32_t d = 0u;
    if (with_res) {
        static_for<4>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            const v2f_t c = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(res, 0.5f, b);        // code / 4
            v2f_t t;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                t[i] = fma_clamp<false>(res_scale, c[i], __fmaf_rn(sc[b / 2][2 * (b & 1) + i], v[2 * b + i], bi[b / 2][2 * (b & 1) + i]));
            two_codes<b>(d, t);
        });
    } else {
        static_for<4>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            v2f_t t;
#pragma unroll
            for (int i = 0; i < 2; ++i) t[i] = fma_clamp<ACCUMULATOR>(sc[b / 2][2 * (b & 1) + i], v[2 * b + i], bi[b / 2][2 * (b & 1) + i]);
            two_codes<b>(d, t);
        });
    }
    return d;
}

// Nibbles of q = 0 and 1 -> plane words of the tile's 32 channels: lanes of half b return the word of plane b.
__device__ __forceinline__ uint32_t plane_words(uint32_t x, uint32_t y, int q_out)
{
    // plane 0 = bit 0 | bit 2, plane 1 = bit 1 | bit 2; bits 0 (x) and 1 (y) of each nibble are kept
    uint32_t p0 = mask_select(0x11111111u, x | (x >> 2), (y << 1) | (y >> 1));
    const uint32_t p1 = mask_select(0x11111111u, (x >> 1) | (x >> 2), y | (y >> 1));
    if (q_out == 1) p0 |= p1;                           // clamp at 1
    const auto both = __builtin_amdgcn_permlane32_swap(p0, p1, false, false);    // half b: plane b of either half's channels
    return mask_select(0x33333333u, both[0], both[1] << 2);
}

}  // namespace apnn
