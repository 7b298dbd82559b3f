// Bit decomposition and packing kernels (Sec. 3.1 Eq. 2; channel-major
// organisation of Sec. 4.2 (a); quantisation layer of Sec. 5.2).
//
// One thread produces the 32-bit word(s) of one (row, k-word) position for all
// planes: it reads 32 source values, takes bit t of each (Eq. 2) and gathers
// them LSB-first into the word of plane t.  The work is HBM-bound: rows*K bytes
// in, rows*K*bits/8 bytes out.
#include <cmath>
#include <type_traits>

#include "common.h"

namespace apnn {

// 4 bytes holding 0/1 each -> 4-bit number, byte 0 in bit 0.  The multiplier
// places byte i at bit 24+i; the stray partial products all land below bit 24
// in distinct positions, so nothing carries into the result.
__device__ __forceinline__ uint32_t gather4(uint32_t ones)
{
    return (ones * 0x01020408u) >> 24;
}

// Per-byte "value > 0" for int8 bytes: low seven bits non-zero and sign clear.
__device__ __forceinline__ uint32_t positive_bytes(uint32_t d)
{
    const uint32_t nz = (((d & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) >> 7) & 0x01010101u;
    return nz & ~(d >> 7);
}

struct PackGeom {
    int64_t rows;      // logical rows (matrix rows, pixels, or Cout*R*S)
    int64_t K;         // values per row
    int64_t row_stride;// source bytes between rows (within one outer block)
    int64_t k_stride;  // source bytes between consecutive k
    int64_t outer_div; // source: row -> (row / outer_div, row % outer_div)
    int64_t outer_stride; // source bytes per outer block
    int64_t inner_n;   // destination: row -> (row / inner_n, row % inner_n)
    int ldw;           // destination words per plane row
    int bits;
    int pm1;
};

// dst word index of (row, plane t, word kw)
__device__ __forceinline__ size_t dst_index(const PackGeom &g, int64_t row, int t, int kw)
{
    const int64_t outer = row / g.inner_n, inner = row - outer * g.inner_n;
    return (static_cast<size_t>(outer * g.bits + t) * g.inner_n + inner) * g.ldw + kw;
}

__global__ __launch_bounds__(256) void pack_generic_kernel(const uint8_t *__restrict__ src,
                                                           uint32_t *__restrict__ dst, PackGeom g, int64_t first)
{
    const int64_t idx = first + static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t total = g.rows * g.ldw;
    if (idx >= total) return;
    const int64_t row = idx / g.ldw;
    const int kw = static_cast<int>(idx - row * g.ldw);
    const int64_t ro = row / g.outer_div, ri = row - ro * g.outer_div;
    const uint8_t *s = src + ro * g.outer_stride + ri * g.row_stride;
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t k0 = static_cast<int64_t>(kw) * 32;
    if (g.k_stride == 1 && k0 + 32 <= g.K && ((reinterpret_cast<uintptr_t>(s + k0) & 15u) == 0)) {
        const uint4 lo = *reinterpret_cast<const uint4 *>(s + k0);
        const uint4 hi = *reinterpret_cast<const uint4 *>(s + k0 + 16);
        const uint32_t d[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (g.pm1) {
                w[0] |= gather4(positive_bytes(d[i])) << (4 * i);
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (t < g.bits) w[t] |= gather4((d[i] >> t) & 0x01010101u) << (4 * i);
            }
        }
    } else {
        for (int b = 0; b < 32; ++b) {
            const int64_t k = k0 + b;
            if (k >= g.K) break;
            const uint8_t v = s[k * g.k_stride];
            if (g.pm1) {
                w[0] |= static_cast<uint32_t>(static_cast<int8_t>(v) > 0) << b;
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (t < g.bits) w[t] |= ((static_cast<uint32_t>(v) >> t) & 1u) << b;
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (t < g.bits) dst[dst_index(g, row, t, kw)] = w[t];
}

// Quantiser + packer.  A wave owns 256 NL consecutive values of a row: NL loads of 16 bytes per lane, all in flight
// together, lane l holding values 4 l .. 4 l + 3 of each 256.  Per value: subtract, multiply or divide, clamp, truncate into a byte
// (v_cvt_pk_u8_f32 of a clamped floor); per load and plane the four bits are gathered by one dot product with (1, 2, 4,
// 8), shifted to their nibble of the word and OR-ed over the eight lanes of the word by three lane exchanges inside
// a row; lane l then keeps word l / 8 of load l % 8, and a plane of the segment leaves in one store.
// Bound by HBM: 4096 x 4096 fp32 -> 2 bits take 12.1 us (5.9 TB/s).  The ballot form it replaces spent some 40 vector
// instructions per value, half of them on the division, and took 20.8 us.
//
// The quotient must be that of one IEEE division, fl(d / step).  EXACT: step is a power of two, so d * (1 / step) is
// that number.  Otherwise v = d * fl(1 / step) is within 2 ulp of it, i.e. within 2^-13 for |v| <= 257, and the code,
// clamp(floor(v)), can differ only if v lies that close to one of the integers 1 .. hi: where the 256 values of a load
// hold one that does, they are divided.  Zeros, as a rectifier leaves them, saturated values and positions beyond K are
// decided without.  The test is of the whole wave, a scalar branch: as a branch of the lane the compiler turned it into a
// division for every value and a selection (4096 x 4096, step 0.7, to 2 bits 14.6 us, to 8 bits 21.4; now 13.1 and 16.9).
//
// SHORT: rows of at most 128 values, whose planes are four words.  A load takes two rows, lanes 0 - 31 and 32 - 63, and a
// wave owns 2 NL rows: with a wave per row most lanes have nothing to do (50000 x 64 -> 2 bits: 10.5 us, here 6.1).
template <int NL, bool EXACT, bool SHORT>
__global__ __launch_bounds__(256) void quantize_pack_wave_kernel(const float *__restrict__ src, uint32_t *__restrict__ dst,
                                                                 uint32_t waves, int segs, uint32_t rows, int K, int ldw,
                                                                 int bits, float zero, float step, float inv)
{
    const int lane = threadIdx.x & 63;
    const uint32_t wave = blockIdx.x * 4u + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);     // scalar: so are segment and row
    if (wave >= waves) return;
    const float hi = static_cast<float>((1 << bits) - 1);
    // this lane's values: k0 .. k0 + 3 of load 0; load i is 256 values on, or (SHORT) two rows
    const uint32_t row = SHORT ? wave * (2u * NL) + (lane >> 5) : wave / static_cast<uint32_t>(segs);
    const int first = SHORT ? 0 : static_cast<int>(wave - row * segs) * (256 * NL);
    const int k0 = SHORT ? 4 * (lane & 31) : first + 4 * lane;
    constexpr int KSTEP = SHORT ? 0 : 256;
    constexpr int RSTEP = SHORT ? 2 : 0;
    const float *s = src + static_cast<size_t>(row) * K + k0;
    float x[NL][4];
    if (!SHORT && first + 256 * NL <= K) {              // wave-uniform: the whole segment exists
#pragma unroll
        for (int i = 0; i < NL; ++i) __builtin_memcpy(x[i], s + 256 * i, 16);
    } else {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const float *si = s + static_cast<size_t>(RSTEP * i) * K + KSTEP * i;
#pragma unroll
            for (int j = 0; j < 4; ++j) x[i][j] = -__builtin_inff();
            if (SHORT && row + RSTEP * i >= rows) continue;
            if (k0 + KSTEP * i + 4 <= K) {
                __builtin_memcpy(x[i], si, 16);
            } else {
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    if (k0 + KSTEP * i + j < K) x[i][j] = si[j];
            }
        }
    }
    uint32_t code[NL];                                  // four codes, one per byte (below zero, -inf, NaN: 0)
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        code[i] = 0;
        float d[4], v[4];
        bool near = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[j] = __fsub_rn(x[i][j], zero);
            v[j] = __fmul_rn(d[j], inv);
            const float in = __builtin_amdgcn_fmed3f(v[j], 0.5f, hi + 0.5f);       // (halves, and for NaN, lie far from integers)
            near |= fabsf(in - rintf(in)) <= 0x1p-13f;
        }
        if (!EXACT && __builtin_amdgcn_ballot_w64(near) != 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = __fdiv_rn(d[j], step);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) code[i] = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(floorf(v[j]), 0.0f, hi), j, code[i]);
        if (first + (SHORT ? 128 : 256 * NL) > K) {     // positions beyond K are 0 (-inf - zero may be NaN or clamp to 0)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k0 + KSTEP * i + j >= K) code[i] &= ~(0xFFu << (8 * j));
        }
    }
    // the word that this lane keeps and stores
    const int nibble = 4 * (lane & 7), k_word = SHORT ? (lane >> 3) & 3 : first / 32 + 8 * (lane & 7) + (lane >> 3);
    const uint32_t my_row = SHORT ? row + 2 * (lane & 7) : row;
    const bool mine = (lane & 7) < NL && (SHORT ? my_row < rows : k_word < ldw);
    for (int t = 0; t < bits; ++t) {
        uint32_t word = 0;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            uint32_t w = __builtin_amdgcn_udot4((code[i] >> t) & 0x01010101u, 0x08040201u, 0u, false) << nibble;
            // OR over the eight lanes of a word: xor 1, xor 2 (quad permutes), mirror of eight
            w |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w), 0xB1, 0xF, 0xF, true));
            w |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w), 0x4E, 0xF, 0xF, true));
            w |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w), 0x141, 0xF, 0xF, true));
            word = (lane & 7) == i ? w : word;
        }
        if (mine) dst[(static_cast<size_t>(my_row) * bits + t) * ldw + k_word] = word;
    }
}

// ---- bytes -> plane words.  x[i], i = 0 .. 7, holds the codes of positions i, 8 + i, 16 + i, 24 + i in its four bytes
// (or, with one byte per pixel, channel i of four pixels): bit t of byte j of x[i] goes to bit 8 j + i of w[t].

// Bits selected by m of b change places with the bits D higher in a.
template <int D> __device__ __forceinline__ void swap_bits(uint32_t &a, uint32_t &b, uint32_t m)
{
    const uint32_t na = (a & m) | ((b << D) & ~m), nb = ((a >> D) & m) | (b & ~m);
    a = na;
    b = nb;
}

// One or two planes: the bits of a plane are OR-ed together position by position.  More: 8 x 8 bit-matrix
// transposition inside every byte column (the stores of planes that do not exist drop the work behind them).
template <int BITS> __device__ __forceinline__ void bytes_to_planes(uint32_t (&x)[8], uint32_t (&w)[BITS])
{
    if constexpr (BITS <= 2) {
#pragma unroll
        for (int t = 0; t < BITS; ++t) {
            w[t] = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[t] |= (i >= t ? x[i] << (i - t) : x[i] >> (t - i)) & (0x01010101u << i);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) swap_bits<4>(x[i], x[i + 4], 0x0F0F0F0Fu);
#pragma unroll
        for (int i = 0; i < 8; i += 4) {
            swap_bits<2>(x[i], x[i + 2], 0x33333333u);
            swap_bits<2>(x[i + 1], x[i + 3], 0x33333333u);
        }
#pragma unroll
        for (int i = 0; i < 8; i += 2) swap_bits<1>(x[i], x[i + 1], 0x55555555u);
#pragma unroll
        for (int t = 0; t < BITS; ++t) w[t] = x[t];
    }
}

// Transposition of 4 x 4 bytes: byte j of r[i] <-> byte i of r[j].
__device__ __forceinline__ void transpose_bytes(uint32_t &r0, uint32_t &r1, uint32_t &r2, uint32_t &r3)
{
    // __builtin_amdgcn_perm(hi, lo, sel): selector 0-3 takes a byte of lo, 4-7 of hi
    const uint32_t a = __builtin_amdgcn_perm(r1, r0, 0x05010400u), b = __builtin_amdgcn_perm(r1, r0, 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(r3, r2, 0x05010400u), d = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
    r0 = __builtin_amdgcn_perm(c, a, 0x05040100u);
    r1 = __builtin_amdgcn_perm(c, a, 0x07060302u);
    r2 = __builtin_amdgcn_perm(d, b, 0x05040100u);
    r3 = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// Row-major source (matrix operand or NHWC feature map), any K and any alignment; one thread per word of a row.  The 32
// bytes of a word are two 16-byte loads at byte addresses; the last, incomplete word of a row loads the row's last 32
// bytes and shifts its planes down, so no byte outside the row is read (rows of fewer than 32 bytes go byte by byte).
// Bound by HBM: 4096 x 4096 2-bit codes take 3.5 us, 1.9 of them the launch.  The generic kernel, which took every row whose length is no
// multiple of 16, read such rows byte by byte: 777 rows of 1999 codes 9.6 us, here under 3 us.
template <int BITS, bool PM1>
__global__ __launch_bounds__(256) void pack_rows_kernel(const uint8_t *__restrict__ src, uint32_t *__restrict__ dst,
                                                        uint32_t total, int K, int ldw)
{
    const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const uint32_t row = idx / static_cast<uint32_t>(ldw);
    const int kw = static_cast<int>(idx - row * ldw);
    const uint8_t *s = src + static_cast<size_t>(row) * K;
    const int k0 = kw * 32;
    uint32_t w[BITS];
#pragma unroll
    for (int t = 0; t < BITS; ++t) w[t] = 0;
    if (k0 < K) {
        uint32_t x[8];
        int down = 0;                                   // plane bits below the word's first position
        if (K >= 32) {
            const int kl = min(k0, K - 32);
            down = k0 - kl;
            uint32_t d[8];
            __builtin_memcpy(d, s + kl, 16);
            __builtin_memcpy(d + 4, s + kl + 16, 16);
            // dwords of positions 8 j .. 8 j + 3 (even) and 8 j + 4 .. 8 j + 7 (odd) -> one register per position mod 8
#pragma unroll
            for (int i = 0; i < 4; ++i) { x[i] = d[2 * i]; x[4 + i] = d[2 * i + 1]; }
            transpose_bytes(x[0], x[1], x[2], x[3]);
            transpose_bytes(x[4], x[5], x[6], x[7]);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = 0;
#pragma unroll
            for (int k = 0; k < 32; ++k)
                if (k < K) x[k & 7] |= static_cast<uint32_t>(s[k]) << (k & 24);
        }
        if constexpr (PM1) {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = positive_bytes(x[i]);
        }
        bytes_to_planes<BITS>(x, w);
#pragma unroll
        for (int t = 0; t < BITS; ++t) w[t] >>= down;
    }
    uint32_t *o = dst + static_cast<size_t>(row) * BITS * ldw + kw;
#pragma unroll
    for (int t = 0; t < BITS; ++t) o[static_cast<size_t>(t) * ldw] = w[t];
}

// N x C x H x W source into the fmap layout.  A block owns PX consecutive pixels of one image: thread = four consecutive
// pixels of one channel word, one dword load per channel (at byte addresses: H W need not be a multiple of 4; the
// last four pixels of an image are loaded whole, overlapping their neighbours), contiguous across PX / 4 lanes.  The
// plane words go to an LDS image of the block's output record ([pixel][plane][channel word], the pixel stride padded
// to an odd number of words) and leave as contiguous 4-byte-per-lane stores: both sides of the transposition are
// coalesced.  PX = 256 keeps whole cache lines together; PX = 64 gives small feature maps four times the blocks (4 x 96
// x 27 x 31, 4 bits: 10.8 us in the generic kernel, one byte per load, here under 4 us).  Dynamic LDS: PX (BITS Cw | 1) words.
template <int BITS, bool PM1, int PX>
__global__ __launch_bounds__(256) void pack_nchw_kernel(const uint8_t *__restrict__ src, uint32_t *__restrict__ dst,
                                                        int C, int HW, int Cw, int blocks_per_image)
{
    extern __shared__ uint32_t rec[];
    constexpr int G = PX / 4;                           // groups of four pixels
    const int n = blockIdx.x / blocks_per_image, p0 = (blockIdx.x - n * blocks_per_image) * PX;    // first pixel of the block
    const int npix = min(PX, HW - p0);
    const int RW = BITS * Cw, PS = RW | 1;              // words per pixel record, padded stride in LDS
    const int l0 = 4 * (static_cast<int>(threadIdx.x) % G);
    const int first = min(p0 + l0, HW - 4);             // (HW >= 4: host)
    if (l0 < npix) {
        for (int cw = threadIdx.x / G; cw < Cw; cw += 256 / G) {
            const uint8_t *s = src + (static_cast<size_t>(n) * C + 32 * cw) * HW + first;
            uint32_t d[32];
#pragma unroll
            for (int c = 0; c < 32; ++c) {
                d[c] = 0;
                if (32 * cw + c < C) __builtin_memcpy(&d[c], s + static_cast<size_t>(c) * HW, 4);
            }
            uint32_t pl[4][BITS];                       // [channels 8 k .. 8 k + 7][plane], byte = pixel
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = PM1 ? positive_bytes(d[8 * k + i]) : d[8 * k + i];
                bytes_to_planes<BITS>(x, pl[k]);
            }
#pragma unroll
            for (int t = 0; t < BITS; ++t) {
                transpose_bytes(pl[0][t], pl[1][t], pl[2][t], pl[3][t]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int px = first - p0 + j;      // below 0: a pixel of the previous block
                    if (px >= 0) rec[px * PS + t * Cw + cw] = pl[j][t];
                }
            }
        }
    }
    __syncthreads();
    uint32_t *o = dst + (static_cast<size_t>(n) * HW + p0) * RW;
    for (int i = threadIdx.x; i < npix * RW; i += 256) {
        const int px = i / RW;
        o[i] = rec[px * PS + (i - px * RW)];
    }
}

__global__ __launch_bounds__(256) void quantize_pack_kernel(const float *__restrict__ src,
                                                            uint32_t *__restrict__ dst, int64_t rows,
                                                            int64_t K, int ldw, int bits, float zero,
                                                            float step, int64_t first)
{
    const int64_t idx = first + static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (idx >= rows * ldw) return;
    const int64_t row = idx / ldw;
    const int kw = static_cast<int>(idx - row * ldw);
    const float hi = static_cast<float>((1 << bits) - 1);
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int b = 0; b < 32; ++b) {
        const int64_t k = static_cast<int64_t>(kw) * 32 + b;
        if (k >= K) break;
        // (x - z) / s with one rounding per operation, then floor and clamp
        const float d = __fsub_rn(src[row * K + k], zero);
        const float v = __fdiv_rn(d, step);
        float f = floorf(v);
        f = (f >= 0.0f) ? f : 0.0f;          // negatives and NaN -> 0
        f = (f > hi) ? hi : f;
        const uint32_t code = static_cast<uint32_t>(f);
#pragma unroll
        for (int t = 0; t < 8; ++t)
            if (t < bits) w[t] |= ((code >> t) & 1u) << b;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (t < bits) dst[(static_cast<size_t>(row) * bits + t) * ldw + kw] = w[t];
}

// Input-layer receptive-field packing: word r of an output pixel holds bit
// (c*S + s) = bit t of image[n][c][ho*stride+r-pad][wo*stride+s-pad].
//
// Row kernel (the usual case).  With the taps of one channel adjacent in the word,
// the S bits of (pixel, r, c, t) are S consecutive bits of the bit string "plane t of
// image row h, channel c".  A block owns one output row (n, ho): it first splits the
// R x C image rows it needs into plane bit strings in LDS (one thread per 32 pixels,
// the same byte gather as the matrix packer; two zero words in front and behind take
// the place of the frame overhang), then every thread assembles output words from
// S-bit fields cut out of those strings with a funnel shift and writes them as
// 16-byte vectors in destination order.  Per output word: C x (two LDS reads, one
// funnel shift, one mask-and-insert) instead of S*C byte loads and gathers.
__global__ __launch_bounds__(256) void pack_patches_rows_kernel(const uint8_t *__restrict__ img,
                                                                uint32_t *__restrict__ dst, int C, int H, int W,
                                                                int Ho, int Wo, int R, int S, int stride, int pad,
                                                                int bits, int LDW, int RW)
{
    extern __shared__ uint32_t rows[];                  // [R][C][bits][RW]; the string starts at word 1
    const int tid = threadIdx.x;
    const int ho = blockIdx.x % Ho;
    const int64_t n = blockIdx.x / Ho;
    const int Ww = (W + 31) / 32;
    for (int i = tid; i < R * C * bits * RW; i += 256) rows[i] = 0;
    __syncthreads();
    for (int item = tid; item < R * C * Ww; item += 256) {
        const int j = item % Ww, rc = item / Ww, c = rc % C, r = rc / C;
        const int h = ho * stride - pad + r;
        if (h < 0 || h >= H) continue;
        const uint8_t *src = img + ((n * C + c) * H + h) * static_cast<int64_t>(W) + 32 * j;
        uint32_t d[8];
        if (32 * j + 32 <= W && (reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = reinterpret_cast<const uint32_t *>(src)[i];
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                d[i] = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (32 * j + 4 * i + b < W) d[i] |= static_cast<uint32_t>(src[4 * i + b]) << (8 * b);
            }
        }
        for (int t = 0; t < bits; ++t) {
            uint32_t w = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) w |= gather4((d[i] >> t) & 0x01010101u) << (4 * i);
            rows[((r * C + c) * bits + t) * RW + 1 + j] = w;
        }
    }
    __syncthreads();
    const uint32_t field = (1u << S) - 1u;
    const int Q = LDW / 4;                              // 16-byte vectors per (pixel, plane)
    uint32_t *out = dst + (static_cast<int64_t>(blockIdx.x) * Wo) * bits * LDW;
    for (int v = tid; v < Wo * bits * Q; v += 256) {
        const int q = v % Q, t = (v / Q) % bits, wo = v / (Q * bits);
        const int xb = wo * stride - pad + 32;          // bit position of tap s = 0 in the string (>= 0: pad <= 32)
        const int wi = xb >> 5, sh = xb & 31;
        uint32_t w4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int r = 4 * q + k;
            uint32_t w = 0;
            if (r < R) {
                for (int c = 0; c < C; ++c) {
                    const uint32_t *str = &rows[((r * C + c) * bits + t) * RW + wi];
                    w |= (__funnelshift_r(str[0], str[1], sh) & field) << (c * S);
                }
            }
            w4[k] = w;
        }
        *reinterpret_cast<uint4 *>(out + static_cast<int64_t>(v) * 4) = make_uint4(w4[0], w4[1], w4[2], w4[3]);
    }
}

// General kernel (any geometry that fits the word): a block handles 32 output
// pixels; thread (pixel, r) collects the S*C bytes of kernel row
// r four to a register, every plane takes one bit of each byte with the same
// gather as the row packer, and the 32 x bits x ldw words of the block, which are
// contiguous in the destination, leave through LDS as coalesced 16-byte stores.
__global__ __launch_bounds__(256) void pack_patches_kernel(const uint8_t *__restrict__ img,
                                                           uint32_t *__restrict__ dst, int64_t npix,
                                                           int C, int H, int W, int Ho, int Wo, int R, int S,
                                                           int stride, int pad, int bits, int LDW)
{
    // LDW = words per plane row, 4 or 8 (host checks R <= 8)
    __shared__ __attribute__((aligned(16))) uint32_t tile[32 * 8 * 8];
    const int tid = threadIdx.x;
    const int r = tid & 7, lp = tid >> 3;                // kernel row, pixel inside the block
    const int64_t pix = static_cast<int64_t>(blockIdx.x) * 32 + lp;
    uint32_t d[8] = {0, 0, 0, 0, 0, 0, 0, 0};            // byte (c*S + s) of the kernel row, 4 per register
    if (pix < npix) {
        const int wo = static_cast<int>(pix % Wo);
        const int ho = static_cast<int>((pix / Wo) % Ho);
        const int64_t n = pix / (static_cast<int64_t>(Wo) * Ho);
        const int h = ho * stride + r - pad;
        if (r < R && h >= 0 && h < H) {
            const int x0 = wo * stride - pad;
            int sc = 0, c = 0;                               // i = c*S + sc, stepped without dividing
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const int x = x0 + sc;
                if (i < S * C && x >= 0 && x < W)
                    d[i >> 2] |= static_cast<uint32_t>(img[((n * C + c) * H + h) * W + x]) << (8 * (i & 3));
                if (++sc == S) { sc = 0; ++c; }
            }
        }
    }
    for (int t = 0; t < bits; ++t) {
        uint32_t w = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) w |= gather4((d[i] >> t) & 0x01010101u) << (4 * i);
        if (r < LDW) tile[(lp * bits + t) * LDW + r] = w;
    }
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * 32 * bits * LDW;      // words
    const int64_t limit = npix * bits * LDW;
    for (int v = tid; v < 32 * bits * LDW / 4; v += 256)
        if (base + 4 * v < limit)
            *reinterpret_cast<uint4 *>(dst + base + 4 * v) = *reinterpret_cast<const uint4 *>(&tile[4 * v]);
}

__global__ __launch_bounds__(256) void pack_patch_weights_kernel(const uint8_t *__restrict__ wsrc,
                                                                 uint32_t *__restrict__ dst, int Cout, int Cin,
                                                                 int R, int S, int bits, int pm1, int ldw)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= Cout * ldw) return;
    const int co = idx / ldw, r = idx - co * ldw;
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (r < R) {
        for (int s = 0; s < S; ++s)
            for (int c = 0; c < Cin; ++c) {
                const uint8_t v = wsrc[((static_cast<size_t>(co) * Cin + c) * R + r) * S + s];
                if (pm1) {
                    w[0] |= static_cast<uint32_t>(static_cast<int8_t>(v) > 0) << (c * S + s);
                } else {
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                        if (t < bits) w[t] |= ((static_cast<uint32_t>(v) >> t) & 1u) << (c * S + s);
                }
            }
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (t < bits) dst[(static_cast<size_t>(co) * bits + t) * ldw + r] = w[t];
}

// f(integral_constant<int, bits>, integral_constant<bool, -1/+1>)
template <class F> static void with_bits(int bits, bool pm1, F &&f)
{
    using std::integral_constant;
    if (pm1) return f(integral_constant<int, 1>{}, std::true_type{});
    switch (bits) {
        case 1: return f(integral_constant<int, 1>{}, std::false_type{});
        case 2: return f(integral_constant<int, 2>{}, std::false_type{});
        case 3: return f(integral_constant<int, 3>{}, std::false_type{});
        case 4: return f(integral_constant<int, 4>{}, std::false_type{});
        case 5: return f(integral_constant<int, 5>{}, std::false_type{});
        case 6: return f(integral_constant<int, 6>{}, std::false_type{});
        case 7: return f(integral_constant<int, 7>{}, std::false_type{});
        default: return f(integral_constant<int, 8>{}, std::false_type{});
    }
}

static int launch_pack(const char *who, const void *src, uint32_t *dst, const PackGeom &g, void *stream)
{
    const int64_t total = g.rows * g.ldw;
    if (total == 0) return APNN_OK;
    if (total > (int64_t(1) << 38)) return fail(APNN_ERR_INVALID_ARG, "%s: tensor too large", who);
    // plain rows of K contiguous bytes, destination planes of a row adjacent
    const bool rows_form = g.k_stride == 1 && g.row_stride == g.K && g.outer_div == g.rows && g.inner_n == 1 &&
                           total < (int64_t(1) << 32) - 256 && g.K <= INT32_MAX - 32;
    if (rows_form)
        with_bits(g.bits, g.pm1, [&](auto bc, auto pc) {
            hipLaunchKernelGGL((pack_rows_kernel<decltype(bc)::value, decltype(pc)::value>), dim3(static_cast<unsigned>(ceil_div(total, 256))), dim3(256), 0, as_stream(stream),
                               static_cast<const uint8_t *>(src), dst, static_cast<uint32_t>(total), static_cast<int>(g.K), g.ldw);
        });
    else
        in_slices(total, [&](int64_t first, unsigned blocks) {
            hipLaunchKernelGGL(pack_generic_kernel, dim3(blocks), dim3(256), 0, as_stream(stream),
                               static_cast<const uint8_t *>(src), dst, g, first);
        });
    return check_launch(who);
}

}  // namespace apnn

using namespace apnn;

extern "C" int apnn_pack(const void *src_dev, int64_t rows, int64_t K, int bits, apnn_encoding enc,
                         uint32_t *dst_dev, void *stream)
{
    clear_error();
    if (int rc = check_bits_enc("apnn_pack", "operand", bits, enc)) return rc;
    if (rows < 0 || K < 0) return fail(APNN_ERR_INVALID_ARG, "apnn_pack: negative size");
    if (rows == 0 || K == 0) return APNN_OK;
    if (!src_dev || !dst_dev) return fail(APNN_ERR_INVALID_ARG, "apnn_pack: null pointer");
    if (!aligned16(dst_dev)) return fail(APNN_ERR_ALIGNMENT, "apnn_pack: dst_dev not 16-byte aligned");
    PackGeom g{rows, K, K, 1, rows, 0, 1, static_cast<int>(apnn_row_words(K)), bits, enc == APNN_ENC_PM1};
    if (apnn_row_words(K) > INT32_MAX) return fail(APNN_ERR_INVALID_ARG, "apnn_pack: K too large");
    return launch_pack("apnn_pack", src_dev, dst_dev, g, stream);
}

extern "C" int apnn_pack_fmap(const void *src_dev, apnn_layout layout, int64_t N, int64_t H, int64_t W,
                              int64_t C, int bits, apnn_encoding enc, uint32_t *dst_dev, void *stream)
{
    clear_error();
    if (int rc = check_bits_enc("apnn_pack_fmap", "feature", bits, enc)) return rc;
    if (N < 0 || H < 0 || W < 0 || C < 0) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_fmap: negative size");
    if (layout != APNN_LAYOUT_NHWC && layout != APNN_LAYOUT_NCHW)
        return fail(APNN_ERR_INVALID_ARG, "apnn_pack_fmap: unknown layout %d", static_cast<int>(layout));
    if (N * H * W * C == 0) return APNN_OK;
    if (!src_dev || !dst_dev) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_fmap: null pointer");
    if (!aligned16(dst_dev)) return fail(APNN_ERR_ALIGNMENT, "apnn_pack_fmap: dst_dev not 16-byte aligned");
    const int64_t HW = H * W;
    PackGeom g;
    g.rows = N * HW; g.K = C; g.inner_n = 1; g.ldw = static_cast<int>(ceil_div(C, 32));
    g.bits = bits; g.pm1 = enc == APNN_ENC_PM1;
    if (layout == APNN_LAYOUT_NHWC) {
        g.row_stride = C; g.k_stride = 1; g.outer_div = g.rows; g.outer_stride = 0;
    } else {
        g.row_stride = 1; g.k_stride = HW; g.outer_div = HW; g.outer_stride = C * HW;
        // 64 pixels per block while 256 would leave compute units without a second one, and where 256 records of wide
        // pixels exceed the LDS
        const int px = N * ceil_div(HW, 256) < 512 || static_cast<int64_t>(bits) * g.ldw > 47 ? 64 : 256;
        const int64_t bpi = ceil_div(HW, px), lds = 4 * px * ((static_cast<int64_t>(bits) * g.ldw) | 1);
        if (HW >= 4 && N * bpi <= kMaxBlocks && lds <= 48 * 1024 && HW <= INT32_MAX - 256 && C <= INT32_MAX - 32) {
            with_bits(bits, g.pm1, [&](auto bc, auto pc) {
                constexpr int BITS = decltype(bc)::value;
                constexpr bool PM1 = decltype(pc)::value;
                hipLaunchKernelGGL((px == 64 ? pack_nchw_kernel<BITS, PM1, 64> : pack_nchw_kernel<BITS, PM1, 256>),
                                   dim3(static_cast<unsigned>(N * bpi)), dim3(256), static_cast<size_t>(lds), as_stream(stream),
                                   static_cast<const uint8_t *>(src_dev), dst_dev, static_cast<int>(C), static_cast<int>(HW), g.ldw,
                                   static_cast<int>(bpi));
            });
            return check_launch("apnn_pack_fmap");
        }
    }
    return launch_pack("apnn_pack_fmap", src_dev, dst_dev, g, stream);
}

extern "C" int apnn_pack_conv_weights(const void *src_dev, int64_t Cout, int64_t Cin, int R, int S, int bits,
                                      apnn_encoding enc, uint32_t *dst_dev, void *stream)
{
    clear_error();
    if (int rc = check_bits_enc("apnn_pack_conv_weights", "weight", bits, enc)) return rc;
    if (Cout < 0 || Cin < 0 || R < 1 || S < 1) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_conv_weights: bad size");
    if (Cout * Cin == 0) return APNN_OK;
    if (!src_dev || !dst_dev) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_conv_weights: null pointer");
    if (!aligned16(dst_dev)) return fail(APNN_ERR_ALIGNMENT, "apnn_pack_conv_weights: dst_dev not 16-byte aligned");
    const int64_t RS = static_cast<int64_t>(R) * S;
    PackGeom g;
    g.rows = Cout * RS; g.K = Cin;           // a "row" is one (cout, r, s) tap, its values are the channels
    g.row_stride = 1; g.k_stride = RS;       // source Cout x Cin x R x S: tap index is contiguous, channels stride RS
    g.outer_div = RS; g.outer_stride = Cin * RS;
    g.inner_n = RS; g.ldw = static_cast<int>(ceil_div(Cin, 32));
    g.bits = bits; g.pm1 = enc == APNN_ENC_PM1;
    return launch_pack("apnn_pack_conv_weights", src_dev, dst_dev, g, stream);
}

extern "C" int apnn_pack_patches(const uint8_t *src_dev, int64_t N, int64_t C, int64_t H, int64_t W, int R, int S,
                                 int stride, int pad, int bits, uint32_t *dst_dev, void *stream)
{
    clear_error();
    if (int rc = check_bits_enc("apnn_pack_patches", "image", bits, APNN_ENC_UNSIGNED)) return rc;
    if (N < 0 || C < 1 || H < 1 || W < 1 || R < 1 || S < 1 || stride < 1 || pad < 0)
        return fail(APNN_ERR_INVALID_ARG, "apnn_pack_patches: bad geometry");
    if (static_cast<int64_t>(S) * C > 32)
        return fail(APNN_ERR_UNSUPPORTED, "apnn_pack_patches: S*C = %lld bits do not fit one word", (long long)(S * C));
    if (H + 2 * pad < R || W + 2 * pad < S) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_patches: kernel larger than padded frame");
    if (N == 0) return APNN_OK;
    if (!src_dev || !dst_dev) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_patches: null pointer");
    if (!aligned16(dst_dev)) return fail(APNN_ERR_ALIGNMENT, "apnn_pack_patches: dst_dev not 16-byte aligned");
    const int Ho = static_cast<int>((H + 2 * pad - R) / stride + 1), Wo = static_cast<int>((W + 2 * pad - S) / stride + 1);
    if (R > 8) return fail(APNN_ERR_UNSUPPORTED, "apnn_pack_patches: kernel height %d above 8", R);
    const int ldw = static_cast<int>(apnn_row_words(32 * static_cast<int64_t>(R)));
    const int64_t npix = N * Ho * Wo;
    // row kernel: needs pad <= 32 (non-negative string positions) and the plane strings of R x C rows in LDS
    const int rw = static_cast<int>((W + 31) / 32) + 4;
    const size_t lds = static_cast<size_t>(R) * C * bits * rw * sizeof(uint32_t);
    if (pad <= 32 && lds <= 48 * 1024 && N * Ho <= kMaxBlocks && (N * C * H * W) < (int64_t(1) << 40)) {
        hipLaunchKernelGGL(pack_patches_rows_kernel, dim3(static_cast<unsigned>(N * Ho)), dim3(256), lds, as_stream(stream),
                           src_dev, dst_dev, static_cast<int>(C), static_cast<int>(H), static_cast<int>(W), Ho, Wo, R, S,
                           stride, pad, bits, ldw, rw);
        return check_launch("apnn_pack_patches");
    }
    if (ceil_div(npix, 32) > kMaxBlocks) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_patches: too many pixels for one launch");
    const unsigned grid = static_cast<unsigned>(ceil_div(npix, 32));
    hipLaunchKernelGGL(pack_patches_kernel, dim3(grid), dim3(256), 0, as_stream(stream), src_dev, dst_dev, npix,
                       static_cast<int>(C), static_cast<int>(H), static_cast<int>(W), Ho, Wo, R, S, stride, pad, bits, ldw);
    return check_launch("apnn_pack_patches");
}

extern "C" int apnn_pack_patch_weights(const void *src_dev, int64_t Cout, int64_t Cin, int R, int S, int bits,
                                       apnn_encoding enc, uint32_t *dst_dev, void *stream)
{
    clear_error();
    if (int rc = check_bits_enc("apnn_pack_patch_weights", "weight", bits, enc)) return rc;
    if (Cout < 0 || Cin < 1 || R < 1 || S < 1) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_patch_weights: bad size");
    if (static_cast<int64_t>(S) * Cin > 32)
        return fail(APNN_ERR_UNSUPPORTED, "apnn_pack_patch_weights: S*Cin = %lld bits do not fit one word", (long long)(S * Cin));
    if (Cout == 0) return APNN_OK;
    if (!src_dev || !dst_dev) return fail(APNN_ERR_INVALID_ARG, "apnn_pack_patch_weights: null pointer");
    if (!aligned16(dst_dev)) return fail(APNN_ERR_ALIGNMENT, "apnn_pack_patch_weights: dst_dev not 16-byte aligned");
    const int ldw = static_cast<int>(apnn_row_words(32 * static_cast<int64_t>(R)));
    const unsigned grid = static_cast<unsigned>(ceil_div(Cout * ldw, 256));
    hipLaunchKernelGGL(pack_patch_weights_kernel, dim3(grid), dim3(256), 0, as_stream(stream),
                       static_cast<const uint8_t *>(src_dev), dst_dev, static_cast<int>(Cout), static_cast<int>(Cin), R, S,
                       bits, enc == APNN_ENC_PM1 ? 1 : 0, ldw);
    return check_launch("apnn_pack_patch_weights");
}

extern "C" int apnn_quantize(const float *src_dev, int64_t rows, int64_t K, float zero, float step, int bits,
                             uint32_t *dst_dev, void *stream)
{
    clear_error();
    if (int rc = check_bits_enc("apnn_quantize", "output", bits, APNN_ENC_UNSIGNED)) return rc;
    if (rows < 0 || K < 0) return fail(APNN_ERR_INVALID_ARG, "apnn_quantize: negative size");
    if (!(step > 0.0f)) return fail(APNN_ERR_INVALID_ARG, "apnn_quantize: step must be > 0");
    if (rows == 0 || K == 0) return APNN_OK;
    if (!src_dev || !dst_dev) return fail(APNN_ERR_INVALID_ARG, "apnn_quantize: null pointer");
    if (!aligned16(dst_dev)) return fail(APNN_ERR_ALIGNMENT, "apnn_quantize: dst_dev not 16-byte aligned");
    const int ldw = static_cast<int>(apnn_row_words(K));
    // 2048 values per wave (or 16 rows of at most 128) where the rows are that long, no more than a third of their last segments
    // would be padding, and 2048 waves get that many values to fill the chip with; else 512 (4 rows), else 256 (2 rows).
    // To 2 bits: 20000 x 2049 30.1 us by 2048, 27.7 by 512; 700 x 4100 5.0 and 3.5.
    const bool short_rows = K <= 128;
    auto fills = [&](int64_t n) {
        if (short_rows) return rows >= 2048 * 2 * n;
        return K >= 256 * n && 2 * round_up(K, 256 * n) <= 3 * K && rows >= ceil_div(2048 * 256 * n, K);
    };
    const int nl = fills(8) ? 8 : fills(2) ? 2 : 1;
    const int64_t segs = short_rows ? 1 : ceil_div(K, 256 * nl), waves = short_rows ? ceil_div(rows, 2 * nl) : rows * segs;
    const float inv = 1.0f / step;
    if (ceil_div(waves, 4) <= kMaxBlocks && rows < (int64_t(1) << 32) - 16 && K <= INT32_MAX - 2048 && inv >= 0x1p-126f && inv <= 0x1p126f) {
        int e;
        const bool exact = std::frexp(step, &e) == 0.5f;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(ceil_div(waves, 4))), dim3(256), 0, as_stream(stream), src_dev,
                               dst_dev, static_cast<uint32_t>(waves), static_cast<int>(segs), static_cast<uint32_t>(rows),
                               static_cast<int>(K), ldw, bits, zero, step, inv);
        };
        auto by_form = [&](auto n) {
            constexpr int NL = decltype(n)::value;
            if (short_rows) exact ? go(quantize_pack_wave_kernel<NL, true, true>) : go(quantize_pack_wave_kernel<NL, false, true>);
            else exact ? go(quantize_pack_wave_kernel<NL, true, false>) : go(quantize_pack_wave_kernel<NL, false, false>);
        };
        if (nl == 8) by_form(std::integral_constant<int, 8>{});
        else if (nl == 2) by_form(std::integral_constant<int, 2>{});
        else by_form(std::integral_constant<int, 1>{});
    } else {
        in_slices(rows * ldw, [&](int64_t item, unsigned blocks) {
            hipLaunchKernelGGL(quantize_pack_kernel, dim3(blocks), dim3(256), 0, as_stream(stream), src_dev, dst_dev, rows, K,
                               ldw, bits, zero, step, item);
        });
    }
    return check_launch("apnn_quantize");
}
