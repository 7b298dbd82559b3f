// Single-pass form of the arbitrary-precision product for operands of more than
// two bits, on the 8-bit integer matrix instruction (v_mfma_i32_32x32x32_i8).
//
// The bit planes of the ABI stay packed in HBM.  The plane words of 32 K positions
// are transposed into 32 bytes, each holding all the bits of one element (Eq. 2
// read backwards: the decoded integer), once per block on their way to LDS, and one
// matrix instruction multiplies 32 x 32 x 32 of them with int32 accumulation.  Where the 1-bit emulation takes p q plane-pair passes and the
// two-plane FP4 form ceil(p/2) ceil(q/2) digit passes, this takes one; the paper
// observes the same about built-in 8-bit arithmetic once operands grow (Sec. 6.1.1).
// Results are the same integers (no range condition: the accumulator is int32, as
// Sec. 4.1 requires of the output).
//
// Encodings (Sec. 3.2).  The instruction multiplies signed bytes.
//   unsigned, up to 7 planes   the byte is the value.
//   unsigned, 8 planes         the top plane is inverted, which makes the byte
//                              value - 128; the product is put right with the row
//                              sums of the other operand (the J-term of Case III,
//                              with 128 in place of 1).
//   -1/+1                      the stored bit b enters as the byte b, and
//                              (2b - 1) x = 2 b x - x is recovered exactly as in
//                              Case III: twice the sum less the other operand's
//                              row sum.
// In general, with a = alphaA a' + oA and b = alphaB b' + oB (a', b' the bytes):
//   Y = alphaA alphaB sum(a' b') + alphaA oB sum(a') + alphaB oA sum(b') + K oA oB.
// The host folds this into Y = accmul acc + mulA RA[m] + mulB RB[n] + c0, RA and RB
// being the decoded row sums sum_s 2^s popc(plane s), which the lanes accumulate
// from the plane words they hold anyway (popcount, as in the AND+popcount kernel).
//
// Schedule.  A block of eight waves owns 128 x 128 outputs and makes the bytes of its 128 + 128 operand rows once - a thread
// per row and word - in LDS, where the waves read them as fragments: about 60 vector instructions a thread per chunk of four
// words (128 positions) and eight matrix instructions at 3 x 5 bits.  (With every wave transposing the words of its own
// fragments, a row's bytes are made by two waves and feed two matrix instructions each, 14 to 23 vector instructions per
// matrix instruction.)  Waves 0 - 3 and 4 - 7 own the same four 64 x 64 tiles and take alternate pairs of steps of a chunk;
// the results are added through LDS at the end.  One half of the waves multiplies a chunk before it makes the next one's
// bytes, the other half after, so that the two waves of a SIMD use the matrix unit and the vector unit in turn.  LDS: [word]
// [lane half][row] pieces of 16 bytes, 129 apart: reads of 32 rows and writes of 2 rows x 4 words both hit all banks.
// The K order inside a step is free as long as both operands agree: dword j, byte g of a transposed word is the element
// at bit 8 g + j.
//
// Measured (us; a form in which every wave transposed for itself, and this one): 2048^3 w3a5 24.9, 22.0; w4a4 20.4, 19.8; w5a5
// 34.5, 23.5; w8a8 40.4, 28.0; 1024^3 w3a5 13.1, 11.0; 4096^3 w3a5 132, 118, w8a8 256, 168.  At 2048^3 w3a5, by counters, a
// SIMD issues vector instructions in 33 % of its cycles and its matrix unit is busy in 20 %: the halves of a block take turns
// and meet at a barrier every chunk, and neither unit is the bound.
#pragma once
#include "mfma_big.h"

namespace apnn {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));

// plane classes: how many planes the LDS rows and the transposition are built for
enum { I8_C2 = 0, I8_C4 = 1, I8_C8 = 2 };
template <int C> struct I8Slots { static constexpr int value = C == I8_C8 ? 8 : C == I8_C4 ? 4 : 2; };

// (a & m) | (b & ~m) in one instruction (truth table a:0xF0, b:0xCC, m:0xAA)
__device__ __forceinline__ uint32_t bit_select(uint32_t a, uint32_t b, uint32_t m)
{
    constexpr int SEL = (0xF0 & 0xAA) | (0xCC & 0x55);
    return __builtin_amdgcn_bitop3_b32(a, b, m, SEL);
}

struct I8Masks { uint32_t m0f, m33, m55, m03; };

// One stage of a bit-matrix transposition on two pairs (a0, b0), (a1, b1): the D-bit blocks selected by ~m of a and
// by m of b change places.  The two left shifts and the two right shifts are each one 64-bit shift of a register
// pair (issued at the rate of a 32-bit one); the bits that cross between the halves land where m drops them.
template <int D> __device__ __forceinline__ void swap_blocks2(uint32_t &a0, uint32_t &b0, uint32_t &a1, uint32_t &b1, uint32_t m)
{
    const uint64_t up = pair_shl<D>(make_pair(b0, b1)), down = pair_shr<D>(make_pair(a0, a1));
    const uint32_t na0 = bit_select(a0, half_of<0>(up), m), na1 = bit_select(a1, half_of<1>(up), m);
    b0 = bit_select(half_of<0>(down), b0, m);
    b1 = bit_select(half_of<1>(down), b1, m);
    a0 = na0;
    a1 = na1;
}

// Plane words w[0 .. slots) of 32 K positions -> 8 dwords of 4 bytes: byte g of d[j] is the element at bit 8 g + j,
// i.e. sum_s 2^s bit(w[s], 8 g + j).  Two parts, so that matrix instructions can be issued in between; x carries
// the state from part 0 to part 1.
template <int C, int PART>
__device__ __forceinline__ void planes_to_bytes(const uint32_t (&w)[I8Slots<C>::value], const I8Masks &k, uint32_t (&x)[8], uint32_t (&d)[8])
{
    if constexpr (C == I8_C8) {
        // 8 x 8 bit-matrix transposition (plane s, bit j of a byte) inside every byte column, three stages
        if constexpr (PART == 0) {
#pragma unroll
            for (int s = 0; s < 8; ++s) x[s] = w[s];
            swap_blocks2<4>(x[0], x[4], x[1], x[5], k.m0f);
            swap_blocks2<4>(x[2], x[6], x[3], x[7], k.m0f);
            swap_blocks2<2>(x[0], x[2], x[1], x[3], k.m33);
        } else {
            swap_blocks2<2>(x[4], x[6], x[5], x[7], k.m33);
            swap_blocks2<1>(x[0], x[1], x[2], x[3], k.m55);
            swap_blocks2<1>(x[4], x[5], x[6], x[7], k.m55);
#pragma unroll
            for (int j = 0; j < 8; ++j) d[j] = x[j];
        }
    } else if constexpr (C == I8_C4) {
        // 4 x 4 transposition inside every nibble: nibble n of x[i] becomes the value at position 4 n + i; then the
        // nibbles are spread over the bytes
        if constexpr (PART == 0) {
            x[0] = w[0]; x[1] = w[1]; x[2] = w[2]; x[3] = w[3];
            swap_blocks2<2>(x[0], x[2], x[1], x[3], k.m33);
            swap_blocks2<1>(x[0], x[1], x[2], x[3], k.m55);
        } else {
            const uint64_t h01 = pair_shr<4>(make_pair(x[0], x[1])), h23 = pair_shr<4>(make_pair(x[2], x[3]));
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = x[i] & k.m0f;
            d[4] = half_of<0>(h01) & k.m0f;
            d[5] = half_of<1>(h01) & k.m0f;
            d[6] = half_of<0>(h23) & k.m0f;
            d[7] = half_of<1>(h23) & k.m0f;
        }
    } else {
        // 2 x 2 transposition inside every bit pair: pair t of x0 is the value at position 2 t, of x1 at 2 t + 1
        if constexpr (PART == 0) {
            const uint32_t a = w[0], b = w[1];
            x[0] = bit_select(a, b << 1, k.m55);
            x[1] = bit_select(a >> 1, b, k.m55);
            const uint64_t h = pair_shr<2>(make_pair(x[0], x[1]));
            d[0] = x[0] & k.m03;
            d[1] = x[1] & k.m03;
            d[2] = half_of<0>(h) & k.m03;
            d[3] = half_of<1>(h) & k.m03;
        } else {
            const uint64_t h4 = pair_shr<4>(make_pair(x[0], x[1])), h6 = pair_shr<6>(make_pair(x[0], x[1]));
            d[4] = half_of<0>(h4) & k.m03;
            d[5] = half_of<1>(h4) & k.m03;
            d[6] = half_of<0>(h6) & k.m03;
            d[7] = half_of<1>(h6) & k.m03;
        }
    }
}

constexpr int kI8Pieces = 8 * 129;                 // 16-byte pieces of a chunk of one operand: (word, half) x rows, padded
constexpr int kI8LdsBytes = 2 * 2 * kI8Pieces * 16 + 2 * 128 * 4;     // two buffers of both operands, row sums

template <int CA, int CB> __global__ __launch_bounds__(512, 2) void mfma_i8_kernel(const MfmaParams p)
{
    constexpr int SA = I8Slots<CA>::value, SB = I8Slots<CB>::value;
    extern __shared__ __attribute__((aligned(1024))) uint32_t smem[];
    uint32_t *const sums = smem + 4 * kI8Pieces * 4;               // row sums of A, of B

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int lr = lane & 31, lh = lane >> 5;
    const int tilesN = (p.N + 127) / 128;
    int tile = blockIdx.x;
    if (p.xcd_regions) {                                 // one rectangular region of tiles per XCD (see mfma_big_kernel)
        const int tilesM = (p.M + 127) / 128;
        const int rw = tilesN >> 2, rh = tilesM >> 1, xcd = tile & 7, idx = tile >> 3;
        tile = ((xcd >> 2) * rh + idx / rw) * tilesN + (xcd & 3) * rw + idx % rw;
    }
    const int m0 = (tile / tilesN) * 128, n0 = (tile % tilesN) * 128;

    I8Masks km;
    km.m0f = reg_const(0x0F0F0F0Fu); km.m33 = reg_const(0x33333333u);
    km.m55 = reg_const(0x55555555u); km.m03 = reg_const(0x03030303u);

    // ---- a thread's row, and its words: 16 bytes of every plane row feed four chunks (word 4 w + c of sixteen goes to chunk c
    // as its word w: the order of K is free), so that their loads are in flight for three or four chunks
    const int row = tid >> 2, word = tid & 3;
    constexpr uint32_t OUT_OF_RANGE = 0x80000000u;       // operands are smaller than 2 GiB (host check)
    const uint32_t bytesA = 4u * p.M * p.PA * p.ldwA, bytesB = 4u * p.N * p.PB * p.ldwB;
    const uint32_t atA = m0 + row < p.M ? 4u * (static_cast<uint32_t>(m0 + row) * p.PA * p.ldwA + 4 * word) : OUT_OF_RANGE;
    const uint32_t atB = n0 + row < p.N ? 4u * (static_cast<uint32_t>(n0 + row) * p.PB * p.ldwB + 4 * word) : OUT_OF_RANGE;
    struct Words { v4i_t a[SA], b[SB]; };
    const __amdgpu_buffer_rsrc_t bufA = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.A), 0, bytesA, 0x00020000);
    const __amdgpu_buffer_rsrc_t bufB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.B), 0, bytesB, 0x00020000);
    // Rows and words beyond the operand read zeros; planes that do not exist are never written and stay zero.  Everything but
    // the two lane offsets is scalar, and only planes that the class may lack are tested (with a test, an address and zeroed
    // registers per plane the loads took a quarter of the kernel: 70 us at K = 8192 with every one a hit of the first-level
    // cache, 53 without them).
    constexpr int FEWEST_A = SA == 8 ? 5 : SA == 4 ? 3 : 1, FEWEST_B = SB == 8 ? 5 : SB == 4 ? 3 : 1;
    auto fetch = [&](int four, Words &w) __attribute__((always_inline)) {
        const uint32_t dead = 16 * four + 4 * word < p.Kw ? 0u : OUT_OF_RANGE, la = atA | dead, lb = atB | dead;
#pragma unroll
        for (int s = 0; s < SA; ++s)
            if (s < FEWEST_A || s < p.PA)
                w.a[s] = __builtin_bit_cast(v4i_t, __builtin_amdgcn_raw_buffer_load_b128(bufA, la, 4u * (s * p.ldwA + 16 * four), 0));
#pragma unroll
        for (int s = 0; s < SB; ++s)
            if (s < FEWEST_B || s < p.PB)
                w.b[s] = __builtin_bit_cast(v4i_t, __builtin_amdgcn_raw_buffer_load_b128(bufB, lb, 4u * (s * p.ldwB + 16 * four), 0));
    };
    const bool need_ra = p.mulA != 0, need_rb = p.mulB != 0;
    uint32_t ra = 0, rb = 0;                             // row sums of this thread's words
    uint32_t *const mine = smem + ((2 * word) * 129 + row) * 4;
    auto stage = [&](int buffer, const Words &w, auto cc) __attribute__((always_inline)) {       // bytes of word c of every piece
        constexpr int c = decltype(cc)::value;
        uint32_t wa[SA], wb[SB];
#pragma unroll
        for (int s = 0; s < SA; ++s) wa[s] = static_cast<uint32_t>(w.a[s][c]);
#pragma unroll
        for (int s = 0; s < SB; ++s) wb[s] = static_cast<uint32_t>(w.b[s][c]);
        if (need_ra) {
#pragma unroll
            for (int s = 0; s < SA; ++s) ra += static_cast<uint32_t>(__popc(wa[s])) << s;
        }
        if (need_rb) {
#pragma unroll
            for (int s = 0; s < SB; ++s) rb += static_cast<uint32_t>(__popc(wb[s])) << s;
        }
        if (CA == I8_C8) wa[SA - 1] ^= p.flipA;          // an 8-bit operand enters as value - 128
        if (CB == I8_C8) wb[SB - 1] ^= p.flipB;
        uint32_t x[8], d[8];
        uint32_t *to = mine + buffer * (2 * kI8Pieces * 4);
        planes_to_bytes<CA, 0>(wa, km, x, d);
        planes_to_bytes<CA, 1>(wa, km, x, d);
        *reinterpret_cast<uint4 *>(to) = make_uint4(d[0], d[1], d[2], d[3]);
        *reinterpret_cast<uint4 *>(to + 129 * 4) = make_uint4(d[4], d[5], d[6], d[7]);
        to += kI8Pieces * 4;
        planes_to_bytes<CB, 0>(wb, km, x, d);
        planes_to_bytes<CB, 1>(wb, km, x, d);
        *reinterpret_cast<uint4 *>(to) = make_uint4(d[0], d[1], d[2], d[3]);
        *reinterpret_cast<uint4 *>(to + 129 * 4) = make_uint4(d[4], d[5], d[6], d[7]);
    };

    v16i_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v16i_t{};
    auto multiply = [&](int buffer) __attribute__((always_inline)) {
        const uint32_t *from = smem + buffer * (2 * kI8Pieces * 4);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t *at = from + (2 * (2 * ks + t) + lh) * (129 * 4) + lr * 4;
            v4i_t a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = *reinterpret_cast<const v4i_t *>(at + (64 * wm + 32 * i) * 4);
                b[i] = *reinterpret_cast<const v4i_t *>(at + kI8Pieces * 4 + (64 * wn + 32 * i) * 4);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };

    auto four_chunks = [&](const Words &now, const Words &next) __attribute__((always_inline)) {
        static_for<4>([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            // buffer c + 1 was read last before the barrier that ended chunk c - 1
            if (ks == 0) multiply(c & 1);
            if constexpr (c < 3) stage((c + 1) & 1, now, std::integral_constant<int, c + 1>{});
            else stage(0, next, std::integral_constant<int, 0>{});
            if (ks) multiply(c & 1);
            __syncthreads();
        });
    };
    Words even{}, odd{};
    fetch(0, even);
    stage(0, even, std::integral_constant<int, 0>{});
    __syncthreads();
    for (int four = 0; four < p.nk / 4; four += 2) {     // (beyond the last words: zeros)
        fetch(four + 1, odd);
        four_chunks(even, odd);
        if (four + 1 == p.nk / 4) break;
        fetch(four + 2, even);
        four_chunks(odd, even);
    }

    // ---- row sums of the four words of a row; the wave halves' results: each keeps one row of tiles
    ra += static_cast<uint32_t>(__shfl_xor(static_cast<int>(ra), 1));
    ra += static_cast<uint32_t>(__shfl_xor(static_cast<int>(ra), 2));
    rb += static_cast<uint32_t>(__shfl_xor(static_cast<int>(rb), 1));
    rb += static_cast<uint32_t>(__shfl_xor(static_cast<int>(rb), 2));
    if (word == 0) {
        sums[row] = ra;
        sums[128 + row] = rb;
    }
    v4i_t *const give = reinterpret_cast<v4i_t *>(smem) + wave * 512 + lane;     // (32 registers a wave: 64 KiB, the bytes are dead)
    const v4i_t *const take = reinterpret_cast<const v4i_t *>(smem) + (wave ^ 4) * 512 + lane;
    v16i_t out[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v4i_t t;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                t[r] = ks ? acc[0][j][4 * q + r] : acc[1][j][4 * q + r];
                out[j][4 * q + r] = ks ? acc[1][j][4 * q + r] : acc[0][j][4 * q + r];
            }
            give[(4 * j + q) * 64] = t;
        }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i_t t = take[(4 * j + q) * 64];
#pragma unroll
            for (int r = 0; r < 4; ++r) out[j][4 * q + r] += t[r];
        }

    // ---- encoding recovery (Sec. 3.2), in wrapping 32-bit arithmetic: Y = accmul acc + mulA RA[row] + mulB RB[column] + c0
    const int mrow0 = m0 + 64 * wm + 32 * ks;
    uint32_t col[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
        col[j] = (need_rb ? sums[128 + 64 * wn + 32 * j + lr] * static_cast<uint32_t>(p.mulB) : 0u) + static_cast<uint32_t>(p.c0);
    // accumulator register r of lane (lh, lr) is row 8 (r / 4) + 4 lh + r % 4, column lr
    static_for<16>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        const uint32_t rowterm = need_ra ? sums[64 * wm + 32 * ks + 8 * (r >> 2) + 4 * lh + (r & 3)] * static_cast<uint32_t>(p.mulA) : 0u;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            out[j][r] = static_cast<int>(static_cast<uint32_t>(out[j][r]) * static_cast<uint32_t>(p.accmul) + rowterm + col[j]);
    });
    if (p.Y) {                                           // straight from the accumulators: two 128-byte row segments a store, rows beyond M out of range
        const __amdgpu_buffer_rsrc_t bufY = __builtin_amdgcn_make_buffer_rsrc(p.Y, 0, 4u * static_cast<uint32_t>(p.M) * p.N, 0x00020000);
        const int gn0 = n0 + 64 * wn + lr;
        const uint32_t vbase = 4u * (static_cast<uint32_t>(mrow0 + 4 * lh) * p.N + gn0);
        static_for<32>([&](auto c) {
            constexpr int j = decltype(c)::value / 16, r = decltype(c)::value % 16, line = 8 * (r >> 2) + (r & 3);
            const uint32_t at = (vbase + 128u * j) | (gn0 + 32 * j < p.N ? 0u : OUT_OF_RANGE);
            __builtin_amdgcn_raw_buffer_store_b32(out[j][r], bufY, at + 4u * line * static_cast<uint32_t>(p.N), 0, 0);
        });
    }
    if (!p.scale) return;
    MfmaParams pe = p;                                   // the shared epilogue sees finished integers
    pe.out_scale = 1.0f; pe.c0 = 0; pe.Y = nullptr;
    static_for<2>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const int gn = n0 + 64 * wn + 32 * j + lr;
        float sc = 0.0f, bi = 0.0f;
        if (gn < p.N) { sc = p.scale[gn]; bi = p.bias[gn]; }
        static_for<4>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const int row0 = mrow0 + 8 * k;
            const float v4[4] = {static_cast<float>(out[j][4 * k]), static_cast<float>(out[j][4 * k + 1]),
                                 static_cast<float>(out[j][4 * k + 2]), static_cast<float>(out[j][4 * k + 3])};
            finish_rows8(pe, v4, row0, gn, sc, bi, load_res_rows8(pe, row0, gn >> 5, lane), lane, lr, lh);
        });
    });
}

}  // namespace apnn
