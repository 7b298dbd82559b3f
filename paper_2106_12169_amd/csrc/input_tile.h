// Input layer with one or two planes out and at most 64 channels: the form the networks' first layers take.
//
// A block of eight waves owns 512 output pixels (64 a wave) and all channels, and stages the image rows their windows touch in
// LDS, as signed bytes x - 128 with the padding filled in.  A K segment is eight consecutive bytes of a row, at any byte
// offset: the rows are kept in COPIES copies, each shifted by STEP = 4 / COPIES bytes against the one before, so that every
// segment is two aligned words of one of them (window starts are multiples of STEP: the stride).  The main loop then has an
// address addition and a load per segment, where input_conv_kernel loads, checks and shifts each for itself.
//
// The weights are the row operand of the matrix instruction and the planes are made in the lane (plane_codes.h); the constant
// that undoes the shift of the image bytes starts the sums.  Block by block the rows are in flight before anything needs
// them only if another block of the compute unit computes meanwhile: two or three fit.
//
// Measured (64 channels, 7 x 7, stride 2, 224 x 224, batch 128 and 8): 41.7 and 6.1 us, with input_conv_kernel 80.0 and 10.4;
// 3 x 3, stride 1: 118 and 12.3, 259 and 20.9; 11 x 11, stride 4: 20.6 and 8.1, 54.4 and 9.8.  Bound by vector instructions
// (7 x 7, batch 128, by counters: issued in 77 % of a SIMD's cycles; 640 a wave, half of them staging, 130 a channel tile for
// the planes).  Small frames and batches are left to input_conv_kernel (the rule is where it is launched).
#pragma once
#include "mfma_kernel.h"
#include "plane_codes.h"

namespace apnn {

typedef int v16i_t __attribute__((ext_vector_type(16)));

struct InputTileParams {
    const uint8_t *img;      // N x C x H x W bytes
    const int8_t *w;         // Cout x Kp signed bytes
    const int32_t *cterm;    // Cout: 128 * sum of the row's weights
    int M, N, C, images, H, W, Hq;           // Hq: lines of the padded frame
    Divisor per_image, per_row;              // output pixels of an image, of a row
    Divisor frame_lines, row_groups;         // Hq, eight-byte groups of a staged row
    int stride, pad, R, Kp, KS, segments;    // bytes of a weight row, its steps of 32 bytes, its segments
    int plane;               // LDS bytes of one copy of one channel's rows
    int pitch;               // bytes of a staged row
    Divisor kernel_rows;     // R
    uint32_t xmask;          // (2^q - 1) in every byte
    const float *scale, *bias;
    uint32_t *out;
    int q_out, NW;
};

// NT: tiles of 32 channels; SEG: eight-byte segments of a kernel row
template <int NT, int SEG, int COPIES> __global__ __launch_bounds__(512, 2) void input_tile_kernel(const InputTileParams p)
{
    constexpr int FP = 2, BP = 8 * 32 * FP, STEP = 4 / COPIES;
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    float *const sP = reinterpret_cast<float *>(lds);                    // [tile][half][register]: scales / 4, biases / 4
    int *const sC = reinterpret_cast<int *>(lds + 64 * NT);              // ... and the constants
    int *const sO = sC + 32 * NT;                                        // byte offset of each segment
    uint32_t *const sW = reinterpret_cast<uint32_t *>(sO + 4 * p.KS);    // weights: [step][tile][lane][16 bytes]
    uint8_t *const sI = reinterpret_cast<uint8_t *>(sW + p.KS * NT * 256);       // image: [channel][copy][row][pitch]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, lh = lane >> 5;
    const int m0 = blockIdx.x * BP, last = min(m0 + BP, p.M) - 1;

    // line of the padded frames and first byte of an output pixel's window
    auto window = [&](int gm, int &x) {
        const int n = divide(gm, p.per_image), rem = gm - n * p.per_image.d;
        const int oy = divide(rem, p.per_row);
        x = (rem - oy * p.per_row.d) * p.stride;
        return n * p.Hq + oy * p.stride;
    };
    int unused;
    const int line0 = __builtin_amdgcn_readfirstlane(window(m0, unused));
    const int lines = __builtin_amdgcn_readfirstlane(window(last, unused)) + p.R - line0;

    // ---- the first weights are in flight while the image rows are fetched
    constexpr int WPRE = 2;
    auto weight = [&](int q) {                                           // (step, tile, lane) -> 16 bytes of its channel
        const int l = q & 63, t = (q >> 6) % NT, s = (q >> 6) / NT, ch = 32 * t + code_channel_of_row(l & 31);
        v4i_t v = {0, 0, 0, 0};
        if (ch < p.N) v = *reinterpret_cast<const v4i_t *>(p.w + ch * p.Kp + 32 * s + 16 * (l >> 5));
        return v;
    };
    const int weights = p.KS * NT * 64;
    v4i_t w0[WPRE];
#pragma unroll
    for (int u = 0; u < WPRE; ++u) w0[u] = weight(min(tid + 512 * u, weights - 1));

    // ---- image rows: a thread stages eight positions of a line, in every copy and channel; U of them in flight
    constexpr int U = 4 / COPIES;
    const int items = lines * p.row_groups.d;
    for (int q0 = tid; q0 < items; q0 += 512 * U) {
        // eight bytes from a start clamped into the row, shifted into place: zeros come in from outside the frame
        const uint8_t *row[U];
        int xs[U][COPIES], shift[U][COPIES], at[U];                      // shift: bits to the left, negative to the right
        bool ok[U][COPIES];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + 512 * u, line = divide(q, p.row_groups), g = q - line * p.row_groups.d;
            const int n = divide(line0 + line, p.frame_lines), y = line0 + line - n * p.frame_lines.d - p.pad;
            const bool row_ok = q < items && n < p.images && static_cast<unsigned>(y) < static_cast<unsigned>(p.H);
            row[u] = p.img + (row_ok ? (static_cast<int64_t>(n) * p.C * p.H + y) * p.W : 0);
            at[u] = line * p.pitch + 8 * g;
#pragma unroll
            for (int j = 0; j < COPIES; ++j) {
                const int x = 8 * g + STEP * j - p.pad;
                xs[u][j] = min(max(x, 0), p.W - 8);
                const int delta = xs[u][j] - x;
                ok[u][j] = row_ok && delta > -8 && delta < 8;
                shift[u][j] = 8 * min(max(delta, -7), 7);                // (groups wholly outside are zero as they are)
            }
        }
        for (int c0 = 0; c0 < p.C; c0 += 3) {                            // three channels in flight
            uint64_t v[U][3][COPIES];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < 3; ++c)
#pragma unroll
                    for (int j = 0; j < COPIES; ++j) {
                        v[u][c][j] = 0;
                        if (ok[u][j] && c0 + c < p.C) __builtin_memcpy(&v[u][c][j], row[u] + static_cast<int64_t>(c0 + c) * p.H * p.W + xs[u][j], 8);
                    }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (q0 + 512 * u >= items) continue;
#pragma unroll
                for (int j = 0; j < COPIES; ++j) {
                    const int shl = max(shift[u][j], 0), shr = max(-shift[u][j], 0);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        constexpr int AND_XOR = (0xF0 & 0xCC) ^ 0xAA;    // (x & mask) ^ 0x80 per byte
                        const uint64_t t = (v[u][c][j] << shl) >> shr;
                        const uint2 s = make_uint2(__builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(t), p.xmask, 0x80808080u, AND_XOR),
                                                   __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(t >> 32), p.xmask, 0x80808080u, AND_XOR));
                        if (c0 + c < p.C) *reinterpret_cast<uint2 *>(sI + at[u] + ((c0 + c) * COPIES + j) * p.plane) = s;
                    }
                }
            }
        }
    }
    // ---- weights, constants, segment offsets
#pragma unroll
    for (int u = 0; u < WPRE; ++u)
        if (tid + 512 * u < weights) *reinterpret_cast<v4i_t *>(sW + 4 * (tid + 512 * u)) = w0[u];
    for (int q = tid + 512 * WPRE; q < weights; q += 512) *reinterpret_cast<v4i_t *>(sW + 4 * q) = weight(q);
    if (tid < 32 * NT) {
        const int ch = (tid & ~31) + code_channel(tid & 15, (tid >> 4) & 1);
        const bool ok = ch < p.N;
        sP[tid] = ok ? 0.25f * p.scale[ch] : 0.0f;       // (what a denormal loses is beyond what the sum keeps)
        sP[32 * NT + tid] = ok ? quarter(p.bias[ch]) : 0.0f;
        sC[tid] = ok ? p.cterm[ch] : 0;
    } else if (const int s = tid - 32 * NT; s < 4 * p.KS) {
        const int krow = s / SEG, c = divide(krow, p.kernel_rows), r = krow - c * p.R;
        sO[s] = s < p.segments ? c * COPIES * p.plane + r * p.pitch + 8 * (s % SEG) : 0;
    }
    __syncthreads();

    // ---- this lane's pixels
    int gm[FP], base[FP];
#pragma unroll
    for (int f = 0; f < FP; ++f) {
        gm[f] = m0 + (wave * FP + f) * 32 + lr;
        int x;
        const int line = window(min(gm[f], last), x) - line0;
        base[f] = line * p.pitch + (x & ~3) + ((x & 3) / STEP) * p.plane;
    }
    v16i_t start[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const v4i_t c = *reinterpret_cast<const v4i_t *>(sC + 32 * t + 16 * lh + 4 * k);
            start[t][4 * k] = c[0]; start[t][4 * k + 1] = c[1]; start[t][4 * k + 2] = c[2]; start[t][4 * k + 3] = c[3];
        }
    v16i_t acc[NT][FP];
    auto step = [&](auto first, int s) {
        const int2 o = *reinterpret_cast<const int2 *>(sO + 4 * s + 2 * lh);
        v4i_t a[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) a[t] = *reinterpret_cast<const v4i_t *>(sW + ((s * NT + t) * 64 + lane) * 4);
#pragma unroll
        for (int f = 0; f < FP; ++f) {
            const uint32_t *s0 = reinterpret_cast<const uint32_t *>(sI + (base[f] + o.x));
            const uint32_t *s1 = reinterpret_cast<const uint32_t *>(sI + (base[f] + o.y));
            const v4i_t b = {static_cast<int>(s0[0]), static_cast<int>(s0[1]), static_cast<int>(s1[0]), static_cast<int>(s1[1])};
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t][f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[t], b, decltype(first)::value ? start[t] : acc[t][f], 0, 0, 0);
        }
    };
    step(std::true_type{}, 0);
    for (int s = 1; s < p.KS; ++s) step(std::false_type{}, s);

    // ---- planes
    static_for<NT>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        uint32_t d[FP][2];
        static_for<2>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const v4f_t *const at = reinterpret_cast<const v4f_t *>(sP + 32 * t + 16 * lh + 8 * q);
            const v4f_t sc[2] = {at[0], at[1]}, bi[2] = {at[8 * NT], at[8 * NT + 1]};
            static_for<FP>([&](auto fc) {
                constexpr int f = decltype(fc)::value;
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = static_cast<float>(acc[t][f][8 * q + j]);
                d[f][q] = nibbles<false>(v, sc, bi, false, 0.0f, 0u);
            });
        });
#pragma unroll
        for (int f = 0; f < FP; ++f) {
            const uint32_t word = plane_words(d[f][0], d[f][1], p.q_out);
            if (gm[f] < p.M && lh < p.q_out && t < p.NW)
                p.out[static_cast<int64_t>(gm[f]) * (p.q_out * p.NW) + (lh * p.NW + t)] = word;
        }
    });
}

}  // namespace apnn
