// Convolution layers whose input pixels are staged once per block: the form for layers with enough output pixels to
// give every compute unit a block.
//
// A block owns 32 FC output channels x 64 FW FP output pixels.  In raster order over a frame padded by `pad` on every side, the
// pixels its taps touch are one contiguous range: the block stages that range in LDS once (the lane-private
// kernels load and check every pixel once per tap and channel tile), padding as zero codes, so that a tap is one added offset
// and needs no range check.  Features and weights become FP4 codes while they are staged, so the main loop only reads operands
// and multiplies: a wave that is alone on its SIMD hides about four other instructions behind a matrix instruction, and five to
// expand each fragment of features at every tap were most of what it issued (64 x 64 outputs a wave, the operands expanded in the
// loop: 82 cycles a matrix instruction, here 54; 38 in a loop of nothing else).  Where twice the LDS for features costs
// resident blocks, they are staged as pairs of bits (PACKED) and expanded in the loop.  Weights pass through in chunks: four lanes
// share a row, since a lane a row made every load touch 64 cache lines (1024 a chunk and compute unit).  With more than 64
// channels eight waves share the pixels of two pairs of channel tiles.
//
// The matrix instruction gets the weights as its row operand, so that a lane holds sixteen channels of one pixel, and the
// planes of their codes are made in the lane (plane_codes.h).
//
// Measured (us; lane-private loads, staged with the expansion in the loop, here): ResNet-18 shape at batch 128, 64 channels 32, 15.1,
// 14.6; 128 22, 14.2, 12.9; 256 24, 13.6, 11.4; 512 28, 15.4, 13.8; 128 -> 256 with stride 2 14.5, 12.4, 9.7.  8 x 112 x 112, 128 channels,
// pooled 19.7, 15.7, 10.8.  What is left: the board's matrix instructions take 20 to 22 ns each with such operands, which is 4.6 us of
// these layers, and 77 % of the SIMDs have work (1568 wave tiles for 1024); launch, first loads and epilogue are 5 us.
#pragma once
#include "mfma_kernel.h"
#include "plane_codes.h"

namespace apnn {

struct ConvHaloParams {
    const uint32_t *A, *B;   // features [pixel][PA][Cw], weights [Cout][PB][taps][Cw]
    uint32_t bytesA, bytesB; // below 2^31
    int M, N;                // output pixels (with pooling four rows per pooled pixel), output channels
    int images, H, W, Hq, Wq;                // frame, padded frame
    Divisor per_image, per_row;              // output pixels (pooled: pooled pixels) of an image, of a row
    Divisor frame, line;                     // Hq Wq, Wq
    int stride, pad, R, S;
    int Cw, half;            // channel words of a pixel, words per lane half (steps of a tap)
    int PA, PB, DA, DB;      // planes and base-4 digits of features / weights
    Divisor digits;          // DA
    int pm1;                 // weights -1/+1, else 0/1 planes
    int plane;               // LDS words from a channel word's codes of the staged positions to the next one's
    int pieces, share;       // pieces a position is staged in, log2 of the threads that share it
    int words_table, words_codes, words_records;     // LDS words of the step offsets, of them and the weight codes, of a buffer of feature codes
    int steps, padded;       // matrix steps of a weight digit, of it as it is walked
    int pairs, buffers;      // pairs of channel tiles of a block, buffers of feature codes
    int packed;              // features are staged as bits, not as codes
    int three;               // (host) three blocks a compute unit at most, steps are read in pairs
    Divisor halves, columns;                 // half, S
    uint32_t first[4], first_codes[4];       // the first entries' words of the table of offsets
    int pool;                // 0 none, 1 maximum, 2 sum
    int scaleA, scaleB;      // block scales (exponent bytes) of features and weights
    Divisor per_column;      // channel tiles
    int tilesM, tile_step;   // tiles of pixels, tiles from one of a block's to its next
    const float *scale, *bias;
    const uint32_t *res;
    int q_res;
    float res_scale;
    uint32_t *out;
    int q_out, NW;
    int32_t *Y;              // int32 results instead of planes
};

// Most weight steps that stay in LDS for all tiles of a block, and of a chunk of longer ones (2 KiB of codes a step)
constexpr int kHaloStay = 26, kHaloChunk = 8;

// Steps whose operands a wave reads together: one step's four and more matrix instructions cover the latency of the next
// one's reads, two instructions do not -- unless four waves share a SIMD, as those of the smaller tile of bits do where weights stay.
// THREE: several digits on 768 tiles at most, or in so much LDS that a compute unit holds three blocks at most, in pairs of steps (time
// relative to one step with room for four waves: from 19 entries on 0.93 on 256 tiles at most, 0.97 on 768, with one or two blocks a unit 0.96;
// with four 1.03 at up to 8 entries).
constexpr int halo_granule(int fp, int fw, bool shared) { return shared || fp * fw >= 4 ? 1 : 2; }

// LDS words of a channel word of a position: codes; pairs of bits; the bits of one plane, or of -1/+1 features and which of them are there
constexpr int halo_words(int kind, bool packed) { return !packed ? 4 : kind == OPK_U1 ? 1 : 2; }

// Where a lane whose words of plane 0 are at byte `at` of the weights finds them in another plane: its own offset and the one that
// all lanes share.  A plane that is not there (the second one of an odd last digit) reads as zero by the lane's own offset, which
// the load checks against the buffer; the shared offset is no part of that check, so it stays inside the buffer.
struct PlaneOffset {
    uint32_t lane, shared;
};
constexpr uint32_t kNowhere = 0x80000000u;                       // beyond every buffer (2^31 bytes at most): reads as zero
__host__ __device__ __forceinline__ PlaneOffset plane_offset(uint32_t at, int plane, int planes, int Kw)
{
    if (plane >= planes) return {kNowhere, 0u};
    return {at, 4u * static_cast<uint32_t>(plane) * static_cast<uint32_t>(Kw)};
}

// SW: channel words of a plane staged together (4, 2, or 1 for an odd number of channel words); FP, FW: 32-pixel and 32-channel
// tiles of a wave (FW = 1: two waves share the pixels).  MULTI: operands of more than one digit.
// POOL (FP = 4): tile f of a wave holds member f of its 32 pooling grids, so that pooling is three instructions per output.
// STAY: the weights stay in LDS while the block walks over its tiles of pixels (grid-stride), and the next tile's pixels are in
// flight during the main loop.  Otherwise a block has one tile, and the weights pass through two buffers, a chunk each, with
// one barrier per chunk.
template <int KA, int SW, int FP, int FW, int FC, bool POOL, bool MULTI, bool PACKED, bool STAY, bool THREE>
__global__ __launch_bounds__(128 * FC, FC == 4 ? 2 : FP * FW == 8 ? 2 : FP == 1 && !THREE && (STAY ? PACKED : !MULTI) ? 4 : 3) void conv_halo_kernel(const ConvHaloParams p)
{
    static_assert(!POOL || FP == 4, "a wave's four pixel tiles are the members of its pooling grids");
    constexpr int HW = SW == 8 ? 4 : SW == 4 ? 2 : 1, PW = SW == 8 ? 4 : SW;     // channel words of a weight load, of a piece of a pixel
    constexpr int G = halo_granule(FP, FW, PACKED && STAY && !THREE);      // steps of a granule
    constexpr int E = MULTI ? 2 : 1;                             // LDS words of a table entry
    constexpr int CW = halo_words(KA, PACKED);                   // LDS words of a channel word of a position
    constexpr int NT = 128 * FC;                                 // threads: four waves for every two channel tiles
    constexpr int BP = 64 * FW * FP;                             // pixels of a tile
    constexpr int FETCH = STAY ? kHaloStay : kHaloChunk;         // weight steps in flight
    constexpr int NI = (FETCH * 2 + 4 * HW - 1) / (4 * HW);      // granules of them a thread has in flight
    constexpr int U = PW == 1 ? 4 : 2;                           // staged pieces of pixels a thread has in flight
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    float *const sP = reinterpret_cast<float *>(lds);            // scales, then biases / 4: [tile][half][register]
    uint32_t *const sB = lds + 64 * FC;                          // weight codes: [buffer][step][tile][lane][4]
    uint32_t *const sT = sB + p.words_codes - p.words_table;     // offsets of the entries
    uint32_t *const sA = sB + p.words_codes;                     // feature codes: [buffer][digit][channel word][position][4]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, lh = lane >> 5;
    const int wg = FC == 4 ? wave >> 2 : 0, w4 = FC == 4 ? wave & 3 : wave;    // pair of channel tiles, wave of the four that share it
    const int wc = 2 * wg + (FW == 1 ? w4 & 1 : 0), wp = FW == 1 ? w4 >> 1 : w4;    // first channel tile, pixels of this wave
    // block -> channel tile, first tile of pixels
    const int tile0 = divide(static_cast<int>(blockIdx.x), p.per_column);
    const int n0 = (static_cast<int>(blockIdx.x) - tile0 * p.per_column.d) * 32 * FC;

    const __amdgpu_buffer_rsrc_t bufA = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.A), 0, p.bytesA, 0x00020000);
    const __amdgpu_buffer_rsrc_t bufB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.B), 0, p.bytesB, 0x00020000);

    // ---- weights.  Packed output: matrix row -> channel as plane_codes.h says; int32 output: in order, four to a store.
    // Rows beyond the last channel read that channel's (their results are not stored); steps beyond the last, and the step a
    // lane half lacks when the number of channel words is odd, read the first words (the features are zero there).
    // Four lanes share a row: (pair of granules, half).
    const int wrow = (16 * w4 + (lane >> 2)) & 31, wtile = 2 * wg + (w4 >> 1), wh = lane & 1, wk = (lane >> 1) & 1;
    const int wch = p.Y ? wrow : code_channel_of_row(wrow);
    const int Kw = p.R * p.S * p.Cw;
    const uint32_t wlane = 4u * static_cast<uint32_t>(min(n0 + 32 * wtile + wch, p.N - 1) * (p.PB * Kw));
    uint32_t wv[NI][2][HW];
    // granule u of this thread, from step s on: the words that its steps' codes are made of
    auto fetch_granule = [&](int u, int digit, int s, auto pm1) __attribute__((always_inline)) {
        const int tap = divide(s, p.halves), cw = wh * p.half + s - tap * p.half;
        const uint32_t at = wlane + 4u * static_cast<uint32_t>(cw < p.Cw ? tap * p.Cw + cw : 0);
        auto load = [&](uint32_t (&w)[HW], PlaneOffset from) __attribute__((always_inline)) {
            if constexpr (HW == 4) {
                const auto t = __builtin_amdgcn_raw_buffer_load_b128(bufB, from.lane, from.shared, 0);
                w[0] = t[0]; w[1] = t[1]; w[2] = t[2]; w[3] = t[3];
            } else if constexpr (HW == 2) {
                const auto t = __builtin_amdgcn_raw_buffer_load_b64(bufB, from.lane, from.shared, 0);
                w[0] = t[0]; w[1] = t[1];
            } else {
                w[0] = __builtin_amdgcn_raw_buffer_load_b32(bufB, from.lane, from.shared, 0);
            }
        };
        load(wv[u][0], plane_offset(at, 2 * digit, p.PB, Kw));
        if constexpr (!decltype(pm1)::value) load(wv[u][1], plane_offset(at, 2 * digit + 1, p.PB, Kw));
    };
    Fp4Masks km;
    km.m1 = reg_const(0x11111111u); km.m2 = reg_const(0x22222222u);
    km.m4 = reg_const(0x44444444u); km.m8 = reg_const(0x88888888u);
    // ... -> codes; steps from `valid` on fill up a granule: zero codes
    auto write_granule = [&](int u, uint32_t *codes, int s, int valid, auto pm1) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < HW; ++i) {
            v8i_t f;
            Fp4Masks m = km;
            if ((MULTI || G == 2) && s + i >= valid) m.m1 = m.m2 = m.m8 = 0u;
            expand_fp4<decltype(pm1)::value ? OPK_PM1 : OPK_U2>(wv[u][0][i], wv[u][1][i], m, f);
            *reinterpret_cast<int4 *>(codes + (((s + i) * FC + wtile) * 64 + 32 * wh + (wrow ^ (2 * wh))) * 4) = make_int4(f[0], f[1], f[2], f[3]);
        }
    };
    // the first `steps` of a digit: weights that stay, or their first chunk
    auto fetch_weights = [&](int steps) {
        auto all = [&](auto pm1) {
#pragma unroll
            for (int u = 0; u < NI; ++u)
                if (2 * u * HW < steps) fetch_granule(u, 0, min((2 * u + wk) * HW, p.steps - HW), pm1);
        };
        if (p.pm1) all(std::true_type{});
        else all(std::false_type{});
    };
    auto write_weights = [&](int steps) {
        auto all = [&](auto pm1) {
#pragma unroll
            for (int u = 0; u < NI; ++u) {
                if (2 * u * HW >= steps) break;                  // uniform
                if (const int s = (2 * u + wk) * HW; s < steps) write_granule(u, sB, s, p.steps, pm1);
            }
        };
        if (p.pm1) all(std::true_type{});
        else all(std::false_type{});
    };

    // ---- the pixels a tile's taps touch: positions lo .. lo + range - 1 of the padded frames
    auto position = [&](int gm) {                                // first tap of an output pixel
        const int px = POOL ? gm >> 2 : gm;
        const int n = divide(px, p.per_image), rem = px - n * p.per_image.d;
        const int oy = divide(rem, p.per_row), ox = rem - oy * p.per_row.d;
        const int y = POOL ? 2 * oy + ((gm >> 1) & 1) : oy, x = POOL ? 2 * ox + (gm & 1) : ox;
        return (n * p.Hq + y * p.stride) * p.Wq + x * p.stride;
    };
    struct Range { int lo, total; };                             // total: pieces, counting those of the share no piece exists for
    auto range_of = [&](int tile) {
        const int m0 = tile * BP;
        Range r;
        r.lo = __builtin_amdgcn_readfirstlane(position(m0));
        r.total = (__builtin_amdgcn_readfirstlane(position(min(m0 + BP, p.M) - 1)) + (p.R - 1) * p.Wq + p.S - r.lo) << p.share;
        return r;
    };
    const int tmask = (1 << p.share) - 1;
    uint32_t a0[U][PW], a1[U][PW];                               // a piece: PW words of each plane of a digit
    bool in[U];
    auto load_piece = [&](uint32_t bytes, uint32_t (&w)[PW]) {
        if constexpr (PW == 4) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(bufA, bytes, 0, 0);
            w[0] = t[0]; w[1] = t[1]; w[2] = t[2]; w[3] = t[3];
        } else if constexpr (PW == 2) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b64(bufA, bytes, 0, 0);
            w[0] = t[0]; w[1] = t[1];
        } else {
            w[0] = __builtin_amdgcn_raw_buffer_load_b32(bufA, bytes, 0, 0);
        }
    };
    auto fetch_pixels = [&](Range r, int q0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + NT * u, pos = r.lo + (q >> p.share), g = q & tmask;
            const int n = divide(pos, p.frame), rem = pos - n * p.frame.d;
            const int yq = divide(rem, p.line), y = yq - p.pad, x = rem - yq * p.Wq - p.pad;
            const int cs = MULTI ? divide(g, p.digits) : g, d = MULTI ? g - cs * p.DA : 0, cw = cs * PW;
            in[u] = q < r.total && n < p.images && static_cast<unsigned>(y) < static_cast<unsigned>(p.H) &&
                    static_cast<unsigned>(x) < static_cast<unsigned>(p.W) && cw < p.Cw;
            const int at = (((n * p.H + y) * p.W + x) * p.PA + 2 * d) * p.Cw + cw;
            load_piece(in[u] ? 4u * static_cast<uint32_t>(at) : kNowhere, a0[u]);
            if (KA == OPK_U2) load_piece(in[u] && 2 * d + 1 < p.PA ? 4u * static_cast<uint32_t>(at + p.Cw) : kNowhere, a1[u]);
        }
    };
    auto write_pixels = [&](uint32_t *features, Range r, int q0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + NT * u, g = q & tmask;
            if (q >= r.total || g >= p.pieces) continue;
            const int cs = MULTI ? divide(g, p.digits) : g, d = MULTI ? g - cs * p.DA : 0;
            uint32_t *const dst = features + (d * 2 * p.half + cs * PW) * p.plane + CW * (q >> p.share);
#pragma unroll
            for (int i = 0; i < PW; ++i) {
                const uint32_t x0 = a0[u][i], x1 = KA == OPK_U2 ? a1[u][i] : in[u] ? ~0u : 0u;
                if constexpr (PACKED && CW == 1) {
                    dst[i * p.plane] = x0;
                } else if constexpr (PACKED) {                   // two planes as pairs of bits: even positions, odd positions
                    const uint2 w = KA == OPK_U2 ? make_uint2(mask_select(0x55555555u, x0, x1 << 1), mask_select(0x55555555u, x0 >> 1, x1)) : make_uint2(x0, x1);
                    *reinterpret_cast<uint2 *>(dst + i * p.plane) = w;
                } else {
                    v8i_t f;
                    expand_fp4<KA>(x0, x1, km, f);
                    *reinterpret_cast<int4 *>(dst + i * p.plane) = make_int4(f[0], f[1], f[2], f[3]);
                }
            }
        }
    };

    // all of a tile's pieces, the first ones of which are fetched already
    auto write_tile = [&](uint32_t *features, Range r) {
        write_pixels(features, r, tid);
        for (int q = tid + NT * U; q < r.total; q += NT * U) {
            fetch_pixels(r, q);
            write_pixels(features, r, q);
        }
    };

    // Weights that pass through: the chunk after one, in the order of the sums (digit DB: none).  A chunk's codes are written
    // while the one before it is multiplied, from words that were fetched a whole chunk earlier.
    struct Chunk { int digit, s0; };
    auto after = [&](Chunk c) {
        const bool wrap = c.s0 + kHaloChunk >= p.steps;
        return Chunk{c.digit + (wrap ? 1 : 0), wrap ? 0 : c.s0 + kHaloChunk};
    };
    // (a chunk's steps beyond the digit's last read step s0; their codes are zero, or not used)
    auto fetch_chunk = [&](Chunk c, auto pm1) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NI; ++u) {
            const int s = c.s0 + (2 * u + wk) * HW;
            fetch_granule(u, min(c.digit, p.DB - 1), s < p.steps ? s : c.s0, pm1);
        }
    };
    // writes the chunk after `c` to the buffer that c is not in (read last before the barrier that began c)
    auto stage_next = [&](Chunk c, int half_buffer) __attribute__((always_inline)) {
        const Chunk next = after(c);
        if (next.digit >= p.DB) return false;
        uint32_t *const to = sB + (half_buffer ^ 1) * (kHaloChunk * FC * 256);
        auto all = [&](auto pm1) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < NI; ++u) write_granule(u, to, (2 * u + wk) * HW, p.steps - next.s0, pm1);
            fetch_chunk(after(next), pm1);
        };
        if (p.pm1) all(std::true_type{});
        else all(std::false_type{});
        return true;
    };

    Range now = range_of(tile0);
    float constant = 0.0f;                                       // scale (first half of the threads) or bias of a channel
    if (!p.Y && tid < 64 * FC) {
        const int k = tid % (32 * FC), ch = n0 + (k & ~31) + code_channel(k & 15, (k >> 4) & 1);
        if (ch < p.N) constant = (tid < 32 * FC ? p.scale : p.bias)[ch];
    }
    fetch_weights(STAY ? p.steps : min(kHaloChunk, p.steps));
    fetch_pixels(now, tid);
    // what needs no load is made while these are in flight
    int gm[FP];                                                  // this lane's pixels
    const uint8_t *base[FP];                                     // the first tap's position, this lane half's words
    auto point = [&](int tile, int buffer) {
        const int m0 = tile * BP, last = min(m0 + BP, p.M) - 1;
#pragma unroll
        for (int f = 0; f < FP; ++f) {
            gm[f] = POOL ? m0 + 4 * (32 * wp + lr) + f : m0 + (wp * FP + f) * 32 + lr;
            base[f] = reinterpret_cast<const uint8_t *>(sA + buffer * p.words_records + CW * (position(min(gm[f], last)) - now.lo) + lh * p.half * p.plane);
        }
    };
    point(tile0, 0);
    // Weights that stay: granules of a tile's sums.  One or two of them come without the table, their offsets with the launch: in sums
    // of up to four steps the table, the step that fills up and what stood between the loads and the barrier were up to a tenth of
    // the layer (40 layers of one digit, 1.054 times what they had taken with operands expanded in the loop, now 1.00 to 1.03; 18 of
    // several digits 1.033, now 1.02; 80 x 32 x 25, 32 -> 64 channels, four feature planes 6.13 us, now 5.98).
    const int entries = (MULTI ? p.steps * p.DA : p.steps), stay_granules = (entries + G - 1) / G;
    const bool few = STAY && stay_granules <= 2;
    // Where an entry's operands are, from those of the first one; an entry is a step or, with several digits, a step and a digit of the
    // features: then the codes of its weights (in the chunk) with the digit in the low bits stand beside it.  Entry e is at e + G.
    for (int i = few ? p.words_table : tid; i < p.words_table / E; i += NT) {
        const int e = max(i - G, 0), st = MULTI ? divide(e, p.digits) : e, d = MULTI ? e - st * p.DA : 0;
        const int tap = divide(st, p.halves), r = divide(tap, p.columns);
        sT[E * i] = st < p.steps ? 4u * CW * static_cast<uint32_t>(r * p.Wq + tap - r * p.S) +
                                       4u * static_cast<uint32_t>((st - tap * p.half + d * 2 * p.half) * p.plane) : 0u;
        if (MULTI) sT[E * i + 1] = 1024u * FC * static_cast<uint32_t>(STAY ? min(st, p.padded - 1) : st % kHaloChunk) + d;
    }
    write_weights(STAY ? p.padded : kHaloChunk);
    if constexpr (!STAY) {
        if (p.pm1) fetch_chunk(after(Chunk{0, 0}), std::true_type{});
        else fetch_chunk(after(Chunk{0, 0}), std::false_type{});
    }
    if (!p.Y && tid < 64 * FC) sP[tid] = tid < 32 * FC ? constant : quarter(constant);
    write_tile(sA, now);
    __syncthreads();

    const int scaleA = static_cast<int>(reg_const(static_cast<uint32_t>(p.scaleA))), scaleB0 = static_cast<int>(reg_const(static_cast<uint32_t>(p.scaleB)));
    const uint32_t m3 = reg_const(0x33333333u);

    for (int tile = tile0, buffer = 0;; buffer ^= p.buffers - 1) {
        // residual words and the next tile's first pixels: their latency hides behind the main loop
        constexpr int FO = POOL ? 1 : FP;                        // output tiles per channel tile
        uint32_t res[FO][FW][2];
#pragma unroll
        for (int f = 0; f < FO; ++f)
#pragma unroll
            for (int c = 0; c < FW; ++c) {
                res[f][c][0] = res[f][c][1] = 0u;
                const int px = POOL ? gm[0] >> 2 : gm[f], ch = n0 + 32 * (wc + c);
                if (p.res && gm[f] < p.M && ch < p.N) {
                    const uint32_t *rp = p.res + static_cast<int64_t>(px) * (p.q_res * p.NW) + (ch >> 5);
                    res[f][c][0] = rp[0];
                    if (p.q_res == 2) res[f][c][1] = rp[p.NW];
                }
            }
        const int next_tile = tile + p.tile_step;
        const bool more_tiles = STAY && next_tile < p.tilesM;
        Range next_range{};
        if (more_tiles) {
            next_range = range_of(next_tile);
            fetch_pixels(next_range, tid);
        }

        // The sums.  K is walked granule by granule; the operands of a granule are read between the matrix instructions of the
        // one before it, into two sets of registers in turn.  Each instruction is fenced, since the compiler otherwise moves the
        // reads to their uses, where a lone wave of a SIMD waits for each.
        v16f_t acc[FW][FP];
        typedef int features_t __attribute__((ext_vector_type(CW == 1 ? 2 : CW)));      // (a vector of one ends up in scratch)
        struct Operands {
            v4i_t a[G][FW];
            features_t b[G][FP];
            int scaleA[G], scaleB;
        } even, odd;
        const uint32_t lane_codes = wc * 256 + (lane ^ (2 * lh)) * 4;
        const uint32_t *codes = sB + lane_codes;
        const uint32_t *table = sT + 2 * G * E;                  // offsets of the second and third granule
        int sB_now = scaleB0;
        typedef uint32_t offsets_t __attribute__((ext_vector_type(G * E)));      // of a granule
        constexpr int READS = G * (FW + FP), PRODUCTS = G * FW * FP;
        // read k of a granule at `off`, its weights at `codes` (several digits: the chunk's)
        auto read = [&](Operands &o, auto kc, const offsets_t &off, const uint32_t *codes) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value, g = k / (FW + FP), i = k % (FW + FP);
            if constexpr (i < FP && CW == 1) o.b[g][i] = features_t{*reinterpret_cast<const int *>(base[i] + off[E * g]), 0};
            else if constexpr (i < FP) o.b[g][i] = *reinterpret_cast<const features_t *>(base[i] + off[E * g]);
            else if constexpr (MULTI) o.a[g][i - FP] = *reinterpret_cast<const v4i_t *>(codes + ((off[E * g + 1] & ~1023u) >> 2) + (i - FP) * 256);
            else o.a[g][i - FP] = *reinterpret_cast<const v4i_t *>(codes + (g * FC + i - FP) * 256);
            if constexpr (MULTI && i == 0) o.scaleA[g] = scaleA + 2 * static_cast<int>(off[E * g + 1] & 1023u);      // (its lowest byte is read)
        };
        v4i_t b;                                                 // the codes of a pixel tile
        auto product = [&](const Operands &o, auto kc, auto first) __attribute__((always_inline)) {         // the first granule starts the sums
            constexpr int k = decltype(kc)::value, g = k / (FW * FP), f = k / FW % FP, c = k % FW;
            const v4i_t a = o.a[g][c];
            if constexpr (!PACKED) {
                b = o.b[g][f];
            } else if constexpr (c == 0) {
                const uint32_t w0 = o.b[g][f][0], w1 = o.b[g][f][1];    // (of one plane: not read)
                if constexpr (KA == OPK_U2) {                    // both words shifted at once: the bits that cross are masked
                    const uint64_t two = (static_cast<uint64_t>(w1) << 32 | w0) >> 2;
                    b = v4i_t{static_cast<int>(w0 & m3), static_cast<int>(w1 & m3), static_cast<int>(static_cast<uint32_t>(two) & m3), static_cast<int>(static_cast<uint32_t>(two >> 32) & m3)};
                } else {
                    v8i_t e;
                    expand_fp4<KA>(w0, w1, km, e);
                    b = v4i_t{e[0], e[1], e[2], e[3]};
                }
            }
            acc[c][f] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(v8i_t{a[0], a[1], a[2], a[3], 0, 0, 0, 0},
                                                                        v8i_t{b[0], b[1], b[2], b[3], 0, 0, 0, 0}, decltype(first)::value && g == 0 ? v16f_t{} : acc[c][f], 4, 4, 0,
                                                                        MULTI ? o.scaleB : scaleB0, 0, MULTI ? o.scaleA[g] : scaleA);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto multiply_and_read = [&](const Operands &o, Operands &next, const offsets_t &off, const uint32_t *codes, auto first) __attribute__((always_inline)) {
            if (MULTI) next.scaleB = sB_now;
            static_for<PRODUCTS>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value, from = k * READS / PRODUCTS, to = (k + 1) * READS / PRODUCTS;
                static_for<to - from>([&](auto jc) __attribute__((always_inline)) { read(next, std::integral_constant<int, from + decltype(jc)::value>{}, off, codes); });
                __builtin_amdgcn_sched_barrier(0);
                product(o, kc, first);
            });
        };
        struct Pair { offsets_t one, two; } t;                   // of the two granules after the one that is in `even`
        auto read_table = [&]() __attribute__((always_inline)) {
            typedef uint32_t pair_t __attribute__((ext_vector_type(2 * G * E), aligned(8 * G)));
            const pair_t v = *reinterpret_cast<const pair_t *>(table);
#pragma unroll
            for (int i = 0; i < G * E; ++i) { t.one[i] = v[i]; t.two[i] = v[G * E + i]; }
        };
        auto launched = [&](int k) __attribute__((always_inline)) {          // offsets of granule k < 2
            offsets_t off;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                off[E * g] = p.first[G * k + g];
                if (MULTI) off[E * g + 1] = p.first_codes[G * k + g];
            }
            return off;
        };
        // the sums' last granule: without the step that fills it up, where weights stay
        auto multiply_last = [&](const Operands &o, auto first) __attribute__((always_inline)) {
            static_for<FW * FP>([&](auto kc) __attribute__((always_inline)) { product(o, kc, first); });
            if (G == 2 && (!STAY || entries % 2 == 0))
                static_for<PRODUCTS - FW * FP>([&](auto kc) __attribute__((always_inline)) { product(o, std::integral_constant<int, FW * FP + decltype(kc)::value>{}, first); });
        };
        if (MULTI) even.scaleB = sB_now;
        const offsets_t off0 = launched(0);
        t.one = launched(1);
        if (!few) t.two = *reinterpret_cast<const offsets_t *>(table + G * E);
        static_for<READS>([&](auto kc) __attribute__((always_inline)) { read(even, kc, off0, codes); });
        if (STAY && FP * FW == 2 && !MULTI && stay_granules == 1) {              // (one granule starts and ends the sums; larger tiles would spill registers)
            multiply_last(even, std::true_type{});
        } else {
            Chunk at{0, 0};
            int half_buffer = 0;
            bool staged = STAY ? false : stage_next(at, half_buffer);            // the chunk after this one is on its way
            // A run: the granules of a chunk.  All but the last one of a weight digit have an even number.
            auto granules = [&]() __attribute__((always_inline)) {
                const int left = (MULTI ? p.steps : p.padded) - at.s0;
                return ((STAY ? left : min(kHaloChunk, left)) * (MULTI ? p.DA : 1) + G - 1) / G;
            };
            offsets_t off;
            auto first_of_pair = [&](auto first) __attribute__((always_inline)) {
                multiply_and_read(even, odd, t.one, MULTI ? codes : codes + G * FC * 256, first);
                off = t.two;
                if (!MULTI) codes += 2 * G * FC * 256;
                table += 2 * G * E;
            };
            auto second_of_pair = [&]() __attribute__((always_inline)) {
                read_table();
                multiply_and_read(odd, even, off, codes, std::false_type{});
            };
            int n = granules();
            if (n > 2) {
                first_of_pair(std::true_type{});
                second_of_pair();
                n -= 2;
            } else {
#pragma unroll
                for (int c = 0; c < FW; ++c)
#pragma unroll
                    for (int f = 0; f < FP; ++f) acc[c][f] = v16f_t{};
            }
            while (true) {
                for (int left = (n - 1) >> 1; left > 0; --left) {
                    first_of_pair(std::false_type{});
                    second_of_pair();
                }
                const bool pair = n % 2 == 0;                        // an odd last granule ends a digit: nothing is read ahead of the next
                if (!MULTI && !pair) break;
                if (!MULTI || pair) first_of_pair(std::false_type{});
                if (STAY || !staged) {                               // nothing to read
                    if (!MULTI || pair) even = odd;
                    break;
                }
                const Chunk next = after(at);                        // on to the next run
                const bool digit = MULTI && next.digit != at.digit;
                at = next;
                half_buffer ^= 1;
                __syncthreads();
                codes = sB + half_buffer * (kHaloChunk * FC * 256) + lane_codes;
                if (digit) {
                    sB_now = block_scale(sB_now, 2);
                    off = *reinterpret_cast<const offsets_t *>(sT + G * E);
                    table = sT + 2 * G * E;
                }
                if (MULTI && !pair) odd = even;
                second_of_pair();
                staged = stage_next(at, half_buffer);
                n = granules();
            }
            multiply_last(even, std::false_type{});
        }
        // the next tile's codes, read last before the barrier that began this tile
        if (more_tiles) {
            if (p.buffers == 1) __syncthreads();                 // (the only buffer: every wave is through with it)
            write_tile(sA + (p.buffers == 1 ? 0 : buffer ^ 1) * p.words_records, next_range);
        }

        // ---- outputs
        static_for<FW>([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            const int ch0 = n0 + 32 * (wc + c);
            if (ch0 >= p.N) return;
            if (p.Y) {
                static_for<FP * 4>([&](auto fk) {
                    constexpr int f = decltype(fk)::value / 4, k = decltype(fk)::value % 4;
                    const int ch = ch0 + 8 * k + 4 * lh;
                    const int4 y = make_int4(static_cast<int>(acc[c][f][4 * k]), static_cast<int>(acc[c][f][4 * k + 1]),
                                             static_cast<int>(acc[c][f][4 * k + 2]), static_cast<int>(acc[c][f][4 * k + 3]));
                    if (gm[f] < p.M && ch < p.N) *reinterpret_cast<int4 *>(p.Y + static_cast<int64_t>(gm[f]) * p.N + ch) = y;
                });
                return;
            }
            uint32_t d[FO][2];
            static_for<2>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                const v4f_t *const at = reinterpret_cast<const v4f_t *>(sP + 32 * (wc + c) + 16 * lh + 8 * q);
                const v4f_t sc[2] = {at[0], at[1]}, bi[2] = {at[8 * FC], at[8 * FC + 1]};
                static_for<FO>([&](auto fc) {
                    constexpr int f = decltype(fc)::value;
                    float v[8];
                    static_for<8>([&](auto rc) {
                        constexpr int j = decltype(rc)::value, r = 8 * q + j;
                        if constexpr (POOL) v[j] = pool4(p.pool, acc[c][0][r], acc[c][1][r], acc[c][2][r], acc[c][3][r]);
                        else v[j] = acc[c][f][r];
                    });
                    // the residual's plane words -> nibbles of this q
                    const uint32_t z0 = res[f][c][0] >> (2 * lh), z1 = res[f][c][1] >> (2 * lh);
                    const uint32_t e = q == 0 ? (z0 & 0x11111111u) | ((z1 << 1) & 0x22222222u) : ((z0 >> 1) & 0x11111111u) | (z1 & 0x22222222u);
                    d[f][q] = nibbles<!POOL>(v, sc, bi, p.res != nullptr, p.res_scale, e);
                });
            });
#pragma unroll
            for (int f = 0; f < FO; ++f) {
                const uint32_t word = plane_words(d[f][0], d[f][1], p.q_out);
                const int px = POOL ? gm[0] >> 2 : gm[f];
                if (gm[f] < p.M && lh < p.q_out)
                    p.out[static_cast<int64_t>(px) * (p.q_out * p.NW) + (lh * p.NW + (ch0 >> 5))] = word;
            }
        });
        if (!more_tiles) break;
        tile = next_tile;
        now = next_range;
        point(tile, buffer ^ (p.buffers - 1));
        __syncthreads();
    }
}

}  // namespace apnn
