// Convolution layers whose input pixels are staged once per block: the form for layers with enough output pixels to
// give every compute unit a block.
//
// A block owns 32 FC output channels x 128 FP output pixels.  In raster order over a frame padded by `pad` on every side, the
// pixels its taps touch are one contiguous range: the block stages the packed planes of that range in LDS once (the lane-private
// kernels load and check every pixel once per tap and channel tile), padding as zero records, so that a tap is one added offset
// and needs no range check.  Weights are expanded to FP4 codes while they are staged, chunk by chunk along K, and shared by
// the block's four waves; features of two planes are stored as interleaved pairs of bits, which leaves five vector
// instructions per 32 codes in the main loop.
//
// The matrix instruction gets the weights as its row operand, so that a lane holds sixteen channels of one pixel, and the
// planes of their codes are made in the lane (plane_codes.h).
//
// Bound by the vector instructions its waves issue up to 64 channels (stage 1 of the ResNet-18 shape at batch 128, by counters: a
// SIMD issues them in 59 % of its cycles, its matrix unit is busy in 23 %; 650 a wave tile of 64 x 64 outputs, prologue
// included), with more channels by what the two to four waves of a SIMD wait for in between (128 channels 44 and 23 %, 256 32
// and 23 %, 512 28 and 21 %).  Measured there, with and without residual: 46 and 32 us with lane-private loads, 16 and 15 here;
// 128 channels 29 and 23, 15 and 14; 256 channels 29, 15; 512 channels 31, 16.
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
    int rec;                 // words of a pixel's LDS record
    int pieces, share;       // pieces a record is staged in, log2 of the threads that share it
    int words_codes, words_records;          // LDS words of the weight codes, of one buffer of records
    int steps, chunk;        // matrix steps of a weight digit, of a weight chunk
    Divisor halves;          // half
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

// HW: channel words (steps) read together from a record; SW: channel words of a plane staged together (HW = 2: 4; HW = 1: 2, or
// 1 for an odd number of channel words); FP, FW: 32-pixel and 32-channel tiles of a wave (FW = 1: two waves share the pixels).
// MULTI: features of more than one digit.
// POOL (FP = 4): tile f of a wave holds member f of its 32 pooling grids, so that pooling is three instructions per output.
// STAY: the weights stay in LDS while the block walks over its tiles of pixels (grid-stride), and the next tile's pixels are in
// flight during the main loop.  Otherwise a block has one tile, and the weights pass through two buffers, a chunk each, with
// one barrier per chunk.
// PT: granules of a tap, 0 if known at run time only.  A lone wave of a SIMD issues an instruction every four or five cycles, and
// long sums on few pixels leave it alone: with PT the offsets inside a tap are part of the loads (s4 of the ResNet-18 shape
// at batch 128, 23 instructions a step instead of 33).
template <int KA, int HW, int SW, int FP, int FW, int PT, bool POOL, bool MULTI, bool STAY>
__global__ __launch_bounds__(256, FP == 1 ? 4 : FP * FW == 8 ? 2 : 3) void conv_halo_kernel(const ConvHaloParams p)
{
    static_assert(!POOL || FP == 4, "a wave's four pixel tiles are the members of its pooling grids");
    constexpr int PL = KA == OPK_U1 ? 1 : 2, GW = PL * HW;       // words of a granule: HW steps of a digit
    constexpr int FC = 2;                                        // channel tiles of a block
    constexpr int BP = 64 * FW * FP;                             // pixels of a tile
    constexpr int FETCH = STAY ? kHaloStay : kHaloChunk;         // weight steps in flight
    constexpr int NI = (FETCH * FC + 4 * HW - 1) / (4 * HW);      // granules of them a thread has in flight
    constexpr int U = SW == 1 ? 4 : 2;                           // staged pieces of pixels a thread has in flight
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    float *const sP = reinterpret_cast<float *>(lds);            // scales, then biases / 4: [tile][half][register]
    uint32_t *const sB = lds + 64 * FC;                          // weight codes: [buffer][step][tile][lane][4]
    uint32_t *const sA = sB + p.words_codes;                     // feature records: [buffer][pixel]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, lh = lane >> 5;
    const int wc = FW == 1 ? wave & 1 : 0, wp = FW == 1 ? wave >> 1 : wave;    // first channel tile, pixels of this wave
    // block -> channel tile, first tile of pixels
    const int tile0 = divide(static_cast<int>(blockIdx.x), p.per_column);
    const int n0 = (static_cast<int>(blockIdx.x) - tile0 * p.per_column.d) * 32 * FC;

    const __amdgpu_buffer_rsrc_t bufA = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.A), 0, p.bytesA, 0x00020000);
    const __amdgpu_buffer_rsrc_t bufB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.B), 0, p.bytesB, 0x00020000);
    constexpr uint32_t NOWHERE = 0x80000000u;                    // beyond every buffer: reads as zero

    // ---- weights.  Packed output: matrix row -> channel as plane_codes.h says; int32 output: in order, four to a store.
    // Rows beyond the last channel read that channel's (their results are not stored); steps beyond the last, and the step a
    // lane half lacks when the number of channel words is odd, read the first words (the features are zero there).
    const int wrow = lane & 31, wtile = lane >> 5;
    const int wch = p.Y ? wrow : code_channel_of_row(wrow);
    const int Kw = p.R * p.S * p.Cw;
    const uint32_t wlane = 4u * static_cast<uint32_t>(min(n0 + 32 * wtile + wch, p.N - 1) * (p.PB * Kw));
    uint32_t wv[NI][2][HW];
    auto fetch_weights = [&](int digit, int s0, int end) {
#pragma unroll
        for (int u = 0; u < NI; ++u) {
            const int it = wave + 4 * u, s = s0 + (it >> 1) * HW;    // (granule, half)
            if (s >= end) break;                                 // uniform
            const int tap = divide(s, p.halves), cw = (it & 1) * p.half + s - tap * p.half;
            const uint32_t at = 4u * static_cast<uint32_t>(2 * digit * Kw + (cw < p.Cw ? tap * p.Cw + cw : 0));
            const uint32_t second = 2 * digit + 1 < p.PB ? 4u * static_cast<uint32_t>(Kw) : 0u;
            if constexpr (HW == 2) {
                const auto t = __builtin_amdgcn_raw_buffer_load_b64(bufB, wlane, at, 0);
                wv[u][0][0] = t[0]; wv[u][0][1] = t[1];
            } else {
                wv[u][0][0] = __builtin_amdgcn_raw_buffer_load_b32(bufB, wlane, at, 0);
            }
            if (!p.pm1) {
                if constexpr (HW == 2) {
                    const auto t = __builtin_amdgcn_raw_buffer_load_b64(bufB, wlane, at + second, 0);
                    wv[u][1][0] = second ? t[0] : 0u; wv[u][1][1] = second ? t[1] : 0u;
                } else {
                    const uint32_t t = __builtin_amdgcn_raw_buffer_load_b32(bufB, wlane, at + second, 0);
                    wv[u][1][0] = second ? t : 0u;
                }
            }
        }
    };
    Fp4Masks km;
    km.m1 = reg_const(0x11111111u); km.m2 = reg_const(0x22222222u);
    km.m4 = reg_const(0x44444444u); km.m8 = reg_const(0x88888888u);
    auto write_weights = [&](uint32_t *codes, int steps) {
        auto all = [&](auto kind) {
#pragma unroll
            for (int u = 0; u < NI; ++u) {
                const int it = wave + 4 * u, s = (it >> 1) * HW, h = it & 1;
                if (s >= steps) break;                           // uniform
#pragma unroll
                for (int i = 0; i < HW; ++i) {
                    v8i_t f;
                    expand_fp4<decltype(kind)::value>(wv[u][0][i], wv[u][1][i], km, f);
                    *reinterpret_cast<int4 *>(codes + (((s + i) * FC + wtile) * 64 + 32 * h + wrow) * 4) = make_int4(f[0], f[1], f[2], f[3]);
                }
            }
        };
        if (p.pm1) all(std::integral_constant<int, OPK_PM1>{});
        else all(std::integral_constant<int, OPK_U2>{});
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
    uint32_t a0[U][SW], a1[U][SW];                               // a piece: SW words of each plane of a digit
    bool in[U];
    auto load_piece = [&](uint32_t bytes, uint32_t (&w)[SW]) {
        if constexpr (SW == 4) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(bufA, bytes, 0, 0);
            w[0] = t[0]; w[1] = t[1]; w[2] = t[2]; w[3] = t[3];
        } else if constexpr (SW == 2) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b64(bufA, bytes, 0, 0);
            w[0] = t[0]; w[1] = t[1];
        } else {
            w[0] = __builtin_amdgcn_raw_buffer_load_b32(bufA, bytes, 0, 0);
        }
    };
    auto fetch_pixels = [&](Range r, int q0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + 256 * u, pos = r.lo + (q >> p.share), g = q & tmask;
            const int n = divide(pos, p.frame), rem = pos - n * p.frame.d;
            const int yq = divide(rem, p.line), y = yq - p.pad, x = rem - yq * p.Wq - p.pad;
            const int cs = MULTI ? divide(g, p.digits) : g, d = MULTI ? g - cs * p.DA : 0, cw = cs * SW;
            in[u] = q < r.total && n < p.images && static_cast<unsigned>(y) < static_cast<unsigned>(p.H) &&
                    static_cast<unsigned>(x) < static_cast<unsigned>(p.W) && cw < p.Cw;
            const int at = (((n * p.H + y) * p.W + x) * p.PA + 2 * d) * p.Cw + cw;
            load_piece(in[u] ? 4u * static_cast<uint32_t>(at) : NOWHERE, a0[u]);
            if (KA == OPK_U2) load_piece(in[u] && 2 * d + 1 < p.PA ? 4u * static_cast<uint32_t>(at + p.Cw) : NOWHERE, a1[u]);
        }
    };
    auto write_pixels = [&](uint32_t *records, Range r, int q0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + 256 * u, g = q & tmask;
            if (q >= r.total || g >= p.pieces) continue;
            const int cs = MULTI ? divide(g, p.digits) : g, d = MULTI ? g - cs * p.DA : 0;
            uint32_t w[SW * PL];
#pragma unroll
            for (int i = 0; i < SW; ++i) {
                if (KA == OPK_U1) {
                    w[i] = a0[u][i];
                } else if (KA == OPK_U2) {                       // pairs of bits: even positions, odd positions
                    w[PL * i] = mask_select(0x55555555u, a0[u][i], a1[u][i] << 1);
                    w[PL * i + 1] = mask_select(0x55555555u, a0[u][i] >> 1, a1[u][i]);
                } else {                                         // signs, and the code's 1.0 inside the frame
                    w[PL * i] = in[u] ? ~a0[u][i] : 0u;
                    w[PL * i + 1] = in[u] ? 0x22222222u : 0u;
                }
            }
            // the piece's granules, DA granules apart
            uint32_t *dst = records + (q >> p.share) * p.rec + (cs * (SW / HW) * p.DA + d) * GW;
            const int apart = MULTI ? p.DA * GW : GW;
#pragma unroll
            for (int k = 0; k < SW / HW; ++k) {
                if constexpr (GW == 4) *reinterpret_cast<uint4 *>(dst + k * apart) = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
                else if constexpr (GW == 2) *reinterpret_cast<uint2 *>(dst + k * apart) = make_uint2(w[2 * k], w[2 * k + 1]);
                else dst[k * apart] = w[k];
            }
        }
    };

    Range now = range_of(tile0);
    fetch_weights(0, 0, STAY ? p.steps : min(p.chunk, p.steps));
    fetch_pixels(now, tid);
    if (!p.Y && tid < 64 * FC) {                                 // scale (first half of the threads) and bias of a channel
        const int k = tid % (32 * FC), ch = n0 + (k & ~31) + code_channel(k & 15, (k >> 4) & 1);
        float v = 0.0f;
        if (ch < p.N) v = tid < 32 * FC ? p.scale[ch] : quarter(p.bias[ch]);
        sP[tid] = v;
    }
    write_weights(sB, STAY ? p.steps : p.chunk);
    write_pixels(sA, now, tid);
    for (int q = tid + 256 * U; q < now.total; q += 256 * U) {
        fetch_pixels(now, q);
        write_pixels(sA, now, q);
    }
    __syncthreads();

    const uint32_t m3 = reg_const(0x33333333u);
    typedef uint32_t words_t __attribute__((ext_vector_type(GW)));
    auto expand = [&](const words_t &w, int i, v8i_t &o) {
        if constexpr (KA == OPK_U1) {
            expand_fp4<OPK_U1>(w[i], 0u, km, o);
        } else if constexpr (KA == OPK_U2) {                     // both words shifted at once: the bits that cross are masked
            const uint64_t two = (static_cast<uint64_t>(w[2 * i + 1]) << 32 | w[2 * i]) >> 2;
            o[0] = w[2 * i] & m3;
            o[1] = w[2 * i + 1] & m3;
            o[2] = static_cast<uint32_t>(two) & m3;
            o[3] = static_cast<uint32_t>(two >> 32) & m3;
            o[4] = o[5] = o[6] = o[7] = 0;
        } else {
            const uint32_t a = w[2 * i], one = w[2 * i + 1];
            o[0] = ((a << 3) & km.m8) | one;
            o[1] = ((a << 2) & km.m8) | one;
            o[2] = ((a << 1) & km.m8) | one;
            o[3] = (a & km.m8) | one;
            o[4] = o[5] = o[6] = o[7] = 0;
        }
    };
    // K is walked granule by granule: the granules of a tap, and the digits of a granule, follow each other in the record.
    const int per_tap = (p.half / HW) * (MULTI ? p.DA : 1);
    const uint32_t tap_step = 4u * static_cast<uint32_t>(p.rec) - 4u * GW * (per_tap - 1);
    const uint32_t row_step = tap_step + 4u * static_cast<uint32_t>((p.Wq - p.S) * p.rec);
    const int scaleA = static_cast<int>(reg_const(static_cast<uint32_t>(p.scaleA)));

    for (int tile = tile0, buffer = 0;; buffer ^= 1) {
        const int m0 = tile * BP, last = min(m0 + BP, p.M) - 1;
        const uint8_t *const records = reinterpret_cast<const uint8_t *>(sA + buffer * p.words_records);
        int gm[FP];                                              // this lane's pixels
        uint32_t base[FP];                                       // bytes: record of the first tap, this lane half's words
#pragma unroll
        for (int f = 0; f < FP; ++f) {
            gm[f] = POOL ? m0 + 4 * (32 * wp + lr) + f : m0 + (wp * FP + f) * 32 + lr;
            base[f] = 4u * static_cast<uint32_t>((position(min(gm[f], last)) - now.lo) * p.rec + lh * per_tap * GW);
        }
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

        v16f_t acc[FW][FP];
        // The operands of a granule are read one granule ahead of its matrix instructions, into two sets of registers in turn;
        // the empty statements keep the compiler from moving the reads back to their use (128 -> 128 channels, 128 x 28 x 28:
        // 16.4 us where it puts them, 13.8 here; it makes no difference where PT is known).
        struct Operands {
            words_t w[FP];
            v4i_t a[HW][FW];
            int scale;
        } even, odd;
        const uint32_t *codes = sB + wc * 256 + lane * 4;
        int scaleB = static_cast<int>(reg_const(static_cast<uint32_t>(p.scaleB)));
        uint32_t off = 0;
        int g = 0, sc = 0, d = 0;
        auto load = [&](Operands &o) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < FP; ++f) o.w[f] = *reinterpret_cast<const words_t *>(records + (base[f] + off));
#pragma unroll
            for (int i = 0; i < HW; ++i)
#pragma unroll
                for (int c = 0; c < FW; ++c) o.a[i][c] = *reinterpret_cast<const v4i_t *>(codes + (i * FC + c) * 256);
            o.scale = MULTI ? block_scale(scaleA, 2 * d) : scaleA;
            asm volatile("" ::: "memory");
        };
        auto advance = [&](bool more) __attribute__((always_inline)) {                          // more: of this chunk
            const bool tap = ++g == per_tap;
            g = tap ? 0 : g;
            sc += tap ? 1 : 0;
            const bool row = sc == p.S;
            sc = row ? 0 : sc;
            off += row ? row_step : tap ? tap_step : 4u * GW;
            if (MULTI) d = d + 1 == p.DA ? 0 : d + 1;
            codes += more && (!MULTI || d == 0) ? HW * FC * 256 : 0;
        };
        auto multiply = [&](auto first, const Operands &o) __attribute__((always_inline)) {     // the first granule starts the sums
#pragma unroll
            for (int i = 0; i < HW; ++i)
#pragma unroll
                for (int f = 0; f < FP; ++f) {
                    v8i_t b;
                    expand(o.w[f], i, b);
#pragma unroll
                    for (int c = 0; c < FW; ++c)
                        acc[c][f] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            v8i_t{o.a[i][c][0], o.a[i][c][1], o.a[i][c][2], o.a[i][c][3], 0, 0, 0, 0}, b,
                            decltype(first)::value && i == 0 ? v16f_t{} : acc[c][f], 4, 4, 0, scaleB, 0, o.scale);
                }
        };
        // `left` granules of a chunk, the first one in odd; more: granules of this weight digit after the chunk
        auto rest_of_chunk = [&](int left, bool more) __attribute__((always_inline)) {
            for (; left >= 2; left -= 2) {
                advance(true);
                load(even);
                multiply(std::false_type{}, odd);
                advance(left > 2);
                off = left > 2 || more ? off : 0u;               // (read, not used)
                load(odd);
                multiply(std::false_type{}, even);
            }
            if (left) {
                multiply(std::false_type{}, odd);
                advance(false);
            }
        };
        const int all = p.steps / HW * (MULTI ? p.DA : 1);       // granules of a weight digit
        if constexpr (STAY) {
            load(even);
            advance(all > 1);
            off = all > 1 ? off : 0u;
            load(odd);
            multiply(std::true_type{}, even);
            rest_of_chunk(all - 1, false);
        } else if constexpr (PT > 0) {
            static_assert(PT % 2 == 0 && !MULTI);
            // granule g of the tap at `off`, whose codes begin at `codes`
            auto load_at = [&](Operands &o, int g, const uint8_t *const (&src)[FP]) __attribute__((always_inline)) {
#pragma unroll
                for (int f = 0; f < FP; ++f) o.w[f] = *reinterpret_cast<const words_t *>(src[f] + 4 * GW * g);
#pragma unroll
                for (int i = 0; i < HW; ++i)
#pragma unroll
                    for (int c = 0; c < FW; ++c) o.a[i][c] = *reinterpret_cast<const v4i_t *>(codes + ((g * HW + i) * FC + c) * 256);
                o.scale = scaleA;
            };
            const uint8_t *src[FP];
            auto point = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int f = 0; f < FP; ++f) src[f] = records + (base[f] + off);
            };
            // a tap, its first granule in even; `next`: the tap after it is in this chunk
            auto tap = [&](auto first, bool next, bool more) __attribute__((always_inline)) {
                static_for<PT>([&](auto gc) {
                    constexpr int g = decltype(gc)::value;
                    constexpr bool starts = decltype(first)::value && g == 0;
                    if constexpr (g + 1 < PT) {
                        if constexpr (g % 2 == 0) load_at(odd, g + 1, src);
                        else load_at(even, g + 1, src);
                    } else {
                        const bool row = ++sc == p.S;
                        sc = row ? 0 : sc;
                        off += row ? row_step + 4u * GW * (PT - 1) : tap_step + 4u * GW * (PT - 1);
                        off = more ? off : 0u;                   // (read, not used)
                        codes += next ? PT * HW * FC * 256 : 0;
                        point();
                        load_at(even, 0, src);
                    }
                    multiply(std::integral_constant<bool, starts>{}, g % 2 == 0 ? even : odd);
                });
            };
            int digit = 0, s0 = 0, half_buffer = 0;              // weight digit, first step and buffer of the chunk
            constexpr int tap_steps = PT * HW, chunk_taps = kHaloChunk / tap_steps;
            int left = min(chunk_taps, p.R * p.S);               // taps of the chunk that are to do
            point();
            load_at(even, 0, src);
            tap(std::true_type{}, left > 1, all > PT);
            --left;
            while (true) {
                int nd = digit, ns = s0 + p.chunk;               // the chunk after this one
                if (ns >= p.steps) { ns = 0; ++nd; }
                const bool more = nd < p.DB;
                if (more) fetch_weights(nd, ns, min(ns + p.chunk, p.steps));
                for (; left > 0; --left) tap(std::false_type{}, left > 1, left > 1 || (more && nd == digit));
                if (!more) break;
                if (nd != digit) {                               // the next weight digit starts at the first tap again
                    off = 0; sc = 0;
                    scaleB = block_scale(scaleB, 2);
                }
                digit = nd;
                s0 = ns;
                half_buffer ^= 1;
                uint32_t *const to = sB + half_buffer * (p.chunk * FC * 256);
                write_weights(to, p.chunk);                      // read last before the barrier two chunks ago
                codes = to + wc * 256 + lane * 4;
                __syncthreads();
                left = divide(min(p.chunk, p.steps - s0), p.halves);
                point();
                load_at(even, 0, src);
            }
        } else {
            int digit = 0, s0 = 0, half_buffer = 0;              // weight digit, first step and buffer of the chunk
            int left = min(p.chunk, p.steps) / HW * (MULTI ? p.DA : 1) - 1;
            load(even);
            advance(left > 0);
            off = all > 1 ? off : 0u;
            load(odd);
            multiply(std::true_type{}, even);
            while (true) {
                int nd = digit, ns = s0 + p.chunk;               // the chunk after this one
                if (ns >= p.steps) { ns = 0; ++nd; }
                const bool more = nd < p.DB;
                if (more) fetch_weights(nd, ns, min(ns + p.chunk, p.steps));
                rest_of_chunk(left, more && nd == digit);
                if (!more) break;
                if (nd != digit) {                               // the next weight digit starts at the first tap again
                    off = 0; g = 0; sc = 0; d = 0;
                    scaleB = block_scale(scaleB, 2);
                }
                digit = nd;
                s0 = ns;
                half_buffer ^= 1;
                uint32_t *const to = sB + half_buffer * (p.chunk * FC * 256);
                write_weights(to, p.chunk);                      // read last before the barrier two chunks ago
                codes = to + wc * 256 + lane * 4;
                __syncthreads();
                left = min(p.chunk, p.steps - s0) / HW * (MULTI ? p.DA : 1);
                load(odd);
            }
        }
        // the next tile's records, read last before the barrier that began this tile
        if (more_tiles) {
            uint32_t *const to = sA + (buffer ^ 1) * p.words_records;
            write_pixels(to, next_range, tid);
            for (int q = tid + 256 * U; q < next_range.total; q += 256 * U) {
                fetch_pixels(next_range, q);
                write_pixels(to, next_range, q);
            }
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
        __syncthreads();
    }
}

}  // namespace apnn
