// FP4 matrix-core kernel for products and convolutions with few outputs: 16 x 16 tiles, the K range of a tile shared out among all
// waves of its block.
//
// Such a product lasts as long as one block does: a launch, one or two memory round trips, and about 35 vector
// instructions to expand the operands of a step, at five cycles each while a SIMD has one wave.  32 x 32 tiles of 8 x 4096
// outputs are 128 blocks on 256 compute units, three quarters of each padding.  Here a step covers twice the K range for
// a quarter of the outputs (the same expansion work), so the same product is 256 blocks with half the steps, and eight
// waves hide each other's latency where K is long.  Measured on w1a2 products in a replayed graph, 32 x 32 tiles before,
// this after (us): 8 x 4096, K = 25088 16.9, 7.5; K = 9216 7.1, 4.9; K = 4096 5.0, 3.9; 64 x 1024, K = 1024 4.0, 3.3;
// 128 x 128, K = 128 (64 x 64 tile before) 4.1, 3.2.  Convolutions: 7 x 7 of 512 channels to 8 x 1 x 1 x 4096 16.5, 8.8;
// 3 x 3, 384 -> 256 channels at 13 x 13 5.9, 4.4.  (A call outside a graph costs the host 3.5 to 4 us: of the smallest of these it
// shows nothing.)
// Four and eight waves are one kernel, two groups in flight: a network's first pass fetches every instance's code from memory, and
// a second one for eight waves (four groups in flight) made that of the AlexNet shape at batch 1 5 to 10 us longer without
// being faster after it (46.1 us either way).
#pragma once
#include "mfma_kernel.h"

namespace apnn {

typedef float v4f_t __attribute__((ext_vector_type(4)));

// Block = one 16 x 16 tile of outputs.  A step is one 16 x 16 x 128 matrix instruction: lane group g = lane / 16
// supplies 32 consecutive K positions (one plane word) of row / column lane % 16.  K is walked in groups of four
// steps = 16 words, of which lane group g loads words 4 g .. 4 g + 3 (one 16-byte load per plane, 64 consecutive
// bytes per row of a matrix); wave w takes groups w, w + waves, ...
// (p.nk: the waves of a block, four or eight)  Words at and beyond Kw read as zero.
template <int KA, int KB, int VW, bool CONV, int GMAX>
__global__ __launch_bounds__(512) void mfma_tile16_kernel(const MfmaParams p)
{
    constexpr int LA = DigitPlanes<KA>::value, LB = DigitPlanes<KB>::value;
    __shared__ float sRed[8][4][64];                    // wave w < 4 finishes accumulator register w

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int tilesN = (p.N + 15) / 16;
    const int m0 = (blockIdx.x / tilesN) * 16, n0 = (blockIdx.x % tilesN) * 16;
    const int gmA = m0 + lr, gn = n0 + lr;
    const bool a_ok = gmA < p.M, b_ok = gn < p.N;
    const uint32_t *a_row = p.A + static_cast<int64_t>(gmA) * p.PA * p.ldwA;      // matrix mode
    const uint32_t *b_row = p.B + static_cast<int64_t>(gn) * p.PB * p.ldwB;

    int a_h0 = 0, a_w0 = 0;
    int64_t a_pix = 0;
    if constexpr (CONV) {
        int wo, ho, n;
        conv_row_to_pixel(p, gmA, n, ho, wo);
        a_h0 = ho * p.stride - p.pad;
        a_w0 = wo * p.stride - p.pad;
        a_pix = static_cast<int64_t>(n) * p.H * p.W;
    }

    Fp4Masks km;
    km.m1 = reg_const(0x11111111u); km.m2 = reg_const(0x22222222u);
    km.m4 = reg_const(0x44444444u); km.m8 = reg_const(0x88888888u);

    const int GT = (p.Kw + 15) / 16;
    const int waves = p.nk, log_waves = waves == 8 ? 3 : 2;
    const int G = wave < GT ? (GT - wave + waves - 1) >> log_waves : 0;    // groups of this wave

    auto load_a = [&](int plane, int kk) -> uint4 {
        const bool validity = KA == OPK_PM1Z && plane == 1;     // all ones for taps inside the frame, made up here
        if (validity) plane = 0;
        if (!a_ok || kk >= p.Kw || plane >= p.PA) return make_uint4(0, 0, 0, 0);
        if constexpr (CONV) return load_conv_a<VW>(p, a_pix, plane, kk, a_h0, a_w0, validity);
        else return *reinterpret_cast<const uint4 *>(a_row + static_cast<int64_t>(plane) * p.ldwA + kk);
    };
    auto load_b = [&](int plane, int kk) -> uint4 {
        if (!b_ok || kk >= p.Kw || plane >= p.PB) return make_uint4(0, 0, 0, 0);
        const uint32_t *src = b_row + static_cast<int64_t>(plane) * p.ldwB + kk;
        if constexpr (CONV) return load_conv_b<VW>(src, p.Kw - kk);
        else return *reinterpret_cast<const uint4 *>(src);
    };

    // the epilogue's per-channel parameters: their latency hides behind the main loop
    float sc = 0.0f, bi = 0.0f;
    if (p.scale && wave < 4 && b_ok) { sc = p.scale[gn]; bi = p.bias[gn]; }

    uint32_t res01[2] = {0, 0};                         // ... and the residual's first two planes
    const uint32_t *rp = p.res;
    if (p.res && wave < 4 && b_ok) {
        const int row = p.pool ? (m0 >> 2) + lg : m0 + 4 * lg + wave;
        if (row < (p.pool ? p.M >> 2 : p.M)) {
            rp += static_cast<int64_t>(row) * p.q_res * p.NW + (gn >> 5);
            res01[0] = rp[0];
            if (p.q_res > 1) res01[1] = rp[p.NW];
        }
    }

    // Digit pairs and the groups of each as one flat sequence, GMAX entries at a time with all their loads in
    // flight; the weight 4^(da + db) of a pair (Eq. 1) enters as the block scales of the matrix instruction.
    v4f_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
    const int total = p.DA * p.DB * G;
    int da = 0, db = 0, grp = 0;
    for (int e0 = 0; e0 < total; e0 += GMAX) {
        uint4 wa[GMAX][LA], wb[GMAX][LB];
        int sa[GMAX], sb[GMAX];
#pragma unroll
        for (int g = 0; g < GMAX; ++g) {
            const int kk = e0 + g < total ? 16 * (wave + (grp << log_waves)) + 4 * lg : p.Kw;
            sa[g] = block_scale(0x7f7f7f7f, 2 * da);
            sb[g] = block_scale(0x7f7f7f7f, 2 * db);
#pragma unroll
            for (int pl = 0; pl < LB; ++pl) wb[g][pl] = load_b((LB == 2 ? 2 * db : db) + pl, kk);
#pragma unroll
            for (int pl = 0; pl < LA; ++pl) wa[g][pl] = load_a((LA == 2 ? 2 * da : da) + pl, kk);
            ++grp;                                      // next group, then next digit of B, then next digit of A
            const bool wg = grp == G;
            grp = wg ? 0 : grp;
            db += wg ? 1 : 0;
            const bool wd = db == p.DB;
            db = wd ? 0 : db;
            da += wd ? 1 : 0;
        }
#pragma unroll
        for (int g = 0; g < GMAX; ++g) {
            if (e0 + g < total) {
                const uint32_t a0[4] = {wa[g][0].x, wa[g][0].y, wa[g][0].z, wa[g][0].w};
                const uint32_t a1[4] = {wa[g][LA - 1].x, wa[g][LA - 1].y, wa[g][LA - 1].z, wa[g][LA - 1].w};
                const uint32_t b0[4] = {wb[g][0].x, wb[g][0].y, wb[g][0].z, wb[g][0].w};
                const uint32_t b1[4] = {wb[g][LB - 1].x, wb[g][LB - 1].y, wb[g][LB - 1].z, wb[g][LB - 1].w};
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    v8i_t fa, fb;
                    expand_fp4<KA>(a0[st], a1[st], km, fa);
                    expand_fp4<KB>(b0[st], b1[st], km, fb);
                    acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa, fb, acc, 4, 4, 0, sa[g], 0, sb[g]);
                }
            }
        }
    }

#pragma unroll
    for (int r = 0; r < 4; ++r) sRed[wave][r][lane] = acc[r];
    __syncthreads();
    if (wave >= 4 || (p.pool && wave > 0)) return;
    float v = 0.0f;                                     // register `wave` of the tile: row 4 lg + wave, column lr
#pragma unroll
    for (int k = 0; k < 4; ++k) v += sRed[k][wave][lane];
    if (waves == 8) {
#pragma unroll
        for (int k = 4; k < 8; ++k) v += sRed[k][wave][lane];
    }
    int gm = m0 + 4 * lg + wave, M = p.M, c0 = p.c0;
    if constexpr (CONV) {
        if (p.pool) {                                   // the four registers of a lane are one pooling grid
            float o[3] = {0.0f, 0.0f, 0.0f};
            for (int k = 0; k < waves; ++k)
#pragma unroll
                for (int r = 0; r < 3; ++r) o[r] += sRed[k][r + 1][lane];
            v = pool4(p.pool, v, o[0], o[1], o[2]);
            gm >>= 2; M >>= 2;
            c0 = p.pool == 2 ? 4 * c0 : c0;
        }
    }
    const bool ok = gm < M && b_ok;
    const int y = static_cast<int>(v * p.out_scale) + c0;             // exact: v is a multiple of 1 / out_scale
    if (p.Y && ok) p.Y[static_cast<int64_t>(gm) * p.N + gn] = y;
    if (!p.scale) return;
    float t = __fmaf_rn(sc, static_cast<float>(y), bi);
    if (p.res) {
        uint32_t code = ((res01[0] >> (gn & 31)) & 1u) | (((res01[1] >> (gn & 31)) & 1u) << 1);
        if (ok)
            for (int b = 2; b < p.q_res; ++b) code |= ((rp[b * p.NW] >> (gn & 31)) & 1u) << b;
        t = __fmaf_rn(p.res_scale, static_cast<float>(code), t);
    }
    if (p.T && ok) p.T[static_cast<int64_t>(gm) * p.N + gn] = t;
    if (!p.out) return;
    // (N is a multiple of 32 whenever planes are written: a tile has all its channels, half a plane word)
    const float qmax = static_cast<float>((1 << p.q_out) - 1);
    float f = floorf(t);
    f = (f >= 0.0f) ? f : 0.0f;
    f = (f > qmax) ? qmax : f;
    const uint32_t code = static_cast<uint32_t>(f);
    uint16_t *op = reinterpret_cast<uint16_t *>(p.out) + 2 * (static_cast<int64_t>(gm) * p.q_out * p.NW) + (gn >> 4);
    for (int b = 0; b < p.q_out; ++b) {
        const unsigned long long bal = __ballot((code >> b) & 1u);
        if (lr == 0 && ok) op[2 * static_cast<int64_t>(b) * p.NW] = static_cast<uint16_t>(bal >> (16 * lg));
    }
}

}  // namespace apnn
