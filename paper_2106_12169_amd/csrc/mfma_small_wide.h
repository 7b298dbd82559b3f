// Small-layer matrix-core kernel with wave tiles of 32 x 32 FN outputs (FN column tiles of 32 channels per wave
// tile): the form for large convolution layers, where every wave owns its own tile (no K split) and the kernel is
// bound by the instructions its waves issue.  The row operand of a wave tile - pixel decoding, tap addresses,
// loads, expansion to FP4 codes - is then shared by 32 FN output channels: at batch 128 the stage-1 layers of the
// ResNet-18 shape take 41 - 54 us with FN = 2 against 59 - 74 us with FN = 1 (FN = 4 with its larger register
// footprint was slower again).  For the same reason the loader is not that of mfma_small_kernel: receptive-field
// positions are walked instead of divided, offsets are 32-bit into range-checked buffers (no branch, select or 64-bit
// address per load), a digit's planes share one position, K is padded to a loader vector per lane half instead of to four
// steps, and the wave's tile is held in scalar registers.  Whole passes with that loader, and with the loads of missing groups
// left out as well: ResNet-18 shape batch 128 690 -> 637 -> 611 us, VGG-16 shape batch 8 322 -> 301 -> 289.  One word per step
// (an odd number of channel words) still divides for its position, once for four words (load_conv_a_words).
#pragma once
#include "mfma_kernel.h"

namespace apnn {

template <int KA, int KB, int VW, int GMAX, int FN>
__device__ __forceinline__ void mfma_small_wide_body(const MfmaParams &p, const int block)
{
    // GMAX: groups of four steps whose loads are in flight together; the load buffers set the register count and with it the
    // waves a SIMD holds.  2 here: four waves for single planes on a side, as 1 x 1 layers need, which are mostly epilogue.
    // FN: 32-column tiles per wave tile: a row operand is loaded, expanded and its pixel decoded once for 32 FN output
    // channels.  A large layer is bound by the instructions its waves issue, and the row side is about a third of them.
    constexpr int LA = DigitPlanes<KA>::value, LB = DigitPlanes<KB>::value;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // scalar: so is the tile's place
    const int lr = lane & 31, lh = lane >> 5;

    // tile of this wave: the block covers four consecutive tiles of the row-major tile grid
    const int tilesN = (p.N + 32 * FN - 1) / (32 * FN), tilesM = (p.M + 31) / 32;
    const int tile = block * 4 + wave;
    const bool live = tile < tilesM * tilesN;           // trailing waves of the last block have no tile
    const int m0 = (tile / tilesN) * 32, n0 = (tile % tilesN) * 32 * FN;

    // A lane half walks NS words (= steps) of K, whole loader vectors, in groups of four; the last group may be shorter.
    const int NS = (((p.Kw + 1) >> 1) + VW - 1) / VW * VW;
    const int G = (NS + 3) / 4;

    Fp4Masks km;
    km.m1 = reg_const(0x11111111u); km.m2 = reg_const(0x22222222u);
    km.m4 = reg_const(0x44444444u); km.m8 = reg_const(0x88888888u);

    // this lane's operand rows
    const int gmA = m0 + lr;
    const bool a_ok = live && gmA < p.M;
    int a_h0 = 0, a_w0 = 0;
    int64_t a_pix = 0;
    {
        int wo, ho, n;
        conv_row_to_pixel(p, gmA, n, ho, wo);
        a_h0 = ho * p.stride - p.pad;
        a_w0 = wo * p.stride - p.pad;
        a_pix = static_cast<int64_t>(n) * p.H * p.W;
    }
    // Both operands are buffers with 32-bit byte offsets (the host checks their sizes), and every load is unconditional:
    // row words that contribute nothing (taps outside the frame, K beyond Kw, rows beyond M, a missing plane) get an offset
    // beyond the buffer, for which the load returns zero.  K beyond Kw and rows beyond the operand need that on the row side
    // alone: a zero code there cancels whatever the column operand holds.  A missing plane needs it on its own side, since the
    // other operand's codes are not zero there: hence `exists` in load_b.
    const __amdgpu_buffer_rsrc_t bufA = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.A), 0, p.bytesA, 0x00020000);
    const __amdgpu_buffer_rsrc_t bufB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.B), 0, p.bytesB, 0x00020000);
    constexpr uint32_t NOWHERE = 0x80000000u;
    auto load_words = [](__amdgpu_buffer_rsrc_t buf, uint32_t bytes, uint32_t *w) {       // one loader vector
        if constexpr (VW == 4) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(buf, bytes, 0, 0);
            w[0] = t[0]; w[1] = t[1]; w[2] = t[2]; w[3] = t[3];
        } else {
            const auto t = __builtin_amdgcn_raw_buffer_load_b64(buf, bytes, 0, 0);
            w[0] = t[0]; w[1] = t[1];
        }
    };
    const uint32_t *a_image = p.A + (a_ok ? a_pix * p.PA * p.Cw : 0);             // one word per step: this lane's image
    const int pixel = p.PA * p.Cw, row_words = p.W * pixel;
    const int a_first = a_ok ? static_cast<int>(a_pix) * pixel + a_h0 * row_words + a_w0 * pixel : 0;
    if (!a_ok) a_h0 = -(1 << 30);                       // no tap of it lies in the frame
    int b_first[FN];                                    // words
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int gnB = n0 + 32 * j + lr;
        b_first[j] = gnB < p.N ? gnB * p.PB * p.ldwB : 0;
    }

    // Position in the receptive field: word k = (r, sc, cw), `off` words beyond the pixel's first tap.  Walked, not divided.
    struct Walk { int k, cw, sc, r, off; };
    auto walk_to = [&](int k) {
        Walk t;
        const int tap = static_cast<int>((static_cast<float>(k) + 0.5f) * p.invCw);
        t.k = k;
        t.cw = k - tap * p.Cw;
        tap_to_rs(p, tap, t.r, t.sc);
        t.off = t.r * row_words + t.sc * pixel + t.cw;
        return t;
    };
    const int next_tap = pixel - p.Cw, next_row = row_words - p.S * pixel;
    auto advance = [&](Walk &t) {                       // by one loader vector
        t.k += VW;
        t.cw += VW;
        t.off += VW;
        const bool wt = t.cw == p.Cw;
        t.cw = wt ? 0 : t.cw;
        t.off += wt ? next_tap : 0;
        t.sc += wt ? 1 : 0;
        const bool wr = t.sc == p.S;
        t.sc = wr ? 0 : t.sc;
        t.off += wr ? next_row : 0;
        t.r += wr ? 1 : 0;
    };
    // Words of planes plane .. plane + LA - 1 of four steps at the position `t`, which moves on by four steps.
    auto load_a = [&](uint4 (&v)[LA], int plane, Walk &t) {
        if constexpr (VW == 1) {
            for (int pl = 0; pl < LA; ++pl) {
                const bool validity = KA == OPK_PM1Z && pl == 1;
                v[pl] = !a_ok || t.k >= p.Kw || (!validity && plane + pl >= p.PA)
                            ? make_uint4(0, 0, 0, 0)
                            : load_conv_a_words(p, a_image, validity ? 0 : plane + pl, t.k, a_h0, a_w0, validity);
            }
            t.k += 4;
        } else {
#pragma unroll
            for (int part = 0; part < 4 / VW; ++part) {
                const bool in = t.k < p.Kw && static_cast<unsigned>(a_h0 + t.r) < static_cast<unsigned>(p.H) &&
                                static_cast<unsigned>(a_w0 + t.sc) < static_cast<unsigned>(p.W);
                const int off = a_first + t.off + plane * p.Cw;
#pragma unroll
                for (int pl = 0; pl < LA; ++pl) {
                    uint32_t w[VW];
                    if (KA == OPK_PM1Z && pl == 1) {    // all ones for taps inside the frame, made up here
#pragma unroll
                        for (int i = 0; i < VW; ++i) w[i] = in ? ~0u : 0u;
                    } else {
                        const bool ok = in && (pl == 0 || plane + pl < p.PA);
                        load_words(bufA, ok ? 4u * static_cast<uint32_t>(off + pl * p.Cw) : NOWHERE, w);
                    }
                    if constexpr (VW == 4) v[pl] = make_uint4(w[0], w[1], w[2], w[3]);
                    else if (part == 0) { v[pl].x = w[0]; v[pl].y = w[1]; }
                    else { v[pl].z = w[0]; v[pl].w = w[1]; }
                }
                advance(t);
            }
        }
    };
    auto load_b = [&](int j, int plane, int pl, int kk) -> uint4 {
        uint4 v = make_uint4(0, 0, 0, 0);
        const bool exists = pl == 0 || plane + pl < p.PB;
        const int at = b_first[j] + (plane + pl) * p.ldwB + kk;
        if constexpr (VW == 1) {
            if (exists && kk < p.Kw) v = load_conv_b_words(p.B + at, p.Kw - kk);
        } else {                                        // rows are whole loader vectors long and aligned to them
            uint32_t w[4];
#pragma unroll
            for (int part = 0; part < 4 / VW; ++part)
                load_words(bufB, exists ? 4u * static_cast<uint32_t>(at + part * VW) : NOWHERE, w + part * VW);
            v = make_uint4(w[0], w[1], w[2], w[3]);
        }
        return v;
    };

    // the epilogue's per-channel parameters and residual words: their latency hides behind the main loop
    // (residual: one load per wave and group of eight rows: lane l holds the word of row l & 7, plane l >> 3)
    constexpr int NG = 4;                               // groups of four registers = eight rows of a tile
    float sc[FN], bi[FN];
    uint32_t pre_res[FN][NG];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int gn = n0 + 32 * j + lr;
        sc[j] = 0.0f; bi[j] = 0.0f;
        if (p.scale && live && gn < p.N) { sc[j] = p.scale[gn]; bi[j] = p.bias[gn]; }
#pragma unroll
        for (int g = 0; g < NG; ++g)
            pre_res[j][g] = (live && p.res && !p.pool) ? load_res_rows8(p, m0 + 8 * g, gn >> 5, lane) : 0u;
    }

    // Digit pairs (da, db) and the groups of four steps of each are walked as one
    // flat sequence, GMAX entries at a time with all their loads in flight together,
    // so that a multi-digit layer (e.g. 8-bit features: four passes) pays one memory
    // round trip, not one per pass.  The weight 4^(da + db) of a pair (Eq. 1) enters
    // as the block scales of the matrix instruction, which makes the order free.
    const int total = p.Kw > 0 ? p.DA * p.DB * G : 0;
    const int kbase = lh * NS;                          // first K word of this lane's first group

    v16f_t acc[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;

    // the four steps of one group: operand words of the lowest and highest plane of the digit (one and the same
    // for single-plane kinds), block scales of the digit pair
    auto run_group = [&](const uint4 (&wa)[LA], const uint4 (&wb)[FN][LB], int sa, int sb, int steps) {
        const uint32_t a0[4] = {wa[0].x, wa[0].y, wa[0].z, wa[0].w};
        const uint32_t a1[4] = {wa[LA - 1].x, wa[LA - 1].y, wa[LA - 1].z, wa[LA - 1].w};
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            if (VW < 4 && st >= VW && st >= steps) break;       // uniform
            v8i_t fa;
            expand_fp4<KA>(a0[st], a1[st], km, fa);
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const uint32_t b0[4] = {wb[j][0].x, wb[j][0].y, wb[j][0].z, wb[j][0].w};
                const uint32_t b1[4] = {wb[j][LB - 1].x, wb[j][LB - 1].y, wb[j][LB - 1].z, wb[j][LB - 1].w};
                v8i_t fb;
                expand_fp4<KB>(b0[st], b1[st], km, fb);
                acc[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa, fb, acc[j], 4, 4, 0, sa, 0, sb);
            }
        }
    };

    // Single planes on both sides: never more than one digit pair.  The general loop, compiled in all the same, and the loads of
    // a group that does not exist had taken these forms from 74 - 80 registers to 97 - 104 (three waves per SIMD instead of
    // four): 64 x 56 x 56, 128 -> 128 channels, 1 x 1, w1a1 24.4 us, without them 19.0.
    constexpr bool ONE_PAIR = KA != OPK_U2 && KB != OPK_U2;
    if (ONE_PAIR || p.DA * p.DB == 1) {                 // one digit pair (most layers): unit scales, plain group loop
        Walk t = walk_to(kbase);
        for (int g0 = 0; g0 < (p.Kw > 0 ? G : 0); g0 += GMAX) {
            uint4 wa[GMAX][LA], wb[GMAX][FN][LB];
#pragma unroll
            for (int g = 0; g < GMAX; ++g) {
                if (g > 0 && g0 + g >= G) break;        // uniform
                const int kk = kbase + 4 * (g0 + g);
                load_a(wa[g], 0, t);
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int pl = 0; pl < LB; ++pl) wb[g][j][pl] = load_b(j, 0, pl, kk);
            }
#pragma unroll
            for (int g = 0; g < GMAX; ++g)
                if (g0 + g < G) run_group(wa[g], wb[g], 0x7f7f7f7f, 0x7f7f7f7f, NS - 4 * (g0 + g));
        }
    }
    int da = 0, db = 0, grp = 0;                        // position in the flat sequence (scalar counters, no divisions)
    const Walk start = walk_to(kbase);
    Walk t = start;
    for (int e0 = 0; e0 < (ONE_PAIR || p.DA * p.DB == 1 ? 0 : total); e0 += GMAX) {
        uint4 wa[GMAX][LA], wb[GMAX][FN][LB];
        int sa[GMAX], sb[GMAX], steps[GMAX];
#pragma unroll
        for (int g = 0; g < GMAX; ++g) {
            const int planeA = LA == 2 ? 2 * da : da, planeB = LB == 2 ? 2 * db : db;
            const int kk = kbase + 4 * grp;             // (beyond the end: read, not used; jumping over it measured slower)
            steps[g] = NS - 4 * grp;
            sa[g] = block_scale(0x7f7f7f7f, 2 * da);
            sb[g] = block_scale(0x7f7f7f7f, 2 * db);
            load_a(wa[g], planeA, t);
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int pl = 0; pl < LB; ++pl) wb[g][j][pl] = load_b(j, planeB, pl, kk);
            ++grp;                                      // next group, then next digit of B, then next digit of A
            const bool wg = grp == G;
            grp = wg ? 0 : grp;
            if (wg) t = start;
            db += wg ? 1 : 0;
            const bool wd = db == p.DB;
            db = wd ? 0 : db;
            da += wd ? 1 : 0;
        }
#pragma unroll
        for (int g = 0; g < GMAX; ++g)
            if (e0 + g < total) run_group(wa[g], wb[g], sa[g], sb[g], steps[g]);
    }

    MfmaParams pq = p;                          // pooled outputs: a quarter of the rows, corrections per grid
    pq.M = p.M >> 2;
    pq.c0 = p.pool == 2 ? 4 * p.c0 : p.c0;
    if (!live) return;                          // wave-uniform: the ballots below stay whole-wave
    static_for<FN>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const int gn = n0 + 32 * j + lr;
        if (p.pool) {                           // registers 4 k .. 4 k + 3 of a lane are one pooling grid
            static_for<4>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                finish_value(pq, pool4(p.pool, acc[j][4 * k], acc[j][4 * k + 1], acc[j][4 * k + 2], acc[j][4 * k + 3]),
                             (m0 + 8 * k + 4 * lh) >> 2, gn, sc[j], bi[j], false, 0u, lr, lh);
            });
        } else {
            static_for<4>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                const float v4[4] = {acc[j][4 * k], acc[j][4 * k + 1], acc[j][4 * k + 2], acc[j][4 * k + 3]};
                finish_rows8(p, v4, m0 + 8 * k, gn, sc[j], bi[j], pre_res[j][k], lane, lr, lh);
            });
        }
    });
}

// One plane of features with two of weights is held to the 128 registers of four waves per SIMD, which it exceeds by a few;
// the forms with one plane of weights stay within them, the others are far above.  64 x 56 x 56, 192 -> 64 channels, 1 x 1,
// w2a1: 16.4 us with three waves, 14.1 with four and two registers kept in memory.
template <int KA, int KB, int VW, int FN>
__global__ __launch_bounds__(256, (KA == OPK_U1 && KB == OPK_U2 ? 4 : 1)) void mfma_small_wide_kernel(const MfmaParams p)
{
    mfma_small_wide_body<KA, KB, VW, 2, FN>(p, blockIdx.x);
}

}  // namespace apnn
