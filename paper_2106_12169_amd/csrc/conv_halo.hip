// Host side of conv_halo_kernel: which layers it takes and how they are laid out in LDS.
#include "conv_halo_launch.h"

#include "common.h"
#include "mfma_launch.h"

namespace apnn {

// Up to 4096 tiles of 32 x 32 outputs: few or short sums on few pixels are better off with the kernels that split K over more waves
// and start sooner.  Both sides' times (us), as fitted to 16000 layers of 64 tiles and more, each measured in every form in a
// replayed graph:
//   those kernels: 2.95, and for 1000 tiles 1.5, for each pair of K words and pair of digits 0.11, 0.095, 0.125 where the channel
//     words are a multiple of four, even, odd (a little over half of it with features of one plane, a tenth more with weights of
//     several where the words are not odd), 0.05 more for odd ones from the fortieth pair on, 0.75 with a residual; 1.3 times
//     that with several digits
//   this one: 4.4, and for each of its entries (steps times pairs of digits) 0.08 where the channel words are a multiple of four,
//     else 0.125; 0.03 more where the weights pass through in chunks; 1.6 times that with pooling (a block has as many pixels
//     before it); 0.065 for each channel word and digit of the pixels that a stride skips; all that again for each further round
//     of blocks that do not fit the compute units together; beyond 256 blocks, 1 + 0.07 entries for as many more; 0.75 for 256
//     blocks of int32 results
// What the rule chooses is on average 0.6 % slower than the faster side (1.2 % with a rule that knew no rounds and one time an entry),
// and 1 % of the layers are 5 % and more slower than without this form (4 % with that rule, up to 1.7 times).  E.g. 9 steps on 8 x
// 56 x 56, 64 channels 6.3 there and 4.9 here; 4 x 56 x 56 4.6, 4.8; 18 on 8 x 28 x 28, 128 channels 5.3 and 5.3, with a residual
// 5.8, 5.5; 9 on 8 x 28 x 28, 64 -> 128 channels 4.6, 4.9; 36 on 4 x 28 x 28, 256 channels 8.3, 7.4.
static bool worth_staging(const MfmaParams &mp, int64_t tiles, int64_t blocks, int64_t steps, bool stay, int64_t rounds)
{
    const bool fours = mp.Cw % 4 == 0, odd = mp.Cw % 2 != 0;
    const double pairs = static_cast<double>(mp.DA) * mp.DB, entries = steps * pairs, words = 0.5 * mp.Kw * pairs;
    const double word = (odd ? 0.125 : fours ? 0.11 : 0.095) * (mp.PA == 1 ? 0.56 : 1.0) * (mp.PB > 1 && !odd ? 1.1 : 1.0);
    const double tile = 1.5 + word * words + (odd && words > 40 ? 0.05 * (words - 40) : 0.0) + (mp.res ? 0.75 : 0.0);
    const double other = 2.95 + 1e-3 * tiles * tile * (pairs > 1 ? 1.3 : 1.0);
    const double spread = 0.065 * (static_cast<double>(mp.stride) * mp.stride - 1) * mp.DA * mp.Cw;
    double each = (fours ? 0.08 : 0.125) + (stay ? 0.0 : 0.03);
    double staged = 4.4 + (mp.Y ? 0.75 / 256 * blocks : 0.0);
    if (mp.pool) each *= 1.6;
    else if (blocks > 256) staged += (blocks / 256.0 - 1.0) * (1.0 + 0.07 * entries);
    return staged + rounds * (spread + each * entries) <= other;
}

bool launch_conv_halo(const MfmaParams &mp, int64_t images, int kindA, int kindB, int force, hipStream_t st)
{
    // int32 results alone, or planes of one or two bits alone (the epilogue keeps no other output)
    const bool ints = mp.Y && !mp.scale && !mp.T && !mp.pool && mp.N % 4 == 0;
    const bool planes = mp.out && !mp.Y && !mp.T && mp.q_out <= 2 && (!mp.res || mp.q_res <= 2);
    if (!ints && !planes) return false;
    const int tilesN = static_cast<int>(ceil_div(mp.N, 64));
    // The chip wants most of its compute units busy: not below 96 tiles of 64 x 128 outputs (128 where the stride spreads the pixels).
    const int64_t blocks = ceil_div(mp.M, mp.pool ? 256 : 128) * tilesN;             // of the smaller tiles
    if (force < 0 && blocks < (mp.stride > 1 ? 128 : 96)) return false;
    // int32 results of one or two steps: their store is all there is (192 channels, 10.3 and 10.6).  Beyond 4096 tiles of 32 x 32
    // the other side has 32 x 64 tiles for every 64 channels, and is ahead for 1 x 1 layers: on average 1.15 times as fast.
    const int64_t small_tiles = ceil_div(mp.M, 32) * ceil_div(mp.N, 32), steps = static_cast<int64_t>(mp.R) * mp.S * ((mp.Cw + 1) / 2);
    if (force < 0 && mp.Y && (steps <= 2 || (small_tiles > 4096 && mp.N % 64 == 0 && mp.R == 1 && mp.S == 1))) return false;
    const int64_t Hq = mp.H + 2 * static_cast<int64_t>(mp.pad), Wq = mp.W + 2 * static_cast<int64_t>(mp.pad);
    const int64_t Kw = static_cast<int64_t>(mp.R) * mp.S * mp.Cw, lim = int64_t(1) << 31;
    // (in 64 bits from the first factor on: four times the channels alone can pass 2^31)
    const int64_t bytesA = 4 * images * mp.H * mp.W * mp.PA * mp.Cw, bytesB = 4 * Kw * mp.PB * mp.N;
    if (Hq >= lim || Wq >= lim || Hq * Wq > (lim - 1) / (images + 1) || bytesA >= lim || bytesB >= lim) return false;
    if (mp.M > lim - 1024) return false;

    ConvHaloParams p{};
    p.A = mp.A; p.B = mp.B;
    p.bytesA = static_cast<uint32_t>(bytesA);
    p.bytesB = static_cast<uint32_t>(bytesB);
    p.M = mp.M; p.N = mp.N;
    p.images = static_cast<int>(images); p.H = mp.H; p.W = mp.W;
    p.Hq = static_cast<int>(Hq); p.Wq = static_cast<int>(Wq);
    const int64_t rows = mp.pool ? mp.Hp : mp.Ho, cols = mp.pool ? mp.Wp : mp.Wo;
    p.per_image = divisor(rows * cols); p.per_row = divisor(cols);
    p.frame = divisor(Hq * Wq); p.line = divisor(Wq);
    p.stride = mp.stride; p.pad = mp.pad; p.R = mp.R; p.S = mp.S;
    p.Cw = mp.Cw; p.half = (mp.Cw + 1) / 2;
    p.PA = mp.PA; p.PB = mp.PB; p.DA = mp.DA; p.DB = mp.DB;
    p.digits = divisor(p.DA); p.halves = divisor(p.half);
    p.pm1 = kindB == OPK_PM1;
    p.pool = mp.pool;
    p.steps = static_cast<int>(steps);
    p.scale = mp.scale; p.bias = mp.bias; p.res = mp.res; p.q_res = mp.q_res; p.res_scale = mp.res_scale;
    p.out = mp.out; p.q_out = mp.q_out; p.NW = mp.NW; p.Y = mp.Y;
    // a two-plane digit enters as half its value; planes are made of a quarter of the result
    p.scaleA = static_cast<int>(0x01010101u * (0x7fu + (kindA == OPK_U2 ? 1u : 0u) - (planes ? 2u : 0u)));
    p.scaleB = static_cast<int>(0x01010101u * (0x7fu + (kindB == OPK_PM1 ? 0u : 1u)));

    // steps read together, words staged together (as the launcher instantiates them)
    const int hw = p.Cw % 4 == 0 ? 2 : 1, sw = p.Cw % 4 == 0 ? 4 : p.Cw % 2 == 0 ? 2 : 1, granule = (kindA == OPK_U1 ? 1 : 2) * hw;
    // records are an odd number of granules apart: a step's reads of consecutive pixels hit all banks
    const int granules = p.DA * 2 * (p.half / hw);
    p.rec = granule * (granules % 2 == 0 ? granules + 1 : granules);
    p.pieces = p.DA * static_cast<int>(ceil_div(2 * p.half, sw));
    while ((1 << p.share) < p.pieces) ++p.share;

    // Weights of up to kHaloStay steps stay in LDS while a block walks over its tiles; longer ones pass through in chunks of
    // whole taps.
    const bool stay = p.DB == 1 && p.steps <= kHaloStay;
    if (!stay && p.half > kHaloChunk) return false;
    p.chunk = stay ? p.steps : kHaloChunk / p.half * p.half;
    const int64_t codes = (stay ? 1 : 2) * p.chunk * 512;

    struct Tiling { int64_t tilesM, records, lds, blocks, buffers; };     // blocks: that a compute unit holds
    auto tiling = [&](int fp) {                            // fp: pixel tiles of a wave; pooled 4 with both channel tiles, 3 with one
        Tiling t{};
        const int64_t pixels = fp == 3 ? 256 : 128 * fp;
        t.tilesM = ceil_div(mp.M, pixels);
        // the longest range of padded positions a tile touches: row steps and image steps between its first and last pixel
        // (the stride of a single row is beyond its image: there the image step counts)
        const int64_t px = mp.pool ? pixels / 4 : pixels, step = mp.pool ? 2 * mp.stride : mp.stride < Hq ? mp.stride : Hq;
        const int64_t new_rows = (px - 1 + cols - 1) / cols, new_images = (px - 1 + rows * cols - 1) / (rows * cols);
        const int64_t between = Hq - rows * step;          // lines an image has beyond its rows' steps
        const int64_t reach = new_rows * step * Wq + (cols - 1) * (mp.pool ? 2 : 1) * mp.stride + new_images * (between > 0 ? between : 0) * Wq +
                              (mp.pool ? mp.stride * (Wq + 1) : 0) + (mp.R - 1) * Wq + mp.S;
        t.records = (reach < images * Hq * Wq ? reach : images * Hq * Wq) * p.rec;
        const int64_t most = fp == 4 ? 2 : fp == 1 ? 4 : 3;    // by registers: waves a SIMD holds
        auto fit = [&](int64_t buffers) {
            t.buffers = buffers;
            t.lds = 4 * (128 + codes + buffers * t.records);
            t.blocks = 160 * 1024 / t.lds < most ? 160 * 1024 / t.lds : most;
        };
        fit(1);
        // a second buffer of records is for blocks that have a second tile, and two of those to a compute unit
        if (stay && t.tilesM * tilesN > 256 * t.blocks / tilesN * tilesN) {
            const int64_t single = t.blocks;
            fit(2);
            if (t.blocks < (single < 2 ? single : 2) || 256 * t.blocks < tilesN) fit(1);
        }
        return t;
    };
    // 64 x 256 outputs a block, or 64 x 128 (measured, us, 64 x 128 against 64 x 256):
    //   weights that stay: 9 steps on 1568 tiles of 256 17.9, 15.3; 18 steps 23.6, 29.2; 9 steps with stride 2 on 784 13.5, 17.9
    //   chunks: what a compute unit holds of pixels decides; 36 steps on 392 tiles 17.2, 14.7 (512 pixels against 384); 72 steps
    //   on 784 tiles 47, 59 (256 either way)
    // Pooled: 64 x 128 pooled outputs a block (a wave has both channel tiles), or 64 x 64 (one; fewer and smaller blocks fill the
    // chip): 36 steps on 196 of the larger tiles 12.4, 18.0; 72 on 104 20.1, 16.0; 36 on 98 12, 9.9; 9 on 784 21.5, 20.9.
    int fp = mp.pool ? 3 : 1;
    Tiling t = tiling(fp);
    if (t.blocks < 1) return false;
    if (force < 0 && small_tiles <= 4096 && !worth_staging(mp, small_tiles, blocks, steps, stay, t.buffers == 2 ? 1 : ceil_div(blocks, 256 * t.blocks)))
        return false;
    if (mp.pool) {
        const Tiling four = tiling(4);
        if (force != 1 && (force == 2 || four.tilesM * tilesN >= 150) && four.blocks >= 1) { fp = 4; t = four; }
    } else {
        const Tiling two = tiling(2);
        fp = force == 1 || force == 2 ? force
             : stay ? (p.steps <= 12 && mp.stride == 1 && two.blocks > 0 && two.tilesM * tilesN >= 256 ? 2 : 1)
                    : (2 * two.blocks > t.blocks && two.tilesM * tilesN >= 192 ? 2 : 1);
        if (fp == 2) t = two;
    }
    const int64_t tiles = t.tilesM * tilesN;
    if (t.blocks < 1 || tiles > kMaxBlocks) return false;
    // Beyond 4096 tiles of 32 x 32: not where staging a tile's pixels is most of the work and little else of the compute unit runs
    // meanwhile.  Matrix instructions of 32 x 32 x 64 for 1000 staged words, and the time relative to the other kernels, on average
    // over 4900 layers: blocks with one tile, one block to a compute unit 2.1 up to 1.4, 1.2 up to 2.8, 1.1 up to 5.7 (level from 4.5 on),
    // 0.8 up to 11, 0.6 to 0.7 beyond; two blocks 1.3 up to 1.4, 0.75 beyond; three 1.0 up to 1.4, four 0.8; blocks that walk, one 1.8 up to 1.4, 0.9
    // beyond, two and more 0.6 (72 x 72, 288 -> 320 channels, 1 x 1, stride 2, pooled, batch 74: 98.6 us and 29.9).
    if (force < 0 && small_tiles > 4096) {
        const double work = static_cast<double>(steps) * mp.DA * mp.DB * (fp == 3 ? 256 : 128 * fp) / 64, words = 1e-3 * t.records;
        const double least = t.buffers == 2 ? (t.blocks == 1 ? 2.0 : 0.0) : t.blocks == 1 ? 4.5 : t.blocks == 2 ? 1.5 : 0.0;
        if (work < least * words) return false;
    }
    int64_t grid = tiles;
    if (t.buffers == 2) grid = 256 * t.blocks / tilesN * tilesN;           // whole rows of channel tiles
    p.tilesM = static_cast<int>(t.tilesM);
    p.per_column = divisor(tilesN);
    p.words_codes = static_cast<int>(codes);
    p.tile_step = static_cast<int>(grid / tilesN);
    p.words_records = static_cast<int>(t.records);
    const unsigned g = static_cast<unsigned>(grid);
    const int bytes = static_cast<int>(t.lds);
    switch (kindA) {
        case OPK_U1: return launch_conv_halo_u1(p, stay, fp, g, bytes, st);
        case OPK_U2: return launch_conv_halo_u2(p, stay, fp, g, bytes, st);
        default: return launch_conv_halo_pm1(p, stay, fp, g, bytes, st);
    }
}

}  // namespace apnn
