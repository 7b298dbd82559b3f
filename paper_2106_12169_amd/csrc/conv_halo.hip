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

// Time (us) of a layer in one of the forms of its blocks, as fitted to 500 layers each measured in all of them (the mean error is 12 %;
// what it chooses is on average 1.4 % slower than the fastest form).  A compute unit works on `resident` blocks in a round, the last
// round's fewer ones share it with nobody.  A round costs its blocks' first loads (less where a block walks: the next tile's pixels are
// in flight), 0.43 for each pair of output tiles of a wave, 0.11 for a thousand words of pixels, and for each matrix instruction 0.022 on
// a SIMD with several waves, 0.041 with a lone one that has four and more to a step, 0.061 with two; a little more where the pixels
// are staged as bits.
static double tiling_cost(int fp, int pairs, int64_t tiles, int64_t resident, bool walks, double words, int64_t entries, bool packed)
{
    const double products = fp == 4 ? 8.0 : fp == 1 ? 2.0 : 4.0, lone = (products >= 4 ? 0.041 : 0.061) + (packed ? 0.005 : 0.0), shared = packed ? 0.029 : 0.0224;
    auto cost = [&](int64_t blocks) {
        const double waves = static_cast<double>(blocks * pairs);
        return (walks ? 1.2 : 3.6) + waves * 0.43 * (fp >= 3 ? products / 2 : products) + 0.11e-3 * blocks * words +
               (waves > 1 ? shared * waves : lone) * products * entries;
    };
    const int64_t round = 256 * resident, rest = tiles % round;
    return static_cast<double>(tiles / round) * cost(resident) + (rest ? cost(ceil_div(rest, 256)) : 0.0);
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
    p.digits = divisor(p.DA); p.halves = divisor(p.half); p.columns = divisor(p.S);
    p.pm1 = kindB == OPK_PM1;
    p.pool = mp.pool;
    p.steps = static_cast<int>(steps);
    p.scale = mp.scale; p.bias = mp.bias; p.res = mp.res; p.q_res = mp.q_res; p.res_scale = mp.res_scale;
    p.out = mp.out; p.q_out = mp.q_out; p.NW = mp.NW; p.Y = mp.Y;
    // a two-plane digit enters as half its value; planes are made of a quarter of the result
    p.scaleA = static_cast<int>(0x01010101u * (0x7fu + (kindA == OPK_U2 ? 1u : 0u) - (planes ? 2u : 0u)));
    p.scaleB = static_cast<int>(0x01010101u * (0x7fu + (kindB == OPK_PM1 ? 0u : 1u)));

    // words of a pixel staged together (as the launcher instantiates them)
    const int sw = p.Cw % 4 == 0 ? 4 : p.Cw % 2 == 0 ? 2 : 1;

    // Weights of up to kHaloStay steps stay in LDS while a block walks over its tiles; longer ones pass through in chunks.
    const bool multi = p.DA > 1 || p.DB > 1;
    const bool stay = p.DB == 1 && round_up(steps, 2) <= kHaloStay;
    auto padded = [&](int fp, bool packed) { return round_up(steps, halo_granule(fp == 3 ? 4 : fp, fp == 3 ? 1 : 2, stay && packed)); };
    if (!stay && p.half > kHaloChunk) return false;

    struct Tiling { bool packed; int64_t tilesM, padded, plane, records, table, codes, lds, blocks, buffers; bool walks; };     // blocks: that a compute unit holds
    // fp: pixel tiles of a wave; pooled 4 with both channel tiles, 3 with one; pairs: of channel tiles; packed: features are staged as
    // bits, not as codes
    auto tiling = [&](int fp, int pairs, bool packed) {
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
        // (with four words a lane an odd number of positions: those that neighbouring lanes write fall on different banks)
        t.plane = halo_words(kindA, packed) * ((reach < images * Hq * Wq ? reach : images * Hq * Wq) | (sw == 4 ? 1 : 0));
        t.packed = packed;
        t.records = t.plane * 2 * p.half * p.DA;
        t.padded = padded(fp, packed);
        t.table = round_up((t.padded * p.DA + 5 * halo_granule(fp == 3 ? 4 : fp, fp == 3 ? 1 : 2, stay && packed)) * (multi ? 2 : 1), 4);
        t.codes = (stay ? t.padded : 2 * kHaloChunk) * 512 * pairs + t.table;
        const int64_t most = pairs == 2 ? 1 : fp == 4 ? 2 : fp == 1 && (stay ? packed : !multi) ? 4 : 3;    // by registers: waves a SIMD holds
        // LDS is given out in granules of 1280 bytes, 128 to a compute unit: three blocks of 42 are resident together, of 43 (53.8 to 54.6 KB,
        // three times that is below 160 KB) two, and a grid of walking blocks for three then takes a second turn (168 x 11 x 74,
        // 128 -> 192 channels, 3 x 3, one buffer of bits: 30.5 us, 23.6 with two).
        auto fit = [&](int64_t buffers) {
            t.buffers = buffers;
            t.lds = 4 * (128 * pairs + t.codes + buffers * t.records);
            const int64_t held = 128 / ceil_div(t.lds, 1280);
            t.blocks = held < most ? held : most;
        };
        fit(1);
        // blocks that have a second tile walk, with a second buffer of records where as many of them fit
        const int64_t columns = ceil_div(mp.N, 64 * pairs), single = t.blocks;
        t.walks = stay && t.tilesM * columns > 256 * t.blocks / columns * columns && 256 * t.blocks >= columns;
        if (t.walks) {
            fit(2);
            if (t.blocks < (force == 1 || force == 2 ? 1 : single) || 256 * t.blocks < columns) fit(1);
        }
        return t;
    };
    int fp = mp.pool ? 3 : 1, pairs = 1;
    Tiling t{};
    double best = 0.0;
    for (int i = 0; i < 4; ++i) {
        const int f = (mp.pool ? 3 : 1) + (i & 1), n = 1 + (i >> 1);
        if (force > 0 && force != i + 1 && !(n == 1 && (force == 5 + (i & 1) || force == 7 + (i & 1)))) continue;
        if (n == 2 && (sw != 4 || multi || mp.N <= 64)) continue;
        for (const bool packed : {false, true}) {
            if (packed ? n == 2 || force > 6 : multi || force == 5 || force == 6) continue;
            const Tiling c = tiling(f, n, packed);
            if (c.blocks < 1) continue;
            const double cost = tiling_cost(f, n, c.tilesM * ceil_div(mp.N, 64 * n), c.blocks, c.walks, 4.0 / halo_words(kindA, packed) * c.records, steps * p.DA * p.DB, packed);
            if (t.blocks > 0 && cost >= best) continue;
            best = cost; t = c; fp = f; pairs = n;
        }
    }
    if (t.blocks < 1) return false;
    if (force < 0 && small_tiles <= 4096) {
        // rounds of the blocks that the model was fitted to: the smaller tiles, chunks of whole taps, features as bits in records of an
        // odd number of granules
        const Tiling small = tiling(mp.pool ? 3 : 1, 1, true);
        const int64_t codes = (stay ? steps : 2 * (kHaloChunk / p.half * p.half)) * 512, most = mp.pool ? 3 : 4;
        const int64_t hw = sw == 4 ? 2 : 1, granules = p.DA * 2 * (p.half / hw);
        const int64_t records = small.plane / halo_words(kindA, true) * (kindA == OPK_U1 ? 1 : 2) * hw * (granules | 1);
        auto resident = [&](int64_t buffers) {
            const int64_t n = 160 * 1024 / (4 * (128 + codes + buffers * records));
            return n < most ? n : most;
        };
        const int64_t one = resident(1), two = resident(2);
        if (one < 1) return false;
        const bool walks = stay && small.tilesM * tilesN > 256 * one / tilesN * tilesN && two >= (one < 2 ? one : 2) && 256 * two >= tilesN;
        if (!worth_staging(mp, small_tiles, blocks, steps, stay, walks ? 1 : ceil_div(blocks, 256 * one))) return false;
    }
    const int columns = static_cast<int>(ceil_div(mp.N, 64 * pairs));
    const int64_t tiles = t.tilesM * columns;
    if (tiles > kMaxBlocks) return false;
    // Beyond 4096 tiles of 32 x 32: not where staging a tile's pixels is most of the work and little else of the compute unit runs
    // meanwhile.  Matrix instructions of 32 x 32 x 64 for 1000 staged words, and the time relative to the other kernels, on average
    // over 4900 layers: blocks with one tile, one block to a compute unit 2.1 up to 1.4, 1.2 up to 2.8, 1.1 up to 5.7 (level from 4.5 on),
    // 0.8 up to 11, 0.6 to 0.7 beyond; two blocks 1.3 up to 1.4, 0.75 beyond; three 1.0 up to 1.4, four 0.8; blocks that walk, one 1.8 up to 1.4, 0.9
    // beyond, two and more 0.6 (72 x 72, 288 -> 320 channels, 1 x 1, stride 2, pooled, batch 74: 98.6 us and 29.9).
    if (force < 0 && small_tiles > 4096) {
        const double work = static_cast<double>(steps) * mp.DA * mp.DB * (fp == 3 ? 256 : 128 * fp) / 64, words = 2e-3 * t.records / halo_words(kindA, t.packed);
        const int64_t groups = t.blocks * pairs;                 // of four waves (128 x 28 x 28, 128 -> 256, 1 x 1, stride 2: 9.3 us, 6.7 in one of eight)
        const double least = t.walks ? (groups == 1 ? 2.0 : 0.0) : groups == 1 ? 4.5 : groups == 2 ? 1.5 : 0.0;
        if (work < least * words) return false;
    }
    int64_t grid = tiles;
    if (t.walks) grid = 256 * t.blocks / columns * columns;           // whole rows of channel tiles
    p.tilesM = static_cast<int>(t.tilesM);
    p.per_column = divisor(columns);
    p.packed = t.packed;
    p.pieces = p.DA * static_cast<int>(ceil_div(2 * p.half, sw));
    while ((1 << p.share) < p.pieces) ++p.share;
    p.pairs = pairs; p.buffers = static_cast<int>(t.buffers);
    p.plane = static_cast<int>(t.plane);
    p.padded = static_cast<int>(t.padded);
    for (int e = 0; e < 4; ++e) {
        const int64_t st = e / p.DA, d = e % p.DA, tap = st / p.half, r = tap / p.S;
        if (st >= steps) break;                            // (zero offsets; codes of a step that fills up a granule)
        p.first[e] = static_cast<uint32_t>(4 * halo_words(kindA, t.packed) * (r * p.Wq + tap - r * p.S) + 4 * (st - tap * p.half + d * 2 * p.half) * t.plane);
    }
    for (int e = 0; multi && e < 4; ++e) p.first_codes[e] = static_cast<uint32_t>(1024 * 2 * (e / p.DA < t.padded ? e / p.DA : t.padded - 1) + e % p.DA);
    p.words_table = static_cast<int>(t.table);
    p.words_codes = static_cast<int>(t.codes);
    p.tile_step = static_cast<int>(grid / columns);
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
