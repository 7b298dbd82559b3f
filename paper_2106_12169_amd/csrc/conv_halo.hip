// Host side of conv_halo_kernel: which layers it takes and how they are laid out in LDS.
#include "conv_halo_launch.h"

#include "common.h"
#include "mfma_launch.h"

namespace apnn {

// Which layers are staged, and in which form: the least of the times (us) that the forms below and the kernels with lane-private
// loads are expected to take.  Both were fitted to 29 600 layers (8 to 20 000 blocks of 64 x 128 outputs, 1 x 1 to 7 x 7, strides 1 and
// 2, up to three planes of weights and four of features, planes and int32 results, each measured in every form in a replayed graph);
// the mean error near the line is 5 and 6 %.  On 7620 other layers what is chosen takes about 1 % more than the fastest of them all (with
// the rules before 3 %, beyond 4096 tiles of 32 x 32 5 %).  By classes: profiles/staged_convolutions_choice.txt.

// The form of a layer's blocks.  fp: pixel tiles of a wave (pooled 4 with both channel tiles of a pair, 3 with one); pairs: of channel
// tiles; packed: features are staged as bits, not as codes; blocks: that a compute unit holds
struct Tiling {
    int fp, pairs;
    bool packed, walks, three;
    int64_t tilesM, columns, padded, plane, records, table, codes, lds, blocks, buffers, grid;
};

// A compute unit works on its resident blocks in rounds.  In one of them
//   the sums read 1.5 operands from LDS for each matrix instruction with one pixel tile a wave, 1 with two, 1.25 and 0.75 pooled, and
//   these reads are most of what an instruction takes: 0.0169 each and 0.00537 on top, nearly twice that on a SIMD with a lone wave;
//   staging passes over the pixels: every thread fetches two pieces (four of one word) and waits, 0.393 a pass, and more for each wave
//   that expands and writes them;
//   weights pass through in chunks, which costs the most where they are loaded word by word (channel words no multiple of four), twice
//   that with two planes;
//   the epilogue takes 0.21 for a 32 x 32 tile of planes, and 0.0334 for each other block that writes into the same lines.
// Where blocks walk, a third of the shorter of the sums and the rest is hidden, by the other waves or by the next tile's pixels being in
// flight; with one buffer and a lone wave nothing is.  A last round that half of the compute units have takes 7 % less, and a lone last
// tile of several blocks that walk 24 %.
static double staged_cost(const MfmaParams &mp, const Tiling &t, int kindA, int64_t steps, bool stay, int sw)
{
    const bool pooled = t.fp >= 3, planes = mp.PB > 1, words = mp.Cw % 4 != 0;       // (weights of two planes, loaded by words)
    const double products = t.fp == 4 ? 8.0 : t.fp == 1 ? 2.0 : 4.0, reads = t.fp == 1 ? 1.5 : t.fp == 2 ? 1.0 : t.fp == 3 ? 1.25 : 0.75;
    const double entries = static_cast<double>(steps) * mp.DA * mp.DB, filled = mp.N / (64.0 * t.pairs * t.columns);
    double outputs = pooled ? 0.0379 + 0.177 * products : (mp.Y ? 0.645 : 0.21) * products;
    if (mp.res) outputs += 0.1 * (pooled ? products / 4 : products);
    outputs *= filled;
    if (!pooled && !mp.Y) outputs += 0.0334 * products * static_cast<double>(t.columns < 8 ? t.columns - 1 : 7);
    int share = 1;                                               // threads that share a position
    while (share < mp.DA * ceil_div(2 * ((mp.Cw + 1) / 2), sw)) share *= 2;
    const double passes = static_cast<double>(ceil_div(t.plane / halo_words(kindA, t.packed) * share, 256 * t.pairs * (sw == 1 ? 4 : 2)));
    const double pass = (sw == 1 ? 0.135 : sw == 2 ? -0.0215 : 0.0215) + (t.packed ? 0.0 : sw == 4 ? 0.0406 : 0.0203) - (mp.PA == 1 ? 0.059 : 0.0);
    const double shared = 0.00537 + 0.0169 * reads + (t.packed ? 0.0016 : 0.0), lone = 0.0302 * reads + (t.packed ? 0.00438 : 0.0);
    const bool two = t.buffers == 2;
    const double resident = static_cast<double>(t.blocks * t.pairs), first = 0.806;                // the first loads of a round
    const double chunk = words ? (planes ? 0.0778 : 0.0428) : planes ? 0.0115 : 0.00859;
    const double fixed = !t.walks ? first + (stay ? 0.0 : (chunk + resident * (planes ? 0.00441 : 0.00145)) * steps * mp.DB)
                       : two ? 0.441 / resident - 0.0695 : 0.474 / resident - 0.304;
    const double weights = stay ? (words ? (planes ? 0.0297 : 0.0163) : planes ? 0.00655 : 0.0) * steps * t.pairs : 0.0;
    auto round = [&](int64_t blocks) {
        const double n = static_cast<double>(blocks), waves = n * t.pairs;
        const double rest = waves * outputs + passes * (0.393 + waves * pass), sums = products * entries * (lone > shared * waves ? lone : shared * waves);
        const double hidden = t.walks && (two || waves > 1) ? 0.631 : 1.0;
        return fixed + (rest > sums ? rest + hidden * sums : sums + hidden * rest) + (t.walks ? 0.0 : n * weights);
    };
    auto last_round = [&](int64_t tiles) {                       // `tiles` blocks, at most one round of them
        const int64_t n = ceil_div(tiles, 256), blocks = n < t.blocks ? n : t.blocks;
        if (t.walks) return round(blocks) * (blocks == 1 && t.blocks > 1 ? 0.758 : 1.0);
        return round(blocks) * (1.0 - 0.137 * (1.0 - tiles / (256.0 * blocks)));
    };
    const int64_t tiles = t.tilesM * t.columns;
    double cost = 3.2;                                          // the launch; 0.2 of it since calls in a row overlap less than those of the others (400 near the line)
    if (t.walks) {
        const int64_t step = t.grid / t.columns, full = ceil_div(t.tilesM, step) - 1;
        cost += full * round(t.blocks) + last_round((t.tilesM - full * step) * t.columns) + (first > fixed ? first - fixed : 0.0) + t.blocks * weights;
    } else {
        const int64_t full = tiles / (256 * t.blocks), rest = tiles % (256 * t.blocks);
        cost += full * round(t.blocks) + (rest ? last_round(rest) : 0.0);
    }
    // int32 results: 1 x 1 layers are 1.12 times as long as that where the other side has tiles of 32 x 64 (605 of them), and beyond the
    // 256 MB that the last cache holds both sides' stores slow down, these more (1 x 1, from 5.0 to 3.9 TB/s, the others from 4.5 to 3.8)
    if (mp.Y && mp.R * mp.S == 1 && mp.N % 64 == 0 && ceil_div(mp.M, 32) * ceil_div(mp.N, 32) > 4096) cost *= 1.12;
    if (mp.Y && static_cast<double>(mp.M) * mp.N > 67108864.0) cost *= 1.14;
    return cost;
}

// The kernels with lane-private loads: so much for a tile of 32 x 32 and for each pair of K words and pair of digits of it, more for
// those from the tenth and the fiftieth on; most of it for whole tiles a compute unit.  Up to 4096 tiles four waves share one; beyond, a
// wave has one, or two of 32 x 32 where the channels are a multiple of 64.
static double private_cost(const MfmaParams &mp, int64_t tiles)
{
    struct Size {
        double launch, chain, whole, tile[3], pair[3], from10[3], from50[3];     // [3]: channel words a multiple of four, even, odd
        double residual, pooled, ints, tile_digits, digits, digits4, one_plane, three_planes, weight_planes, stride;
    };
    static constexpr Size sizes[3] = {
        {3.55, 0.00498, 0.732, {1.17, 1.38, 1.71}, {0.0671, 0.0741, 0.0697}, {0.042, 0.0339, 0.0938}, {-0.00792, 0.0155, 0.022},
         0.374, -0.182, 0.0282, 1.49, 0.952, 0.942, 0.628, 0.886, 1.37, 1.08},
        {4.83, 0.0959, 0.839, {0.625, 0.629, 0.737}, {0.027, 0.0367, 0.0715}, {0.0271, 0.0186, 0.0337}, {0.0328, 0.0447, 0.0292},
         0.493, -0.188, -0.0585, 1.25, 0.877, 0.707, 0.725, 0.916, 2, 1.19},
        {5.14, 0.0291, 0.953, {1.06, 1.3, 1.37}, {0.0546, 0.0665, 0.108}, {0.0356, 0.0449, 0.0492}, {0.0489, 0.0432, 0.0488},
         0.526, -0.278, -0.174, 1.34, 1, 0.876, 0.515, 0.809, 1.46, 1.28}};
    const Size &z = sizes[tiles <= 4096 ? 0 : mp.N % 64 == 0 ? 1 : 2];
    const int words = mp.Cw % 4 == 0 ? 0 : mp.Cw % 2 == 0 ? 1 : 2;
    const int digits = mp.DA * mp.DB;
    const double pairs = 0.5 * mp.Kw * digits;
    double sums = z.pair[words] * pairs + (pairs > 10.0 ? z.from10[words] * (pairs - 10.0) : 0.0) + (pairs > 50.0 ? z.from50[words] * (pairs - 50.0) : 0.0);
    if (mp.PA == 1) sums *= z.one_plane;
    if (mp.PA == 3) sums *= z.three_planes;
    if (mp.PB > 1) sums *= z.weight_planes;
    if (digits > 1) sums *= digits > 2 ? z.digits4 : z.digits;
    if (mp.stride > 1) sums *= z.stride;
    const double tile = z.tile[words] * (digits > 1 ? z.tile_digits : 1.0) + (mp.res ? z.residual : 0.0) + (mp.pool ? z.pooled : 0.0) + (mp.Y ? z.ints : 0.0) + sums;
    const double n = static_cast<double>(tiles), whole = 256.0 * ceil_div(tiles, 256);
    return z.launch + z.chain * pairs + 1e-3 * (n + z.whole * (whole - n)) * tile;
}

bool launch_conv_halo(const MfmaParams &mp, int64_t images, int kindA, int kindB, int force, hipStream_t st)
{
    // int32 results alone, or planes of one or two bits alone (the epilogue keeps no other output)
    const bool ints = mp.Y && !mp.scale && !mp.T && !mp.pool && mp.N % 4 == 0;
    const bool planes = mp.out && !mp.Y && !mp.T && mp.q_out <= 2 && (!mp.res || mp.q_res <= 2);
    if (!ints && !planes) return false;
    // (the times below hold from 64 tiles of 64 x 128 outputs on)
    if (force < 0 && ceil_div(mp.M, mp.pool ? 256 : 128) * ceil_div(mp.N, 64) < 64) return false;
    const int64_t steps = static_cast<int64_t>(mp.R) * mp.S * ((mp.Cw + 1) / 2);
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
    if (!stay && p.half > kHaloChunk) return false;

    auto tiling = [&](int fp, int pairs, bool packed, bool three) {
        Tiling t{};
        const int64_t pixels = fp == 3 ? 256 : 128 * fp;
        t.fp = fp; t.pairs = pairs; t.packed = packed;
        t.columns = ceil_div(mp.N, 64 * pairs);
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
        t.records = t.plane * 2 * p.half * p.DA;
        t.three = three;
        const int granule = halo_granule(fp == 3 ? 4 : fp, fp == 3 ? 1 : 2, stay && packed && !three);
        t.padded = round_up(steps, granule);
        t.table = round_up((t.padded * p.DA + 5 * granule) * (multi ? 2 : 1), 4);
        t.codes = (stay ? t.padded : 2 * kHaloChunk) * 512 * pairs + t.table;
        const int64_t most = pairs == 2 ? 1 : fp == 4 ? 2 : fp == 1 && !three && (stay ? packed : !multi) ? 4 : 3;    // by registers: waves a SIMD holds (eight waves
        // in chunks of 128 pixels take 127: two such blocks can be resident; the times were fitted with one)
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
        // blocks that have a second tile walk, with a second buffer of records where as many of them fit (overrides 1 and 2: where any fits)
        const int64_t single = t.blocks;
        t.walks = stay && t.tilesM * t.columns > 256 * t.blocks / t.columns * t.columns && 256 * t.blocks >= t.columns;
        if (t.walks) {
            fit(2);
            if (t.blocks < (force == 1 || force == 2 ? 1 : single) || 256 * t.blocks < t.columns) fit(1);
        }
        t.grid = t.walks ? 256 * t.blocks / t.columns * t.columns : t.tilesM * t.columns;          // whole rows of channel tiles
        return t;
    };
    Tiling t{};
    double best = 0.0;
    for (int i = 0; i < 4; ++i) {
        const int f = (mp.pool ? 3 : 1) + (i & 1), n = 1 + (i >> 1);
        if (force > 0 && force != i + 1 && !(n == 1 && (force == 5 + (i & 1) || force == 7 + (i & 1)))) continue;
        if (n == 2 && (sw != 4 || multi || mp.N <= 64)) continue;
        for (const bool packed : {false, true}) {
            if (packed ? n == 2 || force > 6 : multi || force == 5 || force == 6) continue;
            Tiling c = tiling(f, n, packed, false);
            if (multi && stay && f == 1 && (c.tilesM * c.columns <= 768 || c.blocks < 4)) {
                const Tiling three = tiling(f, n, packed, true);
                if (three.blocks > 0) c = three;
            }
            if (c.blocks < 1) continue;
            const double cost = staged_cost(mp, c, kindA, steps, stay, sw);
            if (t.blocks > 0 && cost >= best) continue;
            best = cost; t = c;
        }
    }
    if (t.blocks < 1 || t.tilesM * t.columns > kMaxBlocks) return false;
    if (force < 0 && best > private_cost(mp, ceil_div(mp.M, 32) * ceil_div(mp.N, 32))) return false;
    p.tilesM = static_cast<int>(t.tilesM);
    p.per_column = divisor(t.columns);
    p.packed = t.packed; p.three = t.three;
    p.pieces = p.DA * static_cast<int>(ceil_div(2 * p.half, sw));
    while ((1 << p.share) < p.pieces) ++p.share;
    p.pairs = t.pairs; p.buffers = static_cast<int>(t.buffers);
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
    p.tile_step = static_cast<int>(t.grid / t.columns);
    p.words_records = static_cast<int>(t.records);
    const unsigned g = static_cast<unsigned>(t.grid);
    const int bytes = static_cast<int>(t.lds);
    switch (kindA) {
        case OPK_U1: return launch_conv_halo_u1(p, stay, t.fp, g, bytes, st);
        case OPK_U2: return launch_conv_halo_u2(p, stay, t.fp, g, bytes, st);
        default: return launch_conv_halo_pm1(p, stay, t.fp, g, bytes, st);
    }
}

}  // namespace apnn
