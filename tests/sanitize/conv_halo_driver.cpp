// launch_conv_halo (conv_halo.hip), the host side of the staged convolutions, under -fsanitize=address,undefined: which layers
// it takes and the layout it asks for.  The launchers of the kernel's instances are the stand-ins below.
#include <cstdint>
#include <cstdio>

#include "../../paper_2106_12169_amd/csrc/conv_halo_launch.h"

namespace apnn {
static ConvHaloParams g_p;
static bool g_stay;
static int g_fp, g_lds, g_kind;
static unsigned g_grid;
static bool took(int kind, const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds)
{
    g_kind = kind; g_p = p; g_stay = stay; g_fp = fp; g_grid = grid; g_lds = lds;
    return true;
}
bool launch_conv_halo_u1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t) { return took(OPK_U1, p, stay, fp, grid, lds); }
bool launch_conv_halo_u2(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t) { return took(OPK_U2, p, stay, fp, grid, lds); }
bool launch_conv_halo_pm1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t) { return took(OPK_PM1Z, p, stay, fp, grid, lds); }
bool launch_conv_halo(const MfmaParams &mp, int64_t images, int kindA, int kindB, int force, hipStream_t st);
}  // namespace apnn

using namespace apnn;

static int failures = 0;
#define EXPECT(cond) do { if (!(cond)) { std::printf("line %d: %s\n", __LINE__, #cond); ++failures; } } while (0)

struct Layer {
    int64_t images, H, W, Cin, Cout;
    int R, S, stride, pad;
    bool pm1_weights;
    int p;
    bool pm1_features;
    int q;
    int pool = 0;
    bool ints = false;
    int q_out = 2, q_res = 0;
};

// as apnn_layer's dispatch fills the parameters in
static bool staged(const Layer &l, int force)
{
    MfmaParams mp{};
    const int64_t Ho = (l.H + 2 * int64_t(l.pad) - l.R) / l.stride + 1, Wo = (l.W + 2 * int64_t(l.pad) - l.S) / l.stride + 1;
    mp.H = static_cast<int>(l.H); mp.W = static_cast<int>(l.W); mp.Ho = static_cast<int>(Ho); mp.Wo = static_cast<int>(Wo);
    mp.Hp = mp.Ho / 2; mp.Wp = mp.Wo / 2;
    mp.M = static_cast<int>(l.pool ? l.images * mp.Hp * mp.Wp * 4 : l.images * Ho * Wo);
    mp.N = static_cast<int>(l.Cout); mp.NW = mp.N / 32;
    mp.R = l.R; mp.S = l.S; mp.stride = l.stride; mp.pad = l.pad; mp.pool = l.pool;
    mp.Cw = static_cast<int>(l.Cin / 32); mp.Kw = mp.Cw * l.R * l.S;
    mp.PA = l.q; mp.PB = l.p;
    mp.DA = (l.q + 1) / 2; mp.DB = (l.p + 1) / 2;
    alignas(16) static uint32_t there[4];                        // (addresses are passed on, never followed)
    if (l.ints) {
        mp.Y = reinterpret_cast<int32_t *>(there);
    } else {
        mp.out = there; mp.q_out = l.q_out;
        if (l.q_res) { mp.res = there; mp.q_res = l.q_res; }
        mp.scale = mp.bias = reinterpret_cast<const float *>(there);
    }
    g_kind = -1;
    return launch_conv_halo(mp, l.images, l.pm1_features ? OPK_PM1Z : l.q == 1 ? OPK_U1 : OPK_U2,
                            l.pm1_weights ? OPK_PM1 : l.p == 1 ? OPK_U1 : OPK_U2, force, nullptr);
}

// Layers from a file, a line each: the fields of Layer, then the override.  Of each: whether it is staged, and how.
static int layouts(const char *file)
{
    std::FILE *const f = std::fopen(file, "r");
    if (!f) return 2;
    Layer l{};
    int pm1w, pm1f, ints, force;
    while (std::fscanf(f, "%ld %ld %ld %ld %ld %d %d %d %d %d %d %d %d %d %d %d %d %d", &l.images, &l.H, &l.W, &l.Cin, &l.Cout, &l.R, &l.S, &l.stride, &l.pad,
                       &pm1w, &l.p, &pm1f, &l.q, &l.pool, &ints, &l.q_out, &l.q_res, &force) == 18) {
        l.pm1_weights = pm1w; l.pm1_features = pm1f; l.ints = ints;
        if (!staged(l, force)) std::printf("0\n");
        else std::printf("1 kind %d stay %d fp %d pairs %d packed %d three %d buffers %d tilesM %d step %d grid %u lds %d records %d steps %d\n", g_kind, g_stay, g_fp, g_p.pairs,
                         g_p.packed, g_p.three, g_p.buffers, g_p.tilesM, g_p.tile_step, g_grid, g_lds, g_p.words_records, g_p.steps);
    }
    std::fclose(f);
    return 0;
}

int main(int argc, char **argv)
{
    if (argc > 1) return layouts(argv[1]);

    // weights of 2^31 bytes and more are not for 31-bit offsets, whatever their size is modulo 2^32
    const int64_t most = (int64_t(1) << 31) / 8 - 64;            // channels of one 64-channel plane: 8 bytes each
    EXPECT(staged({1, 8, 8, 64, most, 1, 1, 1, 0, true, 1, false, 2}, 1) && g_p.bytesB == 8u * static_cast<uint32_t>(most));
    for (int64_t channels : {most + 64, int64_t(1) << 29, (int64_t(1) << 29) + 64, int64_t(1) << 30})
        EXPECT(!staged({1, 8, 8, 64, channels, 1, 1, 1, 0, true, 1, false, 2}, 1));
    EXPECT(!staged({1, 8, 8, 64, int64_t(1) << 26, 1, 1, 1, 0, false, 8, false, 2}, 1));      // 4 GiB: 0 in 32 bits
    EXPECT(!staged({1, 8, 8, 64, int64_t(1) << 27, 1, 1, 1, 0, false, 4, false, 2}, 1));
    EXPECT(!staged({1, 8, 8, 64, int64_t(1) << 28, 1, 1, 1, 0, false, 2, false, 2}, 1));
    EXPECT(!staged({1, 8, 8, 32, 536870848, 1, 1, 1, 0, false, 3, false, 2}, 1));             // 6442450176: 2147482880

    // frames and strides near 2^30, of which few outputs are left: no size of them wraps
    EXPECT(!staged({8, 8, 8, 64, 64, 3, 3, 1 << 29, 1 << 29, true, 1, false, 2}, 1));          // 9 * 2^60 positions
    EXPECT(!staged({100, 1, 1, 64, 64, 1, 1, 1 << 29, 536870911, true, 1, false, 2}, 1));
    EXPECT(!staged({1, 1, 1 << 28, 32, 64, 1, 1, 2147483647, 0, true, 1, false, 1}, 1));       // 127 strides of 2^28 positions
    EXPECT(!staged({3, 1, 1 << 20, 32, 64, 1, 1, 2147483647, 0, true, 1, false, 1}, 1));
    EXPECT(staged({300, 1, 1, 32, 64, 1, 1, 2147483647, 0, true, 1, false, 1}, 1) && g_p.words_records == 2 * g_p.plane);
    EXPECT(g_p.plane == halo_words(OPK_U1, g_p.packed) * 128);                                // 128 positions of 300 frames

    // block scales: biased exponents in every byte, those of 0/1 weights and of int32 results from 2^7 up
    EXPECT(staged({1, 8, 8, 64, 64, 3, 3, 1, 1, true, 1, false, 2}, 1) && g_p.scaleA == 0x7e7e7e7e && g_p.scaleB == 0x7f7f7f7f);
    EXPECT(staged({4, 27, 31, 96, 160, 3, 3, 1, 1, false, 2, false, 4, 0, true}, 1));
    EXPECT(static_cast<uint32_t>(g_p.scaleA) == 0x80808080u && static_cast<uint32_t>(g_p.scaleB) == 0x80808080u);
    EXPECT(staged({1, 8, 8, 64, 64, 3, 3, 1, 1, false, 1, true, 1}, 1) && g_p.scaleA == 0x7d7d7d7d && static_cast<uint32_t>(g_p.scaleB) == 0x80808080u);

    // blocks that walk over tiles, two buffers of pixels each: the layers of test_blocks_walk_over_tiles (tests/test_gpu_conv_halo.py)
    // give every block a second tile and some a third, the last one ragged
    struct { Layer l; int force, fp, pixels; } const walked[] = {
        {{2, 112, 111, 32, 512, 3, 3, 1, 1, true, 1, false, 2}, 1, 1, 128},    {{2, 157, 158, 64, 480, 1, 1, 1, 0, true, 1, false, 2}, 2, 2, 256},
        {{3, 105, 105, 32, 512, 1, 1, 1, 0, false, 1, false, 1}, 1, 1, 128},   {{3, 104, 105, 32, 512, 2, 1, 1, 1, true, 1, true, 1}, 1, 1, 128},
        {{3, 105, 105, 64, 512, 1, 1, 1, 0, true, 1, false, 3}, 1, 1, 128},    {{1, 550, 551, 32, 64, 1, 1, 1, 0, true, 1, false, 2}, 1, 1, 128},
        {{2, 158, 159, 32, 512, 1, 1, 1, 0, true, 1, false, 2, 1}, 1, 3, 256}, {{2, 183, 183, 32, 512, 1, 1, 1, 0, true, 1, false, 2, 2}, 2, 4, 512}};
    for (const auto &w : walked) {
        EXPECT(staged(w.l, w.force) && g_stay && g_fp == w.fp && g_p.tilesM > 2 * g_p.tile_step && g_p.M % w.pixels != 0);
        EXPECT(g_grid == static_cast<unsigned>(g_p.tile_step * g_p.per_column.d) && g_grid % 256 == 0);
        EXPECT(g_lds == 4 * (128 + g_p.words_codes + 2 * g_p.words_records));
    }

    // blocks that walk are as many as are resident: a compute unit has 128 granules of 1280 bytes of LDS
    EXPECT(staged({168, 11, 74, 128, 192, 3, 3, 1, 1, true, 1, false, 2}, 5) && g_p.packed && g_grid == 510);
    for (int frame = 8; frame <= 200; ++frame)
        for (int Cin : {32, 96, 128, 192})
            for (int force = 1; force <= 8; ++force)
                if (staged({24, frame, frame + 3, Cin, 192, 3, 3, 1, 1, true, 1, false, 2}, force) && g_stay && g_p.tile_step < g_p.tilesM)
                    EXPECT(static_cast<int>(g_grid + 255) / 256 * ((g_lds + 1279) / 1280) <= 128);

    // blocks that walk with one buffer wait for each tile's pixels: not where these are most of the work (224 x 38 x 44, 192 -> 192 channels,
    // 1 x 1, pooled 15.8 us there, 20.8 here), but as soon as there are sums to hide (3 x 3, 128 -> 192, int32 33 there, 24 here)
    EXPECT(!staged({224, 38, 44, 192, 192, 1, 1, 2, 0, true, 1, true, 1, 1}, -1));
    EXPECT(staged({224, 38, 44, 192, 192, 1, 1, 2, 0, true, 1, true, 1, 1}, 5) && g_p.buffers == 1 && g_p.tile_step < g_p.tilesM);
    EXPECT(staged({168, 11, 74, 128, 192, 3, 3, 1, 1, true, 1, false, 2, 0, true}, -1));

    // the offsets that come with the launch are the first ones of the table that the kernel makes: an entry is a step and a digit of the
    // features, one beyond the last step starts over, on the codes of the step that fills a granule up (if there is one)
    for (int Cin : {32, 64, 96, 160, 512})
        for (int R = 1; R <= 3; R += 2)
            for (int q = 1; q <= 5; ++q)
                for (int weights = 1; weights <= 3; weights += 2)
                    for (int force = 1; force <= 8; ++force) {
                        if (!staged({2, 9, 11, Cin, 128, R, R, 1, R / 2, false, weights, false, q}, force)) continue;
                        const bool multi = g_p.DA > 1 || g_p.DB > 1;
                        for (int e = 0; e < 4; ++e) {
                            const int st = e / g_p.DA, d = e % g_p.DA, tap = st / g_p.half, cw = st % g_p.half;
                            const int at = (tap / R * g_p.Wq + tap % R) * halo_words(g_kind, g_p.packed) + (cw + 2 * d * g_p.half) * g_p.plane;
                            EXPECT(g_p.first[e] == (st < g_p.steps ? 4u * static_cast<uint32_t>(at) : 0u));
                            if (!multi) EXPECT(g_p.first_codes[e] == 0);
                            else if (st < g_p.padded) EXPECT(g_p.first_codes[e] == 2048u * static_cast<uint32_t>(st) + static_cast<uint32_t>(d));
                        }
                        EXPECT(g_p.padded >= g_p.steps && g_p.padded <= g_p.steps + 1);
                    }

    // a position of one plane takes half the LDS of one of two: wide frames of many channels fit with the one alone
    for (const Layer &l : {Layer{8, 96, 96, 512, 128, 5, 5, 1, 2, true, 1, false, 1}, Layer{8, 192, 192, 512, 128, 3, 3, 1, 1, true, 1, false, 1},
                           Layer{8, 320, 320, 256, 128, 5, 5, 1, 2, true, 1, false, 1}}) {
        EXPECT(staged(l, -1) && g_kind == OPK_U1 && g_p.packed && g_lds <= 160 * 1024);
    }

    // weight planes: one that is there is inside the weights by both offsets, one that is not is beyond them by the lane's own (the load's
    // range check leaves the shared one out)
    for (int planes = 1; planes <= 8; ++planes)
        for (int Kw : {1, 18, 4608}) {
            const uint32_t row = 4u * static_cast<uint32_t>(planes * Kw), bytes = 640u * row;      // of a channel, of all
            for (int plane = 0; plane < 2 * ((planes + 1) / 2); ++plane) {
                const uint32_t at = 639u * row + 4u * static_cast<uint32_t>(Kw - 1);              // the last word of the last channel
                const PlaneOffset o = plane_offset(at, plane, planes, Kw);
                EXPECT(o.shared < bytes);
                if (plane < planes) EXPECT(o.lane == at && o.shared == 4u * static_cast<uint32_t>(plane * Kw) && o.lane + o.shared < bytes);
                else EXPECT(o.lane >= uint32_t(1) << 31);
            }
        }

    if (failures == 0) std::puts("staged convolution sanitizer run ok");
    return failures != 0;
}
