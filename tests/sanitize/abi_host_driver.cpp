// Host side of the C-ABI library under -fsanitize=address,undefined: size helpers, the batch-norm fold, the
// override table, the tile choice, every argument check, and the dispatch itself.  The sources with the host logic
// (layer.hip, pack.hip, pool.hip, input_layer.hip, conv_halo.hip, common.cpp) are linked with the stand-ins below in place of the
// kernel-instance launchers, which record what the dispatch asked for and launch nothing; so the whole decision path
// of apnn_gemm / apnn_layer runs without a GPU and its constants can be checked.  Device pointers are fakes that host
// code never dereferences.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/apnn.h"
#include "../../include/apnn_debug.h"
#include "../../paper_2106_12169_amd/csrc/conv_halo_launch.h"
#include "../../paper_2106_12169_amd/csrc/mfma_launch.h"
#include "../../paper_2106_12169_amd/csrc/tile_launch.h"

// ---- stand-ins for the kernel-instance launchers -------------------------------------------------------------
static std::string g_kernel;          // which launcher the last dispatch chose
static apnn::MfmaParams g_mp;
static apnn::TileParams g_tp;
static unsigned g_grid;
static int g_pmz;
static int g_nsplit;                  // waves that split K of a tile of the small-layer kernel
static apnn::ConvHaloParams g_halo;
static int g_fp;                      // its pixel tiles
static bool g_stay;                   // ... and whether its weights stay in LDS

// the launches that the sources make themselves (nothing reaches the runtime)
static unsigned g_block;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t)
{
    g_grid = grid.x; g_block = block.x;
    return hipErrorNoDevice;                                  // not launched
}
static int g_device, g_asked;         // the current device, how often a kernel asked for LDS
static hipError_t g_answer = hipSuccess;
extern "C" hipError_t hipGetDevice(int *device) { *device = g_device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { ++g_asked; return g_answer; }

namespace apnn {
static bool took(const char *name, const MfmaParams &p, unsigned grid) { g_kernel = name; g_mp = p; g_grid = grid; return true; }
bool launch_mfma256(const MfmaParams &p, int, int, bool, unsigned grid, hipStream_t) { return took("mfma256", p, grid); }
bool launch_mfma128(const MfmaParams &p, int, int, bool, unsigned grid, hipStream_t) { return took("mfma128", p, grid); }
bool launch_mfma64(const MfmaParams &p, int, int, bool, unsigned grid, hipStream_t) { return took("mfma64", p, grid); }
bool launch_mfma64_k8(const MfmaParams &p, int, int, unsigned grid, hipStream_t) { return took("mfma64_k8", p, grid); }
bool launch_mfma32(const MfmaParams &p, int, int, bool, unsigned grid, hipStream_t) { return took("mfma32", p, grid); }
bool launch_mfma_small_conv(const MfmaParams &p, int, int, int, int nsplit, int, unsigned grid, hipStream_t)
{
    g_nsplit = nsplit;
    return took("small_conv", p, grid);
}
bool launch_mfma_small_conv_wide(const MfmaParams &p, int, int, int, int, unsigned grid, hipStream_t) { return took("small_conv_wide", p, grid); }
bool launch_mfma_small_conv_pair(const MfmaParams &p0, unsigned grid0, const MfmaParams &, unsigned grid1, int, int, int, int, hipStream_t)
{
    return took("small_conv_pair", p0, grid0 + grid1);
}
bool launch_mfma_small_matrix(const MfmaParams &p, int, int, int, unsigned grid, hipStream_t) { return took("small_matrix", p, grid); }
bool launch_mfma_i8(const MfmaParams &p, int, int, unsigned grid, hipStream_t) { return took("i8", p, grid); }
bool launch_mfma_i8_wide(const MfmaParams &p, int, int, unsigned grid, hipStream_t) { return took("i8_wide", p, grid); }
bool launch_mfma_tile16(const MfmaParams &p, int, int, int, unsigned grid, hipStream_t) { return took("tile16", p, grid); }
static bool took_halo(const ConvHaloParams &p, bool stay, int fp, unsigned grid)
{
    g_kernel = "conv_halo"; g_halo = p; g_stay = stay; g_fp = fp; g_grid = grid;
    return true;
}
bool launch_conv_halo_u1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int, hipStream_t) { return took_halo(p, stay, fp, grid); }
bool launch_conv_halo_u2(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int, hipStream_t) { return took_halo(p, stay, fp, grid); }
bool launch_conv_halo_pm1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int, hipStream_t) { return took_halo(p, stay, fp, grid); }
static bool took_tile(const char *name, const TileParams &p, bool pmz, unsigned grid) { g_kernel = name; g_tp = p; g_pmz = pmz; g_grid = grid; return true; }
bool launch_tile8(const TileParams &p, bool conv, int vw, bool, bool pmz, unsigned grid, hipStream_t) { return conv && vw != 4 ? false : took_tile("tile8", p, pmz, grid); }
bool launch_tile4(const TileParams &p, bool conv, int vw, bool, bool pmz, unsigned grid, hipStream_t) { return conv && vw == 1 ? false : took_tile("tile4", p, pmz, grid); }
bool launch_tile2(const TileParams &p, bool, int, bool, bool pmz, unsigned grid, hipStream_t) { return took_tile("tile2", p, pmz, grid); }
}  // namespace apnn

static int failures = 0;
#define EXPECT(cond) do { if (!(cond)) { std::printf("line %d: %s (last error: %s)\n", __LINE__, #cond, apnn_last_error()); ++failures; } } while (0)

int main()
{
    void *fake = reinterpret_cast<void *>(uintptr_t(1) << 20);        // 16-byte aligned, never dereferenced
    const uint32_t *fw = static_cast<const uint32_t *>(fake);
    EXPECT(apnn_row_words(129) == 8 && apnn_packed_words(4096, 4096, 2) == size_t(4096) * 2 * 128);
    EXPECT(apnn_fmap_words(6272, 128, 2) == size_t(6272) * 2 * 4);
    EXPECT(apnn_input_weight_bytes(64, 3, 7, 7) > 0 && apnn_input_weight_bytes(64, 3, 11, 11) > apnn_input_weight_bytes(64, 3, 7, 7));
    EXPECT(apnn_workspace_bytes(nullptr) == 0);

    for (int C : {1, 7, 64, 1000}) {
        std::vector<double> g(C, 1.5), b(C, 0.25), m(C, 0.1), v(C, 2.0);
        std::vector<float> sc(C), bi(C);
        EXPECT(apnn_fold_bn(g.data(), b.data(), m.data(), v.data(), 1e-5, 0.5, 0.25, C, sc.data(), bi.data()) == APNN_OK);
        EXPECT(sc[C - 1] > 0.0f);
    }
    EXPECT(apnn_fold_bn(nullptr, nullptr, nullptr, nullptr, 1e-5, 0.0, 1.0, 4, nullptr, nullptr) == APNN_ERR_INVALID_ARG);

    EXPECT(apnn_debug_force("MFMA", 0) == APNN_OK && apnn_debug_force("INT8", 1) == APNN_OK);
    EXPECT(apnn_debug_force("NOT_A_SWITCH", 1) == APNN_ERR_INVALID_ARG && std::strlen(apnn_last_error()) > 0);
    EXPECT(apnn_debug_force(nullptr, 1) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_debug_force("A_NAME_THAT_IS_MUCH_LONGER_THAN_ANY_SWITCH_OF_THE_LIBRARY_AND_THEN_SOME", 1) == APNN_ERR_INVALID_ARG);
    apnn_debug_reset();
    EXPECT(apnn_debug_tile_choice(4096, 4096, 0, 1) == 256 && apnn_debug_tile_choice(64, 64, 0, 0) == 32);
    EXPECT(apnn_debug_tile_choice(0, 0, 0, 1) == 0);

    // argument checks of the compute entry points (each returns before any launch)
    EXPECT(apnn_gemm(fw, fw, nullptr, 4, 4, 64, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_gemm(fw, fw, static_cast<int32_t *>(fake), 4, 4, 64, 9, 2, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED, nullptr) == APNN_ERR_UNSUPPORTED);
    EXPECT(apnn_gemm(fw, fw, static_cast<int32_t *>(fake), 4, 4, 64, 2, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr) == APNN_ERR_UNSUPPORTED);
    EXPECT(apnn_gemm(fw, fw, static_cast<int32_t *>(fake), -1, 4, 64, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_gemm(fw, fw, static_cast<int32_t *>(fake), 4, 4, int64_t(1) << 40, 8, 8, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED, nullptr) != APNN_OK);
    EXPECT(apnn_gemm(reinterpret_cast<const uint32_t *>(uintptr_t(fake) + 4), fw, static_cast<int32_t *>(fake), 4, 4, 64, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr) == APNN_ERR_ALIGNMENT);
    EXPECT(apnn_gemm(fw, fw, static_cast<int32_t *>(fake), 0, 4, 64, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr) == APNN_OK);   // empty

    apnn_layer_desc L{};
    L.conv = apnn_conv_desc{8, 28, 28, 128, 128, 3, 3, 1, 1, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED};
    L.q_out = 2;
    EXPECT(apnn_layer(&L, fw, fw, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_INVALID_ARG);      // no scale / bias
    L.scale_dev = L.bias_dev = static_cast<const float *>(fake);
    L.pool = 3;
    EXPECT(apnn_layer(&L, fw, fw, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_INVALID_ARG);
    L.pool = 0; L.q_out = 9;
    EXPECT(apnn_layer(&L, fw, fw, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_UNSUPPORTED);
    L.q_out = 2; L.conv.Cin = 100;
    EXPECT(apnn_layer(&L, fw, fw, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_INVALID_ARG);
    L.conv.Cin = 128; L.conv.N = 0;
    EXPECT(apnn_layer(&L, fw, fw, static_cast<uint32_t *>(fake), nullptr) == APNN_OK);                   // empty batch
    EXPECT(apnn_layer(nullptr, fw, fw, nullptr, nullptr) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_layer_pair(nullptr, fw, fw, nullptr, nullptr, fw, fw, nullptr, nullptr) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_conv2d(nullptr, fw, fw, static_cast<int32_t *>(fake), nullptr) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_input_layer(nullptr, fake, static_cast<const uint8_t *>(fake), static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_INVALID_ARG);

    EXPECT(apnn_pack(fake, 4, 64, 9, APNN_ENC_UNSIGNED, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_UNSUPPORTED);
    EXPECT(apnn_pack(fake, 0, 64, 2, APNN_ENC_UNSIGNED, static_cast<uint32_t *>(fake), nullptr) == APNN_OK);
    EXPECT(apnn_quantize(static_cast<const float *>(fake), 4, 64, 0.0f, 0.0f, 2, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_sumpool(fw, 1, 7, 7, 64, 2, 7, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_OVERFLOW);
    EXPECT(apnn_maxpool(fw, 1, 8, 8, 64, 2, 3, 2, 3, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_INVALID_ARG);
    EXPECT(apnn_pack_patches(static_cast<const uint8_t *>(fake), 1, 3, 8, 8, 7, 12, 2, 3, 8, static_cast<uint32_t *>(fake), nullptr) == APNN_ERR_UNSUPPORTED);

    // ---- the dispatch (a launcher stand-in answers; the status is that of the runtime's last-error query, which
    // without a GPU may be a launch error: only the choice and its constants are looked at)
    int32_t *fy = static_cast<int32_t *>(fake);
    apnn_debug_reset();
    g_kernel.clear();
    (void)apnn_gemm(fw, fw, fy, 4096, 4096, 4096, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr);       // the headline product
    EXPECT(g_kernel == "mfma256" && g_grid == 256 && g_mp.out_scale == 2.0f && g_mp.c0 == 0 && g_mp.xcd_regions == 1);
    (void)apnn_gemm(fw, fw, fy, 2048, 2048, 2048, 3, 5, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED, nullptr);  // 6 FP4 passes: one int8 pass
    EXPECT(g_kernel == "i8" && g_grid == 256 && g_mp.accmul == 1 && g_mp.mulA == 0 && g_mp.mulB == 0 && g_mp.c0 == 0);
    (void)apnn_gemm(fw, fw, fy, 2048, 2048, 4096, 3, 5, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED, nullptr);  // long K: shared out among the waves
    EXPECT(g_kernel == "i8_wide" && g_grid == 256 && g_mp.nk % 4 == 0);
    (void)apnn_gemm(fw, fw, fy, 2048, 2048, 4096, 5, 6, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED, nullptr);  // 11 planes: more than its LDS holds
    EXPECT(g_kernel == "i8");
    (void)apnn_gemm(fw, fw, fy, 20, 20, 4000, 8, 8, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED, nullptr);      // beyond the exact range of FP4
    // bytes are value - 128 on both sides: Y = acc + 128 RA + 128 RB + c0, c0 = -npad 128^2 - 2 * 128 * 128 K + 128^2 K
    EXPECT(g_kernel == "i8" && g_mp.mulA == 128 && g_mp.mulB == 128 && g_mp.flipA == ~0u);
    EXPECT(g_mp.c0 == static_cast<int>(-(int64_t(g_mp.nk) * 128 - 4000) * 16384 - 16384 * int64_t(4000)));
    (void)apnn_gemm(fw, fw, fy, 64, 1024, 1024, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr);         // a paper-sized fully connected layer
    EXPECT(g_kernel == "tile16" && g_grid == 4 * 64 && g_mp.nk == 4);
    (void)apnn_gemm(fw, fw, fy, 8, 4096, 25088, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr);         // long K: eight waves
    EXPECT(g_kernel == "tile16" && g_grid == 256 && g_mp.nk == 8);
    (void)apnn_gemm(fw, fw, fy, 256, 1000, 4096, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr);        // more than two tiles a compute unit
    EXPECT(g_kernel == "small_matrix" && g_grid == 8 * 32);
    (void)apnn_gemm(fw, fw, fy, 512, 512, 100, 1, 1, APNN_ENC_PM1, APNN_ENC_PM1, nullptr);               // Case II: pad positions multiply to +1
    EXPECT(g_mp.c0 < 0);
    EXPECT(apnn_debug_force("MFMA", 0) == APNN_OK);
    (void)apnn_gemm(fw, fw, fy, 4096, 4096, 4096, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr);
    EXPECT(g_kernel == "tile4" && g_grid == 4096 && g_tp.alpha == 2 && g_tp.uB == -1 && g_tp.uA == 0 && g_tp.c0 == 0
           && g_tp.xm * g_tp.xn == 8);
    (void)apnn_gemm(fw, fw, fy, 100, 100, 777, 1, 1, APNN_ENC_PM1, APNN_ENC_PM1, nullptr);               // Case II: K - 2 popc(xor)
    EXPECT(g_kernel == "tile2" && g_tp.alpha == -2 && g_tp.c0 == 777);
    // -1/+1 features with padding on the popcount kernel: validity plane, c0 = -32 (walked words) (plane weights)
    apnn_layer_desc P{};
    P.conv = apnn_conv_desc{2, 9, 9, 96, 64, 3, 3, 1, 1, 3, 1, APNN_ENC_UNSIGNED, APNN_ENC_PM1};
    P.acc_out_dev = fy;
    (void)apnn_layer(&P, fw, fw, nullptr, nullptr);
    EXPECT(g_pmz == 1 && g_tp.PA == 2 && g_tp.alpha == 1 && g_tp.Kw == 27 && g_tp.c0 == -32 * 28 * 7);
    P.conv.p = 1; P.conv.encW = APNN_ENC_PM1;
    (void)apnn_layer(&P, fw, fw, nullptr, nullptr);
    EXPECT(g_pmz == 1 && g_tp.alpha == 2 && g_tp.uA == 1 && g_tp.c0 == -64 * 28);
    P.pool = APNN_POOL_SUM2;
    (void)apnn_layer(&P, fw, fw, nullptr, nullptr);
    EXPECT(g_tp.pool == 2 && g_tp.M == 2 * 4 * 4 * 4 && g_tp.Hp == 4);
    apnn_debug_reset();
    P.conv.Cin = 128;                                                                                       // matrix-core shape again
    (void)apnn_layer(&P, fw, fw, nullptr, nullptr);
    EXPECT(g_kernel == "tile16" && g_mp.pool == 2 && g_grid == 8 * 4);
    EXPECT(apnn_debug_force("MFMA_T16", 0) == APNN_OK);
    (void)apnn_layer(&P, fw, fw, nullptr, nullptr);
    EXPECT(g_kernel == "small_conv" && g_mp.pool == 2);
    apnn_debug_reset();

    // ---- 32-bit ranges of the large-layer kernel: operands below 2^31 bytes, one padded image below 2^27 words
    EXPECT(apnn_debug_force("MFMA_HALO", 0) == APNN_OK && apnn_debug_force("MFMA_T16", 0) == APNN_OK);
    apnn_layer_desc V{};
    V.acc_out_dev = fy;
    auto chosen = [&](int64_t images, int64_t H, int64_t W, int64_t Cin, int64_t Cout, int R, int pad, int q, int stride = 1) {
        V.conv = apnn_conv_desc{images, H, W, Cin, Cout, R, R, stride, pad, 1, q, APNN_ENC_PM1, APNN_ENC_UNSIGNED};
        g_kernel.clear();
        (void)apnn_layer(&V, fw, fw, nullptr, nullptr);
        return g_kernel;
    };
    EXPECT(chosen(1023, 128, 128, 512, 64, 3, 1, 2) == "small_conv_wide" && g_mp.bytesA == 1023u << 21 && g_mp.bytesB == 64 * 144 * 4);
    EXPECT(chosen(1024, 128, 128, 512, 64, 3, 1, 2) == "small_conv");                                      // features of 2^31 bytes
    EXPECT(chosen(1, 16, 16, 2048, 932032, 3, 1, 2) == "small_conv_wide" && g_mp.bytesB == 932032u * 2304);
    EXPECT(chosen(1, 16, 16, 2048, 932096, 3, 1, 2) == "small_conv");                                      // weights beyond
    EXPECT(chosen(1, 2043, 2044, 512, 64, 3, 0, 2) == "small_conv_wide");                                   // (2043 + 3)(2044 + 3) 32 words
    EXPECT(chosen(1, 2045, 2045, 512, 64, 3, 0, 2) == "small_conv");                                        // 2048^2 32 = 2^27
    // at most 2^24 - 1 blocks of four 32 x 32 tiles, and no more in the popcount kernel: else refused
    EXPECT(chosen(682, 1024, 1024, 64, 96, 1, 0, 1) == "small_conv" && g_grid == 682u * 3 << 13);
    EXPECT(chosen(683, 1024, 1024, 64, 96, 1, 0, 1) == "" && std::strstr(apnn_last_error(), "too large"));
    // an odd number of channel words: one padded image below 2^31 words, else the popcount kernel
    EXPECT(chosen(1, 32760, 32766, 32, 32, 1, 0, 2, 2) == "small_conv");
    EXPECT(chosen(1, 32767, 32767, 32, 32, 1, 0, 2, 2) == "tile2");                                            // 32768^2 2 = 2^31
    EXPECT(chosen(1, 28, 28, 96, 64, 3, 1, 2) == "small_conv" && g_mp.Cw == 3);
    EXPECT(apnn_debug_force("MFMA_SMALL", 0) == APNN_OK && chosen(1, 28, 28, 96, 64, 3, 1, 2) == "tile2");
    EXPECT(apnn_debug_force("MFMA_SMALL", -1) == APNN_OK);
    EXPECT(chosen(64, 56, 56, 64, 64, 3, 1, 2) == "small_conv_wide" && chosen(64, 56, 56, 64, 96, 3, 1, 2) == "small_conv");
    EXPECT(chosen(1, 14, 14, 64, 64, 3, 1, 2) == "small_conv");                                             // few tiles: K split
    // eight waves a tile: from 72 words of K on up to 512 tiles, from six groups a wave of four on up to 1024
    EXPECT(chosen(4, 14, 14, 256, 512, 3, 1, 2) == "small_conv" && g_nsplit == 8 && chosen(4, 14, 14, 128, 512, 3, 1, 2) == "small_conv" && g_nsplit == 4);
    EXPECT(chosen(4, 28, 28, 256, 256, 3, 1, 2) == "small_conv" && g_nsplit == 4 && chosen(8, 28, 28, 128, 128, 3, 1, 4) == "small_conv" && g_nsplit == 4);
    EXPECT(chosen(8, 14, 14, 512, 512, 3, 1, 2) == "small_conv" && g_nsplit == 4 && chosen(8, 14, 14, 512, 512, 3, 1, 4) == "small_conv" && g_nsplit == 8);
    EXPECT(chosen(8, 28, 28, 512, 256, 3, 1, 4) == "small_conv" && g_nsplit == 4);

    // ---- the library's own choice: staged convolutions (int32 results here) in their limits
    apnn_debug_reset();
    EXPECT(chosen(64, 56, 56, 64, 64, 3, 1, 2) == "conv_halo" && g_stay && g_halo.bytesA == 64u * 56 * 56 * 16 && g_halo.bytesB == 64 * 9 * 8);
    EXPECT(chosen(64, 56, 56, 64, 96, 3, 1, 2) == "conv_halo" && g_halo.per_column.d == 2);
    EXPECT(chosen(85598, 14, 14, 512, 64, 3, 1, 2) == "conv_halo" && !g_stay);
    EXPECT(chosen(85599, 14, 14, 512, 64, 3, 1, 2) == "small_conv");                                       // features of 2^31 bytes
    // large layers: not where a block of one tile has little to do with what it stages, nor int32 results of few steps
    EXPECT(chosen(25, 65, 65, 512, 512, 1, 0, 4) == "small_conv_wide" && chosen(25, 65, 65, 512, 512, 3, 1, 4) == "conv_halo");
    EXPECT(chosen(64, 56, 56, 128, 64, 1, 0, 2) == "small_conv_wide" && chosen(64, 56, 56, 128, 96, 1, 0, 2) == "conv_halo");     // (27.4 us there, 22.1 here)
    // few outputs, or rows of matrices or pixels that would be half of a 32 x 32 tile; not many pixels of few channels
    EXPECT(chosen(1, 14, 14, 64, 64, 3, 1, 2) == "tile16" && chosen(1, 3, 3, 256, 16384, 3, 0, 2) == "tile16");
    EXPECT(chosen(32, 56, 56, 64, 6, 3, 1, 2) == "small_conv" && chosen(32, 56, 56, 96, 10, 1, 0, 2) == "small_conv");
    (void)apnn_gemm(fw, fw, fy, 25000, 10, 1024, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED, nullptr);
    EXPECT(g_kernel == "tile16");
    // more than 256 of them with two groups of K for four waves: the 32 x 32 tiles
    auto product = [&](int64_t M, int64_t N, int64_t K, int p, int q) {
        g_kernel.clear();
        (void)apnn_gemm(fw, fw, fy, M, N, K, p, q, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED, nullptr);
        return g_kernel;
    };
    EXPECT(product(1205, 522, 208, 3, 3) != "i8" && product(1205, 522, 1500, 3, 3) == "i8" && product(1205, 522, 208, 3, 5) == "i8");
    EXPECT(product(1024, 1024, 208, 3, 3) == "i8" && product(512, 1000, 2048, 3, 3) != "i8");
    EXPECT(product(380, 321, 580, 5, 5) == "small_matrix" && product(380, 321, 512, 5, 5) == "tile16" && product(380, 321, 1030, 5, 5) == "tile16");
    EXPECT(product(256, 256, 580, 5, 5) == "tile16" && product(380, 321, 580, 2, 4) == "tile16" && product(380, 321, 580, 3, 3) == "small_matrix");
    EXPECT(chosen(8, 13, 13, 64, 64, 3, 1, 2) == "small_conv" && chosen(8, 12, 12, 96, 64, 3, 1, 2) == "small_conv" && chosen(8, 13, 13, 128, 64, 3, 1, 2) == "tile16");
    EXPECT(chosen(8, 13, 13, 128, 64, 1, 0, 2) == "tile16" && chosen(8, 13, 13, 96, 64, 1, 0, 2) == "small_conv" && chosen(8, 11, 11, 64, 64, 3, 1, 2) == "tile16");
    EXPECT(apnn_debug_force("MFMA_NSPLIT", 1) == APNN_OK && chosen(64, 56, 56, 64, 64, 3, 1, 2) == "small_conv_wide");   // another form asked for
    EXPECT(apnn_debug_force("MFMA_HALO", 1) == APNN_OK && chosen(64, 56, 56, 64, 64, 3, 1, 2) == "conv_halo");
    apnn_debug_reset();
    // eight waves a tile: at most 2^23 - 1 blocks of 512 threads, else the value is ignored
    EXPECT(apnn_debug_force("MFMA_NSPLIT", 8) == APNN_OK && chosen(255, 1024, 1024, 64, 32, 1, 0, 1) == "small_conv" && g_nsplit == 8);
    EXPECT(chosen(256, 1024, 1024, 64, 32, 1, 0, 1) == "small_conv" && g_nsplit == 1 && g_grid == 256u << 13);
    apnn_debug_reset();
    // weights of 4 GiB: not for 31-bit offsets
    V.conv = apnn_conv_desc{1, 8, 8, 64, int64_t(1) << 26, 1, 1, 1, 0, 8, 2, APNN_ENC_UNSIGNED, APNN_ENC_UNSIGNED};
    g_kernel.clear();
    (void)apnn_layer(&V, fw, fw, nullptr, nullptr);
    EXPECT(g_kernel == "small_conv");
    // planes of one or two bits without other outputs, else the kernels that write them
    apnn_layer_desc Q{};
    Q.scale_dev = Q.bias_dev = static_cast<const float *>(fake);
    auto planes = [&](int64_t images, int64_t hw, int64_t Cin, int64_t Cout, int stride, int q_out, int pool) {
        Q.conv = apnn_conv_desc{images, hw, hw, Cin, Cout, 3, 3, stride, 1, 1, 2, APNN_ENC_PM1, APNN_ENC_UNSIGNED};
        Q.q_out = q_out; Q.pool = pool;
        g_kernel.clear();
        (void)apnn_layer(&Q, fw, fw, static_cast<uint32_t *>(fake), nullptr);
        return g_kernel;
    };
    EXPECT(planes(128, 56, 64, 64, 1, 2, 0) == "conv_halo" && g_stay && g_fp == 2);
    EXPECT(planes(128, 56, 64, 64, 1, 3, 0) == "small_conv_wide" && planes(128, 56, 64, 64, 1, 2, 1) == "conv_halo" && g_fp == 4);
    auto pointwise = [&](int64_t images, int64_t hw, int64_t Cin, int64_t Cout, int stride, int q, int pool) {
        Q.conv = apnn_conv_desc{images, hw, hw, Cin, Cout, 1, 1, stride, 0, 1, q, APNN_ENC_PM1, APNN_ENC_UNSIGNED};
        Q.q_out = 2; Q.pool = pool;
        g_kernel.clear();
        (void)apnn_layer(&Q, fw, fw, static_cast<uint32_t *>(fake), nullptr);
        return g_kernel;
    };
    EXPECT(pointwise(128, 56, 64, 128, 2, 2, 0) == "conv_halo" && pointwise(128, 28, 512, 256, 1, 2, 0) == "conv_halo");
    EXPECT(pointwise(74, 72, 288, 320, 2, 1, 1) == "small_conv_wide");
    EXPECT(pointwise(73, 125, 640, 128, 1, 3, 0) == "small_conv_wide");
    // either side of the staged convolutions' rule, and of the pooled 16 x 16 tiles'
    EXPECT(planes(8, 56, 64, 64, 1, 2, 0) == "conv_halo" && planes(4, 56, 64, 64, 1, 2, 0) == "small_conv" && g_nsplit == 4);
    EXPECT(planes(8, 28, 128, 128, 1, 2, 0) == "small_conv" && planes(12, 28, 128, 128, 1, 2, 0) == "conv_halo");
    EXPECT(planes(8, 28, 64, 128, 1, 2, 0) == "small_conv" && planes(12, 28, 192, 128, 1, 2, 0) == "small_conv");
    Q.residual_dev = static_cast<const uint32_t *>(fake); Q.q_res = 2;
    EXPECT(planes(8, 28, 128, 128, 1, 2, 0) == "conv_halo");
    Q.residual_dev = nullptr;
    EXPECT(planes(8, 13, 64, 64, 1, 2, 1) == "small_conv" && planes(8, 13, 128, 64, 1, 2, 1) == "tile16");
    Q.acc_out_dev = fy;
    EXPECT(planes(128, 56, 64, 64, 1, 2, 0) == "small_conv_wide");
    Q.acc_out_dev = nullptr;

    // ---- input layers: 512 pixels a block with the rows staged, or 128
    apnn_layer_desc I{};
    I.scale_dev = I.bias_dev = static_cast<const float *>(fake);
    I.q_out = 2;
    auto input_pixels = [&](int64_t images, int64_t C, int64_t H, int64_t W, int R, int stride, int pad) {
        I.conv = apnn_conv_desc{images, H, W, C, 64, R, R, stride, pad, 1, 8, APNN_ENC_PM1, APNN_ENC_UNSIGNED};
        g_block = 0;
        (void)apnn_input_layer(&I, fake, static_cast<const uint8_t *>(fake), static_cast<uint32_t *>(fake), nullptr);
        return g_block == 512 ? 512 : g_block == 256 ? 128 : 0;
    };
    EXPECT(input_pixels(8, 3, 224, 224, 7, 2, 3) == 512 && g_grid == 8 * 112 * 112 / 512);
    EXPECT(input_pixels(5, 4, 55, 55, 3, 3, 1) == 128);
    EXPECT(input_pixels(64, 3, 56, 56, 3, 1, 1) == 512);
    EXPECT(input_pixels(1, 3, 224, 224, 11, 4, 2) == 512);
    // LDS is asked for once on every device that the kernel runs on; where it is refused the other kernel takes the layer
    auto asks = [&](int device) {
        g_device = device; g_asked = 0;
        EXPECT(input_pixels(8, 3, 224, 224, 7, 2, 3) == 512);
        return g_asked;
    };
    EXPECT(asks(0) == 0 && asks(3) == 1 && asks(3) == 0 && asks(0) == 0 && asks(63) == 1 && asks(63) == 0 && asks(64) == 1 && asks(64) == 1);
    g_device = 1; g_answer = hipErrorInvalidValue;
    EXPECT(input_pixels(8, 3, 224, 224, 7, 2, 3) == 128);
    g_answer = hipSuccess;
    EXPECT(asks(1) == 1 && asks(1) == 0);
    g_device = 0;
    // the last block's pixel numbers stay below 2^31
    EXPECT(input_pixels(1, 1, 268435391, 8, 1, 1, 0) == 512 && g_grid == (1u << 22) - 1);
    EXPECT(input_pixels(1, 1, 268435392, 8, 1, 1, 0) == 128 && input_pixels(1, 1, 268435424, 8, 1, 1, 0) == 128);
    EXPECT(input_pixels(1, 64, 8, 8, 1, (1 << 29) - 8, (1 << 29) - 8) == 128);                              // 2^59 bytes a channel

    if (failures == 0) std::puts("abi host sanitizer run ok");
    return failures != 0;
}
