// Launcher of conv_halo_kernel: one translation unit per kind of features, so they compile in parallel.
#pragma once
#include "common.h"
#include "conv_halo.h"

namespace apnn {

template <int KA, int SW, int FP, int FW, int FC, bool POOL, bool MULTI, bool PACKED, bool STAY, bool THREE = false>
bool launch_conv_halo(const ConvHaloParams &p, unsigned grid, int lds, hipStream_t st)
{
    const auto kernel = conv_halo_kernel<KA, SW, FP, FW, FC, POOL, MULTI, PACKED, STAY, THREE>;
    static std::atomic<uint64_t> granted{0};
    if (!all_of_lds(kernel, granted)) return false;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(128 * FC), lds, st, p);
    return true;
}

template <int KA, int SW, int FC, bool MULTI, bool PACKED, bool STAY> bool launch_conv_halo(const ConvHaloParams &p, int fp, unsigned grid, int lds, hipStream_t st)
{
    if (p.pool) return fp == 4 ? launch_conv_halo<KA, SW, 4, 2, FC, true, MULTI, PACKED, STAY>(p, grid, lds, st)
                               : launch_conv_halo<KA, SW, 4, 1, FC, true, MULTI, PACKED, STAY>(p, grid, lds, st);
    if constexpr (MULTI && STAY) {
        if (p.three) return launch_conv_halo<KA, SW, 1, 2, FC, false, MULTI, PACKED, STAY, true>(p, grid, lds, st);
    }
    return fp == 2 ? launch_conv_halo<KA, SW, 2, 2, FC, false, MULTI, PACKED, STAY>(p, grid, lds, st)
                   : launch_conv_halo<KA, SW, 1, 2, FC, false, MULTI, PACKED, STAY>(p, grid, lds, st);
}

template <int KA, bool MULTI, bool PACKED, bool STAY> bool launch_conv_halo(const ConvHaloParams &p, int fp, unsigned grid, int lds, hipStream_t st)
{
    if constexpr (!PACKED) {
        if (p.pairs == 2) return p.Cw % 8 == 0 ? launch_conv_halo<KA, 8, 4, MULTI, PACKED, STAY>(p, fp, grid, lds, st) : launch_conv_halo<KA, 4, 4, MULTI, PACKED, STAY>(p, fp, grid, lds, st);
    }
    if (p.Cw % 8 == 0) return launch_conv_halo<KA, 8, 2, MULTI, PACKED, STAY>(p, fp, grid, lds, st);
    if (p.Cw % 4 == 0) return launch_conv_halo<KA, 4, 2, MULTI, PACKED, STAY>(p, fp, grid, lds, st);
    if (p.Cw % 2 == 0) return launch_conv_halo<KA, 2, 2, MULTI, PACKED, STAY>(p, fp, grid, lds, st);
    return launch_conv_halo<KA, 1, 2, MULTI, PACKED, STAY>(p, fp, grid, lds, st);
}

// (several digits come as bits; weights that stay are one digit, and so are features of one plane and -1/+1 features)
template <int KA> bool launch_conv_halo(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st)
{
    const bool multi = p.DA > 1 || p.DB > 1;
    if (multi && !stay) return launch_conv_halo<KA, true, true, false>(p, fp, grid, lds, st);
    if constexpr (KA == OPK_U2) {
        if (multi) return launch_conv_halo<KA, true, true, true>(p, fp, grid, lds, st);
    }
    if (p.packed) return stay ? launch_conv_halo<KA, false, true, true>(p, fp, grid, lds, st) : launch_conv_halo<KA, false, true, false>(p, fp, grid, lds, st);
    return stay ? launch_conv_halo<KA, false, false, true>(p, fp, grid, lds, st) : launch_conv_halo<KA, false, false, false>(p, fp, grid, lds, st);
}

bool launch_conv_halo_u1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st);
bool launch_conv_halo_u2(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st);
bool launch_conv_halo_pm1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st);

}  // namespace apnn
