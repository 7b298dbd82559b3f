// Launcher of conv_halo_kernel: one translation unit per kind of features, so they compile in parallel.
#pragma once
#include "common.h"
#include "conv_halo.h"

namespace apnn {

template <int KA, int HW, int SW, int FP, int FW, int PT, bool POOL, bool MULTI, bool STAY>
bool launch_conv_halo(const ConvHaloParams &p, unsigned grid, int lds, hipStream_t st)
{
    const auto kernel = conv_halo_kernel<KA, HW, SW, FP, FW, PT, POOL, MULTI, STAY>;
    static std::atomic<uint64_t> granted{0};
    if (!all_of_lds(kernel, granted)) return false;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), lds, st, p);
    return true;
}

template <int KA, int HW, int SW, int PT, bool MULTI, bool STAY>
bool launch_conv_halo(const ConvHaloParams &p, int fp, unsigned grid, int lds, hipStream_t st)
{
    if (p.pool) return fp == 4 ? launch_conv_halo<KA, HW, SW, 4, 2, PT, true, MULTI, STAY>(p, grid, lds, st)
                               : launch_conv_halo<KA, HW, SW, 4, 1, PT, true, MULTI, STAY>(p, grid, lds, st);
    return fp == 2 ? launch_conv_halo<KA, HW, SW, 2, 2, PT, false, MULTI, STAY>(p, grid, lds, st)
                   : launch_conv_halo<KA, HW, SW, 1, 2, PT, false, MULTI, STAY>(p, grid, lds, st);
}

template <int KA, bool MULTI, bool STAY> bool launch_conv_halo(const ConvHaloParams &p, int fp, unsigned grid, int lds, hipStream_t st)
{
    // 256 and 512 channels: granules of a tap known to the compiler, 23 instructions a step and not 33.  Every count would need an
    // instance of its own (each is code that a first call fetches), so the other multiples of 128 take the general one.
    if constexpr (KA == OPK_U2 && !MULTI && !STAY) {
        if (p.Cw == 8) return launch_conv_halo<KA, 2, 4, 2, MULTI, STAY>(p, fp, grid, lds, st);
        if (p.Cw == 16) return launch_conv_halo<KA, 2, 4, 4, MULTI, STAY>(p, fp, grid, lds, st);
    }
    if (p.Cw % 4 == 0) return launch_conv_halo<KA, 2, 4, 0, MULTI, STAY>(p, fp, grid, lds, st);
    if (p.Cw % 2 == 0) return launch_conv_halo<KA, 1, 2, 0, MULTI, STAY>(p, fp, grid, lds, st);
    return launch_conv_halo<KA, 1, 1, 0, MULTI, STAY>(p, fp, grid, lds, st);
}

template <int KA, bool MULTI> bool launch_conv_halo(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st)
{
    return stay ? launch_conv_halo<KA, MULTI, true>(p, fp, grid, lds, st) : launch_conv_halo<KA, MULTI, false>(p, fp, grid, lds, st);
}

bool launch_conv_halo_u1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st);
bool launch_conv_halo_u2(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st);
bool launch_conv_halo_pm1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st);

}  // namespace apnn
