// Host-side plumbing shared by the C-ABI entry points: status codes, the
// thread-local error text, argument checks and launch error capture.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "../../include/apnn.h"

namespace apnn {

char *error_buffer();                         // thread-local, 512 bytes
int fail(apnn_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

// Checks the status of the launch just issued (no synchronisation).
int check_launch(const char *what);

// A launch has less than 2^32 threads: of a larger one the runtime drops blocks without an error.  A kernel with a thread per
// item is launched in slices: launch(first item, blocks of 256).
template <class F> void in_slices(int64_t items, F &&launch)
{
    constexpr int64_t slice = int64_t(1) << 31;
    for (int64_t first = 0; first < items; first += slice)
        launch(first, static_cast<unsigned>(ceil_div(items - first < slice ? items - first : slice, 256)));
}
constexpr int64_t kMaxBlocks = (int64_t(1) << 24) - 1;      // of 256 threads

// Lets a kernel take all of a compute unit's LDS on the calling thread's device, more than it may have unasked.  Asked for once
// per kernel and device (`granted` has a bit for each): what was granted on one device does not hold on another.  Two
// threads that come here together ask for the same.
template <class Kernel> bool all_of_lds(Kernel kernel, std::atomic<uint64_t> &granted)
{
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return false;
    const uint64_t bit = device < 64 ? uint64_t(1) << device : 0;       // (beyond 64 devices: asked for in every call)
    if (granted.load(std::memory_order_relaxed) & bit) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
        (void)hipGetLastError();                            // another kernel takes the call
        return false;
    }
    granted.fetch_or(bit, std::memory_order_relaxed);
    return true;
}

// Override INPUT_TILE (layer.hip): -1 when it is not set.
int input_tile_override();

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// bits in 1..8; +-1 only with one bit (Sec. 3.2 defines it for 1-bit operands).
int check_bits_enc(const char *who, const char *name, int bits, apnn_encoding enc);

// K (2^p - 1)(2^q - 1) must stay below 2^31 (the result type is int32, Sec. 4.1).
int check_int32_range(const char *who, int64_t K, int p, int q);

}  // namespace apnn
