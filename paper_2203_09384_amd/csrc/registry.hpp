// Host-side registry of compiled kernel variants.  Each kernel translation
// unit registers its instantiations at library load; the planner looks
// them up by (log2 N, log2 EPT, workgroup size, sign).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mifft {

// Launch one FP32 batched transform: `batch` transforms of N = 2^log2n
// interleaved complex64 elements from `in` to `out`, output multiplied by
// `scale`.  `tw` is the 2048-entry table exp(-2 pi i m / 2048); `rows` the
// per-pass twiddle rows of the variant (kind >= 1); `grid_limit` > 0 caps
// the workgroup count of persistent kinds.
using LaunchC32 = hipError_t (*)(const void* in, void* out, const void* tw, const void* rows, int64_t batch,
                                 float scale, int64_t grid_limit, hipStream_t stream);

struct Variant {
    int log2ept, wg, kind;
};

// Built-in choice per log2 N (index 1..11) for FP32: the autotuner's pick on
// MI355X at 2^26 elements per launch (log2 EPT, workgroup size, variant).
constexpr Variant kDefaultC32[21] = {
    {0, 0, 0},     // unused
    {1, 64, 11},   // N=2     one thread per transform, block staged through LDS
    {2, 128, 11},  // N=4
    {3, 64, 11},   // N=8
    {4, 128, 11},  // N=16
    {3, 64, 12},   // N=32    several threads per transform, block staged through LDS
    {3, 256, 12},  // N=64
    {3, 64, 12},   // N=128
    {4, 128, 12},  // N=256
    {3, 64, 12},   // N=512
    {4, 64, 3},    // N=1024  persistent, next-group prefetch
    {4, 128, 3},   // N=2048  persistent, next-group prefetch
    {3, 512, 3},   // N=2^12  one transform per workgroup
    {4, 512, 3},   // N=2^13
    {4, 1024, 2},  // N=2^14  135 KiB LDS
    {0, 0, 9},     // N=2^15 .. 2^20: four-step (column + row pass)
    {0, 0, 9}, {0, 0, 9}, {0, 0, 9}, {0, 0, 9}, {0, 0, 9},
};

struct KernelC32 {
    int log2n, log2ept, wg, sign;
    int kind;                 // 0: one transform group per workgroup, per-pass table reads
                              // 1..4: twiddle-row kernels (1 + TW + 2 PF), see fft_c32.hip
                              // 5..8: the same with wave-local LDS exchanges
    LaunchC32 fn;
    int (*occupancy)();       // workgroups per CU (persistent kinds), else NULL
    int rows;                 // twiddle-row entries the variant needs (kind >= 1)
    int lds_bytes;            // LDS per workgroup
    // the same with plain stores, which stay in the memory-side cache for the
    // next pass of a multidimensional transform; compiled for the built-in
    // variant of each length, else NULL
    LaunchC32 feed;
};

void register_c32(const KernelC32& k);
const KernelC32* find_c32(int log2n, int log2ept, int wg, int sign, int kind);
int count_c32();
const KernelC32* c32_at(int i);

}  // namespace mifft
