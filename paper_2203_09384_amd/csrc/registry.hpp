// Host-side registry of compiled kernel variants.  Each kernel translation
// unit registers its instantiations at library load; the planner looks
// them up by (log2 N, log2 EPT, workgroup size, sign).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
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
    {3, 256, 3},   // N=2048  persistent, next-group prefetch
    {3, 512, 3},   // N=2^12  one transform per workgroup
    {4, 512, 3},   // N=2^13
    {4, 1024, 2},  // N=2^14  135 KiB LDS
    {0, 0, 9},     // N=2^15 .. 2^20: four-step (column + row pass)
    {0, 0, 9}, {0, 0, 9}, {0, 0, 9}, {0, 0, 9}, {0, 0, 9},
};

// Calls of at most `mib` MiB per direction take `v` instead (the first rule
// of their length that covers them).  The defaults were picked where the
// chip is full; below that a persistent grid's workgroups do little more
// than fill and drain their pipelines, and more, smaller threads per
// transform finish sooner.  MI355X, us, default -> rule (three buffer sets
// in turn):
//   N=256   0.5 MiB 3.4 -> 2.9, 8 MiB 5.0 -> 4.5, 32 MiB 13.9 -> 13.4 (64: 24.1 -> 25.5);
//           16 MiB 7.5 -> 8.4: the default's 1024 workgroups end there together,
//           four to a CU (18 MiB 9.3 -> 9.1)
//   N=512   0.5 MiB 2.9 -> 2.7, 8 MiB 5.1 -> 4.9, 15 MiB 7.8 -> 7.3 (16: 8.0 -> 8.5)
//   N=1024  8 MiB 6.1 -> 4.8, 16 MiB 10.2 -> 7.0, 24 MiB 11.5 -> 9.6 (40: 17.1 -> 19.0);
//           64 MiB 25.9 -> 24.8, 128 MiB 47.6 -> 46.4 (512: 182 -> 184)
//   N=2048  8 MiB 5.3 -> 4.9, 16 MiB 8.7 -> 7.8, 24 MiB 12.0 -> 11.6 (32: 14.6 -> 15.2)
//   N=2^12  0.5 MiB 5.0 -> 4.3, 16 MiB 8.8 -> 8.0 (40: 16.6 -> 19.6)
//   N=2^13  0.5 MiB 8.4 -> 7.8, 16 MiB 13.1 -> 12.0, 32 MiB 17.8 -> 16.5 (40: 23.5 -> 24.5)
struct SizeRule {
    int log2;  // of the length (FFT_R32: of the half length)
    int mib;
    Variant v;
    int sign = 0;  // of the plans it holds for; 0: both
};
constexpr SizeRule kRulesC32[] = {
    {8, 14, {3, 64, 6}},    {8, 16, {4, 128, 12}}, {8, 32, {3, 64, 6}},  {9, 15, {3, 64, 6}},  {10, 24, {3, 128, 2}},
    {10, 128, {3, 256, 3}}, {11, 24, {3, 256, 2}}, {12, 16, {3, 512, 2}}, {13, 32, {4, 512, 2}},
};

// The last axis of a multidimensional plan, storing plainly for the next
// pass, keeps 16 points per thread at 2048 points in streams (is_stream).
// MI355X, us, 16 -> 8 points: 2048 x 2048 x 8 191 -> 196, x 16 375 -> 378, 1024 x
// 2048 x 16 166 -> 166, 8 x 2048 x 1600 126 -> 127 (2 x 2048, 16 x 2048 and
// 256 x 2048 differ by at most 2 % either way); below a stream 8 x 2048 x 320
// 35.4 -> 34.0, 64 x 2048 x 64 48.7 -> 46.5, 2048 x 2048 x 2 53.1 -> 51.0.
constexpr Variant kLastAxis2048{4, 128, 3};

template <size_t N>
constexpr Variant rule_or(const SizeRule (&rules)[N], int log2, int64_t bytes, int sign, Variant otherwise)
{
    for (const SizeRule& r : rules)
        if (r.log2 == log2 && (r.sign == 0 || r.sign == sign) && bytes <= (int64_t(r.mib) << 20))
            return r.v;
    return otherwise;
}

struct KernelC32 {
    int log2n, log2ept, wg, sign;
    int kind;                 // 0: one transform group per workgroup, per-pass table reads
                              // 1..4: twiddle-row kernels (1 + TW + 2 PF), see fft_c32.hip
                              // 5..8: the same with wave-local LDS exchanges
    LaunchC32 fn;
    int (*occupancy)();       // workgroups per CU (persistent kinds), else NULL
    int rows;                 // twiddle-row entries the variant needs (kind >= 1)
    int lds_bytes;            // LDS per workgroup
    // the same with plain stores, which stay in the caches for the next pass of
    // a multidimensional transform (plain calls store nontemporally); compiled
    // for the variants that those run, else NULL
    LaunchC32 feed;
};

void register_c32(const KernelC32& k);
const KernelC32* find_c32(int log2n, int log2ept, int wg, int sign, int kind);
int count_c32();
const KernelC32* c32_at(int i);

}  // namespace mifft
