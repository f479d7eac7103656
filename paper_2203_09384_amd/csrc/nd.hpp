// Host-side registry of the axis kernels of multidimensional plans.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mifft {

// In place on `io`: `count` transforms of length 2^log2n along an axis of
// stride 2^log2s elements; transform q starts at element
// (q >> log2s) * 2^(log2n + log2s) + (q & (2^log2s - 1)).  rows: the
// transform's per-pass twiddle rows; every output is multiplied by scale.
// stream: nontemporal loads and stores.
using LaunchAxis = hipError_t (*)(void* io, const void* rows, int64_t count, int log2s, float scale,
                                  bool stream, hipStream_t st);

struct KernelAxis {
    int log2n;
    int log2ept;
    int sign;
    int tile;  // transforms per workgroup
    LaunchAxis fn;
    int rows;       // twiddle-row entries (float2)
    int lds_bytes;
    bool bulk;    // for calls that fill the chip (is_bulk)
    bool narrow;  // for few transforms and short strides (axis_narrow)
};

// Whether transforms of 2048 points keep 16 points per thread, in narrow tiles,
// and not the 32 of longer tiles, and in which: tiles of 4 where one on every CU
// holds all `count` and along strides of up to 16, whose tiles read whole lines
// together; of 8 where those fit once.  MI355X, us, 16 points in tiles of 8 -> 32
// points -> tiles of 4: 2048 x 2 x 8 12.4 -> 13.5 -> 9.2; 512 MiB of 2048 x 2
// 400 -> 440 -> 332; 2048 x 16 x 8 (stride 128) x 8 22.8 -> 24.2 -> 20.3, x 16
// 30.6 -> 31.8 -> 31.5, x 32 60.1 -> 57.1 -> 59.5; 2048 x 2048 x 1 33.0 -> 35.0
// -> 34.4, x 2 56.1 -> 54.0 -> 58.0.
inline bool axis_narrow(int log2n, int64_t count, int log2s) { return log2n == 11 && (count <= 8 * 256 || log2s <= 4); }
inline int narrow_tile(int64_t count, int log2s) { return count > 4 * 256 && count <= 8 * 256 && log2s > 3 ? 8 : 4; }

void register_axis(const KernelAxis& k);
// The kernel for `count` transforms of stride 2^log2s in calls of `bytes` per
// direction.
const KernelAxis* find_axis(int log2n, int sign, int64_t bytes, int64_t count, int log2s);

}  // namespace mifft
