// Registry of the four-step kernels for FP32 lengths 2^12 .. 2^20.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mifft {

// Launch both passes: in -> out (pass 1), out in place (pass 2).  feeds: the
// next kernel reads all of `out`, which fits the memory-side cache, so pass 2
// leaves it there.
using LaunchFourStep = hipError_t (*)(const void* in, void* out, const void* rows1, const void* rows2,
                                      const void* tlo, const void* thi, int64_t batch, float scale, bool feeds,
                                      hipStream_t stream);

// Tables of a real-input plan above 2^15 (half length M = N1 N2, n = 2 M):
// the four-step plan's rows and two-level w_M; rows of 32 points per thread
// of both inner transforms; two-level w_n.
struct RealTables {
    const void *rows1, *rows2, *tlo, *thi;
    const void *wide1, *wide2, *rlo, *rhi;
};

// we / wi weight the edge bins (0 and M) and the interior ones.  R2C's ws
// holds fs_ws_transforms(M, batch) M complex values.
using LaunchFsR2C = hipError_t (*)(const void* in, void* out, void* ws, const RealTables& t, int64_t batch, float we,
                                   float wi, hipStream_t stream);
using LaunchFsC2R = hipError_t (*)(const void* in, void* out, const RealTables& t, int64_t batch, float we, float wi,
                                   hipStream_t stream);

// One pass's workgroups: points per thread (log2), transforms, threads and LDS
// bytes of each.
struct PassShape {
    int log2e, tile, wg, lds;
};
// The passes of a call of `batch` transforms: the complex column and row pass,
// R2C's row pass with the split, C2R's column pass with the reverse split.
enum FsPass { kFsCols, kFsRows, kFsSplitRows, kFsUnsplitCols };
using FsPassShape = PassShape (*)(FsPass pass, int64_t batch);

struct FourStep {
    int log2n, log2n1, log2n2;  // N = N1 * N2, column length N1, row length N2
    int log2e1, log2e2;         // elements per thread of the inner transforms
    int rows1, rows2;           // twiddle-row entries of the inner transforms
    LaunchFourStep fwd, bwd;    // sign -1 / +1
    FsPassShape pass;
    LaunchFsR2C r2c;            // real input of twice the length (M >= 2^15)
    LaunchFsC2R c2r;
    bool bulk;                  // for calls that fill the chip (is_bulk)
};

void register_fourstep(const FourStep& f);
// The kernels for calls of `bytes` per direction.
const FourStep* find_fourstep(int log2n, int64_t bytes);
int64_t fs_ws_transforms(int64_t m, int64_t batch);
hipError_t launch_twiddle_big(void* lo, void* hi, int L, hipStream_t stream);

}  // namespace mifft
