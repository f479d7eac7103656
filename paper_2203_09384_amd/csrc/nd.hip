// Axis passes of multidimensional transforms (FP32), in place.
//
// The multidimensional DFT of a d-dimensional array,
//   X[k] = sum_n x[n] prod_a w_{N_a}^{k_a n_a},
// has a kernel that factors over the axes, so it is the 1D transform of
// Eq. (dft) applied along each axis in turn.  The last (contiguous) axis
// runs through the batched 1D kernels; every other axis runs here: a
// transform along an axis of stride s has its points s elements apart, and
// a workgroup takes a tile of 16 transforms adjacent in memory, so that
// row n of the tile is 16 consecutive complex values (one 128-byte line).  Each transform runs the Stockham passes with its own
// LDS region, and the result is written over the input.
#include "device_fft.hpp"
#include "launch.hpp"
#include "nd.hpp"
#include "tile_fft.hpp"
#include "wide_tile.hpp"

namespace mifft {
namespace {

template <int L, int S, bool NT>
__global__ __launch_bounds__(axis_wg<L>()) void k_axis(cf* __restrict__ io, const cf* __restrict__ rows,
                                                        int64_t count, int log2s, float scale)
{
    __shared__ cf lds[AXIS_TILE * stage_stride<L, axis_e(L)>()];
    axis_tile_staged<L, S, NT>(io, rows, lds, (int64_t)blockIdx.x * AXIS_TILE, count, log2s, scale);
}

// 512 points and more (128 and 256 in large calls): 32 points per thread.
template <int L, int S, bool NT, int T>
__global__ __launch_bounds__((Wide<L, T>::WG), WIDE_WAVES) void k_axis_wide(cf* __restrict__ io,
                                                                      const cf* __restrict__ rows, int64_t count,
                                                                      int log2s, float scale)
{
    __shared__ float lds[Wide<L, T>::PLANE];
    const int64_t q0 = idx::xcd_group_tile(blockIdx.x, WIDE_TILE / T) * T;
    if (q0 < count)
        wide_axis_tile<L, S, NT, T>(io, rows, lds, q0, count, log2s, scale);
}

template <int L, int S, bool NT, int T>
hipError_t launch_axis_wide(cf* io, const cf* rows, int64_t count, int log2s, float scale, hipStream_t st)
{
    const int64_t tiles = (count + T - 1) / T, chunk = 8 * (WIDE_TILE / T);
    const dim3 grid((unsigned)(T == WIDE_TILE ? tiles : (tiles + chunk - 1) / chunk * chunk));
    return launch_kernel((k_axis_wide<L, S, NT, T>), grid, dim3(Wide<L, T>::WG), 0, st, io, rows, count, log2s,
                         scale);
}

template <int L, int S, bool NT, bool W>
hipError_t launch_axis_nt(cf* io, const cf* rows, int64_t count, int log2s, float scale, hipStream_t st)
{
    const dim3 grid((unsigned)((count + AXIS_TILE - 1) / AXIS_TILE));
    if constexpr (!wide_len(L, W)) {
        return launch_kernel((k_axis<L, S, NT>), grid, dim3(axis_wg<L>()), 0, st, io, rows, count, log2s, scale);
    } else {
        if constexpr (!NT)
            if (narrow_tiles(count))
                return launch_axis_wide<L, S, false, 8>(io, rows, count, log2s, scale, st);
        return launch_axis_wide<L, S, NT, 16>(io, rows, count, log2s, scale, st);
    }
}

template <int L, int S, bool W>
hipError_t launch_axis(void* io, const void* rows, int64_t count, int log2s, float scale, bool stream,
                       hipStream_t st)
{
    cf* p = static_cast<cf*>(io);
    const cf* r = static_cast<const cf*>(rows);
    return stream ? launch_axis_nt<L, S, true, W>(p, r, count, log2s, scale, st)
                  : launch_axis_nt<L, S, false, W>(p, r, count, log2s, scale, st);
}

template <int L, bool W = false>
void add_axis()
{
    constexpr int E = wide_len(L, W) ? WIDE_E : axis_e(L);
    const int rows = ((1 << L) >> E) > 1 ? Layout2<L, E>::rows_total() : 0;
    int lds;
    if constexpr (wide_len(L, W))
        lds = Wide<L>::PLANE * (int)sizeof(float);
    else
        lds = AXIS_TILE * stage_stride<L, E>() * (int)sizeof(cf);
    register_axis(KernelAxis{L, E, -1, AXIS_TILE, &launch_axis<L, -1, W>, rows, lds, W});
    register_axis(KernelAxis{L, E, +1, AXIS_TILE, &launch_axis<L, +1, W>, rows, lds, W});
}

struct AxisRegistrar {
    AxisRegistrar()
    {
        add_axis<1>();
        add_axis<2>();
        add_axis<3>();
        add_axis<4>();
        add_axis<5>();
        add_axis<6>();
        add_axis<7>();
        add_axis<7, true>();
        add_axis<8>();
        add_axis<8, true>();
        add_axis<9>();
        add_axis<10>();
        add_axis<11>();
    }
};
AxisRegistrar axis_registrar;

}  // namespace
}  // namespace mifft
