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

// Tiles of 4 or 8 transforms, 16 points per thread, whole complex values in LDS
// (71 KiB a tile of 4 at 2048 points: two workgroups per CU).  axis_narrow says
// where they are the better split: a few transforms are bound by the length of
// one workgroup's work, which this halves, and short strides by accesses of
// less than a line, which 16 stores in flight bear better than 32.  Tiles that
// share 128-byte lines run on one XCD.
constexpr int NARROW_E = 4;

template <int L, int S, int T>
__global__ __launch_bounds__((T * ((1 << L) >> NARROW_E))) void k_axis_narrow(cf* __restrict__ io,
                                                                         const cf* __restrict__ rows, int64_t count,
                                                                         int log2s, float scale)
{
    constexpr int E = NARROW_E, EPT = 1 << E, TPT = (1 << L) >> E, ST = stage_stride<L, E>();
    static_assert(TPT * T > 64, "exchanges span wavefronts");
    __shared__ cf lds[T * ST];
    const int tid = threadIdx.x, c = tid & (T - 1), t = tid / T;
    const int64_t q0 = idx::xcd_group_tile(blockIdx.x, 16 / T) * T, q = q0 + c;
    if (q0 >= count)
        return;
    const bool live = q < count;
    cf* p = io + idx::axis_elem(live ? q : q0, t, L, log2s);
    const int64_t step = (int64_t)TPT << log2s;
    cf v[EPT];
#pragma unroll
    for (int m = 0; m < EPT; m++)
        v[m] = ld_c(p + m * step);
    TwRegs<L, E> tws;
    unit_rows<L, E>(tws);
    run2<L, E, S, 1, false, 0, 0, false>(v, t, rows, tws, lds + c * ST);
    if (live) {
#pragma unroll
        for (int m = 0; m < EPT; m++)
            st_c(p + m * step, cscale(v[m], scale));
    }
}

template <int L, int S, int T>
hipError_t launch_narrow_tiles(void* io, const void* rows, int64_t count, int log2s, float scale, hipStream_t st)
{
    constexpr int GROUP = 8 * (16 / T);  // whole groups for the XCD grouping
    const int64_t tiles = (count + T - 1) / T;
    return launch_kernel((k_axis_narrow<L, S, T>), dim3((unsigned)((tiles + GROUP - 1) / GROUP * GROUP)),
                         dim3(T * ((1 << L) >> NARROW_E)), 0, st, static_cast<cf*>(io), static_cast<const cf*>(rows),
                         count, log2s, scale);
}

template <int L, int S>
hipError_t launch_axis_narrow(void* io, const void* rows, int64_t count, int log2s, float scale, bool, hipStream_t st)
{
    return narrow_tile(count, log2s) == 8 ? launch_narrow_tiles<L, S, 8>(io, rows, count, log2s, scale, st)
                                          : launch_narrow_tiles<L, S, 4>(io, rows, count, log2s, scale, st);
}

template <int L>
void add_axis_narrow()
{
    const int rows = Layout2<L, NARROW_E>::rows_total();
    const int lds = 8 * stage_stride<L, NARROW_E>() * (int)sizeof(cf);
    register_axis(KernelAxis{L, NARROW_E, -1, 4, &launch_axis_narrow<L, -1>, rows, lds, false, true});
    register_axis(KernelAxis{L, NARROW_E, +1, 4, &launch_axis_narrow<L, +1>, rows, lds, false, true});
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
    register_axis(KernelAxis{L, E, -1, AXIS_TILE, &launch_axis<L, -1, W>, rows, lds, W, false});
    register_axis(KernelAxis{L, E, +1, AXIS_TILE, &launch_axis<L, +1, W>, rows, lds, W, false});
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
        add_axis_narrow<11>();
    }
};
AxisRegistrar axis_registrar;

}  // namespace
}  // namespace mifft
