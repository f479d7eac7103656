// Tiles of transforms adjacent in memory, one tile per workgroup: shapes and
// tile bodies shared by the four-step passes and the axis passes of
// multidimensional plans.  Each transform has its own LDS region, at a
// stride that spreads the tile over the 64 banks.
#pragma once

#include "device_fft.hpp"

namespace mifft {

// log2 EPT of an inner transform of length 2^Li: 16 threads per transform
// up to 256 points, then 16 points per thread (at most 64 threads).
constexpr int inner_e(int Li) { return Li <= 6 ? 2 : (Li == 7 ? 3 : 4); }

// Staging stride (complex elements) of one transform's LDS region: the
// padded Stockham region rounded up to 4 (mod 32), which spreads the 16
// transforms of a tile over distinct banks when the tile is staged.
template <int Li, int Ei>
constexpr int stage_stride()
{
    const int reg = Layout2<Li, Ei>::region();
    const int r = reg % 32;
    return reg + ((4 - r + 32) % 32);
}

// ---------------------------------------------------------------- axis tiles
// A tile is TILE transforms of length 2^L along an axis of stride 2^log2s,
// adjacent in memory: transform q starts at element
// (q >> log2s) 2^(L + log2s) + (q & (2^log2s - 1)), its point n is 2^log2s
// elements further per n, so row n of a tile is TILE consecutive values
// when the stride is at least TILE.  Used in place.

// log2 EPT of an axis transform of length 2^L: the whole transform in one
// thread for N <= 4, else as the four-step inner transforms.
constexpr int axis_e(int L) { return L <= 2 ? L : inner_e(L); }
// Transforms per workgroup: whole 128-byte lines.
constexpr int AXIS_TILE = 16;

template <int L>
constexpr int axis_wg()
{
    return AXIS_TILE * ((1 << L) >> axis_e(L));
}

template <int L, int E>
__device__ __forceinline__ void unit_rows(TwRegs<L, E>& tws)
{
#pragma unroll
    for (int p = 0; p < Sched<L, E>::NP; p++)
#pragma unroll
        for (int r = 0; r < (1 << E); r++)
            tws[p][r] = cf{1.f, 0.f};
}

// Transforms of up to 256 points (longer ones: wide_tile.hpp): the tile is
// staged through LDS (rows of TILE values in, one transform per TPT
// consecutive threads), so each transform's exchanges stay inside one
// wavefront; staged back the same way, nontemporally if NT.
template <int L, int S, bool NT>
__device__ __forceinline__ void axis_tile_staged(cf* __restrict__ io, const cf* __restrict__ rows, cf* lds,
                                                 int64_t q0, int64_t count, int log2s, float scale)
{
    constexpr int E = axis_e(L), TILE = AXIS_TILE, LT = 4;
    constexpr int N = 1 << L, EPT = 1 << E, TPT = N / EPT, ST = stage_stride<L, E>(), WG = TILE * TPT;
    constexpr bool WAVE = TPT <= 64;
    const int tid = threadIdx.x;
    // element n of tile transform c
    auto addr = [&](int c, int n) -> int64_t { return idx::axis_elem(q0 + c, n, L, log2s); };
#pragma unroll
    for (int i = 0; i < TILE * N / WG; i++) {
        const int idx = tid + i * WG;
        const int c = idx & (TILE - 1), n = idx >> LT;
        if (q0 + c < count)
            lds[c * ST + n] = ld_data<NT>(reinterpret_cast<const char*>(io + addr(c, n)));
    }
    __syncthreads();
    const int tb = tid / TPT, t = tid % TPT;
    cf* my = lds + tb * ST;
    cf v[EPT];
#pragma unroll
    for (int m = 0; m < EPT; m++)
        v[m] = my[t + m * TPT];
    TwRegs<L, E> tws;
    unit_rows<L, E>(tws);
    // rows after the exchange: enough wavefronts (2^16 at 16 MiB 19.3, ahead 19.5)
    run2<L, E, S, 1, WAVE, 0, 0, false>(v, t, rows, tws, my);
    if constexpr (TPT > 1)
        lds_sync<WAVE>();  // the last exchange is fully read
#pragma unroll
    for (int m = 0; m < EPT; m++)
        my[t + m * TPT] = cscale(v[m], scale);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TILE * N / WG; i++) {
        const int idx = tid + i * WG;
        const int c = idx & (TILE - 1), n = idx >> LT;
        if (q0 + c < count)
            st_data<NT>(reinterpret_cast<char*>(io + addr(c, n)), lds[c * ST + n]);
    }
}

}  // namespace mifft
