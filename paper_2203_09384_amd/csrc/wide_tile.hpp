// Tiles of 16 adjacent transforms of 512, 1024 or 2048 points (in large
// calls 128 and 256 too), 32 points per thread: the long axis passes and the long passes of the four-step.
//
// These passes are bound by memory bandwidth, and reach it only in whole
// 128-byte lines: on MI355X a copy of 2048-point columns at 2^26 points
// takes 284 us in tiles of 8 (64-byte runs), 1024-point columns in tiles
// of 16 take 226 us.  16 transforms of 2048 points fit LDS because an exchange moves
// one float plane (real parts, then imaginary parts) at a time: 34, 66 or
// 132 KiB per tile, so four (512 points) or two (1024) workgroups share a CU
// and one's loads and stores overlap another's passes.  With 32 points per
// thread 512 and 1024 points take two passes and a single exchange.
//
// MI355X at 2^26 points, 16 points per thread and whole complex values in
// LDS -> this: four-step 2^17 476 -> 438 us, 2^18 483 -> 444, 2^19
// 503 -> 448, 2^20 539 -> 446; five transforms of 2^20 points 52 -> 41 us;
// 2D 2048 x 2048 460 -> 441 us, 1024 x 1024 408 -> 385, 512 x 512
// 370 -> 366.
//
// Thread (t, c), c the tile's transform and the fastest lane index, holds
// points t + m TPT.  Plane element d of transform c is at pad(d) T + c:
// the T = 16 transforms are interleaved, so a wavefront's access covers 16
// transforms x 4 points and is conflict-free when the 4 padded indices
// differ mod 4.
#pragma once

#include "device_fft.hpp"

namespace mifft {

constexpr int WIDE_E = 5, WIDE_TILE = 16;
// W: 128 and 256 points too (is_bulk in stream.hpp says when).
constexpr bool wide_len(int L, bool W) { return (L >= 9 && L <= 11) || (W && (L == 7 || L == 8)); }
// pad(d) = d + (d >> B): one spare row of the plane every 2^B points, which
// makes the writes of the first pass (up to 1024 points) and every read
// conflict-free (the radix-2 pass of 2048 points writes two-way).
constexpr int wide_pad(int L) { return L <= 10 ? L - 5 : 5; }

// T transforms (16, or 32 for the two row groups of the real split).
template <int L, int T = WIDE_TILE>
struct Wide {
    using SC = Sched<L, WIDE_E>;
    static constexpr int N = 1 << L, EPT = 32, TPT = N / EPT, WG = TPT * T;
    static constexpr int PLANE = (N + (N >> wide_pad(L))) * T;  // floats
};

// Wavefronts per SIMD that the registers are limited for (128 per lane): one
// workgroup of 1024, two of 512 or four of 256 threads on a CU.
constexpr int WIDE_WAVES = 4;

// Whether pad(d0(t) + q TPT R + r NS) and pad(t + m TPT) of the exchange
// after pass P are pad of the thread's part plus pad of the rest: no carry
// into bit B.
constexpr bool wide_pad_splits(int L, int P)
{
    const int lr = idx::sched_log2r(L, WIDE_E, P), lns = idx::sched_log2ns(L, WIDE_E, P);
    const int tpt = (1 << L) / 32, low = (1 << wide_pad(L)) - 1;
    for (int t = 0; t < tpt; t++) {
        const int d0 = ((t >> lns) << (lns + lr)) + (t & ((1 << lns) - 1));
        for (int q = 0; q < (32 >> lr); q++)
            for (int r = 0; r < (1 << lr); r++)
                if ((d0 & low) + ((((q * tpt) << lr) + (r << lns)) & low) > low)
                    return false;
        for (int m = 0; m < 32; m++)
            if ((t & low) + ((m * tpt) & low) > low)
                return false;
    }
    return true;
}

// One plane of the exchange after pass P: COMP 0 real parts, 1 imaginary.
template <int L, int P, int COMP, int T>
__device__ __forceinline__ void wide_plane(cf (&v)[32], int t, float* lds)
{
    using SC = typename Wide<L>::SC;
    constexpr int LR = SC::log2r(P), R = 1 << LR, LNS = SC::log2ns(P), NS = 1 << LNS;
    constexpr int TPT = Wide<L>::TPT, Q = 32 / R, B = wide_pad(L);
    static_assert(wide_pad_splits(L, P), "padded addresses are a thread base plus immediates");
    const int k = t & (NS - 1), d0 = ((t >> LNS) << (LNS + LR)) + k;
    float* w = lds + (d0 + (d0 >> B)) * T;
#pragma unroll
    for (int q = 0; q < Q; q++)
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int d = q * TPT * R + r * NS;
            w[(d + (d >> B)) * T] = COMP ? v[q + r * Q].y : v[q + r * Q].x;
        }
    __syncthreads();
    const float* rd = lds + (t + (t >> B)) * T;
#pragma unroll
    for (int m = 0; m < 32; m++) {
        const int d = m * TPT;
        const float f = rd[(d + (d >> B)) * T];
        if (COMP)
            v[m].y = f;
        else
            v[m].x = f;
    }
}

// Values 4 K .. 4 K + 3 of the twiddle row of pass P.
template <int L, int S, int P, int K>
__device__ __forceinline__ void wide_row_part(cf (&w)[4], const cf* __restrict__ rows, int t)
{
    using SC = typename Wide<L>::SC;
    constexpr int NS = 1 << SC::log2ns(P);
    const float4* r4 =
        reinterpret_cast<const float4*>(rows + idx::rows_offset(L, WIDE_E, P) + (t & (NS - 1)) * 32) + 2 * K;
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const float4 q = r4[i];
        w[2 * i] = cf{q.x, S > 0 ? -q.y : q.y};
        w[2 * i + 1] = cf{q.z, S > 0 ? -q.w : q.w};
    }
}

// Twiddles of pass P, four at a time with the next four in flight: all 32
// at once would take the registers that the points need.
template <int L, int S, int P, int K = 0>
__device__ __forceinline__ void wide_twiddle(cf (&v)[32], cf (&w)[4], const cf* __restrict__ rows, int t)
{
    cf nx[4];
    if constexpr (K < 7)
        wide_row_part<L, S, P, K + 1>(nx, rows, t);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = K == 0 ? 1 : 0; i < 4; i++)
        v[4 * K + i] = cmul(v[4 * K + i], w[i]);
    if constexpr (K < 7)
        wide_twiddle<L, S, P, K + 1>(v, nx, rows, t);
}

// All passes of the tile's transforms; v in and out as points t + m TPT.
// `lds` is the tile's plane offset by the transform index c; `w` the first
// four twiddles of pass P.
template <int L, int S, int T = WIDE_TILE, int P = 0>
__device__ __forceinline__ void wide_run(cf (&v)[32], int t, const cf* __restrict__ rows, float* lds, cf (&w)[4])
{
    using SC = typename Wide<L>::SC;
    constexpr int R = 1 << SC::log2r(P), Q = 32 / R;
    if constexpr (SC::log2ns(P) > 0)
        wide_twiddle<L, S, P>(v, w, rows, t);
#pragma unroll
    for (int q = 0; q < Q; q++)
        dft_strided<R, S, Q, 32>(v, q);
    if constexpr (P + 1 < SC::NP) {
        if constexpr (P > 0)
            __syncthreads();  // the previous exchange is read
        cf nx[4];
        wide_row_part<L, S, P + 1, 0>(nx, rows, t);
        wide_plane<L, P, 0, T>(v, t, lds);
        __syncthreads();
        wide_plane<L, P, 1, T>(v, t, lds);
        wide_run<L, S, T, P + 1>(v, t, rows, lds, nx);
    }
}

// Axis pass over transforms q0 .. q0 + T - 1 below `count`, in place: a thread
// loads and stores its points straight from and to HBM, at the same
// addresses, nontemporally if NT.  Transforms past the end read transform q0
// and store nothing.
template <int L, int S, bool NT, int T>
__device__ __forceinline__ void wide_axis_tile(cf* __restrict__ io, const cf* __restrict__ rows, float* lds,
                                               int64_t q0, int64_t count, int log2s, float scale)
{
    constexpr int TPT = Wide<L, T>::TPT;
    const int tid = threadIdx.x, c = tid & (T - 1), t = tid / T;
    const int64_t q = q0 + c;
    const bool live = q < count;
    char* p = reinterpret_cast<char*>(io + idx::axis_elem(live ? q : q0, t, L, log2s));
    int64_t step = (int64_t)TPT << (log2s + 3);
    cf v[32];
#pragma unroll
    for (int m = 0; m < 32; m++)
        v[m] = ld_data<NT>(p + m * step);
    cf w[4];
    wide_run<L, S, T>(v, t, rows, lds + c, w);
    // The stores' addresses are computed again: kept from the loads, the 32
    // of them would take 64 registers through the passes.
    asm volatile("" : "+s"(step));
    if (live) {
#pragma unroll
        for (int m = 0; m < 32; m++)
            st_data<NT>(p + m * step, cscale(v[m], scale));
    }
}

// Tiles of 8 transforms where tiles of 16 would be fewer than two per CU:
// 256 CUs with one or two workgroups each finish unevenly, and a single
// transform or image does not reach all of them.  Tiles that share 128-byte
// lines run on one XCD (xcd_group_tile).  MI355X, tiles of 16 -> 8, us:
//   2^20 x 1 23.3 -> 19.4, x 5 39.6 -> 36.0, x 8 (512 tiles) 50.6 -> 54.1
//   2D 2048 x 2048 x 1 39.9 -> 36.6, x 3 85.8 -> 74.5; 1024 x 1024 x 1
//   17.5 -> 16.0, x 8 (512 tiles) 47.1 -> 48.5
//   real 2^20 x 1: R2C 24.4 -> 19.9, C2R 22.3 -> 18.0
// (Tiles of 4 gained at most 0.5 us more, at one or two transforms, and
// lost 2-10 us from 4 transforms on.)
inline bool narrow_tiles(int64_t count) { return count < 2 * 256 * WIDE_TILE; }

}  // namespace mifft
