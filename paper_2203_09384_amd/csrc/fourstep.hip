// Lengths 2^12 .. 2^20 (FP32): four-step Cooley-Tukey split N = N1 * N2.
//
// With n = n1 N2 + n2 and k = k1 + N1 k2 the DFT of Eq. (dft) factors as
//   X[k1 + N1 k2] = sum_n2 w_N2^{n2 k2} ( w_N^{n2 k1} sum_n1 x[n1 N2 + n2] w_N1^{n1 k1} )
// i.e. the radix-N1 / radix-N2 Cooley-Tukey split of Eq. (radix2) taken
// once with large radices.  Two kernels:
//   pass 1  column DFTs of length N1 (stride N2) times w_N^{n2 k1}, stored
//           to Y[k1 + N1 n2] of `out` (so pass 2's tile is read and written
//           in place);
//   pass 2  row DFTs of length N2 over n2, in place in `out`, output
//           X[k1 + N1 k2] (times the plan's scale).
// Each workgroup owns a tile of 16 transforms (16 columns, or 16 rows k1)
// so that every global load and store is a run of 16 complex values (one
// 128-byte line), and transforms them with the same Stockham passes as the
// batched kernels.  Long inner transforms are read straight into registers
// (the tile's transform index is the fastest lane index; from 512 points up
// with the passes of wide_tile.hpp); short ones are staged through LDS so
// that their exchanges stay inside one wavefront.
// w_N^j is built from a two-level FP32 table (w_N^{1024 a} and w_N^{b},
// both from FP64 sincospi); the column pass reads it as three levels in LDS.
#include "device_fft.hpp"
#include "launch.hpp"
#include "fourstep.hpp"
#include "stream.hpp"
#include "tile_fft.hpp"
#include "wide_tile.hpp"

namespace mifft {
namespace {

constexpr int TILE = 16;

template <int S>
__device__ __forceinline__ cf big_twiddle(const cf* __restrict__ lo, const cf* __restrict__ hi, unsigned j)
{
    cf w = cmul(hi[j >> 10], lo[j & 1023u]);
    if constexpr (S > 0)
        w.y = -w.y;
    return w;
}

// The w_N^{n2 k1} lookups are gathers (every lane its own entry); from the
// cached two-level table they cost about a tenth of the four-step's time.
// Each workgroup copies a three-level table into LDS instead (w_N^{1024 a},
// w_N^{32 b}, w_N^{c} for j = 1024 a + 32 b + c: 64 + N / 1024 entries, at
// most 8.5 KiB, taken from the two-level table), at one more complex product
// per point and without losing a workgroup per CU.  MI355X, 2^26 elements:
// 2^15 468 -> 428 us, 2^16 483 -> 440, 2^17 519 -> 478, 2^18 525 -> 485,
// 2^19 552 -> 508, 2^20 567 -> 542.  (The two levels whole in LDS, 10 KiB at
// 2^18, cost a workgroup per CU at 256-point columns.)
constexpr bool tw3_in_lds(int L) { return L >= 15; }

// Columns of 128+ points load straight into registers (MI355X: 2^15
// 485 -> 468 us, 2^16 494 -> 479 us against staging 128- and 256-point
// columns through LDS); the row pass keeps the axis-pass threshold.
constexpr bool col_direct(int L1) { return L1 >= 7; }

// Pass 1, columns of up to 256 points: tile = columns n2 in
// [16 nb, 16 nb + 16) of transform b.  Long columns (col_direct) are read straight into registers
// (the column index is the fastest lane index: rows of T values per
// wavefront access); short ones are staged through LDS so their exchanges
// stay inside one wavefront.  Either way the outputs go out through LDS:
// the tile's outputs Y[k1 + N1 n2] form one contiguous block.
template <int L1, int L2, int S, bool NT>
__global__ __launch_bounds__(TILE*((1 << L1) >> inner_e(L1))) void k_fourstep1(
    const cf* __restrict__ in, cf* __restrict__ out, const cf* __restrict__ rows, const cf* __restrict__ tlo,
    const cf* __restrict__ thi)
{
    constexpr int T = TILE, LT = 4;
    constexpr int E = inner_e(L1), N1 = 1 << L1, N2 = 1 << L2;
    constexpr int EPT = 1 << E, TPT = N1 / EPT, WG = T * TPT, ST = stage_stride<L1, E>();
    constexpr bool DIRECT = col_direct(L1);
    // the three-level table in LDS (tw3_in_lds): twl[c], twl[32 + b],
    // twl[64 + a]
    constexpr bool TW3 = tw3_in_lds(L1 + L2);
    constexpr int NHI = (1 << (L1 + L2)) >> 10;
    constexpr int NTW = TW3 ? 64 + NHI : 1;
    __shared__ cf lds[T * ST];
    __shared__ cf twl[NTW];
    const int tid = threadIdx.x;
    const int64_t tile = blockIdx.x;
    const int nb = (int)(tile % (N2 / T));
    // thread (tb, t): transform tb of the tile, thread t of that transform
    const int tb = DIRECT ? (tid & (T - 1)) : tid / TPT;
    const int t = DIRECT ? (tid >> LT) : tid % TPT;
    cf* my = lds + tb * ST;
    cf v[EPT];
    if constexpr (DIRECT) {
#pragma unroll
        for (int m = 0; m < EPT; m++)
            v[m] = ld_data<NT>(
                reinterpret_cast<const char*>(in + idx::fourstep_col_in(tile, tb, t + m * TPT, L1, L2, T)));
    } else {
        // stage: 16 consecutive columns per row n1 (one 128-byte line)
#pragma unroll
        for (int i = 0; i < T * N1 / WG; i++) {
            const int w = tid + i * WG;
            const int c = w & (T - 1), n1 = w >> LT;
            lds[c * ST + n1] = ld_c(in + idx::fourstep_col_in(tile, c, n1, L1, L2, T));
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < EPT; m++)
            v[m] = my[t + m * TPT];
    }
    if constexpr (TW3) {
        // twl: w_N^c (c < 32), w_N^{32 b} (b < 32), then w_N^{1024 a}
        for (int i = tid; i < NTW; i += WG)
            twl[i] = i < 32 ? tlo[i] : i < 64 ? tlo[32 * (i - 32)] : thi[i - 64];
        __syncthreads();
    }
    TwRegs<L1, E> tws;
    unit_rows<L1, E>(tws);
    constexpr bool WAVE = DIRECT ? TPT * T <= 64 : TPT <= 64;
    run2<L1, E, S, 1, WAVE>(v, t, rows, tws, my);
    const unsigned n2 = nb * T + tb;
#pragma unroll
    for (int m = 0; m < EPT; m++) {
        const unsigned k1 = t + m * TPT;
        const unsigned j = n2 * k1;
        cf w;
        if constexpr (TW3) {
            w = cmul(cmul(twl[64 + (j >> 10)], twl[32 + ((j >> 5) & 31u)]), twl[j & 31u]);
            if constexpr (S > 0)
                w.y = -w.y;
        } else {
            w = big_twiddle<S>(tlo, thi, j);
        }
        v[m] = cmul(v[m], w);
    }
    if constexpr (DIRECT)
        __syncthreads();  // every transform's last exchange is read
    else
        lds_sync<true>();  // this wavefront's last exchange is read
#pragma unroll
    for (int m = 0; m < EPT; m++)
        my[t + m * TPT] = v[m];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < T * N1 / WG; i++) {
        const int w = tid + i * WG;
        const int c = w / N1, k1 = w % N1;
        st_c(out + idx::fourstep_col_out(tile, c, k1, L1, L2, T), lds[c * ST + k1]);
    }
}

// Pass 1 for columns of 512 and more points: 16-column tiles with 32 points
// per thread.  The outputs leave through LDS too, one float plane
// at a time: column c at c (N1 + 4), which puts the 16 columns of a wavefront's
// writes 4 banks apart and each column's 4 points between them.
template <int L1, int L2, int S, bool NT>
__global__ __launch_bounds__(Wide<L1>::WG, WIDE_WAVES) void k_fourstep1_wide(
    const cf* __restrict__ in, cf* __restrict__ out, const cf* __restrict__ rows, const cf* __restrict__ tlo,
    const cf* __restrict__ thi)
{
    using W = Wide<L1>;
    constexpr int N1 = 1 << L1, N2 = 1 << L2, T = WIDE_TILE, WG = W::WG, TPT = W::TPT;
    constexpr int NTW = 64 + ((1 << (L1 + L2)) >> 10), CS = N1 + 4;
    static_assert(T * CS <= W::PLANE, "the output planes fit the exchange plane");
    __shared__ float lds[W::PLANE];
    __shared__ cf twl[NTW];
    const int tid = threadIdx.x, c = tid & (T - 1), t = tid / T;
    const int64_t tile = blockIdx.x;
    const int nb = (int)(tile % (N2 / T));
    cf v[32];
    {
        const char* p = reinterpret_cast<const char*>(in + idx::fourstep_col_in(tile, c, t, L1, L2, T));
#pragma unroll
        for (int m = 0; m < 32; m++)
            v[m] = ld_data<NT>(p + (int64_t)m * (TPT * N2 * 8));
    }
    for (int i = tid; i < NTW; i += WG)
        twl[i] = i < 32 ? tlo[i] : i < 64 ? tlo[32 * (i - 32)] : thi[i - 64];
    cf w4[4];
    wide_run<L1, S>(v, t, rows, lds + c, w4);
    const unsigned n2 = nb * T + c;
#pragma unroll
    for (int m = 0; m < 32; m++) {
        const unsigned j = n2 * (t + m * TPT);
        cf w = cmul(cmul(twl[64 + (j >> 10)], twl[32 + ((j >> 5) & 31u)]), twl[j & 31u]);
        if constexpr (S > 0)
            w.y = -w.y;
        v[m] = cmul(v[m], w);
    }
    // The tile's outputs Y[k1 + N1 n2] are one block: thread tid takes its
    // pairs 2 (tid + i WG), + 1.
    float x[32];
    float* my = lds + c * CS + t;
    const float* blk = lds;
    __syncthreads();  // the last exchange is read
#pragma unroll
    for (int m = 0; m < 32; m++)
        my[m * TPT] = v[m].x;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int e = 2 * (tid + i * WG);
        const float* q = blk + (e / N1) * CS + e % N1;
        x[2 * i] = q[0];
        x[2 * i + 1] = q[1];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 32; m++)
        my[m * TPT] = v[m].y;
    __syncthreads();
    gv4* dst = reinterpret_cast<gv4*>(out + tile * (T * N1)) + tid;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const int e = 2 * (tid + i * WG);
        const float* q = blk + (e / N1) * CS + e % N1;
        gv4 o;
        o.x = x[2 * i];
        o.y = q[0];
        o.z = x[2 * i + 1];
        o.w = q[1];
        dst[i * WG] = o;
    }
}

// Pass 2 with rows of 512 and more points.
template <int L1, int L2, int S, bool NT>
__global__ __launch_bounds__(Wide<L2>::WG, WIDE_WAVES) void k_fourstep2_wide(cf* __restrict__ io,
                                                                            const cf* __restrict__ rows,
                                                                            int64_t count, float scale)
{
    __shared__ float lds[Wide<L2>::PLANE];
    wide_axis_tile<L2, S, NT>(io, rows, lds, (int64_t)blockIdx.x * WIDE_TILE, count, L1, scale);
}

// Pass 2 (in place): tile = rows k1 in [16 kb, 16 kb + 16) of transform b,
// elements Y[k1 + N1 n2] (stride N1 along n2); outputs X[k1 + N1 k2] at the
// same addresses: the axis pass of a multidimensional transform with
// stride N1 over batch * N1 transforms.
template <int L1, int L2, int S, bool NT>
__global__ __launch_bounds__(axis_wg<L2>()) void k_fourstep2(cf* __restrict__ io, const cf* __restrict__ rows,
                                                            int64_t count, float scale)
{
    static_assert(AXIS_TILE == TILE, "row tiles of 16");
    __shared__ cf lds[TILE * stage_stride<L2, axis_e(L2)>()];
    const int64_t q0 = (int64_t)blockIdx.x * TILE;
    axis_tile_staged<L2, S, NT>(io, rows, lds, q0, count, L1, scale);
}

// Both passes over `batch` transforms.  NT: the column pass reads and the
// row pass reads and writes nontemporally; the column pass stores plainly.
template <int L1, int L2, int S, bool NT>
hipError_t launch_passes(const cf* in, cf* out, const cf* rows1, const cf* rows2, const cf* tlo, const cf* thi,
                         int64_t batch, float scale, hipStream_t stream)
{
    const int64_t t1 = batch * ((1 << L2) / TILE), t2 = batch * ((1 << L1) / TILE);
    hipError_t e;
    if constexpr (wide_len(L1))
        e = launch_kernel((k_fourstep1_wide<L1, L2, S, NT>), dim3((unsigned)t1), dim3(Wide<L1>::WG), 0, stream, in,
                          out, rows1, tlo, thi);
    else
        e = launch_kernel((k_fourstep1<L1, L2, S, NT>), dim3((unsigned)t1), dim3(TILE * ((1 << L1) >> inner_e(L1))),
                          0, stream, in, out, rows1, tlo, thi);
    if (e != hipSuccess)
        return e;
    // pass 2 is the axis pass of stride N1 over batch N1 transforms
    if constexpr (wide_len(L2))
        return launch_kernel((k_fourstep2_wide<L1, L2, S, NT>), dim3((unsigned)t2), dim3(Wide<L2>::WG), 0, stream,
                             out, rows2, batch << L1, scale);
    else
        return launch_kernel((k_fourstep2<L1, L2, S, NT>), dim3((unsigned)t2), dim3(axis_wg<L2>()), 0, stream, out,
                             rows2, batch << L1, scale);
}

// Streams run chunk by chunk (stream.hpp): the row pass reads what the
// column pass left in the memory-side cache.  MI355X at 512 MiB, whole batch
// and plain accesses -> this: 2^15 427 -> 351 us, 2^16 437 -> 350, 2^17
// 438 -> 349, 2^18 444 -> 348, 2^19 448 -> 366, 2^20 446 -> 377; at 256 MiB 2^16
// 221 -> 176 (nontemporal accesses alone).
template <int L1, int L2, int S>
hipError_t launch_fourstep(const void* in, void* out, const void* rows1, const void* rows2, const void* tlo,
                           const void* thi, int64_t batch, float scale, hipStream_t stream)
{
    const cf *src = static_cast<const cf*>(in), *lo = static_cast<const cf*>(tlo), *hi = static_cast<const cf*>(thi);
    const cf *r1 = static_cast<const cf*>(rows1), *r2 = static_cast<const cf*>(rows2);
    cf* dst = static_cast<cf*>(out);
    constexpr int64_t EACH = int64_t(sizeof(cf)) << (L1 + L2);
    if (!is_stream(batch * EACH))
        return launch_passes<L1, L2, S, false>(src, dst, r1, r2, lo, hi, batch, scale, stream);
    const int64_t per = chunk_units(EACH);
    for (int64_t b = 0; b < batch; b += per) {
        const int64_t nb = batch - b < per ? batch - b : per;
        const hipError_t e = launch_passes<L1, L2, S, true>(src + (b << (L1 + L2)), dst + (b << (L1 + L2)), r1, r2,
                                                            lo, hi, nb, scale, stream);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// log2 of the points per thread, and the LDS bytes, of an inner transform.
constexpr int fs_e(int Li) { return wide_len(Li) ? WIDE_E : inner_e(Li); }

template <int Li>
constexpr int fs_lds()
{
    if constexpr (wide_len(Li))
        return Wide<Li>::PLANE * (int)sizeof(float);
    else
        return TILE * stage_stride<Li, inner_e(Li)>() * (int)sizeof(cf);
}

template <int L>
void add_len()
{
    constexpr int L1 = (L + 1) / 2, L2 = L / 2;
    constexpr int E1 = fs_e(L1), E2 = fs_e(L2);
    const int tw = tw3_in_lds(L) ? (64 + (1 << (L - 10))) * (int)sizeof(cf) : 0;
    const FourStep fs{L, L1, L2, E1, E2, Layout2<L1, E1>::rows_total(), Layout2<L2, E2>::rows_total(),
                      &launch_fourstep<L1, L2, -1>, &launch_fourstep<L1, L2, +1>, fs_lds<L1>() + tw, fs_lds<L2>(),
                      TILE};
    register_fourstep(fs);
}

struct FourStepRegistrar {
    FourStepRegistrar()
    {
        add_len<12>();
        add_len<13>();
        add_len<14>();
        add_len<15>();
        add_len<16>();
        add_len<17>();
        add_len<18>();
        add_len<19>();
        add_len<20>();
    }
};
FourStepRegistrar fourstep_registrar;

}  // namespace

// Two-level twiddles of length N = 2^L: lo[b] = w_N^b (b < 1024),
// hi[a] = w_N^{1024 a} (a < N / 1024), w_N = exp(-2 pi i / N), FP64 sincospi
// rounded once to FP32.
__global__ void k_twiddle_big(float2* __restrict__ lo, float2* __restrict__ hi, int L)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int nhi = 1 << (L - 10);
    if (i >= 1024 + nhi)
        return;
    const int64_t j = i < 1024 ? i : (int64_t)(i - 1024) << 10;
    double s, c;
    sincospi(2.0 * (double)j / (double)(int64_t(1) << L), &s, &c);
    const float2 w = float2{(float)c, (float)(-s)};
    if (i < 1024)
        lo[i] = w;
    else
        hi[i - 1024] = w;
}

hipError_t launch_twiddle_big(void* lo, void* hi, int L, hipStream_t stream)
{
    const int total = 1024 + (1 << (L - 10));
    return launch_kernel(k_twiddle_big, dim3((total + 255) / 256), dim3(256), 0, stream, static_cast<float2*>(lo),
                       static_cast<float2*>(hi), L);
}

}  // namespace mifft
