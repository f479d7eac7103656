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
    // rows after the exchange: enough wavefronts (2^16 at 16 MiB 19.3, ahead 19.5)
    run2<L1, E, S, 1, WAVE, 0, 0, false>(v, t, rows, tws, my);
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

// ---------------------------------------------------------------- wide columns
// Pass 1 for columns of 512 and more points (and the 256-point columns of
// real input): 16-column tiles with 32 points per thread.

// The three-level table in LDS (tw3_in_lds): w_N^c, w_N^{32 b}, w_N^{1024 a}.
template <int L1, int L2, int T>
__device__ __forceinline__ void col_tables(cf* twl, const cf* __restrict__ tlo, const cf* __restrict__ thi, int tid)
{
    constexpr int NTW = 64 + ((1 << (L1 + L2)) >> 10);
    for (int i = tid; i < NTW; i += Wide<L1, T>::WG)
        twl[i] = i < 32 ? tlo[i] : i < 64 ? tlo[32 * (i - 32)] : thi[i - 64];
}

// v[m] *= w_N^{n2 k1}, k1 = t + m TPT.
template <int L1, int L2, int S>
__device__ __forceinline__ void col_twiddle(cf (&v)[32], const cf* twl, unsigned n2, int t)
{
#pragma unroll
    for (int m = 0; m < 32; m++) {
        const unsigned j = n2 * (t + m * Wide<L1>::TPT);
        cf w = cmul(cmul(twl[64 + (j >> 10)], twl[32 + ((j >> 5) & 31u)]), twl[j & 31u]);
        if constexpr (S > 0)
            w.y = -w.y;
        v[m] = cmul(v[m], w);
    }
}

// The outputs leave through LDS, one float plane at a time: column c at
// c (N1 + 64 / T), which puts the T columns of a wavefront's writes 64 / T
// banks apart and each column's 64 / T points between them.
template <int L1, int T>
constexpr int col_plane()
{
    const int out = T * ((1 << L1) + 64 / T);
    return Wide<L1, T>::PLANE > out ? Wide<L1, T>::PLANE : out;
}

// The tile's outputs Y[k1 + N1 n2] are one block of T N1 values: thread
// tid takes its pairs 2 (tid + i WG), + 1.
template <int L1, int T>
__device__ __forceinline__ void col_store(const cf (&v)[32], float* lds, cf* __restrict__ block, int tid)
{
    constexpr int N1 = 1 << L1, TPT = Wide<L1, T>::TPT, WG = Wide<L1, T>::WG, CS = N1 + 64 / T;
    float x[32];
    float* my = lds + (tid & (T - 1)) * CS + tid / T;
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
    gv4* dst = reinterpret_cast<gv4*>(block) + tid;
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

template <int L1, int L2, int S, bool NT, int T>
__global__ __launch_bounds__((Wide<L1, T>::WG), WIDE_WAVES) void k_fourstep1_wide(
    const cf* __restrict__ in, cf* __restrict__ out, const cf* __restrict__ rows, const cf* __restrict__ tlo,
    const cf* __restrict__ thi)
{
    constexpr int N1 = 1 << L1, N2 = 1 << L2, TPT = Wide<L1, T>::TPT;
    __shared__ float lds[col_plane<L1, T>()];
    __shared__ cf twl[64 + ((1 << (L1 + L2)) >> 10)];
    const int tid = threadIdx.x, c = tid & (T - 1), t = tid / T;
    const int64_t tile = idx::xcd_group_tile(blockIdx.x, WIDE_TILE / T);
    const int nb = (int)(tile % (N2 / T));
    cf v[32];
    {
        const char* p = reinterpret_cast<const char*>(in + idx::fourstep_col_in(tile, c, t, L1, L2, T));
#pragma unroll
        for (int m = 0; m < 32; m++)
            v[m] = ld_data<NT>(p + (int64_t)m * (TPT * N2 * 8));
    }
    col_tables<L1, L2, T>(twl, tlo, thi, tid);
    cf w4[4];
    wide_run<L1, S, T>(v, t, rows, lds + c, w4);
    col_twiddle<L1, L2, S>(v, twl, nb * T + c, t);
    col_store<L1, T>(v, lds, out + tile * (T * N1), tid);
}

// Pass 2 with rows of 512 and more points.
template <int L1, int L2, int S, bool NT, int T>
__global__ __launch_bounds__((Wide<L2, T>::WG), WIDE_WAVES) void k_fourstep2_wide(cf* __restrict__ io,
                                                                            const cf* __restrict__ rows,
                                                                            int64_t count, float scale)
{
    __shared__ float lds[Wide<L2, T>::PLANE];
    const int64_t q0 = idx::xcd_group_tile(blockIdx.x, WIDE_TILE / T) * T;
    wide_axis_tile<L2, S, NT, T>(io, rows, lds, q0, count, L1, scale);
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

// ---------------------------------------------------------------- real input
// Real input above 2^15 (see real.hip for the formulas): the even/odd split
// of the half-length transform (M = N1 N2 points) is folded into the passes,
// so that the spectrum crosses memory twice instead of three times.  MI355X,
// split as a pass of its own -> folded (and chunked, see real_chunk), us:
//   n = 2^20, 256 MiB of reals: R2C 376 -> 209, C2R 377 -> 214
//   n = 2^20, 64 MiB:           R2C  85 ->  53, C2R  86 ->  53
//   n = 2^16, 512 MiB:          R2C 652 -> 456, C2R 644 -> 446
//
// w_n^k, n = 2 M, from the two-level table (rlo[1024], rhi[n / 1024]).

// X_k from a = Z_k, b = Z_{M-k}, w = w_n^k.
__device__ __forceinline__ cf split_bin(cf a, cf b, cf w)
{
    const float sx = 0.5f * (a.x + b.x), sy = 0.5f * (a.y - b.y);
    const float dx = 0.5f * (a.y + b.y), dy = -0.5f * (a.x - b.x);
    return cf{sx + w.x * dx - w.y * dy, sy + w.x * dy + w.y * dx};
}

// Z'_k from a = X_k, b = X_{M-k}, w = w_n^k.
__device__ __forceinline__ cf unsplit_bin(cf a, cf b, cf w)
{
    const float dx = a.x - b.x, dy = a.y + b.y;
    return cf{a.x + b.x - w.x * dy + w.y * dx, a.y - b.y + w.x * dx + w.y * dy};
}

// R2C pass 2: row DFTs of Y in `ws` and the split into `out` (M + 1 bins per
// transform).  Bin k1 + N1 k2 pairs with row N1 - k1, k2' = N2 - 1 - k2, so
// a tile is rows a .. a + H - 1 (slots c < H = T / 2) and their partners
// N1 - a - i (slots H + i).  Row 0 is its own partner (k2' = N2 - k2), and so
// is row N1 / 2, which takes slot H of the first tile.  The partner's values come
// through LDS, one float plane at a time.  All tiles of a transform run on
// one XCD while there are 8 transforms to deal (bins rows start at odd
// multiples of 8 bytes, so tiles share lines, which meet in that XCD's L2).
//
// Narrow tiles (T = 16) of up to 128 threads run where there are few of them:
// registers are not limited for four wavefronts per SIMD, so that all of a
// thread's loads are in flight.  MI355X, R2C in us, limited -> not: n = 2^16 x 2
// 12.1 -> 11.8, 2^17 x 1 13.0 -> 12.4, x 48 29.1 -> 27.5, 2^18 x 6 22.2 -> 20.7 (256 threads,
// 2^19 x 2 19.6 -> 19.9).
template <int L2, int T>
constexpr int split_waves() { return T == 16 && Wide<L2, T>::WG <= 128 ? 1 : WIDE_WAVES; }

template <int L1, int L2, int T>
__global__ __launch_bounds__((Wide<L2, T>::WG), (split_waves<L2, T>())) void k_rows_split(
    const cf* __restrict__ ws, cf* __restrict__ out, const cf* __restrict__ rows, const cf* __restrict__ rlo,
    const cf* __restrict__ rhi, int64_t batch, float we, float wi)
{
    constexpr int H = T / 2, N1 = 1 << L1, N2 = 1 << L2, TPT = Wide<L2, T>::TPT, B = wide_pad(L2), PER = N1 / T;
    constexpr int64_t M = int64_t(1) << (L1 + L2);
    static_assert(TPT % (1024 / N1) == 0, "the low twiddle index is the same for all of a thread's bins");
    // one row of T beyond the plane: row 0 again, as the partner k2' = N2
    __shared__ float lds[Wide<L2, T>::PLANE + T];
    const int tid = threadIdx.x, c = tid & (T - 1), t = tid / T;
    const idx::Tile at = idx::xcd_deal_tile(blockIdx.x, batch, PER);
    const int a = (int)at.tile * H;
    const int k1 = c < H ? a + c : (a == 0 && c == H ? N1 / 2 : N1 - a - (c - H));
    cf v[32];
    {
        const char* p = reinterpret_cast<const char*>(ws + at.b * M + k1 + (int64_t)N1 * t);
#pragma unroll
        for (int m = 0; m < 32; m++)
            v[m] = ld_data<false>(p + (int64_t)m * (TPT * N1 * 8));
    }
    cf w4[4];
    wide_run<L2, -1, T>(v, t, rows, lds + c, w4);
    // partner of (t + m TPT, c): index base + (31 - m) TPT of slot pc
    const bool row0 = a == 0 && c == 0, own = row0 || (a == 0 && c == H);
    const int pt = row0 ? TPT - t : TPT - 1 - t, pc = own ? c : c ^ H;
    float* mine = lds + (t + (t >> B)) * T + c;
    const float* theirs = lds + (pt + (pt >> B)) * T + pc;
    float d[32];
    __syncthreads();  // the last exchange is read
#pragma unroll
    for (int m = 0; m < 32; m++)
        mine[(m * TPT + ((m * TPT) >> B)) * T] = v[m].x;
    if (row0 && t == 0)
        mine[(N2 + (N2 >> B)) * T] = v[0].x;
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 32; m++)
        d[m] = theirs[((31 - m) * TPT + (((31 - m) * TPT) >> B)) * T];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 32; m++)
        mine[(m * TPT + ((m * TPT) >> B)) * T] = v[m].y;
    if (row0 && t == 0)
        mine[(N2 + (N2 >> B)) * T] = v[0].y;
    __syncthreads();
    const cf lo = rlo[(k1 + N1 * t) & 1023];
    const cf* hi = rhi + ((k1 + N1 * t) >> 10);
    cf* dst = out + at.b * (M + 1) + k1 + (int64_t)N1 * t;
#pragma unroll
    for (int m = 0; m < 32; m++) {
        const cf z{d[m], theirs[((31 - m) * TPT + (((31 - m) * TPT) >> B)) * T]};
        const cf x = split_bin(v[m], z, cmul(hi[m * (TPT * N1 / 1024)], lo));
        const float s = m == 0 && t == 0 && k1 == 0 ? we : wi;
        st_c(dst + (int64_t)m * (TPT * N1), cf{x.x * s, x.y * s});
    }
    if (row0 && t == 0)
        st_c(dst + M, cf{(v[0].x - v[0].y) * we, 0.f});  // X_M = E_0 - O_0
}

// Four points of the reverse split, STEP apart: bins k (from up), bins M - k
// (from down) and w_n^k's high factors.
template <int STEP, int I>
struct Unsplit {
    cf p[4], q[4], h[4];
    __device__ __forceinline__ void load(const cf* __restrict__ up, const cf* __restrict__ down,
                                         const cf* __restrict__ hi)
    {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            p[i] = ld_c(up + (4 * I + i) * STEP);
            q[i] = ld_c(down - (4 * I + i) * STEP);
            h[i] = hi[(4 * I + i) * (STEP / 1024)];
        }
    }
};

// The reverse split into v, four points at a time with the next four in
// flight: all at once would take twice the registers that the points need.
template <int STEP, int I = 0>
__device__ __forceinline__ void unsplit_points(cf (&v)[32], Unsplit<STEP, I>& now, const cf* __restrict__ up,
                                               const cf* __restrict__ down, const cf* __restrict__ hi, cf lo,
                                               bool edge, float we, float wi)
{
    Unsplit<STEP, I + 1> nx;
    if constexpr (I < 7)
        nx.load(up, down, hi);
    __builtin_amdgcn_sched_barrier(0);
    if (I == 0 && edge)
        now.p[0].y = now.q[0].y = 0.f;  // a real signal's bins 0 and M are real
#pragma unroll
    for (int i = 0; i < 4; i++)
        v[4 * I + i] =
            cscale(unsplit_bin(now.p[i], now.q[i], cmul(now.h[i], lo)), I == 0 && i == 0 && edge ? we : wi);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (I < 7)
        unsplit_points<STEP, I + 1>(v, nx, up, down, hi, lo, edge, we, wi);
}

// C2R pass 1: the reverse split on loading, then the column pass.  Point
// k = n1 N2 + n2 needs bins k and M - k: the columns of a tile and their
// mirror images, which the mirrored tile reads as well: tiles run in such
// pairs, and all of a transform on one XCD while there are 8 to deal, so that
// the second reading finds the bins in that XCD's L2.
template <int L1, int L2, int T>
__global__ __launch_bounds__((Wide<L1, T>::WG), WIDE_WAVES) void k_unsplit_cols(
    const cf* __restrict__ in, cf* __restrict__ ws, const cf* __restrict__ rows, const cf* __restrict__ tlo,
    const cf* __restrict__ thi, const cf* __restrict__ rlo, const cf* __restrict__ rhi, int64_t batch, float we, float wi)
{
    using W = Wide<L1, T>;
    constexpr int N1 = 1 << L1, N2 = 1 << L2, PER = N2 / T, TPT = W::TPT;
    constexpr int64_t M = int64_t(1) << (L1 + L2);
    static_assert(TPT * N2 % 1024 == 0, "the low twiddle index is the same for all of a thread's points");
    __shared__ float lds[col_plane<L1, T>()];
    __shared__ cf twl[64 + (M >> 10)];
    const int tid = threadIdx.x, c = tid & (T - 1), t = tid / T;
    const idx::Tile at = idx::xcd_deal_tile(blockIdx.x, batch, PER);
    const int64_t b = at.b;
    const int nb = (int)(at.tile & 1 ? PER - 1 - (at.tile >> 1) : at.tile >> 1), k0 = t * N2 + nb * T + c;
    col_tables<L1, L2, T>(twl, tlo, thi, tid);
    const cf* x = in + b * (M + 1);
    const cf lo = rlo[k0 & 1023];
    const cf* hi = rhi + (k0 >> 10);
    cf v[32];
    Unsplit<TPT * N2, 0> first;
    first.load(x + k0, x + M - k0, hi);
    unsplit_points<TPT * N2>(v, first, x + k0, x + M - k0, hi, lo, k0 == 0, we, wi);
    cf w4[4];
    wide_run<L1, +1, T>(v, t, rows, lds + c, w4);
    col_twiddle<L1, L2, +1>(v, twl, nb * T + c, t);
    col_store<L1, T>(v, lds, ws + (b * PER + nb) * (T * N1), tid);
}

// fn(integral_constant<int, T>) with the tile width T for `count` transforms.
// Nontemporal passes keep tiles of 16: half lines would cross the memory side
// twice.  The short last chunk of a stream (one transform of 2^20: 64 tiles) runs
// with them too (25 transforms of 2^20 take 157 us, 33 211, 35 217).
template <bool NT, class F>
hipError_t with_tile(int64_t count, F fn)
{
    if constexpr (!NT)
        if (narrow_tiles(count))
            return fn(std::integral_constant<int, 8>{});
    return fn(std::integral_constant<int, 16>{});
}

// Pass 2 in place: the axis pass of stride N1 over batch N1 transforms.
template <int L1, int L2, int S, bool NT, bool W>
hipError_t launch_rows(cf* io, const void* rows2, int64_t batch, float scale, hipStream_t stream)
{
    const cf* rows = static_cast<const cf*>(rows2);
    if constexpr (wide_len(L2, W))
        return with_tile<NT>(batch << L1, [&](auto tc) {
            constexpr int T = decltype(tc)::value;
            return launch_kernel((k_fourstep2_wide<L1, L2, S, NT, T>), dim3((unsigned)(batch * ((1 << L1) / T))),
                                 dim3(Wide<L2, T>::WG), 0, stream, io, rows, batch << L1, scale);
        });
    else
        return launch_kernel((k_fourstep2<L1, L2, S, NT>), dim3((unsigned)(batch * ((1 << L1) / TILE))), dim3(axis_wg<L2>()), 0, stream, io, rows,
                             batch << L1, scale);
}

// Pass 1.
template <int L1, int L2, int S, bool NT, bool W>
hipError_t launch_cols(const cf* in, cf* out, const cf* rows1, const cf* tlo, const cf* thi, int64_t batch,
                       hipStream_t stream)
{
    if constexpr (wide_len(L1, W))
        return with_tile<NT>(batch << L2, [&](auto tc) {
            constexpr int T = decltype(tc)::value;
            return launch_kernel((k_fourstep1_wide<L1, L2, S, NT, T>), dim3((unsigned)(batch * ((1 << L2) / T))),
                                 dim3(Wide<L1, T>::WG), 0, stream, in, out, rows1, tlo, thi);
        });
    else
        return launch_kernel((k_fourstep1<L1, L2, S, NT>), dim3((unsigned)(batch * ((1 << L2) / TILE))),
                             dim3(TILE * ((1 << L1) >> inner_e(L1))), 0, stream, in, out, rows1, tlo, thi);
}

// Both passes over `batch` transforms.  NTC: the column pass reads
// nontemporally (it stores plainly); NTR: the row pass reads and writes so.
template <int L1, int L2, int S, bool NTC, bool NTR, bool W>
hipError_t launch_passes(const cf* in, cf* out, const cf* rows1, const cf* rows2, const cf* tlo, const cf* thi,
                         int64_t batch, float scale, hipStream_t stream)
{
    const hipError_t e = launch_cols<L1, L2, S, NTC, W>(in, out, rows1, tlo, thi, batch, stream);
    return e == hipSuccess ? launch_rows<L1, L2, S, NTR, W>(out, rows2, batch, scale, stream) : e;
}

// Streams run chunk by chunk (stream.hpp): the row pass reads what the
// column pass left in the memory-side cache.  MI355X at 512 MiB, whole batch
// and plain accesses -> this: 2^15 427 -> 351 us, 2^16 437 -> 350, 2^17
// 438 -> 349, 2^18 444 -> 348, 2^19 448 -> 366, 2^20 446 -> 377; at 256 MiB 2^16
// 221 -> 176 (nontemporal accesses alone).
// As the last axis of a multidimensional plan (feeds) the row pass of one
// chunk stores plainly, for the axis pass that follows: nontemporal -> plain,
// 32 x 65536 at 144 MiB 169 -> 151 us (157 before chunks), at 512 MiB 567 -> 506.
template <int L1, int L2, int S, bool W>
hipError_t launch_fourstep(const void* in, void* out, const void* rows1, const void* rows2, const void* tlo,
                           const void* thi, int64_t batch, float scale, bool feeds, hipStream_t stream)
{
    const cf *src = static_cast<const cf*>(in), *lo = static_cast<const cf*>(tlo), *hi = static_cast<const cf*>(thi);
    const cf *r1 = static_cast<const cf*>(rows1), *r2 = static_cast<const cf*>(rows2);
    cf* dst = static_cast<cf*>(out);
    constexpr int64_t EACH = int64_t(sizeof(cf)) << (L1 + L2);
    if (!is_stream(batch * EACH))
        return launch_passes<L1, L2, S, false, false, W>(src, dst, r1, r2, lo, hi, batch, scale, stream);
    if (feeds)
        return launch_passes<L1, L2, S, true, false, W>(src, dst, r1, r2, lo, hi, batch, scale, stream);
    const int64_t per = chunk_units(EACH);
    for (int64_t b = 0; b < batch; b += per) {
        const int64_t nb = batch - b < per ? batch - b : per;
        const hipError_t e = launch_passes<L1, L2, S, true, true, W>(src + (b << (L1 + L2)), dst + (b << (L1 + L2)), r1,
                                                                  r2, lo, hi, nb, scale, stream);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// Transforms of M points in a chunk: half as many as the complex four-step
// takes, because R2C keeps its bins in the cache beside its workspace, and C2R
// reads its bins twice.  MI355X, n = 2^20, 256 MiB of reals, 256 against
// 128 MiB chunks: R2C 272 -> 209 us, C2R 229 -> 214.
constexpr int64_t real_chunk(int64_t m) { return chunk_units(2 * m * (int64_t)sizeof(cf)); }

// Real input, M = 2^(L1 + L2): R2C through `ws`, which holds one chunk (the
// whole batch unless it is a stream) and is used again by every chunk; C2R
// needs no workspace (column pass into `out`, row pass in place).
template <int L1, int L2, bool W>
hipError_t launch_r2c(const void* in, void* out, void* ws, const RealTables& t, int64_t batch, float we, float wi,
                      hipStream_t stream)
{
    constexpr int64_t M = int64_t(1) << (L1 + L2);
    const cf *rows1 = static_cast<const cf*>(wide_len(L1, W) ? t.wide1 : t.rows1), *lo = static_cast<const cf*>(t.tlo),
             *hi = static_cast<const cf*>(t.thi);
    const bool big = is_stream(batch * M * (int64_t)sizeof(cf));
    const int64_t per = big ? real_chunk(M) : batch;
    for (int64_t b = 0; b < batch; b += per) {
        const int64_t nb = batch - b < per ? batch - b : per;
        const cf* src = static_cast<const cf*>(in) + b * M;
        hipError_t e = big ? launch_cols<L1, L2, -1, true, W>(src, static_cast<cf*>(ws), rows1, lo, hi, nb, stream)
                           : launch_cols<L1, L2, -1, false, W>(src, static_cast<cf*>(ws), rows1, lo, hi, nb, stream);
        if (e == hipSuccess)
            e = with_tile<false>(nb << (L1 - 1), [&](auto tc) {
                constexpr int T = 2 * decltype(tc)::value;
                return launch_kernel((k_rows_split<L1, L2, T>), dim3((unsigned)(nb * ((1 << L1) / T))),
                                     dim3(Wide<L2, T>::WG), 0, stream, static_cast<const cf*>(ws),
                                     static_cast<cf*>(out) + b * (M + 1), static_cast<const cf*>(t.wide2),
                                     static_cast<const cf*>(t.rlo), static_cast<const cf*>(t.rhi), nb, we, wi);
            });
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

template <int L1, int L2, bool W>
hipError_t launch_c2r(const void* in, void* out, const RealTables& t, int64_t batch, float we, float wi,
                      hipStream_t stream)
{
    constexpr int64_t M = int64_t(1) << (L1 + L2);
    const bool big = is_stream(batch * M * (int64_t)sizeof(cf));
    const int64_t per = big ? real_chunk(M) : batch;
    for (int64_t b = 0; b < batch; b += per) {
        const int64_t nb = batch - b < per ? batch - b : per;
        cf* dst = static_cast<cf*>(out) + b * M;
        hipError_t e = with_tile<false>(nb << L2, [&](auto tc) {
            constexpr int T = decltype(tc)::value;
            return launch_kernel((k_unsplit_cols<L1, L2, T>), dim3((unsigned)(nb * ((1 << L2) / T))),
                                 dim3(Wide<L1, T>::WG), 0, stream, static_cast<const cf*>(in) + b * (M + 1), dst,
                                 static_cast<const cf*>(t.wide1), static_cast<const cf*>(t.tlo),
                                 static_cast<const cf*>(t.thi), static_cast<const cf*>(t.rlo),
                                 static_cast<const cf*>(t.rhi), nb, we, wi);
        });
        if (e == hipSuccess)
            e = big ? launch_rows<L1, L2, +1, true, W>(dst, t.rows2, nb, 1.f, stream)
                    : launch_rows<L1, L2, +1, false, W>(dst, t.rows2, nb, 1.f, stream);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// log2 of the points per thread of an inner transform, and the bytes of the
// column pass's twiddle tables in LDS.
constexpr int fs_e(int Li, bool W) { return wide_len(Li, W) ? WIDE_E : inner_e(Li); }

constexpr int fs_tw(int L) { return tw3_in_lds(L) ? (64 + (1 << (L - 10))) * (int)sizeof(cf) : (int)sizeof(cf); }

// Pass shapes as the launches above choose them: an inner transform of 2^Li in
// tiles of 8 where narrow_tiles(count) and not NT, else of 16.
template <int Li, bool W>
PassShape inner_shape(bool nt, int64_t count, bool cols, int tw)
{
    if constexpr (wide_len(Li, W)) {
        const bool narrow = !nt && narrow_tiles(count);
        const int plane = cols ? (narrow ? col_plane<Li, 8>() : col_plane<Li, 16>())
                               : (narrow ? Wide<Li, 8>::PLANE : Wide<Li, 16>::PLANE);
        return PassShape{WIDE_E, narrow ? 8 : 16, narrow ? Wide<Li, 8>::WG : Wide<Li, 16>::WG, plane * (int)sizeof(float) + tw};
    } else {
        constexpr int E = inner_e(Li);
        return PassShape{E, TILE, TILE * ((1 << Li) >> E), TILE * stage_stride<Li, E>() * (int)sizeof(cf) + tw};
    }
}

template <int L1, int L2, bool W>
PassShape pass_shape(FsPass pass, int64_t batch)
{
    constexpr int64_t M = int64_t(1) << (L1 + L2);
    const bool nt = is_stream(batch * M * (int64_t)sizeof(cf));
    const int64_t chunk = fs_ws_transforms(M, batch);  // of real input
    switch (pass) {
    case kFsCols: return inner_shape<L1, W>(nt, batch << L2, true, fs_tw(L1 + L2));
    case kFsRows: return inner_shape<L2, W>(nt, batch << L1, false, 0);
    case kFsSplitRows: {
        const bool narrow = narrow_tiles(chunk << (L1 - 1));
        return narrow ? PassShape{WIDE_E, 16, Wide<L2, 16>::WG, (Wide<L2, 16>::PLANE + 16) * (int)sizeof(float)}
                      : PassShape{WIDE_E, 32, Wide<L2, 32>::WG, (Wide<L2, 32>::PLANE + 32) * (int)sizeof(float)};
    }
    default: return inner_shape<L1, true>(false, chunk << L2, true, fs_tw(L1 + L2));
    }
}

struct RealFns {
    LaunchFsR2C r2c;
    LaunchFsC2R c2r;
};

// Half lengths of the real-input plans above 2^15.
template <int L1, int L2, bool W>
constexpr RealFns real_fns()
{
    if constexpr (L1 + L2 >= 15)
        return RealFns{&launch_r2c<L1, L2, W>, &launch_c2r<L1, L2, W>};
    else
        return RealFns{nullptr, nullptr};
}

template <int L, bool W = false>
void add_len()
{
    constexpr int L1 = (L + 1) / 2, L2 = L / 2;
    constexpr int E1 = fs_e(L1, W), E2 = fs_e(L2, W);
    const FourStep fs{L, L1, L2, E1, E2, Layout2<L1, E1>::rows_total(), Layout2<L2, E2>::rows_total(),
                      &launch_fourstep<L1, L2, -1, W>, &launch_fourstep<L1, L2, +1, W>, &pass_shape<L1, L2, W>,
                      real_fns<L1, L2, W>().r2c, real_fns<L1, L2, W>().c2r, W};
    register_fourstep(fs);
}

struct FourStepRegistrar {
    FourStepRegistrar()
    {
        add_len<12>();
        add_len<13>();
        add_len<14>();
        add_len<15>();
        add_len<15, true>();
        add_len<16>();
        add_len<16, true>();
        add_len<17>();
        add_len<17, true>();
        add_len<18>();
        add_len<19>();
        add_len<20>();
    }
};
FourStepRegistrar fourstep_registrar;

}  // namespace

// Transforms of M points in R2C's workspace: one chunk of a stream, or all.
int64_t fs_ws_transforms(int64_t m, int64_t batch)
{
    return is_stream(batch * m * (int64_t)sizeof(cf)) && real_chunk(m) < batch ? real_chunk(m) : batch;
}

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
