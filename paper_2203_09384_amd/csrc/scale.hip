// out = in * factor[0], complex by a real scalar in device memory: the
// backward of the fused loss, which scales the saved gradient.  A stream, 8
// bytes read and 8 written per point, bound by HBM: 64 KiB to GiB, one
// 16-byte vector per thread.  The gradient is read plainly (the forward left
// it in the memory-side cache) and a stream's output stored nontemporally.
// MI355X, 256 MiB: torch's product 96 us; forward + backward at N = 2048
// 231 -> 216 us with this kernel, 195 with the forward storing plainly.
#include "device_fft.hpp"
#include "launch.hpp"
#include "stream.hpp"

namespace mifft {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int SCALE_WG = 256;

// (a + i b)(f + 0 i), with the zero products, so that infinities and NaN
// come out as in a complex product.
template <bool NT>
__global__ __launch_bounds__(SCALE_WG) void k_scale(const float* __restrict__ in, const float* __restrict__ factor,
                                                    float* __restrict__ out, int64_t points)
{
    const float f = *factor;
    const int64_t i = (int64_t)blockIdx.x * SCALE_WG + threadIdx.x;
    const gv4* src = reinterpret_cast<const gv4*>(in) + i;
    gv4* dst = reinterpret_cast<gv4*>(out) + i;
    if (2 * i + 1 < points) {
        const v4f v = *src;
        const v4f o{v.x * f - v.y * 0.f, v.x * 0.f + v.y * f, v.z * f - v.w * 0.f, v.z * 0.f + v.w * f};
        if constexpr (NT)
            __builtin_nontemporal_store(o, dst);
        else
            *dst = o;
    } else if (2 * i < points) {
        const float a = in[4 * i], b = in[4 * i + 1];
        out[4 * i] = a * f - b * 0.f;
        out[4 * i + 1] = a * 0.f + b * f;
    }
}

}  // namespace
}  // namespace mifft

// For the binding: `points` complex values, 8-byte aligned, in and out apart.
extern "C" int mifft_scale_c32(const void* in, const float* factor, void* out, int64_t points, void* stream)
{
    using namespace mifft;
    const int64_t blocks = ((points + 1) / 2 + SCALE_WG - 1) / SCALE_WG;
    if (points < 1 || blocks > 0x7fffffffLL)
        return -1;
    const hipError_t e =
        launch_kernel(is_stream(points * 8) ? k_scale<true> : k_scale<false>, dim3((unsigned)blocks), dim3(SCALE_WG),
                      0, static_cast<hipStream_t>(stream), static_cast<const float*>(in), factor,
                      static_cast<float*>(out), points);
    return e == hipSuccess ? 0 : -1;
}
