// Blocked convolution on fp16 MFMA with two-term operands (conv_h2.h): the
// kernels over a converted filter, and the conversion.
#include "conv_h2.h"

namespace neo {
namespace conv_detail {

template hipError_t dispatch_h2<true, false>(const ConvConfig&, int, bool, const H2Args&, hipStream_t);

namespace {

__global__ __launch_bounds__(256) void h2_split_filter(const float* w, int KB, int steps, v8h* out, int* wexp) {
    const int k = blockIdx.x, kb = k >> 5, i = k & 31, k16 = k >> 4, li = k & 15;
    const bool real = k16 < KB;
    // element quad q of channel li in step f: float4 q * 16 + li of block (k16, f)
    const v4f* src = reinterpret_cast<const v4f*>(w) + (long)(real ? k16 : 0) * steps * 64 + li;
    __shared__ float red[4];
    float m = 0.f;
    if (real)
        for (long t = threadIdx.x; t < 4L * steps; t += 256) m = h2_max(src[(t >> 2) * 64 + (t & 3) * 16], m);
    m = h2_wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    const int e = h2_exponent(__float_as_uint(m), kH2TopAll);
    const unsigned limit = h2_key(h2_small(e));
    int small = 0;
    const float s2 = ldexpf(1.f, e + 11);
    for (long t = threadIdx.x; t < 2L * steps; t += 256) {
        const long f = t >> 1;
        const int g = (int)(t & 1);
        v4h h[2], l[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const v4f x = real ? src[f * 64 + (2 * g + q) * 16] : v4f{0.f, 0.f, 0.f, 0.f};
            h2_terms(x, s2, h[q], l[q]);
#pragma unroll
            for (int j = 0; j < 4; ++j) small += h2_key(x[j]) < limit ? 1 : 0;
        }
        v8h* dst = out + ((long)kb * steps + f) * 128 + g * 32 + i;
        dst[0] = h2_join(h[0], h[1]);
        dst[64] = h2_join(l[0], l[1]);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) small += __shfl_xor(small, d, 64);
    __shared__ int count[4];
    if ((threadIdx.x & 63) == 0) count[threadIdx.x >> 6] = small;
    __syncthreads();
    if (threadIdx.x == 0) wexp[k] = h2_channel(e, count[0] + count[1] + count[2] + count[3]);
}

}  // namespace

hipError_t launch_h2_split(const float* w, int KB, int steps, void* out, int* wexp, hipStream_t st) {
    hipLaunchKernelGGL(h2_split_filter, dim3((unsigned)(cdiv(KB, 2) * 32)), dim3(256), 0, st, w, KB, steps,
                       static_cast<v8h*>(out), wexp);
    return hipGetLastError();
}

}  // namespace conv_detail
}  // namespace neo
