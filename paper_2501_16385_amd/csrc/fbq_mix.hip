// The element-wise glue of a decoder layer: averaging a layer's result with another tensor, silu(gate) * up.  Launches of
// their own cost about 2.5 us each between launches that stream weights for 4 to 12; the averaging rides on the store of
// the decode kernels where they have an instance for it, the gate is one launch instead of two.  Step of four 7B-shaped decoder
// layers, r = 64, us: INT4, one sequence, 182 with eight launches a layer and 160 with five; INT3, eight sequences, 270 and 249.
#include <hip/hip_fp16.h>

#include "fbq_internal.h"

namespace fbq {

typedef _Float16 half_t;
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

// out = (with + y) / 2 as the decode kernels compute it
__global__ __launch_bounds__(256) void fbq_mix_kernel(const half_t *__restrict__ with, const half_t *__restrict__ y, half_t *__restrict__ out, size_t count)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    auto mix = [](half_t w, half_t v) __attribute__((always_inline)) { return (half_t)((float)v - ((float)v - (float)w) * 0.5f); };
    if (i + 8 <= count) {
        const half8_t w = *reinterpret_cast<const half8_t *>(with + i), v = *reinterpret_cast<const half8_t *>(y + i);
        half8_t o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = mix(w[e], v[e]);
        *reinterpret_cast<half8_t *>(out + i) = o;
    } else {
        for (size_t k = i; k < count; ++k) out[k] = mix(with[k], y[k]);
    }
}

__global__ __launch_bounds__(256) void fbq_silu_mul_kernel(const half_t *__restrict__ gate, const half_t *__restrict__ up, half_t *__restrict__ out, size_t count)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    auto act = [](half_t g, half_t u) __attribute__((always_inline)) {
        const float x = (float)g;
        const half_t s = (half_t)(x / (1.0f + expf(-x)));
        return (half_t)((float)s * (float)u);
    };
    if (i + 8 <= count) {
        const half8_t g = *reinterpret_cast<const half8_t *>(gate + i), u = *reinterpret_cast<const half8_t *>(up + i);
        half8_t o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = act(g[e], u[e]);
        *reinterpret_cast<half8_t *>(out + i) = o;
    } else {
        for (size_t k = i; k < count; ++k) out[k] = act(gate[k], up[k]);
    }
}

hipError_t launch_mix(const LinearArgs &a, hipStream_t stream)
{
    const size_t count = (size_t)a.M * a.N;
    hipLaunchKernelGGL(fbq_mix_kernel, dim3((unsigned)((count + 2047) / 2048)), dim3(256), 0, stream, (const half_t *)a.mix_with, (const half_t *)a.y,
                       (half_t *)a.mix_out, count);
    return hipGetLastError();
}

hipError_t launch_silu_mul(const void *gate, const void *up, void *out, size_t count, hipStream_t stream)
{
    hipLaunchKernelGGL(fbq_silu_mul_kernel, dim3((unsigned)((count + 2047) / 2048)), dim3(256), 0, stream, (const half_t *)gate,
                       (const half_t *)up, (half_t *)out, count);
    return hipGetLastError();
}

}  // namespace fbq
