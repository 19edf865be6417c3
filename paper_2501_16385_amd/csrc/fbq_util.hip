// Kernels off the inference hot path, one thread per element or output and written for clarity: unpacking, W_F, the read-only
// yardstick and the conventional sub-branch that the fused kernels are compared with.
#include <hip/hip_fp16.h>

#include "fbq_internal.h"

namespace fbq {

typedef _Float16 half_t;

// Code k of a packed row, assembled field by field from the device layout.
__device__ __forceinline__ uint32_t code_of_row(const uint32_t *row, int bits, int k)
{
    if (bits == 4) return (row[k >> 3] >> ((k & 7) * 4)) & 15u;
    const uint32_t *u = row + (k >> 5) * 3;
    const int j = k & 31;
    if (j == 30) return ((u[0] >> 15) & 1u) | (((u[1] >> 15) & 1u) << 1) | (((u[2] >> 15) & 1u) << 2);
    if (j == 31) return (u[0] >> 31) | ((u[1] >> 31) << 1) | ((u[2] >> 31) << 2);
    const int wd = j / 10, f = j % 10;
    const int sh = f < 5 ? 3 * f : 16 + 3 * (f - 5);
    return (u[wd] >> sh) & 7u;
}

__global__ __launch_bounds__(256) void fbq_unpack_kernel(const uint32_t *__restrict__ qw, uint8_t *__restrict__ codes,
                                                         int N, int K, int bits, int row_words)
{
    const int n = blockIdx.y;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (n < N && k < K) codes[(size_t)n * K + k] = (uint8_t)code_of_row(qw + (size_t)n * row_words, bits, k);
}

hipError_t launch_unpack(const fbq_desc &d, const uint32_t *qw, uint8_t *codes, hipStream_t stream)
{
    hipLaunchKernelGGL(fbq_unpack_kernel, dim3(ceil_div(d.K, 256), d.N), dim3(256), 0, stream, qw, codes, d.N, d.K, d.bits,
                       (int)row_words(d.K, d.bits));
    return hipGetLastError();
}

// W_F[n,k] = s*(q - z) + sum_j At[j,k] * Bt[n,j]   (Sec. 4.1: W_F = Q(W - Sigma) + Sigma), fp32.
__global__ __launch_bounds__(256) void fbq_reconstruct_kernel(const uint32_t *__restrict__ qw, const uint16_t *__restrict__ scales,
                                                              const uint16_t *__restrict__ zeros, const uint16_t *__restrict__ At,
                                                              const uint16_t *__restrict__ Bt, float *__restrict__ W_hat, int N,
                                                              int K, int r, int bits, int row_words)
{
    const int n = blockIdx.y;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (n >= N || k >= K) return;
    const int G = K / kGroup;
    const float s = (float)__builtin_bit_cast(half_t, scales[(size_t)n * G + k / kGroup]);
    const float z = (float)__builtin_bit_cast(half_t, zeros[(size_t)n * G + k / kGroup]);
    const float q = (float)code_of_row(qw + (size_t)n * row_words, bits, k);
    float sigma = 0.0f;
    for (int j = 0; j < r; ++j)
        sigma = fmaf((float)__builtin_bit_cast(half_t, At[(size_t)j * K + k]),
                     (float)__builtin_bit_cast(half_t, Bt[(size_t)n * r + j]), sigma);
    W_hat[(size_t)n * K + k] = s * (q - z) + sigma;
}

hipError_t launch_reconstruct(const fbq_desc &d, const uint32_t *qw, const uint16_t *scales, const uint16_t *zeros,
                              const uint16_t *At, const uint16_t *Bt, float *W_hat, hipStream_t stream)
{
    hipLaunchKernelGGL(fbq_reconstruct_kernel, dim3(ceil_div(d.K, 256), d.N), dim3(256), 0, stream, qw, scales, zeros, At, Bt,
                       W_hat, d.N, d.K, d.r, d.bits, (int)row_words(d.K, d.bits));
    return hipGetLastError();
}

// ------------------------------------------------------------------ read-stream yardstick

// Reads every 16-byte piece of a buffer once and writes nothing: what the memory system delivers to a
// launch of a given size, measured with the same launch protocol as the decode kernels, is the
// ceiling they are judged against beside the nominal HBM peak.  Eight loads per thread in flight.
__global__ __launch_bounds__(256) void fbq_read_stream_kernel(const uint4 *__restrict__ p, unsigned long long n16)
{
    constexpr int kUnroll = 8;
    unsigned long long i = ((unsigned long long)blockIdx.x * kUnroll) * 256 + threadIdx.x;
    const unsigned long long stride = (unsigned long long)gridDim.x * kUnroll * 256;
    for (; i < n16; i += stride) {
        uint4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const unsigned long long j = i + (unsigned long long)u * 256;
            v[u] = p[j < n16 ? j : n16 - 1];             // past the end: the last piece again, never out of bounds
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) asm volatile("" ::"v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));   // keeps the loads alive
    }
}

hipError_t launch_read_stream(const void *buf, size_t bytes, hipStream_t stream)
{
    const unsigned long long n16 = bytes / 16;
    const int blocks = (int)std::min<unsigned long long>(1024, (n16 + 2047) / 2048);
    hipLaunchKernelGGL(fbq_read_stream_kernel, dim3(blocks), dim3(256), 0, stream, (const uint4 *)buf, n16);
    return hipGetLastError();
}

// ------------------------------------------------------------------ conventional sub-branch (comparator)

// The arrangement the fused kernel replaces (Sec. 3.2, Fig. 4 left): after the quantized main path has written
// y, the sub-branch runs as launches of its own - t = x.A, rounded to fp16 as a stand-alone kernel's output is,
// then y += t.B, which reads y back and writes it again.  Plain kernels: this path exists to be measured against.

// t[m][j] = sum_k x[m][k] At[j][k]: one block per (column j, token m), 256 threads along K.
__global__ __launch_bounds__(256) void fbq_unfused_down_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ At,
                                                               uint16_t *__restrict__ t, int K, int r)
{
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    __shared__ float part[4];
    const int j = blockIdx.x, m = blockIdx.y, tid = threadIdx.x;
    const uint4 *xr = reinterpret_cast<const uint4 *>(x + (size_t)m * K), *ar = reinterpret_cast<const uint4 *>(At + (size_t)j * K);
    float acc = 0.0f;
    for (int i = tid; i < K / 8; i += 256) {
        const uint4 a = xr[i], b = ar[i];
        const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, aw[q]), __builtin_bit_cast(h2, bw[q]), acc, false);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((tid & 63) == 0) part[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) t[(size_t)m * r + j] = __builtin_bit_cast(uint16_t, (_Float16)(part[0] + part[1] + part[2] + part[3]));
}

// y[m][n] += sum_j t[m][j] Bt[n][j]: one thread per output, t of the token in LDS.
__global__ __launch_bounds__(256) void fbq_unfused_up_kernel(const uint16_t *__restrict__ t, const uint16_t *__restrict__ Bt,
                                                             uint16_t *__restrict__ y, int N, int r)
{
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    __shared__ uint32_t tl[kMaxRank / 2];
    const int m = blockIdx.y, n = blockIdx.x * 256 + threadIdx.x;
    for (int i = threadIdx.x; i < r / 2; i += 256) tl[i] = reinterpret_cast<const uint32_t *>(t + (size_t)m * r)[i];
    __syncthreads();
    if (n >= N) return;
    const uint4 *br = reinterpret_cast<const uint4 *>(Bt + (size_t)n * r);
    float acc = (float)__builtin_bit_cast(_Float16, y[(size_t)m * N + n]);
    for (int i = 0; i < r / 8; ++i) {
        const uint4 b = br[i];
        const uint32_t bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, tl[4 * i + q]), __builtin_bit_cast(h2, bw[q]), acc, false);
    }
    y[(size_t)m * N + n] = __builtin_bit_cast(uint16_t, (_Float16)acc);
}

hipError_t launch_unfused_branch(const LinearArgs &a, uint16_t *t, hipStream_t stream)
{
    hipLaunchKernelGGL(fbq_unfused_down_kernel, dim3(a.r, a.M), dim3(256), 0, stream, a.x, a.At, t, a.K, a.r);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fbq_unfused_up_kernel, dim3(ceil_div(a.N, 256), a.M), dim3(256), 0, stream, t, a.Bt, a.y, a.N, a.r);
    return hipGetLastError();
}

}  // namespace fbq
