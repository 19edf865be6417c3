// Kernels off the inference hot path: the feedback quantizer (fp64 matrix instructions: the step before the path, and a third of
// a reconstruction iteration), and, one thread per element or output and written for clarity, unpacking, W_F, the read-only
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

// ------------------------------------------------------------------ feedback quantizer (fp64)

__device__ __forceinline__ double half_bits_to_double(uint16_t h) { return (double)__builtin_bit_cast(half_t, h); }

// double -> fp16 bits, round to nearest even, done on integers so that no intermediate fp32
// rounding can occur.  Input is finite and non-negative here, or negative for the zero point.
__device__ uint16_t double_to_half_bits(double d)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, d);
    const uint16_t sign = (uint16_t)((u >> 48) & 0x8000u);
    const int e = (int)((u >> 52) & 0x7ff) - 1023;           // unbiased exponent
    const uint64_t man = (u & 0xFFFFFFFFFFFFFull) | (1ull << 52);
    if (((u >> 52) & 0x7ff) == 0) return sign;               // zero / fp64 subnormal
    if (e >= 16) return sign | 0x7c00u;                      // overflow (callers never get here with inf/nan)
    if (e < -25) return sign;                                // below half of the smallest subnormal
    // value = man * 2^(e-52).  fp16 keeps bits down to 2^(max(e,-14) - 10).
    const int drop = 52 - 10 + (e < -14 ? -14 - e : 0);      // low bits of man to round away
    uint64_t keep = man >> drop;
    const uint64_t rem = man & ((1ull << drop) - 1), half = 1ull << (drop - 1);
    if (rem > half || (rem == half && (keep & 1))) keep += 1;
    // keep is now in units of the fp16 ulp at this exponent; re-encode (carry handled by addition)
    if (e < -14) return sign | (uint16_t)keep;               // subnormal (or rounds up into the first normal)
    const uint32_t bits = ((uint32_t)(e + 15) << 10) + (uint32_t)(keep - 1024);
    return bits >= 0x7c00u ? (sign | 0x7c00u) : (sign | (uint16_t)bits);
}

// A double from the lane that the data-parallel control word names (quad permutations, row mirrors).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// The 32-bit word of lane V of the lane's quad.
template <int V>
__device__ __forceinline__ uint32_t quad_broadcast(uint32_t w)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, V * 0x55, 0xF, 0xF, true);
}
template <int V>
__device__ __forceinline__ double quad_broadcast(double v) { return dpp_move<V * 0x55>(v); }

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef uint32_t uint4v_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t bounded_buffer(const void *p, long bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ half8_t load_half8(__amdgpu_buffer_rsrc_t b, int off)
{
    return __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
}

// The feedback quantizer of one group of 128 input features and 64 consecutive rows per block, 16 rows per wave.
//
// Sigma = B A is a contraction over the r taps in fp64 and runs on the fp64 matrix instruction (16 rows x 16 columns x
// 4 taps, 2048 flop; 75 TFLOP/s measured on this card, no more than the vector unit has in fp64, but an operand register
// serves sixteen multiply-adds instead of one).  Lane (c = lane % 16, q = lane / 16) supplies tap q of an operand and
// the instruction only needs both operands to agree on which tap that is: of 32 taps, lane group q takes 8 q .. 8 q + 7,
// one per instruction, so a lane's eight taps of its row of Bt are one 16-byte load.  The block converts its tile of At
// (32 taps x 128 features) to fp64 once, in LDS: converted by every wave for itself, the conversions were a tenth of the
// loop.  Column tile t (0..7) is given the features k = 8 c + t of the group: what a lane ends up holding - rows 4 v + q
// (v = 0..3), columns 8 c .. 8 c + 7 - are 16 contiguous bytes of four rows of W, of four rows of Delta_F, and one packed
// INT4 word per row.  The extremes of a group are eight values of a lane and a reduction over its row of 16 lanes: no LDS.
// Bound: the fp64 unit (matrix and vector instructions share it: the two parts' times add).  11008 x 4096, us at r = 0 /
// 32 / 64 / 128: INT3 41 / 89 / 133 / 219, INT4 35 / 79 / 121 / 205; 77 of the 121 are the matrix instructions at their
// peak.  One thread per column with Bt broadcast from LDS - a conversion and an LDS read per multiply-add - took 415
// (INT3, r = 64) and, with Delta_F, 184 at 4096 x 4096 where this takes 63.  Four waves per SIMD: three or two are 3 % and
// 8 % slower.
//
// fp64 throughout, no contraction left to the compiler.  The products of two fp16 values have 22 significant bits, so
// the order of the taps matters only where a sum needs more than 53 bits.
// With DELTA the kernel also writes what the reconstruction step needs from the same registers: Delta_F =
// (W - Sigma) - s (q - z), times `gain`, as fp16 in both orientations (D16 [N][K]; Dt16 [K][ldt] with columns
// N..ldt-1 zero, ldt a multiple of 64), the transposed copy through LDS as whole 128-byte row pieces.
constexpr int kQuantWaves = 4;
constexpr int kQuantRows = 16 * kQuantWaves;
constexpr int kQuantTaps = 32;      // taps per tile of At

template <int BITS, bool DELTA>
__global__ __launch_bounds__(64 * kQuantWaves, 4) void fbq_quantize_kernel(const uint16_t *__restrict__ W, const uint16_t *__restrict__ At,
                                                                        const uint16_t *__restrict__ Bt, uint32_t *__restrict__ qw,
                                                                        uint16_t *__restrict__ scales, uint16_t *__restrict__ zeros, int N,
                                                                        int K, int r, int row_words, uint16_t *__restrict__ D16,
                                                                        uint16_t *__restrict__ Dt16, int ldt, float gain)
{
#pragma clang fp contract(off)
    // the tile of At in fp64, [tap][column tile][c]; afterwards Delta_F by column, [feature][row], rows 144 bytes apart
    __shared__ union { double taps[kQuantTaps][8][16]; uint16_t turn[kGroup][kQuantRows + 8]; } lds;
    constexpr int qmax = (1 << BITS) - 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 15, q = lane >> 4;
    const int g = blockIdx.x, G = K / kGroup;
    const int nb = blockIdx.y * kQuantRows, n0 = nb + 16 * wave;       // the block's first row, the wave's
    const int rows = min(16, N - n0);                                   // may be <= 0: such a wave computes zeros and stores nothing

    // The wave's rows of W and Bt through descriptors that end with row N - 1: rows past it read as zeros.
    const __amdgpu_buffer_rsrc_t wbuf = bounded_buffer(W + (size_t)min(n0, N - 1) * K, rows > 0 ? (long)rows * K * 2 : 0);
    const __amdgpu_buffer_rsrc_t bbuf = bounded_buffer(Bt + (size_t)min(n0, N - 1) * r, rows > 0 ? (long)rows * r * 2 : 0);
    const __amdgpu_buffer_rsrc_t abuf = bounded_buffer(At, (long)r * K * 2);
    half8_t w[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) w[v] = load_half8(wbuf, ((4 * v + q) * K + g * kGroup + 8 * c) * 2);

    double4_t R[8];                                                     // Sigma first: R[t][v] is row 4 v + q, column 8 c + t
#pragma unroll
    for (int t = 0; t < 8; ++t) R[t] = double4_t{0.0, 0.0, 0.0, 0.0};
    constexpr int kNowhere = 0x7FFFFFF0;                                // beyond every buffer: taps past r are zeros in both operands
    // thread i converts pieces i and i + 256 of the block's 32 x 128 tile of At: piece p is features 8 (p % 16) .. + 7 of tap p / 16
    constexpr int kPieces = kQuantTaps * 16 / (64 * kQuantWaves);
    half8_t a8[kPieces], b8;
    auto fetch = [&](int j0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int p = i * 64 * kQuantWaves + threadIdx.x, j = j0 + (p >> 4);
            a8[i] = load_half8(abuf, j < r ? (j * K + g * kGroup + 8 * (p & 15)) * 2 : kNowhere);
        }
        const int j = j0 + 8 * q;                                       // r is a multiple of 8: all of a lane's taps or none
        b8 = load_half8(bbuf, j < r ? (c * r + j) * 2 : kNowhere);
    };
    if (r > 0) fetch(0);
    for (int j0 = 0; j0 < r; j0 += kQuantTaps) {
        if (j0 > 0) __syncthreads();                                    // everybody is done with the tile before
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int p = i * 64 * kQuantWaves + threadIdx.x;
#pragma unroll
            for (int t = 0; t < 8; ++t) lds.taps[p >> 4][t][p & 15] = (double)(float)a8[i][t];
        }
        const half8_t b = b8;
        __syncthreads();
        if (j0 + kQuantTaps < r) fetch(j0 + kQuantTaps);
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int t = 0; t < 8; ++t)
                R[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(float)b[s], lds.taps[8 * q + s][t][c], R[t], 0, 0, 0);
    }

    // feedback: quantize R = W - Sigma.  Extremes of each row's group: the lane's eight values, then its row of 16 lanes.
    // Lane c ends up with those of row 4 (c % 4) + q: the first two steps hand the other rows' values to the lanes that
    // go on with them, so that the four rows cost 2 + 1 + 1 + 1 steps instead of 16.
    double mn[4], mx[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int t = 0; t < 8; ++t) R[t][v] = (double)(float)w[v][t] - R[t][v];
        mn[v] = mx[v] = R[0][v];
#pragma unroll
        for (int t = 1; t < 8; ++t) { mn[v] = fmin(mn[v], R[t][v]); mx[v] = fmax(mx[v], R[t][v]); }
    }
    double lo, hi;
    {
        const bool odd = c & 1, upper = c & 2;
        const double lo0 = fmin(odd ? mn[1] : mn[0], dpp_move<0xB1>(odd ? mn[0] : mn[1]));   // neighbours: row 0 or 1 ...
        const double hi0 = fmax(odd ? mx[1] : mx[0], dpp_move<0xB1>(odd ? mx[0] : mx[1]));
        const double lo1 = fmin(odd ? mn[3] : mn[2], dpp_move<0xB1>(odd ? mn[2] : mn[3]));   // ... and 2 or 3
        const double hi1 = fmax(odd ? mx[3] : mx[2], dpp_move<0xB1>(odd ? mx[2] : mx[3]));
        lo = fmin(upper ? lo1 : lo0, dpp_move<0x4E>(upper ? lo0 : lo1));                     // pairs of a quad: one row
        hi = fmax(upper ? hi1 : hi0, dpp_move<0x4E>(upper ? hi0 : hi1));
        lo = fmin(lo, dpp_move<0x124>(lo)); hi = fmax(hi, dpp_move<0x124>(hi));              // the four quads: row rotated by 4, by 8
        lo = fmin(lo, dpp_move<0x128>(lo)); hi = fmax(hi, dpp_move<0x128>(hi));
    }
    // Scale and zero: every quad's lane c % 4 = v searches for row 4 v + q, the quad then shares the four results.
    uint32_t sz;
    double inv;                                                                 // 1 / scale, correctly rounded
    {
        const int mine = c & 3;
        double s = (hi - lo) / (double)qmax;
        if (!(s > 0.0)) s = 1.0;
        uint16_t s16 = double_to_half_bits(s);
        if (s16 < 0x0400u) s16 = 0x0400u;
        // (extremes that are infinite or NaN never meet the condition below, whatever the scale: straight to the last one)
        if (!(__builtin_fabs(lo) < __builtin_inf() && __builtin_fabs(hi) < __builtin_inf()) && s16 < 0x7bffu) s16 = 0x7bffu;
        uint16_t z16;
        for (;;) {
            const double sd = half_bits_to_double(s16);
            z16 = double_to_half_bits(-lo / sd);
            const double zd = half_bits_to_double(z16);
            if ((lo / sd + zd >= -0.5 && hi / sd + zd <= (double)qmax + 0.5) || s16 >= 0x7bffu) break;
            s16 += 1;
        }
        sz = (uint32_t)s16 | ((uint32_t)z16 << 16);
        inv = 1.0 / half_bits_to_double(s16);
        const int row = 4 * mine + q;
        if (c < 4 && row < rows) {
            scales[(size_t)(n0 + row) * G + g] = s16;
            zeros[(size_t)(n0 + row) * G + g] = z16;
        }
    }
    const uint32_t szv[4] = {quad_broadcast<0>(sz), quad_broadcast<1>(sz), quad_broadcast<2>(sz), quad_broadcast<3>(sz)};
    const double invv[4] = {quad_broadcast<0>(inv), quad_broadcast<1>(inv), quad_broadcast<2>(inv), quad_broadcast<3>(inv)};
    // R / s costs eleven fp64 instructions, R * inv and one correction three, and the result is the same number: with
    // u = R * inv the residual e = R - u s is exact, u + e * inv is off the quotient by about 2^-105 of it before its one
    // rounding, and a quotient of a 53-bit number by an 11-bit one is never that close to the middle between two fp64
    // numbers (it is at least 2^-12 of a last place away from it, and the middle itself would need 54 bits of R).  Only an
    // infinite scale (weights that are infinite) is divided by as before.
    const bool divide = __any((sz & 0xFFFFu) >= 0x7c00u);

    if (DELTA) __syncthreads();                                                 // everybody is done with the tile of At
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = 4 * v + q;
        const double sd = half_bits_to_double((uint16_t)szv[v]), zd = half_bits_to_double((uint16_t)(szv[v] >> 16));
        uint32_t code[8];
        half8_t d8;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            double u;
            if (divide) u = R[t][v] / sd;
            else { u = R[t][v] * invv[v]; u = __builtin_fma(__builtin_fma(-u, sd, R[t][v]), invv[v], u); }
            double x = rint(u + zd);                                             // ties to even
            x = fmin(fmax(x, 0.0), (double)qmax);
            code[t] = (uint32_t)x;
            if (DELTA) d8[t] = (_Float16)(float)((double)gain * (R[t][v] - sd * (x - zd)));   // Delta_F (Sec. 4.2)
        }
        if (DELTA) {
            if (row < rows) *reinterpret_cast<half8_t *>(D16 + (size_t)(n0 + row) * K + g * kGroup + 8 * c) = d8;
#pragma unroll
            for (int t = 0; t < 8; ++t) lds.turn[8 * c + t][16 * wave + row] = row < rows ? __builtin_bit_cast(uint16_t, (_Float16)d8[t]) : (uint16_t)0;
        }
        if constexpr (BITS == 4) {                                               // the lane's eight codes are word c of the group
            uint32_t word = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t) word |= code[t] << (4 * t);
            if (row < rows) qw[(size_t)(n0 + row) * row_words + g * 16 + c] = word;
        } else {
            // 32 codes, three words: a quad.  Lane i of the quad holds codes 8 i .. 8 i + 7, 24 bits of the stream of codes; word i
            // is 15 bits of the stream from 30 i on, 15 more in the upper half, and one bit each of codes 30 and 31.
            const int i = c & 3;
            uint32_t mine = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t) mine |= code[t] << (3 * t);
            const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)mine, 0xF9, 0xF, 0xF, true);   // lanes 1, 2, 3, 3 of the quad
            const uint32_t last = quad_broadcast<3>(mine) >> 18;                                          // codes 30 and 31
            const uint32_t b30 = (uint32_t)((((uint64_t)next << 24) | mine) >> (6 * i));
            const uint32_t word = (b30 & 0x7FFFu) | ((b30 & 0x3FFF8000u) << 1) | ((last >> i) & 1u) << 15 | ((last >> (3 + i)) & 1u) << 31;
            if (i < 3 && row < rows) qw[(size_t)(n0 + row) * row_words + g * 12 + (c >> 2) * 3 + i] = word;
        }
    }
    if (DELTA) {
        __syncthreads();
        // 128 features x 64 rows: eight lanes per feature write its 128 bytes, eight features per instruction
#pragma unroll
        for (int it = 0; it < kGroup * kQuantRows / 8 / (64 * kQuantWaves); ++it) {
            const int piece = it * 64 * kQuantWaves + threadIdx.x, col = piece >> 3, part = piece & 7;
            *reinterpret_cast<uint4 *>(Dt16 + (size_t)(g * kGroup + col) * ldt + nb + 8 * part) = *reinterpret_cast<const uint4 *>(&lds.turn[col][8 * part]);
        }
    }
}

hipError_t launch_quantize(const fbq_desc &d, const uint16_t *W, const uint16_t *At, const uint16_t *Bt, uint32_t *qw,
                           uint16_t *scales, uint16_t *zeros, hipStream_t stream, uint16_t *D16, uint16_t *Dt16, int ldt, float gain)
{
    const dim3 grid(d.K / kGroup, ceil_div(d.N, kQuantRows)), block(64 * kQuantWaves);
    const int words = (int)row_words(d.K, d.bits);
#define FBQ_QUANT(B, D) hipLaunchKernelGGL((fbq_quantize_kernel<B, D>), grid, block, 0, stream, W, At, Bt, qw, scales, zeros, d.N, d.K, d.r, words, D16, Dt16, ldt, gain)
    if (d.bits == 4) { if (D16) FBQ_QUANT(4, true); else FBQ_QUANT(4, false); }
    else { if (D16) FBQ_QUANT(3, true); else FBQ_QUANT(3, false); }
#undef FBQ_QUANT
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
