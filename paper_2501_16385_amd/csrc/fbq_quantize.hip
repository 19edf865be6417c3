// The feedback quantizer Q(W - B A) (Sec. 4.1): the step before the path, and a sixth of a reconstruction iteration.
//
// Codes, scales and zeros are defined in 64 bits.  The kernel gets them from 32-bit sums with a bound on their error: Sigma = B A
// on the fp16 matrix instruction, extremes and codes in fp32.  Where the bound leaves open which fp16 number a scale or a zero
// rounds to, or which whole number a code rounds to, that row of the group is done again in fp64; so the result is that of
// fp64 throughout, and with weights as they come one row in 200 pays for it (r = 64; 1 in 70 at r = 200).
//
// Layout.  One block takes one group of 128 input features and one or two tiles of rows, 16 rows a wave.  Its tile of At is transposed
// into LDS as fp16, [feature][tap]; the features are the rows of the matrix product and the rows of W its columns, features dealt to the
// eight row tiles so that a lane (c = lane % 16, q = lane / 16) ends up with 32 consecutive features 32 q .. 32 q + 31 of row c: whole
// packed words (four of INT4, one unit of three of INT3), one scale and one zero, 64 bytes of W and of Delta_F, and extremes that
// are found in the lane but for two steps between lanes.
//
// What it takes, us, against the same in fp64 throughout (fp64 matrix instruction, a thirtieth of the fp16 rate): 11008 x 4096 INT3, r = 64,
// 124 -> 50; without a sub-branch 38 -> 27; INT4, r = 200, 335 -> 94; 4096 x 4096, r = 128, 79 -> 33.  Of the 50, 23 are the bytes at the rate of
// a large copy, about 15 getting At into LDS and out of it (without a sub-branch 27), 4 the rows in fp64.
// Weights that leave nearly every row open (groups far from zero beside their spread, |z| above 1024; values on half steps) take the attempt and the fp64 product of all rows:
// fp64 throughout / row by row / all sixteen of a wave at once, as now: 11008 x 4096 INT3, r = 64, 124 / 449 / 147, without a sub-branch 37 / 160 / 49; INT4, r = 200, 364 / 1255 / 441.
//
// With DELTA the kernel also writes what the reconstruction step needs from the same registers: Delta_F = (W - Sigma) - s (q - z), times
// `gain`, as fp16 (D16 [N][K]).  It is the fp16 number that fp64 gives: where the bound leaves two open, that element is done again.  Sigma is
// had more exactly for that (below); with the bound of the fp16 products as they are, eight elements in a hundred were open and a step took 233 us,
// now four in a thousand at the start and some two in a hundred after thousands of steps.
// A step with loss, us, fp64 throughout (Delta_F written in both orientations) / now: 4096 x 4096 INT4, r = 64, 182 / 173, without loss 104 / 92;
// 4096 x 11008, r = 64, without loss 298 / 243; 11008 x 4096, r = 200, 719 / 638; taps all of one size, 4096 x 4096, r = 128, without loss 149 / 161 (row by row 413).  What bounds
// the kernel (47 of the 173): vector instructions, about 2300 a tile of 16 rows.
// With a block a CU or less, a wave's chain of instructions bounds a step, and the rows and elements done again are its end.  Such grids go to fp64 as they are (IN64: no norms, no split of
// the taps, nothing done again), and the first tile's W and B are asked for with the taps.  The kernel / a step with loss, us, fp64 throughout / in 32 bits / now: 1000 x 1024, r = 64, 13.9 / 14.5 / 12.9 and
// 50.8 / 52.4 / 50.0; 2000 x 1024, r = 64, 15.0 / 15.8 / 14.5 and 54.1 / 56.4 / 54.0; 1024 x 1024, r = 200, 24.6 / 32.7 / 25.3 and 75.4 / 82.5 / 77.5.  With more blocks than CUs 32 bits win: 1500 x
// 1536, r = 128 (288 blocks), the kernel 25.5 against 29.6; 2048 x 2048, r = 64, 21.0 against 25.4.
#include <hip/hip_fp16.h>

#include "fbq_internal.h"

namespace fbq {

typedef _Float16 half_t;
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef double double4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double half_bits_to_double(uint16_t h) { return (double)__builtin_bit_cast(half_t, h); }

// double -> fp16 bits, rounded once, to nearest even: by way of an fp32 number rounded to odd.  A NaN becomes an infinity of its sign.
__device__ __forceinline__ uint16_t double_to_half_bits(double d)
{
    const float f = (float)d;
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if (__builtin_fabs((double)f) > __builtin_fabs(d)) u -= 1;
    if ((double)f != d) u |= 1;
    const uint16_t h = __builtin_bit_cast(uint16_t, (_Float16)__builtin_bit_cast(float, u));
    return d != d ? (uint16_t)(((__builtin_bit_cast(uint64_t, d) >> 48) & 0x8000u) | 0x7c00u) : h;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t bounded_buffer(const void *p, long bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ half8_t load_half8(__amdgpu_buffer_rsrc_t b, int off)
{
    return __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
}

// Scale (low half) and zero (high half) of a group from its extremes.
__device__ __forceinline__ uint32_t search_scale(double lo, double hi, int qmax)
{
#pragma clang fp contract(off)
    double s = (hi - lo) / (double)qmax;
    if (!(s > 0.0)) s = 1.0;
    uint16_t s16 = double_to_half_bits(s);
    if (s16 < 0x0400u) s16 = 0x0400u;
    // (extremes that are infinite or NaN never meet the condition below, whatever the scale: straight to the last one)
    if (!(__builtin_fabs(lo) < __builtin_inf() && __builtin_fabs(hi) < __builtin_inf()) && s16 < 0x7bffu) s16 = 0x7bffu;
    uint16_t z16;
    for (;;) {
        const double sd = half_bits_to_double(s16), up = -lo / sd;
        z16 = double_to_half_bits(up);
        const double zd = half_bits_to_double(z16);
        if ((zd - up >= -0.5 && hi / sd + zd <= (double)qmax + 0.5) || s16 >= 0x7bffu) break;
        s16 += 1;
    }
    return (uint32_t)s16 | ((uint32_t)z16 << 16);
}

// The packed words of 32 consecutive codes, from the codes as floats.  Fields are added up in fp32, where they are whole numbers below 2^16.
template <int BITS>
__device__ __forceinline__ void pack_codes(const float *x, uint32_t *words)
{
    if constexpr (BITS == 4) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            uint32_t h[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float *f = x + 8 * w + 4 * i;
                h[i] = (uint32_t)__builtin_fmaf(__builtin_fmaf(__builtin_fmaf(f[3], 16.0f, f[2]), 16.0f, f[1]), 16.0f, f[0]);
            }
            words[w] = h[0] | (h[1] << 16);
        }
    } else {
        const uint32_t c30 = (uint32_t)x[30], c31 = (uint32_t)x[31];
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            uint32_t h[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float *f = x + 10 * w + 5 * i;
                h[i] = (uint32_t)__builtin_fmaf(__builtin_fmaf(__builtin_fmaf(__builtin_fmaf(f[4], 8.0f, f[3]), 8.0f, f[2]), 8.0f, f[1]), 8.0f, f[0]);
            }
            words[w] = h[0] | (h[1] << 16) | ((c30 >> w) & 1u) << 15 | ((c31 >> w) & 1u) << 31;
        }
    }
}

// Extremes over the four lanes that hold one row (lanes 16 apart).
__device__ __forceinline__ void row_extremes(float &lo, float &hi)
{
    auto swap16 = [](float v) { return __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, v), false, false); };
    auto swap32 = [](float v) { return __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, v), false, false); };
    auto f = [](uint32_t u) { return __builtin_bit_cast(float, u); };
    auto a = swap16(lo), b = swap16(hi);
    lo = fminf(f(a[0]), f(a[1]));
    hi = fmaxf(f(b[0]), f(b[1]));
    a = swap32(lo);
    b = swap32(hi);
    lo = fminf(f(a[0]), f(a[1]));
    hi = fmaxf(f(b[0]), f(b[1]));
}

// The power of two that takes numbers whose largest is `peak` to 2^10 and above, below 2^11; 1 where that would be a step down.
__device__ __forceinline__ float fixed_point_factor(float peak)
{
    const int exponent = (int)(__builtin_bit_cast(uint32_t, peak) >> 23) - 127;
    return peak == 0.0f || exponent > 10 ? 1.0f : __builtin_bit_cast(float, (uint32_t)(127 + 10 - exponent) << 23);
}

constexpr int kQuantTapStep = 32;      // taps one matrix instruction takes
constexpr float kLongest = 16300.0f;   // of 128 taps or a row of as many, at 2^10 and above: what the exact sums (below) have room for; evenly spread ones are 13400 long
constexpr int kFewOpen = 3;            // open rows of a wave's sixteen that go to 64 bits one by one
constexpr int kOpenList = 128;         // pairs of elements of Delta_F that a wave lists at a time

// Taps in LDS: 16-byte pieces of eight taps, [feature][piece], a piece's place XORed with a key so that the sixteen features that
// one matrix operand reads (bits 0, 1, 5, 6 of the feature differ) lie in sixteen different places of 256 bytes.
__device__ __forceinline__ int tap_key(int f) { return ((f >> 1) & 1) | ((f >> 4) & 6); }

// STEPS: the most steps of 32 taps.  WAVES: a block's.  IN64 (with DELTA only): no attempt in 32 bits.
// DELTA: three waves a SIMD (with four, 128 registers spilled 22: a step with loss 2 % longer).
template <int BITS, bool DELTA, int STEPS, int WAVES, bool IN64>
__global__ __launch_bounds__(64 * WAVES, DELTA ? (WAVES == 8 || STEPS > 4 ? 2 : 3) : 4) void fbq_quantize_kernel(const uint16_t *__restrict__ W, const uint16_t *__restrict__ At,
                                                                  const uint16_t *__restrict__ Bt, uint32_t *__restrict__ qw,
                                                                  uint16_t *__restrict__ scales, uint16_t *__restrict__ zeros, int N,
                                                                  int K, int r, int row_words, uint16_t *__restrict__ D16,
                                                                  float gain, int tiles)
{
#pragma clang fp contract(off)
    constexpr int kRows = 16 * WAVES, kPieces = 4 * STEPS;
    // DELTA, up to 64 taps: taps[] holds their multiples of a unit and rests[] the rest (below); otherwise each wave splits what it reads
    constexpr bool kSplitTaps = DELTA && !IN64 && STEPS <= 2;
    __shared__ half8_t taps[kGroup][kPieces], rests[kSplitTaps ? kGroup : 1][kSplitTaps ? kPieces : 1];
    __shared__ uint32_t longest, straight;                                      // largest squared norm of a feature's taps; whether rows go to 64 bits without an attempt in 32
    // DELTA, by feature: what takes its taps back to At's, and its bound (below)
    __shared__ __attribute__((aligned(16))) float tap_back[DELTA ? kGroup : 4], tap_norm[DELTA ? kGroup : 4];
    __shared__ struct { float code[kGroup]; alignas(16) _Float16 delta[DELTA ? kGroup : 8]; uint16_t list[DELTA ? kOpenList : 8]; } exact[WAVES];
    constexpr int qmax = (1 << BITS) - 1;
    constexpr int kNowhere = 0x7FFFFFF0;                                        // beyond every buffer: taps past r are zeros in both operands
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = K / kGroup, g = blockIdx.x;
    const int steps = (r + kQuantTapStep - 1) / kQuantTapStep;

    if (threadIdx.x == 0) longest = straight = 0;
    // few blocks: what the first tile reads is asked for together with the taps
    half8_t early[5];
    if constexpr (IN64) {
        const int n = min((int)blockIdx.y * tiles * kRows + 16 * wave + (lane & 15), N - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) early[i] = *reinterpret_cast<const half8_t *>(W + (size_t)n * K + g * kGroup + 32 * (lane >> 4) + 8 * i);
        early[4] = *reinterpret_cast<const half8_t *>(Bt + (size_t)n * r + min(8 * (lane >> 4), r - 8));
    }
    const half_t grid = STEPS <= 4 ? (half_t)6144.0f : (half_t)12288.0f;        // 1.5 x 2^10 units: added and taken away, it leaves whole units
    const half8_t grid8 = {grid, grid, grid, grid, grid, grid, grid, grid};
    auto tap8 = [&](int f, int p) __attribute__((always_inline)) {
        if constexpr (kSplitTaps) return taps[f][p ^ tap_key(f)] + rests[f][p ^ tap_key(f)];   // (exact)
        else return taps[f][p ^ tap_key(f)];
    };
    if (r > 0) {
        // eight features of eight taps a thread, turned in registers
        const __amdgpu_buffer_rsrc_t abuf = bounded_buffer(At, (long)r * K * 2);
        for (int u = threadIdx.x; u < 64 * steps; u += 64 * WAVES) {
            const int fb = u & 15, p = u >> 4;
            half8_t a[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) a[j] = load_half8(abuf, 8 * p + j < r ? ((8 * p + j) * K + g * kGroup + 8 * fb) * 2 : kNowhere);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int f = 8 * fb + i;
                taps[f][p ^ tap_key(f)] = half8_t{a[0][i], a[1][i], a[2][i], a[3][i], a[4][i], a[5][i], a[6][i], a[7][i]};
            }
        }
    }
    if (r > 0 && !IN64) {
        __syncthreads();
        // WAVES / 2 threads a feature, side by side
        constexpr int kSide = WAVES / 2;
        const int f = threadIdx.x / kSide;
        float even = 0.0f, odd = 0.0f, peak = 0.0f;
        for (int p = threadIdx.x % kSide; p < 4 * steps; p += kSide) {
            const half8_t a = taps[f][p ^ tap_key(f)];
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                even = __builtin_fmaf((float)a[j], (float)a[j], even);
                odd = __builtin_fmaf((float)a[j + 1], (float)a[j + 1], odd);
            }
            if (DELTA) {
#pragma unroll
                for (int j = 0; j < 8; ++j) peak = fmaxf(peak, fabsf((float)a[j]));
            }
        }
        even += odd;
#pragma unroll
        for (int away = 1; away < kSide; away *= 2) {
            even += __shfl_xor(even, away, 64);
            if (DELTA) peak = fmaxf(peak, __shfl_xor(peak, away, 64));
        }
        if (DELTA) {                                                            // (each thread has the pieces that it read)
            const float factor = fixed_point_factor(peak);
            for (int p = threadIdx.x % kSide; p < 4 * steps; p += kSide) {
                half8_t a = taps[f][p ^ tap_key(f)];
#pragma unroll
                for (int j = 0; j < 8; ++j) a[j] = (half_t)((float)a[j] * factor);
                // (from 2048 on nothing is split: on such a grid the largest fp16 numbers are infinite, and an infinity less itself is none)
                const half8_t whole = kSplitTaps && peak < 2048.0f ? (a + grid8) - grid8 : a;
                taps[f][p ^ tap_key(f)] = whole;
                if constexpr (kSplitTaps) rests[f][p ^ tap_key(f)] = peak < 2048.0f ? a - whole : half8_t{};
            }
            const float back = peak == 0.0f ? 0.0f : 1.0f / factor;
            even = peak == 0.0f ? even : fmaxf(sqrtf(even), 2048.0f * back);    // (at least the largest tap)
            if (threadIdx.x % kSide == 0) {
                tap_back[f] = back;
                tap_norm[f] = even;
                if (peak >= 2048.0f || (STEPS == 4 && even > kLongest * back)) straight = 1;
            }
        }
        uint32_t most = __builtin_bit_cast(uint32_t, even);                    // (not negative; a NaN is larger than all numbers this way)
#pragma unroll
        for (int away = kSide; away < 64; away *= 2) most = max(most, (uint32_t)__shfl_xor((int)most, away, 64));
        if (lane == 0 && most) atomicMax(&longest, most);
    }
    if constexpr (IN64) {
#pragma unroll
        for (int i = 0; i < 5; ++i) asm volatile("" :: "v"(early[i]));
    }
    __syncthreads();
    // (the instruction aligns a subnormal operand as one of 2^-14)
    const float a_norm2 = longest ? __builtin_bit_cast(float, longest) + (float)r * 0x1p-28f : 0.0f;

    for (int tile = 0; tile < tiles; ++tile) {
        const int nb = (blockIdx.y * tiles + tile) * kRows, n0 = nb + 16 * wave;   // the block's first row, the wave's
        if (nb >= N) break;
        int lane_now = lane;                                                    // (not known to be the same in every tile: addresses kept over the loop spill)
        asm volatile("" : "+v"(lane_now));
        const int c = lane_now & 15, q = lane_now >> 4;
        const int rows = min(16, N - n0);                                       // may be <= 0: such a wave computes zeros and stores nothing
        // The wave's rows of W and Bt through descriptors that end with row N - 1: rows past it read as zeros.
        const __amdgpu_buffer_rsrc_t wbuf = bounded_buffer(W + (size_t)min(n0, N - 1) * K, rows > 0 ? (long)rows * K * 2 : 0);
        const __amdgpu_buffer_rsrc_t bbuf = bounded_buffer(Bt + (size_t)min(n0, N - 1) * r, rows > 0 ? (long)rows * r * 2 : 0);
        auto branch_rows = [&](int j) __attribute__((always_inline)) { return load_half8(bbuf, j < r ? (c * r + j) * 2 : kNowhere); };   // (r is a multiple of 8: all of a lane's taps or none)
        auto weights = [&](int i) __attribute__((always_inline)) { return load_half8(wbuf, (c * K + g * kGroup + 32 * q + 8 * i) * 2); };

        // ---- 32 bits, with a bound
        uint32_t words[BITS], sz = 0, open_rows = (1u << max(0, min(16, rows))) - 1;
        half8_t d8[4];
        uint32_t open_delta = 0;                                                // DELTA: pairs of features with an fp16 number that 32 bits leave open, the first pair in bit 15
        if (!IN64 && !__builtin_amdgcn_readfirstlane(__hip_atomic_load(&straight, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))) {   // wave-uniform
            half8_t w[4], b[2];
            b[0] = branch_rows(8 * q);
            b[1] = branch_rows(kQuantTapStep + 8 * q);
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = weights(i);
            float Sigma[32];                                                     // DELTA: times gain, a power of two
#pragma unroll
            for (int i = 0; i < 32; ++i) Sigma[i] = 0.0f;
            float b_norm2 = 0.0f, off_sum, off_rest = 0.0f;                      // off_rest: DELTA, without a rounding of Sigma, for a feature of tap_norm 1
            bool coarse = false;
            if constexpr (!DELTA) {
#pragma unroll 1
                for (int s = 0; s < steps; ++s) {
                    const half8_t b8 = b[0];
                    b[0] = b[1];
                    b[1] = branch_rows(kQuantTapStep * (s + 2) + 8 * q);
#pragma unroll
                    for (int j = 0; j < 8; ++j) b_norm2 = __builtin_fmaf((float)b8[j], (float)b8[j], b_norm2);
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int f = 32 * (c >> 2) + 4 * t + (c & 3);
                        const float4_t sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(taps[f][(4 * s + q) ^ tap_key(f)], b8, float4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 4; ++v) Sigma[4 * t + v] += sum[v];
                    }
                }
                b_norm2 += __shfl_xor(b_norm2, 16, 64);
                b_norm2 += __shfl_xor(b_norm2, 32, 64);
                if (b_norm2 != 0.0f) b_norm2 += (float)(8 * steps) * 0x1p-28f;
                // How far Sigma can be off.  The instruction adds eight products at a time to what it has, cutting each operand off 2^-24 below the
                // largest and rounding the sum once (measured, bit by bit): 10 x 2^-24 of what the operands may be at most, which is |a| |b| of the
                // step's 32 taps, four times a step; then come the steps' sums, rounded in fp32.  Two more and the last factor
                // are for the roundings of this bound itself.
                off_sum = (float)(42 + steps) * 0x1.04p-24f * sqrtf(a_norm2 * b_norm2);
            } else {
                // Delta_F is small beside what adds up to it, so Sigma is had more exactly: taps and rows of B, at 2^10 and above, are each a multiple of
                // `unit` (at most 2^9 units, 2^8 above rank 128) and a rest of half a unit.  Products of the multiples are whole numbers of unit^2 whose sums stay within
                // 2^24 (|a| |b| <= r 2^18 or r 2^16, and between rank 64 and 128 it is checked): exact.  The rests' products are a hundredth of the whole, and so is their error.
                float peak = 0.0f;
#pragma unroll 1
                for (int s = 0; s < steps; ++s) {
                    const half8_t b8 = s == 0 ? b[0] : (s == 1 ? b[1] : branch_rows(kQuantTapStep * s + 8 * q));
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        b_norm2 = __builtin_fmaf((float)b8[j], (float)b8[j], b_norm2);
                        peak = fmaxf(peak, fabsf((float)b8[j]));
                    }
                }
                b_norm2 += __shfl_xor(b_norm2, 16, 64);
                b_norm2 += __shfl_xor(b_norm2, 32, 64);
                peak = fmaxf(peak, __shfl_xor(peak, 16, 64));
                peak = fmaxf(peak, __shfl_xor(peak, 32, 64));
                const float b_factor = fixed_point_factor(peak);
                coarse = peak >= 2048.0f || (STEPS == 4 && b_norm2 * b_factor * b_factor > kLongest * kLongest);   // (to 64 bits)
                float rest[32];
#pragma unroll
                for (int i = 0; i < 32; ++i) rest[i] = 0.0f;
#pragma unroll 1
                for (int s = 0; s < steps; ++s) {
                    half8_t b8 = s == 0 ? b[0] : (s == 1 ? b[1] : branch_rows(kQuantTapStep * s + 8 * q));
#pragma unroll
                    for (int j = 0; j < 8; ++j) b8[j] = (half_t)((float)b8[j] * b_factor);
                    const half8_t b_whole = (b8 + grid8) - grid8, b_rest = b8 - b_whole;
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int f = 32 * (c >> 2) + 4 * t + (c & 3);
                        half8_t a_whole = taps[f][(4 * s + q) ^ tap_key(f)], a_rest;
                        if constexpr (kSplitTaps) a_rest = rests[f][(4 * s + q) ^ tap_key(f)];
                        else {
                            const half8_t a8 = a_whole;
                            a_whole = (a8 + grid8) - grid8;
                            a_rest = a8 - a_whole;
                        }
                        const float4_t had = {Sigma[4 * t], Sigma[4 * t + 1], Sigma[4 * t + 2], Sigma[4 * t + 3]};
                        const float4_t whole = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_whole, b_whole, had, 0, 0, 0);
                        const float4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
                        const float4_t one = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_whole, b_rest, zero4, 0, 0, 0), two = __builtin_amdgcn_mfma_f32_16x16x32_f16(a_rest, b8, zero4, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            Sigma[4 * t + v] = whole[v];
                            rest[4 * t + v] += one[v] + two[v];
                        }
                    }
                }
                const float b_back = 1.0f / b_factor, up = gain * b_back;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float4_t back = *reinterpret_cast<const float4_t *>(&tap_back[32 * q + 4 * t]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) Sigma[4 * t + v] = (Sigma[4 * t + v] + rest[4 * t + v]) * (back[v] * up);
                }
                // The bound of the instruction (above) for the products with a rest, the additions of the rests, and the last one, rounded in fp32.
                // Rests are `half` long at most, where a feature's taps, at 2^10 and above, are tap_norm / tap_back long and tap_norm / tap_back is 2^11 at least.
                const float half = sqrtf((float)r) * (STEPS <= 4 ? 2.0f : 4.0f), b_norm = sqrtf(b_norm2);
                off_rest = peak == 0.0f ? 0.0f : 0x1.06p-24f * (float)(44 + 2 * steps) * half * (b_back + (half * b_back + b_norm) * 0x1p-11f);
                off_sum = (off_rest + 0x1.06p-24f * b_norm) * (longest ? __builtin_bit_cast(float, longest) : 0.0f);
            }
            float R[32];
#pragma unroll
            for (int i = 0; i < 32; ++i) R[i] = DELTA ? __builtin_fmaf(Sigma[i], -1.0f / gain, (float)w[i >> 3][i & 7]) : (float)w[i >> 3][i & 7] - Sigma[i];
            float lo = R[0], hi = R[0];
#pragma unroll
            for (int i = 1; i < 32; ++i) { lo = fminf(lo, R[i]); hi = fmaxf(hi, R[i]); }
            row_extremes(lo, hi);
            // How far R can be off: as Sigma, and by the subtraction.  A branch that is zero leaves R = W exactly.
            const float most = fmaxf(fabsf(lo), fabsf(hi));
            const float off = off_sum == 0.0f ? 0.0f : off_sum + 0x1.04p-24f * (most + off_sum);
            // the search from the widest and from the narrowest extremes that the bound allows (even and odd quarter waves): it is monotone
            // in them while a zero's last place is below one, so where both agree the true ones do
            const double e = q & 1 ? -(double)off : (double)off;
            sz = search_scale((double)lo - e, (double)hi + e, qmax);
            bool sure = (uint32_t)__shfl_xor((int)sz, 16, 64) == sz && (off == 0.0f || hi - lo > 8.0f * off);
            const float s = (float)__builtin_bit_cast(half_t, (uint16_t)sz), z = (float)__builtin_bit_cast(half_t, (uint16_t)(sz >> 16));
            // (far from zero the differences inside a group are lost in R's own rounding)
            sure = sure && fabsf(z) <= 1024.0f;
            if (DELTA) sure = sure && !coarse && (z == 0.0f || fabsf(z) >= 0x1p-9f);   // a code less z is an fp32 number
            const float inv = 1.0f / s;
            // t below is off by R's error, the reciprocal's, and one rounding
            const float lim = 0.5f - (off * inv + 0x1.1p-24f * (most * inv + (float)(qmax + 1)) + 0x1.1p-24f * most * inv);
            float x[32];
            float furthest = 0.0f;                                               // of t from the code it rounds to; NaN where one is
            // Delta_F below is W - s (q - z), one rounding, less Sigma, another one; two more for the bounds themselves
            const float off_delta = gain * 1.1f * off_rest;
            float4_t norm4;
            float below[2], above[2];
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                if (DELTA && !(i & 3)) norm4 = *reinterpret_cast<const float4_t *>(&tap_norm[32 * q + i]);
                const float t = __builtin_fmaf(R[i], inv, z);
                x[i] = rintf(t);                                                 // ties to even
                furthest = __builtin_elementwise_maximum(furthest, fabsf(t - x[i]));
                x[i] = fminf(fmaxf(x[i], 0.0f), (float)qmax);
                if (DELTA) {                                                     // Delta_F (Sec. 4.2)
                    const float d = __builtin_fmaf(gain, __builtin_fmaf(-s, x[i] - z, (float)w[i >> 3][i & 7]), -Sigma[i]), e = __builtin_fmaf(0x1p-22f, fabsf(d), __builtin_fmaf(0x1.1p-23f, fabsf(Sigma[i]), off_delta * norm4[i & 3]));
                    below[i & 1] = d - e;
                    above[i & 1] = d + e;
                    if (i & 1) {
                        const half2_t l = {(half_t)below[0], (half_t)below[1]}, h = {(half_t)above[0], (half_t)above[1]};
                        d8[i >> 3][(i & 7) - 1] = l.x;
                        d8[i >> 3][i & 7] = l.y;
                        open_delta += open_delta + (__builtin_bit_cast(uint32_t, l) != __builtin_bit_cast(uint32_t, h) ? 1u : 0u);
                        asm volatile("" : "+v"(open_delta));                     // (one after the other: as a tree the partial masks spill)
                    }
                }
            }
            sure = sure && furthest <= lim;                                                // (never where nothing is a number: the split of large numbers can make it so)
            pack_codes<BITS>(x, words);
            const unsigned long long unsure = __ballot(!sure);
            open_rows &= (uint32_t)(unsure | unsure >> 16 | unsure >> 32 | unsure >> 48);
        }
        // ---- rows that 32 bits leave open, in 64.  The products of two fp16 values have 22 significant bits, so the
        // order of the taps matters only where a sum needs more than 53 bits.
        // Many of them: all sixteen at once on the fp64 matrix instruction.  Lane (c, q) supplies tap q of four of feature 32 (c % 4) + 4 t + c / 4 and of row c, and ends up
        // with the features 32 q + 4 t .. + 3 of row c, as above.  (An open row takes a quarter of the time of all sixteen.)
        const bool many = IN64 || __builtin_popcount(open_rows) > kFewOpen;
        if (many) {
            int lane_here = lane;                                                // (as above)
            asm volatile("" : "+v"(lane_here));
            const int c = lane_here & 15, q = lane_here >> 4;
            auto branch_rows = [&](int j) __attribute__((always_inline)) { return load_half8(bbuf, j < r ? (c * r + j) * 2 : kNowhere); };
            auto weights = [&](int i) __attribute__((always_inline)) { return load_half8(wbuf, (c * K + g * kGroup + 32 * q + 8 * i) * 2); };
            half8_t w[4];
            auto all_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = weights(i);
            };
            if (DELTA) all_weights();                                            // (no registers for them this early in the other instances)
            double4_t R[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) R[t] = double4_t{0.0, 0.0, 0.0, 0.0};
            half8_t next = branch_rows(8 * q);
#pragma unroll 1
            for (int s = 0; s < steps; ++s) {
                const half8_t b8 = next;
                next = branch_rows(kQuantTapStep * (s + 1) + 8 * q);
                double bd[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) bd[j] = (double)(float)b8[j];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    __builtin_amdgcn_sched_barrier(0);                           // (all eight operands at once spill)
                    const half8_t a8 = tap8(32 * (c & 3) + 4 * t + (c >> 2), 4 * s + q);
#pragma unroll
                    for (int j = 0; j < 8; ++j) R[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(float)a8[j], bd[j], R[t], 0, 0, 0);
                }
            }
            if (!DELTA) all_weights();
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int v = 0; v < 4; ++v) R[t][v] = (double)(float)w[t >> 1][4 * (t & 1) + v] - (DELTA && !IN64 ? R[t][v] * (double)tap_back[32 * q + 4 * t + v] : R[t][v]);
            }
            double lo = R[0][0], hi = R[0][0];
#pragma unroll
            for (int i = 1; i < 32; ++i) { lo = fmin(lo, R[i >> 2][i & 3]); hi = fmax(hi, R[i >> 2][i & 3]); }
#pragma unroll
            for (int away = 16; away < 64; away *= 2) {
                lo = fmin(lo, __shfl_xor(lo, away, 64));
                hi = fmax(hi, __shfl_xor(hi, away, 64));
            }
            const uint32_t found = search_scale(lo, hi, qmax);
            const double sd = half_bits_to_double((uint16_t)found), zd = half_bits_to_double((uint16_t)(found >> 16)), inv = 1.0 / sd;
            // R / s costs eleven fp64 instructions, R * inv and one correction three, and the result is the same number: with
            // u = R * inv the residual e = R - u s is exact, u + e * inv is off the quotient by about 2^-105 of it before its one
            // rounding, and a quotient of a 53-bit number by an 11-bit one is never that close to the middle between two fp64
            // numbers (it is at least 2^-12 of a last place away from it, and the middle itself would need 54 bits of R).  With an
            // infinite scale (weights that are infinite) inv is 0, and so, with no s in the residual, is the quotient of every number.
            const double s_back = (found & 0x7FFFu) == 0x7c00u ? 0.0 : sd;
            float x[32];
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                if (!(i & 3)) __builtin_amdgcn_sched_barrier(0);
                const double Ri = R[i >> 2][i & 3];
                const double u = Ri * inv, code = fmin(fmax(rint(__builtin_fma(__builtin_fma(-u, s_back, Ri), inv, u) + zd), 0.0), (double)qmax);   // ties to even
                x[i] = (float)code;
                if (DELTA) d8[i >> 3][i & 7] = (half_t)(float)((double)gain * (Ri - sd * (code - zd)));   // Delta_F (Sec. 4.2)
            }
            pack_codes<BITS>(x, words);
            sz = found;
            // (rows of one layer are alike; a wave that sees it late finds the same)
            if (!IN64 && lane == 0 && __builtin_popcount(open_rows) > 8) __hip_atomic_store(&straight, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            open_rows = 0xFFFFu;                                                 // (the others come out as they were)
        }
        // A few: one by one, two features a lane.
        for (uint32_t open = many ? 0u : open_rows; open; open &= open - 1) {
            const int n = __builtin_ctz(open);
            uint16_t wi[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) wi[i] = __builtin_amdgcn_raw_buffer_load_b16(wbuf, (n * K + g * kGroup + lane + 64 * i) * 2, 0, 0);
            // the row's taps, four a lane
            const auto b4 = __builtin_amdgcn_raw_buffer_load_b64(bbuf, 4 * lane < r ? (n * r + 4 * lane) * 2 : kNowhere, 0, 0);
            double R[2] = {0.0, 0.0};
            half8_t next[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) next[i] = tap8(lane + 64 * i, 0);
#pragma unroll 1
            for (int p = 0; 8 * p < r; ++p) {
                half8_t a[2];
                const int after = min(p + 1, 4 * steps - 1);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[i] = next[i];
                    next[i] = tap8(lane + 64 * i, after);
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t two = __builtin_amdgcn_readlane(b4[(j >> 1) & 1], 2 * p + (j >> 2));
                    const float bj = (float)__builtin_bit_cast(half_t, (uint16_t)(two >> (16 * (j & 1))));
#pragma unroll
                    for (int i = 0; i < 2; ++i) R[i] += (double)__builtin_fmaf((float)a[i][j], bj, 0.0f);   // (a product of two fp16 is an fp32 number)
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) R[i] = half_bits_to_double(wi[i]) - (DELTA ? R[i] * (double)tap_back[lane + 64 * i] : R[i]);
            double lo = fmin(R[0], R[1]), hi = fmax(R[0], R[1]);
#pragma unroll
            for (int away = 1; away < 64; away *= 2) {
                lo = fmin(lo, __shfl_xor(lo, away, 64));
                hi = fmax(hi, __shfl_xor(hi, away, 64));
            }
            const uint32_t found = search_scale(lo, hi, qmax);
            const double sd = half_bits_to_double((uint16_t)found), zd = half_bits_to_double((uint16_t)(found >> 16));
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const double code = fmin(fmax(rint(R[i] / sd + zd), 0.0), (double)qmax);
                exact[wave].code[lane + 64 * i] = (float)code;
                if (DELTA) exact[wave].delta[lane + 64 * i] = (_Float16)(float)((double)gain * (R[i] - sd * (code - zd)));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (c == n) {
                sz = found;
                float x[32];
#pragma unroll
                for (int i = 0; i < 32; ++i) x[i] = exact[wave].code[32 * q + i];
                pack_codes<BITS>(x, words);
                if (DELTA) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) d8[i] = *reinterpret_cast<const half8_t *>(&exact[wave].delta[32 * q + 8 * i]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }

        if (c < rows) {
            const size_t n = (size_t)(n0 + c);
            if (q == 0) scales[n * G + g] = (uint16_t)sz;
            if (q == 1) zeros[n * G + g] = (uint16_t)(sz >> 16);
            uint32_t *to = qw + n * row_words + g * (4 * BITS) + BITS * q;
            if constexpr (BITS == 4) *reinterpret_cast<uint4 *>(to) = uint4{words[0], words[1], words[2], words[3]};
            else { to[0] = words[0]; to[1] = words[1]; to[2] = words[2]; }
            if (DELTA) {
#pragma unroll
                for (int i = 0; i < 4; ++i) *reinterpret_cast<half8_t *>(D16 + n * K + g * kGroup + 32 * q + 8 * i) = d8[i];
            }
        }
        if (DELTA) {
            // ---- elements that 32 bits leave open (r = 64: four in a thousand, more as the branch grows): the wave lists them, in pairs, and takes 64 at a time,
            // a lane each, or up to eight lanes that share the taps of one.  What they find goes over what was stored above (the
            // wavefront-scope fences order the two).
            auto in_order = []() __attribute__((always_inline)) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            };
            uint32_t pending = c < rows && !(open_rows >> c & 1) ? open_delta : 0u;
            int rank = __builtin_popcount(pending), total;                      // of the lane's first element in the list
            {
                int upto = rank;
#pragma unroll
                for (int away = 1; away < 64; away *= 2) {
                    const int below_me = __shfl_up(upto, away, 64);
                    upto += lane >= away ? below_me : 0;
                }
                total = __builtin_amdgcn_readlane(upto, 63);
                rank = upto - rank;
            }
            uint16_t *const list = exact[wave].list;
            for (int from = 0; from < total; from += kOpenList) {
                in_order();
                for (; pending && rank < from + kOpenList; pending &= pending - 1) list[rank++ - from] = (uint16_t)(c << 7 | (32 * q + 30 - 2 * __builtin_ctz(pending)));
                in_order();
                const int listed = 2 * min(kOpenList, total - from);
#pragma unroll 1
                for (int at = 0; at < listed; at += 64) {
                    const int left = min(64, listed - at), shift = left > 32 ? 0 : (left > 16 ? 1 : (left > 8 ? 2 : 3));
                    const int mine = lane >> shift, entry = at + min(mine, left - 1), element = list[entry >> 1] + (entry & 1);
                    const int n = element >> 7, f = element & 127;
                    const half_t wi = __builtin_bit_cast(half_t, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(wbuf, (n * K + g * kGroup + f) * 2, 0, 0));
                    const uint32_t of_row = (uint32_t)__shfl((int)sz, n, 64);
                    double sum = 0.0;
                    for (int p = lane & ((1 << shift) - 1); 8 * p < r; p += 4 << shift) {   // four pieces asked for at once
                        half8_t a8[4], b8[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const int piece = p + (k << shift);
                            b8[k] = load_half8(bbuf, 8 * piece < r ? (n * r + 8 * piece) * 2 : kNowhere);
                            a8[k] = tap8(f, min(piece, 4 * steps - 1));
                        }
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int j = 0; j < 8; ++j) sum += (double)__builtin_fmaf((float)a8[k][j], (float)b8[k][j], 0.0f);
                    }
                    for (int away = 1; away < 1 << shift; away *= 2) sum += __shfl_xor(sum, away, 64);
                    const double sd = half_bits_to_double((uint16_t)of_row), zd = half_bits_to_double((uint16_t)(of_row >> 16)), R = (double)wi - sum * (double)tap_back[f];
                    const _Float16 d = (_Float16)(float)((double)gain * (R - sd * (fmin(fmax(rint(R / sd + zd), 0.0), (double)qmax) - zd)));
                    if ((lane & ((1 << shift) - 1)) == 0 && mine < left) D16[(size_t)(n0 + n) * K + g * kGroup + f] = __builtin_bit_cast(uint16_t, d);
                }
            }
            in_order();                                                         // (the list and the row of codes are written again)
        }
    }
}

hipError_t launch_quantize(const fbq_desc &d, const uint16_t *W, const uint16_t *At, const uint16_t *Bt, uint32_t *qw,
                           uint16_t *scales, uint16_t *zeros, hipStream_t stream, uint16_t *D16, float gain)
{
    const int words = (int)row_words(d.K, d.bits), G = d.K / kGroup;
    // Waves a block: four, so that four blocks share a CU, but eight where the taps (64 KB above rank 128) leave
    // room for two blocks at most (11008 x 4096 INT4, r = 200: 125 us with four, 96 with eight), unless those are too few to go round.
    // Tiles a block: two, which halves the work of getting At into LDS (r = 64, INT3, 11008 x 4096: 55 us with one tile, 50 with two, 49 with three),
    // where the GPU is full with them; one without a sub-branch (30, 32, 33 us: blocks that start in the order of the rows read memory best).
    // (Not with Delta_F, either, where such blocks go round once and a little: r = 200, 5000 x 1024, 320 blocks, the kernel 67.3 us with eight waves, 62.7 with four; with 384 blocks a step 124.0 and 125.8.)
    const int wide_blocks = G * ceil_div(d.N, 128);
    const bool wide = d.r > 128 && wide_blocks >= 256 && !(D16 && wide_blocks > 256 && wide_blocks < 352);
    const int rows = wide ? 128 : 64, blocks = G * ceil_div(d.N, rows);
    const int tiles = d.r > 0 && blocks >= (wide ? 1024 : 2048) ? 2 : 1;
    const dim3 grid(G, ceil_div(d.N, rows * tiles));
    const bool all_in_64 = blocks <= 256;                                        // (a CU each: see the head of the file)
#define FBQ_QUANT(B, D, S, V, I) hipLaunchKernelGGL((fbq_quantize_kernel<B, D, S, V, I>), grid, dim3(64 * V), 0, stream, W, At, Bt, qw, scales, zeros, d.N, d.K, d.r, words, D16, gain, tiles)
#define FBQ_QUANT_R(B, D, I) do { if (wide) FBQ_QUANT(B, D, 8, 8, false); \
                                  else if (d.r <= 64) FBQ_QUANT(B, D, 2, 4, I); else if (d.r <= 128) FBQ_QUANT(B, D, 4, 4, I); else FBQ_QUANT(B, D, 8, 4, I); } while (0)
    if (d.bits == 4) { if (D16 && all_in_64) FBQ_QUANT_R(4, true, true); else if (D16) FBQ_QUANT_R(4, true, false); else FBQ_QUANT_R(4, false, false); }
    else { if (D16 && all_in_64) FBQ_QUANT_R(3, true, true); else if (D16) FBQ_QUANT_R(3, true, false); else FBQ_QUANT_R(3, false, false); }
#undef FBQ_QUANT_R
#undef FBQ_QUANT
    return hipGetLastError();
}

}  // namespace fbq
