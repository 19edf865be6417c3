// Prefill path (more than 64 tokens): the fused kernel of Sec. 4.3 as an fp16 MFMA GEMM for gfx950.
//
//   y[M,N] = x[M,K] . Wq[N,K]^T + t[M,r] . B[r,N],   t = x . A
//
// Three launches (two without a sub-branch): the down-projection t = x.A as a small MFMA GEMM over K slices
// ("requires relatively minimal time" in the paper's words; its blocks also write the re-ordered copies of x and of the
// scales the fused kernel wants), the slices' sums as t_hi | t_lo, and the fused kernel, which de-quantizes in registers,
// multiplies on the matrix cores and folds the up-projection into the same accumulators as 2r extra K columns,
// so y is written once.  Where there are too few tiles for the CUs, K is split over blocks through fp32 partial results
// and a small summing launch.
//
// Fused kernel.  Four waves side by side along N, block tile (32 TM) x 256, TM = 2, 3, 4, 6 or 8; a wave owns TM x 2
// tiles of v_mfma_f32_32x32x16_f16.  With TM of 6 or 8 that is one wave per SIMD with up to 256 accumulator registers;
// with less the block has eight waves, two groups that split K and meet in LDS (or four waves and several blocks per CU).
// K advances in steps of 64, half a quantization group, and everything a step reads comes out of LDS, copied there three
// steps ahead by buffer_load ... lds (no registers): the activations, the packed words, and scale and zero.  With the
// packed words loaded into registers instead - 32 rows per load, waited for by the compiler's count - the look-ahead
// was worth a step less and the registers it took kept a wave from owning more than 96 rows.
//   * activations: a small pre-pass rewrites x once into the order the kernel wants (see below);
//   * weights: lane (n = lane % 32, h = lane / 32) takes the 32 codes k = 64v + 32h .. +31 of row n (INT4: 16 bytes,
//     INT3: 12) from LDS and turns them into the 8 x fp16 operands of four K steps of 16 in registers.  The MFMA only
//     needs both operands to agree on which k sits in which slot, so the pre-pass puts the
//     activations in the order the code extraction produces (pairs (c, c+4) for INT4, (f, f+5) for
//     INT3), and it XORs the position of each 16-byte piece within its 128-byte row segment with a key of
//     the row, so that the un-padded LDS rows are read without bank conflicts.
//   * de-quantization: one v_and_or_b32 puts a code into the mantissa of 1024.0 (or 1024 + 16c,
//     1024 + 8c, 1024 + 64c for fields at higher bit offsets); one exact packed add or fma recovers
//     the code minus the integer zi nearest to the zero point, d = q - zi; the weight is
//     fma(d, s, c) with c = fp16((zi - z) s): one rounding of the weight (2^-11 relative) and one of
//     c, which is at most 2^-12 of a quantization step.
// The sub-branch enters as t = t_hi + t_lo (two fp16 halves, ~22 bits) against B^T rows.
//
// What bounds it: the matrix cores at the clock they leave.  2048 tokens into 8192 x 8192 (INT4, no sub-branch, us per
// call): 256-row tiles 252; with the de-quantization left out 230, without copies 241, without reading activations 248,
// with nothing but matrix instructions 209 (they alone draw the clock down to 1.9 - 2.0 GHz).  By tile height, us per CU
// and step of 64: 256 rows 1.8, 192 rows 1.43, 128 rows 0.97, 96 rows 0.77, 64 rows 0.59: a step costs about 0.1 and
// each 32 rows 0.21.  The loop before this one (packed words in registers, compiler waits of vmcnt(0) at the top of every
// round) took 977 us for 2048 tokens of 8192 -> 28672 without a sub-branch where this takes 870.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "fbq_internal.h"
#include "fbq_lds_copy.h"

namespace fbq {

typedef _Float16 half_t;
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t uint4v_t __attribute__((ext_vector_type(4)));
typedef uint32_t uint3v_t __attribute__((ext_vector_type(3)));

constexpr int kTN = 2;               // 32-column MFMA tiles per wave along N
constexpr int kWavesN = 4;           // waves side by side along N
constexpr int kBN = kWavesN * kTN * 32;   // 256
constexpr int kStepK = 64;           // K per step: half a quantization group
constexpr int kXRow = 128;           // bytes per activation row and step in LDS: 8 pieces of 8 fp16, piece l at l ^ piece_key(row)
constexpr int kXcds = 8;             // accelerator dies, each with its own L2
constexpr int kStages = 3;           // steps in LDS: the one worked on and the next two on their way from memory

__device__ __forceinline__ half2_t h2_of(uint32_t v) { return __builtin_bit_cast(half2_t, v); }
__device__ __forceinline__ half2_t h2_splat(half_t v) { return half2_t{v, v}; }

struct PrefillParams {
    const uint32_t *qw;
    const uint32_t *sz;    // [G][Np] scale (low half) and zero (high half) by group, written by the pre-pass
    const uint16_t *Bt;    // [N][r]
    const uint16_t *xp;    // [M][K], arranged by the pre-pass
    const uint16_t *thl;   // [M][2r]: t_hi | t_lo
    uint16_t *y;           // [M][N]
    int M, N, K, r;
    int row_words, G, Np;  // Np: N rounded up to kBN
    int row_blocks;        // ceil(M / block tile rows)
    int full_slots;        // blocks per XCD that belong to column blocks this XCD has to itself: (column blocks / 8) * row_blocks * ksplit
    int full_cols;         // column blocks dealt out whole, eight at a time: (column blocks / 8) * 8
    int rem_blocks;        // blocks of the column blocks left over, dealt out singly over the XCDs
    int col0;              // first column block of this launch
    int ksplit;            // blocks that split K for the same tile (1: none)
    float *ypart;          // ksplit > 1 only: [ksplit][M][N] fp32 partial results, added up by fbq_sum_parts_kernel
};

// Order in which the 32 activations of a lane's code block must sit so that slot s of K step i
// (s = 0..7) meets the code the extraction puts there.
template <int BITS>
__device__ __forceinline__ constexpr int slot_source(int s)
{
    if (BITS == 4) {                 // word j = s / 8 yields pairs (0,4) (1,5) (2,6) (3,7)
        const int j = s / 8, t = s % 8;
        return 8 * j + (t / 2) + 4 * (t % 2);
    }
    if (s >= 30) return s;           // the two spread codes pair up last
    const int w = s / 10, t = s % 10;   // word w yields pairs (f, f+5)
    return 10 * w + (t / 2) + 5 * (t % 2);
}

// The lane's 32 codes of one step as 16 fp16 pairs s * (q - z), in slot order, four pairs (one matrix operand) at a time.
template <int BITS>
struct WeightRegs {
    static constexpr int kWords = BITS == 4 ? 4 : 3;
    static constexpr int kRowBytes = 2 * kWords * 4;    // bytes of a weight row per step: two blocks of 32 codes ...
    static constexpr int kLdsRow = 32;                  // ... in LDS 16 bytes apart, used up or not
    uint32_t w[kWords];

    __device__ __forceinline__ void read(const unsigned char *lds)
    {
        if constexpr (BITS == 4) {
            const uint4v_t q = *reinterpret_cast<const uint4v_t *>(lds);
            w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
        } else {
            const uint3v_t q = *reinterpret_cast<const uint3v_t *>(lds);   // (16-byte aligned)
            w[0] = q.x; w[1] = q.y; w[2] = q.z;
        }
    }

    // (w & mask) | 0x6400 in both halves: the masked field lands in the mantissa of 1024.0
    static __device__ __forceinline__ half2_t field(uint32_t w, uint32_t mask, uint32_t k6400)
    {
        uint32_t v;
        asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(v) : "v"(w), "s"(mask), "v"(k6400));
        return h2_of(v);
    }

    // Per-group constants: with zi = the integer nearest to z, the code minus zi is an exact small
    // integer d, and the weight is fma(d, s, c) with c = fp16((zi - z) s), |zi - z| <= 1/2.
    struct Affine {
        half2_t s, c;
        half2_t k0;   // -(1024 + zi): field at bit 0
        half2_t k1;   // INT4: -(64 + zi), field at bit 4;  INT3: -(128 + zi), field at bit 3
        half2_t k2;   // INT3: -(16 + zi), field at bit 6
        __device__ __forceinline__ void set(uint32_t sz)
        {
            const float sf = (float)__builtin_bit_cast(half_t, (uint16_t)sz);
            const float zf = (float)__builtin_bit_cast(half_t, (uint16_t)(sz >> 16));
            const float zi = __builtin_rintf(zf);
            s = h2_splat((half_t)sf);
            c = h2_splat((half_t)((zi - zf) * sf));
            k0 = h2_splat((half_t)(-1024.0f - zi));
            k1 = h2_splat((half_t)((BITS == 4 ? -64.0f : -128.0f) - zi));
            k2 = h2_splat((half_t)(-16.0f - zi));
        }
    };

    // pair p of 16
    __device__ __forceinline__ half2_t pair(int p, const Affine &f, uint32_t k6400) const
    {
        half2_t d;
        if constexpr (BITS == 4) {                      // word p / 4: fields at bits 0, 4, 8, 12 of its halves
            const uint32_t a = p % 4 < 2 ? w[p / 4] : w[p / 4] >> 8;
            if (p % 2 == 0) d = field(a, 0x000F000Fu, k6400) + f.k0;
            else d = field(a, 0x00F000F0u, k6400) * h2_splat((half_t)0.0625f) + f.k1;
        } else if (p == 15) {                           // the two codes spread over bits 15 and 31 of the words
            const uint32_t e = ((w[0] >> 15) & 0x00010001u) | ((w[1] >> 14) & 0x00020002u) | ((w[2] >> 13) & 0x00040004u);
            d = h2_of(e | 0x64006400u) + f.k0;
        } else {                                        // word p / 5: fields at bits 0, 3, 6, 9, 12 of its halves
            const uint32_t a = p % 5 < 3 ? w[p / 5] : w[p / 5] >> 9;
            if (p % 5 % 3 == 0) d = field(a, 0x00070007u, k6400) + f.k0;
            else if (p % 5 % 3 == 1) d = field(a, 0x00380038u, k6400) * h2_splat((half_t)0.125f) + f.k1;
            else d = field(a, 0x01C001C0u, k6400) * h2_splat((half_t)0.015625f) + f.k2;
        }
        return d * f.s + f.c;
    }
    __device__ __forceinline__ half8_t operand(int i, const Affine &f, uint32_t k6400) const
    {
        const half2_t a = pair(4 * i, f, k6400), b = pair(4 * i + 1, f, k6400), c = pair(4 * i + 2, f, k6400), d = pair(4 * i + 3, f, k6400);
        return half8_t{a.x, a.y, b.x, b.y, c.x, c.y, d.x, d.y};
    }
};

// TM: 32-row tiles of a wave and of the block.  KG: groups of four waves that split K for the same tile inside one block
// (1 or 2): the groups take consecutive ranges of K, and group 1 hands its accumulators to group 0 through LDS at the
// end, so nothing but y is ever written.  One block per CU: with TM of 6 or 8 a wave has a SIMD, and its 512
// registers, to itself; with less, two waves share one - of one block with two K groups, or of blocks
// with one (see prefill_cut for which).
template <int BITS, int TM, int KG>
struct GemmTile {
    static constexpr int kBM = 32 * TM;
    static constexpr int kThreads = 64 * kWavesN * KG;
    static constexpr int kXBytes = kBM * kXRow, kQBytes = kBN * WeightRegs<BITS>::kLdsRow;
    static constexpr int kStepBytes = kXBytes + kQBytes;                // one step of one K group
    static constexpr int kSzBytes = kWavesN * KG * 2 * 256;        // two groups' scales and zeros per wave
    static constexpr int kOutRow = 64 * 2 + 16;                         // a wave's output rows in LDS: 64 fp16, 144 bytes apart
    static constexpr int kMain = KG * kStages * kStepBytes + kSzBytes;
    static constexpr int kUp = kBN * 128 + kBM * 256;                   // 64 taps of the block's rows of B^T and of t_hi | t_lo
    static constexpr int kHand = KG > 1 ? TM * kTN * 16 * 64 * 4 * kWavesN : 0;
    static constexpr int kOut = kWavesN * 32 * kOutRow;
    static constexpr int kLds = std::max(std::max(kMain, kUp), std::max(kHand, kOut));
    static_assert(kLds <= 160 * 1024, "a block's buffers must fit the CU's LDS");
};

template <int BITS, int TM, int KG>
__global__ __launch_bounds__((GemmTile<BITS, TM, KG>::kThreads)) __attribute__((amdgpu_waves_per_eu(TM > 4 ? 1 : 2, TM > 4 ? 1 : 2))) void fbq_gemm_kernel(const PrefillParams p)
{
    using T = GemmTile<BITS, TM, KG>;
    constexpr int kBM = T::kBM;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[T::kLds];   // [KG][kStages][x tile | packed words], then [wave][2][64] scale | zero

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave_all / kWavesN, wave = wave_all % kWavesN;   // K group of this wave, position along N
    const int col = lane & 31, h = lane >> 5;
    // Workgroups go to the eight XCDs round-robin by linear id, and each XCD has its own L2.  Give
    // every XCD its own column blocks (all row blocks of one column block run on the same XCD, one
    // after the other in id order), so that a weight tile is fetched into one L2 only.
    // Where a launch would have fewer blocks than the CUs can hold, ksplit blocks share a tile and split
    // K; their fp32 partial results are added by a small launch afterwards.
    // Column blocks are dealt out whole, eight at a time; the blocks of the ones left over (fewer than eight) go to
    // the XCDs one by one, so that every XCD has the same number of them whatever the column count.
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    int bm, bn, part;
    if (slot < p.full_slots) {
        const int q = slot / p.ksplit;
        part = slot % p.ksplit;
        bm = q % p.row_blocks;
        bn = (q / p.row_blocks) * kXcds + xcd;
    } else {
        const int i = (slot - p.full_slots) * kXcds + xcd, q = i / p.ksplit;
        if (i >= p.rem_blocks) return;                  // block-uniform
        part = i % p.ksplit;
        bm = q % p.row_blocks;
        bn = p.full_cols + q / p.row_blocks;
    }
    const int m0 = bm * kBM, n0 = (p.col0 + bn) * kBN;
    const int nw = n0 + wave * (kTN * 32);
    const int shares = KG * p.ksplit;                   // K is shared out over the groups of a block and, for a layer with few tiles, over blocks
    const int U_part = (p.G + shares - 1) / shares;     // quantization groups per share
    const int u0 = min((part * KG + kg) * U_part, p.G - 1);         // this wave's groups: u0 .. u0 + U - 1 (the last shares may have none)
    const int U = max(0, min(U_part, p.G - (part * KG + kg) * U_part));

    // Everything the loop reads comes out of LDS, copied there without passing registers:
    //   x      rows of 128 bytes, eight per copy;  rows past M are outside the descriptor
    //   words  rows of 32 (24) bytes, the blocks of 32 codes side by side, 32 rows per copy;  rows past N likewise
    //   sz     the wave's 64 rows' scale | zero of one group, one copy per group
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(p.xp + (size_t)m0 * p.K, (long)min(kBM, p.M - m0) * p.K * 2);
    const __amdgpu_buffer_rsrc_t qbuf = buffer_of(p.qw + (size_t)n0 * p.row_words, (long)min(kBN, p.N - n0) * p.row_words * 4);
    const __amdgpu_buffer_rsrc_t sbuf = buffer_of(p.sz, (long)p.G * p.Np * 4);
    constexpr int kPiece = WeightRegs<BITS>::kWords * 4;
    const int xoff = (lane >> 3) * p.K * 2 + (lane & 7) * 16;
    const int qoff = (lane >> 1) * p.row_words * 4 + (lane & 1) * kPiece;
    const int soff = (nw + lane) * 4;
    const uint32_t lds0 = lds_offset(lds);
    const uint32_t ring0 = lds0 + kg * (kStages * T::kStepBytes);   // the group's ring of steps
    const int sz_at = KG * kStages * T::kStepBytes + wave_all * 512; // the wave's two slots
    constexpr int kLoadsX = TM, kLoadsQ = 2;       // copies per wave and step; one more, scale and zero, in the first step of a group
    constexpr int kLoads = kLoadsX + kLoadsQ;
    // copy j of step `st` (of this share: group st / 2, half st % 2), into stage `buf`.  Past the share's end: its last
    // group again, never used - every wave issues the same number of copies, so that they can be waited for by count
    auto issue_one = [&](int st, bool first_half, int buf, int j) __attribute__((always_inline)) {
        const int u = min(u0 + (st >> 1), p.G - 1), half = first_half ? 0 : 1;
        const uint32_t stage = ring0 + buf * T::kStepBytes;
        if (j < kLoadsX) {
            const int rows = (wave * kLoadsX + j) * 8;
            copy16_to_lds(xbuf, xoff, rows * p.K * 2 + (2 * u + half) * kXRow, stage + rows * kXRow);
        } else if (j < kLoads) {
            const int rows = (wave * kLoadsQ + j - kLoadsX) * 32;
            const int off = rows * p.row_words * 4 + (2 * u + half) * WeightRegs<BITS>::kRowBytes;
            const uint32_t dst = stage + T::kXBytes + rows * WeightRegs<BITS>::kLdsRow;
            if constexpr (BITS == 4) copy16_to_lds(qbuf, qoff, off, dst);
            else copy12_to_lds(qbuf, qoff, off, dst);
        } else if (j == kLoads && first_half) {
            copy4_to_lds(sbuf, soff, u * p.Np * 4, lds0 + sz_at + ((st >> 1) & 1) * 256);
        }
    };
    // What has to be complete at a barrier is waited for explicitly in front of it: __syncthreads() would wait for every
    // copy in flight.  At most n of this wave's copies may still be on their way.
    auto wait_and_meet = [&](auto N) __attribute__((always_inline)) {
        constexpr int n = decltype(N)::value;
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(n) : "memory");
    };
    auto block_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    float16_t acc[TM][kTN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < kTN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.0f;

    uint32_t k6400 = 0x64006400u;
    asm volatile("" : "+v"(k6400));                     // keep the constant in a VGPR for v_and_or_b32

    // this lane's fragment of K step i (16 values of k) of the step in stage `buf`, row tile tm: piece 4 h + i of its row
    const int a_lane = col * kXRow + (((4 * h) ^ piece_key(col & 15)) << 4);
    const int q_lane = T::kXBytes + (wave * kTN * 32 + col) * WeightRegs<BITS>::kLdsRow + h * 16;
    auto a_frag = [&](int buf, int i, int tm) __attribute__((always_inline)) {
        return *reinterpret_cast<const half8_t *>(lds + (kg * kStages + buf) * T::kStepBytes + (a_lane ^ (i << 4)) + tm * (32 * kXRow));
    };
    WeightRegs<BITS> w[2][kTN];                         // packed words of the step worked on and of the next one
    typename WeightRegs<BITS>::Affine aff[kTN];
    auto read_words = [&](WeightRegs<BITS> (&dst)[kTN], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int tn = 0; tn < kTN; ++tn) dst[tn].read(lds + (kg * kStages + buf) * T::kStepBytes + q_lane + tn * 32 * WeightRegs<BITS>::kLdsRow);
    };
    uint32_t szw[kTN];
    auto read_sz = [&](int parity) __attribute__((always_inline)) {
#pragma unroll
        for (int tn = 0; tn < kTN; ++tn) szw[tn] = *reinterpret_cast<const uint32_t *>(lds + sz_at + parity * 256 + (tn * 32 + col) * 4);
    };

    half8_t af[2][TM], b0, b1;
    // One step: four K steps of 16.  A K step is two phases of TM matrix instructions, one per column tile: during the
    // first the second tile's weights of this K step are de-quantized and the activation fragments of the next one are
    // read from LDS, during the second the first tile's weights of the next K step are de-quantized.  One or two copies of
    // the step after next go out per K step, between the matrix instructions (all at once, they would hold the wave up in
    // the queue of the CU's address unit).  In front of the last K step the waves meet: the next step has landed, and
    // this one's stage has been read by everybody and may be filled again.
    // the copies of a step go out in eight portions, one per phase: copy j of n with portion 8 j / n
    auto issue_portion = [&](int st, auto FIRST, int buf, int portion) __attribute__((always_inline)) {
        constexpr int n = kLoads + (decltype(FIRST)::value ? 1 : 0);
#pragma unroll
        for (int j = 0; j < n; ++j)
            if (8 * j / n == portion) issue_one(st, decltype(FIRST)::value, buf, j);
    };
    auto do_step = [&](auto HALF, int st, int buf, int buf1, int buf2) __attribute__((always_inline)) {
        constexpr int half = decltype(HALF)::value;     // of the group
        constexpr std::integral_constant<bool, half == 0> next_first{};   // step st + 2 begins a group if this one does
        constexpr std::integral_constant<bool, half == 1> next_second{};  // ... and st + 3 if this one does not
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int cur = i & 1, nxt = cur ^ 1;
            __builtin_amdgcn_sched_barrier(0);
            if (i == 3) {
                wait_and_meet(std::integral_constant<int, kLoads + (half == 0 ? 1 : 0)>{});
                issue_portion(st + 3, next_second, buf, 0);
                if (half == 1) read_sz(((st + 1) >> 1) & 1);
                read_words(w[half ^ 1], buf1);
            } else {
                issue_portion(st + 2, next_first, buf2, 2 + 2 * i);
            }
            __builtin_amdgcn_sched_barrier(0);
            b1 = w[half][1].operand(i, aff[1], k6400);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                acc[tm][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[cur][tm], b0, acc[tm][0], 0, 0, 0);
                af[nxt][tm] = i < 3 ? a_frag(buf, i + 1, tm) : a_frag(buf1, 0, tm);
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (i == 3) issue_portion(st + 3, next_second, buf, 1);
            else issue_portion(st + 2, next_first, buf2, 3 + 2 * i);
            __builtin_amdgcn_sched_barrier(0);
            if (i == 3 && half == 1) {
                aff[0].set(szw[0]);
                aff[1].set(szw[1]);
            }
            b0 = i < 3 ? w[half][0].operand(i + 1, aff[0], k6400) : w[half ^ 1][0].operand(0, aff[0], k6400);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) acc[tm][1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[cur][tm], b1, acc[tm][1], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // Start: steps 0 and 1, and the first two portions of step 2 (the others go out in step 0).
#pragma unroll
    for (int j = 0; j <= kLoads; ++j) issue_one(0, true, 0, j);
#pragma unroll
    for (int j = 0; j < kLoads; ++j) issue_one(1, false, 1, j);
    issue_portion(2, std::true_type{}, 2, 0);
    issue_portion(2, std::true_type{}, 2, 1);
    constexpr int kStarted = (2 * (kLoads + 1) + 7) / 8;            // copies j of kLoads + 1 with 8 j / (kLoads + 1) < 2
    wait_and_meet(std::integral_constant<int, kLoads + kStarted>{});
    read_sz(0);
    read_words(w[0], 0);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) af[0][tm] = a_frag(0, 0, tm);
    aff[0].set(szw[0]);
    aff[1].set(szw[1]);
    b0 = w[0][0].operand(0, aff[0], k6400);
    int buf = 0;
    for (int u = 0; u < U; ++u) {
        const int buf1 = buf == 2 ? 0 : buf + 1, buf2 = buf == 0 ? 2 : buf - 1;
        do_step(std::integral_constant<int, 0>{}, 2 * u, buf, buf1, buf2);
        do_step(std::integral_constant<int, 1>{}, 2 * u + 1, buf1, buf2, buf);
        buf = buf2;
    }
    if (KG > 1)                                         // a group of waves with a shorter share of K meets the other one at its barriers
        for (int u = U; u < U_part; ++u) { block_barrier(); block_barrier(); }
    wait_and_meet(std::integral_constant<int, 0>{});    // the copies issued past the end have landed too, and everybody is done: LDS is free

    // the K groups meet: group 1 leaves its accumulators in LDS, group 0 adds them to its own
    if constexpr (KG > 1) {
        static_assert(KG <= 2, "the hand-over below is written for two K groups");
        float *hand = reinterpret_cast<float *>(lds) + (size_t)wave * (TM * kTN * 16 * 64);
        if (kg == 1) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < kTN; ++tn)
#pragma unroll
                    for (int v = 0; v < 16; ++v) hand[((tm * kTN + tn) * 16 + v) * 64 + lane] = acc[tm][tn][v];
        }
        __syncthreads();
        if (kg == 1) return;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < kTN; ++tn)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[tm][tn][v] += hand[((tm * kTN + tn) * 16 + v) * 64 + lane];
    }

    // up-projection: 2r extra K columns, t_hi and t_lo against the same B^T rows
    if (p.r > 0 && part == 0) {
        // 64 taps at a time through LDS.  Every lane fetching its own 16 bytes of
        // its own row - 32 rows per load, some forty loads per wave, all at once - kept the address unit busy for
        // microseconds at the end of every block; copied into LDS, a load moves 1 KiB of whole rows (eight lanes per
        // 128-byte row of B^T, sixteen per 256-byte row of t_hi | t_lo), and the operands come out of LDS.  Rows are
        // stored with the position of each 16-byte piece XOR-ed with the row number, as the activation tiles are.
        // Taps past r, rows past N and tokens past M lie beyond the descriptors or are aimed there: zeros.
        const __amdgpu_buffer_rsrc_t bbuf = buffer_of(p.Bt + (size_t)n0 * p.r, (long)min(kBN, p.N - n0) * p.r * 2);
        const __amdgpu_buffer_rsrc_t tbuf = buffer_of(p.thl + (size_t)m0 * (2 * p.r), (long)min(kBM, p.M - m0) * p.r * 4);
        constexpr int kNowhere = 0x40000000;            // beyond every buffer
        unsigned char *const lds_b = lds;               // [256 rows][8 pieces]
        unsigned char *const lds_t = lds_b + kBN * 128; // [kBM rows][16 pieces: 8 of t_hi, 8 of t_lo]
        for (int c0 = 0; c0 < p.r; c0 += 64) {
            block_barrier();                            // everybody is done with what LDS held before
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int first = (wave * 8 + i) * 8, row = first + (lane >> 3), tap = c0 + ((lane & 7) ^ (row & 7)) * 8;
                copy16_to_lds(bbuf, tap < p.r ? (row * p.r + tap) * 2 : kNowhere, 0, lds0 + first * 128);
            }
#pragma unroll
            for (int j = 0; j < 2 * TM; ++j) {
                const int first = (wave * 2 * TM + j) * 4, row = first + (lane >> 4), piece = (lane & 15) ^ (row & 15), tap = c0 + (piece & 7) * 8;
                copy16_to_lds(tbuf, tap < p.r ? (row * 2 * p.r + (piece < 8 ? tap : p.r + tap)) * 2 : kNowhere, 0, lds0 + kBN * 128 + first * 256);
            }
            wait_and_meet(std::integral_constant<int, 0>{});
            const int steps = min(4, (p.r - c0 + 15) / 16);
            for (int st = 0; st < steps; ++st) {
                half8_t bf[kTN];
#pragma unroll
                for (int tn = 0; tn < kTN; ++tn) {
                    const int row = wave * (kTN * 32) + tn * 32 + col;
                    bf[tn] = *reinterpret_cast<const half8_t *>(lds_b + row * 128 + (((2 * st + h) ^ (row & 7)) << 4));
                }
#pragma unroll
                for (int half = 0; half < 2; ++half)
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm) {
                        const int row = tm * 32 + col;
                        const half8_t t8 = *reinterpret_cast<const half8_t *>(lds_t + row * 256 + (((8 * half + 2 * st + h) ^ (row & 15)) << 4));
#pragma unroll
                        for (int tn = 0; tn < kTN; ++tn)
                            acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(t8, bf[tn], acc[tm][tn], 0, 0, 0);
                    }
            }
        }
    }

    // store of y: accumulator register v of a lane holds row 8*(v/4) + 4*h + v%4, column `col`
    if (p.ksplit == 1 && p.N % 8 == 0) {
        // Stored straight from the accumulators, an instruction writes two 64-byte pieces of two rows, ninety-six such
        // instructions per wave, and the address unit is the busy one again.  Each wave turns 32 rows at a time round in LDS
        // instead (64 fp16 a row, 144 bytes apart so that the two halves of the wave fall on different
        // banks) and writes whole 128-byte row pieces, 16 bytes per lane, eight rows per instruction.
        static_assert(kBN == kPrefillColumns, "the rule that cuts a layer into blocks counts column blocks of this width");
        static_assert(kTN == 2, "a wave's output rows are 64 columns wide");
        unsigned char *const out = lds + wave * (32 * T::kOutRow);
        block_barrier();                                // everybody is done with what LDS held before
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
            for (int tn = 0; tn < kTN; ++tn)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    *reinterpret_cast<half_t *>(out + (8 * (v / 4) + 4 * h + (v % 4)) * T::kOutRow + (tn * 32 + col) * 2) = (half_t)acc[tm][tn][v];
            // (the wave reads what itself wrote: LDS keeps a wave's accesses in order)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = i * 8 + (lane >> 3), piece = lane & 7;
                const uint4 v = *reinterpret_cast<const uint4 *>(out + row * T::kOutRow + piece * 16);
                const int m = m0 + tm * 32 + row, n = nw + piece * 8;
                if (m < p.M && n < p.N) *reinterpret_cast<uint4 *>(p.y + (size_t)m * p.N + n) = v;
            }
        }
        return;
    }
#pragma unroll
    for (int tn = 0; tn < kTN; ++tn) {
        const int n = nw + tn * 32 + col;
        if (n >= p.N) continue;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + tm * 32 + 8 * (v / 4) + 4 * h + (v % 4);
                if (m >= p.M) continue;
                if (p.ksplit > 1) p.ypart[((size_t)part * p.M + m) * p.N + n] = acc[tm][tn][v];
                else p.y[(size_t)m * p.N + n] = __builtin_bit_cast(uint16_t, (half_t)acc[tm][tn][v]);
            }
        }
    }
}

// y = sum of the K parts' fp32 partial results, in index order (only where K is split over blocks).
__global__ __launch_bounds__(256) void fbq_sum_parts_kernel(const float *__restrict__ ypart, uint16_t *__restrict__ y, size_t total, int parts)
{
    if (total % 4 != 0) {                               // (the parts after the first are not 16-byte aligned then)
        for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
            float acc = ypart[i];
            for (int pt = 1; pt < parts; ++pt) acc += ypart[(size_t)pt * total + i];
            y[i] = __builtin_bit_cast(uint16_t, (half_t)acc);
        }
        return;
    }
    for (size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4; i < total; i += (size_t)gridDim.x * 256 * 4) {
        float4 acc = *reinterpret_cast<const float4 *>(ypart + i);
        for (int pt = 1; pt < parts; ++pt) {
            const float4 v = *reinterpret_cast<const float4 *>(ypart + (size_t)pt * total + i);
            acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
        }
        const half2_t lo = half2_t{(half_t)acc.x, (half_t)acc.y}, hi = half2_t{(half_t)acc.z, (half_t)acc.w};
        *reinterpret_cast<uint2 *>(y + i) = make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
    }
}

// ------------------------------------------------------------------ activation pre-pass

// xp[m][64 v + 8 (l ^ piece_key(m % 16)) + e] = x[m][64 v + 32 (l / 4) + slot_source(8 (l % 4) + e)]
// for piece l = 0..7 of every 64-wide step v; one thread per 32 activations (q4: the 64 bytes of piece b of row m).
template <int BITS>
__device__ __forceinline__ void arrange_store(const uint4 (&q4)[4], uint16_t *__restrict__ xp, int K, int m, int b)
{
    half_t v[32];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t wds[4] = {q4[i].x, q4[i].y, q4[i].z, q4[i].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const half2_t hh = h2_of(wds[j]);
            v[i * 8 + j * 2] = hh.x;
            v[i * 8 + j * 2 + 1] = hh.y;
        }
    }
    uint16_t *dst = xp + (size_t)m * K + (b / 2) * 64;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        half2_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            o[j] = half2_t{v[slot_source<BITS>(i * 8 + 2 * j)], v[slot_source<BITS>(i * 8 + 2 * j + 1)]};
        const int l = 4 * (b % 2) + i;
        *reinterpret_cast<uint4 *>(dst + 8 * (l ^ piece_key(m & 15))) =
            make_uint4(__builtin_bit_cast(uint32_t, o[0]), __builtin_bit_cast(uint32_t, o[1]),
                       __builtin_bit_cast(uint32_t, o[2]), __builtin_bit_cast(uint32_t, o[3]));
    }
}

// Items [first, first + count) of a row-major list of (row, 32-wide piece) pairs, `nb` pieces per row starting at piece
// b0 of row m0: `stride` threads share them, thread `t` takes t, t + stride, ...  The loads of kArrangeBatch items are
// requested before the first of them is stored (item by item, every item was a round trip to memory).
constexpr int kArrangeBatch = 3;
template <int BITS>
__device__ __forceinline__ void arrange_items(const uint16_t *__restrict__ x, uint16_t *__restrict__ xp, int K, int m0, int b0, int nb,
                                              long count, long t, long stride)
{
    for (long i0 = t; i0 < count; i0 += stride * kArrangeBatch) {
        uint4 q4[kArrangeBatch][4];
#pragma unroll
        for (int k = 0; k < kArrangeBatch; ++k) {
            const long idx = min(i0 + k * stride, count - 1);          // (past the end: the last item again, not stored)
            const uint4 *src = reinterpret_cast<const uint4 *>(x + (size_t)(m0 + idx / nb) * K + (b0 + idx % nb) * 32);
#pragma unroll
            for (int i = 0; i < 4; ++i) q4[k][i] = src[i];
        }
#pragma unroll
        for (int k = 0; k < kArrangeBatch; ++k) {
            const long idx = i0 + k * stride;
            if (idx < count) arrange_store<BITS>(q4[k], xp, K, m0 + (int)(idx / nb), b0 + (int)(idx % nb));
        }
    }
}

// Scale and zero of 64 rows and 32 groups (tile `t` of the layer's), from [N][G] each to one word per row and group,
// [G][Np]: the fused kernel fetches a group's 256 of them as whole lines.  Rows past N become zeros.  256 threads.
constexpr int kSzRows = 64, kSzGroups = 32;
__device__ void arrange_scales(const uint16_t *__restrict__ scales, const uint16_t *__restrict__ zeros, uint32_t *__restrict__ sz, int N, int Np,
                               int G, int t, uint32_t (*turn)[kSzRows + 1])
{
    const int row_tiles = Np / kSzRows, n0 = (t % row_tiles) * kSzRows, g0 = (t / row_tiles) * kSzGroups;
    const int tid = threadIdx.x;
    uint32_t v[kSzRows / 8];
#pragma unroll
    for (int i = 0; i < kSzRows / 8; ++i) {
        const int n = n0 + i * 8 + tid / 32, g = g0 + tid % 32;
        const bool on = n < N && g < G;
        const size_t at = on ? (size_t)n * G + g : 0;
        v[i] = (uint32_t)scales[at] | ((uint32_t)zeros[at] << 16);
        if (!on) v[i] = 0;
    }
#pragma unroll
    for (int i = 0; i < kSzRows / 8; ++i) turn[tid % 32][i * 8 + tid / 32] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSzGroups / 4; ++i) {
        const int g = g0 + i * 4 + tid / kSzRows;
        if (g < G) sz[(size_t)g * Np + n0 + tid % kSzRows] = turn[i * 4 + tid / kSzRows][tid % kSzRows];
    }
}
static int sz_tiles(int N, int G) { return ceil_div(N, kBN) * (kBN / kSzRows) * ceil_div(G, kSzGroups); }

// What the pre-pass reads and writes besides the down-projection's own arguments.
struct ArrangeParams {
    const uint16_t *x, *scales, *zeros;
    uint16_t *xp;
    uint32_t *sz;
    int M, N, K, G, Np;
    int sz_tiles;
};

// The whole of x, for a layer without a sub-branch (with one, the down-projection's blocks arrange what they read).
// The first sz_tiles blocks arrange scales and zeros.
template <int BITS>
__global__ __launch_bounds__(256) void fbq_arrange_x_kernel(const ArrangeParams a)
{
    __shared__ uint32_t turn[kSzGroups][kSzRows + 1];
    if ((int)blockIdx.x < a.sz_tiles) {
        arrange_scales(a.scales, a.zeros, a.sz, a.N, a.Np, a.G, blockIdx.x, turn);
        return;
    }
    arrange_items<BITS>(a.x, a.xp, a.K, 0, 0, a.K / 32, (long)a.M * (a.K / 32), (long)(blockIdx.x - a.sz_tiles) * 256 + threadIdx.x,
                        (long)(gridDim.x - a.sz_tiles) * 256);
}

// ------------------------------------------------------------------ down-projection (prefill)

// Stage 1: partial[s][m][j] = sum over K slice s of x[m][k] * At[j][k], for one 32-row tile of tokens and all r
// columns.  RT = 32-column tiles (r <= 32 * RT).  The block also writes the arranged copy of the activations it
// reads (its 32 rows, its K slice): one pass over x serves both, and the re-ordering needs no launch of its own.
//
// The slice is walked in chunks of 64: the chunk's 32 rows of x and 32 RT rows of A^T (128 bytes each) are copied
// into LDS, eight whole rows per copy, three chunks ahead of the one worked on (a ring of four; with two chunks of 128 and
// a wait for everything in flight between them, every chunk was a round trip to memory: 2048 x 8192, r = 128, took 35 us and takes 25; 1024 x 4096, r = 64, 10.9 and 7.0).
// (Fetched by the lanes themselves, 16 bytes of one row per lane and instruction, the operands of a
// long slice kept the CU's address unit busy longer than everything else in this kernel took.)  Rows are stored
// with the position of each 16-byte piece XOR-ed with a key of the row, as the fused kernel's tiles are.  Of a
// chunk's four K steps of 16, wave w multiplies step w; the four waves' tiles meet in LDS at the end.
constexpr int kDownStages = 4;
template <int BITS, int RT>
__global__ __launch_bounds__(256) void fbq_down_proj_prefill_kernel(const ArrangeParams a, const uint16_t *__restrict__ At, float *__restrict__ partial,
                                                                    int r, int kslice, int slices, int by_xcd)
{
    constexpr int kRows = 32 + 32 * RT;                 // rows of a chunk in LDS: the tokens, then the columns of A
    constexpr int kChunkBytes = kRows * 128, kCopies = kRows / 8 / 4;   // copies per wave and chunk
    __shared__ __attribute__((aligned(1024))) unsigned char lds_down[kDownStages * kChunkBytes];   // the ring; afterwards float [4][32][32 RT]
    static_assert(sizeof(lds_down) <= 160 * 1024 && sizeof(lds_down) >= 4 * 32 * 32 * RT * sizeof(float), "the ring must fit the CU's LDS and hold the waves' tiles");
    static_assert(sizeof(lds_down) >= kSzGroups * (kSzRows + 1) * sizeof(uint32_t), "the ring must hold a tile of scales");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, h = lane >> 5;
    if ((int)blockIdx.y >= slices) {                    // the rows of blocks behind the K slices arrange scales and zeros
        const int t = ((int)blockIdx.y - slices) * gridDim.x + blockIdx.x;
        if (t < a.sz_tiles) arrange_scales(a.scales, a.zeros, a.sz, a.N, a.Np, a.G, t, reinterpret_cast<uint32_t (*)[kSzRows + 1]>(lds_down));
        return;
    }
    const int M = a.M, K = a.K;
    // The first `by_xcd` slices (a multiple of eight): blocks go to the XCDs round-robin by linear id, and eight slices at a time get an
    // XCD each, with all of their token tiles one after the other.
    int tile = blockIdx.x, slice = blockIdx.y;
    if (slice < by_xcd) {
        const int id = slice * gridDim.x + tile, i = id / kXcds;
        slice = id % kXcds + kXcds * (i / (int)gridDim.x);
        tile = i % (int)gridDim.x;
    }
    const int m0 = tile * 32;
    const int k_lo = slice * kslice, k_hi = min(K, k_lo + kslice);
    const int chunks = (k_hi - k_lo) / kStepK;          // K and the slices are whole groups of 128

    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(a.x + (size_t)m0 * K, (long)min(32, M - m0) * K * 2);   // (tokens past M, columns past r: zeros)
    const __amdgpu_buffer_rsrc_t abuf = buffer_of(At, (long)r * K * 2);
    const uint32_t lds0 = lds_offset(lds_down);
    // copy i of a chunk moves rows 8 i .. 8 i + 7 (lane l: row 8 i + l / 8, put at position l % 8 of it, i.e. piece position ^ key);
    // the first four are the tokens', one per wave
    const int lane_row = lane >> 3;
    auto copy_chunk = [&](int c, int stage) __attribute__((always_inline)) {
        const uint32_t base = lds0 + stage * kChunkBytes;
#pragma unroll
        for (int j = 0; j < kCopies; ++j) {
            const int i = j * 4 + wave, row = 8 * i + lane_row;
            const int off = ((row - (j == 0 ? 0 : 32)) * K + ((lane & 7) ^ piece_key(row & 15)) * 8) * 2, at = (k_lo + c * kStepK) * 2;
            copy16_to_lds(j == 0 ? xbuf : abuf, off, at, base + i * 1024);
        }
    };

    float16_t acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[rt][v] = 0.0f;

    for (int c = 0; c < min(kDownStages - 1, chunks); ++c) copy_chunk(c, c);
    // re-ordered copy: thread t writes position t % 8 of row t / 8 of the chunk, i.e. piece l = (t % 8) ^ key of its step
    const int arow = tid >> 3, apos = tid & 7, al = apos ^ piece_key(arow & 15);
    uint16_t *const xp = a.xp + (size_t)(m0 + arow) * K + k_lo + apos * 8;
    const bool astore = m0 + arow < M;
    for (int c = 0; c < chunks; ++c) {
        // chunk c has landed - with every store of the copy counted as if it were one more copy in flight - and everybody is
        // done with chunk c - 1, whose stage the next copies go to
        if (c + kDownStages - 2 < chunks) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kDownStages - 2) * kCopies) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (c + kDownStages - 1 < chunks) copy_chunk(c + kDownStages - 1, (c + kDownStages - 1) % kDownStages);
        const unsigned char *base = lds_down + (c % kDownStages) * kChunkBytes;
        const int pc = 2 * wave + h;                    // the 16-byte piece with this lane's k of the wave's step
        const half8_t af = *reinterpret_cast<const half8_t *>(base + col * 128 + ((pc ^ piece_key(col & 15)) << 4));
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const half8_t bf = *reinterpret_cast<const half8_t *>(base + (32 + rt * 32 + col) * 128 + ((pc ^ piece_key(col & 15)) << 4));
            acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af, bf, acc[rt], 0, 0, 0);
        }
        const unsigned char *row = base + arow * 128;
        uint4 out;
        if constexpr (BITS == 4) {                      // the eight activations of one piece, re-ordered among themselves
            const uint4 q = *reinterpret_cast<const uint4 *>(row + (apos << 4));   // (piece al sits at position apos)
            out.x = __builtin_amdgcn_perm(q.z, q.x, 0x05040100u); out.y = __builtin_amdgcn_perm(q.z, q.x, 0x07060302u);
            out.z = __builtin_amdgcn_perm(q.w, q.y, 0x05040100u); out.w = __builtin_amdgcn_perm(q.w, q.y, 0x07060302u);
        } else {
            uint16_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int k = 0;                              // slot_source of a piece known only at run time
#pragma unroll
                for (int pi = 0; pi < 4; ++pi) k = (al & 3) == pi ? slot_source<BITS>(8 * pi + e) : k;
                k += 32 * (al >> 2);
                v[e] = *reinterpret_cast<const uint16_t *>(row + (((k >> 3) ^ piece_key(arow & 15)) << 4) + (k & 7) * 2);
            }
            out.x = v[0] | ((uint32_t)v[1] << 16); out.y = v[2] | ((uint32_t)v[3] << 16);
            out.z = v[4] | ((uint32_t)v[5] << 16); out.w = v[6] | ((uint32_t)v[7] << 16);
        }
        if (astore) *reinterpret_cast<uint4 *>(xp + c * kStepK) = out;
    }

    __syncthreads();                                    // the ring is free
    float *sum = reinterpret_cast<float *>(lds_down);
    constexpr int ld = 32 * RT;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[(wave * 32 + 8 * (v / 4) + 4 * h + (v % 4)) * ld + rt * 32 + col] = acc[rt][v];
    __syncthreads();
    float *out = partial + (size_t)slice * M * r;
    for (int idx = tid; idx < 32 * ld; idx += 256) {
        const int i = idx / ld, j = idx % ld;
        if (m0 + i < M && j < r) out[(size_t)(m0 + i) * r + j] = ((sum[i * ld + j] + sum[(32 + i) * ld + j]) + sum[(64 + i) * ld + j]) + sum[(96 + i) * ld + j];
    }
}

// Stage 2: t = sum of the slices in slice order, written as t_hi = fp16(t), t_lo = fp16(t - t_hi).
__global__ __launch_bounds__(256) void fbq_down_proj_finish_kernel(const float *__restrict__ partial, uint16_t *__restrict__ thl,
                                                                   int M, int r, int slices)
{
    const size_t total = (size_t)M * r;
    for (size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (size_t)gridDim.x * 256) {
        // eight slices per round trip to memory, added in slice order
        float t = 0.0f;
        for (int s0 = 0; s0 < slices; s0 += 8) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = partial[(size_t)min(s0 + k, slices - 1) * total + idx];
#pragma unroll
            for (int k = 0; k < 8; ++k) t += s0 + k < slices ? v[k] : 0.0f;
        }
        const size_t m = idx / r, j = idx - m * r;
        const half_t hi = (half_t)t;
        const half_t lo = (half_t)(t - (float)hi);
        thl[m * (2 * r) + j] = __builtin_bit_cast(uint16_t, hi);
        thl[m * (2 * r) + r + j] = __builtin_bit_cast(uint16_t, lo);
    }
}

// workspace: the arranged copy of x ([M][K] fp16), scale | zero by group ([G][Np] words), then [M][2r] fp16 (t_hi | t_lo),
// then down_slices x [M][r] fp32 partial sums, then - where K is split over blocks - ksplit x [M][N] fp32 partial outputs
static size_t pad256(size_t b) { return (b + 255) & ~(size_t)255; }
static size_t xp_bytes(int M, int K) { return pad256((size_t)M * K * sizeof(uint16_t)); }
static size_t sz_bytes(int N, int K) { return (size_t)(K / kGroup) * ceil_div(N, kBN) * kBN * sizeof(uint32_t); }
static size_t thl_bytes(int M, int r) { return pad256((size_t)M * 2 * r * sizeof(uint16_t)); }
static size_t down_partial_bytes(int M, int K, int r) { return pad256((size_t)down_slices(M, K) * M * r * sizeof(float)); }

size_t prefill_workspace_bytes(int M, int N, int K, int r)
{
    const int split = prefill_cut(M, N, K, r).ksplit;
    return xp_bytes(M, K) + sz_bytes(N, K) + thl_bytes(M, r) + down_partial_bytes(M, K, r) + (split > 1 ? (size_t)split * M * N * sizeof(float) : 0);
}

struct PrefillScratch {
    uint16_t *xp;
    uint32_t *sz;
    uint16_t *thl;
    float *partial, *ypart;
};
static PrefillScratch scratch_of(const LinearArgs &a)
{
    char *w = (char *)a.workspace;
    PrefillScratch s;
    s.xp = (uint16_t *)w;       w += xp_bytes(a.M, a.K);
    s.sz = (uint32_t *)w;       w += sz_bytes(a.N, a.K);
    s.thl = (uint16_t *)w;      w += thl_bytes(a.M, a.r);
    s.partial = (float *)w;     w += down_partial_bytes(a.M, a.K, a.r);
    s.ypart = (float *)w;
    return s;
}

// Before the fused kernel: x and the scales re-ordered into the workspace and, with a sub-branch, t = x.A.  With a
// sub-branch two launches (K slices of the down-projection, whose blocks also write the re-ordered x; then the slices'
// sums as t_hi | t_lo); without one, the re-ordering alone.
hipError_t launch_prepass_prefill(const LinearArgs &a, hipStream_t stream)
{
    const PrefillScratch s = scratch_of(a);
    const int G = a.K / kGroup;
    const ArrangeParams ap{a.x, a.scales, a.zeros, s.xp, s.sz, a.M, a.N, a.K, G, ceil_div(a.N, kBN) * kBN, sz_tiles(a.N, G)};
    if (a.r == 0) {
        const size_t items = (size_t)a.M * (a.K / 32);
        const int blocks = (int)std::min<size_t>(4096, (items + 255) / 256) + ap.sz_tiles;
        if (a.bits == 4) hipLaunchKernelGGL(fbq_arrange_x_kernel<4>, dim3(blocks), dim3(256), 0, stream, ap);
        else hipLaunchKernelGGL(fbq_arrange_x_kernel<3>, dim3(blocks), dim3(256), 0, stream, ap);
        return hipGetLastError();
    }
    const int kslice = down_slice_len(a.M, a.K);
    const int slices = down_slices(a.M, a.K);
    const int by_xcd = down_slices_by_xcd(a.M, a.N, a.K, a.r);
    const int row_tiles = ceil_div(a.M, 32);
    const dim3 grid(row_tiles, slices + ceil_div(ap.sz_tiles, row_tiles));
    const int rt = ceil_div(a.r, 32);
#define FBQ_DOWN(B, R) hipLaunchKernelGGL((fbq_down_proj_prefill_kernel<B, R>), grid, dim3(256), 0, stream, ap, a.At, s.partial, a.r, kslice, slices, by_xcd)
    if (a.bits == 4) {
        if (rt <= 1) FBQ_DOWN(4, 1); else if (rt <= 2) FBQ_DOWN(4, 2); else if (rt <= 4) FBQ_DOWN(4, 4); else FBQ_DOWN(4, 8);
    } else {
        if (rt <= 1) FBQ_DOWN(3, 1); else if (rt <= 2) FBQ_DOWN(3, 2); else if (rt <= 4) FBQ_DOWN(3, 4); else FBQ_DOWN(3, 8);
    }
#undef FBQ_DOWN
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int blocks = std::min(1024, ceil_div(a.M * a.r, 256));
    hipLaunchKernelGGL(fbq_down_proj_finish_kernel, dim3(blocks), dim3(256), 0, stream, s.partial, s.thl, a.M, a.r, slices);
    return hipGetLastError();
}

template <int BITS, int TM, int KG>
static void launch_tile(const PrefillParams &p, dim3 grid, hipStream_t stream)
{
    hipLaunchKernelGGL((fbq_gemm_kernel<BITS, TM, KG>), grid, dim3(GemmTile<BITS, TM, KG>::kThreads), 0, stream, p);
}

// `columns` column blocks from p.col0 on, in tiles of 32 tm rows
template <int BITS>
static hipError_t launch_columns(PrefillParams p, int tm, bool single, int columns, hipStream_t stream)
{
    p.row_blocks = ceil_div(p.M, 32 * tm);
    p.full_cols = (columns / kXcds) * kXcds;
    p.full_slots = (columns / kXcds) * p.row_blocks * p.ksplit;
    p.rem_blocks = (columns % kXcds) * p.row_blocks * p.ksplit;
    const dim3 grid(kXcds * (p.full_slots + ceil_div(p.rem_blocks, kXcds)));
    switch (single ? -tm : tm) {
    case 8: launch_tile<BITS, 8, 1>(p, grid, stream); break;
    case 6: launch_tile<BITS, 6, 1>(p, grid, stream); break;
    case 4: launch_tile<BITS, 4, 2>(p, grid, stream); break;
    case 3: launch_tile<BITS, 3, 2>(p, grid, stream); break;
    case 2: launch_tile<BITS, 2, 2>(p, grid, stream); break;
    case -4: launch_tile<BITS, 4, 1>(p, grid, stream); break;
    case -3: launch_tile<BITS, 3, 1>(p, grid, stream); break;
    default: launch_tile<BITS, 2, 1>(p, grid, stream); break;
    }
    return hipGetLastError();
}

hipError_t launch_gemm_prefill(const LinearArgs &a, hipStream_t stream)
{
    const PrefillScratch s = scratch_of(a);
    const PrefillCut c = prefill_cut(a.M, a.N, a.K, a.r);
    PrefillParams p;
    p.qw = a.qw; p.sz = s.sz; p.Bt = a.Bt; p.y = a.y; p.xp = s.xp; p.thl = s.thl;
    p.M = a.M; p.N = a.N; p.K = a.K; p.r = a.r;
    p.row_words = (int)row_words(a.K, a.bits);
    p.G = a.K / kGroup;
    const int nb = ceil_div(a.N, kBN);
    p.Np = nb * kBN;
    p.ksplit = c.ksplit;
    p.ypart = s.ypart;
    p.col0 = 0;
    hipError_t e = a.bits == 4 ? launch_columns<4>(p, c.tm, c.single, c.columns, stream) : launch_columns<3>(p, c.tm, c.single, c.columns, stream);
    if (e == hipSuccess && c.tail_tm) {
        p.col0 = c.columns;
        e = a.bits == 4 ? launch_columns<4>(p, c.tail_tm, false, nb - c.columns, stream) : launch_columns<3>(p, c.tail_tm, false, nb - c.columns, stream);
    }
    if (e == hipSuccess && p.ksplit > 1) {
        const size_t total = (size_t)a.M * a.N;
        hipLaunchKernelGGL(fbq_sum_parts_kernel, dim3((unsigned)std::min<size_t>(2048, (total / 4 + 255) / 256)), dim3(256), 0, stream,
                           p.ypart, a.y, total, p.ksplit);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace fbq
