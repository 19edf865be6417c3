// Layer-wise reconstruction (Alg. 1, Sec. 4.2): one gradient-descent iteration on the sub-branch
// of one layer.
//
// The loss and its gradient depend on the calibration activations X [T,K] only through
// H = X^T X (Sec. 4.2: L = tr(Delta_F H Delta_F^T), dL/dSigma = -2 Delta_F H with the feedback
// detached), so H is formed once per layer and an iteration is
//
//   A16, B16   <- fp16 of the fp32 masters                               (cast kernel)
//   q, s, z    <- Q(W - Sigma16)               feedback quantizer  } fbq_quantize_kernel, Delta_F
//   Delta_F    <- (W - Sigma16) - s (q - z)                        } from its registers
//   Q          <- Bt^T Delta_F        [r,K]                              (GEMM, K split)
//   dL/dAt     <- -2 Q H              [r,K]    } one GEMM on the stacked                                 
//   V^T        <- At H                [r,K]    } operand [Q; At], K split
//   dL/dBt     <- -2 Delta_F V        [N,r]                              (GEMM, K split)
//   L          <- sum (Delta_F^T Delta_F) o H  only if the caller asks   (symmetric product, N K^2 flop, + reduction)
//   masters    <- masters - lr gradient                                  (both in the last launch, with the split sums of dL/dBt:
//                                                                         a call that fails on the way moves neither)
//
// with Sigma[n,k] = sum_j Bt[n,j] At[j,k] in the device layouts At [r,K], Bt [N,r].  The gradients need only products with
// r rows or columns (4 N K r + 4 r K^2 flop) because H is symmetric: Delta_F H At^T = Delta_F (At H)^T.  The loss is the one
// quantity that needs a contraction over N and K x K, and as tr(Delta_F H Delta_F^T) = sum (Delta_F^T Delta_F) o H that is a
// symmetric one, half the work of Delta_F H.
//
// Two matrix-core kernels (v_mfma_f32_32x32x16_f16, fp16 in, fp32 accumulate): fbq_gemm_nt_kernel for the products with r rows or
// columns and fbq_syrk_kernel for A^T A.  Operands whose rows do not run along the contraction (X and Delta_F, but for the last product) lie as they are
// and are turned by the reads from LDS (ds_read_b64_tr_b16).  Both pass their operands through LDS by buffer_load ... lds, several steps of 64 ahead; rows (whole
// cache lines) are stored with their 16-byte pieces XOR-swizzled so that reads have no bank conflict; rows past the end of an
// operand are fetched through a bounds-checked buffer descriptor and arrive as zeros.  fp16 operands carry Delta_F times 256 and H times the caller's h_scale, so
// that neither leaves the normal range; the factors come out again in the epilogues.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "fbq_internal.h"
#include "fbq_lds_copy.h"

namespace fbq {

typedef _Float16 half_t;
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kStepK = 64;           // k per step: one 128-byte row segment per operand row
constexpr float kDeltaGain = 256.0f; // Delta_F is stored as fp16(256 Delta_F)
constexpr int kXcds = 8;

// An operand whose rows run along the contraction, [k][column], in LDS: rows of PIECES 16-byte pieces, piece p of row k at p ^ turned_key.
// Lane 16 b + i of a transposed read asks for 8 bytes of row i / 4 and gets column i of its sixteen lanes' 4 x 16 block: two reads are the eight k of
// a matrix operand's lane.  The key puts the four rows of a block, 32 bytes each for 16 lanes and 64 for 32, on different banks,
// whether the LDS serves 128 or 256 bytes per clock.
__device__ __forceinline__ constexpr int turned_key(int k, int pieces) { return pieces == 16 ? (4 * (k & 3)) ^ (k & 2) : 2 * (k & 3); }
// Of this lane's 8 bytes of the operand's first eight rows (lanes 32 and up: the second eight), columns 8 first_piece and up
template <int PIECES>
__device__ __forceinline__ int turned_offset(int lane, int first_piece)
{
    const int k = (lane & 15) >> 2, piece = first_piece + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    return (8 * (lane >> 5) + k) * (PIECES * 16) + ((piece ^ turned_key(k, PIECES)) << 4) + 8 * (lane & 1);
}
template <int PIECES>
__device__ __forceinline__ half8_t read_turned(const unsigned char *at)
{
    typedef __fp16 four_t __attribute__((vector_size(8)));
    typedef __attribute__((address_space(3))) four_t lds_four_t;
    const half4_t lo = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_four_t *)(__attribute__((address_space(3))) const void *)at));
    const half4_t hi = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_four_t *)(__attribute__((address_space(3))) const void *)(at + 4 * PIECES * 16)));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

struct GemmArgs {
    const uint16_t *A;   // [Mr][lda] fp16
    const uint16_t *B;   // [Nr][ldb] fp16; TURNED: [b_rows][ldb], rows along the contraction, b_rows <= Kd
    int Mr, Nr, Kd;      // Kd a multiple of 64
    int lda, ldb;        // elements
    int b_rows;
    // store epilogue (either may be absent)
    float *C32; int ldc32; float alpha; int c32_rows;   // C32[m,n] = alpha acc for rows m < c32_rows
    uint16_t *C16; int ldc16; float beta; int c16_row0; // C16[m - c16_row0, n] = fp16(beta acc) for rows m >= c16_row0
    // K split over `splits` blocks per tile (few tiles, long K): raw sums go to part [splits][Mr][Nr]
    // and fbq_sum_splits_kernel applies the store epilogue
    int splits; float *part;
};

__device__ __forceinline__ void store_result(const GemmArgs &g, int m, int n, float a)
{
    if (g.C32 && m < g.c32_rows) g.C32[(size_t)m * g.ldc32 + n] = g.alpha * a;
    if (g.C16 && m >= g.c16_row0) g.C16[(size_t)(m - g.c16_row0) * g.ldc16 + n] = __builtin_bit_cast(uint16_t, (half_t)(g.beta * a));
}

// WM x WN: 32x32 tiles a wave owns (rows x columns); the block's 2 x 2 waves cover 64 WM x 64 WN.
// These products have few rows or columns (r or 2r) and read one large operand once: bound by memory.  The steps of 64 pass
// through a ring of four stages in LDS, copied there without passing registers three steps ahead (through registers, one step
// ahead, the three products of a 4096 x 4096 step at r = 64 took 43 us and take 34).
constexpr int kNtStages = 4;
// TURNED: B's rows run along the contraction and are turned by the reads from LDS (Q = B^T Delta_F: the quantizer writes Delta_F once).
template <int WM, int WN, bool TURNED>
__global__ __launch_bounds__(256) void fbq_gemm_nt_kernel(GemmArgs g)
{
    constexpr int BM = 64 * WM, BN = 64 * WN;
    constexpr int kStageBytes = (BM + BN) * kStepK * 2;
    constexpr int kCopies = (BM + BN) / 8 / 4;          // per wave and step, eight rows each
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kNtStages * kStageBytes];   // [stage][A rows | B rows][128 bytes]

    // Consecutive tiles (same rows of A, neighbouring rows of B) run on the same XCD and share its L2.
    const int tiles_n = (g.Nr + BN - 1) / BN, tiles_m = (g.Mr + BM - 1) / BM;
    const int total = tiles_m * tiles_n * g.splits, per_xcd = (total + kXcds - 1) / kXcds;
    const int unit = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if ((int)(blockIdx.x / kXcds) >= per_xcd || unit >= total) return;
    // (wave-uniform as it is, but the divisions run on the vector unit: descriptors and copies want scalar registers)
    const int tile = __builtin_amdgcn_readfirstlane(unit / g.splits), split = __builtin_amdgcn_readfirstlane(unit % g.splits);
    const int m0 = __builtin_amdgcn_readfirstlane(tile / tiles_n) * BM, n0 = __builtin_amdgcn_readfirstlane(tile % tiles_n) * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int col = lane & 31, h = lane >> 5;

    const __amdgpu_buffer_rsrc_t abuf = buffer_of(g.A + (size_t)m0 * g.lda, (long)min(BM, g.Mr - m0) * g.lda * 2);   // rows past the end: zeros
    const __amdgpu_buffer_rsrc_t bbuf = buffer_of(g.B + (size_t)n0 * g.ldb, TURNED ? 0 : (long)min(BN, g.Nr - n0) * g.ldb * 2);
    const int all_steps = g.Kd / kStepK, per_split = (all_steps + g.splits - 1) / g.splits;
    const int first = split * per_split, steps = min(all_steps, first + per_split) - first;   // >= 1: the launcher sees to it
    const int lrow = lane >> 3;
    const uint32_t lds0 = lds_offset(lds);
    // TURNED: a step's 64 rows of B by BN columns, as they lie, kPieces pieces a row; Nr columns are whole pieces, those past Nr aim nowhere
    constexpr int kPieces = BN / 8;
    const int trow = lane / kPieces, tcolumn = ((lane % kPieces) ^ turned_key(trow, kPieces)) * 8;
    const int toff = n0 + tcolumn < g.Nr ? (trow * g.ldb + tcolumn) * 2 : 0x40000000;
    auto copy_step = [&](int s, int stage) __attribute__((always_inline)) {
        const uint32_t base = lds0 + stage * kStageBytes;
        const int k0 = (first + s) * kStepK;
        const __amdgpu_buffer_rsrc_t tbuf = TURNED ? buffer_of(g.B + (size_t)k0 * g.ldb + n0, __builtin_amdgcn_readfirstlane(max(0, (min(kStepK, g.b_rows - k0) * g.ldb - n0) * 2))) : bbuf;
#pragma unroll
        for (int j = 0; j < kCopies; ++j) {
            const int row = 8 * (4 * j + wave);         // of [A rows | B rows]; BM is a multiple of 32, so the side is the same for all waves
            const int piece = ((lane & 7) ^ piece_key((row + lrow) & 15)) * 16;
            if (TURNED && 32 * j >= BM) copy16_to_lds(tbuf, toff, (row - BM) / 8 * (64 / kPieces) * g.ldb * 2, base + row * 128);
            else if (32 * j < BM) copy16_to_lds(abuf, lrow * g.lda * 2 + piece, row * g.lda * 2 + (first + s) * 128, base + row * 128);
            else copy16_to_lds(bbuf, lrow * g.ldb * 2 + piece, (row - BM) * g.ldb * 2 + (first + s) * 128, base + row * 128);
        }
    };

    float16_t acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // operand rows of this lane: 32 rows apart, so they share the key
    const int key = piece_key(col & 15);
    const int arow = (wm * 32 * WM + col) * 128, brow = (BM + wn * 32 * WN + col) * 128;
    int tlane[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j) tlane[j] = TURNED ? turned_offset<kPieces>(lane, (wn * WN + j) * 4) : 0;
    for (int s = 0; s < min(kNtStages - 1, steps); ++s) copy_step(s, s);
    for (int s = 0; s < steps; ++s) {
        // step s has landed, and everybody is done with step s - 1, whose stage the next copies go to
        if (s + kNtStages - 2 < steps) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kNtStages - 2) * kCopies) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (s + kNtStages - 1 < steps) copy_step(s + kNtStages - 1, (s + kNtStages - 1) % kNtStages);
        const unsigned char *base = lds + (s % kNtStages) * kStageBytes;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int chunk = ((kk * 2 + h) ^ key) * 16;
            half8_t af[WM], bf[WN];
#pragma unroll
            for (int i = 0; i < WM; ++i) af[i] = *reinterpret_cast<const half8_t *>(base + arow + i * 32 * 128 + chunk);
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                if constexpr (TURNED) bf[j] = read_turned<kPieces>(base + BM * 128 + tlane[j] + kk * (16 * kPieces * 16));
                else bf[j] = *reinterpret_cast<const half8_t *>(base + brow + j * 32 * 128 + chunk);
            }
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[i], bf[j], acc[i][j], 0, 0, 0);
        }
    }

    // accumulator register v of a lane: row 8 (v / 4) + 4 h + v % 4 of the 32x32 tile, column `col`
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            const int n = n0 + (wn * WN + j) * 32 + col;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + (wm * WM + i) * 32 + 8 * (v / 4) + 4 * h + (v % 4);
                if (m >= g.Mr || n >= g.Nr) continue;
                if (g.splits > 1) g.part[((size_t)split * g.Mr + m) * g.Nr + n] = acc[i][j][v];
                else store_result(g, m, n, acc[i][j][v]);
            }
        }
}

// loss = scale x (sum of the tiles' partial sums, in index order), by one block.
struct LossArgs { const float *part; int n; float scale; float *out; };
__device__ void sum_loss(const LossArgs &l)
{
    __shared__ double s[256];
    double a = 0.0;
    for (int i = threadIdx.x; i < l.n; i += 256) a += (double)l.part[i];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) *l.out = (float)(s[0] * (double)l.scale);
}

// What the last launch of a step does besides its split sums.
struct LastArgs {
    LossArgs loss;                                      // loss.part null: none
    float *At32, *Bt32;                                 // masters <- masters - lr gradient (Alg. 1, the update line); null: not this launch
    const float *gAt, *gBt;
    float lr;
    unsigned sum_blocks, a_blocks, b_blocks;            // blocks that add up splits - and move Bt32 as they go -, that move At32, and, without splits, Bt32
    size_t nA, nB;
};
__device__ __forceinline__ void descend(float *__restrict__ master, const float *__restrict__ grad, float lr, size_t i, size_t n)   // n a multiple of 4
{
    if (i >= n) return;
    const float4 v = *reinterpret_cast<const float4 *>(grad + i);
    float4 m = *reinterpret_cast<const float4 *>(master + i);
    m.x -= lr * v.x; m.y -= lr * v.y; m.z -= lr * v.z; m.w -= lr * v.w;
    *reinterpret_cast<float4 *>(master + i) = m;
}

// The store epilogue over the sum of the K splits' partial results, splits in index order; four results per thread (Nr is a
// multiple of 4).
__global__ __launch_bounds__(256) void fbq_sum_splits_kernel(GemmArgs g, LastArgs last)
{
    if (blockIdx.x >= last.sum_blocks) {                // block-uniform
        const unsigned b = blockIdx.x - last.sum_blocks;
        if (b < last.a_blocks) descend(last.At32, last.gAt, last.lr, ((size_t)b * 256 + threadIdx.x) * 4, last.nA);
        else if (b < last.a_blocks + last.b_blocks) descend(last.Bt32, last.gBt, last.lr, ((size_t)(b - last.a_blocks) * 256 + threadIdx.x) * 4, last.nB);
        else sum_loss(last.loss);
        return;
    }
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4, count = (size_t)g.Mr * g.Nr;
    if (i >= count) return;
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int s0 = 0; s0 < g.splits; s0 += 8) {          // eight splits per round trip to memory
        float4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const float4 *>(g.part + (size_t)min(s0 + k, g.splits - 1) * count + i);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (s0 + k < g.splits) { a.x += v[k].x; a.y += v[k].y; a.z += v[k].z; a.w += v[k].w; }
    }
    const int m = (int)(i / g.Nr), n = (int)(i % g.Nr);
    store_result(g, m, n, a.x);
    store_result(g, m, n + 1, a.y);
    store_result(g, m, n + 2, a.z);
    store_result(g, m, n + 3, a.w);
    if (last.Bt32) {                                    // (g.C32 is dL/dBt, laid out like the master; the thread has just written these four)
        const size_t at = (size_t)m * g.ldc32 + n;
        float4 b = *reinterpret_cast<const float4 *>(last.Bt32 + at);
        b.x -= last.lr * (g.alpha * a.x); b.y -= last.lr * (g.alpha * a.y); b.z -= last.lr * (g.alpha * a.z); b.w -= last.lr * (g.alpha * a.w);
        *reinterpret_cast<float4 *>(last.Bt32 + at) = b;
    }
}

// Tile shapes: 64 rows or columns where an operand has no more, and 64 of the other one, so that there are as many tiles, as few
// K splits and as little traffic of partial results as possible (4096 x 4096, r = 64, us with 64 x 64 and 128 x 64 tiles / 64 x 128
// and 128 x 128: B^T Delta 9.7 / 11.0, [Q; At] H 14.2 / 16.7, Delta V 9.7 / 11.6).  Half as many splits: 0.3 to 1 us slower.
struct TileShape { int wm, wn; };
static TileShape tile_for(int Mr, int Nr)
{
    if (Mr <= 64) return {1, 1};
    if (Mr <= 128) return {2, 1};
    if (Nr <= 64) return {1, 1};
    if (Nr <= 128) return {1, 2};
    return {2, 2};
}
static int tiles_of(int Mr, int Nr)
{
    const TileShape t = tile_for(Mr, Nr);
    return ceil_div(Mr, 64 * t.wm) * ceil_div(Nr, 64 * t.wn);
}

// Blocks that split K for one tile: enough to give every CU a block when the tiles alone do not,
// at least 4 steps each, and none left without a step.
static int splits_for(int Mr, int Nr, int Kd)
{
    const int tiles = tiles_of(Mr, Nr), steps = Kd / kStepK;
    const int want = std::min(256 / std::max(tiles, 1), steps / 4);
    if (want < 2) return 1;
    return ceil_div(steps, ceil_div(steps, want));
}

static size_t split_scratch_bytes(int Mr, int Nr, int Kd)
{
    const int sp = splits_for(Mr, Nr, Kd);
    return sp > 1 ? (size_t)sp * Mr * Nr * 4 : 0;
}

template <int WM, int WN>
static void launch_gemm_tile(const GemmArgs &g, dim3 grid, hipStream_t stream)
{
    if (g.b_rows) hipLaunchKernelGGL((fbq_gemm_nt_kernel<WM, WN, true>), grid, dim3(256), 0, stream, g);
    else hipLaunchKernelGGL((fbq_gemm_nt_kernel<WM, WN, false>), grid, dim3(256), 0, stream, g);
}

// last: the launch that ends a step, or null
static hipError_t launch_gemm(GemmArgs g, float *split_scratch, hipStream_t stream, const LastArgs *last = nullptr)
{
    g.splits = splits_for(g.Mr, g.Nr, g.Kd);
    g.part = split_scratch;
    const TileShape t = tile_for(g.Mr, g.Nr);
    const int units = tiles_of(g.Mr, g.Nr) * g.splits;
    const dim3 grid(ceil_div(units, kXcds) * kXcds);
    if (t.wm == 1 && t.wn == 1) launch_gemm_tile<1, 1>(g, grid, stream);
    else if (t.wm == 1) launch_gemm_tile<1, 2>(g, grid, stream);
    else if (t.wn == 1) launch_gemm_tile<2, 1>(g, grid, stream);
    else launch_gemm_tile<2, 2>(g, grid, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const auto blocks_of = [](size_t n) { return (unsigned)((n / 4 + 255) / 256); };
    LastArgs l{};
    if (last) l = *last;
    l.sum_blocks = g.splits > 1 ? blocks_of((size_t)g.Mr * g.Nr) : 0u;   // Nr is a multiple of 8 (r or K)
    if (last) {
        l.a_blocks = blocks_of(l.nA);
        l.b_blocks = g.splits > 1 ? 0u : blocks_of(l.nB);
    }
    const unsigned blocks = l.sum_blocks + l.a_blocks + l.b_blocks + (l.loss.part ? 1u : 0u);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(fbq_sum_splits_kernel, dim3(blocks), dim3(256), 0, stream, g, l);
    return hipGetLastError();
}

static GemmArgs gemm_args(const uint16_t *A, int Mr, int lda, const uint16_t *B, int Nr, int ldb, int Kd)
{
    GemmArgs g{};
    g.A = A; g.B = B; g.Mr = Mr; g.Nr = Nr; g.Kd = Kd; g.lda = lda; g.ldb = ldb;
    g.c32_rows = Mr; g.c16_row0 = 0; g.splits = 1;
    return g;
}

// ------------------------------------------------------------------ symmetric products

// G = A^T A of one operand A [Kd][R]: the lower triangle of tiles of 192 x 192 is computed, half the work of the square.
//   DOT false: C = fp16(beta G), both triangles (H = X^T X with A = X)
//   DOT true:  dot[unit] = the tile's share of sum G o H (the loss with A = Delta_F: tr(Delta H Delta^T) = sum
//              (Delta^T Delta) o H; a tile below the diagonal stands for its mirror image as well and meets H + H^T)
// Four waves of 96 x 96 (3 x 3 of v_mfma_f32_32x32x16_f16), one per SIMD; k advances in steps of 64, three steps in LDS
// (48 KiB each), copied there without passing registers and waited for by count as in the prefill kernel.  The copies of
// a step go out one by one between groups of three matrix instructions.  192 rows: 4096 rows make 253 such tiles, one for
// nearly every CU, where 256-row tiles would leave half the chip idle (136 tiles of the triangle) and 128-row tiles need 2.1
// rounds.  Few tiles: the contraction is split over blocks - for free where only the dot product is wanted (it is linear in
// G), through fp32 partial tiles and a summing launch otherwise.
// Bound: matrix cores; 4096 x 4096 in us, the whole square in 128-row tiles staged through registers / this: H over 2048 tokens
// 103 / 41, the loss over 4096 rows 196 / 74 (34 and 69 GFLOP of the triangle: 0.84 and 0.93 PFLOP/s).
// H used to be taken from a transposed copy of X, 7 us more at this size (46.4 / 40.6 for all of H, 128 features over some tokens 18.0 / 15.6), and the loss from a second, transposed Delta_F.  The
// turned reads are twice as many instructions for the same bytes and cost the loss 4 us (70.6 / 74.6 on one box), of the 13 that writing Delta_F twice cost the quantizer.
// Other sizes leave the last round emptier and keep the gain; H with that transpose, the square / this: 3072 features, 4096 tokens
// 152 / 66 (136 tiles); 5120, 2048 185 / 81 (378); 8192, 512 168 / 80 (946); 11008, 4096 1362 / 493 (1711).
constexpr int kSyTile = 192, kSyWave = 96, kSyStages = 3;
constexpr int kSySide = kSyTile * 128, kSyStep = 2 * kSySide;       // LDS bytes of one operand's rows and of a step
constexpr int kSyBand = 6;                                          // tiles are numbered in bands of six tile rows

struct SyrkArgs {
    const uint16_t *A;                   // [Kd][R], R a multiple of 8
    int R, Kd;
    int side, tiles, splits;             // tiles per side, tiles of the lower triangle, blocks that share a tile's contraction
    uint16_t *C; int ldc; float beta;
    float *part;                         // splits > 1 and not DOT: [splits][tiles][192][192]
    const uint16_t *H; float *dot;       // DOT: H [R][R]
};

// Tile t of the lower triangle: bands of six tile rows, column by column within a band, so that the tiles an XCD works on at
// the same time (consecutive ones) lie in a block of about six by five and share their operands' rows in its L2.
__device__ __forceinline__ void syrk_tile(int t, int side, int *ti, int *tj)
{
    int b = 0, h;
    for (;; ++b) {
        h = min(kSyBand, side - b * kSyBand);
        const int count = b * kSyBand * h + h * (h + 1) / 2;
        if (t < count) break;
        t -= count;
    }
    if (t < b * kSyBand * h) {
        *tj = t / h;
        *ti = b * kSyBand + t % h;
        return;
    }
    t -= b * kSyBand * h;
    int c = 0;
    for (; t >= h - c; ++c) t -= h - c;
    *tj = b * kSyBand + c;
    *ti = *tj + t;
}

template <bool DOT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void fbq_syrk_kernel(const SyrkArgs g)
{
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kSyStages * kSyStep];
    const int units = g.tiles * g.splits, per_xcd = (units + kXcds - 1) / kXcds;
    const int unit = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;      // consecutive units on the same XCD
    if ((int)(blockIdx.x / kXcds) >= per_xcd || unit >= units) return;
    // (wave-uniform as it is, but the divisions run on the vector unit: descriptors and copies want scalar registers)
    const int split = __builtin_amdgcn_readfirstlane(unit / g.tiles), tile = __builtin_amdgcn_readfirstlane(unit % g.tiles);
    int ti, tj;
    syrk_tile(tile, g.side, &ti, &tj);
    ti = __builtin_amdgcn_readfirstlane(ti);
    tj = __builtin_amdgcn_readfirstlane(tj);
    const int m0 = ti * kSyTile, n0 = tj * kSyTile;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int col = lane & 31, h = lane >> 5;

    // Waves 0 and 1 copy the tile's row side, 64 rows of A by 192 columns a step, 32 rows each, waves 2 and 3 its column side.  A copy moves 64
    // pieces of 24 a row, as they lie in LDS: three copies are eight rows.  A descriptor ends with the step's last row (rows past A's: zeros);
    // columns past A's aim nowhere.
    const int side0 = wm ? n0 : m0;
    int loff[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const int row = (b * 64 + lane) / 24, column = (((b * 64 + lane) % 24) ^ turned_key(row, 24)) * 8;
        loff[b] = side0 + column < g.R ? (row * g.R + column) * 2 : 0x40000000;
    }
    const uint32_t lds0 = lds_offset(lds);
    const int all_steps = (g.Kd + 63) / 64, per_split = (all_steps + g.splits - 1) / g.splits;
    const int first = split * per_split, steps = max(0, min(all_steps, first + per_split) - first);
    constexpr int kCopies = kSyWave / 8;                // per wave and step
    auto rows_of = [&](int st) __attribute__((always_inline)) {               // (past the end: the last step again, never used)
        const int k0 = __builtin_amdgcn_readfirstlane(min(first + st, all_steps - 1) * 64);
        return buffer_of(g.A + (size_t)k0 * g.R + side0, __builtin_amdgcn_readfirstlane((min(64, g.Kd - k0) * g.R - side0) * 2));
    };
    auto issue = [&](const __amdgpu_buffer_rsrc_t &buf, int stage, int j) __attribute__((always_inline)) {
        copy16_to_lds(buf, loff[j % 3], (wn * 32 + j / 3 * 8) * g.R * 2, lds0 + stage * kSyStep + wm * kSySide + (wn * kCopies + j) * 1024);
    };
    auto wait_and_meet = [&](auto N) __attribute__((always_inline)) {
        constexpr int n = decltype(N)::value;
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(n) : "memory");
    };

    float16_t acc[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // fragment of K step i: rows 16 i + 8 h and up of A, 32 columns
    int a_lane[3], b_lane[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        a_lane[t] = turned_offset<24>(lane, wm * (kSyWave / 8) + 4 * t);
        b_lane[t] = kSySide + turned_offset<24>(lane, wn * (kSyWave / 8) + 4 * t);
    }
    auto frag = [&](int stage, const int (&lane_off)[3], int i, int t) __attribute__((always_inline)) {
        return read_turned<24>(lds + stage * kSyStep + lane_off[t] + i * (16 * 24 * 16));
    };
    half8_t af[2][3], bf[2][3];
    auto do_step = [&](int st, int s0, int s1, int s2) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int cur = i & 1, nxt = cur ^ 1;
            const __amdgpu_buffer_rsrc_t buf = rows_of(i == 3 ? st + 3 : st + 2);
            __builtin_amdgcn_sched_barrier(0);
            // the next step has landed, and everybody has read all of this one: its stage may be filled again
            if (i == 3) wait_and_meet(std::integral_constant<int, kCopies>{});
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                if (i == 3) issue(buf, s0, t);
                else issue(buf, s2, 3 + 3 * i + t);
                af[nxt][t] = i < 3 ? frag(s0, a_lane, i + 1, t) : frag(s1, a_lane, 0, t);
                bf[nxt][t] = i < 3 ? frag(s0, b_lane, i + 1, t) : frag(s1, b_lane, 0, t);
#pragma unroll
                for (int u = 0; u < 3; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[cur][t], bf[cur][u], acc[t][u], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < kCopies; ++j) issue(rows_of(s), s, j);
#pragma unroll
    for (int j = 0; j < 3; ++j) issue(rows_of(2), 2, j);
    wait_and_meet(std::integral_constant<int, kCopies + 3>{});
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        af[0][t] = frag(0, a_lane, 0, t);
        bf[0][t] = frag(0, b_lane, 0, t);
    }
    int s0 = 0;
    for (int st = 0; st < steps; ++st) {
        const int s1 = s0 == 2 ? 0 : s0 + 1, s2 = s0 == 0 ? 2 : s0 - 1;
        do_step(st, s0, s1, s2);
        s0 = s1;
    }
    wait_and_meet(std::integral_constant<int, 0>{});    // the copies issued past the end have landed too, and everybody is done: LDS is free

    // accumulator register v of a lane: row 8 (v / 4) + 4 h + v % 4 of the 32x32 tile, column `col`
    const int mw = m0 + wm * kSyWave, nw = n0 + wn * kSyWave;       // the wave's rows and columns
    constexpr int kPieces = kSyWave * kSyWave / 8 / 64;             // 16-byte pieces of a 96 x 96 fp16 tile per lane
    if constexpr (DOT) {
        // the two tiles of H that the wave's 96 x 96 meet, by way of LDS: rows mw.., columns nw.. and the mirror image
        constexpr int kHTile = kSyWave * kSyWave * 2;
        auto copy_h = [&](int r0, int c0, int o) __attribute__((always_inline)) {
            const __amdgpu_buffer_rsrc_t hbuf = buffer_of(g.H + (size_t)r0 * g.R, __builtin_amdgcn_readfirstlane(max(0, min(kSyWave, g.R - r0)) * g.R * 2));   // (the clamp runs on the vector unit)
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                const int piece = i * 64 + lane, row = piece / 12, p = piece % 12;   // 192 bytes a row
                copy16_to_lds(hbuf, c0 + p * 8 < g.R ? row * g.R * 2 + (c0 + p * 8) * 2 : 0x7FFFFFF0, 0, lds0 + (wave * 2 + o) * kHTile + i * 1024);
            }
        };
        copy_h(mw, nw, 0);
        copy_h(nw, mw, 1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // (each wave reads what itself copied)
        const uint16_t *hd = reinterpret_cast<const uint16_t *>(lds + wave * 2 * kHTile), *hm = hd + kSyWave * kSyWave;
        const float mirror = ti == tj ? 0.0f : 1.0f;                // a diagonal tile is its own mirror image
        float dot = 0.0f;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                float part = 0.0f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = t * 32 + 8 * (v / 4) + 4 * h + (v % 4), n = u * 32 + col;
                    const float direct = (float)__builtin_bit_cast(half_t, hd[m * kSyWave + n]), turned = (float)__builtin_bit_cast(half_t, hm[n * kSyWave + m]);
                    part = fmaf(acc[t][u][v], fmaf(mirror, turned, direct), part);
                }
                dot += part;
            }
        // fixed order: lanes by xor-shuffles, then the four waves in turn
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off, 64);
        __syncthreads();
        float *wsum = reinterpret_cast<float *>(lds);
        if (lane == 0) wsum[wave] = dot;
        __syncthreads();
        if (tid == 0) g.dot[unit] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
        return;
    }
    if (g.splits > 1) {
        float *part = g.part + ((size_t)split * g.tiles + tile) * (kSyTile * kSyTile) + (wm * kSyWave) * kSyTile + wn * kSyWave;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int u = 0; u < 3; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v) part[(t * 32 + 8 * (v / 4) + 4 * h + (v % 4)) * kSyTile + u * 32 + col] = acc[t][u][v];
        return;
    }
    // (scaled here and not in the conversions: fused into some of them, the two triangles would not round alike)
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float scaled = g.beta * acc[t][u][v];
                asm volatile("" : "+v"(scaled));
                acc[t][u][v] = scaled;
            }
    // fp16 tiles turned round in the wave's own piece of LDS (rows of 96 fp16, 208 bytes apart) and stored as 16-byte pieces
    constexpr int kOutRow = kSyWave * 2 + 16;
    static_assert(4 * kSyWave * kOutRow <= (int)sizeof(lds), "the waves' tiles must fit the stages");
    unsigned char *const out = lds + wave * (kSyWave * kOutRow);
    auto store = [&](int r0, int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int piece = i * 64 + lane, row = piece / 12, p = piece % 12;
            const uint4 v = *reinterpret_cast<const uint4 *>(out + row * kOutRow + p * 16);
            if (r0 + row < g.R && c0 + p * 8 < g.R) *reinterpret_cast<uint4 *>(g.C + (size_t)(r0 + row) * g.ldc + c0 + p * 8) = v;
        }
    };
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                *reinterpret_cast<half_t *>(out + (t * 32 + 8 * (v / 4) + 4 * h + (v % 4)) * kOutRow + (u * 32 + col) * 2) = (half_t)acc[t][u][v];
    store(mw, nw);                                      // (the wave reads what itself wrote: LDS keeps a wave's accesses in order)
    if (ti == tj) return;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                half4_t v4;
#pragma unroll
                for (int e = 0; e < 4; ++e) v4[e] = (half_t)acc[t][u][4 * q + e];
                *reinterpret_cast<half4_t *>(out + (u * 32 + col) * kOutRow + (t * 32 + 8 * q + 4 * h) * 2) = v4;
            }
    store(nw, mw);
}

// C = fp16(beta x sum of the splits' partial tiles), splits in index order, both triangles.  Block: a 32 x 32 piece of a tile,
// four values per thread; R is a multiple of 128, so a piece lies in the matrix whole or not at all.
// Bound: the round trips over the splits, eight at a time.  (64 x 64 pieces, sixteen rows of a thread and every split one after
// the other: the whole H of 128 features over 4096 tokens 73 us, of 1024 features 57; 17 and 28 with these pieces.)
constexpr int kSyPiece = 32, kSyPieces = kSyTile / kSyPiece;       // pieces along a side of a tile
__global__ __launch_bounds__(256) void fbq_syrk_sum_kernel(const SyrkArgs g)
{
    __shared__ uint32_t turn[kSyPiece][kSyPiece / 2 + 1];
    int ti, tj;
    syrk_tile(blockIdx.x, g.side, &ti, &tj);
    const int pr = (blockIdx.y / kSyPieces) * kSyPiece, pc = (blockIdx.y % kSyPieces) * kSyPiece;
    const int m0 = ti * kSyTile + pr, n0 = tj * kSyTile + pc;
    if (m0 >= g.R || n0 >= g.R) return;                 // block-uniform
    const int r = threadIdx.x >> 3, c = (threadIdx.x & 7) * 4;
    const float *part = g.part + (size_t)blockIdx.x * (kSyTile * kSyTile) + (pr + r) * kSyTile + pc + c;
    const size_t stride = (size_t)g.tiles * (kSyTile * kSyTile);
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int s0 = 0; s0 < g.splits; s0 += 8) {          // eight splits per round trip to memory
        float4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const float4 *>(part + (size_t)min(s0 + k, g.splits - 1) * stride);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (s0 + k < g.splits) { a.x += v[k].x; a.y += v[k].y; a.z += v[k].z; a.w += v[k].w; }
    }
    // (scaled here and not in the conversions, as in the kernel above: a diagonal tile's two halves have to round alike)
    float scaled[4] = {g.beta * a.x, g.beta * a.y, g.beta * a.z, g.beta * a.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(scaled[e]));
    const half4_t o = half4_t{(half_t)scaled[0], (half_t)scaled[1], (half_t)scaled[2], (half_t)scaled[3]};
    *reinterpret_cast<half4_t *>(g.C + (size_t)(m0 + r) * g.ldc + n0 + c) = o;
    if (ti == tj) return;                               // block-uniform
#pragma unroll
    for (int e = 0; e < 4; ++e) reinterpret_cast<half_t *>(turn[c + e])[r] = o[e];
    __syncthreads();
    const uint2 w = make_uint2(turn[r][c / 2], turn[r][c / 2 + 1]);
    *reinterpret_cast<uint2 *>(g.C + (size_t)(n0 + r) * g.ldc + m0 + c) = w;
}

// Blocks that share a tile's contraction: what makes the estimate in us smallest, 256 CUs assumed: rounds x (steps + 7 of
// start and end), a step taking 0.55 and up to 0.3 more as the round fills the CUs; where the partial tiles have to be written
// and summed, 0.3 per partial tile of a sum and 0.03 of traffic per tile in flight as well.  Fitted to H at 128 to 5120
// features and 128 to 65536 tokens with 1 to 256 splits: where the choice itself was measured it is within 7 % of the best one.
// Examples, us without a split / as chosen / with twice the splits: 1024 features, 4096 tokens 54 / 28 (5) / 28; 2048 features,
// 2048 tokens 39 / 32 (2) / 40; 128 features, 4096 tokens 47 / 17 (8) / 18; 2944 features, 4096 tokens 67 (1) / 78.
struct SyrkShape { int side, tiles, splits; };
static SyrkShape syrk_shape(int R, int Kd, bool dot)
{
    const int side = ceil_div(R, kSyTile), tiles = side * (side + 1) / 2, steps = ceil_div(Kd, 64);
    SyrkShape best{side, tiles, 1};
    double best_cost = 1e300;
    for (int s = 1; s <= 64 && s <= steps && (s == 1 || tiles * s <= 768); ++s) {
        const double rounds = ceil_div(tiles * s, 256), filled = tiles * s / (256.0 * rounds);
        double cost = rounds * (ceil_div(steps, s) * (0.55 + 0.3 * filled) + 7.0);
        if (s > 1 && !dot) cost += 0.5 + 0.3 * s + 0.03 * tiles * s;
        if (cost < best_cost * 0.98) { best_cost = cost; best.splits = s; }
    }
    return best;
}
static size_t syrk_units(const SyrkShape &s) { return (size_t)s.tiles * s.splits; }
static size_t syrk_scratch_bytes(int R, int Kd)
{
    const SyrkShape s = syrk_shape(R, Kd, false);
    return s.splits > 1 ? syrk_units(s) * kSyTile * kSyTile * 4 : 0;
}

template <bool DOT>
static hipError_t launch_syrk(SyrkArgs g, hipStream_t stream)
{
    const SyrkShape s = syrk_shape(g.R, g.Kd, DOT);
    g.side = s.side; g.tiles = s.tiles; g.splits = s.splits;
    const int units = s.tiles * s.splits;
    hipLaunchKernelGGL(fbq_syrk_kernel<DOT>, dim3(ceil_div(units, kXcds) * kXcds), dim3(256), 0, stream, g);
    if (!DOT && g.splits > 1) hipLaunchKernelGGL(fbq_syrk_sum_kernel, dim3(g.tiles, kSyPieces * kSyPieces), dim3(256), 0, stream, g);
    return hipGetLastError();
}

// fp16 views of the fp32 masters: At16 [r][K] and Bt16 [N][r] (the inference layouts, outputs of the
// step; At16 once more as the lower half of the stacked operand [Q; At]) and Bc [r][Np] = B with
// rows contiguous along n, columns N..Np-1 zero.
__global__ __launch_bounds__(256) void fbq_cast_masters_kernel(const float *__restrict__ At32, const float *__restrict__ Bt32,
                                                               uint16_t *__restrict__ At16, uint16_t *__restrict__ Bt16,
                                                               uint16_t *__restrict__ At16_stacked, uint16_t *__restrict__ Bc,
                                                               int N, int K, int r, int Np)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t nA = (size_t)r * K, nB = (size_t)N * r, nC = (size_t)r * Np;
    if (i < nA) {
        const uint16_t v = __builtin_bit_cast(uint16_t, (half_t)At32[i]);
        At16[i] = v;
        At16_stacked[i] = v;
    } else if (i < nA + nB) {
        Bt16[i - nA] = __builtin_bit_cast(uint16_t, (half_t)Bt32[i - nA]);
    } else if (i < nA + nB + nC) {
        const size_t e = i - nA - nB;
        const int j = (int)(e / Np), n = (int)(e % Np);
        Bc[e] = n < N ? __builtin_bit_cast(uint16_t, (half_t)Bt32[(size_t)n * r + j]) : (uint16_t)0;
    }
}

static size_t pad256(size_t b) { return (b + 255) & ~(size_t)255; }
static int pad64(int v) { return (v + 63) & ~63; }

constexpr float kVGain = 64.0f;      // V^T = At H is stored as fp16(64 h_scale At H)

struct TrainLayout {
    size_t Bc, D16, S16, Vt16, dot, split, total;
};

static TrainLayout train_layout(int N, int K, int r)
{
    const int Np = pad64(N);
    TrainLayout l{};
    size_t o = 0;
    l.Bc = o;   o += pad256((size_t)r * Np * 2);
    l.D16 = o;  o += pad256((size_t)N * K * 2);
    l.S16 = o;  o += pad256((size_t)2 * r * K * 2);          // stacked operand [Q; At]
    l.Vt16 = o; o += pad256((size_t)r * K * 2);
    l.dot = o;  o += pad256(syrk_units(syrk_shape(K, Np, true)) * 4);
    l.split = o;
    o += pad256(std::max(std::max(split_scratch_bytes(r, K, Np), split_scratch_bytes(2 * r, K, K)), split_scratch_bytes(N, r, K)));
    o += pad256((size_t)K * Np * 2);                         // not used: what is asked for, and what is refused, stays as it was when Delta_F was kept in both orientations
    l.total = o;
    return l;
}

size_t train_workspace_bytes(int N, int K, int r, int T)
{
    const int Tp = pad64(T);
    return std::max(train_layout(N, K, r).total, pad256((size_t)K * Tp * 2) + pad256(syrk_scratch_bytes(K, Tp)));
}

hipError_t launch_gram(int K, int T, const uint16_t *X, float h_scale, uint16_t *H16, void *workspace, hipStream_t stream)
{
    // (a result over the activations themselves: from a copy of them)
    const size_t x_bytes = (size_t)T * K * 2;
    if ((uintptr_t)X < (uintptr_t)H16 + (size_t)K * K * 2 && (uintptr_t)H16 < (uintptr_t)X + x_bytes) {
        const hipError_t e = hipMemcpyAsync(workspace, X, x_bytes, hipMemcpyDeviceToDevice, stream);
        if (e != hipSuccess) return e;
        X = (const uint16_t *)workspace;
    }
    SyrkArgs g{};
    g.A = X; g.R = K; g.Kd = T;
    g.C = H16; g.ldc = K; g.beta = h_scale; g.part = (float *)((unsigned char *)workspace + pad256((size_t)K * pad64(T) * 2));
    return launch_syrk<false>(g, stream);
}

hipError_t launch_train_step(const TrainArgs &a, hipStream_t stream)
{
    const int N = a.d.N, K = a.d.K, r = a.d.r, Np = pad64(N);
    const TrainLayout l = train_layout(N, K, r);
    unsigned char *ws = (unsigned char *)a.workspace;
    uint16_t *Bc = (uint16_t *)(ws + l.Bc);
    uint16_t *D16 = (uint16_t *)(ws + l.D16);
    uint16_t *S16 = (uint16_t *)(ws + l.S16), *Vt16 = (uint16_t *)(ws + l.Vt16);
    float *dot = (float *)(ws + l.dot), *scratch = (float *)(ws + l.split);

    // fp16 views of the masters: what the forward pass of Alg. 1 computes with
    const size_t casts = (size_t)r * K + (size_t)N * r + (size_t)r * Np;
    hipLaunchKernelGGL(fbq_cast_masters_kernel, dim3((unsigned)((casts + 255) / 256)), dim3(256), 0, stream, a.At32, a.Bt32, a.At16,
                       a.Bt16, S16 + (size_t)r * K, Bc, N, K, r, Np);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // Q(W - Sigma16), written in the inference layout, and Delta_F = (W - Sigma16) - Q(W - Sigma16), times 256
    e = launch_quantize(a.d, a.W, a.At16, a.Bt16, a.qw, a.scales, a.zeros, stream, D16, kDeltaGain);
    if (e != hipSuccess) return e;
    // Q = Bt^T Delta_F (times 256), the upper half of the stacked operand
    {
        GemmArgs g = gemm_args(Bc, r, Np, D16, K, K, Np);
        g.b_rows = N;
        g.C16 = S16; g.ldc16 = K; g.beta = 1.0f;
        if ((e = launch_gemm(g, scratch, stream)) != hipSuccess) return e;
    }
    // [Q; At] H (H symmetric): rows of Q give dL/dAt = -2 Q H, rows of At give V^T = At H
    {
        GemmArgs g = gemm_args(S16, 2 * r, K, a.H16, K, K, K);
        g.C32 = a.gAt; g.ldc32 = K; g.alpha = -2.0f / (kDeltaGain * a.h_scale); g.c32_rows = r;
        g.C16 = Vt16; g.ldc16 = K; g.beta = kVGain; g.c16_row0 = r;
        if ((e = launch_gemm(g, scratch, stream)) != hipSuccess) return e;
    }
    // L = sum (Delta_F^T Delta_F) o H: the only contraction of this size, and only on request
    LastArgs last{};
    if (a.loss) {
        SyrkArgs g{};
        g.A = D16; g.R = K; g.Kd = N;
        g.H = a.H16; g.dot = dot;
        if ((e = launch_syrk<true>(g, stream)) != hipSuccess) return e;
        last.loss = {dot, (int)syrk_units(syrk_shape(K, Np, true)), 1.0f / (kDeltaGain * kDeltaGain * a.h_scale), a.loss};
    }
    // dL/dBt = -2 Delta_F H At^T = -2 Delta_F V; its summing launch moves the masters and adds up the loss as well
    GemmArgs g = gemm_args(D16, N, K, Vt16, r, K, K);
    g.C32 = a.gBt; g.ldc32 = r; g.alpha = -2.0f / (kDeltaGain * kVGain * a.h_scale);
    last.At32 = a.At32; last.Bt32 = a.Bt32; last.gAt = a.gAt; last.gBt = a.gBt; last.lr = a.lr;
    last.nA = (size_t)r * K; last.nB = (size_t)N * r;
    return launch_gemm(g, scratch, stream, &last);
}

}  // namespace fbq
