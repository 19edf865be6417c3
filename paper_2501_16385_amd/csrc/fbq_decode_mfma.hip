// Decode path for a few tokens (3 <= M <= 16): the fused kernel of Sec. 4.3 with the packed codes
// streamed exactly once, the tokens riding along as the 16 rows of a matrix-core tile.
//
//   y[M,N] = x[M,K] . Wq[N,K]^T + t[M,r] . B[r,N],   t = x . A
//
// One launch.  The first blocks of a grid row do the layer's down-projection and hand t over inside
// the launch (every partial sum travels as one 8-byte word {value, launch tag}, written and read at
// device scope: no flag, no fence, nothing to reset); all others stream weights from the start and
// ask for t only when their main part is done.  (The paper has a second launch there; on this GPU
// a launch boundary costs 4-5 us, a third of this kernel.)
//
// v_mfma_f32_16x16x32_f16 multiplies a 16 (token) x 32 (k) activation fragment with a 32 (k) x 16
// (output row) weight fragment.  Lane (c = lane % 16, q = lane / 16) supplies 8 values of k for
// token c in the first operand and for output row c in the second, and the instruction only needs
// both operands to agree on which k that is.
//
// Weights.  For one quantization group (128 codes) of 16 consecutive output rows, lane (c, q) needs
// the 32 codes k = 32 q .. 32 q + 31 of row c: one 16-byte (INT4) or 12-byte (INT3) load straight
// from the packed row into registers, no LDS memory in between (in most instances a neighbouring
// lane does the load, so that the four lanes of a load quad read one row, and the words change lanes
// afterwards).  A wave owns four consecutive groups, so the 16 row segments it reads are 256 (192)
// contiguous bytes each.  Masking a packed word with
// 0x000F000F and OR-ing 0x64006400 leaves two codes as the fp16 pair (1024 + q, 1024 + q'); fields
// that sit 4 (3, 6) bits higher come out as 1024 + 16 q (8 q, 64 q).  These go into the matrix
// instruction as they are: one v_and_or_b32 per two codes is all the de-quantization the inner
// loop does.
//
// Activations.  For every group, lane (c, q) reads the 32 activations k = 32 q .. 32 q + 31 of token c
// (four 16-byte loads, while the weights are under way) and re-orders them in registers into the four
// operands that meet its weight operands - divided by 16 (8, 64) where the weight field is scaled.
// A wave keeps the operands of its four groups in registers and walks over the block's row tiles
// with them, so a block reads the activations once, whatever the number of rows it owns.  Per group
// and token, X = sum x and XS = 1024 sum x' (x' the scaled activations) come from the matrix core as
// well: the operands against a column of ones, and against the column of field gains.
//
// One group of one row tile then is  D' = sum x' (1024 + m q) = XS + sum x q  (four matrix
// instructions, fp32, every product exact), and the lane that holds output row n adds
// s (D' - XS - z X) to its accumulator: the same factorisation as in the one-token kernel.
//
// A block's eight waves split K.  The up-projection enters the same accumulators as r more values of
// k (t split into two fp16 halves: t_hi + t_lo carries 22 bits of the fp32 sum), 32 taps a wave for all tiles of
// the block; then the waves' partial tiles meet in LDS and y is stored once.  Layers that read the same activations (q/k/v, gate/up) share the launch.
#include <type_traits>

#include "fbq_few_burst.h"

namespace fbq {

constexpr int kMaxTiles = 4;         // 16-row tiles per block (more would not fit the register file next to the activations)

struct SmallParams {
    const uint32_t *qw;
    const uint16_t *scales;
    const uint16_t *zeros;
    const uint16_t *At;    // [r][K]
    const uint16_t *Bt;    // [N][r]
    const uint16_t *x;     // [M][K]
    uint16_t *y;           // [M][N]
    uint64_t *tpart;       // workspace: [slices][16][r] words {fp32 partial sum of t = x.A over one K slice, launch tag}
    uint64_t *tsum;        // workspace: [16][r] words {t, launch tag}: the slices added up
    int M, N, K, r;
    int row_words, G;
    int slices, kslice;    // down-projection: number of K slices and their length (a multiple of 512)
    int down_blocks;       // blocks at the start of this layer's grid row that do its down-projection, slice by slice ...
    int sum_blocks;        // ... and the blocks after them that add the slices up (16 columns each)
    int tiles_per_block;   // 16-row tiles a consumer block owns
    int spin_limit;        // polls for t before a wave computes it itself; negative: at once (test hook)
};

// Layers that share their activations (q/k/v, gate/up) share the launch.  In the grid y is the layer
// and x the block of that layer; the layer's parameters are found from the block index alone, so
// they are fetched in one go with the rest of the kernel arguments (a second, dependent round trip
// to them costs more than half a microsecond).  Surplus blocks of rows with fewer blocks than the
// widest leave at once.
// The instances that write averages with the results have what to average with behind a layer's other parameters.
struct MixSmallParams : SmallParams {
    const uint16_t *mix_with;   // [M][N]
    uint16_t *mix_out;          // null: none
};
template <bool MIX>
struct SmallGroup {
    int n_layers;
    std::conditional_t<MIX, MixSmallParams, SmallParams> layer[kMaxSmallGroup];
};

// ------------------------------------------------------------------ fused kernel

// BITS, T, BRANCH, TAIL, MIX: see few_burst_block.
template <int BITS, int T, bool BRANCH, bool TAIL, bool MIX>
__global__ __launch_bounds__(64 * kMainWaves) void fbq_small_m_kernel(const SmallGroup<MIX> g)
{
    __shared__ float4_t red[kMainWaves][T][64];
    __shared__ uint4_t xslab[kMainWaves][kTokens * 17];
    float4_t (*red_prep)[64] = reinterpret_cast<float4_t (*)[64]>(&red[0][0][0]);   // [8][64], what a down-projection block needs

    const auto p = g.layer[blockIdx.y];
    // (all of them before the first branch: left alone, the compiler fetches only what the branch needs first)
    asm volatile("" :: "s"(p.qw), "s"(p.scales), "s"(p.zeros), "s"(p.x), "s"(p.y), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.row_words), "s"(p.G), "s"(p.tiles_per_block));
    if (BRANCH) asm volatile("" :: "s"(p.Bt), "s"(p.At), "s"(p.tpart), "s"(p.tsum), "s"(p.r), "s"(p.slices), "s"(p.kslice), "s"(p.down_blocks), "s"(p.sum_blocks), "s"(p.spin_limit));
    const uint32_t tag = BRANCH ? small_m_launch_tag() : 0u;

    // The first blocks of a grid row do the layer's down-projection.  They come first in dispatch
    // order, so whoever waits for their words waits for blocks that are already running.
    if (BRANCH && (int)blockIdx.x < p.down_blocks + p.sum_blocks) {
        if ((int)blockIdx.x < p.down_blocks) down_proj_block(p, blockIdx.x, tag, red_prep);
        else sum_slices_block(p, blockIdx.x - p.down_blocks, tag);
        return;
    }
    const int block = blockIdx.x - (BRANCH ? p.down_blocks + p.sum_blocks : 0);
    if (block * p.tiles_per_block >= (p.N + 15) / 16) return;   // a narrower layer of the group
    few_burst_block<BITS, T, BRANCH, TAIL, MIX>(p, block * p.tiles_per_block, tag, red, xslab);
}

template <int BITS, int T, bool BRANCH, bool TAIL>
static void launch_instance(const SmallGroup<true> &g, bool mix, dim3 grid, hipStream_t stream)
{
    if constexpr (!TAIL) {
        if (mix) {
            hipLaunchKernelGGL((fbq_small_m_kernel<BITS, T, BRANCH, TAIL, true>), grid, dim3(64 * kMainWaves), 0, stream, g);
            return;
        }
    }
    SmallGroup<false> plain;
    plain.n_layers = g.n_layers;
    std::copy(g.layer, g.layer + kMaxSmallGroup, plain.layer);
    hipLaunchKernelGGL((fbq_small_m_kernel<BITS, T, BRANCH, TAIL, false>), grid, dim3(64 * kMainWaves), 0, stream, plain);
}

template <int BITS, int T, bool TAIL>
static hipError_t launch_tiles(const SmallGroup<true> &g, bool branch, bool mix, dim3 grid, hipStream_t stream)
{
    // (the INT3 three- and four-tile instances without the branch come out of the compiler with spills of
    // 160 bytes and more; the ones with the branch spill nothing or 36 bytes, and with r = 0 they do the same work)
    if constexpr (BITS == 3 && T >= 3) {
        launch_instance<BITS, T, true, TAIL>(g, mix, grid, stream);
    } else {
        if (branch) launch_instance<BITS, T, true, TAIL>(g, mix, grid, stream);
        else launch_instance<BITS, T, false, TAIL>(g, mix, grid, stream);
    }
    return hipGetLastError();
}

template <int BITS>
static hipError_t launch_bits(const SmallGroup<true> &g, bool tail, bool mix, int row_blocks, hipStream_t stream)
{
    const bool branch = g.layer[0].r > 0;
    const dim3 grid(row_blocks, g.n_layers);
    switch (g.layer[0].tiles_per_block * 2 + (tail ? 1 : 0)) {
    case 2: return launch_tiles<BITS, 1, false>(g, branch, mix, grid, stream);
    case 3: return launch_tiles<BITS, 1, true>(g, branch, mix, grid, stream);
    case 4: return launch_tiles<BITS, 2, false>(g, branch, mix, grid, stream);
    case 5: return launch_tiles<BITS, 2, true>(g, branch, mix, grid, stream);
    case 6: return launch_tiles<BITS, 3, false>(g, branch, mix, grid, stream);
    case 7: return launch_tiles<BITS, 3, true>(g, branch, mix, grid, stream);
    case 8: return launch_tiles<BITS, 4, false>(g, branch, mix, grid, stream);
    default: return launch_tiles<BITS, 4, true>(g, branch, mix, grid, stream);
    }
}

// workspace: [16 slices][16][r] 8-byte words {fp32 partial sum of t, launch tag}, then [16][r] words {t, launch tag};
// zero-filled once by the caller
constexpr int kMaxSlices = 16;       // K slices of the down-projection
static_assert(kMaxSlices == kSumSlices, "the summing blocks ask for every slice at once");
static_assert((size_t)(kMaxSlices + 1) * kTokens * kMaxRank * 8 <= kStaticScratchBytes, "the static scratch must hold the largest few-token hand-over");
size_t small_m_workspace_bytes(int K, int r) { (void)K; return (size_t)(kMaxSlices + 1) * kTokens * r * 8; }

static int tiles_per_block_of(int total_tiles, int preparing_blocks, int passes)
{
    // Blocks run one per compute unit, in rounds; a block's time grows with passes x (tiles + about one tile's
    // worth of fixed work: arranging the activations, the reduction).  The blocks that do the down-projection come
    // first in the grid and are gone after about two such units - which only matters where they and the
    // consumers together do not fit the GPU at once: then some consumers start that much later.  (Counting them
    // as full blocks of a round, as an earlier version did, chose one tile per block for long K with few rows:
    // 28672 -> 8192 at 16 tokens 58 us, with two tiles 46; 13824 -> 5120 28.6 and 24.7.)  So: the tile count that
    // makes rounds x passes x (tiles + 1), plus that delay where it applies, smallest.  4096 rows: two tiles in
    // one round beside the preparing blocks instead of one tile and a late start; q/k/v together: four tiles
    // instead of three for the same reason; gate/up together: three tiles in two full rounds rather than four in
    // one and a half; 11008 -> 4096: one tile per block (16.3 us against 17.9 with two).
    constexpr int kPrepUnits = 2;
    int best = 1, best_cost = 1 << 30;
    for (int t = 1; t <= kMaxTiles; ++t) {
        const int consumers = ceil_div(total_tiles, t);
        const int cost = ceil_div(consumers, cu_count()) * passes * (t + 1) + (consumers + preparing_blocks > cu_count() ? kPrepUnits : 0);
        if (cost < best_cost) { best = t; best_cost = cost; }
    }
    return best;
}

// What the kernel itself needs of the layers of one launch: the same instance (a branch-free layer never joins layers
// with a sub-branch).  Activations, token count, outputs and workspace are per layer.
static bool same_instance(const LinearArgs &a, const LinearArgs &b)
{
    return a.K == b.K && a.bits == b.bits && (a.r > 0) == (b.r > 0);
}

// Layers of a grouped call share the launch when they also read the same activations.
bool small_m_group_compatible(const LinearArgs &a, const LinearArgs &b)
{
    return a.x == b.x && a.M == b.M && same_instance(a, b);
}

hipError_t launch_gemv_small_m(const LinearArgs *layers, int n_layers, hipStream_t stream)
{
    if (n_layers < 1 || n_layers > kMaxSmallGroup) return hipErrorInvalidValue;
    const LinearArgs &first = layers[0];
    int total_tiles = 0;
    for (int i = 0; i < n_layers; ++i) {
        if (layers[i].M < 1 || layers[i].M > kTokens || !same_instance(first, layers[i])) return hipErrorInvalidValue;
        total_tiles += ceil_div(layers[i].N, 16);
    }
    // sets of 16 tokens side by side have activations of their own, the layers of a group the same ones
    const bool sets = n_layers > 1 && layers[0].x != layers[1].x;
    bool burst[kMaxSmallGroup] = {false};
    int streamed = 0;
    for (int i = 0; i < n_layers; ++i) {
        burst[i] = !few_stream((sets ? n_layers : 1) * (long)layers[i].N, first.K);
        streamed += !burst[i];
    }
    if (streamed == n_layers || (streamed > 0 && burst_joins_stream(layers, n_layers, burst))) return launch_few_stream(layers, n_layers, burst, stream);
    if (streamed > 0) {                                  // each kind in a launch of its own
        LinearArgs part[kMaxSmallGroup];
        for (const bool small : {false, true}) {
            int n = 0;
            for (int i = 0; i < n_layers; ++i)
                if (burst[i] == small) part[n++] = layers[i];
            const hipError_t e = launch_gemv_small_m(part, n, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    int preparing = 0;
    for (int i = 0; i < n_layers; ++i)
        if (layers[i].r > 0) preparing += ceil_div(layers[i].r, 16) * (ceil_div(layers[i].K, burst_slice_length(layers[i].K)) + 1);
    const int tpb = tiles_per_block_of(total_tiles, preparing, ceil_div(first.K / kGroup, kPassGroups));
    SmallGroup<true> g;
    g.n_layers = n_layers;
    int row_blocks = 0;                                  // widest row of the grid
    for (int i = 0; i < n_layers; ++i) {
        const LinearArgs &a = layers[i];
        MixSmallParams &p = g.layer[i];
        p.qw = a.qw; p.scales = a.scales; p.zeros = a.zeros; p.At = a.At; p.Bt = a.Bt; p.x = a.x; p.y = a.y;
        p.tpart = (uint64_t *)a.workspace;               // each layer's own partial sums of t ...
        p.tsum = p.tpart + (size_t)kMaxSlices * kTokens * a.r;   // ... and their sums
        p.M = a.M; p.N = a.N; p.K = a.K; p.r = a.r;
        p.row_words = (int)row_words(a.K, a.bits);
        p.G = a.K / kGroup;
        // Every consumer block reads all of t at device scope, slice by slice, so few slices: one up to K = 8192 (its
        // producers have the whole main part of the consumers to finish in), at most four.
        p.kslice = burst_slice_length(a.K);
        p.slices = ceil_div(a.K, p.kslice);
        p.down_blocks = a.r > 0 ? ceil_div(a.r, 16) * p.slices : 0;
        p.sum_blocks = a.r > 0 ? ceil_div(a.r, 16) : 0;
        p.tiles_per_block = tpb;
        p.spin_limit = spin_limit();
        p.mix_with = a.mix_with; p.mix_out = a.mix_out;
        row_blocks = std::max(row_blocks, p.down_blocks + p.sum_blocks + ceil_div(ceil_div(a.N, 16), tpb));
    }
    for (int i = n_layers; i < kMaxSmallGroup; ++i) g.layer[i] = g.layer[0];   // never indexed: grid.y stops at n_layers
    bool tail = false;                                  // a layer whose scale array ends in the middle of a dword
    bool mix = false;                                   // averages to be written: with the results, or behind the launch where a layer has such a tail
    for (int i = 0; i < n_layers; ++i) {
        tail = tail || (((long)layers[i].N * g.layer[i].G) & 1);
        mix = mix || layers[i].mix_out;
    }
    hipError_t e = first.bits == 4 ? launch_bits<4>(g, tail, mix, row_blocks, stream) : launch_bits<3>(g, tail, mix, row_blocks, stream);
    for (int i = 0; i < n_layers && e == hipSuccess && tail; ++i)
        if (layers[i].mix_out) e = launch_mix(layers[i], stream);
    return e;
}

}  // namespace fbq
