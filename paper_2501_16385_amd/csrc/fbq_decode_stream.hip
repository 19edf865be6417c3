// Decode path for a few tokens (3 <= M <= 16) of larger layers: the fused kernel of Sec. 4.3 as a stream of packed codes that
// every compute unit reads once from end to end, the tokens riding along as the 16 rows of a matrix-core tile.
//
//   y[M,N] = x[M,K] . Wq[N,K]^T + t[M,r] . B[r,N],   t = x . A
//
// One block per CU, one launch.  A block owns a run of rows; its eight waves split K and keep the activations of their share in
// registers, as matrix operands, while the rows go by in tiles of 16.  What a wave needs of a tile - codes, scales and zeros,
// a unit of 4.5 KB - is copied into a ring of LDS slots of its own, three units ahead, without passing registers; a wave waits
// for its oldest unit by count, takes it into registers and has the slot filled again before it multiplies, so requests stay under
// way whatever the waves do, and nobody waits for anybody but once in four tiles, when the waves' partial results meet.
// (The other kernel for these token counts asks for a pass of a block's tiles in one burst and works on it
// when all is there, one block after the other.)
//
// Products.  A code field stays where it is in the packed word, masked: as an fp16 number it is the subnormal code x gain x 2^-24,
// which the matrix cores multiply exactly (measured); activations that meet a gain are divided by it.  So no offset rides on
// the sums, and per two codes there is one instruction.  The zero points of a unit are one more product,
// sums of activations [token][group] times -s z [group][row], in fp32 on the matrix core.
//
// Down-projection.  The first blocks of a layer do it, slices of K first and their sums behind them, and are gone after some 4 us; the
// rows' blocks that start in their place own fewer rows.  (As a job on the rows' own blocks, which have the activations
// anyway, t came 2 us later: 14336 x 4096, r = 64, 8 tokens 13.5 us with blocks of their own and 14.8 without.)
//
// What bounds it: memory, at about 5.4 TB/s over a long stream, and in front of it 2.7 us for the activations: launch, first round
// trip, change of order (K up to 8192: once; beyond, once a pass and four tiles, 1.5 us each with little under way).  us, the other kernel
// and this one: 28672 x 8192, INT4, r = 128, 16 tokens 46.5 / 31.1 (r = 0: 43.8 / 28.6, of which launch 2, activations 3.4);
// 13824 x 5120, r = 64, 8 tokens 20.3 / 15.8; two layers of 11008 x 4096, INT3, r = 64, 8 tokens 18.7 / 15.5; 5120 x 13824, INT3, r = 128, 48 tokens
// as three sets 38.8 / 36.1.  Tried: four waves with twice the registers (one wave per SIMD issues too slowly: 16 us where this takes 14);
// activations by way of the ring as well (a branch more per unit and twice the code: 15.1 against 13.9); the next
// pass's activations asked for while one is worked on (the wait for them is one for the ring behind them: 38.8 against 33.1); rows dealt
// out in sweeps over the layer instead of runs (35.8 against 33.3).  Instances must not spill vector registers: scratch memory alone costs a launch
// 2 us (50 to 97 scalar ones spill into vector lanes).
#include <type_traits>

#include "fbq_few_burst.h"
#include "fbq_stream_plan.h"

namespace fbq {

constexpr int kUnitGroups = 4;       // quantization groups of a unit: 16 rows x 4 groups, what one ring slot holds
static_assert(kPassGroups == kMainWaves * kUnitGroups, "both kernels take as many groups a pass");
constexpr int kRing = 3;             // ring slots per wave
constexpr int kRoundTiles = 4;       // row tiles between two meetings of the waves

constexpr int kUnitBytes = 16 * 256 + 2 * 256;               // codes (16 bytes per 32, used up or not), scales, zeros
constexpr int kUnitLoads = 6;
constexpr int kAreaAt = kMainWaves * kRing * kUnitBytes;         // 4 KB per wave: a group of activations changing order; partial results
constexpr int kTapAt = kAreaAt + kMainWaves * 4096;
constexpr int kTapBytes = kMaxRank / 32 * 2048;              // t as operands: per 32 taps 1 KB of high halves, 1 KB of low ones
constexpr int kXSumAt = kTapAt + kTapBytes;   // [wave][group][token] sums of the activations
constexpr int kLdsBytes = kXSumAt + kMainWaves * kUnitGroups * 64;   // (a unit's at a time)
static_assert(kLdsBytes <= 160 * 1024, "a block's buffers must fit the CU's LDS");
static_assert(kRoundTiles * 1024 <= 4096 && 2 * kRoundTiles == kMainWaves, "a wave's area holds its part of a round; every wave ends up with one tile of two rounds");

struct StreamParams {
    const uint32_t *qw;
    const uint16_t *scales;
    const uint16_t *zeros;
    const uint16_t *At;    // [r][K]
    const uint16_t *Bt;    // [N][r]
    const uint16_t *x;     // [M][K]
    uint16_t *y;           // [M][N]
    uint64_t *tpart;       // workspace: [slices][16][r] words {fp32 partial sum of t = x.A over one K slice, launch tag}
    uint64_t *tsum;        // workspace: [16][r] words {t, launch tag}: the slices added up
    const uint16_t *mix_with;   // [M][N]
    uint16_t *mix_out;          // null: none
    int M, N, K, r;
    int row_words, G;
    int slices, kslice;    // down-projection: number of K slices and their length (a multiple of 256)
    int down_blocks;       // the layer's first blocks, which do its down-projection, slice by slice ...
    int sum_blocks;        // ... and the blocks after them that add the slices up (16 columns each)
    int early, rows, late_rows;   // the first blocks behind those, `early` of them, own `rows` output rows each, the others fewer
    int passes, share;     // passes over K, and the groups a wave takes in each
    int spin_limit;        // polls for t before a wave computes it itself; negative: at once (test hook)
};
template <bool LINE>
struct StreamGroup {
    StreamParams layer[kMaxSmallGroup];
};
// Blocks in line (see fbq_stream_plan.h): segments 0..3 are the layers' preparing blocks, 4..7 those with their rows; where each starts.
// Layers that are too small for this kernel can come along: `early` is kBurst, and blocks of the other kernel are among their preparing ones.
template <>
struct StreamGroup<true> {
    StreamParams layer[kMaxSmallGroup];
    int segment[2 * kMaxSmallGroup];
};
constexpr int kBurst = -1;
constexpr int burst_tiles(int G) { return G <= kPassGroups ? 3 : 2; }   // tiles of rows of such a block (two or three up to K = 4096: {11008, 4096} x 4096, INT3, no sub-branch 12.6 / 11.8 us)

// Whether small layers share the launch of streamed ones.  Not where rows are so short that a block of theirs is all fixed cost, so long that their
// blocks' passes outlast the stream, or, with two passes and more, where they alone fill the GPU.  us, each kind in a launch of its own / together, 8 tokens
// without a sub-branch and 16 with r = 64: {11008, 4096} x 4096, INT4, 15.6 / 12.6 and 18.9 / 15.4; {10240, 1024, 1024} x 4096, INT3, 14.4 / 10.4 and 17.9 / 13.6;
// {32768, 1024, 1024} x 2048, INT4, 19.0 / 16.1 and 25.1 / 19.7; {12288, 1024, 1024} x 12288, INT4, 34.8 / 27.9 and 39.9 / 38.5.  On the other
// side: {110000, 4000} x 384, INT3, 37.9 / 42.9 and 44.8 / 51.0; {40000, 2048, 2048, 2048} x 1024, INT3, 22.4 / 23.9 and 26.7 / 29.4;
// {16384, 1024, 1024} x 16384, INT3, 47.5 / 50.7 and 56.0 / 69.6; {13000, 1000} x 14336, INT3, 43.7 / 29.6 and 48.2 / 49.5; {10240, 8192} x
// 8192, INT4, 28.4 / 26.4 and, r = 128, 33.1 / 34.9.
bool burst_joins_stream(const LinearArgs *layers, int n_layers, const bool *burst)
{
    int bursts = 0;
    for (int i = 0; i < n_layers; ++i) bursts += burst[i] ? ceil_div(layers[i].N, 16 * burst_tiles(layers[i].K / kGroup)) : 0;
    const int K = layers[0].K;
    return K >= 2048 && (K <= 4096 || (K <= (layers[0].r > 0 ? 12288 : 14336) && bursts < cu_count()));
}
static_assert(kMainWaves * (3 * 1024 + kTokens * 17 * 16) <= kLdsBytes, "the other kernel's buffers must fit into this one's");

// ------------------------------------------------------------------ fused kernel

// BITS: 3 or 4.  C: units of weights a wave takes per tile and pass (4 C groups).  MULTI: several passes over K.  XL: loads of four token rows a group of activations takes.
// LINE: layers dealt out in line; instances of their own, as finding out the layer costs every block 0.05 to 0.1 us.
template <int BITS, int C, int XL, bool MULTI, bool LINE>
__global__ __launch_bounds__(64 * kMainWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void fbq_few_stream_kernel(const StreamGroup<LINE> g)
{
    constexpr int kPiece = BITS == 4 ? 16 : 12;         // bytes of 32 codes
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kLdsBytes];

    int layer = blockIdx.x, index = blockIdx.y;         // the block's place in its layer, preparing blocks first
    if constexpr (LINE) {
        const int id = blockIdx.x;
        int s = 0;
#pragma unroll
        for (int i = 1; i < 2 * kMaxSmallGroup; ++i) s = id >= g.segment[i] ? i : s;
        layer = s & (kMaxSmallGroup - 1);
        index = id - g.segment[s] + (s < kMaxSmallGroup ? 0 : g.segment[layer + 1] - g.segment[layer]);
    }
    const auto p = g.layer[layer];
    // (all of them before the first branch: left alone, the compiler fetches only what the branch needs first)
    asm volatile("" :: "s"(p.qw), "s"(p.scales), "s"(p.zeros), "s"(p.x), "s"(p.y), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.row_words), "s"(p.G), "s"(p.early), "s"(p.rows), "s"(p.late_rows), "s"(p.down_blocks), "s"(p.sum_blocks));
    asm volatile("" :: "s"(p.Bt), "s"(p.At), "s"(p.tpart), "s"(p.tsum), "s"(p.r), "s"(p.passes), "s"(p.share), "s"(p.spin_limit));
    const uint32_t tag = small_m_launch_tag();
    // A layer's first blocks do its down-projection.  They come first in dispatch order, so whoever waits for their
    // words waits for blocks that are already running.
    if (index < p.down_blocks + p.sum_blocks) {
        if (index < p.down_blocks) down_proj_block(p, index, tag, reinterpret_cast<float4_t (*)[64]>(lds));
        else sum_slices_block(p, index - p.down_blocks, tag);
        return;
    }
    const int block = index - p.down_blocks - p.sum_blocks;
    if constexpr (LINE) {
        if (p.early == kBurst) {
            constexpr int kBurstTiles = burst_tiles(C == 1 && !MULTI ? kPassGroups : 2 * kPassGroups);
            few_burst_block<BITS, kBurstTiles, true, true, true>(p, block * kBurstTiles, tag, reinterpret_cast<float4_t (*)[kBurstTiles][64]>(lds),
                                                                 reinterpret_cast<uint4_t (*)[kTokens * 17]>(lds + kMainWaves * kBurstTiles * 1024));
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    // which eighth of a pass is the wave's: turned from block to block, so that the CUs of an XCD do not all ask for the same activations at once
    const int kw = (wave + block + (block >> 3)) & (kMainWaves - 1);
    const int row0 = min(block < p.early ? block * p.rows : p.early * p.rows + (block - p.early) * p.late_rows, p.N);
    const int row_end = min(p.N, row0 + (block < p.early ? p.rows : p.late_rows));
    const int tiles = (row_end - row0 + 15) >> 4;
    if (tiles == 0) return;                             // (a column of the grid with a block less than the others)
    const int passes = MULTI ? p.passes : 1;
    const int row_bytes = p.row_words * 4;
    constexpr int kNowhere = 0x40000000;                // beyond every buffer
    constexpr int kFar = 0x20000000;                    // beyond x and A, also on top of it

    // Rows past the block's own are outside the descriptors: zeros, without a memory access.  The range check is per dword, so the
    // counts of scales and zeros are rounded up to whole dwords (the half behind an odd-sized array is masked out below).
    const __amdgpu_buffer_rsrc_t qbuf = buffer_of(p.qw, (long)row_end * row_bytes);
    const __amdgpu_buffer_rsrc_t sbuf = buffer_of(p.scales, ((long)row_end * p.G * 2 + 3) & ~3L);
    const __amdgpu_buffer_rsrc_t zbuf = buffer_of(p.zeros, ((long)row_end * p.G * 2 + 3) & ~3L);

    unsigned char *const ring = lds + wave * (kRing * kUnitBytes);
    unsigned char *const slab = lds + kAreaAt + kw * 4096;
    float4_t *const sums = reinterpret_cast<float4_t *>(slab);
    const uint32_t ring_lds = lds_offset(ring);

    // A unit's copies.  Copy j of the codes moves rows 4 j .. 4 j + 3, 16 lanes and up to 256 contiguous bytes a row; row n's piece i
    // (32 codes) lies at position i ^ n of it, so that the 16 rows of a matrix operand touch every bank once.  Scales and zeros: the
    // aligned dwords that hold the four groups' halves, four lanes a row.  Groups past the wave's share aim nowhere; those of the share that lie
    // past the end of K are whatever follows, and meet activations of zero.
    int qoff[4], qoff_last[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = 4 * j + q, piece = c ^ row;
        qoff[j] = row * row_bytes + piece * kPiece;
        qoff_last[j] = (piece >> 2) < p.share - kUnitGroups * (C - 1) ? qoff[j] : kNowhere;
    }
    const int soff = (lane >> 2) * p.G, sdword = 4 * min(lane & 3, 2);
    auto first_group = [&](int pass) __attribute__((always_inline)) { return (pass * kMainWaves + kw) * p.share; };
    auto issue_unit = [&](int slot, int tile, int chunk, int pass) __attribute__((always_inline)) {
        const int g0 = first_group(pass) + kUnitGroups * chunk, n0 = row0 + 16 * tile;
        const int base = n0 * row_bytes + g0 * (4 * kPiece);
        const uint32_t dst = ring_lds + slot * kUnitBytes;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int off = (C == 1 || chunk == C - 1 ? qoff_last[j] : qoff[j]) + base;
            if constexpr (BITS == 4) copy16_to_lds(qbuf, off, 0, dst + j * 1024);
            else copy12_to_lds(qbuf, off, 0, dst + j * 1024);
        }
        const int so = ((soff + n0 * p.G + g0) * 2 & ~3) + sdword;
        copy4_to_lds(sbuf, so, 0, dst + 4096);
        copy4_to_lds(zbuf, so, 0, dst + 4096 + 256);
    };
    // The sequence of units: rounds of kRoundTiles tiles, in each the passes over K, in each the tiles, in each the chunks of K.
    int i_tile = 0, i_first = 0, i_end = min(kRoundTiles, tiles), i_chunk = 0, i_pass = 0, i_slot = 0;
    int ahead = 0;                                      // units under way or landed and not yet used
    auto issue_next = [&]() __attribute__((always_inline)) {
        if (i_first >= tiles) return;
        issue_unit(i_slot, i_tile, i_chunk, i_pass);
        ++ahead;
        i_slot = i_slot + 1 == kRing ? 0 : i_slot + 1;
        if (++i_chunk < C) return;
        i_chunk = 0;
        if (++i_tile < i_end) return;
        i_tile = i_first;
        if (++i_pass < passes) return;
        i_pass = 0;
        i_first = i_tile = i_end;
        i_end = min(i_first + kRoundTiles, tiles);
    };
    // The oldest unit has landed: at most the younger ones' copies are under way.  (Other loads only make the wait longer.)
    auto wait_unit = [&]() __attribute__((always_inline)) {
        static_assert(kRing == 3 && kUnitLoads == 6, "the counts below");
        if (ahead >= 3) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
        else if (ahead == 2) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    auto block_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    const int tap_steps = (p.r + 31) >> 5;
    constexpr int kHeld = 4;             // operands of the rows of B^T of the wave's tile among the first eight, asked for early
    half8_t ubf[kHeld];                                 // (outside the loops, where a wait for them would be one for the ring)
    const __amdgpu_buffer_rsrc_t bbuf = buffer_of(p.Bt, (long)row_end * p.r * 2);
    auto taps = [&](int row, int js) __attribute__((always_inline)) {
        const int j = js * 32 + q * 8;
        return __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(bbuf, j < p.r ? (row * p.r + j) * 2 : kNowhere, 0, 0));
    };
    issue_next();                                       // the first tile's weights are on their way before the activations
#pragma unroll
    for (int k = 0; k < kHeld; ++k) ubf[k] = half8_t{};
    if (C == 1 && tap_steps > 0) {
#pragma unroll
        for (int k = 0; k < kHeld; ++k) ubf[k] = taps(row0 + wave * 16 + c, k);
    }

    const float4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    half8_t xa[C][kUnitGroups][4];
    float xs[C];                                        // sums of the activations of token c and a unit's group q
    unsigned char *const xsum = lds + kXSumAt + kw * (kUnitGroups * 64);
    uint32_t smask[C][2];                               // which halves of a unit's scales belong to groups of the wave's share
    int valid[C];                                       // how many of a unit's groups do

    // The wave's activations of a pass: loaded a group at a time, four token rows per load (16 lanes, 256 contiguous bytes a row), passed
    // through LDS into operand order.  kWindow groups are under way at a time.
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(p.x, (long)p.M * p.K * 2);
    constexpr int kWindow = C == 1 || XL < 4 ? 4 : 2;
    uint4_t xraw[kWindow][XL];
    // (Addresses are worked out where they are used: kept from pass to pass, they would take the registers that the operands need.)
    auto afresh = [](int v) __attribute__((always_inline)) { asm volatile("" : "+v"(v)); return v; };
    auto request_group = [&](int pass, int i, int c, int q) __attribute__((always_inline)) {
        const int group = first_group(pass) + i;
        const int at = i < p.share && group < p.G ? group * 256 + c * 16 : kFar;
#pragma unroll
        for (int k = 0; k < XL; ++k) xraw[i % kWindow][k] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (4 * k + q < p.M ? (4 * k + q) * p.K * 2 : kNowhere) + at, 0, 0);
    };
    auto request_x = [&](int pass) __attribute__((always_inline)) {
        const int l = afresh(lane);
#pragma unroll
        for (int i = 0; i < kWindow; ++i) request_group(pass, i, l & 15, l >> 4);
    };
    auto arrange_x = [&](int pass) __attribute__((always_inline)) {
        const int l = afresh(lane), c = l & 15, q = l >> 4;
#pragma unroll
        for (int ch = 0; ch < C; ++ch) {
#pragma unroll
            for (int gi = 0; gi < kUnitGroups; ++gi) {
                const int n = ch * kUnitGroups + gi;
                uint4_t mine[4];
#pragma unroll
                for (int i = 0; i < XL; ++i) *reinterpret_cast<uint4_t *>(slab + (4 * i + q) * 256 + ((c ^ (4 * i + q)) << 4)) = xraw[n % kWindow][i];
                if (n + kWindow < C * kUnitGroups) request_group(pass, n + kWindow, c, q);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < 4; ++i) mine[i] = *reinterpret_cast<const uint4_t *>(slab + c * 256 + (((4 * q + i) ^ c) << 4));
                __builtin_amdgcn_wave_barrier();
                arrange_operands<BITS>(mine, xa[ch][gi]);
                float4_t sx = zero4;
#pragma unroll
                for (int t = 0; t < 4; ++t) sx = mfma(xa[ch][gi][t], gain_operand<BITS>(t), sx);
                if (c == 0) *reinterpret_cast<float4_t *>(xsum + gi * 64 + q * 16) = sx * 0x1p-24f;
            }
            __builtin_amdgcn_wave_barrier();
            const float4_t *const row = reinterpret_cast<const float4_t *>(xsum + q * 64 + (c & 12) * 4);   // (as it was stored: the compiler must not take these for unrelated)
            const float4_t four = *row;
            xs[ch] = c & 2 ? (c & 1 ? four.w : four.z) : (c & 1 ? four.y : four.x);
            valid[ch] = min(p.share, p.G - first_group(pass)) - kUnitGroups * ch;
            smask[ch][0] = (valid[ch] > 0 ? 0xFFFFu : 0u) | (valid[ch] > 1 ? 0xFFFF0000u : 0u);
            smask[ch][1] = (valid[ch] > 2 ? 0xFFFFu : 0u) | (valid[ch] > 3 ? 0xFFFF0000u : 0u);
        }
    };
    // Eight words {t, tag} of this wave's 32 taps.
    const __amdgpu_buffer_rsrc_t tbuf = buffer_of(p.tsum, (long)kTokens * p.r * 8);
    uint4_t tw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tw[k] = uint4_t{0, 0, 0, 0};
    auto ask_t = [&]() __attribute__((always_inline)) {
        const int l = afresh(lane), j = 32 * wave + 8 * (l >> 4);
        const int off = (l & 15) < 4 * XL && j < p.r ? ((l & 15) * p.r + j) * 8 : kNowhere;
#pragma unroll
        for (int k = 0; k < 4; ++k) tw[k] = __builtin_amdgcn_raw_buffer_load_b128(tbuf, off + 16 * k, 0, kCacheSc1);
    };
    int u_slot = 0;
    bool start = true;
    float4_t mine = zero4;                              // the wave's tile: number `wave` of the eight of two rounds
    for (int first_tile = 0;;) {
        const int nt = min(kRoundTiles, tiles - first_tile);
        const int eight = first_tile & ~(kMainWaves - 1);   // first tile of the eight
        for (int pass = 0; pass < passes; ++pass) {
            if (start || MULTI) {
                float4_t kept[kRoundTiles];             // the area holds partial results of the passes before
                if (MULTI && pass > 0) {
#pragma unroll
                    for (int ti = 0; ti < kRoundTiles; ++ti) kept[ti] = sums[ti * 64 + lane];
                    asm volatile("" ::: "memory");  // (the same LDS under another type: the compiler keeps the order)
                }
                request_x(pass);
                arrange_x(pass);
                if (MULTI && pass > 0) {
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int ti = 0; ti < kRoundTiles; ++ti) sums[ti * 64 + lane] = kept[ti];
                }
                start = false;
            }
            while (ahead < kRing && i_first < tiles) issue_next();
            for (int ti = 0; ti < nt; ++ti) {
                float4_t acc = zero4;
                // the row's first half may be the upper one of its dword
                const int odd = ((row0 + (first_tile + ti) * 16 + c) * p.G + first_group(pass)) & 1;   // (chunks are four groups apart)
#pragma unroll
                for (int ch = 0; ch < C; ++ch) {
                    wait_unit();
                    const unsigned char *const unit = ring + u_slot * kUnitBytes;
                    uint4_t w[kUnitGroups];
#pragma unroll
                    for (int gi = 0; gi < kUnitGroups; ++gi) w[gi] = *reinterpret_cast<const uint4_t *>(unit + c * 256 + (((4 * gi + q) ^ c) << 4));
                    const uint4_t s4 = *reinterpret_cast<const uint4_t *>(unit + 4096 + c * 16);
                    const half_t sq = *reinterpret_cast<const half_t *>(unit + 4096 + c * 16 + (odd + q) * 2), zq = *reinterpret_cast<const half_t *>(unit + 4096 + 256 + c * 16 + (odd + q) * 2);
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // in registers: the slot may be filled again
                    u_slot = u_slot + 1 == kRing ? 0 : u_slot + 1;
                    --ahead;
                    issue_next();
                    const uint32_t s01 = __builtin_amdgcn_alignbit(s4.y, s4.x, 16 * odd) & smask[ch][0], s23 = __builtin_amdgcn_alignbit(s4.z, s4.y, 16 * odd) & smask[ch][1];
                    // the zero points of all four groups are one more product: sums of activations [token][group] times -s z [group][row]
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[ch], q < valid[ch] ? -(float)sq * (float)zq : 0.0f, acc, 0, 0, 0);
#pragma unroll
                    for (int gi = 0; gi < kUnitGroups; ++gi) {
                        half8_t b[4];
                        code_operands<BITS>(w[gi], b);
                        float4_t D = zero4;
#pragma unroll
                        for (int t = 0; t < 4; ++t) D = mfma(xa[ch][gi][t], b[t], D);
                        const half2_t sh = h2_of(gi < 2 ? s01 : s23);
                        const float s = (float)(gi & 1 ? sh.y : sh.x);
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[v] = fmaf(s, D[v], acc[v]);
                    }
                }
                float4_t *const slot = sums + ti * 64 + lane;
                *slot = pass == 0 ? acc * 0x1p24f : *slot + acc * 0x1p24f;
            }
        }

        // The waves meet; tile ti of the round goes to wave ti or, in the second round of two, ti + 4.
        const bool last = first_tile + kRoundTiles >= tiles;
        const bool store = last || first_tile != eight;
        // With the results to be stored: t, 32 taps a wave, lane (c, q) eight of them for token c, as two fp16 halves (22 bits) in
        // operand order: [32 taps][hi, lo][8 taps][token].  Should the tags not turn up, the lane computes its eight values itself.
        half8_t late[kHeld];
        if (store && p.r > 0) {
            const int my_row = row0 + (eight + wave) * 16 + c;
            if (C > 1 || eight > 0) {
#pragma unroll
                for (int k = 0; k < kHeld; ++k) late[k] = taps(my_row, k);
            }
            if (wave < tap_steps) {
                // (Not while the last tile is worked on: an answer that comes too early costs a second round trip, and more blocks
                // wait for words that are not there yet.  11008 x 4096, r = 64, 16 tokens: INT4 11.4 us with the early request, 11.1 without, INT3 10.5 / 10.0.)
                if (p.spin_limit > 0) ask_t();
                const int l = afresh(lane), c = l & 15, j = 32 * wave + 8 * (l >> 4);
                const bool mine_too = c < 4 * XL && j < p.r;
                bool ready = false;
#pragma unroll 1
                for (int spin = 0; spin < p.spin_limit; ++spin) {
                    bool ok = true;
#pragma unroll
                    for (int k = 0; k < 4; ++k) ok = ok && (!mine_too || (tw[k].y == tag && tw[k].w == tag));
                    ready = __all(ok);
                    if (ready) break;
                    ask_t();
                }
                __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): no load that the compiler would wait for in the tile loop
                half8_t hi, lo;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t word = e & 1 ? tw[e / 2].z : tw[e / 2].x;
                    float t = __builtin_bit_cast(float, word);
                    if (!ready && mine_too) {
                        const uint16_t *xr = p.x + (size_t)min(c, p.M - 1) * p.K, *ar = p.At + (size_t)(j + e) * p.K;
                        t = 0.0f;
#pragma unroll 1
                        for (int i = 0; i < p.K; ++i) t = fmaf((float)__builtin_bit_cast(half_t, xr[i]), (float)__builtin_bit_cast(half_t, ar[i]), t);
                    }
                    hi[e] = (half_t)t;
                    lo[e] = (half_t)(t - (float)hi[e]);
                }
                *reinterpret_cast<half8_t *>(lds + kTapAt + wave * 2048 + l * 16) = hi;
                *reinterpret_cast<half8_t *>(lds + kTapAt + wave * 2048 + 1024 + l * 16) = lo;
            }
        }
        block_barrier();
        const int mt = wave - (first_tile - eight);
        if (mt >= 0 && mt < nt) {                       // wave-uniform
            const float4_t *const part = reinterpret_cast<const float4_t *>(lds + kAreaAt) + mt * 64 + afresh(lane);
            mine = part[0];
#pragma unroll
            for (int k = 1; k < kMainWaves; ++k) mine += part[k * 256];
        }
        if (store && eight + wave < min(tiles, first_tile + kRoundTiles)) {   // wave-uniform
            const int l = afresh(lane), c = l & 15, q = l >> 4, my_row = row0 + (eight + wave) * 16 + c;
            auto fold = [&](int js, half8_t bf) __attribute__((always_inline)) {
                const unsigned char *const at = lds + kTapAt + js * 2048 + l * 16;
                float4_t d = mfma(*reinterpret_cast<const half8_t *>(at), bf, zero4);
                mine += mfma(*reinterpret_cast<const half8_t *>(at + 1024), bf, d);
            };
#pragma unroll
            for (int k = 0; k < kHeld; ++k)
                if (k < tap_steps) fold(k, C == 1 && eight == 0 ? ubf[k] : late[k]);
            if (tap_steps > kHeld) {
#pragma unroll
                for (int k = 0; k < kHeld; ++k) late[k] = taps(my_row, kHeld + k);
#pragma unroll
                for (int k = 0; k < kHeld; ++k)
                    if (kHeld + k < tap_steps) fold(kHeld + k, late[k]);
            }
            // lane (c, q) holds output row my_row and tokens 4 q + v
            if (my_row < row_end) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = 4 * q + v;
                    if (m < p.M) {
                        const half_t y = (half_t)mine[v];
                        p.y[(size_t)m * p.N + my_row] = __builtin_bit_cast(uint16_t, y);
                        if (p.mix_out) {
                            const float with = (float)__builtin_bit_cast(half_t, p.mix_with[(size_t)m * p.N + my_row]);
                            p.mix_out[(size_t)m * p.N + my_row] = __builtin_bit_cast(uint16_t, (half_t)((float)y - ((float)y - with) * 0.5f));
                        }
                    }
                }
            }
        }
        if (last) return;
        if (store) __builtin_amdgcn_s_waitcnt(0x0F70);
        block_barrier();                                // (the partial results, and t, may be written again)
        first_tile += kRoundTiles;
    }
}

template <int BITS, int C, bool MULTI, bool LINE>
static void launch_instance(const StreamGroup<LINE> &g, bool half, dim3 grid, hipStream_t stream)
{
    if (half) hipLaunchKernelGGL((fbq_few_stream_kernel<BITS, C, 2, MULTI, LINE>), grid, dim3(64 * kMainWaves), 0, stream, g);
    else hipLaunchKernelGGL((fbq_few_stream_kernel<BITS, C, 4, MULTI, LINE>), grid, dim3(64 * kMainWaves), 0, stream, g);
}
template <bool LINE>
static hipError_t launch_group(const StreamGroup<LINE> &g, int bits, int chunks, bool multi, bool half, dim3 grid, hipStream_t stream)
{
    if (bits == 4) {
        if (chunks > 1) launch_instance<4, 2, false>(g, half, grid, stream);
        else if (multi) launch_instance<4, 1, true>(g, half, grid, stream);
        else launch_instance<4, 1, false>(g, half, grid, stream);
    } else {
        if (chunks > 1) launch_instance<3, 2, false>(g, half, grid, stream);
        else if (multi) launch_instance<3, 1, true>(g, half, grid, stream);
        else launch_instance<3, 1, false>(g, half, grid, stream);
    }
    return hipGetLastError();
}

// Length of a K slice of the down-projection: slices only exist to put more CUs to work on a short, latency-bound step, and every block
// of it is a CU that starts late on its rows (28672 x 8192, r = 128, 16 tokens: up to 32 such blocks 32.7 us, 64 30.7, 128 30.8).
constexpr int kMaxDownBlocks = 64;
static int slice_length(int K, int r)
{
    constexpr int kStep = 32 * kMainWaves;
    int len = std::max(1024, ceil_div(ceil_div(K, kSumSlices), kStep) * kStep);
    while (ceil_div(r, 16) * ceil_div(K, len) > kMaxDownBlocks) len += kStep;
    return len;
}
static int down_blocks(const LinearArgs &a, int slice) { return a.r > 0 ? ceil_div(a.r, 16) * (ceil_div(a.K, slice) + 1) : 0; }

hipError_t launch_few_stream(const LinearArgs *layers, int n_layers, const bool *burst, hipStream_t stream)
{
    const LinearArgs &first = layers[0];
    const int G = first.K / kGroup;
    const int chunks = G > kPassGroups && G <= 2 * kPassGroups ? 2 : 1;
    const int passes = ceil_div(G, chunks * kPassGroups), share = ceil_div(G, kMainWaves * passes);
    int order[kMaxSmallGroup], rows_of[kMaxSmallGroup], preparing[kMaxSmallGroup], slice[kMaxSmallGroup], most = 0, n = 0;
    long busy = 0;                                       // what CUs would stream in while they run preparing blocks, in bytes
    int prep = 0;
    for (int kind = 1; kind >= 0; --kind) {              // small layers first: their blocks are short
        for (int i = 0; i < n_layers; ++i) {
            if (burst[i] != (bool)kind) continue;
            const LinearArgs &a = layers[i];
            slice[n] = kind ? burst_slice_length(a.K) : slice_length(a.K, a.r);
            const int down = down_blocks(a, slice[n]), bursts = kind ? ceil_div(a.N, 16 * burst_tiles(G)) : 0;
            rows_of[n] = kind ? 0 : a.N;
            preparing[n] = down + bursts;
            busy += (long)down * stream_down_bytes(slice[n]) + (long)bursts * stream_burst_bytes(a.K);
            prep += preparing[n];
            most = std::max(most, a.M);
            order[n++] = i;
        }
    }
    const int row_bytes = (int)row_words(first.K, first.bits) * 4 + 4 * G;
    const int behind = prep ? std::max(1, (int)(busy / prep / row_bytes)) : 0;
    const bool line = stream_in_line(rows_of, preparing, n_layers);
    const StreamPlan plan = plan_stream(rows_of, preparing, n_layers, behind, passes, cu_count());
    StreamGroup<true> g;
    int widest = 0;
    for (int i = 0; i < n_layers; ++i) {
        const LinearArgs &a = layers[order[i]];
        StreamParams &p = g.layer[i];
        p.qw = a.qw; p.scales = a.scales; p.zeros = a.zeros; p.At = a.At; p.Bt = a.Bt; p.x = a.x; p.y = a.y;
        p.tpart = (uint64_t *)a.workspace;               // each layer's own partial sums of t ...
        p.tsum = p.tpart + (size_t)kSumSlices * kTokens * a.r;   // ... and their sums
        p.mix_with = a.mix_with; p.mix_out = a.mix_out;
        p.M = a.M; p.N = a.N; p.K = a.K; p.r = a.r;
        p.row_words = (int)row_words(a.K, a.bits);
        p.G = G;
        p.kslice = slice[i];
        p.slices = ceil_div(a.K, p.kslice);
        p.down_blocks = a.r > 0 ? ceil_div(a.r, 16) * p.slices : 0;
        p.sum_blocks = a.r > 0 ? ceil_div(a.r, 16) : 0;
        p.rows = plan.rows;
        p.late_rows = plan.late_rows;
        p.early = burst[order[i]] ? kBurst : plan.early[i];
        p.passes = passes; p.share = share;
        p.spin_limit = spin_limit();
        widest = std::max(widest, preparing[i] + plan.early[i] + plan.late[i]);
    }
    for (int i = n_layers; i < kMaxSmallGroup; ++i) g.layer[i] = g.layer[0];   // never indexed: the grid stops before
    const bool half = most <= 8;
    if (line) {
        int start = 0;
        for (int s = 0; s < 2 * kMaxSmallGroup; ++s) {
            const int i = s & (kMaxSmallGroup - 1);
            g.segment[s] = start;
            if (i < n_layers) start += s < kMaxSmallGroup ? preparing[i] : plan.early[i] + plan.late[i];
        }
        return launch_group(g, first.bits, chunks, passes > 1, half, dim3(start), stream);
    }
    StreamGroup<false> alike;
    std::copy(g.layer, g.layer + kMaxSmallGroup, alike.layer);
    return launch_group(alike, first.bits, chunks, passes > 1, half, dim3(n_layers, widest), stream);
}

}  // namespace fbq
