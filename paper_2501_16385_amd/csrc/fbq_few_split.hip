// 3 to 64 tokens of layers with long rows: K is split over blocks, all tokens of the call meet the codes in one block, and a second
// launch adds up.
//
//   y[M,N] = x[M,K] . Wq[N,K]^T + t[M,r] . B[r,N],   t = x . A
//
// The other two kernels for a few tokens own all of K for their rows, so every CU reads all activations (48 tokens of 13824: 1.3 MB for
// 104 KB of codes) in several passes, and 16 tokens at a time, so every set of 16 reads the words again.  Here a block owns a run of rows and a
// segment of K.  Its eight waves split the segment and keep the activations of their share, of all S sets of 16 tokens, in registers as
// operands for the whole run; codes, scales and zeros come through rings of LDS slots of each wave's own, one or two units ahead, as in
// the streaming kernel, from which the products are taken too (masked fields as subnormal fp16 numbers, zero points as an fp32 product).  After every
// one to four units the waves' partial sums meet in LDS, and go to the workspace in fp32, as the accumulators lie: [segment][set][tile][lane].
//
// Down-projection: blocks of their own, in front, take rows of A^T instead of rows of codes, with the same segments of K: partial sums of t, in the
// same layout.
//
// The second launch (fbq_few_join_kernel) adds the segments up, t included, adds t . B on the matrix cores with t as two fp16 halves (22
// bits), and stores y, averaged with another tensor if asked.  Nothing waits inside a launch, and no words are handed over.
//
// What it takes, us, before (three sets of the streaming kernel, its several passes, or the prefill GEMM) and now: 13824 -> 5120, INT3, r = 128,
// 48 tokens 35.1 / 23.7; 28672 -> 8192, INT3, r = 128, 32 tokens 58.3 / 36.7; 8192 -> 28672, INT4, r = 128, 64 tokens 70.7 / 59; 28672 -> 8192, INT4,
// r = 128, 16 tokens 43.6 / 36.1.  Of the 23.7, with parts left out: products 5, copies of codes not hidden behind them 3, activations 2, partial
// sums to the workspace and meetings 5, the second launch 5.6.  With four sets of a wide layer the partial sums bound it (29 MB each way).
#include <algorithm>

#include "fbq_few_tokens.h"
#include "fbq_split_plan.h"

namespace fbq {

struct SplitParams {
    const uint32_t *qw;
    const uint16_t *scales;
    const uint16_t *zeros;
    const uint16_t *At;    // [r][K]
    const uint16_t *x;     // [M][K]
    float4_t *part;        // [segment][set][tile of 16 rows][lane] sums: lane (c, q) has row c and tokens 4 q .. 4 q + 3 of the set
    float4_t *tpart;       // [segment][set][tile of 16 taps][lane]
    int M, N, K, r;
    int row_words, G;
    int segments, share;   // segments of K, and the groups a wave takes of one
    int tap_blocks, taps;  // blocks for A^T per segment, and tiles of 16 taps each owns
    int row_blocks, units; // blocks for rows per segment, and units of rows each owns
};
struct SplitGroup {
    SplitParams layer[kMaxSmallGroup];
    int start[kMaxSmallGroup];   // a layer's first block
};

// S sets of 16 tokens.
template <int S>
struct SplitShape {
    static constexpr int kGroups = S <= 2 ? 4 : 2;       // groups a wave can hold the activations of: 64 (S = 1), 128, 96, 128 registers
    static constexpr int kUnitRows = 64 / kGroups;       // a unit: 16 rows x 4 groups or 32 x 2
    static constexpr int kUnitTiles = kUnitRows / 16;
    static constexpr int kRing = S == 4 ? 2 : 3;
    static constexpr int kRoundUnits = S == 1 ? 4 : (S == 2 ? 2 : 1);    // units between two meetings of the waves
    static constexpr int kAreaBytes = kRoundUnits * kUnitTiles * S * 1024;   // a wave's partial sums of a round; before, a group of activations changing order (4 KB)
    static constexpr int kUnitBytes = 16 * 256 + 2 * 256;   // codes (16 bytes per 32, used up or not), scales, zeros
    static constexpr int kAreaAt = kMainWaves * kRing * kUnitBytes;
    static constexpr int kXSumAt = kAreaAt + kMainWaves * kAreaBytes;
    static constexpr int kLdsBytes = kXSumAt + kMainWaves * kGroups * 64;
    static_assert(kLdsBytes <= 160 * 1024 && kAreaBytes >= 4096 && kRoundUnits * kUnitTiles * S <= kMainWaves, "a block's buffers, a wave's slab, a wave per pair of tile and set");
};

template <int BITS, int S, int XL>
__global__ __launch_bounds__(64 * kMainWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void fbq_few_split_kernel(const SplitGroup g)
{
    using Shape = SplitShape<S>;
    constexpr int kGroups = Shape::kGroups, kUnitRows = Shape::kUnitRows, kUnitTiles = Shape::kUnitTiles, kRing = Shape::kRing, kUnitBytes = Shape::kUnitBytes;
    constexpr int kPiece = BITS == 4 ? 16 : 12;         // bytes of 32 codes
    constexpr int kNowhere = 0x40000000;                // beyond every buffer
    constexpr int kFar = 0x20000000;                    // beyond x and A, also on top of it
    __shared__ __attribute__((aligned(1024))) unsigned char lds[Shape::kLdsBytes];

    int layer = 0;
#pragma unroll
    for (int i = 1; i < kMaxSmallGroup; ++i) layer = (int)blockIdx.x >= g.start[i] ? i : layer;
    const auto p = g.layer[layer];
    int index = blockIdx.x - g.start[layer];
    const bool of_taps = index < p.segments * p.tap_blocks;
    if (!of_taps) index -= p.segments * p.tap_blocks;
    const int run = index / p.segments, segment = index - run * p.segments;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    // which eighth of the segment is the wave's: turned from block to block, so that the CUs of an XCD do not all ask for the same activations at once
    const int kw = (wave + run + (run >> 3)) & (kMainWaves - 1);
    const int first_group = (segment * kMainWaves + kw) * p.share;
    const int valid = max(0, min(p.share, p.G - first_group));   // groups of the wave's that exist

    unsigned char *const slab = lds + Shape::kAreaAt + kw * Shape::kAreaBytes;
    float4_t *const sums = reinterpret_cast<float4_t *>(slab);
    float *const xsum = reinterpret_cast<float *>(lds + Shape::kXSumAt + kw * (kGroups * 64));   // [group][token]
    auto block_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // After a meeting: wave w adds up pair w of tile and set and passes it on.
    auto join_waves = [&](int pair) __attribute__((always_inline)) {
        const float4_t *const from = reinterpret_cast<const float4_t *>(lds + Shape::kAreaAt) + pair * 64 + lane;
        float4_t sum = from[0];
#pragma unroll
        for (int k = 1; k < kMainWaves; ++k) sum += from[k * (Shape::kAreaBytes / 16)];
        return sum;
    };
    const float4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};

    // ---- codes, scales and zeros into the ring
    const int row0 = of_taps ? 0 : run * p.units * kUnitRows, row_end = of_taps ? 0 : min(p.N, row0 + p.units * kUnitRows);
    const int units = max(0, row_end - row0 + kUnitRows - 1) / kUnitRows;
    if (!of_taps && units == 0) return;
    const int row_bytes = p.row_words * 4;
    // Rows past the block's own are outside the descriptors: zeros, without a memory access.  The range check is per dword, so the
    // counts of scales and zeros are rounded up to whole dwords (the half behind an odd-sized array is masked out below).
    const __amdgpu_buffer_rsrc_t qbuf = buffer_of(p.qw, (long)row_end * row_bytes);
    const __amdgpu_buffer_rsrc_t sbuf = buffer_of(p.scales, ((long)row_end * p.G * 2 + 3) & ~3L);
    const __amdgpu_buffer_rsrc_t zbuf = buffer_of(p.zeros, ((long)row_end * p.G * 2 + 3) & ~3L);
    unsigned char *const ring = lds + wave * (kRing * kUnitBytes);
    const uint32_t ring_lds = lds_offset(ring);
    // A unit's copies.  Copy j of the codes moves 4 rows of 16 pieces or 8 of 8 (a piece is 32 codes), up to 256 contiguous bytes a row; a row's
    // pieces are XORed with a key of the row, so that the 16 rows of a matrix operand touch every bank once.  Scales and zeros: the
    // aligned dwords that hold the groups' halves, four or two lanes a row.  Pieces of groups that do not exist aim nowhere.
    auto key = [](int row) __attribute__((always_inline)) { return kGroups == 4 ? row : (row >> 1) & 7; };
    int qoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = kGroups == 4 ? 4 * j + q : 8 * j + (lane >> 3), piece = (kGroups == 4 ? c : lane & 7) ^ key(row);
        qoff[j] = (piece >> 2) < valid ? row * row_bytes + piece * kPiece : kNowhere;
    }
    const int soff = (kGroups == 4 ? lane >> 2 : lane >> 1) * p.G, sdword = 4 * (kGroups == 4 ? min(lane & 3, 2) : lane & 1);
    int i_unit = 0, i_slot = 0, u_slot = 0, ahead = 0;  // next unit to ask for, its slot, the slot to be used next, units under way or landed
    auto issue_next = [&]() __attribute__((always_inline)) {
        if (i_unit >= units) return;
        const int n0 = row0 + i_unit * kUnitRows, base = n0 * row_bytes + first_group * (4 * kPiece);
        const uint32_t dst = ring_lds + i_slot * kUnitBytes;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (BITS == 4) copy16_to_lds(qbuf, qoff[j] + base, 0, dst + j * 1024);
            else copy12_to_lds(qbuf, qoff[j] + base, 0, dst + j * 1024);
        }
        const int so = ((soff + n0 * p.G + first_group) * 2 & ~3) + sdword;
        copy4_to_lds(sbuf, so, 0, dst + 4096);
        copy4_to_lds(zbuf, so, 0, dst + 4096 + 256);
        ++i_unit;
        ++ahead;
        i_slot = i_slot + 1 == kRing ? 0 : i_slot + 1;
    };
    // The oldest unit has landed: at most the younger ones' six copies each are under way.  (Other loads and stores only make the wait longer.)
    auto wait_unit = [&]() __attribute__((always_inline)) {
        if (ahead >= 3) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
        else if (ahead == 2) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };

    // ---- activations: a group at a time, four token rows per load (16 lanes, 256 contiguous bytes a row), through LDS into operand order
    auto request = [&](const __amdgpu_buffer_rsrc_t &from, int row, int end, int gi, uint4_t *raw, int loads) __attribute__((always_inline)) {
        const int at = gi < valid ? (first_group + gi) * 256 + c * 16 : kFar;
#pragma unroll
        for (int k = 0; k < loads; ++k) raw[k] = __builtin_amdgcn_raw_buffer_load_b128(from, (row + 4 * k + q < end ? (row + 4 * k + q) * p.K * 2 : kNowhere) + at, 0, 0);
    };
    auto turn = [&](const uint4_t *raw, int loads, uint4_t (&mine)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < loads; ++i) *reinterpret_cast<uint4_t *>(slab + (4 * i + q) * 256 + ((c ^ (4 * i + q)) << 4)) = raw[i];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 4; ++i) mine[i] = *reinterpret_cast<const uint4_t *>(slab + c * 256 + (((4 * q + i) ^ c) << 4));
        __builtin_amdgcn_wave_barrier();
    };
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(p.x, (long)p.M * p.K * 2);
    half8_t xa[S][kGroups][4];
    float xs[S];                                        // sums of the activations of token c and group q
    constexpr int kWindow = S * kGroups == 6 ? 6 : 4;    // groups under way
    {
        uint4_t raw[kWindow][XL];
#pragma unroll
        for (int n = 0; n < kWindow; ++n) request(xbuf, 16 * (n / kGroups), p.M, n % kGroups, raw[n], XL);
        if (!of_taps) issue_next();                     // (behind the activations: loads come back in order)
#pragma unroll
        for (int n = 0; n < S * kGroups; ++n) {
            const int set = n / kGroups, gi = n % kGroups;
            uint4_t mine[4];
            turn(raw[n % kWindow], XL, mine);
            if (n + kWindow < S * kGroups) request(xbuf, 16 * ((n + kWindow) / kGroups), p.M, (n + kWindow) % kGroups, raw[n % kWindow], XL);
            if (of_taps) {
#pragma unroll
                for (int t = 0; t < 4; ++t) xa[set][gi][t] = __builtin_bit_cast(half8_t, mine[t]);
                continue;
            }
            arrange_operands<BITS>(mine, xa[set][gi]);
            float4_t sx = zero4;
#pragma unroll
            for (int t = 0; t < 4; ++t) sx = mfma(xa[set][gi][t], gain_operand<BITS>(t), sx);
            if (c == 0) *reinterpret_cast<float4_t *>(xsum + gi * 16 + q * 4) = sx * 0x1p-24f;
            if (gi == kGroups - 1) {
                __builtin_amdgcn_wave_barrier();
                const float4_t four = *reinterpret_cast<const float4_t *>(xsum + (q & (kGroups - 1)) * 16 + (c & 12));   // (as it was stored: the compiler must not take these for unrelated)
                xs[set] = c & 2 ? (c & 1 ? four.w : four.z) : (c & 1 ? four.y : four.x);
                __builtin_amdgcn_wave_barrier();
            }
        }
    }

    // ---- blocks for A^T: as many rows of it as activations a group, by the same way
    if (of_taps) {
        const int tap_tiles = (p.r + 15) >> 4;
        const __amdgpu_buffer_rsrc_t abuf = buffer_of(p.At, (long)p.r * p.K * 2);
        const int end = min((run + 1) * p.taps, tap_tiles);
        for (int tile = run * p.taps; tile < end; ++tile) {
            uint4_t raw[kGroups][4];
#pragma unroll
            for (int gi = 0; gi < kGroups; ++gi) request(abuf, 16 * tile, p.r, gi, raw[gi], 4);
            float4_t acc[S];
#pragma unroll
            for (int set = 0; set < S; ++set) acc[set] = zero4;
#pragma unroll
            for (int gi = 0; gi < kGroups; ++gi) {
                uint4_t mine[4];
                turn(raw[gi], 4, mine);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int set = 0; set < S; ++set) acc[set] = mfma(xa[set][gi][t], __builtin_bit_cast(half8_t, mine[t]), acc[set]);
            }
            asm volatile("" ::: "memory");              // (the same LDS under another type: the compiler keeps the order)
#pragma unroll
            for (int set = 0; set < S; ++set) sums[set * 64 + lane] = acc[set];
            block_barrier();
            if (wave < S) p.tpart[((size_t)(segment * S + wave) * tap_tiles + tile) * 64 + lane] = join_waves(wave);
            block_barrier();
        }
        return;
    }

    // ---- rows
    const int tiles = (p.N + 15) >> 4;
    const uint32_t smask[2] = {(valid > 0 ? 0xFFFFu : 0u) | (valid > 1 ? 0xFFFF0000u : 0u), (valid > 2 ? 0xFFFFu : 0u) | (valid > 3 ? 0xFFFF0000u : 0u)};
    while (ahead < kRing && i_unit < units) issue_next();
    for (int first = 0; first < units; first += Shape::kRoundUnits) {
        const int nu = min(Shape::kRoundUnits, units - first);
        for (int ui = 0; ui < nu; ++ui) {
            wait_unit();
            const unsigned char *const unit = ring + u_slot * kUnitBytes;
            uint4_t w[kUnitTiles][kGroups], s4[kUnitTiles];
            half_t sq[kUnitTiles], zq[kUnitTiles];
            int odd[kUnitTiles];
#pragma unroll
            for (int tt = 0; tt < kUnitTiles; ++tt) {
                const int row = 16 * tt + c;
                odd[tt] = ((row0 + (first + ui) * kUnitRows + row) * p.G + first_group) & 1;   // the row's first half may be the upper one of its dword
#pragma unroll
                for (int gi = 0; gi < kGroups; ++gi) w[tt][gi] = *reinterpret_cast<const uint4_t *>(unit + row * (64 * kGroups) + (((4 * gi + q) ^ key(row)) << 4));
                const unsigned char *const at = unit + 4096 + row * (4 * kGroups);
                if constexpr (kGroups == 4) s4[tt] = *reinterpret_cast<const uint4_t *>(at);
                else { const uint2_t two = *reinterpret_cast<const uint2_t *>(at); s4[tt] = uint4_t{two.x, two.y, 0, 0}; }
                const int half = (odd[tt] + (q & (kGroups - 1))) * 2;
                sq[tt] = *reinterpret_cast<const half_t *>(at + half);
                zq[tt] = *reinterpret_cast<const half_t *>(at + 256 + half);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // in registers: the slot may be filled again
            u_slot = u_slot + 1 == kRing ? 0 : u_slot + 1;
            --ahead;
            issue_next();
#pragma unroll
            for (int tt = 0; tt < kUnitTiles; ++tt) {
                const uint32_t s01 = __builtin_amdgcn_alignbit(s4[tt].y, s4[tt].x, 16 * odd[tt]) & smask[0], s23 = __builtin_amdgcn_alignbit(s4[tt].z, s4[tt].y, 16 * odd[tt]) & smask[1];
                // the zero points of all groups are one more product: sums of activations [token][group] times -s z [group][row]
                const float minus_sz = q < valid && q < kGroups ? -(float)sq[tt] * (float)zq[tt] : 0.0f;
                float4_t acc[S];
#pragma unroll
                for (int set = 0; set < S; ++set) acc[set] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[set], minus_sz, zero4, 0, 0, 0);
#pragma unroll
                for (int gi = 0; gi < kGroups; ++gi) {
                    half8_t b[4];
                    code_operands<BITS>(w[tt][gi], b);
                    const half2_t sh = h2_of(gi < 2 ? s01 : s23);
                    const float s = (float)(gi & 1 ? sh.y : sh.x);
#pragma unroll
                    for (int set = 0; set < S; ++set) {
                        float4_t D = zero4;
#pragma unroll
                        for (int t = 0; t < 4; ++t) D = mfma(xa[set][gi][t], b[t], D);
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[set][v] = fmaf(s, D[v], acc[set][v]);
                    }
                }
#pragma unroll
                for (int set = 0; set < S; ++set) sums[((ui * kUnitTiles + tt) * S + set) * 64 + lane] = acc[set] * 0x1p24f;
            }
        }
        block_barrier();
        const int tile = (row0 >> 4) + first * kUnitTiles + wave / S, set = wave % S;
        if (wave < nu * kUnitTiles * S && tile < tiles)      // wave-uniform
            p.part[((size_t)(segment * S + set) * tiles + tile) * 64 + lane] = join_waves(wave);
        block_barrier();                                // (the sums may be written again)
    }
}

// ------------------------------------------------------------------ the segments' sums

struct JoinParams {
    const float4_t *part;
    const float4_t *tpart;
    const uint16_t *Bt;         // [N][r]
    uint16_t *y;                // [M][N]
    const uint16_t *mix_with;   // [M][N]
    uint16_t *mix_out;          // null: none
    int M, N, r, segments, sets;
};
struct JoinGroup {
    JoinParams layer[kMaxSmallGroup];
    int start[kMaxSmallGroup];
};

// A block: eight tiles of 16 rows, one a wave, of one set of tokens.
__global__ __launch_bounds__(64 * kMainWaves) void fbq_few_join_kernel(const JoinGroup g)
{
    __shared__ __attribute__((aligned(16))) unsigned char tap[kMaxRank / 32 * 2048];   // t as operands: per 32 taps 1 KB of high halves, 1 KB of low ones
    int layer = 0;
#pragma unroll
    for (int i = 1; i < kMaxSmallGroup; ++i) layer = (int)blockIdx.x >= g.start[i] ? i : layer;
    const auto p = g.layer[layer];
    const int index = blockIdx.x - g.start[layer], set = index % p.sets;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, q = lane >> 4;
    const int tiles = (p.N + 15) >> 4, tile = index / p.sets * kMainWaves + wave, my_row = tile * 16 + c;
    const int tap_tiles = (p.r + 15) >> 4, tap_steps = (p.r + 31) >> 5;
    const float4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int kNowhere = 0x40000000;
    const __amdgpu_buffer_rsrc_t bbuf = buffer_of(p.Bt, (long)p.N * p.r * 2);
    auto taps = [&](int js) __attribute__((always_inline)) {
        const int j = js * 32 + q * 8;
        return __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(bbuf, j < p.r && my_row < p.N ? (my_row * p.r + j) * 2 : kNowhere, 0, 0));
    };
    constexpr int kHeld = 4;
    half8_t bf[kHeld];
#pragma unroll
    for (int k = 0; k < kHeld; ++k) bf[k] = taps(k);
    // segments of one tile, `step` accumulators apart, eight asked for at once
    auto add_up = [&](const float4_t *from, size_t step) __attribute__((always_inline)) {
        float4_t sum = zero4;
        for (int s0 = 0; s0 < p.segments; s0 += 8) {
            float4_t v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = from[(size_t)min(s0 + i, p.segments - 1) * step];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (s0 + i < p.segments) sum += v[i];
        }
        return sum;
    };
    for (int jt = wave; jt < 2 * tap_steps; jt += kMainWaves) {
        const float4_t t = jt < tap_tiles ? add_up(p.tpart + ((size_t)set * tap_tiles + jt) * 64 + lane, (size_t)p.sets * tap_tiles * 64) : zero4;
        // lane (c, q) holds tap 16 jt + c of tokens 4 q + v: half (tap % 8) of lane (token, tap / 8 % 4) of its 32 taps
        half_t *const to = reinterpret_cast<half_t *>(tap + (jt >> 1) * 2048) + ((2 * (jt & 1) + (c >> 3)) * 16 + 4 * q) * 8 + (c & 7);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const half_t hi = (half_t)t[v];
            to[v * 8] = hi;
            to[512 + v * 8] = (half_t)(t[v] - (float)hi);
        }
    }
    float4_t mine = add_up(p.part + ((size_t)set * tiles + min(tile, tiles - 1)) * 64 + lane, (size_t)p.sets * tiles * 64);
    __syncthreads();
    auto fold = [&](int js, half8_t b) __attribute__((always_inline)) {
        const float4_t d = mfma(*reinterpret_cast<const half8_t *>(tap + js * 2048 + lane * 16), b, zero4);
        mine += mfma(*reinterpret_cast<const half8_t *>(tap + js * 2048 + 1024 + lane * 16), b, d);
    };
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
        if (k < tap_steps) fold(k, bf[k]);
    for (int k = kHeld; k < tap_steps; ++k) fold(k, taps(k));
    if (my_row >= p.N) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int m = 16 * set + 4 * q + v;
        if (m >= p.M) continue;
        const half_t y = (half_t)mine[v];
        p.y[(size_t)m * p.N + my_row] = __builtin_bit_cast(uint16_t, y);
        if (p.mix_out) {
            const float with = (float)__builtin_bit_cast(half_t, p.mix_with[(size_t)m * p.N + my_row]);
            p.mix_out[(size_t)m * p.N + my_row] = __builtin_bit_cast(uint16_t, (half_t)((float)y - ((float)y - with) * 0.5f));
        }
    }
}

// ------------------------------------------------------------------ launches

template <int BITS, int S, int XL>
static void launch_instance(const SplitGroup &g, int blocks, hipStream_t stream)
{
    hipLaunchKernelGGL((fbq_few_split_kernel<BITS, S, XL>), dim3(blocks), dim3(64 * kMainWaves), 0, stream, g);
}
template <int BITS>
static void launch_bits(const SplitGroup &g, int sets, bool half, int blocks, hipStream_t stream)
{
    if (sets == 1 && half) launch_instance<BITS, 1, 2>(g, blocks, stream);
    else if (sets == 1) launch_instance<BITS, 1, 4>(g, blocks, stream);
    else if (sets == 2) launch_instance<BITS, 2, 4>(g, blocks, stream);
    else if (sets == 3) launch_instance<BITS, 3, 4>(g, blocks, stream);
    else launch_instance<BITS, 4, 4>(g, blocks, stream);
}

hipError_t launch_few_split(const LinearArgs *layers, int n_layers, hipStream_t stream)
{
    if (n_layers < 1 || n_layers > kMaxSmallGroup) return hipErrorInvalidValue;
    const int sets = ceil_div(layers[0].M, kTokens), cus = cu_count();
    double work[kMaxSmallGroup], total = 0.0;            // in tiles of rows of all K
    for (int i = 0; i < n_layers; ++i) {
        if (ceil_div(layers[i].M, kTokens) != sets || sets > kMaxSmallGroup) return hipErrorInvalidValue;
        total += work[i] = ceil_div(layers[i].N, 16) + kSplitTapCost * ceil_div(layers[i].r, 16);
    }
    SplitGroup g;
    JoinGroup j;
    int blocks = 0, joins = 0;
    for (int i = 0; i < n_layers; ++i) {
        const LinearArgs &a = layers[i];
        const FewSplit f = a.split;
        SplitParams &p = g.layer[i];
        p.qw = a.qw; p.scales = a.scales; p.zeros = a.zeros; p.At = a.At; p.x = a.x;
        p.part = (float4_t *)((char *)a.workspace + handover_reserve(a.K, a.r));
        p.tpart = p.part + (size_t)f.segments * sets * ceil_div(a.N, 16) * 64;
        p.M = a.M; p.N = a.N; p.K = a.K; p.r = a.r;
        p.row_words = (int)row_words(a.K, a.bits);
        p.G = a.K / kGroup;
        p.segments = f.segments; p.share = f.share;
        const FewSplitRuns runs = few_split_runs(sets, a.N, a.r, std::max(1, (int)(cus * (work[i] / total)) / f.segments));
        p.tap_blocks = runs.tap_blocks; p.taps = runs.taps;
        p.row_blocks = runs.row_blocks; p.units = runs.units;
        g.start[i] = blocks;
        blocks += f.segments * (p.tap_blocks + p.row_blocks);
        JoinParams &o = j.layer[i];
        o.part = p.part; o.tpart = p.tpart; o.Bt = a.Bt; o.y = a.y; o.mix_with = a.mix_with; o.mix_out = a.mix_out;
        o.M = a.M; o.N = a.N; o.r = a.r; o.segments = f.segments; o.sets = sets;
        j.start[i] = joins;
        joins += ceil_div(ceil_div(a.N, 16), kMainWaves) * sets;
    }
    for (int i = n_layers; i < kMaxSmallGroup; ++i) {
        g.layer[i] = g.layer[0]; j.layer[i] = j.layer[0];   // never indexed
        g.start[i] = j.start[i] = 0x7FFFFFFF;
    }
    int most = 0;
    for (int i = 0; i < n_layers; ++i) most = std::max(most, layers[i].M);
    if (layers[0].bits == 4) launch_bits<4>(g, sets, most <= 8, blocks, stream);
    else launch_bits<3>(g, sets, most <= 8, blocks, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fbq_few_join_kernel, dim3(joins), dim3(64 * kMainWaves), 0, stream, j);
    return hipGetLastError();
}

}  // namespace fbq
