// Internal declarations shared by the library's own translation units (not part of the ABI).
#ifndef FBQ_INTERNAL_H
#define FBQ_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "fbq.h"

namespace fbq {

constexpr int kGroup = 128;          // codes per (scale, zero) pair
constexpr int kLaneCodes = 32;       // codes one lane takes from one wave-wide load
constexpr int kChunk = 64 * kLaneCodes;   // codes one wave-wide load covers (2048)
constexpr int kMaxRank = 256;
constexpr int kMaxK = 16 * kChunk;      // 32768: the decode kernel keeps a wave's activations in registers
constexpr int kDecodeMaxM = 16;
constexpr int kChunkedMaxM = 64;     // up to here the few-token kernel, 16 tokens at a time, can beat the prefill GEMM
constexpr int kPerTokenMaxM = 2;     // up to here the GEMV streams the weights once per token; above, the matrix-core tile wins
constexpr int kMaxTSlices = 4;       // K slices of the decode down-projection: kMaxK / (4 passes * 2048)
constexpr int kMaxGroup = 8;         // layers one grouped decode launch can serve
constexpr int kMaxSmallGroup = 4;    // ... for 4..16 tokens

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// How often a consumer polls for the down-projection's words before it computes them itself.  The value
// in force is process-wide and only the test hook fbq_test_set_spin_limit changes it: a negative value
// makes every consumer take the fall-back path at once (every kernel still runs to its end), so the
// path that a healthy run never takes can be checked against the oracle.
constexpr int kDefaultSpinLimit = 1 << 15;   // polls of about 0.3 us each
int spin_limit();

// Words per packed row.
inline size_t row_words(int K, int bits) { return (size_t)K * bits / 32; }

// Segments of K, 0: not split, and the groups each of a block's eight waves takes of one (fbq_few_split.hip).
struct FewSplit { int segments, share; };

struct LinearArgs {
    const uint32_t *qw;
    const uint16_t *scales;
    const uint16_t *zeros;
    const uint16_t *At;
    const uint16_t *Bt;
    const uint16_t *x;
    uint16_t *y;
    void *workspace;  // see decode_workspace_bytes / small_m_workspace_bytes / prefill_workspace_bytes
    size_t workspace_need;   // fbq_workspace_bytes of the call (above 64 tokens a search, so looked up once) ...
    size_t unsplit_need;     // ... and of the same call with K unsplit
    int M, N, K, r, bits;
    const uint16_t *mix_with;   // [M][N] and ...
    uint16_t *mix_out;          // ... null, or [M][N] that the decode launchers write y averaged with mix_with to (see launch_mix)
    FewSplit split;             // 3 to 64 tokens: how K is split over blocks (see split_of), where the workspace has room for it
};

// 3 to 16 tokens: which of the two kernels serves a layer of N rows (for sets of 16 tokens side by side: rows times sets).  Of
// the layer alone, so that a layer of a grouped call gets exactly what a call of its own gives it.  The streaming kernel
// keeps a wave's activations for all tiles of its block and has the next tiles' codes under way while it works on one; it wins where a
// CU has several tiles.  The other one is a single burst of requests, and takes what is small.  us, burst / stream, 16 tokens or as
// stated, r = 64 or as stated: 28672 x 8192 INT4 r = 128 46.5 / 31.1; two of 11008 x 4096 INT3 at 8 tokens 18.7 / 15.5, INT4 18.6 / 16.6; one alone
// INT3 11.0 / 10.0, but INT4 10.0 / 11.1 and 10240 x 4096 INT4 9.9 / 10.7, which the pairs decide; 14336 x 4096 r = 128 at 8 15.4 / 14.0; 50257 x 1024 r = 16 at
// 8 31.6 / 19.5.  On the burst's side of the line 8192 x 4096 INT4 9.3 / 10.3, 4096 x 4096 7.8 / 9.2, 4096 x 11008 INT3 at 8 15.7 / 16.1, INT4 16.0 / 17.7,
// {4096, 1024, 1024} x 4096 at 8 8.6 / 9.4; the line is on the safe side where it leaves the burst 8192 x 5120 (15.8 / 13.7), 8192 x 8192 (16.7 / 14.9, INT3 19.1 / 14.7)
// and 12288 x 2048 (11.8 / 9.9).
inline bool few_stream(long rows, int K) { return rows >= 10240 && rows * K >= 40000000L; }

// Launchers (validated arguments only).  Each returns the hipError_t of its launches.
hipError_t launch_gemv_decode(const LinearArgs *layers, int n_layers, hipStream_t stream);
bool decode_group_compatible(const LinearArgs &a, const LinearArgs &b);
hipError_t launch_gemv_small_m(const LinearArgs *layers, int n_layers, hipStream_t stream);
bool small_m_group_compatible(const LinearArgs &a, const LinearArgs &b);
bool burst_joins_stream(const LinearArgs *layers, int n_layers, const bool *burst);
hipError_t launch_few_stream(const LinearArgs *layers, int n_layers, const bool *burst, hipStream_t stream);   // (by way of launch_gemv_small_m, which says which layers are too small)
hipError_t launch_few_split(const LinearArgs *layers, int n_layers, hipStream_t stream);
hipError_t launch_prepass_prefill(const LinearArgs &a, hipStream_t stream);
hipError_t launch_gemm_prefill(const LinearArgs &a, hipStream_t stream);
hipError_t launch_unpack(const fbq_desc &d, const uint32_t *qw, uint8_t *codes, hipStream_t stream);
hipError_t launch_reconstruct(const fbq_desc &d, const uint32_t *qw, const uint16_t *scales, const uint16_t *zeros,
                              const uint16_t *At, const uint16_t *Bt, float *W_hat, hipStream_t stream);
// D16 (optional): Delta_F times `gain` as fp16, [N][K].
hipError_t launch_quantize(const fbq_desc &d, const uint16_t *W, const uint16_t *At, const uint16_t *Bt, uint32_t *qw,
                           uint16_t *scales, uint16_t *zeros, hipStream_t stream, uint16_t *D16 = nullptr,
                           float gain = 0.0f);

// a.mix_out = a.y averaged with a.mix_with, behind the launch that writes y
hipError_t launch_mix(const LinearArgs &a, hipStream_t stream);
hipError_t launch_silu_mul(const void *gate, const void *up, void *out, size_t count, hipStream_t stream);

hipError_t launch_read_stream(const void *buf, size_t bytes, hipStream_t stream);
// the sub-branch as two launches of its own on top of a y the main path has written (t: [M][r] fp16 scratch)
hipError_t launch_unfused_branch(const LinearArgs &a, uint16_t *t, hipStream_t stream);

// Arguments of one reconstruction iteration (validated): see fbq_train_step.
struct TrainArgs {
    fbq_desc d;
    const uint16_t *W;
    const uint16_t *H16;
    float h_scale, lr;
    float *At32, *Bt32;
    uint32_t *qw;
    uint16_t *scales, *zeros, *At16, *Bt16;
    float *gAt, *gBt, *loss;
    void *workspace;
};
hipError_t launch_gram(int K, int T, const uint16_t *X, float h_scale, uint16_t *H16, void *workspace, hipStream_t stream);
hipError_t launch_train_step(const TrainArgs &a, hipStream_t stream);
size_t train_workspace_bytes(int N, int K, int r, int T);

// Shared by the entry points (fbq_api.cpp, fbq_static.hip): argument validation that fills the launch
// record without launching, the dispatch on the token count, and the mapping of a HIP error to a status.
fbq_status check_layer(const fbq_desc *d, int M, const void *x, const void *qweight, const void *scales, const void *zeros,
                       const void *At, const void *Bt, void *y, void *workspace, size_t workspace_bytes, LinearArgs *a);
hipError_t launch_one(const LinearArgs &a, hipStream_t s);
fbq_status hip_status(hipError_t e);

// Largest hand-over scratch any call of up to kDecodeMaxM tokens needs (r = kMaxRank): 16 K slices and their
// sums, 16 token rows each, one 8-byte word per value.
constexpr size_t kStaticScratchBytes = (size_t)(16 + 1) * 16 * kMaxRank * 8;

constexpr int kPrefillColumns = 256;   // columns of a block tile of the prefill GEMM

// How a layer is cut into blocks: tiles of 32 tm rows (tm = 8, 6: four waves; 4, 3, 2: eight waves in two K groups), K
// split over ksplit blocks.  One block per CU at a time, 8 XCDs of 32 CUs assumed (the workspace is sized without a device):
// a launch takes rounds x (steps x step time + fixed part), plus the summing launch and its traffic where K is split over
// blocks.  Column blocks are dealt to the XCDs whole, eight at a time, the rest block by block: the fullest XCD counts.
// The constants (us) are fitted to 2700 measurements: both bit widths, 65 to 2048 tokens, eleven layers from
// 1000 x 1408 to 28672 x 8192 and 8192 x 28672, every tile height with every split; over them the choice is 0.6 % slower
// than the best one on average and 14 % at most.  A CU runs faster while others are idle (the clock follows the load): a
// step of a round that fills the fraction f of the CUs takes 0.48 (1 - f) less.  Examples, the choice and the two that
// bracket it, us: 4096 -> 11008 at 1024 tokens 102 (256 rows), 109 (96), 118 (128); 8192 -> 28672 at 384 tokens 172 (192
// rows), 190 (96), 202 (128); 28672 -> 8192 at 256 tokens 137 (128 rows, K split in 4), 144 (in 3), 144 (in 8).
//
// Columns left over by full rounds: where the last round would leave many CUs idle, the column blocks that fill whole rounds are
// one launch and the others a second one in tiles of their own height (4 us for the launch).  8192 -> 28672 at 2048 tokens,
// INT4, r = 128, us: four rounds of 256-row tiles, the last half empty, 896; three rounds, and the rest as 256 tiles of 128 rows, 844.
//
// Low tiles of one K group: two blocks of 128 or 96 rows, three of 64, share a CU, and one works while another starts or ends.  That
// is worth most where a block has few steps and a CU several blocks; what it lacks is the second group's help with the
// steps.  Estimated the same way, from what a set of one, two or three blocks on a CU takes per step and at its start and end
// (fitted to 400 layers without a sub-branch, 128 to 6144 activations, 256 to 150000 rows, 65 to 4096 tokens).  Without a
// sub-branch they are taken over that range of activations up to 5 % above the other estimate; with one, up to 2048 where theirs is
// 5 % below: a block's end with a sub-branch, which lower tiles have more of, undoes the gain (11008 x 4096 at 1024 tokens, r = 64:
// 102 us in 256 rows, 105 in 96 like this).  Against the estimate above alone: 160 drawn layers of up to 2176 activations with a
// sub-branch 7 % faster on average, 1 % slower at worst; 800 without one, 7 % on average.  Examples, us
// without / with: 14402 x 128 at 922 tokens, INT4, no sub-branch 30.1 / 21; 26880 x 256 at 577, r = 64, 37.5 / 28.8;
// 50257 x 1024 at 700, r = 16, 130 / 105; 9000 x 1536 at 2000, r = 64, 94 / 81; 18796 x 2304 at 849, INT3, no sub-branch 102 / 92.
constexpr int kSingleGroups = 16, kSingleGroupsNoBranch = 48;
struct PrefillCut { int tm, ksplit, columns, tail_tm; bool single; };   // columns: column blocks of the first launch; tail_tm: tile height of the second, 0: none; single: one K group though tm < 6

inline PrefillCut prefill_cut(int M, int N, int K, int r)
{
    static constexpr struct { int tm, kg; double step, fixed; } kTiles[] = {
        {8, 1, 1.614, 16.2}, {6, 1, 1.241, 11.6}, {4, 2, 1.731, 9.4}, {3, 2, 1.402, 7.6}, {2, 2, 1.144, 6.0}};
    const int G = K / kGroup, columns = ceil_div(N, kPrefillColumns);
    auto launch_us = [&](int tile, int cols, int split) {
        const auto &t = kTiles[tile];
        const int rows = ceil_div(M, 32 * t.tm);
        const double per_xcd = (double)(cols / 8) * rows * split + std::ceil((cols % 8) * (double)rows * split / 8.0);
        const double rounds = std::ceil(per_xcd / 32.0), filled = (double)cols * rows * split / (256.0 * rounds);
        const int steps = 2 * ceil_div(G, split * t.kg);
        const double us = rounds * (steps * t.step * (1.0 - 0.48 * (1.0 - filled)) + t.fixed) +
                          (split > 1 ? 5.6 + 0.886e-6 * M * (double)N * (split + 0.5) : 0.0);
        return us * (1.0 - 0.01 * t.tm);                // (taller tiles draw less power per product: measured, they win where this estimate is a tie)
    };
    PrefillCut best{0, 1, columns, 0, false};
    double best_us = 1e300;
    for (int i = 0; i < 5; ++i) {
        const double tiles = (double)columns * ceil_div(M, 32 * kTiles[i].tm);
        for (int split = 1; split <= 8; ++split) {
            if (split > 1 && (tiles * split > 600 || G / (split * kTiles[i].kg) < 2)) break;
            const double us = launch_us(i, columns, split);
            if (us < best_us) { best_us = us; best = {kTiles[i].tm, split, columns, 0, false}; }
        }
    }
    for (int i = 0; i < 5; ++i) {
        const int rows = ceil_div(M, 32 * kTiles[i].tm);
        const int whole = (int)((double)columns * rows / 256.0) * 256 / rows / 8 * 8;   // column blocks, in eights, that fill whole rounds
        if (whole < 8 || whole >= columns) continue;
        for (int j = 0; j < 5; ++j) {
            const double us = launch_us(i, whole, 1) + launch_us(j, columns - whole, 1) + 4.0;
            if (us < 0.98 * best_us) { best_us = us; best = {kTiles[i].tm, 1, whole, kTiles[j].tm, false}; }
        }
    }
    static constexpr struct { int tm, together; double step[3], fixed[3], idle; } kSingle[] = {
        {4, 2, {0.93, 1.65, 0}, {6.8, 8.3, 0}, 0.29}, {3, 2, {0.79, 1.32, 0}, {5.7, 6.5, 0}, 0.27}, {2, 3, {0.71, 1.07, 1.68}, {4.5, 6.3, 5.5}, 0.26}};
    best_us *= r > 0 ? 0.95 : 1.05;
    for (int i = 0; i < 3 && G <= (r > 0 ? kSingleGroups : kSingleGroupsNoBranch); ++i) {
        const auto &t = kSingle[i];
        const int rows = ceil_div(M, 32 * t.tm);
        const double per_cu = std::ceil(((double)(columns / 8) * rows + std::ceil((columns % 8) * (double)rows / 8.0)) / 32.0);
        auto set_us = [&](int blocks) { return blocks ? 2 * G * t.step[blocks - 1] + t.fixed[blocks - 1] : 0.0; };
        const double sets = std::floor(per_cu / t.together);
        const double us = (sets * set_us(t.together) + set_us((int)(per_cu - sets * t.together))) *
                          (1.0 - t.idle * (1.0 - (double)columns * rows / (256.0 * per_cu))) * (1.0 - 0.01 * t.tm);
        if (us < best_us) { best_us = us; best = {t.tm, 1, columns, 0, true}; }
    }
    return best;
}

// K slices of the prefill down-projection, one block per slice and 32-token tile: eight for a thousand tokens, more
// for fewer tokens so that the pass has about one block per compute unit (256 assumed: the workspace is sized
// without a device), never narrower than 256 activations.  Slices are whole quantization groups: the kernel walks
// them in chunks of 128.
inline int down_slice_len(int M, int K)
{
    const int want = std::min(32, std::max(8, ceil_div(256, ceil_div(M, 32))));
    return std::max(256, ceil_div(ceil_div(K, want), kGroup) * kGroup);
}
inline int down_slices(int M, int K) { return ceil_div(K, down_slice_len(M, K)); }

// How many of the slices, in eights, are dealt out to the XCDs whole, so that a slice of A^T comes into one L2 and not into each that has
// one of its token tiles (256 tokens of 28672 x 128, INT3: the pass reads 30 MB instead of 81 and takes 17.4 us instead of 19.6).  It pays
// where A^T is large and eight tiles or more read it and where all blocks fit the GPU at once; the fused kernel finds the re-ordered x in other
// L2s then, which costs the more of the call the narrower and shorter the layer is.  The call, us, before /
// with it: 256 tokens of 20480 -> 1024, r = 256, 66.2 / 61.6, of 28672 -> 5120, r = 128, 115.3 / 112.5, of 13824 -> 1024, r = 128, 42.5 / 41.9, of
// 28672 -> 512, r = 64, 54.4 / 53.3; on the other side of a line 256 tokens of 8192 -> 1024, r = 200, 44.6 / 46.7, of 6144 -> 512, r = 256, 3 % slower, of
// 16384 -> 512, r = 96, 4 %, of 4096 -> 3456, r = 128, 36.3 / 37.1; 160 of 8192 -> 1024, r = 256, 41.6 / 43.2; 1092, 280 blocks, of 13952 -> 3456, r = 128, 151 / 156.
inline int down_slices_by_xcd(int M, int N, int K, int r)
{
    const int tiles = ceil_div(M, 32), slices = down_slices(M, K);
    const bool pays = r * K >= 1500000 && ((long)K * std::min(N, 2304) >= 14000000 || r * K >= 2600000);
    return pays && tiles >= 8 && tiles * slices <= 256 ? slices & ~7 : 0;
}

// In front of what the prefill path and the K split keep in a workspace: room for the hand-over words of the decode paths, which those
// never touch.  A workspace that serves calls of every token count then only ever holds words with a
// launch's tag, or the zeros it started with, where the decode kernels look for tags - never activations or partial
// sums that happen to look like one.
size_t handover_reserve(int K, int r);

size_t decode_workspace_bytes(int M, int K, int r);
size_t small_m_workspace_bytes(int K, int r);
size_t prefill_workspace_bytes(int M, int N, int K, int r);

}  // namespace fbq

#endif
