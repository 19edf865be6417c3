// C ABI of the library: argument validation, host-side packing and kernel dispatch.
// Every operation is defined in include/fbq.h; nothing here computes on the CPU except fbq_pack
// (a one-off layout conversion that is off the hot path by definition).
#include <string.h>

#include <atomic>

#include "fbq_internal.h"
#include "fbq_split_plan.h"

using namespace fbq;

extern "C" const char *fbq_status_string(fbq_status s)
{
    switch (s) {
    case FBQ_OK: return "ok";
    case FBQ_ERR_NULL: return "null pointer";
    case FBQ_ERR_SHAPE: return "bad shape or value";
    case FBQ_ERR_UNSUPPORTED: return "unsupported configuration";
    case FBQ_ERR_ALIGN: return "device pointer not 16-byte aligned";
    case FBQ_ERR_WORKSPACE: return "workspace too small";
    case FBQ_ERR_HIP: return "HIP launch error";
    }
    return "unknown status";
}

extern "C" fbq_status fbq_check_desc(const fbq_desc *d)
{
    if (!d) return FBQ_ERR_NULL;
    if (d->bits != 3 && d->bits != 4) return FBQ_ERR_UNSUPPORTED;
    if (d->group != kGroup) return FBQ_ERR_UNSUPPORTED;
    if (d->N < 1 || d->K < 1 || d->r < 0) return FBQ_ERR_SHAPE;
    if (d->K % d->group || d->K % 32 || d->r % 8) return FBQ_ERR_SHAPE;
    if (d->r > kMaxRank || d->K > kMaxK) return FBQ_ERR_UNSUPPORTED;
    // the kernels address a layer's buffers with 32-bit byte offsets and keep 2^30 as "nowhere"
    if ((size_t)d->N * row_words(d->K, d->bits) * sizeof(uint32_t) >= ((size_t)1 << 30)) return FBQ_ERR_UNSUPPORTED;
    if ((size_t)d->N * d->r * sizeof(uint16_t) >= ((size_t)1 << 30)) return FBQ_ERR_UNSUPPORTED;   // (B^T likewise)
    return FBQ_OK;
}

extern "C" size_t fbq_packed_bytes(const fbq_desc *d)
{
    if (fbq_check_desc(d) != FBQ_OK) return 0;
    return (size_t)d->N * row_words(d->K, d->bits) * sizeof(uint32_t);
}

// 17..64 tokens: whether the few-token kernels, the sets of 16 tokens side by side in one launch, take the call, or the prefill
// GEMM.  The sets stream the packed words once per set and multiply the codes exactly (relative error of y 2.2e-4); the GEMM reads the words
// once and rounds the weights to fp16 (2.9e-4).  The first line is the cost of both, in us, that was fitted to ten shapes when there was neither
// the streaming kernel nor the GEMM of today: sets 2 + sets x (2.2 + 0.165 MC), in passes of 4096 along K, GEMM 30 + 0.135 MC + 1.5 K / 1024 (MC = millions
// of codes, K counted in whole passes for the sets).  As an estimate it is obsolete; it stays as the line up to which a call has the smaller error: who had it
// keeps it.  What that costs by now, sets / GEMM, us: nothing for 4096 x 4096 (8.8 / 28 at 32 tokens, 13.7 / 30 at 64), 4096 -> 11008 (20 / 31 at 48,
// 24 / 32 at 64), 8192 -> 8192 at 48 (27 / 37), 13824 -> 5120 at 48 (37.5 / 42.0, INT3 36.0 / 43.7) and 28672 -> 8192 at 32 (61 / 69); 28672 -> 5120 at 48 62.6 / 60.6.
//
// Beyond that line the sets are faster too where they add up to a launch of the streaming kernel and K is 3072 to 8192 (longer rows:
// a wave's activations come again and again; shorter ones: too little work per row): two sets at any N, four up to 70 million codes.
// Sets / GEMM, us, r = 64 or as stated.  Two, at 32 tokens: 8192 -> 28672, r = 128, 49.0 / 65.5; 3072 -> 40000 32.7 / 40.7; 4096 -> 131072 99 / 116; but
// 2048 -> 60000 40.2 / 35.7, 1024 -> 40000 29.6 / 23.9, 8320 -> 20001, r = 0, 55.4 / 42.7.  Four, at 64: 4096 -> 17088 31.5 / 37.5, 3072 -> 22784 33.7 / 38.6,
// 8192 -> 8544, r = 128, 36.5 / 42.0; but 6144 -> 20000 49.3 / 47.2, 8192 -> 28672 87.9 / 70.9.  Three were left to the GEMM while their launches had more
// blocks than CUs; at 48 tokens they would now win over the same K: 3072 -> 22784 28.5 / 37.8, 5120 -> 11008, r = 128, 27.6 / 36.8, 5120 -> 13824, r = 128, 32.6 / 38.1,
// 6144 -> 20000 40.2 / 45.2, 8192 -> 28672 68.0 / 68.4 (INT3 61.1 / 69.0).
static bool takes_sets(int M, int N, int K)
{
    const int sets = (M + kDecodeMaxM - 1) / kDecodeMaxM;
    const double k_passes = 4096.0 * ((K + 4095) / 4096);
    const double cost_sets = 2.0 + sets * (2.2 + 0.165e-6 * N * k_passes);
    const double cost_gemm = 30.0 + 0.135e-6 * N * (double)K + 1.5 * K / 1024.0;
    if (cost_sets <= cost_gemm) return true;
    return K >= 3072 && K <= 8192 && few_stream((long)sets * N, K) && (sets == 2 || (sets == 4 && (long)N * K <= 70000000L));
}

namespace fbq {
size_t handover_reserve(int K, int r)
{
    return r > 0 ? (size_t)kMaxSmallGroup * small_m_workspace_bytes(K, r) : 0;
}
}  // namespace fbq

// How a call of 3 to 64 tokens has its K split over blocks (fbq_few_split.hip) instead of going where it would go otherwise; segments 0: not at all.  Times of the split
// over those of the other way, r = 64, INT3 and INT4.
// Up to 16 tokens, instead of streaming or bursts: above 16384 activations, from 2048 to 10239 rows: 28672 -> 2048 0.62 to 0.72, -> 8192 0.76 to 0.95; 17408 -> 2048 to 10000 0.82 to 1.03; but
// 16384 -> 2500 1.06 to 1.19, 14336 -> 6000 INT4 1.1.  (Wider layers stream; narrower ones share launches with them.)
// Instead of sets of 16, above 8192 activations and from 25 million codes on: three and four sets 0.65 to 1.0; two sets where they take four passes, above 12288: 13824 -> 2304 to 8192 0.77 to 0.97; below
// that from 4600 rows on: 8320 -> 4700 0.82 to 0.90, 10240 -> 5120 0.95 to 1.01, 11008 -> 8192 0.88; but 11008 -> 2304 1.16, -> 4096 1.04; with one or two tokens left over, which the sets take one by one, from 3400: 8320 to 12288
// -> 3500 0.80 to 0.86, -> 3001 0.88 to 1.03.
// Instead of the GEMM, from 2048 activations on, up to the rows whose partial sums, written and read once a segment, cost what is saved.  Two sets 44000 rows: 2048 -> 28000 0.82, 34000 0.94, 44000 0.98, 52000 1.08
// (long rows at any N: 20480 -> 52000 0.57); three sets 46000, less as the segments are less full: 2048 -> 44000 0.98, 52000 1.04; 2176 -> 24000 (full 17/32) 0.97, 28000 1.02, 34000 1.17; 4224 -> 28000 0.93, 44000 1.17;
// four sets 35000 likewise, 30000 where there is one segment: 2048 -> 28000 0.96, 34000 1.06; 2304 -> 20000 0.94, 28000 1.15; 3072 -> 28000 0.96, 34000 1.1; 4224 -> 24000 1.0, 34000 1.15; 8192 -> 34000 0.84, 64000 1.1.  And
// 1024 -> 28672 at 48 tokens 20.9 us against 21.7 split.
static FewSplit split_of(const fbq_desc *d, int M)
{
    const FewSplit none{0, 0};
    const int N = d->N, K = d->K, G = K / kGroup, sets = ceil_div(M, kDecodeMaxM);
    if (M <= kPerTokenMaxM || M > kChunkedMaxM) return none;
    const bool few = M <= kDecodeMaxM, instead_of_sets = !few && takes_sets(M, N, K);
    if (few ? K <= 16384 || N < 2048 || N >= 10240 : K < (instead_of_sets ? 8193 : 2048) || (instead_of_sets && (long)N * K < 25000000L)) return none;
    const FewSplit f = few_split(sets, N, K, d->r, d->bits);
    const double full = G / (8.0 * f.share * f.segments);       // of what the waves could hold, what there is of K
    if (few) return f;
    if (instead_of_sets) return sets > 2 || K > 12288 || N >= (M <= kDecodeMaxM + kPerTokenMaxM ? 3400 : 4600) ? f : none;
    if (sets == 2) return K > 8192 || N <= 44000 ? f : none;
    return N <= (sets == 3 ? 46000 : K == 2048 ? 30000 : 35000) * full ? f : none;
}

// What a call cannot do without.
static size_t least_workspace(const fbq_desc *d, int M)
{
    if (fbq_check_desc(d) != FBQ_OK || M < 1) return 0;
    if (M <= kPerTokenMaxM) return d->r == 0 ? 0 : decode_workspace_bytes(M, d->K, d->r);
    // up to 64 tokens go through the few-token kernel 16 at a time, all in one launch, every 16 tokens with hand-over
    // words of their own (one or two left over, where they go through the GEMV afterwards, have words that fit the first set);
    // nothing to hand over without a sub-branch
    if (M <= kDecodeMaxM) return small_m_workspace_bytes(d->K, d->r);
    if (M <= kChunkedMaxM && takes_sets(M, d->N, d->K))
        return (size_t)((M + kDecodeMaxM - 1) / kDecodeMaxM) * small_m_workspace_bytes(d->K, d->r);
    return handover_reserve(d->K, d->r) + prefill_workspace_bytes(M, d->N, d->K, d->r);      // holds the re-ordered activations even when r == 0
}

// The workspace of a split call: the hand-over words' room and the partial sums, or what it needs without the split.
static size_t split_workspace(const fbq_desc *d, int M, const FewSplit &f, size_t least)
{
    return std::max(least, handover_reserve(d->K, d->r) + few_split_bytes(f, ceil_div(M, kDecodeMaxM), d->N, d->r));
}

extern "C" size_t fbq_workspace_bytes(const fbq_desc *d, int M)
{
    const size_t least = least_workspace(d, M);
    if (fbq_check_desc(d) != FBQ_OK || M < 1) return 0;
    const FewSplit f = split_of(d, M);
    return f.segments ? split_workspace(d, M, f, least) : least;
}

// ------------------------------------------------------------------ host-side packing

// Bit c of code k within a packed row: word index and bit position (layout in fbq.h).
static inline void code_bit_slot(int bits, int k, int c, size_t *word, int *bit)
{
    if (bits == 4) {
        *word = (size_t)k >> 3;
        *bit = ((k & 7) << 2) + c;
        return;
    }
    const int unit = k >> 5, j = k & 31;
    if (j >= 30) {
        *word = (size_t)unit * 3 + c;
        *bit = j == 30 ? 15 : 31;
        return;
    }
    const int wd = j / 10, f = j - wd * 10;
    *word = (size_t)unit * 3 + wd;
    *bit = (f >= 5 ? 16 + 3 * (f - 5) : 3 * f) + c;
}

extern "C" fbq_status fbq_pack(const fbq_desc *d, const uint8_t *codes, const uint16_t *scales, const uint16_t *zeros,
                               const uint16_t *A, const uint16_t *B, uint32_t *qweight_out, uint16_t *scales_out,
                               uint16_t *zeros_out, uint16_t *At_out, uint16_t *Bt_out)
{
    fbq_status st = fbq_check_desc(d);
    if (st != FBQ_OK) return st;
    if (!codes || !scales || !zeros || !qweight_out || !scales_out || !zeros_out) return FBQ_ERR_NULL;
    if (d->r > 0 && (!A || !B || !At_out || !Bt_out)) return FBQ_ERR_NULL;

    const int N = d->N, K = d->K, r = d->r, bits = d->bits;
    const size_t rw = row_words(K, bits);
    const unsigned qmax = (1u << bits) - 1u;
    memset(qweight_out, 0, rw * (size_t)N * sizeof(uint32_t));
    for (int n = 0; n < N; ++n) {
        uint32_t *row = qweight_out + rw * (size_t)n;
        const uint8_t *crow = codes + (size_t)n * K;
        for (int k = 0; k < K; ++k) {
            const unsigned q = crow[k];
            if (q > qmax) return FBQ_ERR_SHAPE;
            for (int c = 0; c < bits; ++c) {
                size_t w;
                int bit;
                code_bit_slot(bits, k, c, &w, &bit);
                row[w] |= ((q >> c) & 1u) << bit;
            }
        }
    }
    const size_t ng = (size_t)N * (K / d->group);
    memcpy(scales_out, scales, ng * sizeof(uint16_t));
    memcpy(zeros_out, zeros, ng * sizeof(uint16_t));
    if (r > 0) {
        for (int k = 0; k < K; ++k)
            for (int j = 0; j < r; ++j) At_out[(size_t)j * K + k] = A[(size_t)k * r + j];
        for (int n = 0; n < N; ++n)
            for (int j = 0; j < r; ++j) Bt_out[(size_t)n * r + j] = B[(size_t)j * N + n];
    }
    return FBQ_OK;
}

// ------------------------------------------------------------------ device entry points

static inline bool misaligned(const void *p) { return ((uintptr_t)p & 15u) != 0; }

namespace fbq {
fbq_status hip_status(hipError_t e)
{
    if (e == hipSuccess) e = hipGetLastError();
    return e == hipSuccess ? FBQ_OK : FBQ_ERR_HIP;
}
}  // namespace fbq

namespace fbq {

// Validates one layer's arguments and fills the launch record; nothing is launched here.
fbq_status check_layer(const fbq_desc *d, int M, const void *x, const void *qweight, const void *scales,
                              const void *zeros, const void *At, const void *Bt, void *y, void *workspace,
                              size_t workspace_bytes, LinearArgs *a)
{
    fbq_status st = fbq_check_desc(d);
    if (st != FBQ_OK) return st;
    if (M < 1) return FBQ_ERR_SHAPE;
    if (!x || !qweight || !scales || !zeros || !y) return FBQ_ERR_NULL;
    if (d->r > 0 && (!At || !Bt)) return FBQ_ERR_NULL;
    const size_t need = least_workspace(d, M);
    if (need > 0 && !workspace) return FBQ_ERR_NULL;
    if (misaligned(x) || misaligned(qweight) || misaligned(scales) || misaligned(zeros) || misaligned(y)) return FBQ_ERR_ALIGN;
    if (d->r > 0 && (misaligned(At) || misaligned(Bt))) return FBQ_ERR_ALIGN;
    if (need > 0 && misaligned(workspace)) return FBQ_ERR_ALIGN;
    if (workspace_bytes < need) return FBQ_ERR_WORKSPACE;
    // (a workspace without room for the partial sums is accepted, and served without the split)
    a->split = split_of(d, M);
    const size_t whole = a->split.segments ? split_workspace(d, M, a->split, need) : need;
    if (!workspace || misaligned(workspace) || workspace_bytes < whole) a->split = {0, 0};
    a->qw = (const uint32_t *)qweight;
    a->scales = (const uint16_t *)scales;
    a->zeros = (const uint16_t *)zeros;
    a->At = (const uint16_t *)At;
    a->Bt = (const uint16_t *)Bt;
    a->x = (const uint16_t *)x;
    a->y = (uint16_t *)y;
    a->workspace = workspace;
    a->workspace_need = a->split.segments ? whole : need;
    a->unsplit_need = need;
    a->M = M; a->N = d->N; a->K = d->K; a->r = d->r; a->bits = d->bits;
    a->mix_with = nullptr; a->mix_out = nullptr;
    return FBQ_OK;
}

static hipError_t launch_prefill(const LinearArgs &call, hipStream_t s)
{
    LinearArgs a = call;
    a.workspace = (char *)call.workspace + handover_reserve(call.K, call.r);
    hipError_t e = launch_prepass_prefill(a, s);
    if (e == hipSuccess) e = launch_gemm_prefill(a, s);
    return e;
}

// One or two tokens: streaming GEMV, one pass per token, with the down-projection inside the launch.
// 3..16 tokens: one pass over the packed words against a matrix-core tile of tokens.  17..64 tokens:
// the same, 16 tokens at a time, the sets of 16 side by side in ONE launch as if they were layers of a group,
// unless the layer lies beyond the line of takes_sets.  More: the prefill GEMM.
hipError_t launch_one(const LinearArgs &a, hipStream_t s)
{
    if (a.M <= kPerTokenMaxM) return launch_gemv_decode(&a, 1, s);
    if (a.split.segments) return launch_few_split(&a, 1, s);
    if (a.M <= kDecodeMaxM) return launch_gemv_small_m(&a, 1, s);
    if (a.M <= kChunkedMaxM && takes_sets(a.M, a.N, a.K)) {
        static_assert(kChunkedMaxM <= kMaxSmallGroup * kDecodeMaxM, "the sets of 16 tokens must fit one grouped launch");
        LinearArgs set[kMaxSmallGroup], rest = a;
        const size_t ws_each = small_m_workspace_bytes(a.K, a.r);
        // One or two tokens left over are a set like the others where the streaming kernel takes the sets: a pass of their own would
        // read the words again.  As a set / with the GEMV, us: 28672 -> 8192 at 17 tokens 58 / 73, at 18 57 / 119 (INT3); 4096 -> 11008 at 18
        // 15 / 21; 4096 -> 4096 at 49 13.8 / 15.7.  One beside two sets is left to the GEMV; three sets in one launch have since become faster
        // (8192 -> 8192 at 33 30.3 with the GEMV, at 48 27.4; 5120 -> 5120 20.4 at 33, 17.9 at 34).
        const bool all_in_sets = a.M != 2 * kDecodeMaxM + 1 && few_stream((long)ceil_div(a.M, kDecodeMaxM) * a.N, a.K);
        int n = 0;
        rest.M = 0;
        for (int m0 = 0; m0 < a.M; m0 += kDecodeMaxM) {
            LinearArgs c = a;
            c.M = std::min(kDecodeMaxM, a.M - m0);
            c.x = a.x + (size_t)m0 * a.K;
            c.y = a.y + (size_t)m0 * a.N;
            if (c.M <= kPerTokenMaxM && !all_in_sets) { rest = c; continue; }
            c.workspace = a.workspace ? (char *)a.workspace + (size_t)n * ws_each : nullptr;
            set[n++] = c;
        }
        hipError_t e = launch_gemv_small_m(set, n, s);
        // (the GEMV runs behind the grouped launch on the stream and marks its words with its own tag, whoever wrote there before)
        if (e == hipSuccess && rest.M > 0) e = launch_gemv_decode(&rest, 1, s);
        return e;
    }
    return launch_prefill(a, s);
}

}  // namespace fbq

extern "C" fbq_status fbq_linear_unfused(const fbq_desc *d, int M, const void *x, const void *qweight, const void *scales,
                                         const void *zeros, const void *At, const void *Bt, void *y, void *workspace,
                                         size_t workspace_bytes, fbq_stream stream)
{
    LinearArgs a;
    const fbq_status st = check_layer(d, M, x, qweight, scales, zeros, At, Bt, y, workspace, workspace_bytes, &a);
    if (st != FBQ_OK) return st;
    if (M > kDecodeMaxM) return FBQ_ERR_UNSUPPORTED;
    if (d->r > 0 && workspace_bytes < (size_t)M * d->r * sizeof(uint16_t)) return FBQ_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    LinearArgs main_path = a;                           // the quantized layer without its sub-branch ...
    main_path.r = 0; main_path.At = nullptr; main_path.Bt = nullptr;
    main_path.split = {0, 0};                           // (in one launch)
    hipError_t e = launch_one(main_path, s);
    if (e == hipSuccess && d->r > 0) e = launch_unfused_branch(a, (uint16_t *)workspace, s);   // ... and the sub-branch on top
    return hip_status(e);
}

extern "C" fbq_status fbq_linear(const fbq_desc *d, int M, const void *x, const void *qweight, const void *scales,
                                 const void *zeros, const void *At, const void *Bt, void *y, void *workspace,
                                 size_t workspace_bytes, fbq_stream stream)
{
    LinearArgs a;
    const fbq_status st = check_layer(d, M, x, qweight, scales, zeros, At, Bt, y, workspace, workspace_bytes, &a);
    if (st != FBQ_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    return hip_status(launch_one(a, s));
}

static bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

// What an average is written to may be nothing that a layer of the call reads or writes, and what it is taken with may be no
// layer's result: within a launch, and between the launches of a call, nothing orders the one against the other.
static bool mix_tensors_overlap(const LinearArgs *args, int n)
{
    for (int i = 0; i < n; ++i) {
        if (!args[i].mix_out) continue;
        const size_t ni = (size_t)args[i].M * args[i].N * sizeof(uint16_t);
        for (int j = 0; j < n; ++j) {
            const LinearArgs &b = args[j];
            const size_t nx = (size_t)b.M * b.K * sizeof(uint16_t), ny = (size_t)b.M * b.N * sizeof(uint16_t);
            if (overlap(args[i].mix_out, ni, b.x, nx) || overlap(args[i].mix_out, ni, b.y, ny) || overlap(args[i].mix_with, ni, b.y, ny)) return true;
            if (b.mix_out && overlap(args[i].mix_out, ni, b.mix_with, ny)) return true;
            if (b.mix_out && j > i && overlap(args[i].mix_out, ni, b.mix_out, ny)) return true;
        }
    }
    return false;
}

// mix: null or n entries
static fbq_status linear_group(const fbq_layer_call *calls, const fbq_mix *mix, int n, int M, hipStream_t s)
{
    constexpr int kMaxCalls = 64;
    if (!calls) return FBQ_ERR_NULL;
    if (n < 1 || n > kMaxCalls) return FBQ_ERR_SHAPE;
    LinearArgs args[kMaxCalls];
    for (int i = 0; i < n; ++i) {
        const fbq_layer_call &c = calls[i];
        const fbq_status st = check_layer(&c.desc, M, c.x, c.qweight, c.scales, c.zeros, c.At, c.Bt, c.y, c.workspace,
                                          c.workspace_bytes, &args[i]);
        if (st != FBQ_OK) return st;
        if (!mix || !mix[i].out) continue;
        if (!mix[i].with) return FBQ_ERR_NULL;
        if (misaligned(mix[i].with) || misaligned(mix[i].out)) return FBQ_ERR_ALIGN;
        args[i].mix_with = (const uint16_t *)mix[i].with;
        args[i].mix_out = (uint16_t *)mix[i].out;
    }
    // A layer whose room for partial sums meets another layer's workspace goes unsplit: what such calls did before K was split, sharing nothing
    // that they needed, they still do.
    const auto meet = [&](int i, int j) {
        return args[i].workspace_need && args[j].workspace_need && overlap(args[i].workspace, args[i].workspace_need, args[j].workspace, args[j].workspace_need);
    };
    bool unsplit[kMaxCalls] = {false};
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) unsplit[i] = unsplit[i] || (i != j && args[i].split.segments && meet(i, j));
    for (int i = 0; i < n; ++i) {
        if (!unsplit[i]) continue;
        args[i].split = {0, 0};
        args[i].workspace_need = args[i].unsplit_need;
    }
    // Layers that share a launch carry the same launch tag: two of them writing their hand-over words into the same
    // memory would accept each other's t.  Workspaces must not overlap.
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < i; ++j)
            if (meet(i, j)) return FBQ_ERR_WORKSPACE;
    if (mix && mix_tensors_overlap(args, n)) return FBQ_ERR_UNSUPPORTED;
    hipError_t e = hipSuccess;
    if (M > kDecodeMaxM) {
        for (int i = 0; i < n && e == hipSuccess; ++i) {
            LinearArgs plain = args[i];
            plain.mix_with = nullptr; plain.mix_out = nullptr;
            e = launch_one(plain, s);
            if (e == hipSuccess && args[i].mix_out) e = launch_mix(args[i], s);
        }
        return hip_status(e);
    }
    // Decode: layers that fit one launch (the same kernel instance; for 4..16 tokens also the same
    // activations) are served together.
    const bool few = M > kPerTokenMaxM;
    const int cap = few ? kMaxSmallGroup : kMaxGroup;
    bool done[kMaxCalls] = {false};
    for (int i = 0; i < n && e == hipSuccess; ++i) {
        if (done[i]) continue;
        LinearArgs batch[kMaxGroup];
        int nb = 0;
        for (int j = i; j < n && nb < cap; ++j) {
            if (!done[j] && (few ? !args[j].split.segments == !args[i].split.segments && small_m_group_compatible(args[i], args[j]) : decode_group_compatible(args[i], args[j]))) {
                batch[nb++] = args[j];
                done[j] = true;
            }
        }
        e = !few ? launch_gemv_decode(batch, nb, s) : batch[0].split.segments ? launch_few_split(batch, nb, s) : launch_gemv_small_m(batch, nb, s);
    }
    return hip_status(e);
}

extern "C" fbq_status fbq_linear_group(const fbq_layer_call *calls, int n, int M, fbq_stream stream)
{
    return linear_group(calls, nullptr, n, M, (hipStream_t)stream);
}

extern "C" fbq_status fbq_linear_group_mix(const fbq_layer_call *calls, const fbq_mix *mix, int n, int M, fbq_stream stream)
{
    if (!mix) return FBQ_ERR_NULL;
    return linear_group(calls, mix, n, M, (hipStream_t)stream);
}

extern "C" fbq_status fbq_silu_mul(const void *gate, const void *up, void *out, size_t count, fbq_stream stream)
{
    if (!gate || !up || !out) return FBQ_ERR_NULL;
    if (count < 1) return FBQ_ERR_SHAPE;
    if (misaligned(gate) || misaligned(up) || misaligned(out)) return FBQ_ERR_ALIGN;
    return hip_status(launch_silu_mul(gate, up, out, count, (hipStream_t)stream));
}

extern "C" fbq_status fbq_reconstruct(const fbq_desc *d, const void *qweight, const void *scales, const void *zeros,
                                      const void *At, const void *Bt, float *W_hat, fbq_stream stream)
{
    fbq_status st = fbq_check_desc(d);
    if (st != FBQ_OK) return st;
    if (!qweight || !scales || !zeros || !W_hat) return FBQ_ERR_NULL;
    if (d->r > 0 && (!At || !Bt)) return FBQ_ERR_NULL;
    if (misaligned(qweight) || misaligned(scales) || misaligned(zeros) || misaligned(W_hat)) return FBQ_ERR_ALIGN;
    if (d->r > 0 && (misaligned(At) || misaligned(Bt))) return FBQ_ERR_ALIGN;
    return hip_status(launch_reconstruct(*d, (const uint32_t *)qweight, (const uint16_t *)scales, (const uint16_t *)zeros,
                                         (const uint16_t *)At, (const uint16_t *)Bt, W_hat, (hipStream_t)stream));
}

extern "C" fbq_status fbq_unpack_codes(const fbq_desc *d, const void *qweight, uint8_t *codes_out, fbq_stream stream)
{
    fbq_status st = fbq_check_desc(d);
    if (st != FBQ_OK) return st;
    if (!qweight || !codes_out) return FBQ_ERR_NULL;
    if (misaligned(qweight) || misaligned(codes_out)) return FBQ_ERR_ALIGN;
    return hip_status(launch_unpack(*d, (const uint32_t *)qweight, codes_out, (hipStream_t)stream));
}

extern "C" fbq_status fbq_quantize_feedback(const fbq_desc *d, const void *W, const void *At, const void *Bt,
                                            void *qweight_out, void *scales_out, void *zeros_out, fbq_stream stream)
{
    fbq_status st = fbq_check_desc(d);
    if (st != FBQ_OK) return st;
    if (!W || !qweight_out || !scales_out || !zeros_out) return FBQ_ERR_NULL;
    if (d->r > 0 && (!At || !Bt)) return FBQ_ERR_NULL;
    if (misaligned(W) || misaligned(qweight_out) || misaligned(scales_out) || misaligned(zeros_out)) return FBQ_ERR_ALIGN;
    if (d->r > 0 && (misaligned(At) || misaligned(Bt))) return FBQ_ERR_ALIGN;
    return hip_status(launch_quantize(*d, (const uint16_t *)W, (const uint16_t *)At, (const uint16_t *)Bt,
                                      (uint32_t *)qweight_out, (uint16_t *)scales_out, (uint16_t *)zeros_out,
                                      (hipStream_t)stream));
}

namespace fbq {
static std::atomic<int> g_spin_limit{kDefaultSpinLimit};
int spin_limit() { return g_spin_limit.load(std::memory_order_relaxed); }
}  // namespace fbq

extern "C" int fbq_test_set_spin_limit(int polls)
{
    const int clamped = polls < 0 ? -1 : std::min(polls, kDefaultSpinLimit);
    return g_spin_limit.exchange(clamped, std::memory_order_relaxed);
}

extern "C" fbq_status fbq_measure_read_stream(const void *buf, size_t bytes, fbq_stream stream)
{
    if (!buf) return FBQ_ERR_NULL;
    if (bytes < 16) return FBQ_ERR_SHAPE;
    if (misaligned(buf)) return FBQ_ERR_ALIGN;
    return hip_status(launch_read_stream(buf, bytes, (hipStream_t)stream));
}

extern "C" size_t fbq_train_workspace_bytes(const fbq_desc *d, int T)
{
    if (fbq_check_desc(d) != FBQ_OK || d->r < 1 || T < 1) return 0;
    return train_workspace_bytes(d->N, d->K, d->r, T);
}

extern "C" fbq_status fbq_gram(const fbq_desc *d, int T, const void *X, float h_scale, void *H16_out, void *workspace,
                               size_t workspace_bytes, fbq_stream stream)
{
    fbq_status st = fbq_check_desc(d);
    if (st != FBQ_OK) return st;
    if (T < 1 || T > (1 << 20) || !(h_scale > 0.0f)) return FBQ_ERR_SHAPE;
    if (!X || !H16_out || !workspace) return FBQ_ERR_NULL;
    if (misaligned(X) || misaligned(H16_out) || misaligned(workspace)) return FBQ_ERR_ALIGN;
    if (workspace_bytes < train_workspace_bytes(d->N, d->K, d->r > 0 ? d->r : 8, T)) return FBQ_ERR_WORKSPACE;
    return hip_status(launch_gram(d->K, T, (const uint16_t *)X, h_scale, (uint16_t *)H16_out, workspace, (hipStream_t)stream));
}

extern "C" fbq_status fbq_train_step(const fbq_desc *d, const void *W, const void *H16, float h_scale, float *At32, float *Bt32,
                                     float lr, void *qweight_out, void *scales_out, void *zeros_out, void *At16_out,
                                     void *Bt16_out, float *grad_At, float *grad_Bt, float *loss, void *workspace,
                                     size_t workspace_bytes, fbq_stream stream)
{
    fbq_status st = fbq_check_desc(d);
    if (st != FBQ_OK) return st;
    if (d->r < 1 || !(h_scale > 0.0f) || !(lr >= 0.0f)) return FBQ_ERR_SHAPE;
    if (!W || !H16 || !At32 || !Bt32 || !qweight_out || !scales_out || !zeros_out || !At16_out || !Bt16_out || !grad_At ||
        !grad_Bt || !workspace)
        return FBQ_ERR_NULL;
    if (misaligned(W) || misaligned(H16) || misaligned(At32) || misaligned(Bt32) || misaligned(qweight_out) ||
        misaligned(scales_out) || misaligned(zeros_out) || misaligned(At16_out) || misaligned(Bt16_out) || misaligned(grad_At) ||
        misaligned(grad_Bt) || misaligned(workspace))
        return FBQ_ERR_ALIGN;
    if (workspace_bytes < train_workspace_bytes(d->N, d->K, d->r, 1)) return FBQ_ERR_WORKSPACE;
    TrainArgs a{};
    a.d = *d;
    a.W = (const uint16_t *)W; a.H16 = (const uint16_t *)H16; a.h_scale = h_scale; a.lr = lr;
    a.At32 = At32; a.Bt32 = Bt32;
    a.qw = (uint32_t *)qweight_out; a.scales = (uint16_t *)scales_out; a.zeros = (uint16_t *)zeros_out;
    a.At16 = (uint16_t *)At16_out; a.Bt16 = (uint16_t *)Bt16_out;
    a.gAt = grad_At; a.gBt = grad_Bt; a.loss = loss; a.workspace = workspace;
    return hip_status(launch_train_step(a, (hipStream_t)stream));
}
