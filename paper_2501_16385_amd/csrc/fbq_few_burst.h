// A block of the few-token kernel that works on a burst of row tiles (device code; see fbq_decode_mfma.hip for the method), for the launches of
// small layers and for small layers that share a launch with streamed ones.
#ifndef FBQ_FEW_BURST_H
#define FBQ_FEW_BURST_H

#include "fbq_few_tokens.h"

namespace fbq {

constexpr int kWaveGroups = 4;       // consecutive quantization groups a wave takes per pass over the block's tiles
constexpr int kPassGroups = kMainWaves * kWaveGroups;   // groups one pass covers (4096 codes)

// Length of a K slice of a down-projection: slices of 1024 (they only exist to put more compute units to work on a short, latency-bound
// step), longer where K > 16384.
inline int burst_slice_length(int K) { return std::max(1024, ceil_div(ceil_div(K, kSumSlices), 32 * kMainWaves) * (32 * kMainWaves)); }

// (w & mask) | 0x6400 in both halves: the masked field lands in the mantissa of 1024.0.  Plain C on
// purpose (it becomes one v_and_or_b32): the result feeds a matrix instruction directly, and only
// for instructions it has selected itself does the compiler keep the required distance.
__device__ __forceinline__ half2_t field(uint32_t w, uint32_t mask, uint32_t k6400)
{
    return h2_of((w & mask) | k6400);
}

// The lane's 32 codes of one group and their four matrix operands.  Pair order (also the order of
// the arranged activations): INT4 word j -> codes (8j+f, 8j+f+4), f = 0..3;  INT3 word j -> codes
// (10j+f, 10j+f+5), f = 0..4, and codes (30, 31) last.
template <int BITS>
struct SmallCodes {
    static constexpr int kWords = BITS == 4 ? 4 : 3;
    uint32_t w[kWords];

    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t buf, int lane_off, int tile_off)
    {
        if constexpr (BITS == 4) {
            const uint4_t v = __builtin_amdgcn_raw_buffer_load_b128(buf, lane_off, tile_off, 0);
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else {
            const uint3_t v = __builtin_amdgcn_raw_buffer_load_b96(buf, lane_off, tile_off, 0);
            w[0] = v.x; w[1] = v.y; w[2] = v.z;
        }
    }

    // With from_lane >= 0 the words arrived in load order (lane l: row l / 4, quarter l % 4) and move to matrix order first.
    __device__ __forceinline__ void operands(uint32_t k6400, int from_lane, half8_t (&b)[4])
    {
        if (from_lane >= 0) {
#pragma unroll
            for (int j = 0; j < kWords; ++j) w[j] = (uint32_t)__builtin_amdgcn_ds_bpermute(from_lane, (int)w[j]);
        }
        if constexpr (BITS == 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t lo = w[j], hi = w[j] >> 8;
                b[j] = pack8(field(lo, 0x000F000Fu, k6400), field(lo, 0x00F000F0u, k6400), field(hi, 0x000F000Fu, k6400),
                             field(hi, 0x00F000F0u, k6400));
            }
        } else {
            half2_t d[16];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const uint32_t lo = w[j], hi = w[j] >> 9;
                d[5 * j + 0] = field(lo, 0x00070007u, k6400);
                d[5 * j + 1] = field(lo, 0x00380038u, k6400);
                d[5 * j + 2] = field(lo, 0x01C001C0u, k6400);
                d[5 * j + 3] = field(hi, 0x00070007u, k6400);
                d[5 * j + 4] = field(hi, 0x00380038u, k6400);
            }
            const uint32_t e = ((w[0] >> 15) & 0x00010001u) | ((w[1] >> 14) & 0x00020002u) | ((w[2] >> 13) & 0x00040004u);
            d[15] = h2_of(e | 0x64006400u);
#pragma unroll
            for (int t = 0; t < 4; ++t) b[t] = pack8(d[4 * t], d[4 * t + 1], d[4 * t + 2], d[4 * t + 3]);
        }
    }
};

// fp16 number i (0..4) of three consecutive words
__device__ __forceinline__ half_t half_at(uint3_t w, int i)
{
    const uint32_t lo = i < 2 ? w.x : (i < 4 ? w.y : w.z);
    return __builtin_bit_cast(half_t, (uint16_t)((i & 1) ? lo >> 16 : lo));
}

// Tiles tile0 .. tile0 + T - 1 of layer p.  red and xslab are the block's LDS: the waves' partial tiles, and per wave a group of activations
// on its way from row order (as loaded, coalesced) to lane order, [token][16 pieces of 16 bytes + 1 of padding] (the padding keeps both
// directions free of bank conflicts).
// BITS: 3 or 4.  T: 16-row tiles per block.  BRANCH: r > 0.
// TAIL: some layer of the launch has an odd number of scales (N G odd): see where scale and zero are taken.
// MIX: averages are written with the results; instances of their own for the same reason.
// (p by value: by reference the compiler schedules the INT3 instances otherwise, 8192 x 8192, no sub-branch, 8 tokens 13.8 us by value and 14.8 by reference.)
template <int BITS, int T, bool BRANCH, bool TAIL, bool MIX, typename Params>
__device__ __forceinline__ void few_burst_block(const Params p, int tile0, uint32_t tag, float4_t (*red)[T][64], uint4_t (*xslab)[kTokens * 17])
{
    constexpr int kPiece = BITS == 4 ? 16 : 12;         // bytes of 32 codes
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, q = lane >> 4;
    const int ntiles = (p.N + 15) / 16;
    const int row_bytes = p.row_words * 4;

    const __amdgpu_buffer_rsrc_t qbuf = buffer_of(p.qw, (long)p.N * row_bytes);
    // The range check is per dword, so the count is rounded up to whole dwords: with N·G odd the last
    // half shares an aligned dword with two bytes past the array (same cache line, never another page).
    const __amdgpu_buffer_rsrc_t sbuf = buffer_of(p.scales, ((long)p.N * p.G * 2 + 3) & ~3L);
    const __amdgpu_buffer_rsrc_t zbuf = buffer_of(p.zeros, ((long)p.N * p.G * 2 + 3) & ~3L);
    const __amdgpu_buffer_rsrc_t xbuf = buffer_of(p.x, (long)p.M * p.K * 2);
    // activations are fetched a group at a time in four loads of four token rows each: 16 lanes per row,
    // 256 contiguous bytes (the lane's own 64 bytes of its token would make every load a 64-segment gather)
    const int xtok = lane >> 4, xpiece = lane & 15;

    // Who loads what.  The matrix instruction wants lane (c, q) = lane q * 16 + c to hold quarter q of row c,
    // but loaded that way the four neighbouring lanes of a load quad read four different rows, i.e. four
    // cache lines, and a wave-wide load costs the address path 64 cycles.  So lane l fetches quarter l % 4 of
    // row l / 4 - a quad reads 64 (48) contiguous bytes of one row, 16 cycles per load - and the words change
    // lanes afterwards (ds_bpermute: lane (c, q) takes those of lane 4 c + q).  Scale and zero likewise: the
    // four lanes of a quad read the same 12 bytes of row l / 4, lane (c, q) takes them from lane 4 c.
    // Measured: 4096 -> 11008 11.9 -> 10.8 us, the {gate,up} pair 21.2 -> 19.9, 28672 -> 8192 52.7 -> 49.1.  Not
    // for INT4 with four tiles per block (the extra lane traffic costs more than the address path gains: q/k/v
    // 13.3 -> 14.0; INT3 with four tiles gains, 14.3 -> 13.0) and not for INT3 with two tiles (that instance then spills).
    // Rows past N re-read the last row: computed, never stored.
    constexpr bool kQuadLoads = BITS == 4 ? T <= 3 : T != 2;
    const int from_lane = (4 * c + q) * 4, from_quad = (4 * c) * 4;   // byte addresses of the source lanes
    int qrow[T], srow[T], odd[T];
#pragma unroll
    for (int ti = 0; ti < T; ++ti) {
        const int n = min((tile0 + ti) * 16 + c, p.N - 1);
        const int n_ld = kQuadLoads ? min((tile0 + ti) * 16 + (lane >> 2), p.N - 1) : n;
        qrow[ti] = n_ld * row_bytes + (kQuadLoads ? lane & 3 : q) * kPiece;
        srow[ti] = n_ld * p.G * 2;
        odd[ti] = (n * p.G) & 1;                        // of the row the lane ends up with; the wave's first group is a multiple of four
    }

    // Up-projection: r more values of k, 32 taps a wave.  Lane (c, q) needs t[token c][j .. j + 7] and Bt[row c of every tile][j .. j + 7],
    // j = 32 wave + 8 q; taps past r read beyond the buffers, i.e. zeros.  The Bt part of the first tile or two (cold, from HBM) is requested
    // here with everything else; t (a few KB that every block reads) is fetched when it is needed.
    // The wave follows from the taps alone: dealt out by (tile, taps), what is added to which partial sum, and with it a result's last
    // bit, depended on how many tiles a block owned, i.e. on what the layer shared the launch with.  And a wave polls for t once and not
    // for every tile, and the first waves, which are done first, do it: us, INT3, r = 64, 16 tokens of 4096 x 4096 8.6 dealt out by (tile, taps) of the
    // block, 9.2 by the tile's place in the layer, 8.4 like this; 8192 x 4096, r = 200, 8 tokens 12.7 / 10.2; 4096 x 11008, INT4, 8 tokens 14.9 / 15.0.
    const int tap_steps = BRANCH ? (p.r + 31) / 32 : 0;
    const __amdgpu_buffer_rsrc_t tbuf = buffer_of(p.tsum, BRANCH ? (long)kTokens * p.r * 8 : 0);
    const __amdgpu_buffer_rsrc_t bbuf = buffer_of(p.Bt, BRANCH ? (long)p.N * p.r * 2 : 0);
    constexpr int kNowhere = 0x7FFFFFF0;                // beyond every buffer
    constexpr int kEarlyTaps = T <= 2 ? T : (BITS == 4 && T == 3 ? 0 : 1);   // (no register left for it there)
    half8_t ubf[kEarlyTaps > 0 ? kEarlyTaps : 1];
    auto taps_of = [&](int ti) __attribute__((always_inline)) {
        const int j = wave * 32 + q * 8;
        const int n = min((tile0 + ti) * 16 + c, p.N - 1);
        return __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(bbuf, j < p.r ? (n * p.r + j) * 2 : kNowhere, 0, 0));   // r is a multiple of 8: all eight taps or none
    };
    if (BRANCH) {
#pragma unroll
        for (int ti = 0; ti < kEarlyTaps; ++ti) ubf[ti] = taps_of(ti);
    }

    uint32_t k6400 = 0x64006400u;
    asm volatile("" : "+v"(k6400));                     // keep the constant in a VGPR for v_and_or_b32
    const float4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    float4_t acc[T];
#pragma unroll
    for (int ti = 0; ti < T; ++ti) acc[ti] = zero4;

    // One pass: the wave's four groups g0 .. g0 + 3 against every tile of the block.  Everything the
    // pass needs is requested up front.  Every offset that depends on the group is part of the
    // bounds-checked per-lane offset of its buffer load: groups past the end of K read activation
    // operands and sums beyond their buffers, i.e. zeros without a memory access, and add nothing
    // (their weights are whatever follows in the row, or zero behind the last row: finite either way;
    // their scales and zeros are replaced by zero).
    const int passes = (p.G + kPassGroups - 1) / kPassGroups;
    for (int pass = 0; pass < passes; ++pass) {
        const int g0 = pass * kPassGroups + wave * kWaveGroups;
        // Token rows past M are all zero and are not fetched (their lanes aim beyond the buffer).
        // Order of the requests: the first tile's weights, then the activations, then the other tiles -
        // the weights are the long pole (HBM), so some are under way before the block's share of the
        // activations (L2) occupies the load path, and the first tile can be worked on while the rest streams.
        half8_t xa[kWaveGroups][4];
        float4_t X[kWaveGroups], XS[kWaveGroups];
        SmallCodes<BITS> cw[T][kWaveGroups];
        // Four fp16 scales / zeros, groups g0 .. g0 + 3 of the lane's row: they start at an even or an odd
        // fp16 index, so three aligned words are loaded and shifted by a half where needed.
        uint3_t sc[T], zp[T];
        auto request_tile = [&](int ti) __attribute__((always_inline)) {
#pragma unroll
            for (int gi = 0; gi < kWaveGroups; ++gi) cw[ti][gi].load(qbuf, qrow[ti] + (g0 + gi) * 4 * kPiece, 0);
            sc[ti] = __builtin_amdgcn_raw_buffer_load_b96(sbuf, (srow[ti] + g0 * 2) & ~3, 0, 0);
            zp[ti] = __builtin_amdgcn_raw_buffer_load_b96(zbuf, (srow[ti] + g0 * 2) & ~3, 0, 0);
        };
        request_tile(0);
        // Activations: all four groups at once, or two at a time where the instance is short of registers (INT3,
        // four tiles): the second pair is then requested when the first has been arranged, long before the weights are in.
        constexpr int kXG = BITS == 4 && T <= 3 ? kWaveGroups : 2;
        uint4_t xraw[kXG][4];
        auto request_x = [&](int part) __attribute__((always_inline)) {
#pragma unroll
            for (int gj = 0; gj < kXG; ++gj)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int grp = g0 + kXG * part + gj;
                    xraw[gj][i] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, 4 * i + xtok < p.M && grp < p.G ? (4 * i + xtok) * p.K * 2 + grp * 256 + xpiece * 16 : kNowhere, 0, 0);
                }
        };
        request_x(0);
#pragma unroll
        for (int ti = 1; ti < T; ++ti) request_tile(ti);
        __builtin_amdgcn_sched_barrier(0);
        // while the weights stream: operands, and both sums per token from the matrix core (accumulator
        // register v of lane (., q) belongs to token 4 q + v, which is where the sums are needed)
        half8_t ones;
#pragma unroll
        for (int e = 0; e < 8; ++e) ones[e] = (half_t)1.0f;
#pragma unroll
        for (int part = 0; part < kWaveGroups / kXG; ++part) {
            uint4_t mine[kXG][4];
#pragma unroll
            for (int gj = 0; gj < kXG; ++gj) {
                // through the wave's slab: token rows in, the lane's 64 bytes (token c, quarter q) out
#pragma unroll
                for (int i = 0; i < 4; ++i) xslab[wave][(4 * i + xtok) * 17 + xpiece] = xraw[gj][i];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < 4; ++i) mine[gj][i] = xslab[wave][c * 17 + 4 * q + i];
                __builtin_amdgcn_wave_barrier();
            }
            if (part + 1 < kWaveGroups / kXG) request_x(part + 1);
#pragma unroll
            for (int gj = 0; gj < kXG; ++gj) {
                const int gi = kXG * part + gj;
                arrange_operands<BITS>(mine[gj], xa[gi]);
                float4_t sx = zero4, sxs = zero4;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    sx = mfma(xa[gi][t], gain_operand<BITS>(t), sx);
                    sxs = mfma(xa[gi][t], ones, sxs);
                }
                X[gi] = sx;
                XS[gi] = 1024.0f * sxs;
            }
        }
#pragma unroll
        for (int ti = 0; ti < T; ++ti) {
            // scale and zero of the lane's row from the lane that fetched them
            if constexpr (kQuadLoads) {
            sc[ti] = uint3_t{(uint32_t)__builtin_amdgcn_ds_bpermute(from_quad, (int)sc[ti].x), (uint32_t)__builtin_amdgcn_ds_bpermute(from_quad, (int)sc[ti].y),
                             (uint32_t)__builtin_amdgcn_ds_bpermute(from_quad, (int)sc[ti].z)};
            zp[ti] = uint3_t{(uint32_t)__builtin_amdgcn_ds_bpermute(from_quad, (int)zp[ti].x), (uint32_t)__builtin_amdgcn_ds_bpermute(from_quad, (int)zp[ti].y),
                             (uint32_t)__builtin_amdgcn_ds_bpermute(from_quad, (int)zp[ti].z)};
            }
            // Groups past the end of K add nothing as long as what is read in their place is finite: the next row's
            // scales, or zero beyond the descriptor.  One half is neither: with N G odd the descriptor, whole dwords,
            // also admits the two bytes behind the array, which may hold anything, a NaN included.  That half is cleared
            // (any row within a pass's 32 groups of the array's end can have fetched it).
            if (TAIL && ((p.N * p.G) & 1)) {               // block-uniform; an instance of its own, so that layers with an even number of scales run the code they always ran
                const int n = min((tile0 + ti) * 16 + c, p.N - 1);
                const int kk = ((p.N * p.G) >> 1) - ((n * p.G + g0) >> 1);   // which of the lane's three dwords is the array's last
                sc[ti] = uint3_t{kk == 0 ? sc[ti].x & 0xFFFFu : sc[ti].x, kk == 1 ? sc[ti].y & 0xFFFFu : sc[ti].y, kk == 2 ? sc[ti].z & 0xFFFFu : sc[ti].z};
                zp[ti] = uint3_t{kk == 0 ? zp[ti].x & 0xFFFFu : zp[ti].x, kk == 1 ? zp[ti].y & 0xFFFFu : zp[ti].y, kk == 2 ? zp[ti].z & 0xFFFFu : zp[ti].z};
            }
#pragma unroll
            for (int gi = 0; gi < kWaveGroups; ++gi) {
                half8_t b[4];
                cw[ti][gi].operands(k6400, kQuadLoads ? from_lane : -1, b);
                float4_t D = zero4;
#pragma unroll
                for (int t = 0; t < 4; ++t) D = mfma(xa[gi][t], b[t], D);
                const float s = (float)half_at(sc[ti], gi + odd[ti]), z = (float)half_at(zp[ti], gi + odd[ti]);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[ti][v] = fmaf(s, D[v] - fmaf(z, X[gi][v], XS[gi][v]), acc[ti][v]);
            }
        }
    }

    if (BRANCH && wave < tap_steps) {                   // wave-uniform
        half8_t late[T];
#pragma unroll
        for (int ti = kEarlyTaps; ti < T; ++ti) late[ti] = taps_of(ti);
        const int j = wave * 32 + q * 8;
        // t[token c][j .. j + 7]: eight words {t, launch tag} (four 16-byte device-scope loads), written long ago
        // as a rule.  Should the tags not turn up, the lane computes its eight values itself.
        float t[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};   // (taps past r stay zero also when nothing is ever polled)
        bool ready = false;
        const int off = j < p.r ? (c * p.r + j) * 8 : kNowhere;
        for (int spin = 0; spin < p.spin_limit && !ready; ++spin) {
            bool ok = true;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4_t w = __builtin_amdgcn_raw_buffer_load_b128(tbuf, off + 16 * i, 0, kCacheSc1);
                const uint32_t v0 = w.x, v1 = w.z;
                t[2 * i] = __builtin_bit_cast(float, v0);
                t[2 * i + 1] = __builtin_bit_cast(float, v1);
                ok = ok && (j >= p.r || (w.y == tag && w.w == tag));
            }
            ready = __all(ok);
            if (!ready) __builtin_amdgcn_s_sleep(4);
        }
        if (!ready && j < p.r) {
            const uint16_t *xr = p.x + (size_t)min(c, p.M - 1) * p.K;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint16_t *ar = p.At + (size_t)(j + e) * p.K;
                float a = 0.0f;
                for (int k = 0; k < p.K; ++k) a = fmaf((float)__builtin_bit_cast(half_t, xr[k]), (float)__builtin_bit_cast(half_t, ar[k]), a);
                t[e] = a;
            }
        }
        half8_t thi, tlo;                               // t_hi + t_lo carries 22 bits of the fp32 sum
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            thi[e] = (half_t)t[e];
            tlo[e] = (half_t)(t[e] - (float)thi[e]);
        }
#pragma unroll
        for (int ti = 0; ti < T; ++ti) {
            const half8_t b = ti < kEarlyTaps ? ubf[ti < kEarlyTaps ? ti : 0] : late[ti];
            float4_t d = mfma(thi, b, zero4);
            acc[ti] += mfma(tlo, b, d);
        }
    }

    // K split: every wave leaves its tiles in LDS; wave ti adds them up for tile ti and stores.
#pragma unroll
    for (int ti = 0; ti < T; ++ti) red[wave][ti][lane] = acc[ti];
    // the values to average with, on their way while the waves meet (wave ti stores tile ti)
    static_assert(T <= kMainWaves, "a wave stores at most one tile");
    uint16_t with[4] = {0, 0, 0, 0};
    if constexpr (MIX) {
        if (p.mix_out && wave < T) {                    // wave-uniform
            const __amdgpu_buffer_rsrc_t mbuf = buffer_of(p.mix_with, (long)p.M * p.N * 2);
            const int n = (tile0 + wave) * 16 + c;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                with[v] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(mbuf, n < p.N && 4 * q + v < p.M ? ((4 * q + v) * p.N + n) * 2 : kNowhere, 0, 0);
        }
    }
    __syncthreads();
    for (int ti = wave; ti < T; ti += kMainWaves) {     // wave-uniform
        if (tile0 + ti >= ntiles) break;
        float4_t sum = red[0][ti][lane];
#pragma unroll
        for (int w = 1; w < kMainWaves; ++w) sum += red[w][ti][lane];
        const int n = (tile0 + ti) * 16 + c;
        // lane (c, q) holds output row n and tokens 4 q + v
        if (n < p.N) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 4 * q + v;
                if (m < p.M) {
                    const half_t y = (half_t)sum[v];
                    p.y[(size_t)m * p.N + n] = __builtin_bit_cast(uint16_t, y);
                    if constexpr (MIX) {
                        if (p.mix_out) {
                            const float w = (float)__builtin_bit_cast(half_t, with[v]);
                            p.mix_out[(size_t)m * p.N + n] = __builtin_bit_cast(uint16_t, (half_t)((float)y - ((float)y - w) * 0.5f));
                        }
                    }
                }
            }
        }
    }
}

}  // namespace fbq

#endif
