// What the kernels of the 12-bit decode share: sizes, code unpacking, search in an ascending list.
#pragma once

#include "common.h"

namespace antkv {

constexpr int kT12 = 1024;               // threads
constexpr int kW12 = kT12 / 64;          // waves
constexpr int kC12 = 4096;
constexpr int kNH = 4;                   // head slots of a query group (G <= 4)
constexpr int kChunkMax = 32768;         // tokens per workgroup (bitmaps of 1024 words)
constexpr float kEmptyRef12 = -1.0e4f;   // softmax reference before any token: finite, far above the masked score
constexpr int kLutMax12 = 32767;
constexpr int kTabThreads = 256;
constexpr int tab_blocks(int ds) { return (kD / ds) * kC12 / (kTabThreads * 4); }   // per (sequence, KV head), 4 entries per thread
constexpr int heads_per_table(int ds) { return ds == 32 ? 4 : 2; }                  // heads whose int16 table fits 128 KB
constexpr float kPShift12 = 12.f;        // weights are kept scaled by 2^12 so that small ones stay normal in fp16

__device__ __forceinline__ float dot8f(const half8_t& a, const half8_t& b, float acc)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const half2_t x = {a[2 * i], a[2 * i + 1]}, y = {b[2 * i], b[2 * i + 1]};
        acc = __builtin_amdgcn_fdot2(x, y, acc, false);
    }
    return acc;
}

// first position in ascending idx[0..n) whose value is >= target; 64-ary search, every lane returns the same value
__device__ __forceinline__ int lower_bound64(const int32_t* __restrict__ idx, int n, int target, int lane)
{
    int lo = 0, hi = n;                                   // the answer lies in [lo, hi]
    while (hi > lo) {
        const int len = hi - lo;
        const int step = (len + 63) / 64;                 // 64 probes at lo + lane * step cover [lo, hi)
        const int pos = lo + lane * step;
        const bool below = pos < hi && idx[pos] < target;
        const int cnt = (int)__popcll(__ballot(below));   // the list ascends, so these lanes form a prefix
        if (cnt == 0) { hi = lo; break; }
        int nhi = lo + cnt * step;                        // probe cnt is not below the target (or past the end)
        if (nhi > hi) nhi = hi;
        lo = lo + (cnt - 1) * step + 1;                   // probe cnt - 1 is below it
        hi = nhi;                                         // hi - lo <= step - 1 < len: the loop ends
    }
    return lo;
}

template <int N>
__device__ __forceinline__ float row_ror_add(float v)              // plus the value of the lane N places further round in the row of 16
{
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}

// a token's code words: 48 or 96 bits, code m at bits 12 m .. 12 m + 11
template <int DS>
__device__ __forceinline__ void load_cw(const uint8_t* __restrict__ base, int64_t tok, uint32_t (&w)[3])
{
    if constexpr (DS == 32) {
        const uint16_t* s = (const uint16_t*)(base + tok * 6);
        w[0] = (uint32_t)s[0] | ((uint32_t)s[1] << 16);
        w[1] = (uint32_t)s[2];
        w[2] = 0u;
    } else {
        const uint32_t* s = (const uint32_t*)(base + tok * 12);
        w[0] = s[0];
        w[1] = s[1];
        w[2] = s[2];
    }
}

__device__ __forceinline__ uint32_t code12(const uint32_t (&w)[3], int m)
{
    const int bit = 12 * m, d = bit >> 5, sh = bit & 31;       // m is a compile-time constant wherever this is called
    uint32_t v = w[d] >> sh;
    if (sh > 20) v |= w[d + 1] << (32 - sh);
    return v & 0xFFFu;
}

// d12_weights_kernel and d12_values_kernel (decode12_by_code.hip)
struct D12LongParams {
    const half_t* q;
    const uint8_t *codes_k, *codes_v;
    const half_t* cb_v;
    const int32_t *idx_k, *idx_v;
    const half_t *rows_k, *rows_v;
    const float2* tab;                    // [B][Hkv][2 pairs of heads][M][4096] fp32 scores
    const float* tab_amax;                // [B][Hkv][table blocks][4] per-block maxima of |score|
    const float4_t* given;                // or, instead of a table, [B][Hkv][N] the four heads' scores (then k_k is 0)
    float* part;                          // [B][Hq][slots][kD + 2]: S slots of the first kernel, S2 of the second
    float2* stat;                         // [B][Hq][S] reference and sum of the weights that the first kernel wrote
    uint32_t* wts;                        // [pairs of heads][B][Hkv][N] weights, two fp16; both negative: a V-anchored token, where
                                          // it is scored apart -1 if it is not in the K list
    const float4_t* v_scores;             // those scores: [B][Hkv][k_v] of four heads
    float* tile_ref;                      // [B][Hkv][tiles of 64 tokens][4] the references they were taken against
    int64_t N, N_cap, range;              // range: tokens of a workgroup of the second kernel, a multiple of 64
    int k_k, k_v;
    float c1;
    int Hq, Hkv, G, S, chunk, S2, slots;
};
hipError_t launch_decode12_by_code(const Geom& g, const D12LongParams& p, hipStream_t st);

}  // namespace antkv
