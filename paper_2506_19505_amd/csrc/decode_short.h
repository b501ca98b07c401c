// Decode attention over 12-bit codes for short token ranges (decode_short.hip).
#pragma once

#include "decode12.h"

namespace antkv {

constexpr int kShortRanges = 32;        // most ranges per (sequence, KV head)
constexpr int kShortTokens = 3072;      // most tokens of a range
constexpr int kShortLeast = 128;        // and the fewest a split leaves it

struct ShortParams {
    const half_t* q;
    const uint8_t *codes_k, *codes_v;
    const half_t *cb_k, *cb_v;
    const int32_t *idx_k, *idx_v;
    const half_t *rows_k, *rows_v;
    half_t* out;
    unsigned long long* done;           // [B][Hkv] arrival words (launch_tag.h)
    float* part;                        // [B][Hq][S][kD + 2]: sums, reference, sum of weights
    uint64_t tag;
    int64_t N, N_cap;
    int k_k, k_v;
    float c1;                           // scale * log2(e)
    int B, Hq, Hkv, G;
    int S, chunk;                       // ranges per (sequence, KV head), tokens of a range
};

struct ShortPlan {
    bool on;                            // these kernels are the faster ones for the shape
    int S, chunk;
    size_t off_part, total;             // workspace
};

ShortPlan short_plan(const Geom& g, int64_t N);
hipError_t launch_decode_short(const Geom& g, const ShortPlan& pl, const DecodeArgs& a, void* ws, uint64_t tag, hipStream_t st);

}  // namespace antkv
