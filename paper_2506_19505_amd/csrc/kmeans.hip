// One iteration of the offline token-weighted k-means that learns the codebooks (paper Sec. 3.1, "Offline
// Token-Aware Centroids Learning": the sub-vectors of K / V are clustered with one weight per token, the weight
// standing for that token's error-propagation factor).  The assignment step is the online encode kernel; this file
// holds the update step: per (KV head, sub-space, centroid) the weighted sum of the assigned sub-vectors and the
// assigned weight, then the weighted mean.
//
// Accumulation (256 centroids): a workgroup takes one sub-space and walks a range of tokens in chunks of 2048 (d = 16:
// 1024).  It sorts a chunk's sub-vectors by their code into LDS (counting sort: the rank comes from the histogram's
// fetch-add), every thread adds up a run of consecutive sorted tokens in registers, and the runs of a code meet without
// atomics: a code that ends inside a thread's run has exactly one such thread, and a thread ends with exactly one code, so
// both kinds of partial sums have slots of their own.  Totals stay in registers over the chunks.  A workgroup that has a
// sub-space to itself writes the new centroids from there; otherwise one addition per centroid and channel goes to the global
// sums, which the encode kernel has cleared, with hardware float atomics, and km_finalize divides them.  (The ranges' sums as plain
// stores that km_finalize adds up: d 16, 8 ranges, 3 us more; added up by the last workgroup to arrive 7 us more.)  Sums are fp32
// and their order is not fixed: results agree to fp32 rounding, not bit for bit, from run to run.
// The workgroups of one range's sub-spaces run on one XCD, since they read the same lines of x.  Bound: the latency of
// the chain of six barriers per chunk (loads, ranks, sums and merge take about 6 us each).  Adding every product into LDS
// with ds_add_f32, as before, runs at three clocks per lane: 8 heads x 32768 tokens (d8) 195 us, 38 now (a call, with the encode:
// 87, 84 without a launch that clears the sums; 500 tokens 22 and 17); sorting indices and gathering the sub-vectors from memory in
// sorted order thrashes the L2: 55 us.
// With 4096 centroids (12-bit codes) a workgroup owns up to 512 centroids of one sub-space, picks their tokens out of all
// codes and writes the new centroids itself (km_update12).
#include "common.h"

namespace antkv {

namespace {

constexpr int kKsThreads = 512;    // 256 centroids
constexpr int kKwThreads = 1024;   // 4096 centroids
constexpr int kKwCodes = 512;      // most centroids of a workgroup
constexpr int kKwList = 8192;      // sorted tokens in LDS
constexpr int kKwLook = 32768;     // tokens of a chunk: about 4096 of them are the workgroup's
constexpr int ks_per(int d) { return d == 16 ? 2 : 4; }                  // tokens of a chunk per thread
constexpr int ks_chunk(int d) { return kKsThreads * ks_per(d); }

__global__ __launch_bounds__(256) void km_zero(uint32_t* a, int64_t n_a, uint32_t* b, int64_t n_b)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_a) a[i] = 0u;
    else if (i < n_a + n_b) b[i - n_a] = 0u;
}

// no tokens: the codebook stays
__global__ __launch_bounds__(256) void km_keep(const uint32_t* from, uint32_t* to, int64_t n, uint32_t* a, int64_t n_a, uint32_t* b, int64_t n_b)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) to[i] = from[i];
    else if (i < n + n_a) a[i - n] = 0u;
    else if (i < n + n_a + n_b) b[i - n - n_a] = 0u;
}

// The sums of several ranges, and what one range's workgroup writes itself
struct KmOut {
    float* sums;                                                // [Hkv][M][kC][DSUB]
    float* wsum;                                                // [Hkv][M][kC]
    double* obj;                                                // [Hkv][M]
    half_t* cb;
    float* wsum_out;                                            // optional
    double* objective;                                          // optional
};

// LDS of km_accumulate: the sorted sub-vectors, weights and codes, later the last runs of the threads (row e at stride
// kKsThreads + 1: neighbouring e fall on neighbouring banks); runs that ended inside a thread; the centroids
constexpr size_t km_lds_sort(int d)
{
    const size_t sorted = (size_t)ks_chunk(d) * (2 * d + 8), last = (size_t)(d + 1) * (kKsThreads + 1) * 4;
    return ((sorted > last ? sorted : last) + 15) / 16 * 16;
}
constexpr size_t km_lds(int d) { return km_lds_sort(d) + (size_t)kC * (d + 1) * 4 + (size_t)kC * d * 2 + (2 * kC + 4 + 16) * 4; }

// grid: 8 * M * ceil(units / 8) workgroups, a unit being (KV head, range of `range` tokens); `range` is a multiple of the chunk
template <int DSUB>
__global__ __launch_bounds__(kKsThreads, 4) void km_accumulate(
    const half_t* __restrict__ x, const float* __restrict__ w, const uint8_t* __restrict__ codes,
    const half_t* __restrict__ cb, int64_t n_tok, int64_t total, int64_t range, int Hkv, int units, const KmOut out)
{
    constexpr int M = kD / DSUB, NV = DSUB + 1;                 // values of a run: DSUB sums and the weight
    constexpr int kPer = ks_per(DSUB), kChunk = ks_chunk(DSUB), kStride = kKsThreads + 1;
    constexpr int kItems = (kC * NV + kKsThreads - 1) / kKsThreads;     // (centroid, value) pairs of a thread
    typedef half_t vec_t __attribute__((ext_vector_type(DSUB)));
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    vec_t* s_x = (vec_t*)lds;                                   // sorted sub-vectors,
    float* s_w = (float*)(s_x + kChunk);                        // weights
    uint32_t* s_c = (uint32_t*)(s_w + kChunk);                  // and codes
    float* s_last = (float*)lds;                                // [NV][kStride], after the sorted tokens have been read
    float* s_end = (float*)(lds + km_lds_sort(DSUB));           // [kC][NV]
    vec_t* s_cb = (vec_t*)(s_end + kC * NV);
    uint32_t* s_cnt = (uint32_t*)(s_cb + kC);                   // histogram
    uint32_t* s_off = s_cnt + kC;                               // first sorted position of a code; [kC] = tokens
    double* s_obj = (double*)(s_off + kC + 4);                  // one per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int unit = (int)(blockIdx.x / (8 * M)) * 8 + (int)(blockIdx.x & 7), m = (int)(blockIdx.x >> 3) % M;
    if (unit >= units) return;
    const int g = unit % Hkv;
    const bool alone = units == Hkv;                            // one range
    const int64_t j_lo = (int64_t)(unit / Hkv) * range;         // tokens are counted over all sequences
    const int64_t j_hi = total - j_lo < range ? total : j_lo + range;

    int code[kPer];
    float wt[kPer];
    vec_t xv[kPer];
    int64_t seq = j_lo / n_tok, pos = j_lo - seq * n_tok + tid; // this thread's next token: sequence and position in it
    auto fetch = [&](int64_t j0) {                              // tokens j0 + tid, + kKsThreads, ... of the range
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            code[i] = -1;
            if (j0 + tid + i * kKsThreads < j_hi) {
                while (pos >= n_tok) { pos -= n_tok; ++seq; }
                const int64_t r = (seq * Hkv + g) * n_tok + pos;
                code[i] = codes[r * M + m];
                wt[i] = w[r];
                xv[i] = *(const vec_t*)(x + r * kD + m * DSUB);
            }
            pos += kKsThreads;
        }
    };
    fetch(j_lo);
    for (int i = tid; i < kC; i += kKsThreads) s_cb[i] = *(const vec_t*)(cb + (((int64_t)g * M + m) * kC + i) * DSUB);
    float sum[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) sum[k] = 0.f;
    double obj = 0.0;
    for (int64_t j0 = j_lo; j0 < j_hi; j0 += kChunk) {
        const int n = (int)(j_hi - j0 < kChunk ? j_hi - j0 : kChunk);
        if (tid < kC) s_cnt[tid] = 0u;
        lds_barrier();
        uint32_t rank[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) rank[i] = code[i] >= 0 ? atomicAdd(&s_cnt[code[i]], 1u) : 0u;
        lds_barrier();
        if (tid < 64) {                                         // prefix sums, four codes per lane
            uint32_t c[4], own = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) { c[i] = s_cnt[4 * tid + i]; own += c[i]; }
            uint32_t pre = own;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = __shfl_up(pre, off, 64);
                if (tid >= off) pre += o;
            }
            pre -= own;
#pragma unroll
            for (int i = 0; i < 4; ++i) { s_off[4 * tid + i] = pre; pre += c[i]; }
            if (tid == 63) s_off[kC] = pre;
        }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (code[i] >= 0) {
                const uint32_t p = s_off[code[i]] + rank[i];
                s_x[p] = xv[i];
                s_w[p] = wt[i];
                s_c[p] = (uint32_t)code[i];
            }
        }
        lds_barrier();
        if (j0 + kChunk < j_hi) fetch(j0 + kChunk);             // lands while this chunk is added up
        const int p0 = kPer * tid, len = n - p0 < kPer ? n - p0 : kPer;   // this thread's sorted positions (len <= 0: none)
        float acc[NV];
#pragma unroll
        for (int e = 0; e < NV; ++e) acc[e] = 0.f;
        int cur = len > 0 ? (int)s_c[p0] : 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (i < len) {
                const int c = (int)s_c[p0 + i];
                if (c != cur) {                                 // the run of `cur` ends here and nowhere else
#pragma unroll
                    for (int e = 0; e < NV; ++e) { s_end[cur * NV + e] = acc[e]; acc[e] = 0.f; }
                    cur = c;
                }
                const float wi = s_w[p0 + i];
                const vec_t xi = s_x[p0 + i], cv = s_cb[c];
                float dist = 0.f;
#pragma unroll
                for (int e = 0; e < DSUB; ++e) {
                    const float xe = (float)xi[e], df = xe - (float)cv[e];
                    dist = fmaf(df, df, dist);
                    acc[e] = fmaf(wi, xe, acc[e]);
                }
                acc[DSUB] += wi;
                obj += (double)wi * (double)dist;
            }
        }
        lds_barrier();                                        // the sorted tokens' memory becomes the last runs'
        if (len > 0) {
#pragma unroll
            for (int e = 0; e < NV; ++e) s_last[e * kStride + tid] = acc[e];
        }
        lds_barrier();
        // a code's sum: the run that ended inside a thread, if any, and the last runs of the threads whose last position
        // is one of the code's
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int i = tid + k * kKsThreads;
            if (i >= kC * NV) continue;
            const int c = i < kC * DSUB ? i / DSUB : i - kC * DSUB, e = i < kC * DSUB ? i % DSUB : DSUB;
            const int lo = (int)s_off[c], hi = (int)s_off[c + 1];
            if (lo == hi) continue;
            float v = hi % kPer != 0 && hi != n ? s_end[c * NV + e] : 0.f;
            const int t_hi = hi == n ? (n + kPer - 1) / kPer : hi / kPer;
            for (int t = lo / kPer; t < t_hi; ++t) v += s_last[e * kStride + t];
            sum[k] += v;
        }
        // (the next chunk's first barrier keeps s_off and s_last until everybody is here)
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) obj += __shfl_xor(obj, off, 64);
    if (lane == 0) s_obj[wave] = obj;
    __syncthreads();
    const int64_t gm = (int64_t)g * M + m;
    if (tid == 0) {
        double o = 0.0;
        for (int i = 0; i < kKsThreads / 64; ++i) o += s_obj[i];
        if (!alone) unsafeAtomicAdd(out.obj + gm, o);
        else if (out.objective) out.objective[gm] = o;
    }
    if (!alone) {
        float* gs = out.sums + gm * kC * DSUB;
        float* gw = out.wsum + gm * kC;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int i = tid + k * kKsThreads;
            if (i < kC * NV && sum[k] != 0.f) unsafeAtomicAdd(i < kC * DSUB ? gs + i : gw + (i - kC * DSUB), sum[k]);
        }
        return;
    }
    // weighted means; a centroid without assigned weight keeps its old value
    float* s_ws = s_end;                                        // [kC] weights
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = tid + k * kKsThreads;
        if (i >= kC * DSUB && i < kC * NV) {
            s_ws[i - kC * DSUB] = sum[k];
            if (out.wsum_out) out.wsum_out[gm * kC + i - kC * DSUB] = sum[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = tid + k * kKsThreads;
        if (i < kC * DSUB) {
            const float ws = s_ws[i / DSUB];
            out.cb[gm * kC * DSUB + i] = ws > 0.f ? (half_t)(sum[k] / ws) : cb[gm * kC * DSUB + i];
        }
    }
}

// 4096 centroids, codes packed 12 bits each (code m at bits 12 m .. 12 m + 11 of the token's row).  A workgroup owns `cw`
// centroids of one sub-space and walks all tokens in chunks: it counts the codes of its own range, sorts those tokens by
// code in LDS, and DSUB / 8 lanes each add up a window of consecutive sorted tokens, gathering their sub-vectors.  A run
// belongs to the window that it starts in, which alone adds to its centroid's sums in LDS; what a window continues of the
// run before it has a slot of its own and is added after a barrier.  Sums need no atomics; their order inside a code does
// vary from run to run (positions come from fetch-adds).
// Bound: latency of the count, sort and gather passes of a chunk.  Every product added to the global sums with hardware float
// atomics, as before, ran at the L2's atomic rate: 8 heads x 32768 tokens, 35 M additions, 1.77 ms (d32) and 1.63 ms (d16);
// 56 and 82 us now, 500 tokens 17 and 27 us.
constexpr int kw_groups(int d) { return kKwThreads / (d / 8); }
constexpr size_t kw_lds(int d)
{
    return (size_t)kKwList * 4 + (size_t)(kKwCodes + kw_groups(d)) * (d + 1) * 4 + (kKwCodes + 4 + kKwCodes) * 4 + 16 * 8;
}

// grid: Hkv * M * (4096 / cw) workgroups, heads fastest (8 heads, one per XCD)
template <int DSUB>
__global__ __launch_bounds__(kKwThreads) void km_update12(
    const half_t* __restrict__ x, const float* __restrict__ w, const uint8_t* __restrict__ codes,
    const half_t* __restrict__ cb_in, half_t* __restrict__ cb_out, float* __restrict__ wsum_out,
    double* __restrict__ objective, int64_t n_tok, int64_t total, int Hkv, int cw)
{
    constexpr int M = kD / DSUB, L = DSUB / 8, CB = 3 * M / 2, NC = 4096, NV = DSUB + 1, NG = kw_groups(DSUB);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    uint32_t* s_list = (uint32_t*)lds;                          // code << 16 | token, sorted by code
    float* s_sum = (float*)(s_list + kKwList);                  // [kKwCodes][NV]: DSUB sums and the weight
    float* s_first = s_sum + kKwCodes * NV;                     // [NG][NV]: what a window continues
    uint32_t* s_off = (uint32_t*)(s_first + NG * NV);           // first sorted position of a code; [kKwCodes] = tokens
    uint32_t* s_cur = s_off + kKwCodes + 4;                     // histogram, then the next free position of a code
    double* s_obj = (double*)(s_cur + kKwCodes);                // one per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ranges = NC / cw;
    const int g = (int)(blockIdx.x % Hkv), rest = (int)(blockIdx.x / Hkv), m = rest / ranges, c0 = rest % ranges * cw;
    const int gi = tid / L, part = tid % L;                     // the thread's window, and its channels 8 part .. 8 part + 7
    const int64_t gm = (int64_t)g * M + m;
    const half_t* cen = cb_in + (gm * NC + c0) * DSUB + 8 * part;
    const uint8_t* code_at = codes + (12 * m >> 3);             // the 12 bits of code m: in two bytes of the row
    const int code_shift = (12 * m) & 7;
    for (int i = tid; i < kKwCodes * NV; i += kKwThreads) s_sum[i] = 0.f;

    int64_t seq0 = 0, pos0 = 0;                                 // first token of the chunk (counted over all sequences)
    auto row_of = [&](int t) {
        int64_t seq = seq0, pos = pos0 + t;                     // (pos0 + t < n_tok + 32768 fits 32 bits)
        if (pos >= n_tok) {
            const uint32_t more = (uint32_t)pos / (uint32_t)n_tok;
            seq += more;
            pos -= (int64_t)more * n_tok;
        }
        return (seq * Hkv + g) * n_tok + pos;
    };
    auto each_own = [&](int len, auto&& f) {                    // f(token, code - c0) for the chunk's tokens of this range
        for (int t0 = tid; t0 < len; t0 += 8 * kKwThreads) {
            uint32_t two[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int t = t0 + u * kKwThreads;
                two[u] = 0u;
                if (t < len) {
                    const uint8_t* cr = code_at + row_of(t) * CB;
                    two[u] = (uint32_t)cr[0] | ((uint32_t)cr[1] << 8);
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t c = ((two[u] >> code_shift) & 0xFFFu) - (uint32_t)c0;
                const int t = t0 + u * kKwThreads;
                if (t < len && c < (uint32_t)cw) f(t, c);
            }
        }
    };
    double obj = 0.0;
    for (int64_t j0 = 0; j0 < total;) {
        int len = (int)(total - j0 < kKwLook ? total - j0 : kKwLook);
        for (;;) {                                              // at most twice: kKwList tokens always fit the list
            if (tid < kKwCodes) s_cur[tid] = 0u;
            __syncthreads();
            each_own(len, [&](int, uint32_t c) { atomicAdd(&s_cur[c], 1u); });
            __syncthreads();
            if (tid < 64) {                                     // prefix sums, eight codes per lane
                uint32_t c[kKwCodes / 64], own = 0u;
#pragma unroll
                for (int i = 0; i < kKwCodes / 64; ++i) { c[i] = s_cur[kKwCodes / 64 * tid + i]; own += c[i]; }
                uint32_t pre = own;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t o = __shfl_up(pre, off, 64);
                    if (tid >= off) pre += o;
                }
                pre -= own;
#pragma unroll
                for (int i = 0; i < kKwCodes / 64; ++i) {
                    s_off[kKwCodes / 64 * tid + i] = pre;
                    s_cur[kKwCodes / 64 * tid + i] = pre;
                    pre += c[i];
                }
                if (tid == 63) s_off[kKwCodes] = pre;
            }
            __syncthreads();
            if (s_off[kKwCodes] <= kKwList) break;
            len = kKwList;                                      // (crowded codes: a shorter chunk)
        }
        const int n = (int)s_off[kKwCodes];
        each_own(len, [&](int t, uint32_t c) { s_list[atomicAdd(&s_cur[c], 1u)] = (c << 16) | (uint32_t)t; });
        __syncthreads();

        const int per = n > 8 * NG ? (n + NG - 1) / NG : 8;     // sorted positions of a window
        const int p0 = gi * per, p1 = p0 + per < n ? p0 + per : n;
        float acc[8], wacc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
        int cur = p0 < p1 ? (int)(s_list[p0] >> 16) : 0;
        bool continues = p0 < p1 && (int)s_off[cur] < p0;
        auto flush = [&] {
            float* to = continues ? s_first + gi * NV : s_sum + cur * NV;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float* at = to + 8 * part + e;
                *at = continues ? acc[e] : *at + acc[e];
                acc[e] = 0.f;
            }
            if (part == 0) to[DSUB] = continues ? wacc : to[DSUB] + wacc;
            wacc = 0.f;
            continues = false;
        };
        for (int p = p0; p < p1; p += 4) {
            half8_t xv[4], cv[4];
            float wt[4];
            int c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t e = s_list[p + u < p1 ? p + u : p];
                const int64_t r = row_of((int)(e & 0xFFFFu));
                c[u] = (int)(e >> 16);
                wt[u] = w[r];
                xv[u] = *(const half8_t*)(x + r * kD + m * DSUB + 8 * part);
                cv[u] = *(const half8_t*)(cen + (int64_t)c[u] * DSUB);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (p + u < p1) {
                    if (c[u] != cur) { flush(); cur = c[u]; }
                    float dist = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float xe = (float)xv[u][e], df = xe - (float)cv[u][e];
                        dist = fmaf(df, df, dist);
                        acc[e] = fmaf(wt[u], xe, acc[e]);
                    }
                    wacc += wt[u];
                    obj += (double)wt[u] * (double)dist;
                }
            }
        }
        if (p0 < p1) flush();
        __syncthreads();
        for (int i = tid; i < kKwCodes * NV; i += kKwThreads) { // the windows that a run goes on in
            const int c = i / NV, e = i - c * NV, lo = (int)s_off[c], hi = (int)s_off[c + 1];
            if (lo == hi) continue;
            float v = 0.f;
            for (int k = lo / per + 1; k * per < hi; ++k) v += s_first[k * NV + e];
            s_sum[i] += v;
        }
        j0 += len;
        pos0 += len;
        seq0 += pos0 / n_tok;
        pos0 %= n_tok;
        // (the next chunk's first two barriers keep s_off, s_first and s_list until everybody is here)
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) obj += __shfl_xor(obj, off, 64);
    if (lane == 0) s_obj[wave] = obj;
    __syncthreads();
    if (tid == 0 && objective) {
        double o = 0.0;
        for (int i = 0; i < kKwThreads / 64; ++i) o += s_obj[i];
        unsafeAtomicAdd(objective + gm, o);
    }
    // weighted means; a centroid without assigned weight keeps its old value
    for (int i = tid; i < cw * L; i += kKwThreads) {            // (kKwThreads is a multiple of L: `part` is i % L)
        const int c = i / L;
        const float* sum = s_sum + c * NV;
        const float ws = sum[DSUB];
        const half8_t old = *(const half8_t*)(cen + (int64_t)c * DSUB);
        half8_t to;
#pragma unroll
        for (int e = 0; e < 8; ++e) to[e] = ws > 0.f ? (half_t)(sum[8 * part + e] / ws) : old[e];
        *(half8_t*)(cb_out + (gm * NC + c0 + c) * DSUB + 8 * part) = to;
        if (part == 0 && wsum_out) wsum_out[gm * NC + c0 + c] = ws;
    }
}

// the same from the sums of several ranges
template <int DSUB>
__global__ __launch_bounds__(256) void km_finalize(const half_t* __restrict__ cb_in, const KmOut out, int64_t n_centroids)
{
    // a thread takes up to 8 channels of one centroid, so that neighbouring threads touch neighbouring memory
    constexpr int PER = DSUB < 8 ? DSUB : 8, PARTS = DSUB / PER;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / PARTS;                                         // (g, m, c) flattened
    const int part = (int)(t % PARTS);
    if (i >= n_centroids) return;
    const float ws = out.wsum[i];
    if (out.wsum_out && part == 0) out.wsum_out[i] = ws;
    if (out.objective && part == 0 && i % kC == 0) out.objective[i / kC] = out.obj[i / kC];
#pragma unroll
    for (int e = PER * part; e < PER * part + PER; ++e)
        out.cb[i * DSUB + e] = ws > 0.f ? (half_t)(out.sums[i * DSUB + e] / ws) : cb_in[i * DSUB + e];
}

struct KmPlan {
    size_t off_sums, off_wsum, off_obj, total;
};

KmPlan km_plan(const Geom& g)
{
    KmPlan p;                                                   // (with 4096 centroids nothing of it is read or written)
    size_t off = 0;
    p.off_sums = off; off += align_up((size_t)g.Hkv * kD * g.C * sizeof(float));      // M * d_sub = D
    p.off_wsum = off; off += align_up((size_t)g.Hkv * g.M * g.C * sizeof(float));
    p.off_obj = off;  off += align_up((size_t)g.Hkv * g.M * sizeof(double));
    p.total = off;
    return p;
}

// tokens of a workgroup: about two workgroups per CU; a range is whole chunks, since every range adds 256 x (DSUB + 1) values to
// the sums
int64_t km_range(const Geom& g, int64_t n_tok)
{
    const int64_t total = (int64_t)g.B * n_tok, pairs = (int64_t)g.Hkv * g.M, chunk = ks_chunk(g.d);
    return ((total * pairs + 511) / 512 + chunk - 1) / chunk * chunk;
}

template <int DSUB>
hipError_t launch_t(const Geom& g, const half_t* x, const float* w, int64_t n_tok, const half_t* cb_in, half_t* cb_out,
                    const uint8_t* codes, float* wsum_out, double* objective, char* ws, hipStream_t st)
{
    if (n_tok == 0) {
        const int64_t n_cb = (int64_t)g.Hkv * kD * kC / 2, n_w = wsum_out ? (int64_t)g.Hkv * g.M * kC : 0, n_obj = objective ? (int64_t)g.Hkv * g.M * 2 : 0;
        hipLaunchKernelGGL(km_keep, dim3((unsigned)((n_cb + n_w + n_obj + 255) / 256)), dim3(256), 0, st, (const uint32_t*)cb_in,
                           (uint32_t*)cb_out, n_cb, (uint32_t*)wsum_out, n_w, (uint32_t*)objective, n_obj);
        return hipGetLastError();
    }
    const KmPlan p = km_plan(g);
    const KmOut out = {(float*)(ws + p.off_sums), (float*)(ws + p.off_wsum), (double*)(ws + p.off_obj), cb_out, wsum_out, objective};
    static OncePerDevice once;
    const hipError_t setup = allow_lds(once, (const void*)km_accumulate<DSUB>, km_lds(DSUB));
    if (setup != hipSuccess) return setup;
    const int64_t total = (int64_t)g.B * n_tok, range = km_range(g, n_tok), units = (total + range - 1) / range * g.Hkv;
    hipLaunchKernelGGL(km_accumulate<DSUB>, dim3((unsigned)((units + 7) / 8 * 8 * g.M)), dim3(kKsThreads), km_lds(DSUB), st,
                       x, w, codes, cb_in, n_tok, total, range, g.Hkv, (int)units, out);
    if (units > g.Hkv) {
        const int64_t n_cen = (int64_t)g.Hkv * g.M * kC, n_fin = n_cen * (DSUB < 8 ? 1 : DSUB / 8);
        hipLaunchKernelGGL(km_finalize<DSUB>, dim3((unsigned)((n_fin + 255) / 256)), dim3(256), 0, st, cb_in, out, n_cen);
    }
    return hipGetLastError();
}

template <int DSUB>
hipError_t launch_wide(const Geom& g, const half_t* x, const float* w, int64_t n_tok, const half_t* cb_in, half_t* cb_out,
                       const uint8_t* codes, float* wsum_out, double* objective, hipStream_t st)
{
    static OncePerDevice once;
    const hipError_t setup = allow_lds(once, (const void*)km_update12<DSUB>, kw_lds(DSUB));
    if (setup != hipSuccess) return setup;
    if (objective) {
        const int64_t n_obj = (int64_t)g.Hkv * g.M * 2;
        hipLaunchKernelGGL(km_zero, dim3((unsigned)((n_obj + 255) / 256)), dim3(256), 0, st, (uint32_t*)objective, n_obj,
                           (uint32_t*)nullptr, (int64_t)0);
    }
    // Every workgroup looks at all codes of its sub-space, so fewer than 512 centroids each only where 512 leave CUs idle.
    int cw = kKwCodes;
    while (cw > 64 && (int64_t)g.Hkv * g.M * (4096 / cw) < 256) cw /= 2;
    hipLaunchKernelGGL(km_update12<DSUB>, dim3((unsigned)(g.Hkv * g.M * (4096 / cw))), dim3(kKwThreads), kw_lds(DSUB), st, x, w,
                       codes, cb_in, cb_out, wsum_out, objective, n_tok, (int64_t)g.B * n_tok, g.Hkv, cw);
    return hipGetLastError();
}

}  // namespace

size_t kmeans_workspace_bytes(const Geom& g) { return km_plan(g).total; }

ClearWords kmeans_clear(const Geom& g, int64_t n_tok, void* ws)
{
    if ((int64_t)g.B * n_tok <= km_range(g, n_tok)) return {nullptr, 0};       // one range: no sums to share
    return {(uint32_t*)ws, (int64_t)(km_plan(g).total / 4)};
}

// codes [B][Hkv][n_tok][code bytes] must already hold the assignment of x to cb_in, and kmeans_clear's words be zero
hipError_t launch_kmeans_update(const Geom& g, const half_t* x, const float* w, int64_t n_tok, const half_t* cb_in,
                                half_t* cb_out, const uint8_t* codes, float* wsum_out, double* objective, void* ws,
                                hipStream_t st)
{
    if (g.C == 4096) {
        if (g.d == 32) return launch_wide<32>(g, x, w, n_tok, cb_in, cb_out, codes, wsum_out, objective, st);
        return launch_wide<16>(g, x, w, n_tok, cb_in, cb_out, codes, wsum_out, objective, st);
    }
    switch (g.d) {
    case 4: return launch_t<4>(g, x, w, n_tok, cb_in, cb_out, codes, wsum_out, objective, (char*)ws, st);
    case 8: return launch_t<8>(g, x, w, n_tok, cb_in, cb_out, codes, wsum_out, objective, (char*)ws, st);
    default: return launch_t<16>(g, x, w, n_tok, cb_in, cb_out, codes, wsum_out, objective, (char*)ws, st);
    }
}

}  // namespace antkv
