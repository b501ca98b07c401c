// Top-k selection of Anchor Scores (keep the ~1 % highest-scoring tokens in FP16; paper Sec. 3,
// Fig. 2(b)) and the gather of the selected FP16 rows.
//
// Exact radix select on an order-preserving 32-bit key:
//   1. histogram of the top 11 key bits per row;
//   2. every workgroup (slice of 8192 scores) finds the bin d0 that holds the k-th largest key.  Where k is small beside all
//      scores (rule: list_above) and the keys of that bin and above fit the row's list (about N/8 + 4096 entries; the usual case
//      for heavy-tailed scores), the workgroup appends its own ones, with their positions and in their order, as a segment of
//      it.  Otherwise it lists its keys of bin d0 alone, if those fit, and counts the ones above.  If they don't (scores crowded
//      into a narrow range) it adds its keys of bin d0 to a second histogram over the next 11 bits;
//   3. only for rows that took the last branch: the same once more, one level down, with prefix (d0, d1) in the place of d0;
//      workgroups of other rows return at once;
//   4. one workgroup per row selects the exact k-th largest key tau among the list's (radix rounds on the remaining bits,
//      histograms in LDS) and counts every slice's keys > tau and == tau; a row whose keys agree in 22 bits for more than the
//      list holds is walked by that workgroup instead;
//   5. an ordered emission pass over the segments, or over the scores of rows without them, writes the positions of all keys > tau
//      plus the lowest-positioned keys == tau needed to reach k, in ascending position order.  (By the one workgroup per row
//      of step 4 it took 20 us for 16 rows of 840000.)
// The scores are read once with segments, and once more where the producer has not counted them for the first histogram.
// Rows of up to 32768 scores fit the registers of one workgroup: topk_row does all of it in one launch (the launches
// above cost 38 us for 128 rows of 1531 scores, this one 6).  The kernels for
// longer rows are bound by latency up to some 100000 scores and by reading the scores beyond.  16 rows of
// 840000 scores whose histogram the producer counted, k 1 %, kernel trace: 61 us when step 2 listed bin d0 alone and step 5 read all
// scores again, 44 now; one call with 256 rows of 40000, k 1 %, 53 and 43.
#include "common.h"

namespace antkv {

namespace {

constexpr int kSlice = 8192;
constexpr int kTopkThreads = 256;
constexpr int kBins = kTopkBins;

// Find the bin where the count of keys taken from the top reaches k_rem.
// On return digit = that bin, k_new = how many keys are still needed inside it.
template <int THREADS = kTopkThreads>
__device__ void find_digit(const uint32_t* __restrict__ hist, int nbins, uint32_t k_rem,
                           uint32_t& digit, uint32_t& k_new, uint32_t* sh)   // sh: 2 + THREADS / 64 words
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bpt = nbins / THREADS;
    uint32_t c[kBins / THREADS];
    uint32_t tot = 0;
    for (int i = 0; i < bpt; ++i) {
        c[i] = hist[nbins - 1 - (tid * bpt + i)];
        tot += c[i];
    }
    uint32_t incl = tot;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t n = __shfl_up(incl, off, 64);
        if (lane >= off) incl += n;
    }
    if (lane == 63) sh[2 + wave] = incl;
    __syncthreads();
    uint32_t prefix = incl - tot;
    for (int w = 0; w < wave; ++w) prefix += sh[2 + w];
    for (int i = 0; i < bpt; ++i) {
        if (prefix < k_rem && prefix + c[i] >= k_rem) {
            sh[0] = (uint32_t)(nbins - 1 - (tid * bpt + i));
            sh[1] = k_rem - prefix;
        }
        prefix += c[i];
    }
    __syncthreads();
    digit = sh[0];
    k_new = sh[1];
    __syncthreads();
}

__global__ __launch_bounds__(256) void zero_u32(uint32_t* p, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

__device__ __forceinline__ const float* row_scores(const float* scores, const float* scores_b, int rows_a, int64_t row,
                                                   int64_t N)
{
    return (row < rows_a) ? scores + row * N : scores_b + (row - rows_a) * N;
}

// per-row header in the workspace
enum { kHeadCount = 0, kHeadTau = 1, kHeadNeedEq = 2, kHeadCrowded = 3, kHeadSegments = 4, kHeadWords = 8 };

__global__ __launch_bounds__(kTopkThreads) void topk_hist0(const float* __restrict__ scores,
                                                           const float* __restrict__ scores_b, int rows_a, int64_t N,
                                                           uint32_t* __restrict__ ws_hist)
{
    __shared__ uint32_t lh[kBins];
    const int64_t row = blockIdx.y;
    for (int i = threadIdx.x; i < kBins; i += kTopkThreads) lh[i] = 0u;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * kSlice;
    const int64_t hi = (lo + kSlice < N) ? lo + kSlice : N;
    const float* src = row_scores(scores, scores_b, rows_a, row, N);
    if (hi - lo == kSlice && (((uintptr_t)(src + lo)) & 15) == 0) {
#pragma unroll
        for (int j = 0; j < kSlice / (4 * kTopkThreads); ++j) {
            const float4_t v = *(const float4_t*)(src + lo + 4 * (threadIdx.x + kTopkThreads * j));
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(&lh[float_key(v[e]) >> 21], 1u);
        }
    } else {
        for (int64_t i = lo + threadIdx.x; i < hi; i += kTopkThreads) atomicAdd(&lh[float_key(src[i]) >> 21], 1u);
    }
    __syncthreads();
    uint32_t* hist = ws_hist + row * 2 * kBins;
    for (int i = threadIdx.x; i < kBins; i += kTopkThreads)
        if (lh[i]) atomicAdd(&hist[i], lh[i]);
}

// Keys of a slice in a thread.  A whole, 16-byte aligned slice: a thread owns 32 consecutive scores; any other: a wave owns 2048
// consecutive ones, 64 at a time (coalesced), element j of lane l at 64 j + l.  (16 rows of 840000, listing: aligned 14 us by
// threads, 20 by waves; 840003 scores, not aligned, 87 by threads (a dword at a time), 16 by waves.)
constexpr int kPer = kSlice / kTopkThreads;

// What a row's list holds, for `above` keys in higher bins and `bin` in the k-th key's: every key from that bin up (in segments),
// the bin's, or nothing
enum { kListAbove, kListBin, kListNone };
__device__ __forceinline__ int list_kind(uint32_t above, uint32_t bin, uint32_t cap, bool list_above)
{
    return list_above && above + bin <= cap ? kListAbove : (bin <= cap ? kListBin : kListNone);
}

// LEVEL 1: list the keys from bin d0 up, or bin d0's, or (crowded) histogram the next 11 bits of bin d0's.  LEVEL 2, crowded rows
// only: the same for the prefix (d0, d1).  segs: [rows][slices] (start, length) of the slice's segment of the row's list;
// counts, where the list holds the bin alone: [rows][slices] (keys above it, 0).
template <int LEVEL>
__global__ __launch_bounds__(kTopkThreads) void topk_collect(const float* __restrict__ scores,
                                                             const float* __restrict__ scores_b, int rows_a, int64_t N,
                                                             uint32_t k, uint32_t* __restrict__ ws_hist,
                                                             uint32_t* __restrict__ head, uint2_t* __restrict__ segs,
                                                             uint2_t* __restrict__ counts, int n_slices,
                                                             uint2_t* __restrict__ cand, uint32_t cap, bool list_above)
{
    __shared__ uint32_t lh[LEVEL == 1 ? kBins : 1];
    __shared__ uint32_t sh[8];
    __shared__ uint32_t red[2][4];
    __shared__ uint32_t s_base;
    const int64_t row = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t* hist0 = ws_hist + row * 2 * kBins;
    uint32_t* hist1 = hist0 + kBins;
    if (LEVEL == 2 && head[row * kHeadWords + kHeadCrowded] == 0u) return;
    // the scores are requested ahead of the histogram, whose latency they share
    const int64_t slice_lo = (int64_t)blockIdx.x * kSlice;
    const float* src = row_scores(scores, scores_b, rows_a, row, N);
    const bool fast = slice_lo + kSlice <= N && (((uintptr_t)(src + slice_lo)) & 15) == 0;
    const int64_t lo = slice_lo + (fast ? tid * kPer : wave * (64 * kPer) + lane);
    uint32_t key[kPer];
    if (fast) {
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j) {
            const float4_t v = *(const float4_t*)(src + lo + 4 * j);
#pragma unroll
            for (int e = 0; e < 4; ++e) key[4 * j + e] = __float_as_uint(v[e]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j) key[j] = lo + 64 * j < N ? __float_as_uint(src[lo + 64 * j]) : 0xffffffffu;
    }
    // (past the end keys are 0, the lowest; the NaN 0xffffffff has it too, so those are left out by position)
    const int own = fast ? kPer : (lo < N ? (int)((N - lo + 63) / 64 < kPer ? (N - lo + 63) / 64 : kPer) : 0);
    uint32_t d0, k_rem;
    find_digit(hist0, kBins, k, d0, k_rem, sh);
    int kind = list_kind(k - k_rem, hist0[d0], cap, list_above);   // the same for every workgroup of the row
    uint32_t prefix = d0;
    if (LEVEL == 2) {
        uint32_t d1;
        find_digit(hist1, kBins, k_rem, d1, k_rem, sh);
        prefix = (d0 << 11) | d1;
        kind = list_kind(k - k_rem, hist1[d1], cap, list_above);
        if (kind == kListNone) return;                          // topk_resolve walks the row
    }
    constexpr int kShift = LEVEL == 1 ? 21 : 10;
#pragma unroll
    for (int j = 0; j < kPer; ++j) key[j] = float_key(__uint_as_float(key[j]));
    if (LEVEL == 1 && kind == kListNone) {                      // bin d0's next 11 bits go to the second histogram
        if (blockIdx.x == 0 && tid == 0) head[row * kHeadWords + kHeadCrowded] = 1u;
        for (int i = tid; i < kBins; i += kTopkThreads) lh[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (j < own && (key[j] >> 21) == d0) atomicAdd(&lh[(key[j] >> 10) & 2047u], 1u);
        __syncthreads();
        for (int i = tid; i < kBins; i += kTopkThreads)
            if (lh[i]) atomicAdd(&hist1[i], lh[i]);
        return;
    }
    // entries (keys from first to first + span) of the thread (aligned slices) or of the wave, and what comes before them in the slice
    uint32_t first = prefix << kShift, span = kind == kListAbove ? ~first : (1u << kShift) - 1u;
    uint32_t mine = 0, incl;
    if (kind == kListBin) {
        uint32_t gt = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) gt += key[j] > first + span;
        gt = wave_sum_u32(gt);
        if (lane == 0) red[1][wave] = gt;
    }
    if (fast) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) mine += key[j] - first <= span;
        incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t a = __shfl_up(incl, off, 64);
            if (lane >= off) incl += a;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j) mine += (uint32_t)__popcll(__ballot(j < own && key[j] - first <= span));
        incl = mine;
    }
    if (lane == 63) red[0][wave] = incl;
    __syncthreads();
    if (tid == 0) {
        const uint32_t n = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        s_base = n ? atomicAdd(&head[row * kHeadWords + kHeadCount], n) : 0u;
        if (kind == kListAbove) segs[row * n_slices + blockIdx.x] = uint2_t{s_base, n};
        else counts[row * n_slices + blockIdx.x] = uint2_t{red[1][0] + red[1][1] + red[1][2] + red[1][3], 0u};
    }
    __syncthreads();
    uint32_t at = s_base + incl - mine;
    for (int w = 0; w < wave; ++w) at += red[0][w];
    uint2_t* out = cand + row * (int64_t)cap;
    // (compared again: kept, 32 results spilled scalar registers and cost a wave per SIMD)
    pin(first);
    if (fast) {
        if (mine == 0) return;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (key[j] - first <= span) {
                if (at < cap) out[at] = uint2_t{key[j], (uint32_t)(lo + j)};
                ++at;
            }
        }
    } else {
        const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const bool in = j < own && key[j] - first <= span;
            const uint64_t m = __ballot(in);
            if (m == 0ull) continue;
            const uint32_t my = at + (uint32_t)__popcll(m & below);
            if (in && my < cap) out[my] = uint2_t{key[j], (uint32_t)(lo + 64 * j)};
            at += (uint32_t)__popcll(m);
        }
    }
}

// one more in lh[bin] for every lane that calls; lanes with the first one's bin are counted by one atomic
__device__ __forceinline__ void count_in(uint32_t* lh, uint32_t bin)
{
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    const uint64_t same = __ballot(bin == first);
    if (bin != first) atomicAdd(&lh[bin], 1u);
    else if (__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u)) == 0u)
        atomicAdd(&lh[first], (uint32_t)__popcll(same));
}

// per row: exact k-th largest key among the listed ones (or among all, where the list does not hold them), and the keys > tau
// and == tau of every slice
constexpr int kResolveThreads = 1024;

__global__ __launch_bounds__(kResolveThreads) void topk_resolve(const float* __restrict__ scores,
                                                             const float* __restrict__ scores_b, int rows_a, int64_t N,
                                                             uint32_t k, const uint32_t* __restrict__ ws_hist,
                                                             uint32_t* __restrict__ head, uint2_t* __restrict__ counts,
                                                             int n_slices, const uint2_t* __restrict__ cand, uint32_t cap,
                                                             bool list_above)
{
    __shared__ uint32_t lh[kBins];
    __shared__ uint32_t lh_eq[kBins];
    __shared__ uint32_t sh[2 + kResolveThreads / 64];
    const int64_t row = blockIdx.x;
    const int tid = threadIdx.x;
    const uint32_t* hist0 = ws_hist + row * 2 * kBins;
    const uint32_t* hist1 = hist0 + kBins;
    uint32_t d0, d1 = 0, d2, k_rem, need_eq;
    find_digit<kResolveThreads>(hist0, kBins, k, d0, k_rem, sh);
    uint32_t bin = hist0[d0];
    int kind = list_kind(k - k_rem, bin, cap, list_above);
    const bool crowded = kind == kListNone;
    if (crowded) {
        find_digit<kResolveThreads>(hist1, kBins, k_rem, d1, k_rem, sh);
        bin = hist1[d1];
        kind = list_kind(k - k_rem, bin, cap, list_above);
    }
    const bool listed = kind != kListNone;                       // else more than the list holds agree in 22 bits: walk the row
    const uint32_t n_list = kind == kListAbove ? k - k_rem + bin : bin;
    const uint2_t* list = cand + row * (int64_t)cap;
    const float* src = row_scores(scores, scores_b, rows_a, row, N);
    auto for_each = [&](auto fn) {
        if (listed) {
            constexpr int kAhead = 4;                            // loads of a thread in flight (8: 2 us slower on short lists)
            for (uint32_t i0 = tid; i0 < n_list; i0 += kAhead * kResolveThreads) {
                uint2_t e[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const uint32_t i = i0 + u * kResolveThreads;
                    e[u] = list[i < n_list ? i : n_list - 1];
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    if (i0 + u * kResolveThreads < n_list) fn(e[u][0], e[u][1]);
            }
        } else {
            constexpr int kAhead = 8;
            for (int64_t i0 = tid; i0 < N; i0 += kAhead * kResolveThreads) {
                float e[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int64_t i = i0 + u * kResolveThreads;
                    e[u] = src[i < N ? i : N - 1];
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    if (i0 + u * kResolveThreads < N) fn(float_key(e[u]), (uint32_t)(i0 + u * kResolveThreads));
            }
        }
    };
    if (!crowded) {                                              // the k-th key shares d0 only: round on bits 20..10
        for (int i = tid; i < kBins; i += kResolveThreads) lh[i] = 0u;
        __syncthreads();
        for_each([&](uint32_t key, uint32_t) { if ((key >> 21) == d0) count_in(lh, (key >> 10) & 2047u); });
        __syncthreads();
        find_digit<kResolveThreads>(lh, kBins, k_rem, d1, k_rem, sh);
    }
    const uint32_t prefix22 = (d0 << 11) | d1;
    for (int i = tid; i < kBins; i += kResolveThreads) lh[i] = 0u;
    __syncthreads();
    for_each([&](uint32_t key, uint32_t) { if ((key >> 10) == prefix22) count_in(lh, key & 1023u); });
    __syncthreads();
    find_digit<kResolveThreads>(lh, 1024, k_rem, d2, need_eq, sh);
    const uint32_t tau = (prefix22 << 10) | d2;
    // counts per slice, in LDS for 2048 slices at a time
    uint2_t* c = counts + row * (int64_t)n_slices;
    for (int s0 = 0; s0 < n_slices; s0 += kBins) {
        __syncthreads();
        for (int i = tid; i < kBins; i += kResolveThreads) { lh[i] = 0u; lh_eq[i] = 0u; }
        __syncthreads();
        for_each([&](uint32_t key, uint32_t i) {
            const uint32_t s = i / kSlice - (uint32_t)s0;
            if (s >= (uint32_t)kBins) return;                    // (neighbours in the list are in one slice)
            if (key > tau) count_in(lh, s);
            else if (key == tau) count_in(lh_eq, s);
        });
        __syncthreads();
        for (int i = tid; i < kBins && s0 + i < n_slices; i += kResolveThreads)
            c[s0 + i] = uint2_t{lh[i] + (kind == kListBin ? c[s0 + i][0] : 0u), lh_eq[i]};
    }
    if (tid == 0) {
        head[row * kHeadWords + kHeadTau] = tau;
        head[row * kHeadWords + kHeadNeedEq] = need_eq;
        head[row * kHeadWords + kHeadSegments] = kind == kListAbove ? 1u : 0u;
    }
}

// Writes a wave's selected positions: keys > tau and, up to need_eq of the row, keys == tau.  key[j] of lane l is the score
// at position lo + 64 j (lo includes the lane), so positions ascend over (j, lane); run_gt / run_eq count what lies before.
template <int PER>
__device__ __forceinline__ void emit_ordered(const uint32_t (&key)[PER], uint32_t tau, uint32_t need_eq, uint32_t run_gt,
                                             uint32_t run_eq, int lane, int64_t lo, int32_t* __restrict__ out)
{
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint64_t mg = __ballot(key[j] > tau), me = __ballot(key[j] == tau);
        if ((mg | me) == 0ull) continue;                         // uniform, the usual case at 1 %
        const uint32_t my_gt = run_gt + (uint32_t)__popcll(mg & below), my_eq = run_eq + (uint32_t)__popcll(me & below);
        if (key[j] > tau) out[my_gt + (my_eq < need_eq ? my_eq : need_eq)] = (int32_t)(lo + 64 * j);
        else if (key[j] == tau && my_eq < need_eq) out[my_gt + my_eq] = (int32_t)(lo + 64 * j);
        run_gt += (uint32_t)__popcll(mg);
        run_eq += (uint32_t)__popcll(me);
    }
}

// SEGMENTS: a row's segments are read if it has them, a wave per quarter of one, ranked through ballots.  Otherwise the scores,
// requested ahead of the counts, whose latency they share.
template <bool SEGMENTS>
__global__ __launch_bounds__(kTopkThreads) void topk_emit(const float* __restrict__ scores,
                                                          const float* __restrict__ scores_b, int rows_a, int64_t N,
                                                          uint32_t k, const uint32_t* __restrict__ head,
                                                          const uint2_t* __restrict__ counts, const uint2_t* __restrict__ segs,
                                                          int n_slices, const uint2_t* __restrict__ cand, uint32_t cap,
                                                          int32_t* __restrict__ idx, int32_t* __restrict__ idx_b)
{
    __shared__ uint32_t red[4][4];
    const int64_t row = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t slice_lo = (int64_t)blockIdx.x * kSlice;
    const float* src = row_scores(scores, scores_b, rows_a, row, N);
    const bool fast = slice_lo + kSlice <= N && (((uintptr_t)(src + slice_lo)) & 15) == 0;
    const int64_t lo = slice_lo + (fast ? tid * kPer : wave * (64 * kPer) + lane);
    uint32_t key[kPer];
    // (Past the end keys are 0, the lowest.  The NaN 0xffffffff has it too, but at earlier positions, and need_eq counts only
    // those.)
    auto request = [&]() {
        if (fast) {
#pragma unroll
            for (int j = 0; j < kPer / 4; ++j) {
                const float4_t v = *(const float4_t*)(src + lo + 4 * j);
#pragma unroll
                for (int e = 0; e < 4; ++e) key[4 * j + e] = __float_as_uint(v[e]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j) key[j] = lo + 64 * j < N ? __float_as_uint(src[lo + 64 * j]) : 0xffffffffu;
        }
    };
    if constexpr (!SEGMENTS) request();
    const uint32_t tau = head[row * kHeadWords + kHeadTau], need_eq = head[row * kHeadWords + kHeadNeedEq];
    const bool segments = SEGMENTS && head[row * kHeadWords + kHeadSegments] != 0u;
    const uint2_t seg = SEGMENTS ? segs[row * n_slices + blockIdx.x] : uint2_t{0u, 0u};
    // keys > tau and == tau in the slices before this one
    uint32_t bgt = 0, beq = 0;
    for (int s = tid; s < (int)blockIdx.x; s += kTopkThreads) {
        const uint2_t c = counts[row * n_slices + s];
        bgt += c[0];
        beq += c[1];
    }
    bgt = wave_sum_u32(bgt);
    beq = wave_sum_u32(beq);
    if (lane == 0) { red[0][wave] = bgt; red[1][wave] = beq; }
    int32_t* out = (row < rows_a) ? idx + row * (int64_t)k : idx_b + (row - rows_a) * (int64_t)k;
    uint32_t gt = 0, eq = 0, my_gt = 0, my_eq = 0;               // of the wave; of the thread and, then, of the lanes up to it
    if (segments) {
        const uint2_t* list = cand + row * (int64_t)cap + seg[0];
        const uint32_t quarter = (seg[1] + 255) / 256 * 64, e_lo = wave * quarter, e_hi = e_lo + quarter < seg[1] ? e_lo + quarter : seg[1];
        for (uint32_t i = e_lo + lane; i < e_hi; i += 64) {
            const uint32_t x = list[i][0];
            gt += x > tau;
            eq += x == tau;
        }
        gt = wave_sum_u32(gt);
        eq = wave_sum_u32(eq);
        if (lane == 0) { red[2][wave] = gt; red[3][wave] = eq; }
        __syncthreads();
        uint32_t run_gt = red[0][0] + red[0][1] + red[0][2] + red[0][3], run_eq = red[1][0] + red[1][1] + red[1][2] + red[1][3];
        for (int w = 0; w < wave; ++w) { run_gt += red[2][w]; run_eq += red[3][w]; }
        const uint64_t below = (1ull << lane) - 1ull;
        for (uint32_t i0 = e_lo; i0 < e_hi; i0 += 64) {
            const bool in = i0 + lane < e_hi;
            const uint2_t e = list[in ? i0 + lane : e_lo];
            const bool is_gt = in && e[0] > tau, is_eq = in && e[0] == tau;
            const uint64_t mg = __ballot(is_gt), me = __ballot(is_eq);
            const uint32_t at_gt = run_gt + (uint32_t)__popcll(mg & below), at_eq = run_eq + (uint32_t)__popcll(me & below);
            if (is_gt) out[at_gt + (at_eq < need_eq ? at_eq : need_eq)] = (int32_t)e[1];
            else if (is_eq && at_eq < need_eq) out[at_gt + at_eq] = (int32_t)e[1];
            run_gt += (uint32_t)__popcll(mg);
            run_eq += (uint32_t)__popcll(me);
        }
        return;
    }
    if constexpr (SEGMENTS) request();
#pragma unroll
    for (int j = 0; j < kPer; ++j) key[j] = float_key(__uint_as_float(key[j]));
    if (fast) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) { my_gt += key[j] > tau; my_eq += key[j] == tau; }
        gt = my_gt;
        eq = my_eq;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t a = __shfl_up(gt, off, 64), b = __shfl_up(eq, off, 64);
            if (lane >= off) { gt += a; eq += b; }
        }
        if (lane == 63) { red[2][wave] = gt; red[3][wave] = eq; }
    } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            gt += (uint32_t)__popcll(__ballot(key[j] > tau));
            eq += (uint32_t)__popcll(__ballot(key[j] == tau));
        }
        if (lane == 0) { red[2][wave] = gt; red[3][wave] = eq; }
    }
    __syncthreads();
    uint32_t run_gt = red[0][0] + red[0][1] + red[0][2] + red[0][3], run_eq = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    for (int w = 0; w < wave; ++w) { run_gt += red[2][w]; run_eq += red[3][w]; }
    if (!fast) {
        emit_ordered<kPer>(key, tau, need_eq, run_gt, run_eq, lane, lo, out);
        return;
    }
    run_gt += gt - my_gt;
    run_eq += eq - my_eq;
    if (my_gt == 0 && (my_eq == 0 || run_eq >= need_eq)) return; // nothing of this thread is selected
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (key[j] > tau) {
            out[run_gt + (run_eq < need_eq ? run_eq : need_eq)] = (int32_t)(lo + j);
            ++run_gt;
        } else if (key[j] == tau) {
            if (run_eq < need_eq) out[run_gt + run_eq] = (int32_t)(lo + j);
            ++run_eq;
        }
    }
}

// A whole row of at most 1024 * PER scores in one workgroup: the k-th largest key by three rounds of histograms in LDS (11,
// 11 and 10 bits), then the ordered emission.  Bound: the chain of barriers of the three rounds.
constexpr int kRowThreads = 1024;

template <int PER>
__global__ __launch_bounds__(kRowThreads) void topk_row(const float* __restrict__ scores, const float* __restrict__ scores_b,
                                                        int rows_a, int N, uint32_t k, int32_t* __restrict__ idx,
                                                        int32_t* __restrict__ idx_b)
{
    __shared__ uint32_t lh[3][kBins];
    __shared__ uint32_t sh[2 + kRowThreads / 64];
    __shared__ uint32_t red[2][kRowThreads / 64];
    const int64_t row = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* src = row_scores(scores, scores_b, rows_a, row, N);
    const int lo = wave * (64 * PER) + lane;                     // a wave owns 64 * PER consecutive scores
    uint32_t key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) key[j] = lo + 64 * j < N ? float_key(src[lo + 64 * j]) : 0u;   // (the lowest key; the NaN
                                                                 // 0xffffffff has it too, but at earlier positions, and need_eq counts only those)
    for (int i = tid; i < 3 * kBins; i += kRowThreads) (&lh[0][0])[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (lo + 64 * j < N) atomicAdd(&lh[0][key[j] >> 21], 1u);
    __syncthreads();
    uint32_t d0, d1, d2, k_rem, need_eq;
    find_digit<kRowThreads>(lh[0], kBins, k, d0, k_rem, sh);
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if ((key[j] >> 21) == d0 && lo + 64 * j < N) atomicAdd(&lh[1][(key[j] >> 10) & 2047u], 1u);
    __syncthreads();
    find_digit<kRowThreads>(lh[1], kBins, k_rem, d1, k_rem, sh);
    const uint32_t prefix22 = (d0 << 11) | d1;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if ((key[j] >> 10) == prefix22 && lo + 64 * j < N) atomicAdd(&lh[2][key[j] & 1023u], 1u);
    __syncthreads();
    find_digit<kRowThreads>(lh[2], 1024, k_rem, d2, need_eq, sh);
    const uint32_t tau = (d0 << 21) | (d1 << 10) | d2;
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        gt += (uint32_t)__popcll(__ballot(key[j] > tau));
        eq += (uint32_t)__popcll(__ballot(key[j] == tau));
    }
    if (lane == 0) { red[0][wave] = gt; red[1][wave] = eq; }
    __syncthreads();
    uint32_t run_gt = 0, run_eq = 0;
    for (int w = 0; w < wave; ++w) { run_gt += red[0][w]; run_eq += red[1][w]; }
    int32_t* out = (row < rows_a) ? idx + row * (int64_t)k : idx_b + (row - rows_a) * (int64_t)k;
    emit_ordered<PER>(key, tau, need_eq, run_gt, run_eq, lane, lo, out);
}

__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4_t* __restrict__ x, int64_t N,
                                                          const int32_t* __restrict__ idx, int64_t k,
                                                          uint4_t* __restrict__ rows, int64_t n_items)
{
    // one 16-lane group per row of 128 fp16 = 16 x 16 B
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t item = t >> 4;
    const int part = (int)(t & 15);
    if (item >= n_items) return;
    const int64_t bg = item / k;
    const int64_t j = idx[item];
    rows[item * 16 + part] = x[(bg * N + j) * 16 + part];
}

}  // namespace

namespace {

struct TopkPlan {
    int n_slices;
    uint32_t cap;                      // candidate entries per row
    size_t off_hist, off_head, off_segs, off_counts, off_cand, total;
};

TopkPlan topk_plan(int64_t rows, int64_t N)
{
    TopkPlan p;
    p.n_slices = (int)((N + kSlice - 1) / kSlice);
    if (p.n_slices < 1) p.n_slices = 1;
    // the bin of the k-th key usually holds a few percent of a row; a fuller bin makes topk_resolve walk the row
    p.cap = (uint32_t)(N / 8 + 4096 - p.n_slices);
    size_t off = 0;
    p.off_hist = off;   off += align_up((size_t)rows * 2 * kBins * 4);            // two histogram levels per row
    p.off_head = off;   off += align_up((size_t)rows * kHeadWords * 4);     // directly after the histograms: zeroed together
    p.off_counts = off; off += align_up((size_t)rows * p.n_slices * sizeof(uint2_t));
    p.off_segs = off;                                                             // segments and lists together N / 8 + 4096 per row
    p.off_cand = off + (size_t)rows * p.n_slices * sizeof(uint2_t);
    off += align_up((size_t)rows * (p.n_slices + p.cap) * sizeof(uint2_t));
    p.total = off;
    return p;
}

// Listing every key from the threshold's bin up saves the emission a second pass over the scores; in return the one workgroup per
// row that resolves the threshold walks k more entries, some 0.7 ns each.  The two meet at a k of about 4000 (2 rows of 840000),
// 6500 (16 of 131072), 6000 (2 of 2000000), 15000 (16 of 840000) and 21000 (64 of 400000).  One call, us, listed above and
// not: 16 rows of 840000, k 1 % 54 and 59, 5 % 81 and 64, 25 % 218 and 76; 2 of 2000000, 0.1 % 36 and 38, 1 % 50 and 41, 25 % 404 and 57.
bool list_above(int64_t rows, int64_t N, int64_t k) { return k <= 3000 + rows * N / 1280; }

}  // namespace

size_t topk_workspace_bytes(int64_t n_rows, int64_t N, int64_t k)
{
    (void)k;
    return topk_plan(n_rows, N).total;
}

// Two score arrays of n_rows rows each can be selected in one go (scores_b / idx_b may be NULL): the launches then
// cover 2 n_rows rows, the first n_rows from `scores` into `idx`, the rest from `scores_b` into `idx_b`.
namespace {

// clears the histograms and headers of `rows` rows
uint32_t* topk_clear(int64_t rows, int64_t N, void* ws, hipStream_t st)
{
    const TopkPlan p = topk_plan(rows, N);
    uint32_t* hist = (uint32_t*)((char*)ws + p.off_hist);
    const int64_t nz = (int64_t)(p.off_counts / 4);             // histograms and headers
    hipLaunchKernelGGL(zero_u32, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, st, hist, nz);
    return hist;
}

// everything after the first-level histogram
hipError_t topk_select(const float* scores, int32_t* idx, const float* scores_b, int32_t* idx_b, int64_t n_rows,
                       int64_t N, int64_t k, void* ws, hipStream_t st)
{
    const int64_t rows = scores_b ? 2 * n_rows : n_rows;
    const TopkPlan p = topk_plan(rows, N);
    char* w = (char*)ws;
    uint32_t* hist = (uint32_t*)(w + p.off_hist);
    uint32_t* head = (uint32_t*)(w + p.off_head);
    uint2_t* segs = (uint2_t*)(w + p.off_segs);
    uint2_t* counts = (uint2_t*)(w + p.off_counts);
    uint2_t* cand = (uint2_t*)(w + p.off_cand);
    const int ra = (int)n_rows;
    const bool above = list_above(rows, N, k);
    dim3 grid(p.n_slices, (unsigned)rows);
    hipLaunchKernelGGL(topk_collect<1>, grid, dim3(kTopkThreads), 0, st, scores, scores_b, ra, N, (uint32_t)k, hist, head,
                       segs, counts, p.n_slices, cand, p.cap, above);
    hipLaunchKernelGGL(topk_collect<2>, grid, dim3(kTopkThreads), 0, st, scores, scores_b, ra, N, (uint32_t)k, hist, head,
                       segs, counts, p.n_slices, cand, p.cap, above);
    hipLaunchKernelGGL(topk_resolve, dim3((unsigned)rows), dim3(kResolveThreads), 0, st, scores, scores_b, ra, N, (uint32_t)k,
                       hist, head, counts, p.n_slices, cand, p.cap, above);
    hipLaunchKernelGGL(above ? topk_emit<true> : topk_emit<false>, grid, dim3(kTopkThreads), 0, st, scores, scores_b, ra, N, (uint32_t)k,
                       head, counts, segs, p.n_slices, cand, p.cap, idx, idx_b);
    return hipGetLastError();
}

}  // namespace

// A row in one workgroup needs no workspace.  Beyond 32 scores per thread they no longer fit the registers, and the few
// workgroups of a long row would leave the chip idle: 16 rows of 32768 take 22 us in one launch and 27 in six, 256 rows 23 and 38.
static bool topk_in_rows(int64_t N) { return N <= 32 * kRowThreads; }

// The same where the producer of the scores could count them for the first histogram: the longer launches then save a read of
// the scores, and fewer than 64 aligned rows of more than 16384 are quicker that way.  Decode step with re-selection, d_sub 8,
// 16 rows of 24576 / 32768: 62 / 64 us counted, 66 / 70 in one launch; 256 rows 113 / 132 and 106 / 126; 16 rows of 20001,
// not aligned, 71 and 64; 16 rows of 16384 60 and 62, of 12288 64 and 61.
static bool topk_in_rows_counted(int64_t rows, int64_t N)
{
    return topk_in_rows(N) && (N <= 16384 || rows >= 64 || N % 4 != 0);
}

static hipError_t launch_topk_rows(const float* scores, int32_t* idx, const float* scores_b, int32_t* idx_b, int64_t n_rows,
                                   int64_t N, int64_t k, hipStream_t st)
{
    const unsigned rows = (unsigned)(scores_b ? 2 * n_rows : n_rows);
#define ANTKV_TR(PER)                                                                                                    \
    hipLaunchKernelGGL(topk_row<PER>, dim3(rows), dim3(kRowThreads), 0, st, scores, scores_b, (int)n_rows, (int)N, (uint32_t)k, \
                       idx, idx_b)
    if (N <= 2 * kRowThreads) ANTKV_TR(2);
    else if (N <= 8 * kRowThreads) ANTKV_TR(8);
    else ANTKV_TR(32);
#undef ANTKV_TR
    return hipGetLastError();
}

hipError_t launch_topk2(const float* scores, int32_t* idx, const float* scores_b, int32_t* idx_b, int64_t n_rows,
                        int64_t N, int64_t k, void* ws, hipStream_t st)
{
    if (k == 0 || n_rows == 0) return hipSuccess;
    if (topk_in_rows(N)) return launch_topk_rows(scores, idx, scores_b, idx_b, n_rows, N, k, st);
    const int64_t rows = scores_b ? 2 * n_rows : n_rows;
    uint32_t* hist = topk_clear(rows, N, ws, st);
    const TopkPlan p = topk_plan(rows, N);
    dim3 grid(p.n_slices, (unsigned)rows);
    hipLaunchKernelGGL(topk_hist0, grid, dim3(kTopkThreads), 0, st, scores, scores_b, (int)n_rows, N, hist);
    return topk_select(scores, idx, scores_b, idx_b, n_rows, N, k, ws, st);
}

TopkCounts topk2_begin(int64_t n_rows, int64_t N, void* ws)
{
    if (topk_in_rows_counted(2 * n_rows, N)) return {nullptr, 0};
    const TopkPlan p = topk_plan(2 * n_rows, N);
    return {(uint32_t*)((char*)ws + p.off_hist), (int64_t)(p.off_counts / 4)};    // histograms and headers
}

hipError_t launch_topk2_finish(const float* scores, int32_t* idx, const float* scores_b, int32_t* idx_b, int64_t n_rows,
                               int64_t N, int64_t k, void* ws, hipStream_t st)
{
    if (k == 0 || n_rows == 0) return hipSuccess;
    if (topk_in_rows_counted(2 * n_rows, N)) return launch_topk_rows(scores, idx, scores_b, idx_b, n_rows, N, k, st);
    return topk_select(scores, idx, scores_b, idx_b, n_rows, N, k, ws, st);
}

hipError_t launch_topk(const float* scores, int64_t n_rows, int64_t N, int64_t k, int32_t* idx, void* ws,
                       hipStream_t st)
{
    return launch_topk2(scores, idx, nullptr, nullptr, n_rows, N, k, ws, st);
}

hipError_t launch_gather_rows(const Geom& g, const half_t* x, int64_t N, const int32_t* idx, int64_t k,
                              half_t* rows, hipStream_t st)
{
    const int64_t n_items = (int64_t)g.B * g.Hkv * k;
    if (n_items == 0) return hipSuccess;
    const int64_t threads = n_items * 16;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st,
                       (const uint4_t*)x, N, idx, k, (uint4_t*)rows, n_items);
    return hipGetLastError();
}

}  // namespace antkv
