// Decode append with an FP16 sliding window of recent tokens (paper Sec. 3.2, last paragraph; window of 32 in
// Sec. 4).  The window lives in the last W entries of the anchor lists.  One launch per step: the retiring token's row
// is encoded (nearest centroid per sub-vector, Sec. 3.1), the window moves one place down and the new row is appended.
//
// Bound: latency.  A step touches one row per head; what costs is the chain launch -> row and centroid loads -> arg-max
// -> store, so every load is issued up front and nothing runs in a loop over sub-spaces.  A (sequence, KV head, K|V) is
// cut by channels: a workgroup encodes the sub-vectors of its own channels and moves the same channels of the window
// rows, so workgroups share no data and need no order among themselves.  A wave takes a whole sub-space (256 centroids:
// four per lane) or, with 4096 centroids, an eighth of one, and finds the arg-max with row rotations instead of LDS
// exchanges.  Neighbouring lanes read one centroid, so that a load instruction covers whole cache lines (one lane per
// 64-byte centroid cost four times the L1 cycles).  8 KV heads, kernel trace: d_sub 4 / 8 / 16 at batch 1 from
// 25 / 13 / 10 us (one workgroup looping over the sub-spaces) to 4.0 / 4.0 / 4.6 us, d32m4096 from 35 to 7.8 us
// with codebooks that a step in between has pushed out of the L2 (12.5 with a workgroup per pair of sub-spaces).
#include "common.h"

namespace antkv {

namespace {

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)      // v of another lane of the row (quad permutation, row rotation)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}

// the wave's maximum / minimum in every lane: row rotations inside 16 lanes, then the four rows through scalar registers
__device__ __forceinline__ float wave_max_all(float x)
{
    x = fmaxf(x, __uint_as_float(dpp<0x121>(__float_as_uint(x))));
    x = fmaxf(x, __uint_as_float(dpp<0x122>(__float_as_uint(x))));
    x = fmaxf(x, __uint_as_float(dpp<0x124>(__float_as_uint(x))));
    x = fmaxf(x, __uint_as_float(dpp<0x128>(__float_as_uint(x))));
    float r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), 16 * i));
    return fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3]));
}
__device__ __forceinline__ uint32_t wave_min_all(uint32_t x)
{
    x = min(x, dpp<0x121>(x));
    x = min(x, dpp<0x122>(x));
    x = min(x, dpp<0x124>(x));
    x = min(x, dpp<0x128>(x));
    uint32_t r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (uint32_t)__builtin_amdgcn_readlane((int)x, 16 * i);
    return min(min(r[0], r[1]), min(r[2], r[3]));
}

// Channels per workgroup and waves: 256 centroids, 32 channels x 4 waves (16 KB of codebook); 4096 centroids, one sub-space
// x 16 waves (128 or 256 KB of codebook) or, PAIR, two of them, whose 12-bit codes fill whole bytes.
template <int DSUB, int NC, bool PAIR>
struct Ap {
    static constexpr int channels = NC == 256 ? 32 : (PAIR ? 2 : 1) * DSUB;
    static constexpr int waves = NC == 256 ? 4 : 16;
    static constexpr int threads = waves * 64;
    static constexpr int subs = channels / DSUB;                          // sub-spaces of the workgroup
    static constexpr int waves_per_sub = waves >= subs ? waves / subs : 1;
    static constexpr int subs_per_wave = waves >= subs ? 1 : subs / waves;
    static constexpr int chunk = DSUB < 8 ? DSUB : 8;                     // channels of a sub-vector that one lane loads
    static constexpr int lanes = DSUB / chunk;                            // lanes of a sub-vector: neighbours read it as one line
    static constexpr int step = 64 / lanes;                               // centroids of one load instruction
    static constexpr int per_wave = NC / waves_per_sub;                   // centroids of a wave
    static_assert(threads >= 64 * channels / 8, "a window of 64 rows is one 16-byte piece per thread");
};

// NC = centroids per sub-space: 256 (one code byte per sub-space) or 4096 (M 12-bit codes packed into 3 M / 2 bytes)
template <int DSUB, int NC, bool PAIR>
__global__ __launch_bounds__((Ap<DSUB, NC, PAIR>::threads)) void append_kernel(
    const half_t* __restrict__ k_new, const half_t* __restrict__ v_new, const half_t* __restrict__ cb_k,
    const half_t* __restrict__ cb_v, uint8_t* __restrict__ codes_k, uint8_t* __restrict__ codes_v, int64_t N_cap,
    int32_t* __restrict__ idx_k, half_t* __restrict__ rows_k, int64_t k_k, int32_t* __restrict__ idx_v,
    half_t* __restrict__ rows_v, int64_t k_v, int64_t N, int W, int Hkv)
{
    using P = Ap<DSUB, NC, PAIR>;
    typedef half_t piece_t __attribute__((ext_vector_type(P::chunk)));
    constexpr int M = kD / DSUB;
    constexpr int kCodeBytes = NC == 256 ? M : 3 * M / 2;
    __shared__ float s_val[P::waves];
    __shared__ uint32_t s_who[P::waves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t bg = blockIdx.x;
    const int g = (int)(bg % Hkv);
    const bool is_v = blockIdx.y != 0;
    const int ch0 = (int)blockIdx.z * P::channels;                               // first channel of the workgroup
    const int64_t kk = is_v ? k_v : k_k;
    half_t* rows = (is_v ? rows_v : rows_k) + (bg * kk + (kk - W)) * kD;          // first window row
    int32_t* idx = (is_v ? idx_v : idx_k) + bg * kk + (kk - W);
    const half_t* fresh = (is_v ? v_new : k_new) + bg * kD;
    const half_t* cb = (is_v ? cb_v : cb_k) + (size_t)g * kD * NC;
    uint8_t* codes = (is_v ? codes_v : codes_k) + (bg * N_cap + (N - W)) * kCodeBytes;   // codes of the retiring position

    // window move: row e takes row e + 1 (the last one the new row); one 16-byte piece per thread, read now, written
    // after the barrier below
    constexpr int kPieces = P::channels / 8;
    const int e = tid / kPieces, off = ch0 + 8 * (tid % kPieces);
    uint4_t mv = {0u, 0u, 0u, 0u};
    if (e < W) mv = (e + 1 < W) ? *(const uint4_t*)(rows + (e + 1) * kD + off) : *(const uint4_t*)(fresh + off);

    // one 12-bit code per workgroup: the words that it lies in, as they are (nobody else changes its bits)
    uint32_t* word = nullptr;
    uint32_t bit = 0, old0 = 0, old1 = 0;
    if constexpr (NC == 4096 && !PAIR) {
        const int64_t at = (bg * N_cap + (N - W)) * kCodeBytes * 8 + 12 * (int64_t)blockIdx.z;
        word = (uint32_t*)(is_v ? codes_v : codes_k) + (at >> 5);
        bit = (uint32_t)at & 31;
        if (tid == 0) {
            old0 = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (bit > 20) old1 = __hip_atomic_load(word + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    // the row that becomes codes: the window's oldest, or the new row itself when there is no window
    const half_t* src = (W > 0) ? rows : fresh;
    const int part = wave % P::waves_per_sub;                                     // the wave's share of its sub-space
    const int li = lane % P::lanes;                                               // the lane's channels inside a sub-vector
    float best[P::subs_per_wave];
    uint32_t who[P::subs_per_wave];
#pragma unroll
    for (int s = 0; s < P::subs_per_wave; ++s) {
        const int m = ch0 / DSUB + (wave / P::waves_per_sub) * P::subs_per_wave + s;
        const uint32_t c_lo = (uint32_t)(part * P::per_wave + lane / P::lanes);
        const half_t* cen = cb + ((int64_t)m * NC + c_lo) * DSUB + li * P::chunk;
        const piece_t x = *(const piece_t*)(src + m * DSUB + li * P::chunk);
        float val = -3.0e38f;
        uint32_t c_best = c_lo;
        // centroids c_lo, c_lo + step, ...: x.c - |c|^2 / 2 (largest = nearest), ascending with a strict '>' so that ties
        // keep the lower index
#pragma unroll 16
        for (int j = 0; j < P::per_wave / P::step; ++j) {
            const piece_t c = *(const piece_t*)(cen + j * P::step * DSUB);
            float nn = 0.f, dot = 0.f;
#pragma unroll
            for (int t = 0; t < P::chunk; t += 2) {                               // fp16 products are exact, sums are fp32
                const half2_t c2 = {c[t], c[t + 1]}, x2 = {x[t], x[t + 1]};
                nn = __builtin_amdgcn_fdot2(c2, c2, nn, false);
                dot = __builtin_amdgcn_fdot2(x2, c2, dot, false);
            }
            float sc = fmaf(-0.5f, nn, dot);
            if constexpr (P::lanes >= 2) sc += __uint_as_float(dpp<0xB1>(__float_as_uint(sc)));   // quad lanes 1 0 3 2
            if constexpr (P::lanes == 4) sc += __uint_as_float(dpp<0x4E>(__float_as_uint(sc)));   // quad lanes 2 3 0 1
            if (sc > val) { val = sc; c_best = c_lo + P::step * j; }
        }
        best[s] = wave_max_all(val);
        who[s] = wave_min_all(val == best[s] ? c_best : 0xffffffffu);             // the lowest index among equals
    }
    if constexpr (P::waves_per_sub > 1) {
        if (lane == 0) { s_val[wave] = best[0]; s_who[wave] = who[0]; }
    }
    __syncthreads();                                                              // window and row are read everywhere
    if constexpr (NC == 256) {
        if constexpr (P::waves_per_sub == 1) {
#pragma unroll
            for (int s = 0; s < P::subs_per_wave; ++s)
                if (lane == 0) codes[ch0 / DSUB + wave * P::subs_per_wave + s] = (uint8_t)who[s];
        } else if (tid < P::subs) {
            float val = s_val[tid * P::waves_per_sub];
            uint32_t c = s_who[tid * P::waves_per_sub];
#pragma unroll
            for (int w = 1; w < P::waves_per_sub; ++w)                            // ascending shares, strict '>'
                if (s_val[tid * P::waves_per_sub + w] > val) { val = s_val[tid * P::waves_per_sub + w]; c = s_who[tid * P::waves_per_sub + w]; }
            codes[ch0 / DSUB + tid] = (uint8_t)c;
        }
    } else if constexpr (!PAIR) {
        if (wave == 0) {                                                          // the lowest index among the waves' equals
            const float val = lane < P::waves ? s_val[lane] : -3.0e38f;
            const float top = wave_max_all(val);
            const uint32_t code = wave_min_all(lane < P::waves && val == top ? s_who[lane] : 0xffffffffu) & 0xfffu;
            if (lane == 0) {
                // Other workgroups change other bits of these words at the same time: what differs in the code's own bits is flipped.
                __hip_atomic_fetch_xor(word, (old0 ^ (code << bit)) & (0xfffu << bit), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (bit > 20)
                    __hip_atomic_fetch_xor(word + 1, (old1 ^ (code >> (32 - bit))) & (0xfffu >> (32 - bit)), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    } else if (tid == 0) {
        uint32_t c2[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float val = s_val[s * P::waves_per_sub];
            c2[s] = s_who[s * P::waves_per_sub];
#pragma unroll
            for (int w = 1; w < P::waves_per_sub; ++w)
                if (s_val[s * P::waves_per_sub + w] > val) { val = s_val[s * P::waves_per_sub + w]; c2[s] = s_who[s * P::waves_per_sub + w]; }
        }
        // 12-bit codes, little-endian, code m at bits 12 m .. 12 m + 11: two codes are three whole bytes
        uint8_t* dst = codes + 3 * blockIdx.z;
        dst[0] = (uint8_t)c2[0];
        dst[1] = (uint8_t)((c2[0] >> 8) | (c2[1] << 4));
        dst[2] = (uint8_t)(c2[1] >> 4);
    }
    if (e < W) {
        *(uint4_t*)(rows + e * kD + off) = mv;
        if (blockIdx.z == 0 && tid % kPieces == 0) idx[e] = (int32_t)(N - W + 1 + e);
    }
}

}  // namespace

hipError_t launch_append(const Geom& g, const half_t* k_new, const half_t* v_new, const half_t* cb_k, const half_t* cb_v,
                         uint8_t* codes_k, uint8_t* codes_v, int64_t N_cap, int32_t* idx_k, half_t* rows_k, int64_t k_k,
                         int32_t* idx_v, half_t* rows_v, int64_t k_v, int64_t N, int W, hipStream_t st)
{
    if (g.B == 0) return hipSuccess;
#define ANTKV_AP(DS, NCEN, PAIR)                                                                                     \
    hipLaunchKernelGGL((append_kernel<DS, NCEN, PAIR>), dim3((unsigned)(g.B * g.Hkv), 2, kD / Ap<DS, NCEN, PAIR>::channels), \
                       dim3(Ap<DS, NCEN, PAIR>::threads), 0, st, k_new, v_new, cb_k, cb_v, codes_k, codes_v, N_cap, idx_k,    \
                       rows_k, k_k, idx_v, rows_v, k_v, N, W, g.Hkv)
    // 12-bit codes: a workgroup per sub-space while that leaves each a CU of its own (a CU takes 57 GB/s of a cold codebook: d 32,
    // 8 heads 12.5 us in pairs, 7.8 alone; d 16, 24 heads are 384 workgroups, a whole step 71.1 us in pairs and 72.3 alone).  It
    // changes its bits of 32-bit words, which the buffer has to consist of (d 32 has rows of six bytes).
    const int64_t rows = (int64_t)g.B * g.Hkv;
    const bool alone = rows * 2 * g.M <= 256 && rows * N_cap * g.code_bytes % 4 == 0;
    if (g.C == 4096 && g.d == 32 && alone) ANTKV_AP(32, 4096, false);
    else if (g.C == 4096 && g.d == 32) ANTKV_AP(32, 4096, true);
    else if (g.C == 4096 && alone) ANTKV_AP(16, 4096, false);
    else if (g.C == 4096) ANTKV_AP(16, 4096, true);
    else if (g.d == 4) ANTKV_AP(4, 256, false);
    else if (g.d == 8) ANTKV_AP(8, 256, false);
    else ANTKV_AP(16, 256, false);
#undef ANTKV_AP
    return hipGetLastError();
}

}  // namespace antkv
