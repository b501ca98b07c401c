// VQ encode: nearest-centroid assignment of K / V sub-vectors (paper Sec. 3.1).
//
// argmin_c ||x - c||^2 = argmax_c (x.c - ||c||^2 / 2).  The comparison value of 32 tokens against 32 centroids
// comes out of the matrix core directly: v_mfma_f32_32x32x16_f16 has 16 k slots, the sub-vector fills 4 or 8 of them
// and three more carry -||c||^2/2 split into three fp16 terms (hi + mid + lo reproduce the fp32 value) against ones
// on the token side; for 16-channel sub-vectors the three terms go through a second MFMA.  Centroids sit on the MFMA
// row axis and tokens on the column axis: a lane then owns one token and sees 16 centroid scores per tile in its
// accumulator registers, which makes the running arg-max a per-lane affair: it narrows the winner down to a quad of
// four neighbouring centroids, whose scores are then looked at once more.  Lanes l and l+32 hold complementary centroid
// subsets of the same token and are combined once per sub-space.  Ties resolve to the lower centroid index (strict '>'
// while indices ascend, explicit index compare across the lane pair).
//
// A workgroup (8 waves, two per CU) owns four neighbouring sub-spaces of one KV head -- their four code bytes are one
// word -- keeps their centroids in LDS in operand layout together with the three norm terms per centroid, and walks over
// 32-token blocks; token sub-vectors are loaded straight from global memory in MFMA operand layout, one block ahead.
// Splitting by sub-spaces and not by tokens alone keeps the chip busy for short inputs: a wave's unit is 32 tokens x 4
// sub-spaces.
//
// Bound: VALU issue.  Per tile of 32 x 32 a wave spends 8 instructions on the maximum, 4 on the bookkeeping and, spread
// over the tiles of a sub-space, about 7 on settling the winner: some 20 at 4.35 clocks, beside which the matrix
// instruction costs 8 more.  8 heads x 32768 tokens, one call, d_sub 4 / 8 / 16: 156 / 82 / 53 us with one workgroup per
// head's whole codebook and a group's eight scores kept by selects, 104 / 57 / 39 us now; 2003 tokens: 77 / 39 / 23 us
// then, 10 now.
#include "common.h"

namespace antkv {

namespace {

// maxima of finite scores; this file is compiled with -fno-honor-nans so that the chains below become
// v_max3_f32 / v_max_f32 without NaN canonicalisation of the MFMA results
__device__ __forceinline__ float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
__device__ __forceinline__ float max2f(float a, float b) { return fmaxf(a, b); }

__device__ __forceinline__ float dot8(const half8_t& a, const half8_t& b, float acc)
{
    acc = __builtin_amdgcn_fdot2(half2_t{a[0], a[1]}, half2_t{b[0], b[1]}, acc, false);
    acc = __builtin_amdgcn_fdot2(half2_t{a[2], a[3]}, half2_t{b[2], b[3]}, acc, false);
    acc = __builtin_amdgcn_fdot2(half2_t{a[4], a[5]}, half2_t{b[4], b[5]}, acc, false);
    return __builtin_amdgcn_fdot2(half2_t{a[6], a[7]}, half2_t{b[6], b[7]}, acc, false);
}

typedef float pair_t __attribute__((ext_vector_type(2)));

// lanes 0-31: a's value of either half-wave in (a, b), lanes 32-63: b's
__device__ __forceinline__ void cross(uint32_t& a, uint32_t& b)
{
    const uint2_t r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

constexpr int kEncThreads = 512;
constexpr int kEncWaves = kEncThreads / 64;
constexpr int kQuad = 4;               // sub-spaces of a workgroup
constexpr float kNormScale = 16.f;     // see the norm terms in the kernel: sub-vector norms up to ||c||^2 = 2.09e6 stay finite
constexpr float kNormLimit = 2.f * 65520.f * kNormScale;               // from here on the first term rounds to infinity

// LDS layout per sub-vector width (halfs per centroid): the A operand of a lane is 8 consecutive halfs
//   d = 4   one array  [4][256][8]  = {c0..c3, n_hi, n_mid, n_lo, 0}: lanes 0-31 read it, lanes 32-63 multiply by zero
//   d = 8   two arrays [4][256][8]: the centroid (lanes 0-31) and {n_hi, n_mid, n_lo, 0 x 5} (lanes 32-63)
//   d = 16  the centroid [4][256][16] (lanes 0-31 the first 8 channels, lanes 32-63 the rest) and a second array
//           [4][256][4] = {n_hi, n_mid, n_lo, 0} for the second MFMA
// The four rows of a group (centroids 4 i .. 4 i + 3) are permuted by a xor with swizzle(i): the lanes of a gather that
// reads row e of a different group each then meet all bank quads and not a quarter of them.
constexpr int enc_row(int d) { return d == 16 ? 16 : 8; }                                // halfs of a row
constexpr int enc_a_halfs(int d) { return kQuad * kC * (d == 4 ? 8 : 16); }
constexpr int enc_n_halfs(int d) { return d == 16 ? kQuad * kC * 4 : 8; }
template <int DSUB>
__device__ __forceinline__ int swizzle(int group) { return (DSUB == 16 ? group >> 1 : group >> 2) & 3; }

template <int DSUB>
__global__ __launch_bounds__(kEncThreads, 4) void encode_kernel(
    const half_t* __restrict__ x, int64_t xs_b, int64_t xs_h, int64_t xs_t, int64_t n_tok,
    const half_t* __restrict__ cb, uint8_t* __restrict__ codes, int64_t N_cap, int64_t token_offset,
    int B, int Hkv, int chunks)
{
    constexpr int M = kD / DSUB;
    constexpr int NQ = M / kQuad;
    constexpr int kRow = enc_row(DSUB);
    constexpr int kPlane = kQuad * kC * 8;                                             // d = 8: the second array inside s_a
    __shared__ __attribute__((aligned(256))) half_t s_a[enc_a_halfs(DSUB)];            // see above
    __shared__ __attribute__((aligned(16))) half_t s_n[enc_n_halfs(DSUB)];             // d = 16 only: norm terms,
    __shared__ __attribute__((aligned(16))) float s_f[kQuad * kC];                     // -||c||^2 / 2 in fp32
    __shared__ uint64_t s_good[kQuad * kC / 64];                                       // centroids within the norm limit
    static_assert(kQuad * kC / 64 == 16, "16 lanes read the words");
    const int tid = threadIdx.x;
    // heads fastest: with 8 heads each XCD works on one, and the workgroups that read the same token rows share its L2
    const int g = blockIdx.x % Hkv, quad = (blockIdx.x / Hkv) % NQ, chunk = blockIdx.x / (Hkv * NQ);

    // ---- the quad's centroids into LDS, with -||c||^2/2 as three fp16 terms per centroid
    const half_t* src = cb + ((size_t)g * M + quad * kQuad) * kC * DSUB;
    // row e = (sub-space, centroid) takes centroid `from`; false if that one is beyond the norm limit (or not finite)
    auto stage = [&](int e, int from) -> bool {
        half_t* row = s_a + (e ^ swizzle<DSUB>(e >> 2)) * kRow;
        float cf[DSUB];
        if constexpr (DSUB == 4) {
            const half4_t v = *(const half4_t*)(src + from * 4);
#pragma unroll
            for (int t = 0; t < 4; ++t) cf[t] = (float)v[t];
        } else {
#pragma unroll
            for (int u = 0; u < DSUB / 8; ++u) {
                const half8_t v = *(const half8_t*)(src + from * DSUB + 8 * u);
#pragma unroll
                for (int t = 0; t < 8; ++t) cf[8 * u + t] = (float)v[t];
                *(half8_t*)(row + 8 * u) = v;
            }
        }
        float nn = 0.f;
#pragma unroll
        for (int t = 0; t < DSUB; ++t) nn = fmaf(cf[t], cf[t], nn);
        // (stored divided by kNormScale and met by kNormScale in the token operand: a power of two, so nothing is
        // rounded, and -||c||^2/2 stays finite in fp16 up to ||c||^2 = 2 * 65504 * kNormScale)
        const float nv = -0.5f * nn * (1.0f / kNormScale);
        const half_t n_hi = (half_t)nv;
        const float r1 = nv - (float)n_hi;
        const half_t n_mid = (half_t)r1;
        const half_t n_lo = (half_t)(r1 - (float)n_mid);
        const half_t z = (half_t)0.f;
        if constexpr (DSUB == 4) {
            *(half8_t*)row = half8_t{(half_t)cf[0], (half_t)cf[1], (half_t)cf[2], (half_t)cf[3], n_hi, n_mid, n_lo, z};
        } else if constexpr (DSUB == 8) {
            *(half8_t*)(row + kPlane) = half8_t{n_hi, n_mid, n_lo, z, z, z, z, z};
        } else {
            *(half4_t*)(s_n + e * 4) = half4_t{n_hi, n_mid, n_lo, z};
        }
        s_f[e] = -0.5f * nn;
        return __float_as_uint(nn) < __float_as_uint(kNormLimit);      // (as integers: a NaN is above every number)
    };
#pragma unroll
    for (int e = tid; e < kQuad * kC; e += kEncThreads) {
        const uint64_t good = __ballot(stage(e, e));
        if ((tid & 63) == 0) s_good[e >> 6] = good;
    }

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const half_t one = (half_t)kNormScale, zero = (half_t)0.f;        // multiplies the three norm terms
    const half8_t ones3 = {one, one, one, zero, zero, zero, zero, zero};
    const half8_t zeros = {zero, zero, zero, zero, zero, zero, zero, zero};
    const half8_t bn = (DSUB == 16 && h == 0) ? ones3 : zeros;        // d = 16: token side of the norm terms
    const int64_t blocks_per_b = (n_tok + 31) / 32;
    const int64_t total = (int64_t)B * blocks_per_b;
    // token operands of a block's four sub-spaces: the sub-vector in the k slots of the centroid, ones against the
    // three norm terms
    auto fetch = [&](int64_t unit, half8_t (&bx)[kQuad]) {
        const int64_t b = unit / blocks_per_b;
        const int64_t tok = (unit % blocks_per_b) * 32 + n;
        const half_t* xr = x + b * xs_b + (int64_t)g * xs_h + (tok < n_tok ? tok : n_tok - 1) * xs_t + quad * kQuad * DSUB;
#pragma unroll
        for (int mm = 0; mm < kQuad; ++mm) {
            if constexpr (DSUB == 4) {
                bx[mm] = zeros;
                if (h == 0) {
                    const half4_t v = *(const half4_t*)(xr + mm * 4);
                    bx[mm] = half8_t{v[0], v[1], v[2], v[3], one, one, one, zero};
                }
            } else if constexpr (DSUB == 8) {
                bx[mm] = ones3;
                if (h == 0) bx[mm] = *(const half8_t*)(xr + mm * 8);
            } else {
                bx[mm] = *(const half8_t*)(xr + mm * 16 + 8 * h);
            }
        }
    };
    // this lane's A-operand rows: n of every tile (d = 4, 8: the swizzle alternates between even and odd tiles)
    const int my_k = DSUB == 16 ? 8 * h : (DSUB == 8 ? kPlane * h : 0);
    const half_t* ap[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) ap[i] = s_a + ((32 * i + n) ^ swizzle<DSUB>((32 * i + n) >> 2)) * kRow + my_k;
    const half_t* an = s_n + n * 4;                                   // d = 16 only

    half8_t bx[kQuad];
    int64_t unit = (int64_t)wave * chunks + chunk;
    if (unit < total) fetch(unit, bx);
    __syncthreads();
    // Centroids beyond the norm limit are never chosen: their terms, which are infinities and NaN, give way to a copy of the
    // sub-space's first good centroid.  A copy behind it loses the tie; one before it is told by its index.
    int first_good[kQuad / 2] = {0, 0};                               // of sub-space 2 i (lanes 0-31) or 2 i + 1
    if (__builtin_expect(__any(s_good[lane & 15] != ~0ull), 0)) {     // (the same in every wave)
        int first[kQuad];
#pragma unroll
        for (int mm = 0; mm < kQuad; ++mm) {
            first[mm] = 0;
            for (int i = kC / 64 - 1; i >= 0; --i) {
                const uint64_t good = s_good[mm * (kC / 64) + i];
                if (good != 0ull) first[mm] = 64 * i + __builtin_ctzll(good);
            }
            first[mm] = __builtin_amdgcn_readfirstlane(first[mm]);
        }
        for (int e = tid; e < kQuad * kC; e += kEncThreads)
            if ((s_good[e >> 6] >> (e & 63) & 1) == 0) stage(e, (e & ~(kC - 1)) + first[e / kC]);
#pragma unroll
        for (int i = 0; i < kQuad / 2; ++i) first_good[i] = h ? first[2 * i + 1] : first[2 * i];
        __syncthreads();
    }
    while (unit < total) {
        const int64_t next = unit + (int64_t)chunks * kEncWaves;
        half8_t nx[kQuad];
        fetch(next < total ? next : unit, nx);
        float16_t acc[2];
        half8_t a[2];
        half4_t a4[2];
        auto operand = [&](int s) {                                    // step s: sub-space s / 8, tile s % 8
            a[s & 1] = *(const half8_t*)(ap[s & 1] + (s >> 1) * 64 * kRow);
            if constexpr (DSUB == 16) a4[s & 1] = *(const half4_t*)(an + s * 32 * 4);
        };
        auto scores = [&](int s) {
            float16_t z;
#pragma unroll
            for (int r = 0; r < 16; ++r) z[r] = 0.f;
            acc[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[s & 1], bx[s >> 3], z, 0, 0, 0);
            if constexpr (DSUB == 16) {
                const half4_t v = a4[s & 1];
                const half8_t a2 = {v[0], v[1], v[2], v[3], zero, zero, zero, zero};
                acc[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, bn, acc[s & 1], 0, 0, 0);
            }
        };
        // Running maximum over tiles of 16 candidates per lane: a chain of max3 over the best so far and four quads (rows
        // 8 q + 4 h .. + 3).  When a tile raises it (strictly, so the lowest tile wins ties) the tile's id and the chain's value
        // after each of the first three quads are kept, by moves under the lanes' mask (every lane is active before and
        // after).  The next tile's product is in flight meanwhile, with its operand read one tile earlier still.
        pair_t keep[kQuad];                                            // chain after quads 0, 1 of the best tile,
        float keep2[kQuad], best[kQuad];                               // after quad 2, and its end
        int tile[kQuad];
        operand(0);
        operand(1);
        scores(0);
#pragma unroll
        for (int mm = 0; mm < kQuad; ++mm) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int s = 8 * mm + t;
                if (s + 1 < 8 * kQuad) scores(s + 1);
                if (s + 2 < 8 * kQuad) operand(s + 2);
                __builtin_amdgcn_sched_barrier(0);
                const float16_t& v = acc[s & 1];
                pair_t lo;
                lo[0] = max3f(t == 0 ? max2f(v[0], v[1]) : max3f(best[mm], v[0], v[1]), v[2], v[3]);
                lo[1] = max3f(max3f(lo[0], v[4], v[5]), v[6], v[7]);
                const float hi = max3f(max3f(lo[1], v[8], v[9]), v[10], v[11]);
                const float top = max3f(max3f(hi, v[12], v[13]), v[14], v[15]);
                if (t == 0) {
                    keep[mm] = lo;
                    keep2[mm] = hi;
                    tile[mm] = 0;
                } else {
                    asm volatile("v_cmpx_gt_f32 vcc, %6, %7\n\tv_mov_b64 %0, %3\n\tv_mov_b32 %1, %4\n\tv_mov_b32 %2, %5\n\ts_mov_b64 exec, -1"
                                 : "+v"(keep[mm]), "+v"(keep2[mm]), "+v"(tile[mm])
                                 : "v"(lo), "v"(hi), "n"(t), "v"(top), "v"(best[mm])
                                 : "vcc");
                }
                best[mm] = top;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // The winner is in the first quad whose chain value is the maximum.  Two sub-spaces are settled at once, lanes 0-31 for the
        // first and 32-63 for the second: the token's two candidates (equal scores: the lower quad) change places between
        // the half-waves, as the sub-vectors do, and a lane scores the four centroids of its quad with packed dot products
        // (v_dot2_f32_f16) and takes the lowest index among equals.
        uint32_t pair_codes[kQuad / 2];
#pragma unroll
        for (int pr = 0; pr < kQuad / 2; ++pr) {
            uint32_t grp[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int mm = 2 * pr + i;
                const int q = (keep[mm][0] < best[mm] ? 1 : 0) + (keep[mm][1] < best[mm] ? 1 : 0) + (keep2[mm] < best[mm] ? 1 : 0);
                grp[i] = (uint32_t)(8 * tile[mm] + 2 * q + h);
            }
            uint32_t b0 = __float_as_uint(best[2 * pr]), b1 = __float_as_uint(best[2 * pr + 1]);
            cross(b0, b1);                                             // of this lane's sub-space: lower, upper half-wave
            cross(grp[0], grp[1]);
            const float top0 = __uint_as_float(b0), top1 = __uint_as_float(b1);
            const bool up = top1 > top0 || (top1 == top0 && grp[1] < grp[0]);
            const int gr = (int)(up ? grp[1] : grp[0]);                // centroids 4 gr .. 4 gr + 3
            uint4_t x0 = __builtin_bit_cast(uint4_t, bx[2 * pr]), x1 = __builtin_bit_cast(uint4_t, bx[2 * pr + 1]);
#pragma unroll
            for (int i = 0; i < (DSUB == 4 ? 2 : 4); ++i) {            // x0: channels 0 .. 7, x1 (d = 16): the others
                uint32_t a0 = x0[i], a1 = x1[i];
                cross(a0, a1);
                x0[i] = a0;
                x1[i] = a1;
            }
            const int sub = (2 * pr + h) * kC;
            const half_t* rows = s_a + (sub + 4 * gr) * kRow;
            const int at = swizzle<DSUB>(gr) * kRow;
            const float4_t nrm = *(const float4_t*)(s_f + sub + 4 * gr);
            float sc[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const half_t* row = rows + (at ^ (e * kRow));
                if constexpr (DSUB == 4) {
                    const half4_t c = *(const half4_t*)row;
                    const half4_t xv = __builtin_bit_cast(half4_t, uint2_t{x0[0], x0[1]});
                    sc[e] = __builtin_amdgcn_fdot2(half2_t{c[0], c[1]}, half2_t{xv[0], xv[1]}, nrm[e], false);
                    sc[e] = __builtin_amdgcn_fdot2(half2_t{c[2], c[3]}, half2_t{xv[2], xv[3]}, sc[e], false);
                } else {
                    sc[e] = dot8(*(const half8_t*)row, __builtin_bit_cast(half8_t, x0), nrm[e]);
                    if constexpr (DSUB == 16) sc[e] = dot8(*(const half8_t*)(row + 8), __builtin_bit_cast(half8_t, x1), sc[e]);
                }
            }
            const float s_max = max2f(max3f(sc[0], sc[1], sc[2]), sc[3]);
            const int e = sc[0] == s_max ? 0 : (sc[1] == s_max ? 1 : (sc[2] == s_max ? 2 : 3));
            const int code = 4 * gr + e;
            pair_codes[pr] = (uint32_t)(code > first_good[pr] ? code : first_good[pr]);
        }
        uint32_t word = pair_codes[0] | pair_codes[1] << 16, word_hi = word;
        cross(word, word_hi);                                          // sub-spaces 0 and 2, 1 and 3
        word |= word_hi << 8;
        const int64_t b = unit / blocks_per_b, tok = (unit % blocks_per_b) * 32 + n;
        if (tok < n_tok && h == 0)
            *(uint32_t*)(codes + (((int64_t)b * Hkv + g) * N_cap + token_offset + tok) * M + kQuad * quad) = word;
#pragma unroll
        for (int mm = 0; mm < kQuad; ++mm) bx[mm] = nx[mm];
        unit = next;
    }
}

}  // namespace

hipError_t launch_encode(const Geom& g, const half_t* x, int64_t xs_b, int64_t xs_h, int64_t xs_t, int64_t n_tok,
                         const half_t* cb, uint8_t* codes, int64_t N_cap, int64_t token_offset, hipStream_t st)
{
    if (n_tok == 0 || g.B == 0) return hipSuccess;
    // two workgroups per CU in total; a workgroup takes every chunks-th block, wave by wave, so that a last uneven round
    // spreads over all of them
    const int64_t blocks = (int64_t)g.B * ((n_tok + 31) / 32);
    const int groups = g.Hkv * (g.M / kQuad);
    int64_t chunks = (512 + groups - 1) / groups;
    if (chunks > blocks) chunks = blocks;
#define ANTKV_ENC(DS)                                                                                              \
    hipLaunchKernelGGL(encode_kernel<DS>, dim3((unsigned)(groups * chunks)), dim3(kEncThreads), 0, st, x, xs_b, xs_h, xs_t, \
                       n_tok, cb, codes, N_cap, token_offset, g.B, g.Hkv, (int)chunks)
    if (g.d == 4) ANTKV_ENC(4);
    else if (g.d == 8) ANTKV_ENC(8);
    else ANTKV_ENC(16);
#undef ANTKV_ENC
    return hipGetLastError();
}

}  // namespace antkv
