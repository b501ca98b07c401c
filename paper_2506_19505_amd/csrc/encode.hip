// VQ encode: nearest-centroid assignment of K / V sub-vectors (paper Sec. 3.1).
//
// argmin_c ||x - c||^2 = argmax_c (x.c - ||c||^2 / 2).  The comparison value of 32 tokens against 32 centroids
// comes out of the matrix core directly: v_mfma_f32_32x32x16_f16 has 16 k slots, the sub-vector fills 4 or 8 of them
// and three more carry -||c||^2/2 split into three fp16 terms (hi + mid + lo reproduce the fp32 value) against ones
// on the token side; 16-channel sub-vectors leave no slot and take -||c||^2/2 as the C operand, read from LDS.  Centroids sit
// on the MFMA row axis and tokens on the column axis: a lane then owns one token and sees 16 centroid scores per tile in its
// accumulator registers, which makes the running arg-max a per-lane affair: it narrows the winner down to a quad of
// four neighbouring centroids, whose scores are then looked at once more.  Lanes l and l+32 hold complementary centroid
// subsets of the same token and are combined once per sub-space.  Ties resolve to the lower centroid index (strict '>'
// while indices ascend, explicit index compare across the lane pair).
//
// A workgroup (8 waves) owns four neighbouring sub-spaces of one KV head, keeps their centroids in LDS in operand layout
// together with the norm terms, and walks over units of 64 tokens, a wave on one sub-space; token sub-vectors are loaded straight
// from global memory in MFMA operand layout, one unit ahead.  Splitting by sub-spaces and not by tokens alone keeps the chip busy
// for short inputs.
//
// Bound: VALU issue.  Per tile of 32 x 32 a wave spends 8 instructions on the maximum, 4 on the bookkeeping and, spread
// over the tiles of a sub-space, about 4 on settling the winner and 2 on the rest, at 4.1 clocks, and the matrix instruction
// costs 9 clocks of issue beside them: 84 of the 96 clocks that a tile takes (d 8).  8 heads x 32768 tokens, one call, d_sub
// 4 / 8 / 16: 118 / 57.5 / 40 us with one wave on four sub-spaces of 32 tokens, both half-waves settling the same winner
// and the norm terms of d 16 in a second matrix instruction; 83 / 45.7 / 31 us now; 2003 tokens 8.0 / 6.0 / 5.7.
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
constexpr int kSlots = kEncWaves / kQuad;                              // units of tokens that it works on at a time
constexpr int NG = 2;                  // groups of 32 tokens of a unit, which share the operands that a wave reads from LDS
constexpr float kNormScale = 16.f;     // see the norm terms in the kernel: sub-vector norms up to ||c||^2 = 2.09e6 stay finite
constexpr float kNormLimit = 2.f * 65520.f * kNormScale;               // from here on the first term rounds to infinity

// LDS layout per sub-vector width: rows of 8 halfs, the A operand of a lane
//   d = 4   one plane  [4][256][8]  = {c0..c3, n_hi, n_mid, n_lo, 0}: lanes 0-31 read it, lanes 32-63 multiply by zero
//   d = 8   two planes [4][256][8]: the centroid (lanes 0-31) and {n_hi, n_mid, n_lo, 0 x 5} (lanes 32-63)
//   d = 16  two planes [4][256][8]: the first 8 channels (lanes 0-31) and the rest (lanes 32-63)
// The four rows of a group (centroids 4 i .. 4 i + 3) are permuted by a xor with swizzle(i): the lanes of a gather that
// reads row e of a different group each then meet all bank quads and not a quarter of them.
constexpr int kRow = 8;                                                // halfs of a row
constexpr int kPlane = kQuad * kC * kRow;
__device__ __forceinline__ int swizzle(int group) { return (group >> 2) & 3; }

// A wave takes one of the workgroup's sub-spaces and the units of its slot.  (waves per SIMD: three workgroups per CU, d = 16 two:
// with three it spills)
template <int DSUB, bool CLEAR>
__global__ __launch_bounds__(kEncThreads, DSUB == 16 ? 4 : 6) void encode_kernel(
    const half_t* __restrict__ x, int64_t xs_b, int64_t xs_h, int64_t xs_t, int64_t n_tok,
    const half_t* __restrict__ cb, uint8_t* __restrict__ codes, int64_t N_cap, int64_t token_offset,
    int Hkv, int chunks, uint32_t units_per_b, uint32_t units, ClearWords clear)
{
    constexpr int M = kD / DSUB;
    constexpr int NQ = M / kQuad;
    __shared__ __attribute__((aligned(256))) half_t s_a[(DSUB == 4 ? 1 : 2) * kPlane];  // see above
    __shared__ __attribute__((aligned(16))) float s_f[kQuad * kC];                     // -||c||^2 / 2
    __shared__ uint64_t s_good[kQuad * kC / 64];                                       // centroids within the norm limit
    static_assert(kQuad * kC / 64 == 16, "16 lanes read the words");
    const int tid = threadIdx.x;
    // heads fastest: with 8 heads each XCD works on one, and the workgroups that read the same token rows share its L2
    const int g = blockIdx.x % Hkv, quad = (blockIdx.x / Hkv) % NQ, chunk = blockIdx.x / (Hkv * NQ);

    // ---- the quad's centroids into LDS, with -||c||^2/2 as three fp16 terms per centroid
    const half_t* src = cb + ((size_t)g * M + quad * kQuad) * kC * DSUB;
    // row e = (sub-space, centroid) takes centroid `from`; false if that one is beyond the norm limit (or not finite)
    auto stage = [&](int e, int from) -> bool {
        half_t* row = s_a + (e ^ swizzle(e >> 2)) * kRow;
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
                *(half8_t*)(row + u * kPlane) = v;
            }
        }
        float nn = 0.f;
#pragma unroll
        for (int t = 0; t < DSUB; ++t) nn = fmaf(cf[t], cf[t], nn);
        s_f[e] = -0.5f * nn;
        // (stored divided by kNormScale and met by kNormScale in the token operand: a power of two, so nothing is
        // rounded, and -||c||^2/2 stays finite in fp16 up to ||c||^2 = 2 * 65504 * kNormScale)
        const float nv = -0.5f * nn * (1.0f / kNormScale);
        const half_t n_hi = (half_t)nv;
        const float r1 = nv - (float)n_hi;
        const half_t n_mid = (half_t)r1;
        const half_t n_lo = (half_t)(r1 - (float)n_mid);
        const half_t z = (half_t)0.f;
        if constexpr (DSUB == 4) *(half8_t*)row = half8_t{(half_t)cf[0], (half_t)cf[1], (half_t)cf[2], (half_t)cf[3], n_hi, n_mid, n_lo, z};
        if constexpr (DSUB == 8) *(half8_t*)(row + kPlane) = half8_t{n_hi, n_mid, n_lo, z, z, z, z, z};
        return __float_as_uint(nn) < __float_as_uint(kNormLimit);      // (as integers: a NaN is above every number)
    };
#pragma unroll
    for (int e = tid; e < kQuad * kC; e += kEncThreads) {
        const uint64_t good = __ballot(stage(e, e));
        if ((tid & 63) == 0) s_good[e >> 6] = good;
    }
    if constexpr (CLEAR)                                               // (asked at run time, 0.4 us of an encode of 500 tokens)
        for (int64_t i = (int64_t)blockIdx.x * kEncThreads + tid; i < clear.n; i += (int64_t)gridDim.x * kEncThreads) clear.at[i] = 0u;

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mm = wave % kQuad;                                      // this wave's sub-space
    const int n = lane & 31, h = lane >> 5;
    const half_t one = (half_t)kNormScale, zero = (half_t)0.f;        // multiplies the three norm terms
    const half8_t ones3 = {one, one, one, zero, zero, zero, zero, zero};
    const half8_t zeros = {zero, zero, zero, zero, zero, zero, zero, zero};
    const half_t* xg = x + (int64_t)g * xs_h + (quad * kQuad + mm) * DSUB;
    // token operands of a unit's groups: the sub-vector in the k slots of the centroid, ones against the three norm terms
    auto fetch = [&](uint32_t unit, half8_t (&bx)[NG]) {
        const uint32_t b = unit / units_per_b;
        const int64_t t0 = (int64_t)(unit - b * units_per_b) * (32 * NG) + n;
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int64_t tok = t0 + 32 * i;
            const half_t* xr = xg + b * xs_b + (tok < n_tok ? tok : n_tok - 1) * xs_t;
            if constexpr (DSUB == 4) {
                bx[i] = zeros;
                if (h == 0) {
                    const half4_t v = *(const half4_t*)xr;
                    bx[i] = half8_t{v[0], v[1], v[2], v[3], one, one, one, zero};
                }
            } else if constexpr (DSUB == 8) {
                bx[i] = ones3;
                if (h == 0) bx[i] = *(const half8_t*)xr;
            } else {
                bx[i] = *(const half8_t*)(xr + 8 * h);
            }
        }
    };
    // this lane's A-operand rows: n of every tile (the swizzle alternates between even and odd tiles)
    const half_t* ap[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        ap[i] = s_a + (mm * kC + ((32 * i + n) ^ swizzle((32 * i + n) >> 2))) * kRow + (DSUB == 4 ? 0 : h * kPlane);
    const float* np = s_f + mm * kC + 4 * h;

    half8_t bx[NG];
    uint32_t unit = (uint32_t)(wave / kQuad) * chunks + chunk;
    if (unit < units) fetch(unit, bx);
    __syncthreads();
    // Centroids beyond the norm limit are never chosen: their terms, which are infinities and NaN, give way to a copy of the
    // sub-space's first good centroid.  A copy behind it loses the tie; one before it is told by its index.
    int first_good = 0;
    if (__builtin_expect(__any(s_good[lane & 15] != ~0ull), 0)) {     // (the same in every wave)
        auto first_of = [&](int sub) {
            int first = 0;
            for (int i = kC / 64 - 1; i >= 0; --i) {
                const uint64_t good = s_good[sub * (kC / 64) + i];
                if (good != 0ull) first = 64 * i + __builtin_ctzll(good);
            }
            return first;
        };
        first_good = first_of(mm);
        for (int e = tid; e < kQuad * kC; e += kEncThreads)
            if ((s_good[e >> 6] >> (e & 63) & 1) == 0) stage(e, (e & ~(kC - 1)) + first_of(e / kC));
        __syncthreads();
    }
#pragma unroll 1
    while (unit < units) {
        const uint32_t next = unit + (uint32_t)chunks * kSlots;
        half8_t nx[NG];
        fetch(next < units ? next : unit, nx);
        const uint64_t active = __builtin_amdgcn_read_exec();
        float16_t acc[2], nb;
        half8_t a[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) nb[r] = 0.f;
        auto operand = [&](int t) {                                    // of tile t; d = 16: the C operand is -||c||^2/2
            a[t & 1] = *(const half8_t*)(ap[t & 1] + (t >> 1) * 64 * kRow);
            if constexpr (DSUB == 16) {
#pragma unroll
                for (int qd = 0; qd < 4; ++qd) {                       // rows 8 qd + 4 h + e live in register 4 qd + e
                    const float4_t v = *(const float4_t*)(np + 32 * t + 8 * qd);
#pragma unroll
                    for (int e = 0; e < 4; ++e) nb[4 * qd + e] = v[e];
                }
            }
        };
        auto scores = [&](int s) {                                     // step s: tile s / NG, group s % NG
            acc[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[(s / NG) & 1], bx[s % NG], nb, 0, 0, 0);
        };
        // Running maximum over tiles of 16 candidates per lane: a chain of max3 over the best so far and four quads (rows
        // 8 q + 4 h .. + 3).  When a tile raises it (strictly, so the lowest tile wins ties) the tile's id and the chain's value
        // after each of the first three quads are kept, by moves under the lanes' mask, which is put back.  The next step's product is in flight meanwhile; a tile's operands serve the wave's NG groups.
        pair_t keep[NG];                                               // chain after quads 0, 1 of the best tile,
        float keep2[NG], best[NG];                                     // after quad 2, and its end
        int tile[NG];
        operand(0);
        if constexpr (DSUB != 16) operand(1);
        scores(0);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                const int s = NG * t + i;
                if (s + 1 < 8 * NG) scores(s + 1);
                if (DSUB == 16 ? (i == NG - 2 && t + 1 < 8) : (i == NG - 1 && t + 2 < 8)) operand(DSUB == 16 ? t + 1 : t + 2);
                __builtin_amdgcn_sched_barrier(0);
                const float16_t& v = acc[s & 1];
                pair_t lo;
                lo[0] = max3f(t == 0 ? max2f(v[0], v[1]) : max3f(best[i], v[0], v[1]), v[2], v[3]);
                lo[1] = max3f(max3f(lo[0], v[4], v[5]), v[6], v[7]);
                const float hi = max3f(max3f(lo[1], v[8], v[9]), v[10], v[11]);
                const float top = max3f(max3f(hi, v[12], v[13]), v[14], v[15]);
                if (t == 0) {
                    keep[i] = lo;
                    keep2[i] = hi;
                    tile[i] = 0;
                } else {
                    asm volatile("v_cmpx_gt_f32 vcc, %6, %7\n\tv_mov_b64 %0, %3\n\tv_mov_b32 %1, %4\n\tv_mov_b32 %2, %5\n\ts_mov_b64 exec, %8"
                                 : "+v"(keep[i]), "+v"(keep2[i]), "+v"(tile[i])
                                 : "v"(lo), "v"(hi), "n"(t), "v"(top), "v"(best[i]), "s"(active)
                                 : "vcc");
                }
                best[i] = top;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // The winner is in the first quad whose chain value is the maximum.  Two groups are settled at once, lanes 0-31 for the
        // first and 32-63 for the second: a token's two candidates (equal scores: the lower quad) change places between
        // the half-waves, as the sub-vectors do, and a lane scores the four centroids of its quad with packed dot products
        // (v_dot2_f32_f16) and takes the lowest index among equals.
        const uint32_t b = unit / units_per_b;
        const int64_t t0 = (int64_t)(unit - b * units_per_b) * (32 * NG) + lane;
        uint8_t* out = codes + (((int64_t)b * Hkv + g) * N_cap + token_offset + t0) * M + kQuad * quad + mm;
#pragma unroll
        for (int pr = 0; pr < NG / 2; ++pr) {
            uint32_t grp[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int i = 2 * pr + j;
                const int q = (keep[i][0] < best[i] ? 1 : 0) + (keep[i][1] < best[i] ? 1 : 0) + (keep2[i] < best[i] ? 1 : 0);
                grp[j] = (uint32_t)(8 * tile[i] + 2 * q + h);
            }
            uint32_t b0 = __float_as_uint(best[2 * pr]), b1 = __float_as_uint(best[2 * pr + 1]);
            cross(b0, b1);                                             // of this lane's token: lower, upper half-wave
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
            const half_t* rows = s_a + (mm * kC + 4 * gr) * kRow;
            const int at = swizzle(gr) * kRow;
            const float4_t nrm = *(const float4_t*)(s_f + mm * kC + 4 * gr);
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
                    if constexpr (DSUB == 16) sc[e] = dot8(*(const half8_t*)(row + kPlane), __builtin_bit_cast(half8_t, x1), sc[e]);
                }
            }
            const float s_max = max2f(max3f(sc[0], sc[1], sc[2]), sc[3]);
            const int e = sc[0] == s_max ? 0 : (sc[1] == s_max ? 1 : (sc[2] == s_max ? 2 : 3));
            const int code = 4 * gr + e;
            if (t0 + 64 * pr < n_tok) out[(int64_t)(64 * pr) * M] = (uint8_t)(code > first_good ? code : first_good);
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) bx[i] = nx[i];
        unit = next;
    }
}

}  // namespace

hipError_t launch_encode(const Geom& g, const half_t* x, int64_t xs_b, int64_t xs_h, int64_t xs_t, int64_t n_tok,
                         const half_t* cb, uint8_t* codes, int64_t N_cap, int64_t token_offset, hipStream_t st, ClearWords clear)
{
    if (n_tok == 0 || g.B == 0) return hipSuccess;
    // Two workgroups per CU, or three (d = 4, 8) where that still leaves a wave several units: 8 heads, d 8, 32768 tokens 47.7 and
    // 45.7 us, 9001 tokens 15.1 and 15.7.  (Units of four groups: 46.3 and 15.5; 3000 tokens 8.1 against 6.9; d 16 spills.)
    const int64_t units_per_b = (n_tok + 32 * NG - 1) / (32 * NG), units = g.B * units_per_b;
    if (units > 0x7fffffffLL) return hipErrorInvalidValue;             // (2^37 tokens)
    const int groups = g.Hkv * (g.M / kQuad);
    const int64_t all = (units + kSlots - 1) / kSlots;
    int64_t chunks = (512 + groups - 1) / groups;
    if (g.d != 16 && all >= 6 * chunks) chunks = (768 + groups - 1) / groups;
    if (chunks > all) chunks = all;
#define ANTKV_ENC(DS, CLEAR)                                                                                       \
    hipLaunchKernelGGL((encode_kernel<DS, CLEAR>), dim3((unsigned)(groups * chunks)), dim3(kEncThreads), 0, st, x, xs_b, xs_h, xs_t, \
                       n_tok, cb, codes, N_cap, token_offset, g.Hkv, (int)chunks, (uint32_t)units_per_b, (uint32_t)units, clear)
    if (clear.n > 0) {
        if (g.d == 4) ANTKV_ENC(4, true);
        else if (g.d == 8) ANTKV_ENC(8, true);
        else ANTKV_ENC(16, true);
    } else {
        if (g.d == 4) ANTKV_ENC(4, false);
        else if (g.d == 8) ANTKV_ENC(8, false);
        else ANTKV_ENC(16, false);
    }
#undef ANTKV_ENC
    return hipGetLastError();
}

}  // namespace antkv
