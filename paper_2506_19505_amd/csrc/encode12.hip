// VQ encode for the 12-bit codebooks (paper Sec. 3.1 with the 4096-centroid settings of Sec. 4: d32, "0.375 bit", and
// d16, "0.75 bit"): nearest of 4096 centroids for each 32- or 16-channel sub-vector, the M = 4 or 8 codes of a token
// row packed into 6 or 12 bytes.
//
// argmin_c ||x - c||^2 = argmax_c (x.c - ||c||^2 / 2).  A workgroup (16 waves, one per CU) takes two neighbouring
// sub-spaces -- their two codes are three whole bytes -- for up to 64 (d32: 48) groups of 32 tokens, one sub-space after the other,
// with the sub-space's centroids in LDS in MFMA operand order (d16: all 128 KB; d32: one half of 2048 after the other)
// and -||c||^2/2 beside them.
//   level 1  per 32 tokens x 32 centroids: v_mfma_f32_32x32x16_f16 (one per 16 channels) with centroids on the row
//            axis and tokens on the column axis, the C operand being -||c||^2/2.  A lane owns one token and 16 of the 32
//            centroid scores; it keeps the best score and the tile it came from (a max3 tree, one compare, one select:
//            ten VALU instructions per 16 candidates, and one or two of addressing).  A wave holds up to four (three) token groups, which share every
//            operand it reads from LDS.
//   level 2  the 16 scores of the winning tile and half-wave again, with packed dot products (v_dot2_f32_f16), eight in
//            each of the token's two lanes; lanes start at different rows so that the reads spread over the banks.
// Ties go to the lower index: level 1 keeps the first tile, level 2 compares (score, index), and when both half-waves
// reach the same score in the same tile, level 2 looks at all 32.  Both levels are fp32-accurate; they may order two
// centroids differently only when their scores agree to fp32 rounding.
//
// Bound: VALU issue first: level 1 takes 50 clocks of it per tile and group beside 32 or 64 of MFMA.  Over the whole kernel a tile
// and group takes 81 clocks (d16, 32768 tokens; VALU busy 73 %, MFMA 39 %): the rest is level 2 and bringing a sub-space's
// centroids into LDS, behind barriers with nothing running beside it.  With the centroids read from the
// L2 by four-wave workgroups that walked all sub-spaces, short inputs left one wave per SIMD and nothing hid the reads:
// 8 heads x 9001 tokens, d16, took 381 us; this one 104 (32768 tokens: 760 to 338; d32: 578 to 305).
#include "common.h"

#include <type_traits>

namespace antkv {

namespace {

constexpr int kE12Waves = 16;
constexpr int kE12Threads = kE12Waves * 64;
constexpr int e12_groups(int d) { return d == 32 ? 3 : 4; }   // token groups of a wave (registers: 128 at 16 waves)
constexpr int kC12 = 4096;
constexpr float kE12Low = -3.0e38f;

// d = 16: the whole sub-space in LDS; d = 32: halves of 2048 centroids
constexpr int e12_parts(int d) { return d == 32 ? 2 : 1; }
constexpr size_t e12_lds(int d) { return 131072 + (size_t)(kC12 / e12_parts(d)) * 4 + kE12Threads * 8; }

__device__ __forceinline__ float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

__device__ __forceinline__ float dot8(const half8_t& a, const half8_t& b, float acc)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const half2_t x = {a[2 * i], a[2 * i + 1]}, y = {b[2 * i], b[2 * i + 1]};
        acc = __builtin_amdgcn_fdot2(x, y, acc, false);
    }
    return acc;
}

__device__ __forceinline__ half8_t other_half(const half8_t& v)          // the same registers of lane ^ 32
{
    uint4_t u = __builtin_bit_cast(uint4_t, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = (uint32_t)__shfl_xor((int)u[i], 32, 64);
    return __builtin_bit_cast(half8_t, u);
}

template <int CTRL>
__device__ __forceinline__ float quad_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// grid = (B * Hkv, token chunks, M / 2).  A chunk is groups_per_wg groups of 32 tokens; with few groups, 1 << cs_log2
// waves share a group and each walks its share of the tiles (then a wave has one group).
template <int DS>
__global__ __launch_bounds__(kE12Threads) void encode12_kernel(
    const half_t* __restrict__ x, int64_t xs_b, int64_t xs_h, int64_t xs_t, int64_t n_tok,
    const half_t* __restrict__ cb, uint8_t* __restrict__ codes, int64_t N_cap, int64_t token_offset, int Hkv,
    int groups_per_wg, int cs_log2)
{
    constexpr int M = kD / DS;
    constexpr int kGroups = e12_groups(DS);
    constexpr int NU = DS / 8;                                      // 16-byte chunks of a sub-vector
    constexpr int NS = DS / 16;                                     // MFMA k-steps
    constexpr int kParts = e12_parts(DS);
    constexpr int kHC = kC12 / kParts;                              // centroids in LDS at a time
    constexpr int kHT = kHC / 32;                                   // tiles of 32
    constexpr int kTileB = 64 * DS;                                 // bytes of a tile: [k-step][channel half][32 rows][16]
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    float* s_nrm = (float*)(lds + 131072);                          // -||c||^2 / 2
    float* s_best = s_nrm + kHC;                                    // [wave][lane], only with shared groups
    int* s_blk = (int*)(s_best + kE12Threads);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, kh = lane >> 5;
    const int b = blockIdx.x / Hkv, g = blockIdx.x % Hkv;
    const half_t* xbase = x + (int64_t)b * xs_b + (int64_t)g * xs_h;
    const int64_t all_groups = (n_tok + 31) >> 5;
    const int64_t g0 = (int64_t)blockIdx.y * groups_per_wg;
    const int n_g = (int)(all_groups - g0 < groups_per_wg ? all_groups - g0 : groups_per_wg);
    const int share = wave & ((1 << cs_log2) - 1), slot = wave >> cs_log2, slots = kE12Waves >> cs_log2;
    const int ng = n_g > slot ? (n_g - slot + slots - 1) / slots : 0;   // groups slot, slot + slots, ... of the chunk
    const int t_lo = share * (kHT >> cs_log2), t_hi = t_lo + (kHT >> cs_log2);

    auto token = [&](int i) -> int64_t { return (g0 + slot + (int64_t)i * slots) * 32 + n; };   // this lane's token of group i
    uint32_t code[kGroups];                                      // the pair's codes: first | second << 12
#pragma unroll
    for (int i = 0; i < kGroups; ++i) code[i] = 0;

#pragma unroll 1
    for (int mm = 0; mm < 2; ++mm) {
        const int m = 2 * blockIdx.z + mm;
        half8_t xb[kGroups][NS];                                 // B operand: k-step s holds channels 16 s + 8 kh .. + 7
        float best[kGroups];
        int blk[kGroups];
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            best[i] = kE12Low;
            blk[i] = 0;
            if (i < ng) {
                const int64_t t = token(i);
                const half_t* xr = xbase + (t < n_tok ? t : n_tok - 1) * xs_t + m * DS + 8 * kh;
#pragma unroll
                for (int s = 0; s < NS; ++s) xb[i][s] = *(const half8_t*)(xr + 16 * s);
            }
        }
#pragma unroll 1
        for (int part = 0; part < kParts; ++part) {
            // ---- centroids into LDS: neighbouring lanes take the chunks of one centroid
            const half_t* cbm = cb + (((int64_t)g * M + m) * kC12 + part * kHC) * DS;
            half8_t stage[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) stage[i] = *(const half8_t*)(cbm + (int64_t)(tid + i * kE12Threads) * 8);
            __syncthreads();                                        // the previous centroids are no longer read
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = tid + i * kE12Threads, c = e / NU, u = e % NU;
                *(half8_t*)(lds + (c >> 5) * kTileB + u * 512 + (c & 31) * 16) = stage[i];
                float s = dot8(stage[i], stage[i], 0.f);
                s = quad_add<0xB1>(s);                              // quad lanes 1 0 3 2
                if constexpr (NU == 4) s = quad_add<0x4E>(s);       // quad lanes 2 3 0 1
                if (u == 0) s_nrm[c] = -0.5f * s;
            }
            __syncthreads();
            // ---- level 1
            auto walk = [&](auto count) {
                constexpr int NG = decltype(count)::value;
                const unsigned char* ap = lds + t_lo * kTileB + lane * 16;
                const float* np = s_nrm + t_lo * 32 + 4 * kh;
                half8_t a[NS];
                float16_t nb;
                auto operands = [&]() {
#pragma unroll
                    for (int s = 0; s < NS; ++s) a[s] = *(const half8_t*)(ap + s * 1024);
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd) {                // rows 8 qd + 4 kh + e live in register 4 qd + e
                        const float4_t v = *(const float4_t*)(np + 8 * qd);
#pragma unroll
                        for (int e = 0; e < 4; ++e) nb[4 * qd + e] = v[e];
                    }
                };
                float16_t acc[2];
                auto scores = [&](int i) {
                    acc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], xb[i][0], nb, 0, 0, 0);
                    if constexpr (NS == 2) acc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], xb[i][1], acc[i & 1], 0, 0, 0);
                };
                operands();
#pragma unroll 1
                for (int t2 = t_lo; t2 < t_hi; t2 += 2) {           // (two copies of the body: the operand registers alternate)
#pragma unroll
                  for (int t = t2; t < t2 + 2; ++t) {
                    // the next group's product is issued before the current one's scores are looked at, the next tile's
                    // operands are requested after the last product
                    scores(0);
#pragma unroll
                    for (int i = 0; i < NG; ++i) {
                        if (i + 1 < NG) scores(i + 1);
                        if (i + 2 >= NG && i < NG - 1 + (NG == 1)) {
                            ap += kTileB;                           // (one tile past the end: still inside the allocation)
                            np += 32;
                            operands();
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        const float16_t& v = acc[i & 1];
                        float mx = max3f(v[0], v[1], v[2]);
#pragma unroll
                        for (int r = 3; r < 15; r += 2) mx = max3f(mx, v[r], v[r + 1]);
                        mx = max3f(mx, v[15], best[i]);
                        blk[i] = mx > best[i] ? part * kHT + t : blk[i];   // strict: an equal later tile does not replace
                        best[i] = mx;
                        __builtin_amdgcn_sched_barrier(0);
                    }
                  }
                }
            };
            if (ng == 1) walk(std::integral_constant<int, 1>{});
            else if (ng == 2) walk(std::integral_constant<int, 2>{});
            else if (ng == 3) walk(std::integral_constant<int, 3>{});
            else if (ng == 4) walk(std::integral_constant<int, kGroups>{});
            if (cs_log2) {                                          // the group's waves agree on the best tile
                s_best[tid] = best[0];
                s_blk[tid] = blk[0];
                __syncthreads();
                const int w0 = (slot << cs_log2) * 64 + lane;
                best[0] = s_best[w0];
                blk[0] = s_blk[w0];
                for (int w = 1; w < (1 << cs_log2); ++w) {
                    const float v = s_best[w0 + 64 * w];
                    const int k2 = s_blk[w0 + 64 * w];
                    if (v > best[0] || (v == best[0] && k2 < blk[0])) { best[0] = v; blk[0] = k2; }
                }
            }
            // ---- level 2
#pragma unroll
            for (int i = 0; i < kGroups; ++i) {
                if (i >= ng) continue;
                const float ob = __shfl_xor(best[i], 32, 64);
                const int oblk = __shfl_xor(blk[i], 32, 64);
                const bool tie = ob == best[i] && oblk == blk[i];
                const bool other = ob > best[i] || (ob == best[i] && oblk < blk[i]);
                const int win = other ? oblk : blk[i];
                const bool here = win >= part * kHT;                // (a tile of the first half was settled there)
                const int wt = here ? win - part * kHT : 0;
                half8_t xf[NU];
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const half8_t o = other_half(xb[i][s]);
                    xf[2 * s] = kh ? o : xb[i][s];
                    xf[2 * s + 1] = kh ? xb[i][s] : o;
                }
                float bv = kE12Low;
                int bc = 0;
                const int passes = __any(tie) ? 2 : 1;
#pragma unroll 1
                for (int p = 0; p < passes; ++p) {
                    const int hw = kh ^ (int)other ^ p;             // the half-wave whose candidates are looked at
#pragma unroll 4
                    for (int j = 0; j < 8; ++j) {
                        const int r = (2 * j + kh + 2 * n) & 15;
                        const int row = 8 * (r >> 2) + 4 * hw + (r & 3);
                        const unsigned char* cp = lds + wt * kTileB + row * 16;
                        float s = s_nrm[wt * 32 + row];
#pragma unroll
                        for (int u = 0; u < NU; ++u) s = dot8(*(const half8_t*)(cp + u * 512), xf[u], s);
                        if (s > bv || (s == bv && row < bc)) { bv = s; bc = row; }
                    }
                }
                const float ov = __shfl_xor(bv, 32, 64);
                const int oc = __shfl_xor(bc, 32, 64);
                if (ov > bv || (ov == bv && oc < bc)) bc = oc;
                const uint32_t c = (uint32_t)(win * 32 + bc);
                if (here) code[i] = mm ? (code[i] & 0xfffu) | c << 12 : c;
            }
        }
    }
    // codes little-endian, code m at bits 12 m .. 12 m + 11 of the row: the pair's three bytes
    if (kh == 0 && share == 0) {
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            if (i < ng && token(i) < n_tok) {
                uint8_t* dst = codes + (((int64_t)b * Hkv + g) * N_cap + token_offset + token(i)) * (M * 3 / 2) + 3 * blockIdx.z;
                dst[0] = (uint8_t)code[i];
                dst[1] = (uint8_t)(code[i] >> 8);
                dst[2] = (uint8_t)(code[i] >> 16);
            }
        }
    }
}

// Chunks per (sequence, KV head, pair): the waves of a CU share its issue slots, so a chunk's time grows with its groups
// (plus about three groups' worth of staging and set-up) and the launch takes as many rounds as its workgroups fill the
// 256 CUs.
int e12_chunks(int64_t groups, int64_t wgs_per_chunk, int groups_per_wave)
{
    const int64_t lo = (groups + kE12Waves * groups_per_wave - 1) / (kE12Waves * groups_per_wave);
    int64_t hi = lo + 16 > 512 / wgs_per_chunk ? lo + 16 : 512 / wgs_per_chunk;
    if (hi > groups) hi = groups;
    int64_t best_w = lo, best_cost = INT64_MAX;
    for (int64_t w = lo; w <= hi; ++w) {
        const int64_t cost = ((wgs_per_chunk * w + 255) / 256) * ((groups + w - 1) / w + 3);
        if (cost < best_cost) { best_cost = cost; best_w = w; }
    }
    return (int)best_w;
}

}  // namespace

template <int DS>
static hipError_t launch_encode12_t(const Geom& g, const half_t* x, int64_t xs_b, int64_t xs_h, int64_t xs_t,
                                    int64_t n_tok, const half_t* cb, uint8_t* codes, int64_t N_cap,
                                    int64_t token_offset, hipStream_t st)
{
    static OncePerDevice once;
    const hipError_t setup = allow_lds(once, (const void*)encode12_kernel<DS>, e12_lds(DS));
    if (setup != hipSuccess) return setup;
    const int64_t groups = (n_tok + 31) / 32;
    const int chunks = e12_chunks(groups, (int64_t)g.B * g.Hkv * (g.M / 2), e12_groups(DS));
    const int per_wg = (int)((groups + chunks - 1) / chunks);
    const int used = (int)((groups + per_wg - 1) / per_wg);
    int cs_log2 = 0;
    while (cs_log2 < 4 && (per_wg << (cs_log2 + 1)) <= kE12Waves) ++cs_log2;
    hipLaunchKernelGGL(encode12_kernel<DS>, dim3((unsigned)(g.B * g.Hkv), (unsigned)used, (unsigned)(g.M / 2)),
                       dim3(kE12Threads), e12_lds(DS), st, x, xs_b, xs_h, xs_t, n_tok, cb, codes, N_cap, token_offset, g.Hkv,
                       per_wg, cs_log2);
    return hipGetLastError();
}

hipError_t launch_encode12(const Geom& g, const half_t* x, int64_t xs_b, int64_t xs_h, int64_t xs_t, int64_t n_tok,
                           const half_t* cb, uint8_t* codes, int64_t N_cap, int64_t token_offset, hipStream_t st)
{
    if (g.B == 0) return hipSuccess;
    // the token chunks (of at least 1536 tokens when there are many) are the grid's second axis, which ends at 65536
    constexpr int64_t kMost = 1 << 26;
    for (int64_t t = 0; t < n_tok; t += kMost) {
        const int64_t n = n_tok - t < kMost ? n_tok - t : kMost;
        const hipError_t e =
            g.d == 32 ? launch_encode12_t<32>(g, x + t * xs_t, xs_b, xs_h, xs_t, n, cb, codes, N_cap, token_offset + t, st)
                      : launch_encode12_t<16>(g, x + t * xs_t, xs_b, xs_h, xs_t, n, cb, codes, N_cap, token_offset + t, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace antkv
