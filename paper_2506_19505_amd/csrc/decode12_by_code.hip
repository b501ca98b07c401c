// Decode attention over 12-bit VQ codes for long contexts: the values are added up by code.
//
//   sum_t P_h(t) v(t) = sum over (sub-space, code) of W_h[code] * centroid[code],   W_h[code] = sum of P_h over the tokens with that code
//
// so that a token costs a few integer atomics in LDS instead of its 256 bytes of centroids out of the L2.  Two kernels, since
// neither the q . centroid table of the K side (128 KB of int16 entries) nor the sums (two sub-spaces x 4096 codes x four
// heads x 32 bits) leave room for the other:
//   d12_weights_kernel  a workgroup per token range.  Table in LDS (the fp32 scores come from d12_table_kernel), lane = token:
//            unpack the K codes, one table read per sub-space, integer sums, softmax weights against the wave's largest
//            score so far.  The weights go out as fp16, 8 bytes per token, with the reference of every 64 tokens.
//            K-anchored tokens get weight zero; V-anchored ones are marked by the sign.  Then the K list's entries, 16
//            lanes each, scores from the FP16 rows, values added up here.
//   d12_values_kernel   a workgroup per token range and pair of sub-spaces.  Weights as fixed point into W_h[code], the V list's
//            rows times their tokens' weights, W_h times the centroids at the end.
// Where a table does not hold every head (d16) a V-anchored token outside the K list is scored in fp32, as in decode12_kernel: by
// workgroups beside those of d12_table_kernel.  Its weight then counts in d12_values_kernel alone.
// Bound: VALU issue first, with no pipe full: d12_weights_kernel is VALU-busy for 73 % of its cycles, d12_values_kernel for 67 %
// beside 45 % of LDS (d32) or 63 and 59 % (d16: twice the atomics per weight).  A 64-bit integer atomic, two heads each, takes 12.5
// clocks per wave instruction on random codes, a float atomic 192.  Gathering centroids instead costs 36 clocks per KB as
// pieces of 64 bytes (d32) and 71 as pieces of 32 (d16).
#include "decode12.h"

#include <type_traits>

namespace antkv {

namespace {

typedef float float2_t __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(4))) float4_t scalar_float4;      // uniform reads of what earlier kernels wrote

constexpr int kKI = 5, kKBlock = 4 * kKI;  // entries of the K list that a wave takes at a time
constexpr int kProbes = 512;               // samples of the V list in LDS

__device__ __forceinline__ float swap_add32(float a, float b)      // lanes 0-31: a, lanes 32-63: b, over the two half-waves
{
    const uint2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_add16(float a, float b)      // even rows of 16 lanes: a, odd rows: b, over the two rows
{
    const uint2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float rows_max(float v)                 // of the lanes l mod 16 of the four rows
{
    uint2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float all_max(float v)                  // of the wave, in every lane
{
#define ANTKV_ROR_MAX(N) v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + N, 0xf, 0xf, true)))
    ANTKV_ROR_MAX(8);
    ANTKV_ROR_MAX(4);
    ANTKV_ROR_MAX(2);
    ANTKV_ROR_MAX(1);
#undef ANTKV_ROR_MAX
    return rows_max(v);
}
// four heads' values, added up over the wave: lane 16 h + anything then holds head h
__device__ __forceinline__ float fold_sums(const float (&l)[kNH])
{
    float v = swap_add16(swap_add32(l[0], l[2]), swap_add32(l[1], l[3]));
    v = row_ror_add<8>(v);
    v = row_ror_add<4>(v);
    v = row_ror_add<2>(v);
    return row_ror_add<1>(v);
}
// four heads' values of a lane's eight channels, added up over the lanes that hold the same channels (l mod STEP): lane
// 16 h + l then holds head h
template <int STEP>
__device__ __forceinline__ void fold_heads(const float (&a)[kNH][8], float (&out)[8])
{
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float v = swap_add16(swap_add32(a[0][c], a[2][c]), swap_add32(a[1][c], a[3][c]));
        if constexpr (STEP <= 8) v = row_ror_add<8>(v);
        if constexpr (STEP <= 4) v = row_ror_add<4>(v);
        if constexpr (STEP <= 2) v = row_ror_add<2>(v);
        out[c] = v;
    }
}

// LDS of d12_weights_kernel: table, bitmaps of the range's K- and V-anchored tokens, q, samples of the V list, words, the waves'
// references and sums of the stream
constexpr size_t kWLds = (size_t)128 * 1024 + 2 * 1024 * 4 + kNH * kD * 2 + kProbes * 4 + 16 * 4 + 2 * kW12 * kNH * 4;
static_assert(kWLds <= 160 * 1024, "LDS budget");

template <int DS, bool GIVEN>
__global__ __launch_bounds__(kT12) void d12_weights_kernel(const D12LongParams p)
{
    constexpr int M = kD / DS, CB = 3 * M / 2;
    constexpr int NHT = GIVEN ? kNH : heads_per_table(DS);             // heads of a walk over the tokens
    constexpr bool kVApart = NHT < kNH;                                // V entries outside the K list are scored elsewhere
    constexpr int kTabBlocks = tab_blocks(DS);
    constexpr int kPairs = M * kC12 / 2 / kT12;                        // pairs of neighbouring table entries per thread and plane
    constexpr int kReq = kPairs * (heads_per_table(DS) / 2);           // 16-byte pieces of the table per thread
    extern __shared__ uint4_t smem_u4[];
    char* smem = (char*)smem_u4;
    uint32_t* s_mask = (uint32_t*)(smem + 128 * 1024);                 // [1024] words of (K-anchored or past the end, V-anchored)
    half_t* s_q = (half_t*)(s_mask + 2 * 1024);
    int* s_probe = (int*)(s_q + kNH * kD);
    int* s_misc = s_probe + kProbes;
    float* s_ms = (float*)(s_misc + 16);                               // [waves][heads]
    float* s_ls = s_ms + kW12 * kNH;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x % p.Hkv, rest = blockIdx.x / p.Hkv;       // KV head g on XCD g mod 8
    const int b = rest / p.S, sp = rest % p.S, bg = b * p.Hkv + g;
    const int64_t bgs = (int64_t)(gridDim.x / p.S), nt = (p.N + 63) >> 6;
    const int nh = p.G;
    const int64_t t0 = (int64_t)sp * p.chunk;
    const int n_tok = (int)((t0 + p.chunk < p.N ? t0 + p.chunk : p.N) - t0);
    const int n_tiles = (n_tok + 63) >> 6;
    const int32_t* idx_k = p.idx_k + (int64_t)bg * p.k_k;
    const int32_t* idx_v = p.idx_v + (int64_t)bg * p.k_v;
    const int n_walks = (nh + NHT - 1) / NHT;                          // 2 for d16 with more than two heads
    const int stride = (p.k_v + kProbes - 1) / kProbes;                // sample j of the V list is entry j * stride

    // ---- prologue: the table's pieces are requested first and arrive while the lists are searched
    float4_t piece[kReq];
    auto request = [&](int walk) {
        const float4_t* tb = (const float4_t*)p.tab + (int64_t)bg * M * kC12;      // [plane][entry] of two heads
#pragma unroll
        for (int i = 0; i < kReq; ++i) {
            const int plane = DS == 32 ? i / kPairs : walk;
            piece[i] = tb[plane * (M * kC12 / 2) + (i % kPairs) * kT12 + tid];
        }
    };
    float lut_q[NHT];                                                  // table quantum per head (log2 units)
    auto write_table = [&](int walk) {
        float inv[NHT];
        const scalar_float4* am = (const scalar_float4*)p.tab_amax + (int64_t)bg * kTabBlocks;
        float4_t a = am[0];
        for (int k = 1; k < kTabBlocks; ++k) {
            const float4_t x = am[k];
#pragma unroll
            for (int h = 0; h < kNH; ++h) a[h] = fmaxf(a[h], x[h]);
        }
#pragma unroll
        for (int h = 0; h < NHT; ++h) {
            const float top = NHT == kNH ? a[h] : (walk ? a[(2 + h) & 3] : a[h]);
            inv[h] = top > 0.f ? (float)kLutMax12 / top : 0.f;
            lut_q[h] = top * (1.0f / (float)kLutMax12);
        }
        // two entries to 16-bit integers: adding 1.5 * 2^23 leaves the rounded value in the low half
        auto pack = [](float x, float ix, float y, float iy) {
            const uint32_t lo = __float_as_uint(fmaf(x, ix, 12582912.f)), hi = __float_as_uint(fmaf(y, iy, 12582912.f));
            return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
        };
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            const float4_t x = piece[i];
            if constexpr (DS == 32) {
                const float4_t y = piece[i + kPairs];
                smem_u4[i * kT12 + tid] = uint4_t{pack(x[0], inv[0], x[1], inv[1]), pack(y[0], inv[2], y[1], inv[3]),
                                                  pack(x[2], inv[0], x[3], inv[1]), pack(y[2], inv[2], y[3], inv[3])};
            } else {
                ((uint2_t*)smem_u4)[i * kT12 + tid] = uint2_t{pack(x[0], inv[0], x[1], inv[1]), pack(x[2], inv[0], x[3], inv[1])};
            }
        }
    };
    if constexpr (!GIVEN) request(0);
    {
        const int over = tid * 32 + 32 - n_tok;                        // tokens of this word past the end
        *(uint2_t*)(s_mask + 2 * tid) = uint2_t{over <= 0 ? 0u : (over >= 32 ? ~0u : ~0u << (32 - over)), 0u};
    }
    if (tid < kNH * kD) s_q[tid] = (tid >> 7) < nh ? p.q[((int64_t)b * p.Hq + g * nh) * kD + tid] : (half_t)0.f;
    if (tid < kProbes && p.k_k > 0 && (int64_t)tid * stride < p.k_v) s_probe[tid] = idx_v[tid * stride];
    if (wave < 4) {                                                    // list ranges that fall into the token range
        const int r = lower_bound64(wave < 2 ? idx_k : idx_v, wave < 2 ? p.k_k : p.k_v, (int)t0 + ((wave & 1) ? n_tok : 0), lane);
        if (lane == 0) s_misc[wave] = r;
    }
    lds_barrier();
    // (a thread takes eight neighbouring entries: clustered anchors fill whole words)
    auto mark_list = [&](const int32_t* idx, int lo, int hi, int which) {
        for (int i = lo + 8 * tid; i < hi; i += 8 * kT12) {
            int rel[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) rel[j] = idx[i + j < hi ? i + j : hi - 1] - (int)t0;
            uint32_t bits = 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                bits |= 1u << (rel[j] & 31);
                if (j == 7 || rel[j + 1] >> 5 != rel[j] >> 5) {
                    atomicOr(s_mask + 2 * (rel[j] >> 5) + which, bits);
                    bits = 0u;
                }
            }
        }
    };
    mark_list(idx_k, s_misc[0], s_misc[1], 0);
    mark_list(idx_v, s_misc[2], s_misc[3], 1);
    // ---- the K list's entries: blocks of 20 dealt round-robin over all waves of the (sequence, KV head) whatever range an
    // entry's token is in (anchors cluster at the ends of a context); 16 lanes per entry.  Their V rows are looked
    // up in the V list: samples of it in LDS narrow the search down.
    const int grp = lane >> 4, li = lane & 15;
    constexpr int LPM = DS / 8;                                        // lanes per sub-space
    const int n_blocks = (p.k_k + kKBlock - 1) / kKBlock;
    const uint8_t* cv = p.codes_v + (int64_t)bg * p.N_cap * CB;
    const half_t* cbv = p.cb_v + (int64_t)g * M * kC12 * DS;
    half8_t row[kKI], src[kKI];                                            // K rows and values of a block's entries 4 i + grp
    auto fetch_block = [&](int blk) {
        const half_t* rows = p.rows_k + ((int64_t)bg * p.k_k + blk * kKBlock) * kD + 8 * li;
        const int left = p.k_k - blk * kKBlock;                             // entries of the block
        const int my = idx_k[blk * kKBlock + (lane < left ? lane : left - 1)];   // entry `lane`'s token, and its place in the V list or -1
#pragma unroll
        for (int i = 0; i < kKI; ++i) {
            const int e = 4 * i + grp;
            row[i] = *(const half8_t*)(rows + (e < left ? e : left - 1) * kD);
        }
        int pos = -1;
        {
            int lo = 0, hi = p.k_v > 0 ? (p.k_v - 1) / stride + 1 : 0; // first sample above the token
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (s_probe[mid] <= my) lo = mid + 1;
                else hi = mid;
            }
            if (lo > 0) {
                int a = (lo - 1) * stride, z = a + stride < p.k_v ? a + stride : p.k_v;
                while (z - a > 1) {                                    // entry a is not above the token
                    const int mid = (a + z) >> 1;
                    if (idx_v[mid] <= my) a = mid;
                    else z = mid;
                }
                if (idx_v[a] == my) pos = a;
            }
        }
#pragma unroll
        for (int i = 0; i < kKI; ++i) {
            const int tok = __shfl(my, 4 * i + grp, 64), at = __shfl(pos, 4 * i + grp, 64);
            const half_t* s;
            if (at >= 0) {
                s = p.rows_v + ((int64_t)bg * p.k_v + at) * kD + 8 * li;
            } else {
                const int m = li / LPM;
                const uint8_t* c = cv + (int64_t)tok * CB + m + (m >> 1);
                const uint32_t code = ((uint32_t)c[0] | (uint32_t)c[1] << 8) >> (4 * (m & 1)) & 0xFFFu;
                s = cbv + ((int64_t)m * kC12 + code) * DS + 8 * (li % LPM);
            }
            src[i] = *(const half8_t*)s;
        }
    };
    int blk = sp * kW12 + wave;
    if constexpr (!GIVEN) write_table(0);
    __syncthreads();

    // ---- stream
    float m_ref[kNH], l_lane[kNH];
#pragma unroll
    for (int h = 0; h < kNH; ++h) {
        m_ref[h] = kEmptyRef12;
        l_lane[h] = 0.f;
    }
    const uint8_t* ck = p.codes_k + ((int64_t)bg * p.N_cap + t0) * CB;
    const float4_t* given = GIVEN ? p.given + (int64_t)bg * p.N + t0 : nullptr;
    uint32_t* out[2] = {p.wts + (int64_t)bg * p.N + t0, p.wts + (bgs + bg) * p.N + t0};
    float* ref_out = p.tile_ref + ((int64_t)bg * nt + (t0 >> 6)) * kNH;
    struct Codes {
        uint32_t w[3];
        float4_t given;
    };
    auto fetch = [&](int tile, Codes& c) {
        const int tok = tile * 64 + lane, lt = tok < n_tok ? tok : n_tok - 1;
        if constexpr (GIVEN) {
            c.given = given[(uint32_t)lt];
        } else if constexpr (DS == 32) {
            const uint16_t* s = (const uint16_t*)(ck + (uint32_t)(lt * 6));
            c.w[0] = (uint32_t)s[0] | ((uint32_t)s[1] << 16);
            c.w[1] = (uint32_t)s[2];
            c.w[2] = 0u;
        } else {
            const uint32_t* s = (const uint32_t*)(ck + (uint32_t)(lt * 12));
            c.w[0] = s[0];
            c.w[1] = s[1];
            c.w[2] = s[2];
        }
    };
    // A wave takes two tiles at a time (their table reads and exponentials do not wait for each other) and the codes of the
    // next two are on their way meanwhile.  A second tile past the end has no tokens: all its mask bits are set.
    auto walk_tokens = [&](auto first) {
        constexpr int H0 = decltype(first)::value;                     // first head of the walk
        Codes cur[2], nxt[2];
        auto fetch2 = [&](int t, Codes (&c)[2]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) fetch(t + u * kW12 < n_tiles ? t + u * kW12 : n_tiles - 1, c[u]);
        };
        if (wave < n_tiles) fetch2(wave, cur);
#pragma unroll 1
        for (int t = wave; t < n_tiles; t += 2 * kW12) {
            fetch2(t + 2 * kW12, nxt);
            float x[2][NHT], over = kNegBig;
            uint32_t mark[2];
            bool off[2];
            const uint32_t bit = lane & 31;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int tile = t + u * kW12;
                const uint2_t mk = *(const uint2_t*)(s_mask + 2 * ((2 * tile + (lane >> 5)) & 1023));
                off[u] = (mk[0] >> bit & 1u) != 0u;
                mark[u] = (mk[1] >> bit & 1u) * 0x80008000u;
                if constexpr (kVApart) {                               // a weight of 0 here, and -1 as the mark
                    if (off[u]) mark[u] = 0u;
                    off[u] = off[u] || mark[u] != 0u;
                    mark[u] = mark[u] != 0u ? 0xBC00BC00u : 0u;
                }
                if (u == 1 && tile >= n_tiles) off[u] = true;
                if constexpr (GIVEN) {
#pragma unroll
                    for (int h = 0; h < kNH; ++h) x[u][h] = cur[u].given[h];
                } else {
                    int sum[NHT];
#pragma unroll
                    for (int h = 0; h < NHT; ++h) sum[h] = 0;
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        if constexpr (DS == 32) {
                            const uint2_t e = ((const uint2_t*)smem_u4)[m * kC12 + code12(cur[u].w, m)];
                            sum[0] += (int)(short)(e[0] & 0xFFFFu);
                            sum[1] += (int)e[0] >> 16;
                            sum[2] += (int)(short)(e[1] & 0xFFFFu);
                            sum[3] += (int)e[1] >> 16;
                        } else {
                            const uint32_t e = ((const uint32_t*)smem_u4)[m * kC12 + code12(cur[u].w, m)];
                            sum[0] += (int)(short)(e & 0xFFFFu);
                            sum[1] += (int)e >> 16;
                        }
                    }
#pragma unroll
                    for (int h = 0; h < NHT; ++h) x[u][h] = (float)sum[h] * lut_q[h];
                }
#pragma unroll
                for (int h = 0; h < NHT; ++h) {
                    x[u][h] = off[u] ? kNegBig : x[u][h];
                    over = fmaxf(over, x[u][h] - m_ref[H0 + h]);
                }
            }
            // (the reference is the largest score so far, whose weight then is a power of two and rounds to itself: with references
            // up to 3 log2 units below it the output's error was 2 % larger)
            if (__any(over > 0.f)) {
#pragma unroll
                for (int h = 0; h < NHT; ++h) {
                    const float top = all_max(fmaxf(x[0][h], x[1][h]));
                    if (top > m_ref[H0 + h]) {
                        l_lane[H0 + h] *= fast_exp2(m_ref[H0 + h] - top);
                        m_ref[H0 + h] = top;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int tile = t + u * kW12, tok = tile * 64 + lane;
                half_t w[NHT];
#pragma unroll
                for (int h = 0; h < NHT; ++h) {
                    const float pw = fast_exp2(x[u][h] - m_ref[H0 + h] + kPShift12);
                    l_lane[H0 + h] += pw;
                    w[h] = (half_t)pw;
                }
                if (tok < n_tok) {
#pragma unroll
                    for (int pl = 0; pl < NHT / 2; ++pl)
                        if (H0 + 2 * pl < nh) out[H0 / 2 + pl][(uint32_t)tok] = __builtin_bit_cast(uint32_t, half2_t{w[2 * pl], w[2 * pl + 1]}) ^ mark[u];
                    if (lane == 0) {
                        if constexpr (NHT == kNH) *(float4_t*)(ref_out + tile * kNH) = float4_t{m_ref[0], m_ref[1], m_ref[2], m_ref[3]};
                        else *(float2_t*)(ref_out + tile * kNH + H0) = float2_t{m_ref[H0], m_ref[H0 + 1]};
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) cur[u] = nxt[u];
        }
    };
    walk_tokens(std::integral_constant<int, 0>{});
    if constexpr (NHT < kNH) {
        if (n_walks > 1) {                                             // heads 2 and 3: their table takes the first one's place
            request(1);
            lds_barrier();
            write_table(1);
            lds_barrier();
            walk_tokens(std::integral_constant<int, kNH - NHT>{});
        }
    }

    // ---- the K list's entries.  (Their weights are summed apart: the fixed-point unit of d12_values_kernel follows the stream's.)
    {
        const float l = fold_sums(l_lane);
        if (li == 0) s_ls[wave * kNH + grp] = l;
    }
    if (lane == 0) *(float4_t*)(s_ms + wave * kNH) = float4_t{m_ref[0], m_ref[1], m_ref[2], m_ref[3]};
    float acc[kNH][8];
#pragma unroll
    for (int h = 0; h < kNH; ++h) {
        l_lane[h] = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[h][c] = 0.f;
    }
#pragma unroll 1
    for (; blk < n_blocks; blk += p.S * kW12) {
        fetch_block(blk);
        const int left = p.k_k - blk * kKBlock;
        float sc[kKI][kNH], top[kNH];
#pragma unroll
        for (int h = 0; h < kNH; ++h) {
            const half8_t qh = *(const half8_t*)(s_q + h * kD + 8 * li);
#pragma unroll
            for (int i = 0; i < kKI; ++i) {
                float d = dot8f(row[i], qh, 0.f);
                d = row_ror_add<8>(d);
                d = row_ror_add<4>(d);
                d = row_ror_add<2>(d);
                d = row_ror_add<1>(d);
                sc[i][h] = 4 * i + grp < left ? d * p.c1 : kNegBig;
            }
            float t = sc[0][h];
#pragma unroll
            for (int i = 1; i < kKI; ++i) t = fmaxf(t, sc[i][h]);
            top[h] = rows_max(t);
            if (top[h] > m_ref[h]) {
                const float alpha = fast_exp2(m_ref[h] - top[h]);
                l_lane[h] *= alpha;
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[h][c] *= alpha;
                m_ref[h] = top[h];
            }
        }
#pragma unroll
        for (int i = 0; i < kKI; ++i) {
            float pw[kNH];
#pragma unroll
            for (int h = 0; h < kNH; ++h) {
                pw[h] = fast_exp2(sc[i][h] - m_ref[h] + kPShift12);
                l_lane[h] += li == 0 ? pw[h] : 0.f;
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float vf = 4 * i + grp < left ? (float)src[i][c] : 0.f;
#pragma unroll
                for (int h = 0; h < kNH; ++h) acc[h][c] = fmaf(pw[h], vf, acc[h][c]);
            }
        }
    }

    // ---- merge the waves, write the workgroup's partial
    __syncthreads();                                                   // nobody reads the table any more
    float* s_m = (float*)smem;                                         // [waves][heads] references
    float* s_l = s_m + kW12 * kNH;                                     // [waves][heads] sums
    float* s_acc = s_l + kW12 * kNH;                                   // [waves][heads][128]
    const float l_entries = fold_sums(l_lane);
    if (lane == 0) *(float4_t*)(s_m + wave * kNH) = float4_t{m_ref[0], m_ref[1], m_ref[2], m_ref[3]};
    __builtin_amdgcn_wave_barrier();                                   // LDS operations of one wave stay in order
    if (li == 0) s_l[wave * kNH + grp] = fmaf(s_ls[wave * kNH + grp], fast_exp2(s_ms[wave * kNH + grp] - s_m[wave * kNH + grp]), l_entries);
    float fold[8];
    fold_heads<16>(acc, fold);
#pragma unroll
    for (int c = 0; c < 8; ++c) s_acc[(wave * kNH + grp) * kD + 8 * li + c] = fold[c];
    __syncthreads();
    if (tid < kNH * kD) {
        const int h = tid >> 7, ch = tid & 127;
        if (h < nh) {
            float m = kEmptyRef12;
            for (int w = 0; w < kW12; ++w) m = fmaxf(m, s_m[w * kNH + h]);
            float l = 0.f, a = 0.f;
            for (int w = 0; w < kW12; ++w) {
                const float f = fast_exp2(s_m[w * kNH + h] - m);
                l = fmaf(s_l[w * kNH + h], f, l);
                a = fmaf(s_acc[(w * kNH + h) * kD + ch], f, a);
            }
            float* dst = p.part + (((int64_t)b * p.Hq + g * nh + h) * p.slots + sp) * (kD + 2);
            dst[2 + ch] = a;
            if (ch == 0) {
                dst[0] = m;
                dst[1] = l;
            }
        }
    } else if (tid < kNH * kD + nh) {
        const int h = tid - kNH * kD;
        float m = kEmptyRef12, l = 0.f;
        for (int w = 0; w < kW12; ++w) m = fmaxf(m, s_ms[w * kNH + h]);
        for (int w = 0; w < kW12; ++w) l = fmaf(s_ls[w * kNH + h], fast_exp2(s_ms[w * kNH + h] - m), l);
        p.stat[((int64_t)b * p.Hq + g * nh + h) * p.S + sp] = float2{m, l};
    }
}

// A batch is kU rounds of 1024 tokens, the next batch is requested before the current one is added up.  The factors that turn a
// tile's weights into fixed point are worked out once per tile, for sections of kSec tiles.
constexpr int kU = 4;
constexpr int kUV = 5;                      // entries of the V list per lane in flight
constexpr int kSec = 1792;
constexpr size_t kVLds = (size_t)128 * 1024 + kSec * 16 + 3 * kNH * sizeof(float);
static_assert(kVLds <= 160 * 1024, "LDS budget");

// SCORED: the V list's entries come with scores, not with the stream's weights
template <int DS, bool SCORED>
__global__ __launch_bounds__(kT12) void d12_values_kernel(const D12LongParams p)
{
    constexpr int M = kD / DS, CB = 3 * M / 2, NP = M / 2;
    extern __shared__ uint4_t smem_u4[];
    unsigned long long* s_hist = (unsigned long long*)smem_u4;         // [2 sub-spaces][2 head pairs][4096]
    float4_t* s_f = (float4_t*)((char*)smem_u4 + 128 * 1024);          // [tiles of the section] factors of the four heads
    float* s_top = (float*)(s_f + kSec);                               // [heads] reference of the range,
    float* s_all = s_top + kNH;                                        // and of the sequence
    int* s_exp = (int*)(s_all + kNH);                                  // [heads] log2 of the fixed-point scale
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x % p.Hkv;                                  // KV head g on XCD g mod 8
    int rest = blockIdx.x / p.Hkv;
    const int pr = rest % NP;
    rest /= NP;
    const int r = rest % p.S2, b = rest / p.S2, bg = b * p.Hkv + g;
    const int64_t bgs = (int64_t)(gridDim.x / (NP * p.S2)), nt = (p.N + 63) >> 6;
    const int64_t r0 = (int64_t)r * p.range, r1 = r0 + p.range < p.N ? r0 + p.range : p.N;
    const int planes = p.G > 2 ? 2 : 1;
    const uint32_t* wt[2] = {p.wts + (int64_t)bg * p.N, p.wts + ((planes - 1) * bgs + bg) * p.N};
    const float4_t* refs = (const float4_t*)p.tile_ref + (int64_t)bg * nt;
    // The V list's rows, this pair's 2 DS channels of them, LR lanes per row; blocks of RP entries are dealt over all waves.
    constexpr int LR = 2 * DS / 8, RP = 64 / LR;
    const int v_step = p.S2 * kW12 * RP;
    int ve = (r * kW12 + wave) * RP + lane / LR;
#pragma unroll
    for (int i = 0; i < 8; ++i) smem_u4[i * kT12 + tid] = uint4_t{0u, 0u, 0u, 0u};
    // References, and the sum of the stream's weights over the ranges of d12_weights_kernel that this one touches.  The fixed-point
    // unit is 2^-e, so that 17/16 of that sum has at most 2^32 of them and at least 2^31: no sum of weights overflows, since a
    // sixteenth is more than their rounding to fp16 and one unit for each of 2^27 tokens (rule: d12_by_code).
    if (wave < kNH) {
        float all = kEmptyRef12, top = kEmptyRef12;
        int e = 0;
        if (wave < p.G) {
            const float2* st = p.stat + ((int64_t)b * p.Hq + g * p.G + wave) * p.S;
            const int s_lo = (int)(r0 / p.chunk), s_hi = (int)((r1 - 1) / p.chunk);
            for (int s = lane; s < p.S; s += 64) {
                const float x = st[s].x;
                all = fmaxf(all, x);
                if (s >= s_lo && s <= s_hi) top = fmaxf(top, x);
            }
            all = all_max(all);
            top = all_max(top);
            float l = 0.f;
            for (int s = s_lo + lane; s <= s_hi; s += 64) l = fmaf(st[s].y, fast_exp2(st[s].x - top), l);
            l = wave_sum(l);
            (void)frexpf(l * 1.0625f, &e);
            e = 32 - e;
        }
        if (lane == 0) {
            s_all[wave] = all;
            s_top[wave] = top;
            s_exp[wave] = e;
        }
    }
    __syncthreads();
    float top[kNH], scale[kNH];                                        // weight to fixed point: 2^(reference of the tile - top) scale
#pragma unroll
    for (int h = 0; h < kNH; ++h) {
        top[h] = s_top[h];
        scale[h] = h < p.G ? ldexpf(1.f, s_exp[h]) : 0.f;              // (0: the slot has no head)
    }
    // What a weight is short of whole units counts as one or none by the lane's share of a unit, spread evenly over the 64 tokens
    // of a tile: rounded to the nearest, the small weights beside a large one would all err the same way.
    const float share = ((float)(__brev((uint32_t)lane) >> 26) + 0.5f) * (1.f / 64.f);
    auto to_fixed = [&](float w, float f) -> uint32_t {
        uint32_t r;
        asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(fmaf(w, f, share)));    // (0 for marked weights, which are negative, and NaN)
        return r;
    };
    const int coff = (3 * pr) & ~1, cshift = 8 * ((3 * pr) & 1);       // the pair's three bytes of a row lie in two 16-bit words
    const uint8_t* cv = p.codes_v + (int64_t)bg * p.N_cap * CB + coff;

    struct Batch {
        uint16_t lo[kU], hi[kU];
        uint32_t w[kU][2];
    };
#pragma unroll 1
    for (int64_t s0 = r0; s0 < r1; s0 += (int64_t)kSec * 64) {
        const int n = (int)(r1 - s0 < (int64_t)kSec * 64 ? r1 - s0 : (int64_t)kSec * 64);
        const uint8_t* cs = cv + s0 * CB;
        const uint32_t *ws0 = wt[0] + s0, *ws1 = wt[1] + s0;
        auto fetch = [&](int base, Batch& t) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int tok = base + u * kT12 + tid;
                const uint32_t lt = (uint32_t)(tok < n ? tok : n - 1);
                const uint16_t* cp = (const uint16_t*)(cs + lt * (uint32_t)CB);
                t.lo[u] = cp[0];
                t.hi[u] = cp[1];
                t.w[u][0] = ws0[lt];
                t.w[u][1] = ws1[lt];
            }
        };
        auto add = [&](int base, const Batch& t) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int at = (base + u * kT12) / 64 + wave;          // tile of the section
                if (at * 64 >= n) continue;
                const float4_t f = s_f[at];
                const bool on = at * 64 + lane < n;
                const uint32_t code = ((uint32_t)t.lo[u] | ((uint32_t)t.hi[u] << 16)) >> cshift;
                unsigned long long* h0 = s_hist + (code & 0xFFFu);
                unsigned long long* h1 = s_hist + (code >> 12 & 0xFFFu) + 2 * kC12;
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) {
                    if (pl >= planes) continue;
                    const half2_t w2 = __builtin_bit_cast(half2_t, t.w[u][pl]);
                    // (marked weights are negative and become 0)
                    const uint32_t x = to_fixed((float)w2[0], f[2 * pl]), y = to_fixed((float)w2[1], f[2 * pl + 1]);
                    if (on && (x | y) != 0u) {
                        const unsigned long long v = (unsigned long long)y << 32 | x;
                        atomicAdd(h0 + pl * kC12, v);
                        atomicAdd(h1 + pl * kC12, v);
                    }
                }
            }
        };
        Batch cur, nxt;
        fetch(0, cur);
        for (int t = tid; t < (n + 63) / 64; t += kT12) {
            const float4_t ref = refs[(s0 >> 6) + t];
            float4_t f;
#pragma unroll
            for (int h = 0; h < kNH; ++h) f[h] = fast_exp2(ref[h] - top[h]) * scale[h];
            s_f[t] = f;
        }
        lds_barrier();
#pragma unroll 1
        for (int base = 0; base < n; base += kU * kT12) {
            fetch(base + kU * kT12, nxt);
            add(base, cur);
            cur = nxt;
        }
        lds_barrier();
    }

    // ---- the V list's rows times their tokens' weights: those that the stream left (negative; a K-anchored token, whose weight is 0,
    // is settled there), or of the entry's score, against the wave's largest so far
    float av[kNH][8], m_v[kNH], l_v[kNH];
#pragma unroll
    for (int h = 0; h < kNH; ++h) {
        m_v[h] = SCORED ? kEmptyRef12 : s_all[h];
        l_v[h] = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) av[h][c] = 0.f;
    }
    const int32_t* idx_v = p.idx_v + (int64_t)bg * p.k_v;
    const half_t* rows = p.rows_v + (int64_t)bg * p.k_v * kD + 2 * DS * pr + 8 * (lane % LR);
    const float4_t* scores = p.v_scores + (int64_t)bg * p.k_v;
#pragma unroll 1
    for (; __any(ve < p.k_v); ve += kUV * v_step) {
        uint4_t vrow[kUV];
        uint32_t w2[kUV][2];
        float4_t from[kUV];                                            // score, or reference of the token's tile
        int tok[kUV];
#pragma unroll
        for (int u = 0; u < kUV; ++u) {
            const int e = ve + u * v_step;
            tok[u] = -1;
            vrow[u] = uint4_t{0u, 0u, 0u, 0u};
            from[u] = float4_t{0.f, 0.f, 0.f, 0.f};
            if (e < p.k_v) {
                tok[u] = idx_v[e];
                vrow[u] = *(const uint4_t*)(rows + (int64_t)e * kD);
                if constexpr (SCORED) from[u] = scores[e];
            }
        }
#pragma unroll
        for (int u = 0; u < kUV; ++u) {
            const int t = tok[u] < 0 ? 0 : tok[u];
            w2[u][0] = wt[0][t];
            if constexpr (!SCORED) {
                w2[u][1] = wt[1][t];
                from[u] = refs[t >> 6];
            }
        }
        float w[kUV][kNH];
        if constexpr (SCORED) {
#pragma unroll
            for (int h = 0; h < kNH; ++h) {
                float t = kNegBig;
#pragma unroll
                for (int u = 0; u < kUV; ++u) {
                    w[u][h] = tok[u] >= 0 && (w2[u][0] & 0x8000u) != 0u ? from[u][h] : kNegBig;
                    t = fmaxf(t, w[u][h]);
                }
                t = all_max(t);
                if (t > m_v[h]) {
                    const float alpha = fast_exp2(m_v[h] - t);
                    l_v[h] *= alpha;
#pragma unroll
                    for (int c = 0; c < 8; ++c) av[h][c] *= alpha;
                    m_v[h] = t;
                }
#pragma unroll
                for (int u = 0; u < kUV; ++u) {
                    w[u][h] = fast_exp2(w[u][h] - m_v[h] + kPShift12);
                    l_v[h] += lane % LR == 0 ? w[u][h] : 0.f;
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < kUV; ++u)
#pragma unroll
                for (int h = 0; h < kNH; ++h)
                    w[u][h] = tok[u] < 0 ? 0.f : -(float)__builtin_bit_cast(half2_t, w2[u][h >> 1])[h & 1] * fast_exp2(from[u][h] - m_v[h]);
        }
#pragma unroll
        for (int u = 0; u < kUV; ++u) {
            const half8_t v = __builtin_bit_cast(half8_t, vrow[u]);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float vf = (float)v[c];
#pragma unroll
                for (int h = 0; h < kNH; ++h) av[h][c] = fmaf(w[u][h], vf, av[h][c]);
            }
        }
    }
    float out_v[8];
    fold_heads<LR>(av, out_v);
    const float sum_v = SCORED ? fold_sums(l_v) : 0.f;

    // ---- the 2 x 4096 sums times their centroids: LPC lanes per centroid, a wave takes 256 codes of either sub-space, the next
    // four centroids are on their way while four are multiplied
    constexpr int LPC = DS / 8, kPer = 64 / LPC, kIter = 256 / kPer;
    const int li = lane % LPC, c0 = wave * 256 + lane / LPC;
    const half_t* cbv = p.cb_v + ((int64_t)g * M + 2 * pr) * kC12 * DS + 8 * li;
    float out_s[2][8];
    {
        uint4_t cur[4], nxt[4];
        auto request = [&](int i0, uint4_t (&dst)[4]) {                // rounds i0 .. i0 + 3 of both sub-spaces' 2 kIter
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = i0 + i < 2 * kIter ? i0 + i : 2 * kIter - 1, sub = at / kIter, it = at % kIter;
                dst[i] = *(const uint4_t*)(cbv + (uint32_t)((sub * kC12 + c0 + it * kPer) * DS));
            }
        };
        request(0, cur);
        lds_barrier();                                                 // the sums are complete
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            float acc[kNH][8];
#pragma unroll
            for (int h = 0; h < kNH; ++h)
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[h][c] = 0.f;
#pragma unroll 1
            for (int i0 = 0; i0 < kIter; i0 += 4) {
                request(sub * kIter + i0 + 4, nxt);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int code = c0 + (i0 + i) * kPer;
                    const unsigned long long x = s_hist[2 * sub * kC12 + code], y = s_hist[(2 * sub + 1) * kC12 + code];
                    // a centroid that no token uses may hold anything
                    const half8_t v = __builtin_bit_cast(half8_t, (x | y) != 0ull ? cur[i] : uint4_t{0u, 0u, 0u, 0u});
                    const float wf[kNH] = {(float)(uint32_t)x, (float)(uint32_t)(x >> 32), (float)(uint32_t)y, (float)(uint32_t)(y >> 32)};
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        const float vf = (float)v[c];
#pragma unroll
                        for (int h = 0; h < kNH; ++h) acc[h][c] = fmaf(wf[h], vf, acc[h][c]);
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) cur[i] = nxt[i];
            }
            fold_heads<LPC>(acc, out_s[sub]);
        }
    }
    __syncthreads();                                                   // the sums are no longer read
    float* s_o = (float*)smem_u4;                                      // [waves][heads][2 DS], then the same of the V list
    float* s_ov = s_o + kW12 * kNH * 2 * DS;
    float* s_mv = s_ov + kW12 * kNH * 2 * DS;                          // [waves][heads] its references and sums
    float* s_lv = s_mv + kW12 * kNH;
    const int row = wave * kNH + (lane >> 4);
    if ((lane & 15) < LPC) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            s_o[row * 2 * DS + 8 * li + c] = out_s[0][c];
            s_o[row * 2 * DS + DS + 8 * li + c] = out_s[1][c];
        }
    }
    if ((lane & 15) < LR) {
#pragma unroll
        for (int c = 0; c < 8; ++c) s_ov[row * 2 * DS + 8 * (lane % LR) + c] = out_v[c];
    }
    if constexpr (SCORED) {
        if ((lane & 15) == 0) s_lv[row] = sum_v;
        if (lane == 0) *(float4_t*)(s_mv + wave * kNH) = float4_t{m_v[0], m_v[1], m_v[2], m_v[3]};
    }
    __syncthreads();
    if (tid < kNH * 2 * DS) {
        const int h = tid / (2 * DS), ch = tid % (2 * DS);
        if (h < p.G) {
            float a = 0.f, v = 0.f, m = SCORED ? s_top[h] : s_all[h], l = 0.f;
#pragma unroll
            for (int w = 0; w < kW12; ++w) a += s_o[(w * kNH + h) * 2 * DS + ch];
            if constexpr (SCORED) {
#pragma unroll
                for (int w = 0; w < kW12; ++w) m = fmaxf(m, s_mv[w * kNH + h]);
            }
            a = ldexpf(a, -s_exp[h]) * fast_exp2(s_top[h] - m);
#pragma unroll
            for (int w = 0; w < kW12; ++w) {
                const float f = SCORED ? fast_exp2(s_mv[w * kNH + h] - m) : 1.f;
                v = fmaf(s_ov[(w * kNH + h) * 2 * DS + ch], f, v);
                if constexpr (SCORED) l = fmaf(s_lv[w * kNH + h], f, l);
            }
            float* dst = p.part + (((int64_t)b * p.Hq + g * p.G + h) * p.slots + p.S + r) * (kD + 2);
            dst[2 + 2 * DS * pr + ch] = a + v;
            if (pr == 0 && ch == 0) {                                  // (the stream's weights are counted in d12_weights_kernel's sums)
                dst[0] = m;
                dst[1] = l;
            }
        }
    }
}

template <int DS>
hipError_t launch(const Geom& g, const D12LongParams& p, hipStream_t st)
{
    constexpr bool kApart = heads_per_table(DS) < kNH;
    static OncePerDevice once;
    const hipError_t setup = on_this_device(once, []() {
        const std::pair<const void*, size_t> kernels[] = {{(const void*)d12_weights_kernel<DS, false>, kWLds},
                                                          {(const void*)d12_weights_kernel<DS, true>, kWLds},
                                                          {(const void*)d12_values_kernel<DS, kApart>, kVLds},
                                                          {(const void*)d12_values_kernel<DS, false>, kVLds}};
        for (const auto& k : kernels) {
            const hipError_t e = hipFuncSetAttribute(k.first, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.second);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    });
    if (setup != hipSuccess) return setup;
    const dim3 ranges((unsigned)(g.B * g.Hkv * p.S)), parts((unsigned)(g.B * g.Hkv * p.S2 * (g.M / 2)));
    if (p.given) {
        hipLaunchKernelGGL((d12_weights_kernel<DS, true>), ranges, dim3(kT12), kWLds, st, p);
        hipLaunchKernelGGL((d12_values_kernel<DS, false>), parts, dim3(kT12), kVLds, st, p);
    } else {
        hipLaunchKernelGGL((d12_weights_kernel<DS, false>), ranges, dim3(kT12), kWLds, st, p);
        hipLaunchKernelGGL((d12_values_kernel<DS, kApart>), parts, dim3(kT12), kVLds, st, p);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_decode12_by_code(const Geom& g, const D12LongParams& p, hipStream_t st)
{
    return g.d == 32 ? launch<32>(g, p, st) : launch<16>(g, p, st);
}

}  // namespace antkv
