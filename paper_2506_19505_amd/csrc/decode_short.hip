// Decode attention over 12-bit codes for short token ranges, one launch: every token's key and value row is put together
// from its centroids (or its FP16 anchor row) and goes through the matrix cores as it stands.
//
// For long contexts a table of q . centroid products is worth its own kernel, its quantisation in every workgroup, and
// anchor lists as work of their own.  Here a workgroup (8 waves) has a few hundred tokens of one (sequence, KV head):
//
//  prologue  one round of loads: the anchor lists (their entries in the range leave their slot numbers in LDS, one word
//            per token and side; long lists are cut to the range by a search first), the codes of the waves' first tiles, the
//            query.  The codebooks (1 MB each) stay in the L2.
//  tile      32 tokens per wave.  Scores: 16 tokens x 128 channels on the rows of the MFMA, the query heads on its
//            columns, a lane's eight channels being one 16-byte piece of a centroid or of an FP16 K row: anchored tokens
//            differ in the address only.  The result leaves four consecutive tokens of one head in a lane, which is the
//            form the value product takes its weights in.  Values: the tile's rows, centroids or FP16 rows alike, go from
//            memory straight into the wave's LDS area; 16 channels x 32 tokens per MFMA through transposed reads.
//  merge     waves through LDS, workgroups through device-scope partials: the last to arrive adds them up.
//
// Scores are fp16 x fp16 products in fp32, tiles are dealt statically and all sums have a fixed order.
//
// Bound: latency up to a few hundred tokens per workgroup (10 us: launch, one round of loads, gathers, the two merges), then the
// gathers: 23 clocks per token and CU for d 32 (18 at the measured rate of 2.2 clocks per piece of a row), 40 for d 16.  One step
// (append and attention), 8 heads, d 32 / d 16: 1000 tokens 37.3 / 46.7 -> 14.6 / 14.2 us, 16384 38.6 / 51.5 -> 20 / 22, 50000
// 43.6 / 62.6 -> 31 / 42.
#include "decode_short.h"
#include "lds_tile.h"

namespace antkv {

namespace {

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kTile = 32;               // tokens of a wave's tile
// A list of up to kScan entries is read whole by every workgroup, a longer one cut to its range by a search (two or three dependent
// loads).  8 heads, read whole and cut: d 32, 90000 tokens, all anchored 216 and 77 us (165 through a table), one in ten 50.6 and 43;
// 16384 tokens, all 35 and 21; d 16, 57000 tokens, all 104 and 43, one in ten 51 and 42.
constexpr int kScan = 4 * kThreads;

struct Lds {
    static constexpr int rows = 0;                                  // [waves][32 rows of 256 bytes]
    static constexpr int mrg = 0;                                   // merge: [waves][channel][4 heads] fp32
    static constexpr int slot_k = kWaves * kTileBytes;              // [token] index into the K list or -1
    static constexpr int slot_v = slot_k + kShortTokens * 4;
    static constexpr int red = slot_v + kShortTokens * 4;           // [waves][8]: references and sums; then one word
    static constexpr int total = red + kWaves * 32 + 64;
    static_assert(kWaves * kD * kNH * 4 <= slot_k && total <= 163840, "LDS of one CU");
};

typedef __attribute__((address_space(3))) const char lds_cchar;

__device__ __forceinline__ half4_t read_tr16(uint32_t addr)
{
    return __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)addr));
}
__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row16_max(float v)
{
    v = fmaxf(v, dpp<0xB1>(v));                                     // quad_perm [1,0,3,2]
    v = fmaxf(v, dpp<0x4E>(v));                                     // quad_perm [2,3,0,1]
    v = fmaxf(v, dpp<0x141>(v));                                    // row_half_mirror
    return fmaxf(v, dpp<0x140>(v));                                 // row_mirror
}
__device__ __forceinline__ float row16_sum(float v)
{
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    return v + dpp<0x140>(v);
}
// 16 bytes per lane from the lane's own address to LDS address `to` + 16 * lane (waited for as load_to_lds16 is)
__device__ __forceinline__ void gather_to_lds16(const void* from, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(to), "v"(from) : "m0", "memory");
}

// What a lane needs of a tile's codes.  K: the code row of token 16 u + lane % 16.  V: the code behind the lane's 16-byte piece
// of row 4 i + lane / 16, i = 0..7.
template <int DSUB>
struct TileCodes {
    static constexpr int row = 12 * kD / DSUB / 8;                  // bytes of a token's codes
    uint32_t k[2][3], v[8];

    // the piece: rows are swizzled in LDS (lds_tile.h)
    __device__ __forceinline__ static int piece(int i, int lane) { return (lane & 15) ^ swz(4 * i + (lane >> 4)); }

    __device__ __forceinline__ void load(const uint8_t* ck, const uint8_t* cv, int tile, int n, int lane)
    {
        auto token = [&](int t) { return t < n ? t : n - 1; };
#pragma unroll
        for (int u = 0; u < 2; ++u) load_cw<DSUB>(ck, token(tile * kTile + 16 * u + (lane & 15)), k[u]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int m = piece(i, lane) * 8 / DSUB;
            const uint8_t* s = cv + token(tile * kTile + 4 * i + (lane >> 4)) * row + m + (m >> 1);
            v[i] = ((uint32_t)s[0] | (uint32_t)s[1] << 8) >> (4 * (m & 1)) & 0xFFFu;
        }
    }
};

template <int DSUB>
__global__ __launch_bounds__(kThreads) void decode_short_kernel(const ShortParams p)
{
    using Codes = TileCodes<DSUB>;
    constexpr int C = kC12;
    extern __shared__ uint4_t smem_u4[];
    char* smem = (char*)smem_u4;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_cchar*)smem_u4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups go to the 8 XCDs round-robin.  Where the number of KV heads allows, head g stays on XCD g mod 8, whose L2 then
    // holds the codebooks of its own heads only (4 x 8 heads, 12000 tokens, d 32 / d 16: a step 28 / 40 us, 42 / 69 with the ranges of a sequence on one XCD).
    const int groups = (p.Hkv & 7) == 0 ? 8 : 1;
    const int rest = (int)blockIdx.x / groups, sp = rest % p.S, b = rest / p.S % p.B, g = (int)blockIdx.x % groups + groups * (rest / p.S / p.B);
    const int bg = b * p.Hkv + g, h0 = g * p.G, nheads = p.G;
    const int t0 = sp * p.chunk;
    const int n = (int)(p.N - t0 < p.chunk ? p.N - t0 : p.chunk);
    const int n_tiles = (n + kTile - 1) / kTile;
    const uint8_t* ck = p.codes_k + ((int64_t)bg * p.N_cap + t0) * Codes::row;
    const uint8_t* cv = p.codes_v + ((int64_t)bg * p.N_cap + t0) * Codes::row;
    const half_t* cbk = p.cb_k + (size_t)g * kD * C;
    const half_t* cbv = p.cb_v + (size_t)g * kD * C;
    const int32_t* idx_k = p.idx_k + (int64_t)bg * p.k_k;
    const int32_t* idx_v = p.idx_v + (int64_t)bg * p.k_v;
    const half_t* rows_k = p.rows_k + (int64_t)bg * p.k_k * kD;
    const half_t* rows_v = p.rows_v + (int64_t)bg * p.k_v * kD;
    int* s_slot_k = (int*)(smem + Lds::slot_k);
    int* s_slot_v = (int*)(smem + Lds::slot_v);
    float* s_red = (float*)(smem + Lds::red);
    int* s_count = (int*)(smem + Lds::red + kWaves * 32);           // one word; then the bounds of the K and of the V list
    int* s_cut = s_count + 1;
    // MFMA lane coordinates: row / column and k-group; token and 8-byte piece of a transposed read
    const int ln = lane & 15, kg = lane >> 4, tj = lane >> 2 & 3, tq = lane & 3;

    // ------------------------------------------------------------------------------------------ prologue
    unsigned long long seen = 0ull;                                 // arrival word
    if (tid == 0 && p.S > 1) seen = __hip_atomic_load(&p.done[bg], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool cut_k = p.k_k > kScan, cut_v = p.k_v > kScan;
    const int first_k = !cut_k && tid < p.k_k ? idx_k[tid] : -1, first_v = !cut_v && tid < p.k_v ? idx_v[tid] : -1;
    Codes codes;
    if (wave < n_tiles) codes.load(ck, cv, wave, n, lane);
    half8_t qop[4];                                                 // query: column ln is head ln % 4
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        qop[st] = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
        if ((ln & 3) < nheads) qop[st] = *(const half8_t*)(p.q + ((int64_t)b * p.Hq + h0 + (ln & 3)) * kD + 32 * st + 8 * kg);
    }
    for (int i = tid; i < n_tiles * kTile; i += kThreads) {
        s_slot_k[i] = -1;
        s_slot_v[i] = -1;
    }
    lds_barrier();
    auto note = [&](int* slots, int token, int slot) {              // (the filler -1 and positions below t0 wrap to huge values)
        const uint32_t rel = (uint32_t)token - (uint32_t)t0;
        if (token >= 0 && rel < (uint32_t)n) slots[rel] = slot;
    };
    note(s_slot_k, first_k, tid);
    note(s_slot_v, first_v, tid);
    if (cut_k || cut_v) {
        if (wave < 4 && (wave < 2 ? cut_k : cut_v)) {
            const int at = lower_bound64(wave < 2 ? idx_k : idx_v, wave < 2 ? p.k_k : p.k_v, wave & 1 ? t0 + n : t0, lane);
            if (lane == 0) s_cut[wave] = at;
        }
        lds_barrier();
        const int lo_k = cut_k ? s_cut[0] : kThreads, len_k = (cut_k ? s_cut[1] : p.k_k) - lo_k;
        const int lo_v = cut_v ? s_cut[2] : kThreads, len_v = (cut_v ? s_cut[3] : p.k_v) - lo_v;
        for (int j = tid; j < max(len_k, len_v); j += 2 * kThreads) {
            int e[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                e[0][u] = j + u * kThreads < len_k ? idx_k[lo_k + j + u * kThreads] : -1;
                e[1][u] = j + u * kThreads < len_v ? idx_v[lo_v + j + u * kThreads] : -1;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                note(s_slot_k, e[0][u], lo_k + j + u * kThreads);
                note(s_slot_v, e[1][u], lo_v + j + u * kThreads);
            }
        }
    } else {
        for (int j = tid + kThreads; j < p.k_k; j += kThreads) note(s_slot_k, idx_k[j], j);
        for (int j = tid + kThreads; j < p.k_v; j += kThreads) note(s_slot_v, idx_v[j], j);
    }
    // a word left by another launch, or by this one if it is replayed, is replaced by (tag, 0) by whoever gets there first
    if (tid == 0 && p.S > 1 && arrivals_are_stale(seen, p.tag, (uint32_t)p.S))
        __hip_atomic_compare_exchange_strong(&p.done[bg], &seen, (unsigned long long)p.tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    lds_barrier();

    // ------------------------------------------------------------------------------------------ tiles
    float m_ref = kNegBig, l_sum = 0.f;                             // head ln % 4: reference, this lane's share of the weights
    float4_t acc[8];                                                // register h: head h, channel 16 s + ln
#pragma unroll
    for (int s = 0; s < 8; ++s) acc[s] = float4_t{0.f, 0.f, 0.f, 0.f};
    const uint32_t rows0 = lds0 + Lds::rows + (uint32_t)wave * kTileBytes;

    for (int tile = wave; tile < n_tiles; tile += kWaves) {
        const int base = tile * kTile;
        // ---- operand rows of the keys: 8 channels 32 st + 8 kg of token 16 u + ln
        half8_t kop[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int slot = s_slot_k[base + 16 * u + ln];
            const half_t* row = rows_k + (int64_t)(slot < 0 ? 0 : slot) * kD + 8 * kg;
            const uint32_t (&w)[3] = codes.k[u];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const half_t* c;
                if constexpr (DSUB == 32) {
                    c = cbk + (uint32_t)(st * C + (int)code12(w, st)) * 32u + 8u * kg;
                } else {
                    const uint32_t code = kg & 2 ? code12(w, 2 * st + 1) : code12(w, 2 * st);
                    c = cbk + (uint32_t)((2 * st + (kg >> 1)) * C + (int)code) * 16u + 8u * (kg & 1);
                }
                kop[u][st] = *(const half8_t*)(slot < 0 ? c : row + 32 * st);
            }
        }
        // ---- the values' rows into LDS
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // those of the tile before have been read
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int slot = s_slot_v[base + 4 * i + kg];
            const int c = Codes::piece(i, lane);
            const half_t* cen = cbv + (uint32_t)(c * 8 / DSUB * C + (int)codes.v[i]) * (uint32_t)DSUB + (uint32_t)(8 * c % DSUB);
            gather_to_lds16(slot < 0 ? cen : rows_v + (int64_t)slot * kD + 8 * c, rows0 + 1024u * i);
        }
        if (tile + kWaves < n_tiles) codes.load(ck, cv, tile + kWaves, n, lane);
        // ---- scores: register r is token 16 u + 4 kg + r, head ln % 4
        float x[2][4], m_tile = kNegBig;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float4_t c4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < 4; ++st) c4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kop[u][st], qop[st], c4, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                x[u][r] = base + 16 * u + 4 * kg + r < n ? c4[r] * p.c1 : kNegBig;
                m_tile = fmaxf(m_tile, x[u][r]);
            }
        }
        m_tile = fmaxf(m_tile, __shfl_xor(m_tile, 16, 64));
        m_tile = fmaxf(m_tile, __shfl_xor(m_tile, 32, 64));
        const float m_new = fmaxf(m_ref, m_tile - kPShift12);
        if (tile != wave) {
            const float alpha = fast_exp2(m_ref - m_new);
            l_sum *= alpha;
#pragma unroll
            for (int h = 0; h < kNH; ++h) {
                const float ah = lane_value(alpha, h);
#pragma unroll
                for (int s = 0; s < 8; ++s) acc[s][h] *= ah;
            }
        }
        m_ref = m_new;
        // ---- weights, as the operand of the value product: element 4 u + r of k-group kg
        half8_t pa;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float w = fast_exp2(x[u][r] - m_new);         // masked: exp2 of -1e30
                l_sum += w;
                pa[4 * u + r] = (half_t)w;
            }
        // ---- values: slab s is channels 16 s .. + 15; a lane asks for 8 bytes (piece tq) of token 16 u + 4 kg + tj
        wait_all_loads();
        if (n - base < kTile) {                                     // rows behind the last token: whatever their code names, zeros
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (4 * i + kg >= n - base) *(uint4_t*)(smem + Lds::rows + wave * kTileBytes + 1024 * i + 16 * lane) = uint4_t{0u, 0u, 0u, 0u};
        }
        uint32_t at[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = 16 * u + 4 * kg + tj;
            at[u] = rows0 + (uint32_t)r * 256u + (uint32_t)(((tq >> 1) ^ swz(r)) << 4) + 8u * (tq & 1);
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const half4_t lo = read_tr16(at[0] ^ 32u * s), hi = read_tr16(at[1] ^ 32u * s);
            const half8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa, v, acc[s], 0, 0, 0);
        }
    }

    // ------------------------------------------------------------------------------------------ merge of the waves
    l_sum += __shfl_xor(l_sum, 16, 64);
    l_sum += __shfl_xor(l_sum, 32, 64);
    if (lane < kNH) {
        s_red[wave * 8 + lane] = m_ref;
        s_red[wave * 8 + 4 + lane] = l_sum;
    }
    lds_barrier();                                                  // everyone is done with the rows, too
    const int waves = n_tiles < kWaves ? n_tiles : kWaves;          // waves that had a tile
    float m_all[kNH], l_all[kNH];
    {
        const int ws = ln < waves ? ln : 0;                         // lane (kg, ln) looks at head kg of wave ln
        const float m_w = s_red[ws * 8 + kg], l_w = ln < waves ? s_red[ws * 8 + 4 + kg] : 0.f;
        const float m_r = row16_max(m_w), l_r = row16_sum(l_w * fast_exp2(m_w - m_r));
#pragma unroll
        for (int h = 0; h < kNH; ++h) {
            m_all[h] = lane_value(m_r, 16 * h);
            l_all[h] = lane_value(l_r, 16 * h);
        }
    }
    float4_t* s_mrg = (float4_t*)(smem + Lds::mrg);
    if (wave < waves) {
        float4_t f;
#pragma unroll
        for (int h = 0; h < kNH; ++h) f[h] = fast_exp2(lane_value(m_ref, h) - m_all[h]);
        // all four k-groups hold the same sums: each writes two slabs
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float4_t v = acc[i];
#pragma unroll
            for (int q = 1; q < 4; ++q)
#pragma unroll
                for (int h = 0; h < kNH; ++h) v[h] = kg == q ? acc[2 * q + i][h] : v[h];
            s_mrg[wave * kD + 16 * (2 * kg + i) + ln] = v * f;
        }
    }
    lds_barrier();
    float* part_bg = p.part + ((int64_t)b * p.Hq + h0) * p.S * (kD + 2);
    {
        const int h = tid & 3, dim = tid >> 2;
        const float* src = (const float*)s_mrg + tid;
        float v[kWaves], sum = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) v[w] = w < waves ? src[w * kNH * kD] : 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += v[w];
        if (h < nheads) {
            float m = m_all[0], l = l_all[0];
#pragma unroll
            for (int i = 1; i < kNH; ++i) {
                m = h == i ? m_all[i] : m;
                l = h == i ? l_all[i] : l;
            }
            if (p.S == 1) {
                p.out[((int64_t)b * p.Hq + h0 + h) * kD + dim] = (half_t)(l > 0.f ? sum / l : 0.f);
            } else {
                // device-scope stores write through this die's L2: the workgroup that merges may sit on another die
                float* dst = part_bg + ((int64_t)h * p.S + sp) * (kD + 2);
                __hip_atomic_store(dst + dim, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (dim == 0) {
                    __hip_atomic_store(dst + kD, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(dst + kD + 1, l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
    }
    if (p.S == 1) return;
    // ------------------------------------------------------------------------------------------ merge of the workgroups
    // Each wave waits until its stores are acknowledged, the barrier collects the waves, then one thread arrives: the last
    // arrival reads partials that have all reached the level its device-scope loads read from.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) *s_count = (int)(__hip_atomic_fetch_add(&p.done[bg], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kArrivalMask) + 1;
    __syncthreads();
    if (*s_count != p.S) return;
    auto ld = [](const float* q) { return __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    const int S = p.S;
    float m = kNegBig, l = 0.f;                                     // thread 32 h + s: statistics of slot s
    if (tid < kNH * kShortRanges && (tid >> 5) < nheads && (tid & 31) < S) {
        const float* ps = part_bg + ((int64_t)(tid >> 5) * S + (tid & 31)) * (kD + 2) + kD;
        m = ld(ps);
        l = ld(ps + 1);
    }
    static_assert(kThreads == kNH * kD, "a thread per head and channel");
    const int h = tid >> 7, dim = tid & (kD - 1);
    const float* pb = part_bg + (int64_t)h * S * (kD + 2) + dim;
    float v[kShortRanges];
#pragma unroll
    for (int i = 0; i < kShortRanges; ++i) v[i] = h < nheads && i < S ? ld(pb + i * (kD + 2)) : 0.f;
    float* s_w = (float*)(smem + Lds::slot_k);                      // [4 heads][32]: 2^(m_s - m)
    float* s_tot = s_w + kNH * kShortRanges;                        // [4]: sum of weights
    if (tid < kNH * kShortRanges) {
        float mm = row16_max(m);
        mm = fmaxf(mm, __shfl_xor(mm, 16, 64));
        const float w = fast_exp2(m - mm);
        float t = row16_sum(l * w);
        t += __shfl_xor(t, 16, 64);
        s_w[tid] = w;
        if ((tid & 31) == 0) s_tot[tid >> 5] = t;
    }
    lds_barrier();
    float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kShortRanges; ++i) a[i & 3] = fmaf(v[i], s_w[h * kShortRanges + i], a[i & 3]);
    if (h < nheads) {
        const float lt = s_tot[h];
        p.out[((int64_t)b * p.Hq + h0 + h) * kD + dim] = (half_t)(lt > 0.f ? ((a[0] + a[1]) + (a[2] + a[3])) / lt : 0.f);
    }
}

template <int DSUB>
hipError_t launch_t(unsigned grid, const ShortParams& p, hipStream_t st)
{
    static OncePerDevice once;
    const hipError_t e = allow_lds(once, (const void*)decode_short_kernel<DSUB>, Lds::total);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_short_kernel<DSUB>), dim3(grid), dim3(kThreads), Lds::total, st, p);
    return hipGetLastError();
}

}  // namespace

// The longest range that is faster here than through a table.  A token costs the gathers of its pieces out of the L2, which
// codebooks of more than two KV heads on one XCD (2 MB each, 4 MB of L2) overflow; fewer than 8 pairs do not fill the chip with
// 32 ranges each.  One step, tokens of a range here and through a table: d 32, 8 heads, 2500 40.5 and 47.4 us, 3125 46.8 and
// 50.4, 3750 55.5 and 54.9; 16 heads 3000 48.9 and 50.2, 4000 61.5 and 56.5; 2 heads 2000 37.8 and 42.6, 3000 49.6 and 44.6; 64
// pairs of 32 heads 1536 46 and 55, 3072 75 and 62; 128 pairs 2048 61 and 68.  d 16, 8 heads, 2500 62 and 67, 3125 73 and 69 (one
// or two query heads per KV head 2000 50.8 and 54.7, 3000 71 and 60); 16 heads 2000 57.4 and 57.0; 4 heads 1000 38 and 53, 2000
// 66 and 61; 32 heads, 64 pairs 256 26 and 59, 1536 74 and 68, 128 pairs 768 49 and 70, 1536 78 and 76.
static int most_tokens(const Geom& g)
{
    const int heads_per_xcd = g.Hkv % 8 == 0 ? g.Hkv / 8 : g.Hkv;
    const bool near = heads_per_xcd <= 2 && (int64_t)g.B * g.Hkv * kShortRanges >= 256;
    return g.d == 32 ? (near ? kShortTokens : 2048) : (near ? 1792 : 1280);
}

ShortPlan short_plan(const Geom& g, int64_t N)
{
    ShortPlan pl = {false, 0, 0, 0, 0};
    const int64_t pairs = (int64_t)g.B * g.Hkv;
    if (N < 1 || pairs < 1) return pl;
    int64_t most = pairs < 256 ? 256 / pairs : 1;
    if (most > kShortRanges) most = kShortRanges;
    int64_t chunk = ((N + most - 1) / most + 63) / 64 * 64;
    if (chunk < kShortLeast) chunk = kShortLeast;
    if (chunk > most_tokens(g)) return pl;
    pl.chunk = (int)chunk;
    pl.S = (int)((N + chunk - 1) / chunk);
    if (pairs * pl.S > 0x7fffffffLL) return pl;
    pl.on = true;
    pl.off_part = align_up((size_t)pairs * sizeof(unsigned long long));
    pl.total = pl.off_part + (pl.S > 1 ? align_up((size_t)g.B * g.Hq * pl.S * (kD + 2) * sizeof(float)) : 0);
    return pl;
}

hipError_t launch_decode_short(const Geom& g, const ShortPlan& pl, const DecodeArgs& a, void* ws, uint64_t tag, hipStream_t st)
{
    ShortParams p;
    p.q = a.q; p.codes_k = a.codes_k; p.codes_v = a.codes_v; p.cb_k = a.cb_k; p.cb_v = a.cb_v;
    p.idx_k = a.idx_k; p.idx_v = a.idx_v; p.rows_k = a.rows_k; p.rows_v = a.rows_v; p.out = a.out;
    p.done = (unsigned long long*)ws; p.part = (float*)((char*)ws + pl.off_part); p.tag = tag;
    p.N = a.N; p.N_cap = a.N_cap; p.k_k = (int)a.k_k; p.k_v = (int)a.k_v;
    p.c1 = a.scale * kLog2e; p.B = g.B; p.Hq = g.Hq; p.Hkv = g.Hkv; p.G = g.G; p.S = pl.S; p.chunk = pl.chunk;
    const unsigned grid = (unsigned)((int64_t)g.B * g.Hkv * pl.S);
    return g.d == 32 ? launch_t<32>(grid, p, st) : launch_t<16>(grid, p, st);
}

}  // namespace antkv
