// Causal attention over the prompt (paper Sec. 2.1) that also writes the softmax row statistics which the
// Anchor Score pass consumes (Alg. 1, first step: attention extended to return row maximum and row sum).
//
// A workgroup is 8 waves = G heads of a KV head's group x 8/G query tiles of 32 (4 x 2, 2 x 4 or 1 x 8), or 4 waves and half the
// query tiles: short prompts leave CUs idle or end with their longest rows, which then take half as long.  Its waves share
// the 32-key tiles of K and V, which go from global memory straight into LDS (16 bytes per lane, no registers), four
// tiles of each in flight or in use.
//   scores   S^T tile (keys on the MFMA row axis, queries on the column axis): lane (n, kh) owns query n and
//            16 of the tile's 32 keys, so the running softmax is lane-local; the two half-waves of a query meet only
//            when the reference moves and at the end.
//   output   O^T += V^T P^T, again with queries on the column axis: the B operand is the lane's own 16
//            probabilities (fp16), the A operand comes out of the V tile through ds_read_b64_tr_b16, and the
//            accumulator rows of a lane all belong to its query, so a moved reference rescales registers only.
// Probabilities are exp2 against a per-query reference that trails the running maximum: it moves only when a
// tile brings a score more than kPMax (log2 units) above it, which keeps fp16 P below 2^kPMax.
// One step of the loop works on three tiles at once: the softmax of tile t (VALU) is interleaved with the scores of tile
// t + 1 and the value product of tile t - 1 (16 MFMAs), none of which waits for it.
// Bound: the matrix cores under the power limit.  32768 tokens, 32 heads (8.8 TFLOP): with tiles staged through registers
// and softmax and products in turn 10.9 ms (matrix cores 38 % busy at 1.97 GHz), now 8.2 ms = 1.07 PFLOP/s (63 % at
// 1.61 GHz).  2 x 1531 tokens, 32 KV heads: 101 -> 55 us.
#include "lds_tile.h"

#include <type_traits>

namespace antkv {

namespace {

constexpr int kRing = 4;                                // tiles of K, and of V, in LDS
constexpr float kPMax = 12.f;
constexpr int64_t kPaMany = 384;                        // workgroups of eight waves from which they are used
constexpr float kMasked = -INFINITY;                    // a score that takes no part

__device__ __forceinline__ float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

template <int NW>                                       // waves of a workgroup: 8 or 4
__global__ __launch_bounds__(NW * 64, 2) void prefill_attn_kernel(
    const half_t* __restrict__ q, const half_t* __restrict__ k, const half_t* __restrict__ v, int64_t N, int64_t Nq,
    float c1, half_t* __restrict__ out, float* __restrict__ row_max, float* __restrict__ row_sum, int Hq, int Hkv, int G,
    int q_blocks)
{
    __shared__ __attribute__((aligned(1024))) unsigned char s_kv[2 * kRing * kTileBytes];     // K ring, V ring
    constexpr int kParts = 8 / NW;                                 // pieces of 1 KB of a tile that a wave moves
    lds_byte* lds = (lds_byte*)s_kv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // scalar, so that per-wave conditions are scalar branches
    const int n = lane & 31, kh = lane >> 5;
    const int bgs = gridDim.x / q_blocks;                          // B * Hkv
    const int bg = blockIdx.x % bgs, b = bg / Hkv, g = bg % Hkv;   // (heads fastest: 8 heads, one per XCD)
    const int64_t qblk = q_blocks - 1 - blockIdx.x / bgs;          // longest rows first
    const int q_tiles = NW / G;                                    // query tiles of the workgroup
    const int64_t q0 = (qblk * q_tiles + wave / G) * 32;
    const int h = g * G + wave % G;
    const int64_t qi = q0 + n;
    const int64_t qrow = qi < Nq ? qi : Nq - 1;
    const int qpos = (int)(N - Nq + qrow);                         // last key this lane's query sees
    const int first_pos = (int)(N - Nq + q0);                      // position of the tile's first query
    auto tiles_to = [&](int64_t q_end) { return (int)((N - Nq + (q_end < Nq ? q_end : Nq) + 31) >> 5); };   // key tiles seen by rows < q_end
    const int n_tiles = tiles_to((qblk + 1) * q_tiles * 32);       // of the workgroup
    const int my_tiles = q0 < Nq ? tiles_to(q0 + 32) : 0;          // of the wave
    const half_t* kbase = k + (int64_t)bg * N * kD;
    const half_t* vbase = v + (int64_t)bg * N * kD;

    // staging: a wave moves kParts x 4 rows of a tile, a lane the chunk that belongs at its place of the 1 KB; rows
    // past the end repeat the last one, tiles past the end the last tile
    const int last_tile = (int)((N - 1) >> 5);
    uint32_t soff[kParts], soff_last[kParts];
#pragma unroll
    for (int i = 0; i < kParts; ++i) {
        soff[i] = stage_off(wave * kParts + i, lane, 31);
        soff_last[i] = stage_off(wave * kParts + i, lane, (int)(N - 1) & 31);
    }
    const uint32_t to0 = (uint32_t)(uintptr_t)lds + wave * (kParts * 1024);
    auto stage = [&](const half_t* base, int tile, uint32_t slot) {
        const int tc = tile < last_tile ? tile : last_tile;
#pragma unroll
        for (int i = 0; i < kParts; ++i)
            load_to_lds16((const unsigned char*)base + (int64_t)tc * kTileBytes, tc == last_tile ? soff_last[i] : soff[i],
                          to0 + slot * kTileBytes + 1024 * i);
    };
    // operand addresses inside a tile: K row n, channels 16 s + 8 kh .. + 7; V transposed: inside a 16-lane block, lane
    // 4 e + c reads key row e of the lane's four, channels 4 c .. 4 c + 3 of 16; blocks 0/1 cover the two channel halves
    // of a 32-channel group, blocks 2/3 the same for the other key half
    uint32_t k_at[8], v_at[4][2];
#pragma unroll
    for (int s = 0; s < 8; ++s) { k_at[s] = tile_at(n, s, kh); pin(k_at[s]); }
    {
        const int e = (lane & 15) >> 2, c = lane & 3, blk = (lane >> 4) & 1;
#pragma unroll
        for (int cg = 0; cg < 4; ++cg)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int row = 8 * j + 4 * kh + e;
                v_at[cg][j] = kRing * kTileBytes + row * 256 + (((4 * cg + 2 * blk + (c >> 1)) ^ swz(row)) << 4) + 8 * (c & 1);
                pin(v_at[cg][j]);
            }
    }

    for (int i = 0; i < 4; ++i) stage(kbase, i, i);
    for (int i = 0; i < 2; ++i) stage(vbase, i, kRing + i);
    // the V slot of "tile -1" is multiplied with zero probabilities: it has to be finite
#pragma unroll
    for (int i = 0; i < kParts; ++i) *(uint4_t*)(s_kv + (2 * kRing - 1) * kTileBytes + (i * NW * 64 + tid) * 16) = uint4_t{0u, 0u, 0u, 0u};
    half8_t tq[8];
    {
        const half_t* qp = q + (((int64_t)b * Hq + h) * Nq + qrow) * kD + 8 * kh;
#pragma unroll
        for (int s = 0; s < 8; ++s) tq[s] = *(const half8_t*)(qp + 16 * s);
#pragma unroll
        for (int s = 0; s < 8; ++s) pin(tq[s]);
    }
    wait_all_loads();
    __syncthreads();

    float16_t o[4], sc[2];
    half8_t p[2][2];
#pragma unroll
    for (int cg = 0; cg < 4; ++cg)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[cg][r] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) p[1][i][j] = (half_t)0.f;
    float m_ref = kNegBig, s_max = kMasked, l_run = 0.f;            // reference (log2 units), largest raw score, sum
    auto k_op = [&](int s, int slot) { return *(lds_half8*)(lds + k_at[s] + slot * kTileBytes); };
    auto v_op = [&](int i, int slot) {                              // i = 4 * (16-key half) + channel group
        const lds_byte* at = lds + slot * kTileBytes + (i >> 2) * 16 * 256;
        const half4_t a = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(at + v_at[i & 3][0])));
        const half4_t c = __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(at + v_at[i & 3][1])));
        return half8_t{a[0], a[1], a[2], a[3], c[0], c[1], c[2], c[3]};
    };
    {
        float16_t z;
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r] = 0.f;
        sc[0] = z;
#pragma unroll
        for (int s = 0; s < 8; ++s) sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(k_op(s, 0), tq[s], sc[0], 0, 0, 0);
    }
    __syncthreads();                                                // step 0 stages over the tile that has just been read

    // before the exponentials of tile t: mask, largest score, reference; true if it moves (o has to be rescaled by alpha)
    auto open_tile = [&](float16_t& s, int t, float& alpha) __attribute__((always_inline)) {
        if (__builtin_expect(t * 32 + 31 > first_pos, 0)) {         // the causal diagonal: key offset <= lim is visible
            const int lim = qpos - t * 32;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + 4 * kh + (r & 3) > lim) s[r] = kMasked;
        }
        s_max = max3f(s_max, s[0], s[1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) s_max = max3f(s_max, s[r], s[r + 1]);
        alpha = 1.f;
        const bool moves = __any(fmaf(s_max, c1, -m_ref) > kPMax);
        if (__builtin_expect(moves, 0)) {                           // the reference moves to the largest score so far
            const float m_new = fmaxf(s_max, __shfl_xor(s_max, 32, 64)) * c1;
            if (m_new - m_ref > kPMax) {
                alpha = fast_exp2(m_ref - m_new);
                l_run *= alpha;
                m_ref = m_new;
            }
        }
        return moves;
    };
    auto rescale = [&](float alpha) __attribute__((always_inline)) {
#pragma unroll
        for (int cg = 0; cg < 4; ++cg)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[cg][r] *= alpha;
    };

    // step t, T = t mod 4
    auto step = [&](int t, auto phase) __attribute__((always_inline)) {
        constexpr int T = decltype(phase)::value;
        constexpr int kNext = (T + 1) & 3, kPrev = (T + 3) & 3, cur = T & 1, nxt = cur ^ 1;
        stage(kbase, t + 4, T);                                     // (tiles past the end repeat the last row)
        stage(vbase, t + 2, kRing + ((T + 2) & 3));
        float16_t& s = sc[cur];
        float alpha;
        const bool moves = open_tile(s, t, alpha);
        half8_t ka[8], va[8];
        ka[0] = k_op(0, kNext); va[0] = v_op(0, kPrev);
        ka[1] = k_op(1, kNext); va[1] = v_op(1, kPrev);
        float sum[2] = {0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[nxt][r] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i + 2 < 8) { ka[i + 2] = k_op(i + 2, kNext); va[i + 2] = v_op(i + 2, kPrev); }
            sc[nxt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ka[i], tq[i], sc[nxt], 0, 0, 0);              // rows = keys, cols = queries
            float p0 = fast_exp2(fmaf(s[2 * i], c1, -m_ref));
            sum[0] += p0;
            o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[i], p[nxt][i >> 2], o[i & 3], 0, 0, 0);   // rows = channels
            float p1 = fast_exp2(fmaf(s[2 * i + 1], c1, -m_ref));
            sum[1] += p1;
            pin(sum[0]);                                            // (the products must not sink below the loop)
            pin(sum[1]);
            // k-slot j of half kh in 16-key half i is key 16 i + 8 (j >> 2) + 4 kh + (j & 3), on both operands
            p[cur][i >> 2][(2 * i) & 7] = (half_t)p0;
            p[cur][i >> 2][(2 * i + 1) & 7] = (half_t)p1;
            __builtin_amdgcn_sched_barrier(0);
        }
        l_run += sum[0] + sum[1];
        if (__builtin_expect(moves, 0)) rescale(alpha);
        landed_but<4 * kParts>();                                   // this step's two tiles and the last one's
    };
    // Whole groups of four tiles are interleaved; up to three more go one after the other, so that the loop has one end with
    // the registers in the same roles (four ends spill).  No tile past the wave's last is touched: its V rows, which no
    // query of the wave sees, would meet zero probabilities (inf * 0).
    int t = 0;
    for (; t + 4 <= my_tiles; t += 4) {
        step(t, std::integral_constant<int, 0>{});
        step(t + 1, std::integral_constant<int, 1>{});
        step(t + 2, std::integral_constant<int, 2>{});
        step(t + 3, std::integral_constant<int, 3>{});
    }
    auto stage_ahead = [&](int t) {
        stage(kbase, t + 4, t & 3);
        stage(vbase, t + 2, kRing + ((t + 2) & 3));
    };
    auto last_product = [&](int t) __attribute__((always_inline)) {                                // the value product of tile t - 1
#pragma unroll
        for (int i = 0; i < 8; ++i)
            o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(v_op(i, (t + 3) & 3), p[1][i >> 2], o[i & 3], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);                          // (V has been read before another wave stages over it)
    };
#pragma unroll 1
    for (; t < my_tiles; ++t) {
        stage_ahead(t);
        last_product(t);
        float alpha;
        if (open_tile(sc[0], t, alpha)) rescale(alpha);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float e = fast_exp2(fmaf(sc[0][r], c1, -m_ref));
            l_run += e;
            p[1][r >> 3][r & 7] = (half_t)e;
            sc[0][r] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(k_op(i, (t + 1) & 3), tq[i], sc[0], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        landed_but<4 * kParts>();
    }
    last_product(t);
    for (; t < n_tiles; ++t) {                                      // waves that are done keep staging for the others
        stage_ahead(t);
        landed_but<4 * kParts>();
    }
    wait_all_loads();                                               // nothing may land in LDS after the workgroup's end
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    s_max = fmaxf(s_max, __shfl_xor(s_max, 32, 64));
    if (qi < Nq) {
        const int64_t row = ((int64_t)b * Hq + h) * Nq + qi;
        const float inv = 1.f / l_tot;
        half_t* op = out + row * kD + 4 * kh;
#pragma unroll
        for (int cg = 0; cg < 4; ++cg)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {                        // accumulator rows 8 qd + 4 kh + e = channels of group cg
                half4_t w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = (half_t)(o[cg][4 * qd + e] * inv);
                *(half4_t*)(op + 32 * cg + 8 * qd) = w;
            }
        if (kh == 0 && row_max) {
            row_max[row] = s_max * c1 * (1.f / kLog2e);
            row_sum[row] = l_tot * fast_exp2(fmaf(-s_max, c1, m_ref));
        }
    }
}

}  // namespace

hipError_t launch_prefill_attn(const Geom& g, const half_t* q, const half_t* k, const half_t* v, int64_t N, int64_t Nq,
                               float scale, half_t* out, float* row_max, float* row_sum, hipStream_t st)
{
    const int64_t pairs = (int64_t)g.B * g.Hkv;
    auto blocks = [&](int nw) { const int64_t span = 32 * (nw / g.G); return (Nq + span - 1) / span; };
#define ANTKV_PA(NW)                                                                                                       \
    hipLaunchKernelGGL(prefill_attn_kernel<NW>, dim3((unsigned)(blocks(NW) * pairs)), dim3(NW * 64), 0, st, q, k, v, N, Nq, scale * kLog2e, \
                       out, row_max, row_sum, g.Hq, g.Hkv, g.G, (int)blocks(NW))
    // Twice the workgroups read K and V twice as often.  32 heads, 8 and 4 waves, by workgroups of 8: 64 (500 tokens) 19.1 and 14.7 us,
    // 128 29.5 and 22.9, 192 41.2 and 34.5, 256 33.5 and 29.7, 320 69.8 and 63.7, 376 161 and 150, 384 52.0 and 52.2, 512 136 and 140,
    // 640 123 and 119, 1024 271 and 272, 2048 560 and 580.
    if (blocks(8) * pairs < kPaMany) ANTKV_PA(4);
    else ANTKV_PA(8);
#undef ANTKV_PA
    return hipGetLastError();
}

}  // namespace antkv
