// Anchor Score (paper Eq. (4); two-phase procedure of Alg. 1, Sec. 3.3):
//   AnS(V_j) = sum_i A_ij,   AnS(K_j) = sum_i A_ij (1 - A_ij) ||Q_i||_2,   A = causal softmax(scale Q K^T),
// summed over the query heads of a KV head.  A is never materialised.
//
//   phase 1  row statistics: per (head, query row) the running max and sum of exp over the visible keys.
//            MFMA tile with keys on the row axis and queries on the column axis, so a lane owns one query
//            and reduces over keys in its own registers.  Long contexts with few query rows are split
//            over the key axis; a small kernel merges the splits and adds ||Q_i||_2.
//            (Skipped when the caller supplies row max / row sum, as an extended attention kernel would.)
//   phase 2  column reduction: per (KV head, block of keys) loop over the group's heads and all query
//            tiles that can see the block, rebuild A = exp2(S*c1 - c_i) from the row statistic
//            c_i = max_i*log2(e) + log2(sum_i), and reduce over queries.  Queries sit on the MFMA row
//            axis and keys on the column axis, so a lane owns one key; per-tile partial sums are fp32,
//            the running column sums are fp64.
// All contractions are v_mfma_f32_32x32x16_f16 on the raw fp16 Q and K (exact products, fp32 accumulate);
// the softmax scale is applied to the fp32 result.
#include "lds_tile.h"

#include <type_traits>

namespace antkv {

namespace {

constexpr int kAsThreads = 512;   // 8 waves

// MFMA operand for 32 rows x 128 channels: lane (r = lane%32, kh = lane/32) holds, for each of the
// 8 k-steps s, the 8 channels 16*s + 8*kh .. +7 of row r.
struct Tile128 {
    half8_t v[8];
};

__device__ __forceinline__ void load_tile(Tile128& t, const half_t* row_ptr, int kh)
{
#pragma unroll
    for (int s = 0; s < 8; ++s) t.v[s] = *(const half8_t*)(row_ptr + 16 * s + 8 * kh);
#pragma unroll
    for (int s = 0; s < 8; ++s) pin(t.v[s]);
}

// A 32-row x 128-channel tile shared by the waves of a workgroup sits in LDS with rows padded to 136 halfs
// (272 bytes): the 16 lanes that one 16-byte LDS read serves per clock then fall on 16 different bank quads.
constexpr int kRowPad = 136;
constexpr int kTileHalfs = 32 * kRowPad;

// rows x staged tile: the staged tile is the A operand (rows of the result), the register tile the B operand
__device__ __forceinline__ float16_t tile_dot_lds_a(const half_t* __restrict__ st, const Tile128& b, int n, int kh)
{
    float16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const half8_t a = *(const half8_t*)(st + n * kRowPad + 16 * s + 8 * kh);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b.v[s], acc, 0, 0, 0);
    }
    return acc;
}

// -------------------------------------------------------------------------------------------------
// phase 1: partial row statistics.  grid = (key splits, query blocks, B*Hkv); 8 waves = HG heads of the
// group x 8/HG query tiles of 32 with HG = min(G, 4), so that no wave idles for small groups (larger groups loop).
// part: [B][Hq][Nq][KS][2] = (max in log2 units, sum of exp2)
// -------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kAsThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void ans_row_stats(
    const half_t* __restrict__ q, const half_t* __restrict__ k, int64_t N, int64_t Nq, float c1,
    float* __restrict__ part, int Hq, int Hkv, int G, int KS, int64_t keys_per_split)
{
    __shared__ __attribute__((aligned(16))) half_t s_k[2][kTileHalfs];   // key tiles, double-buffered
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, kh = lane >> 5;
    const int ks = blockIdx.x;
    const int64_t qblk = blockIdx.y;
    const int b = blockIdx.z / Hkv, g = blockIdx.z % Hkv;
    const int HG = G >= 4 ? 4 : G;                              // head slots of the workgroup
    const int qspan = 32 * (8 / HG);                            // query rows per workgroup
    const int64_t q0 = qblk * qspan + (wave >> (HG >> 1)) * 32;        // first query row of this wave's tile
    const bool wave_on = q0 < Nq;
    const int64_t qi = q0 + n;                                  // this lane's query row
    const int64_t qrow = qi < Nq ? qi : Nq - 1;
    const int64_t qpos = N - Nq + qrow;                         // absolute position = last visible key
    const int64_t tile_last_pos = N - Nq + ((q0 + 31 < Nq) ? q0 + 31 : Nq - 1);
    const int64_t k_lo = (int64_t)ks * keys_per_split;
    // keys this workgroup walks: up to the last key any of its queries can see
    const int64_t blk_last_pos = N - Nq + ((qblk * qspan + qspan - 1 < Nq) ? qblk * qspan + qspan - 1 : Nq - 1);
    int64_t k_end = k_lo + keys_per_split;
    if (k_end > blk_last_pos + 1) k_end = blk_last_pos + 1;
    int64_t k_hi = k_lo + keys_per_split;                       // this wave's own limit
    if (k_hi > tile_last_pos + 1) k_hi = tile_last_pos + 1;
    const half_t* kbase = k + ((int64_t)b * Hkv + g) * N * kD;
    // staging: thread t moves 16 bytes: row t / 16, chunk t % 16 of the tile
    const int srow = tid >> 4, schunk = tid & 15;
    auto fetch = [&](int64_t kt) -> uint4_t {
        const int64_t krow = (kt + srow < N) ? kt + srow : N - 1;
        return *(const uint4_t*)(kbase + krow * kD + 8 * schunk);
    };

    for (int h_it = 0; h_it < (G + HG - 1) / HG; ++h_it) {
        const int hh = HG * h_it + (wave & (HG - 1));
        const bool head_on = wave_on && hh < G;
        const int h = g * G + (hh < G ? hh : G - 1);
        Tile128 tq;
        load_tile(tq, q + (((int64_t)b * Hq + h) * Nq + qrow) * kD, kh);
        wait_all_loads();
        float m_run = kNegBig, l_run = 0.f;
        // One-step software pipeline: the scores of tile t+1 are computed while the statistics of tile t are
        // updated, so LDS holds tiles t+1 (read) and t+2 (being written); tile t's buffer is the one rewritten.
        if (k_lo < k_end) *(uint4_t*)(&s_k[0][srow * kRowPad + 8 * schunk]) = fetch(k_lo);
        if (k_lo + 32 < k_end) *(uint4_t*)(&s_k[1][srow * kRowPad + 8 * schunk]) = fetch(k_lo + 32);
        __syncthreads();
        float16_t acc_cur;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_cur[r] = 0.f;
        if (head_on && k_lo < k_hi) acc_cur = tile_dot_lds_a(s_k[0], tq, n, kh);   // rows = keys, cols = queries
        __syncthreads();                                            // the first step writes tile 2 over the tile that has just been read
        int buf = 0;                                                // buffer of tile t
        for (int64_t kt = k_lo; kt < k_end; kt += 32) {
            const bool more = kt + 64 < k_end;
            uint4_t nxt = {0u, 0u, 0u, 0u};
            if (more) nxt = fetch(kt + 64);
            if (head_on && kt < k_hi) {
                // Exponents are taken against this lane's reference m_run, which only moves when a tile brings
                // a score more than 64 (log2 units) above it, or when the lane has seen nothing yet: the common
                // tile costs one fma, one exp2, one add and one max per element.
                const bool init = m_run > kNegBig;
                const float base = init ? m_run : 0.f;
                float arg[16];
                float mx = kNegBig, sum = 0.f;
                float16_t acc_next;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_next[r] = 0.f;
                const int lim_q = (int)(qpos - kt), lim_k = (int)(k_hi - kt);   // visible: offset <= lim_q, < lim_k
                auto body = [&](auto masked) {
                    const half_t* ap = &s_k[buf ^ 1][n * kRowPad + 8 * kh];
                    half8_t a_op[8];
                    a_op[0] = *(const half8_t*)(ap);
                    a_op[1] = *(const half8_t*)(ap + 16);
#pragma unroll
                    for (int s = 0; s < 8; ++s) {
                        if (s + 2 < 8) a_op[s + 2] = *(const half8_t*)(ap + 16 * (s + 2));
                        acc_next = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_op[s], tq.v[s], acc_next, 0, 0, 0);
#pragma unroll
                        for (int e2 = 0; e2 < 2; ++e2) {
                            const int r = 2 * s + e2;
                            float x = fmaf(acc_cur[r], c1, -base);
                            if (decltype(masked)::value) {
                                const int off = 8 * (r >> 2) + 4 * kh + (r & 3);
                                if (!((off <= lim_q) && (off < lim_k))) x = kNegBig;
                            }
                            arg[r] = x;
                            mx = fmaxf(mx, x);
                            sum += fast_exp2(x);
                        }
                    }
                };
                // every key of the tile is visible to every query of the wave: no mask
                if (kt + 31 <= N - Nq + q0 && kt + 31 < k_hi) body(std::false_type{});
                else body(std::true_type{});
                if (init && mx <= 64.f) {
                    l_run += sum;
                } else if (mx > 0.5f * kNegBig) {                  // the tile has a visible element: move the reference
                    float sum2 = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum2 += fast_exp2(arg[r] - mx);
                    l_run = (init ? l_run * fast_exp2(-mx) : 0.f) + sum2;
                    m_run = base + mx;
                }
                acc_cur = acc_next;
            }
            if (more) *(uint4_t*)(&s_k[buf][srow * kRowPad + 8 * schunk]) = nxt;
            __syncthreads();
            buf ^= 1;
        }
        // merge the two half-waves (they saw complementary keys of the same query)
        const float m_o = __shfl_xor(m_run, 32, 64), l_o = __shfl_xor(l_run, 32, 64);
        const float m_f = fmaxf(m_run, m_o);
        const float l_f = l_run * fast_exp2(m_run - m_f) + l_o * fast_exp2(m_o - m_f);
        if (head_on && kh == 0 && qi < Nq) {
            float* p = part + ((((int64_t)b * Hq + h) * Nq + qi) * KS + ks) * 2;
            p[0] = m_f;
            p[1] = l_f;
        }
        __syncthreads();
    }
}

// merge key splits -> c_i = m + log2(l); also ||Q_i||_2.  One 16-lane group per (b, h, i).  Written as tiles of 32 rows,
// {-c_i x 32, ||Q_i|| x 32}; rows past Nq and one tile behind the last hold {-inf, 0}, which makes their weights zero.
// Clears the arrival counters of phase 2, too.
constexpr int kStatTile = 64;

__global__ __launch_bounds__(256) void ans_finalize_stats(
    const half_t* __restrict__ q, const float* __restrict__ part, int KS, const float* __restrict__ row_max,
    const float* __restrict__ row_sum, float* __restrict__ stat, int64_t Nq, int q_tiles, int64_t n_heads, const ClearWords clear)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t; i < clear.n; i += (int64_t)gridDim.x * blockDim.x) clear.at[i] = 0u;
    const int64_t slot = t >> 4;                                 // padded row
    const int part_i = (int)(t & 15);
    const int64_t head = slot / ((int64_t)q_tiles * 32), i = slot - head * q_tiles * 32;
    if (head > n_heads || (head == n_heads && i >= 32)) return;
    float* out = stat + (slot >> 5) * kStatTile + (slot & 31);
    if (head == n_heads || i >= Nq) {
        if (part_i == 0) { out[0] = -INFINITY; out[32] = 0.f; }
        return;
    }
    const int64_t row = head * Nq + i;
    const half8_t v = *(const half8_t*)(q + row * kD + part_i * 8);
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) s = fmaf((float)v[e], (float)v[e], s);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (row_max) {
        if (part_i == 0) {
            out[0] = -(row_max[row] * kLog2e + log2f(row_sum[row]));
            out[32] = sqrtf(s);
        }
        return;
    }
    // the 16 lanes of the group share the KS partial (reference, sum) pairs, then combine
    float m = kNegBig, l = 0.f;
    for (int j = part_i; j < KS; j += 16) {
        const float2 ml = *(const float2*)(part + (row * KS + j) * 2);
        const float mn = fmaxf(m, ml.x);
        l = l * exp2f(m - mn) + ml.y * exp2f(ml.x - mn);
        m = mn;
    }
    float mg = m;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) mg = fmaxf(mg, __shfl_xor(mg, off, 64));
    l *= exp2f(m - mg);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) l += __shfl_xor(l, off, 64);
    if (part_i == 0) {
        out[0] = -(mg + log2f(l));
        out[32] = sqrtf(s);
    }
}

// -------------------------------------------------------------------------------------------------
// phase 2: column reduction.  A workgroup of NW waves walks the (head, query tile) steps that can see its keys; a wave owns
// KT tiles of 32 keys, kept in registers, and reads the query tile and its row statistics from LDS, where they go straight
// from global memory, three to four steps ahead.  While the VALU rebuilds and reduces the probabilities of step t the
// matrix cores compute the scores of step t + 1.
// Bound: VALU issue, per element one fma, one exp2 (8 clocks), one add and two fma (2.6 each).  32768 x 32768, 32 heads:
// 8.8 ms with tiles staged through registers and 32 keys per wave, 5.4 ms now.
// -------------------------------------------------------------------------------------------------
// SPLIT: few keys leave CUs idle while a workgroup walks all heads and queries; `splits` workgroups then take a part of the steps
// each, and the last of a key block to arrive adds up their fp64 sums.
struct ColSplit {
    int splits;
    double* sums;                                               // [splits][V, K][B * Hkv][N]
    uint32_t* done;                                             // [key blocks][B * Hkv] arrivals, cleared by ans_finalize_stats
};

template <int KT, int NW, bool SPLIT>
__global__ __launch_bounds__(NW * 64, 2) void ans_col_reduce(
    const half_t* __restrict__ q, const half_t* __restrict__ k, int64_t N, int64_t Nq, float c1,
    const float* __restrict__ stat, float* __restrict__ ans_k, float* __restrict__ ans_v, int Hq, int Hkv, int G,
    int64_t n_bg, int q_tiles, const ColSplit sp)
{
    constexpr int kRing = 4, kParts = 8 / NW;                   // pieces of 1 KB of a query tile per wave
    constexpr int kStatBytes = kStatTile * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[kRing * (kTileBytes + kStatBytes)];
    lds_byte* lds = (lds_byte*)s_mem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, kh = lane >> 5;
    const int bg = (int)(blockIdx.x % n_bg), b = bg / Hkv, g = bg % Hkv;    // (heads fastest: 8 heads, one per XCD)
    const int64_t rest = blockIdx.x / n_bg, kblk = SPLIT ? rest / sp.splits : rest;
    const int part = SPLIT ? (int)(rest % sp.splits) : 0;
    const int64_t kblk0 = kblk * (32 * KT * NW);                            // the first keys have the most queries: longest first
    const int64_t k0 = kblk0 + wave * (32 * KT);                            // first key of this wave
    half8_t tk[KT][8];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
        const int64_t key = k0 + 32 * kt + n;
        const half_t* kp = k + ((int64_t)bg * N + (key < N ? key : N - 1)) * kD + 8 * kh;
#pragma unroll
        for (int s = 0; s < 8; ++s) tk[kt][s] = *(const half8_t*)(kp + 16 * s);
    }
    // first query tile that can see a key of this block:  N - Nq + i >= kblk0
    int64_t i_first = kblk0 - (N - Nq);
    if (i_first < 0) i_first = 0;
    const int qt_first = (int)(i_first >> 5);
    const int n_qt = q_tiles - qt_first, all_steps = n_qt * G;   // query tiles per head; step = (head of the group, query tile)
    const int step0 = SPLIT ? (int)((int64_t)all_steps * part / sp.splits) : 0;
    const int n_steps = (SPLIT ? (int)((int64_t)all_steps * (part + 1) / sp.splits) : all_steps) - step0;    // (a part may be empty)
    const int qt_0 = SPLIT ? step0 % n_qt : 0;                   // query tile of the first step
    const int64_t head0 = (int64_t)b * Hq + (int64_t)g * G + (SPLIT ? step0 / n_qt : 0);

    uint32_t soff[kParts], soff_last[kParts];
#pragma unroll
    for (int i = 0; i < kParts; ++i) {
        soff[i] = stage_off(wave * kParts + i, lane, 31);
        soff_last[i] = stage_off(wave * kParts + i, lane, (int)(Nq - 1) & 31);
    }
    const uint32_t to_q = (uint32_t)(uintptr_t)lds, to_s = to_q + kRing * kTileBytes;
    // the steps are staged in order: from tile to tile, from a head's last tile to the next head's first, and behind the
    // last step the last tile again with the neutral statistics
    const int64_t q_wrap = Nq * (kD * 2) - (int64_t)(n_qt - 1) * kTileBytes, s_wrap = (int64_t)(qt_first + 1) * kStatBytes;
    const unsigned char* q_ptr = (const unsigned char*)(q + (head0 * Nq + (int64_t)(qt_first + qt_0) * 32) * kD);
    const unsigned char* s_ptr = (const unsigned char*)(stat + (head0 * q_tiles + qt_first + qt_0) * kStatTile);
    const unsigned char* s_none = (const unsigned char*)(stat + (n_bg / Hkv) * Hq * q_tiles * kStatTile);
    int q_left = n_steps, s_left = n_steps, q_row = n_qt - qt_0, s_row = n_qt - qt_0;      // steps to stage, tiles left of the head
    auto stage_q = [&](uint32_t slot) {
        const bool last = q_row == 1;
#pragma unroll
        for (int i = 0; i < kParts; ++i)
            load_to_lds16(q_ptr, last ? soff_last[i] : soff[i], to_q + slot * kTileBytes + (wave * kParts + i) * 1024);
        if (--q_left > 0) {
            q_ptr += last ? q_wrap : (int64_t)kTileBytes;
            q_row = last ? n_qt : q_row - 1;
        }
    };
    auto stage_s = [&](uint32_t slot) {                          // (every wave writes the same values)
        load_to_lds4(s_left > 0 ? s_ptr : s_none, lane * 4, to_s + slot * kStatBytes);
        --s_left;
        const bool last = s_row == 1;
        s_ptr += last ? s_wrap : (int64_t)kStatBytes;
        s_row = last ? n_qt : s_row - 1;
    };
    uint32_t q_at[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) { q_at[s] = tile_at(n, s, kh); pin(q_at[s]); }
    const uint32_t s_at = kRing * kTileBytes + 16 * kh;
    auto q_op = [&](int s, int slot) { return *(lds_half8*)(lds + q_at[s] + slot * kTileBytes); };
    auto stat_op = [&](int qd, int which, int slot) { return *(lds_float4*)(lds + s_at + slot * kStatBytes + which * 128 + qd * 32); };

    for (int i = 0; i < 4; ++i) stage_q(i);
    for (int i = 0; i < 3; ++i) stage_s(i);
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int s = 0; s < 8; ++s) pin(tk[kt][s]);
    wait_all_loads();
    __syncthreads();
    float16_t sc[2][KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[0][kt][r] = 0.f;
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const half8_t a = q_op(s, 0);
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) sc[0][kt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, tk[kt][s], sc[0][kt], 0, 0, 0);   // rows = queries, cols = keys
    }
    __syncthreads();                                             // step 0 stages over the tile that has just been read
    double sum_v[KT], sum_k[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) sum_v[kt] = sum_k[kt] = 0.0;
    int qt = qt_0;                                               // query tile of the current step
    const int rel0 = (int)(N - Nq + (int64_t)qt_first * 32 - k0);   // position of tile 0's first query minus this wave's first key

    auto step = [&](auto phase) __attribute__((always_inline)) { // a step whose number is T mod 4
        constexpr int T = decltype(phase)::value;
        constexpr int kNext = (T + 1) & 3, cur = T & 1, nxt = cur ^ 1;
        stage_q(T);                                              // step + 4
        stage_s((T + 3) & 3);                                    // step + 3
        const int rel = rel0 + 32 * qt;
        if (__builtin_expect(rel < 32 * KT - 1, 0)) {            // some query of the tile does not see some key of the wave
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const int lim = n + 32 * kt - rel;               // tile row r sees this lane's key iff r >= lim
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + 4 * kh + (r & 3) < lim) sc[cur][kt][r] = -INFINITY;
            }
        }
        if (++qt == n_qt) qt = 0;
        half8_t a[8];
        float4_t c4[4], n4[4];
        a[0] = q_op(0, kNext);
        c4[0] = stat_op(0, 0, T);
        n4[0] = stat_op(0, 1, T);
        a[1] = q_op(1, kNext);
        float pv[KT], pk[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            pv[kt] = pk[kt] = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) sc[nxt][kt][r] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {                            // tile rows 8 qd + 4 kh + e live in register 4 qd + e
            if (i + 2 < 8) a[i + 2] = q_op(i + 2, kNext);
            if ((i & 1) == 1 && i < 7) { c4[(i >> 1) + 1] = stat_op((i >> 1) + 1, 0, T); n4[(i >> 1) + 1] = stat_op((i >> 1) + 1, 1, T); }
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                sc[nxt][kt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], tk[kt][i], sc[nxt][kt], 0, 0, 0);
#pragma unroll
                for (int e2 = 0; e2 < 2; ++e2) {
                    const int r = 2 * i + e2;
                    const float c = c4[r >> 2][r & 3], nn = n4[r >> 2][r & 3];
                    const float w = fast_exp2(fmaf(sc[cur][kt][r], c1, c));
                    pv[kt] += w;
                    pk[kt] = fmaf(w, fmaf(-w, nn, nn), pk[kt]);  // a (1 - a) ||q||
                }
                pin(pv[kt]);                                     // (keeps the work where it is written)
                pin(pk[kt]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {                        // fp32 per tile, fp64 over tiles
            sum_v[kt] += (double)pv[kt];
            sum_k[kt] += (double)pk[kt];
        }
        landed_but<2 * (kParts + 1)>();                          // this step's loads and the last one's
    };
    // Whole groups of four in the loop, the rest behind it: rounded up to four (with neutral statistics) 300 queries x 131072
    // keys x 8 heads of one query head each took 350 us for the whole selection, now 327.
    int left = n_steps;
    for (; left >= 4; left -= 4) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
    }
    if (left > 0) step(std::integral_constant<int, 0>{});
    if (left > 1) step(std::integral_constant<int, 1>{});
    if (left > 2) step(std::integral_constant<int, 2>{});
    wait_all_loads();                                            // nothing may land in LDS after the workgroup's end
    if constexpr (SPLIT) {
        static_assert(KT == 1, "a key per lane");
        double v = sum_v[0] + __shfl_xor(sum_v[0], 32, 64), kk = sum_k[0] + __shfl_xor(sum_k[0], 32, 64);
        const int64_t key = k0 + n, plane = n_bg * N, at = (int64_t)bg * N + key;
        const bool on = kh == 0 && key < N;
        if (on) {                                                // device-scope stores: the last workgroup may sit on another die
            __hip_atomic_store(sp.sums + 2 * part * plane + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(sp.sums + (2 * part + 1) * plane + at, kk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_s_waitcnt(0);                           // acknowledged before the workgroup arrives
        __syncthreads();
        int* s_last = (int*)s_mem;
        if (tid == 0)
            *s_last = (int)__hip_atomic_fetch_add(&sp.done[kblk * n_bg + bg], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
        __syncthreads();
        if (*s_last != sp.splits || !on) return;
        v = kk = 0.0;
        for (int i = 0; i < sp.splits; ++i) {
            v += __hip_atomic_load(sp.sums + 2 * i * plane + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            kk += __hip_atomic_load(sp.sums + (2 * i + 1) * plane + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        ans_v[at] = (float)v;
        ans_k[at] = (float)kk;
        return;
    }
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {                            // lanes l and l+32 hold complementary query rows of the same key
        const double ov = __shfl_xor(sum_v[kt], 32, 64), ok = __shfl_xor(sum_k[kt], 32, 64);
        const int64_t key = k0 + 32 * kt + n;
        if (kh == 0 && key < N) {
            ans_v[(int64_t)bg * N + key] = (float)(sum_v[kt] + ov);
            ans_k[(int64_t)bg * N + key] = (float)(sum_k[kt] + ok);
        }
    }
}

// -------------------------------------------------------------------------------------------------
// Few query rows (an observation window): steps = heads of the group x query tiles <= kWinSteps.  Both phases then keep the
// query tiles in LDS and stream the keys once: a wave takes tiles of 32 keys, the next tile's rows on their way into registers while
// this one meets every step, without a barrier in the loop.
// Bound: neither the keys nor the arithmetic alone.  131072 keys x 8 heads, four steps, kernel trace and counters: phase 1 53 us,
// phase 2 59, of which reading the keys once (268 MB) takes 46 at the rate of a large copy and the steps 32 (550 clocks of a SIMD
// each); VALU 57 and 63 % of the time, MFMA 36 and 35 %, waves wait for memory or a counter 36 and 33 % of theirs: a wave asks for
// its next tile at once and meets four steps before it needs it, and loads and steps of the three waves of a SIMD overlap in part.
// -------------------------------------------------------------------------------------------------
constexpr int kWinSteps = 4, kWinWaves = 4, kWinThreads = kWinWaves * 64, kWinPerCu = 3;
constexpr int kWinPairs = 192;                                  // (sequence, KV head) pairs from which a wave has at least two tiles

// query tiles of the (sequence, KV head) into LDS: step = (head of the group, query tile)
template <int STEPS>
__device__ __forceinline__ void stage_window(const half_t* __restrict__ q, int64_t head0, int64_t Nq, int q_tiles, uint32_t to, int wave, int lane)
{
    constexpr int kParts = 8 / kWinWaves;                       // pieces of 1 KB of a tile per wave
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const int hh = s / q_tiles, qt = s - hh * q_tiles;
        const int64_t left = Nq - 32 * qt;
#pragma unroll
        for (int i = 0; i < kParts; ++i)
            load_to_lds16(q + ((head0 + hh) * Nq + 32 * qt) * kD, stage_off(wave * kParts + i, lane, left < 32 ? (int)left - 1 : 31),
                          to + s * kTileBytes + (wave * kParts + i) * 1024);
    }
}

// the keys of a tile as an MFMA operand; keys past N repeat the last one
__device__ __forceinline__ void load_keys(half8_t (&t)[8], const half_t* __restrict__ kb, int64_t key0, int64_t N, int n, int kh)
{
    const int64_t key = key0 + n;
    const half_t* kp = kb + (key < N ? key : N - 1) * kD + 8 * kh;
#pragma unroll
    for (int s = 0; s < 8; ++s) t[s] = *(const half8_t*)(kp + 16 * s);
}

// phase 1: keys on the row axis, queries on the column axis, so that a lane owns a query.  part as above, KS = S.
template <int STEPS>
__global__ __launch_bounds__(kWinThreads, kWinPerCu) void ans_window_stats(
    const half_t* __restrict__ q, const half_t* __restrict__ k, int64_t N, int64_t Nq, float c1, float* __restrict__ part,
    int Hq, int Hkv, int G, int S, int64_t tiles_per_wg)
{
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[STEPS * kTileBytes];
    lds_byte* lds = (lds_byte*)s_mem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, kh = lane >> 5;
    const int bg = blockIdx.x / S, sp = blockIdx.x % S, b = bg / Hkv, g = bg % Hkv;
    const int q_tiles = STEPS / G;
    const int64_t n_tiles = (N + 31) / 32, tile0 = sp * tiles_per_wg;
    const int64_t tile1 = tile0 + tiles_per_wg < n_tiles ? tile0 + tiles_per_wg : n_tiles;
    const int64_t head0 = (int64_t)b * Hq + (int64_t)g * G;
    const half_t* kb = k + (int64_t)bg * N * kD;
    stage_window<STEPS>(q, head0, Nq, q_tiles, (uint32_t)(uintptr_t)lds, wave, lane);
    half8_t tk[2][8];
    int64_t tile = tile0 + wave;
    load_keys(tk[0], kb, tile * 32, N, n, kh);
    uint32_t q_at[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) { q_at[s] = tile_at(n, s, kh); pin(q_at[s]); }
    auto q_op = [&](int s, int step) { return *(lds_half8*)(lds + q_at[s] + step * kTileBytes); };
    float m_run[STEPS], l_run[STEPS];
    int64_t qpos[STEPS], q_first[STEPS];                         // positions of this lane's query and of the tile's first
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        m_run[s] = kNegBig;
        l_run[s] = 0.f;
        const int64_t i0 = 32 * (s % q_tiles), i = i0 + n;
        q_first[s] = N - Nq + i0;
        qpos[s] = N - Nq + (i < Nq ? i : Nq - 1);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) pin(tk[0][s]);
    wait_all_loads();
    __syncthreads();
    // scores of one step; the statistics of the step before are updated between the matrix instructions
    float16_t sc[2];
    auto run_tile = [&](half8_t (&cur)[8], half8_t (&nxt)[8]) __attribute__((always_inline)) {
        if (tile + kWinWaves < tile1) load_keys(nxt, kb, (tile + kWinWaves) * 32, N, n, kh);
        const int64_t kt = tile * 32;
#pragma unroll
        for (int s = 0; s <= STEPS; ++s) {                       // products of step s, statistics of step s - 1
            half8_t op[8];
            if (s < STEPS) {
                op[0] = q_op(0, s);
                op[1] = q_op(1, s);
#pragma unroll
                for (int r = 0; r < 16; ++r) sc[s & 1][r] = 0.f;
            }
            const int u = s > 0 ? s - 1 : 0;
            const bool init = m_run[u] > kNegBig;
            const float base = init ? m_run[u] : 0.f;
            float arg[16];
            float mx = kNegBig, sum = 0.f;
            auto body = [&](auto masked) {
                const int lim_q = (int)(qpos[u] - kt);           // visible: offset <= lim_q (the last query sees the last key)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (s < STEPS) {
                        if (i + 2 < 8) op[i + 2] = q_op(i + 2, s);
                        sc[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cur[i], op[i], sc[s & 1], 0, 0, 0);
                    }
                    if (s > 0) {
#pragma unroll
                        for (int e2 = 0; e2 < 2; ++e2) {
                            const int r = 2 * i + e2;
                            float x = fmaf(sc[u & 1][r], c1, -base);
                            if (decltype(masked)::value && 8 * (r >> 2) + 4 * kh + (r & 3) > lim_q) x = kNegBig;
                            arg[r] = x;
                            mx = fmaxf(mx, x);
                            sum += fast_exp2(x);
                        }
                        pin(sum);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (s == 0 || kt + 31 <= q_first[u]) body(std::false_type{});
            else body(std::true_type{});
            if (s > 0) {
                if (init && mx <= 64.f) {
                    l_run[u] += sum;
                } else if (mx > 0.5f * kNegBig) {                // the tile has a visible element: move the reference
                    float sum2 = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum2 += fast_exp2(arg[r] - mx);
                    l_run[u] = (init ? l_run[u] * fast_exp2(-mx) : 0.f) + sum2;
                    m_run[u] = base + mx;
                }
            }
        }
        tile += kWinWaves;
    };
    while (tile < tile1) {
        run_tile(tk[0], tk[1]);
        if (tile >= tile1) break;
        run_tile(tk[1], tk[0]);
    }
    // the half-waves saw complementary keys of the same queries, the waves other tiles
    __syncthreads();                                             // the query tiles are no longer needed
    float2* s_ml = (float2*)s_mem;                               // [wave][step][32]
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const float m_o = __shfl_xor(m_run[s], 32, 64), l_o = __shfl_xor(l_run[s], 32, 64);
        const float m_f = fmaxf(m_run[s], m_o);
        const float l_f = l_run[s] * fast_exp2(m_run[s] - m_f) + l_o * fast_exp2(m_o - m_f);
        if (kh == 0) s_ml[(wave * STEPS + s) * 32 + n] = float2{m_f, l_f};
    }
    __syncthreads();
    if (tid < STEPS * 32) {
        float2 w[kWinWaves];
#pragma unroll
        for (int i = 0; i < kWinWaves; ++i) w[i] = s_ml[i * STEPS * 32 + tid];
        float m = w[0].x;
#pragma unroll
        for (int i = 1; i < kWinWaves; ++i) m = fmaxf(m, w[i].x);
        float l = 0.f;
#pragma unroll
        for (int i = 0; i < kWinWaves; ++i) l += w[i].y * fast_exp2(w[i].x - m);
        const int s = tid >> 5, hh = s / q_tiles;
        const int64_t i = 32 * (s - hh * q_tiles) + (tid & 31);
        if (i < Nq) *(float2*)(part + (((head0 + hh) * Nq + i) * S + sp) * 2) = float2{m, l};
    }
}

// phase 2: queries on the row axis, keys on the column axis, sums as in ans_col_reduce.  The tiles go backwards: the last ones
// that phase 1 read are the ones that the caches still hold.
template <int STEPS>
__global__ __launch_bounds__(kWinThreads, kWinPerCu) void ans_window_cols(
    const half_t* __restrict__ q, const half_t* __restrict__ k, int64_t N, int64_t Nq, float c1, const float* __restrict__ stat,
    float* __restrict__ ans_k, float* __restrict__ ans_v, int Hq, int Hkv, int G, int S, int64_t tiles_per_wg)
{
    constexpr int kStatBytes = kStatTile * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[STEPS * (kTileBytes + kStatBytes)];
    lds_byte* lds = (lds_byte*)s_mem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, kh = lane >> 5;
    const int bg = blockIdx.x / S, sp = blockIdx.x % S, b = bg / Hkv, g = bg % Hkv;
    const int q_tiles = STEPS / G;
    const int64_t n_tiles = (N + 31) / 32, tile0 = sp * tiles_per_wg;
    const int64_t tile1 = tile0 + tiles_per_wg < n_tiles ? tile0 + tiles_per_wg : n_tiles;
    const int64_t head0 = (int64_t)b * Hq + (int64_t)g * G;
    const half_t* kb = k + (int64_t)bg * N * kD;
    stage_window<STEPS>(q, head0, Nq, q_tiles, (uint32_t)(uintptr_t)lds, wave, lane);
    if (wave < STEPS) load_to_lds4(stat + (head0 * q_tiles + wave) * kStatTile, lane * 4, (uint32_t)(uintptr_t)lds + STEPS * kTileBytes + wave * kStatBytes);
    half8_t tk[2][8];
    int64_t tile = tile1 - 1 - wave;
    if (tile < tile0) tile = tile0 - 1;                          // (nothing to do; tile0 - 1 may be -1, which is not loaded)
    load_keys(tk[0], kb, (tile < 0 ? 0 : tile) * 32, N, n, kh);
    uint32_t q_at[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) { q_at[s] = tile_at(n, s, kh); pin(q_at[s]); }
    const uint32_t s_at = STEPS * kTileBytes + 16 * kh;
    auto q_op = [&](int s, int step) { return *(lds_half8*)(lds + q_at[s] + step * kTileBytes); };
    auto stat_op = [&](int qd, int which, int step) { return *(lds_float4*)(lds + s_at + step * kStatBytes + which * 128 + qd * 32); };
#pragma unroll
    for (int s = 0; s < 8; ++s) pin(tk[0][s]);
    wait_all_loads();
    __syncthreads();
    int q_off[STEPS];                                            // first row of the step's query tile
#pragma unroll
    for (int s = 0; s < STEPS; ++s) q_off[s] = 32 * (s % q_tiles);
    float16_t sc[2];
    auto run_tile = [&](half8_t (&cur)[8], half8_t (&nxt)[8]) __attribute__((always_inline)) {
        if (tile - kWinWaves >= tile0) load_keys(nxt, kb, (tile - kWinWaves) * 32, N, n, kh);
        double sum_v = 0.0, sum_k = 0.0;
        const int rel0 = (int)(N - Nq - tile * 32);              // position of the first query minus the tile's first key
#pragma unroll
        for (int s = 0; s <= STEPS; ++s) {                       // products of step s, sums of step s - 1
            half8_t a[8];
            float4_t c4[4], n4[4];
            const int u = s > 0 ? s - 1 : 0;
            if (s < STEPS) {
                a[0] = q_op(0, s);
                a[1] = q_op(1, s);
#pragma unroll
                for (int r = 0; r < 16; ++r) sc[s & 1][r] = 0.f;
            }
            if (s > 0) {
                c4[0] = stat_op(0, 0, u);
                n4[0] = stat_op(0, 1, u);
                const int rel = rel0 + q_off[u];
                if (__builtin_expect(rel < 31, 0)) {             // some query of the tile does not see some key
                    const int lim = n - rel;                     // tile row r sees this lane's key iff r >= lim
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (8 * (r >> 2) + 4 * kh + (r & 3) < lim) sc[u & 1][r] = -INFINITY;
                }
            }
            float pv = 0.f, pk = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {                        // tile rows 8 qd + 4 kh + e live in register 4 qd + e
                if (s < STEPS) {
                    if (i + 2 < 8) a[i + 2] = q_op(i + 2, s);
                    sc[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], cur[i], sc[s & 1], 0, 0, 0);
                }
                if (s > 0) {
                    if ((i & 1) == 1 && i < 7) { c4[(i >> 1) + 1] = stat_op((i >> 1) + 1, 0, u); n4[(i >> 1) + 1] = stat_op((i >> 1) + 1, 1, u); }
#pragma unroll
                    for (int e2 = 0; e2 < 2; ++e2) {
                        const int r = 2 * i + e2;
                        const float c = c4[r >> 2][r & 3], nn = n4[r >> 2][r & 3];
                        const float w = fast_exp2(fmaf(sc[u & 1][r], c1, c));
                        pv += w;
                        pk = fmaf(w, fmaf(-w, nn, nn), pk);      // a (1 - a) ||q||
                    }
                    pin(pv);
                    pin(pk);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (s > 0) {                                         // fp32 per tile, fp64 over tiles
                sum_v += (double)pv;
                sum_k += (double)pk;
            }
        }
        const double ov = __shfl_xor(sum_v, 32, 64), ok = __shfl_xor(sum_k, 32, 64);   // lanes l and l + 32: the same key
        const int64_t key = tile * 32 + n;
        if (kh == 0 && key < N) {
            ans_v[(int64_t)bg * N + key] = (float)(sum_v + ov);
            ans_k[(int64_t)bg * N + key] = (float)(sum_k + ok);
        }
        tile -= kWinWaves;
    };
    while (tile >= tile0) {
        run_tile(tk[0], tk[1]);
        if (tile < tile0) break;
        run_tile(tk[1], tk[0]);
    }
}

constexpr int kColKeys = 128;                                   // keys of the small workgroups of phase 2

// Workgroups that share the steps of a key block.  Unsplit, the first block's workgroup walks every query of every head, 0.27 us a step,
// while most CUs have nothing: 32 heads of 8 KV heads, whole selection, unsplit and as below: 500 tokens 41 and 23 us, 1200 79 and 30,
// 3000 179 and 80, 7000 422 and 288, 16000 1443 and 1351.  A part costs some 8 us besides its steps, so that the longest walk, the
// first key block's, has at least 16 of them per part (of a causal prompt's later blocks the parts have fewer, the last ones' one or
// none; every block has the same number of parts); short walks are split up to 512 blocks (one query head per KV head, 2 x 32 heads, 640 blocks of at most 38 steps: 40 us, in halves
// 48; 320 blocks 33 and 31), longer ones up to 2048, into more than four parts below 128 blocks (3 x 8 heads, 240 blocks:
// quarters 52 us, eighths 58; 80 blocks 35 and 30).
int col_splits(int64_t blocks, int64_t n_steps)
{
    const int most = blocks < 128 ? 8 : 4;
    const int64_t few = n_steps >= 128 ? 2048 : 512;
    int s = 1;
    while (s < most && blocks * s < few && n_steps >= 32 * s) s *= 2;
    return s;
}

struct AsPlan {
    int splits;                                                 // workgroups that share the heads of a key block, phase 2
    int steps;                                                  // 0, or what the window kernels take
    int KS;
    int64_t keys_per_split, n_done;
    size_t off_done, off_part, off_stat, off_ans_k, off_ans_v, total;
};

AsPlan plan(const Geom& g, int64_t N, int64_t Nq, bool room)
{
    AsPlan p;
    const int64_t n_steps = g.G * ((Nq + 31) / 32), n_bg = (int64_t)g.B * g.Hkv;
    p.steps = n_steps <= kWinSteps ? (int)n_steps : 0;
    const int qspan = 32 * (8 / (g.G >= 4 ? 4 : g.G));          // query rows per workgroup of phase 1
    const int64_t qblocks = (Nq + qspan - 1) / qspan;
    const int64_t base_wgs = (int64_t)g.B * g.Hkv * qblocks;
    int64_t ks = base_wgs > 0 ? (1024 + base_wgs - 1) / base_wgs : 1;
    // Ranges of 1024 keys: few query rows leave phase 1 no other parallelism (whole selection, 131072 keys x 8 heads, one query head
    // each, 160 queries: 229 us with ranges of 4096, 222 with these, 213 with 2048; four query heads each, 64 queries 256, 259, 252,
    // 128 queries 427, 430, 430).
    const int64_t max_ks = (N + 1023) / 1024;
    if (ks > max_ks) ks = max_ks;
    if (ks < 1) ks = 1;
    int64_t per = (N + ks - 1) / ks;
    per = (per + 31) / 32 * 32;
    p.keys_per_split = per;
    p.KS = (int)((N + per - 1) / per);
    if (p.steps) {
        // Workgroups of a (sequence, KV head): all CUs full once, at least a tile per wave, and two where the pairs themselves come
        // near a workgroup per CU (query tiles are then loaded less often).  Whole selection, 4 heads x 32 queries, through the general
        // kernels, with one tile and with two: 224 pairs x 300 keys 32.7, 34.3, 31.7 us, 256 x 450 39.9, 40.3, 36.1, 384 x 150 38.5,
        // 40.2, 36.9; 128 x 150 23.7, 22.5, 24.7.  General and these, 8192 keys: 8 pairs 44 and 33, 64 88 and 80, 128 160 and 129, 384
        // 505 and 361, 400 524 and 413 (a workgroup per pair from 385 on), 768 959 and 712, 800 1040 and 863, 2048 2527 and 1894.
        const int64_t n_tiles = (N + 31) / 32, fill = n_bg > 0 ? 256 * kWinPerCu / n_bg : 1, least = kWinWaves * (n_bg < kWinPairs ? 1 : 2);
        const int64_t most = (n_tiles + least - 1) / least;
        const int64_t S = fill < 1 ? 1 : (fill < most ? fill : most);
        const int64_t tiles = (n_tiles + S - 1) / S;
        p.keys_per_split = 32 * tiles;
        p.KS = (int)((n_tiles + tiles - 1) / tiles);
    }
    const int64_t blocks = (N + kColKeys - 1) / kColKeys;
    p.splits = room && !p.steps ? col_splits(blocks * n_bg, n_steps) : 1;
    // phase 1's partials, or phase 2's: the former are done with when phase 2 starts.  The arrival counters lie behind both, since they
    // are cleared while phase 1's are read.
    const size_t rows = (size_t)g.B * g.Hq * Nq, sums = (size_t)p.splits * 2 * n_bg * N * sizeof(double);
    size_t part = align_up(rows * p.KS * 2 * sizeof(float));
    p.n_done = p.splits > 1 ? blocks * n_bg : 0;
    if (p.splits > 1) {
        if (part < align_up(sums)) part = align_up(sums);
        p.off_done = part;
        part += align_up(p.n_done * sizeof(uint32_t));
    } else {
        p.off_done = 0;
    }
    size_t off = 0;
    p.off_part = off; off += p.steps ? 0 : part;
    p.off_stat = off; off += align_up(((size_t)g.B * g.Hq * ((Nq + 31) / 32) + 1) * kStatTile * sizeof(float));
    p.off_ans_k = off; off += align_up((size_t)g.B * g.Hkv * N * sizeof(float));
    p.off_ans_v = off; off += align_up((size_t)g.B * g.Hkv * N * sizeof(float));
    p.total = off;
    if (p.steps) {                                              // the partials lie where phase 2 puts its scores afterwards
        p.off_part = p.off_ans_k;
        if (p.total < p.off_part + part) p.total = p.off_part + part;
    }
    return p;
}

}  // namespace

size_t anchor_score_workspace_bytes(const Geom& g, int64_t N, int64_t Nq, bool room) { return plan(g, N, Nq, room).total; }

// ans_k / ans_v may be NULL: the scores then live in the workspace at the offsets of the plan.
hipError_t launch_anchor_score(const Geom& g, const half_t* q, const half_t* k, int64_t N, int64_t Nq, float scale,
                               const float* row_max, const float* row_sum, float* ans_k, float* ans_v, void* ws, bool room,
                               hipStream_t st)
{
    const AsPlan p = plan(g, N, Nq, room);
    char* w = (char*)ws;
    float* part = (float*)(w + p.off_part);
    float* stat = (float*)(w + p.off_stat);
    if (!ans_k) ans_k = (float*)(w + p.off_ans_k);
    if (!ans_v) ans_v = (float*)(w + p.off_ans_v);
    const float c1 = scale * kLog2e;
    const int64_t n_bg = (int64_t)g.B * g.Hkv;
#define ANTKV_WIN(KERNEL, STEPS, ...)                                                                                      \
    hipLaunchKernelGGL((KERNEL<STEPS>), dim3((unsigned)(p.KS * n_bg)), dim3(kWinThreads), 0, st, q, k, N, Nq, c1, __VA_ARGS__, \
                       g.Hq, g.Hkv, g.G, p.KS, p.keys_per_split / 32)
#define ANTKV_WIN_STEPS(KERNEL, ...)                                                                                       \
    do {                                                                                                                   \
        if (p.steps == 1) ANTKV_WIN(KERNEL, 1, __VA_ARGS__);                                                               \
        else if (p.steps == 2) ANTKV_WIN(KERNEL, 2, __VA_ARGS__);                                                          \
        else if (p.steps == 3) ANTKV_WIN(KERNEL, 3, __VA_ARGS__);                                                          \
        else ANTKV_WIN(KERNEL, 4, __VA_ARGS__);                                                                            \
    } while (0)
    if (!row_max && p.steps) {
        ANTKV_WIN_STEPS(ans_window_stats, part);
    } else if (!row_max) {
        const int qspan = 32 * (8 / (g.G >= 4 ? 4 : g.G));
        dim3 grid((unsigned)p.KS, (unsigned)((Nq + qspan - 1) / qspan), (unsigned)(g.B * g.Hkv));
        hipLaunchKernelGGL(ans_row_stats, grid, dim3(kAsThreads), 0, st, q, k, N, Nq, c1, part, g.Hq, g.Hkv, g.G,
                           p.KS, p.keys_per_split);
    }
    const int64_t q_tiles = (Nq + 31) / 32, n_heads = (int64_t)g.B * g.Hq;
    const int64_t padded = (n_heads * q_tiles + 1) * 32;
    const ColSplit split = {p.splits, (double*)part, (uint32_t*)(w + p.off_part + p.off_done)};
    hipLaunchKernelGGL(ans_finalize_stats, dim3((unsigned)((padded * 16 + 255) / 256)), dim3(256), 0, st, q, part, p.KS,
                       row_max, row_sum, stat, Nq, (int)q_tiles, n_heads, ClearWords{split.done, p.n_done});
    // 64 keys per wave (the query tiles and statistics are read once for two key tiles) while that fills the chip and the
    // walk over the queries is long beside loading the keys (whole selection, 131072 keys x 32 heads: 64 queries 275 us against 259
    // with the smaller ones, 300 988 and 985, 512 1396 and 1432); smaller workgroups otherwise
#define ANTKV_CR(KT, NW, SPLIT)                                                                                           \
    hipLaunchKernelGGL((ans_col_reduce<KT, NW, SPLIT>), dim3((unsigned)((N + 32 * KT * NW - 1) / (32 * KT * NW) * n_bg * (SPLIT ? p.splits : 1))), \
                       dim3(NW * 64), 0, st, q, k, N, Nq, c1, stat, ans_k, ans_v, g.Hq, g.Hkv, g.G, n_bg, (int)q_tiles, split)
    if (p.steps) ANTKV_WIN_STEPS(ans_window_cols, stat, ans_k, ans_v);
    else if (p.splits > 1) ANTKV_CR(1, kColKeys / 32, true);
    else if (Nq > 256 && (N + 511) / 512 * n_bg >= 512) ANTKV_CR(2, 8, false);
    else ANTKV_CR(1, 4, false);
#undef ANTKV_CR
#undef ANTKV_WIN_STEPS
#undef ANTKV_WIN
    return hipGetLastError();
}

}  // namespace antkv
