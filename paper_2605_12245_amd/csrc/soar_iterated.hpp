// The iterated path: Algorithm 1 in full (Sec. 3.3-3.4, Appendix B.3) and the arms of the
// component study: k_iter_init builds the Eq. 1-2 state, k_iter carries out one iteration.
#pragma once
#include "soar_device.hpp"

namespace {

// Sums of up to three per-block binary64 terms over the blocks of a workgroup, as the
// adjacent-pair tree over the flat block index: wave tree, four waves, then a
// binary-counter stack over the workgroup's consecutive tiles.  Call once per tile
// (tile k of the workgroup, all lanes); after the last tile lane 0 holds the sums.
template <int NS>
struct TileTree {
    double (*s_wave)[4];     // [NS][4]
    double (*s_stack)[32];   // [NS][32]
    double wg[NS] = {};
    __device__ __forceinline__ void add_tile(uint32_t k, const double term[NS])
    {
        double v[NS];
#pragma unroll
        for (int n = 0; n < NS; ++n) v[n] = wave_pair_tree(term[n]);
        __syncthreads();                                   // s_wave free again
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int n = 0; n < NS; ++n) s_wave[n][threadIdx.x >> 6] = v[n];
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int n = 0; n < NS; ++n) {
                double x = (s_wave[n][0] + s_wave[n][1]) + (s_wave[n][2] + s_wave[n][3]);
                uint32_t lvl = 0;
                while ((k >> lvl) & 1u) { x = s_stack[n][lvl] + x; ++lvl; }
                s_stack[n][lvl] = x;
                wg[n] = x;
            }
        }
    }
};

// The same three sums for the memory-bound kernels, at a fraction of the cross-lane work: what a block
// contributes -- a = sum w q, b = sum q^2, its stored scale d and its error, four floats -- is staged in LDS
// for up to kStage consecutive tiles; lane t then forms the binary64 terms a d, b d^2, err of the adjacent
// blocks t*T .. t*T+T-1 (exact products, wherever they are formed), folds them in registers, and ONE wave
// tree, the four waves and the binary-counter stack finish the group -- the adjacent-pair tree again
// (k_stats does the same for its two sums).  Per group of T tiles: stage() once per tile by every lane,
// then close() by every lane; after the last group lane 0 holds the sums (N, M, error) in wg[].
template <int LANES = kWG>
struct StagedTree {
    static constexpr int kWaves = LANES / 64;
    float4 *s_blocks;            // [kStage * LANES]: a, b, d, err; zeros for a block that does not exist
    double (*s_wave)[kWaves];    // [3][kWaves]
    double (*s_stack)[32];       // [3][32]
    double wg[3] = {};
    __device__ __forceinline__ void stage(uint32_t kk, float a, float b, float d, float err)
    {
        s_blocks[kk * LANES + threadIdx.x] = make_float4(a, b, d, err);
    }
    static __device__ __forceinline__ void terms(const float4 &x, double v[3])
    {
        v[0] = (double)x.x * (double)x.z;
        v[1] = ((double)x.y * (double)x.z) * (double)x.z;
        v[2] = (double)x.w;
    }
    // group `k` of the workgroup, T tiles staged (T a power of two <= kStage)
    __device__ __forceinline__ void close(uint32_t k, uint32_t T)
    {
        __syncthreads();
        const float4 *x = s_blocks + threadIdx.x * T;
        double v[3];
        terms(x[0], v);
        if (T >= 2) {
            double u[3];
            terms(x[1], u);
#pragma unroll
            for (int n = 0; n < 3; ++n) v[n] = v[n] + u[n];
        }
        if (T == 4) {
            double u[3], z[3];
            terms(x[2], u);
            terms(x[3], z);
#pragma unroll
            for (int n = 0; n < 3; ++n) v[n] = v[n] + (u[n] + z[n]);
        }
#pragma unroll
        for (int n = 0; n < 3; ++n) v[n] = wave_pair_tree(v[n]);
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int n = 0; n < 3; ++n) s_wave[n][threadIdx.x >> 6] = v[n];
        __syncthreads();
        if (threadIdx.x < (kWaves == 4 ? 1u : 64u)) {
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                double y;
                if constexpr (kWaves == 4)
                    y = (s_wave[n][0] + s_wave[n][1]) + (s_wave[n][2] + s_wave[n][3]);
                else
                    y = wave_pair_tree(threadIdx.x < (uint32_t)kWaves ? s_wave[n][threadIdx.x] : 0.0);
                if (threadIdx.x == 0) {
                    uint32_t lvl = 0;
                    while ((k >> lvl) & 1u) { y = s_stack[n][lvl] + y; ++lvl; }
                    s_stack[n][lvl] = y;
                    wg[n] = y;
                }
            }
        }
    }
};
static_assert(kStage == 4, "StagedTree::close folds up to four tiles");

// largest E4M3 code in [0x01, 0x7E] whose value does not exceed y (0x01 if none does)
__device__ __forceinline__ int e4m3_floor_code(float y)
{
    if (!(y > 0.0f)) return (int)kE4M3Min;                  // zero, negative, NaN
    const int normal = (int)(__float_as_uint(y) >> 20) - (120 << 3);
    const int sub = (int)(fminf(y, 1.0f) * 512.0f);
    const int code = (y >= 0x1p-6f) ? normal : sub;
    return min(max(code, (int)kE4M3Min), (int)kE4M3Max);
}

// assign_codes with the reciprocal chosen at compile time; nib carries the previous codes in
// (every byte is overwritten) so that no register has to be cleared first
template <bool FAST>
__device__ __forceinline__ void assign_codes_rcp(const float w[16], float scale, uint32_t nib[2], float q[16])
{
    const float r = FAST ? rcp_midrange(scale) : 1.0f / scale;
    float x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = w[j] * r;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t v = nib[h];
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 0], x[8 * h + 1], 1.0f, 0);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 2], x[8 * h + 3], 1.0f, 1);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 4], x[8 * h + 5], 1.0f, 2);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 6], x[8 * h + 7], 1.0f, 3);
        nib[h] = v;
    }
    fp4x8_values(nib[0], q);
    fp4x8_values(nib[1], q + 8);
}

// The joint search of Sec. 3.3 for one block: factors beta ascending, for each the stored-scale
// candidates in their order (bracket: c0 then c0+1; window: c0, -1, +1, ...), the first pair with
// the smallest binary32 error wins.  Only the error and the winning factor are tracked in the
// loop; the winner's codes are formed once more at the end.
template <bool FAST, int UNROLL>
__device__ __forceinline__ void joint_search(const float w[16], float alpha, float delta_star, const float *s_beta,
                                             int n_beta, bool bracket, int c0, int radius, float &best_err,
                                             int &best_code, uint32_t best_nib[2], float q[16])
{

    uint32_t nib[2] = {0u, 0u};
    float best = __builtin_inff();           // an error is never NaN; "first wins" for an infinite one too
    float best_beta = s_beta[0];
    if (bracket) {
        const int lo = c0;
        const int hi = min(lo + 1, (int)kE4M3Max);           // hi == lo can never win
        const float s_lo = alpha * e4m3_value_of(lo);
        const float s_hi = alpha * e4m3_value_of(hi);
#pragma unroll UNROLL
        for (int kb = 0; kb < n_beta; ++kb) {
            const float bk = s_beta[kb];
            assign_codes_rcp<FAST>(w, alpha * (delta_star * bk), nib, q);
            const float e_lo = block_error(w, q, s_lo);
            const float e_hi = block_error(w, q, s_hi);
            const float m = fminf(fminf(best, e_lo), e_hi);
            best_beta = (m < best) ? bk : best_beta;         // strictly better only: the first factor keeps a tie
            best = m;
        }
        // the winning factor once more: its codes, and which of the two stored scales it won with
        assign_codes_rcp<FAST>(w, alpha * (delta_star * best_beta), best_nib, q);
        const float e_lo = block_error(w, q, s_lo);
        const float e_hi = block_error(w, q, s_hi);
        const bool upper = e_hi < e_lo;                      // the lower code comes first and keeps a tie
        best_code = upper ? hi : lo;
        best_err = upper ? e_hi : e_lo;
    } else {
        best_code = c0;
        for (int kb = 0; kb < n_beta; ++kb) {
            const float bk = s_beta[kb];
            assign_codes_rcp<FAST>(w, alpha * (delta_star * bk), nib, q);
            // a code clamped into [0x01, 0x7E] repeats an earlier candidate of the same factor
            // and can then never win
            for (int c = 0; c <= 2 * radius; ++c) {
                const int o = (c + 1) >> 1;
                const int code = (c & 1) ? max(c0 - o, (int)kE4M3Min) : min(c0 + o, (int)kE4M3Max);
                const float e = block_error(w, q, alpha * e4m3_value_of(code));
                if (e < best) { best = e; best_beta = bk; best_code = code; }
            }
        }
        best_err = best;
        assign_codes_rcp<FAST>(w, alpha * (delta_star * best_beta), best_nib, q);
    }
}

// assign_codes_rcp without the decoded values (codes only)
template <bool FAST>
__device__ __forceinline__ void codes_only_rcp(const float w[16], float scale, uint32_t nib[2])
{
    const float r = FAST ? rcp_midrange(scale) : 1.0f / scale;
    float x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = w[j] * r;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t v = nib[h];
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 0], x[8 * h + 1], 1.0f, 0);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 2], x[8 * h + 3], 1.0f, 1);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 4], x[8 * h + 5], 1.0f, 2);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[8 * h + 6], x[8 * h + 7], 1.0f, 3);
        nib[h] = v;
    }
}

// The factors of a stretch of the grid at which a lane's codes change, one bit each, in registers (a list in LDS would
// take 26 KB of a workgroup for the paper's grid).  Filled word by word, the factor number uniform over the wave; taken
// out by each lane at its own pace.
constexpr int kStretch = 128;
struct ChangeSet {
    uint32_t now = 0u, later[3] = {0u, 0u, 0u};
    int at = -kStretch;              // number of the first factor of `now` within the stretch
    __device__ __forceinline__ void push(uint32_t word)
    {
        now = later[0];
        later[0] = later[1];
        later[1] = later[2];
        later[2] = word;
        at += 32;
    }
    // after the last push, and whenever `now` has been used up: `now` is zero in an empty set only
    __device__ __forceinline__ void settle()
    {
        while (now == 0u && (later[0] | later[1] | later[2]) != 0u) push(0u);
    }
    __device__ __forceinline__ bool empty() const { return now == 0u; }
    // the smallest of a set that is not empty, taken out
    __device__ __forceinline__ int pop()
    {
        const int k = at + __builtin_ctz(now);
        now &= now - 1u;
        if (now == 0u) {
            asm volatile("");        // a few times per stretch: kept out of the straight line
            settle();
        }
        return k;
    }
};

// The same joint search in two passes, for what joint_search_nearest does not take or would do more work for (see
// nearest_search).  Neighbouring factors very often give a block the same 16 codes (a quarter of the paper's 101 factors
// give new ones, on average, on heavy-tailed weights), and a pair whose codes equal those of the factor before it has
// the same errors and can never be strictly better.  Per stretch of the grid: pass 1 forms the codes only and notes the
// factors at which this block's codes change; pass 2 evaluates the errors for those alone (its trip count is the
// largest set in the wave).  The result is that of joint_search, pair for pair.
// 2048 x 4096 bf16, three iterations, paper settings: 0.46 ms, joint_search 0.52, joint_search_nearest 0.06; window of
// radius 4: 0.87, 1.34, 0.13; 300 factors, radius 100: 12.3, 75, 51.
template <bool FAST>
__device__ __forceinline__ void joint_search_changes(const float w[16], float alpha, float delta_star, const float *s_beta, int n_beta,
                                                     bool bracket, int c0, int radius, float &best_err, int &best_code,
                                                     uint32_t best_nib[2], float q[16])
{
    uint32_t nib[2] = {0u, 0u}, even[2] = {0u, 0u}, odd[2] = {0u, 0u};
    float best = __builtin_inff();
    float best_beta = s_beta[0];
    const int lo = c0;
    const int hi = min(lo + 1, (int)kE4M3Max);
    const float s_lo = alpha * e4m3_value_of(lo);
    const float s_hi = alpha * e4m3_value_of(hi);
    best_code = c0;
    for (int base = 0; base < n_beta; base += kStretch) {
        ChangeSet set;
        for (int first = base; first < min(n_beta, base + kStretch); first += 32) {
            uint32_t word = first == 0 ? 1u : 0u;
            // two factors a round: each set of codes is compared with the other one, and none has to be copied
            for (int k = 0; k < min(n_beta - first, 32); k += 2) {
                codes_only_rcp<FAST>(w, alpha * (delta_star * s_beta[first + k]), even);
                word |= ((even[0] ^ odd[0]) | (even[1] ^ odd[1])) != 0u ? 1u << k : 0u;
                if (first + k + 1 == n_beta) break;
                codes_only_rcp<FAST>(w, alpha * (delta_star * s_beta[first + k + 1]), odd);
                word |= ((even[0] ^ odd[0]) | (even[1] ^ odd[1])) != 0u ? 2u << k : 0u;
            }
            set.push(word);
        }
        set.settle();
        while (__builtin_amdgcn_ballot_w64(!set.empty()) != 0ull) {
            if (!set.empty()) {
                const float bk = s_beta[base + set.pop()];
                assign_codes_rcp<FAST>(w, alpha * (delta_star * bk), nib, q);
                if (bracket) {
                    const float e_lo = block_error(w, q, s_lo);
                    const float e_hi = block_error(w, q, s_hi);
                    const float m = fminf(fminf(best, e_lo), e_hi);
                    best_beta = (m < best) ? bk : best_beta;
                    best = m;
                } else {
                    for (int c = 0; c <= 2 * radius; ++c) {
                        const int o = (c + 1) >> 1;
                        const int code = (c & 1) ? max(c0 - o, (int)kE4M3Min) : min(c0 + o, (int)kE4M3Max);
                        const float e = block_error(w, q, alpha * e4m3_value_of(code));
                        if (e < best) { best = e; best_beta = bk; best_code = code; }
                    }
                }
            }
        }
    }
    assign_codes_rcp<FAST>(w, alpha * (delta_star * best_beta), best_nib, q);
    if (bracket) {
        const float e_lo = block_error(w, q, s_lo);
        const float e_hi = block_error(w, q, s_hi);
        const bool upper = e_hi < e_lo;
        best_code = upper ? hi : lo;
        best_err = upper ? e_hi : e_lo;
    } else {
        best_err = best;
    }
}

// four times twice the rounding of a block error of 16 or 32 elements, (n + 2) 2^-24, rounded up by a tenth
constexpr float kFarSideRounding16 = 1.0e-5f, kFarSideRounding32 = 1.8e-5f;

// The same joint search without walking the factor grid.  For ONE stored scale s the exact block error, as a
// function of the factor, falls towards the assignment scale t = s and rises beyond it: the codes of one element
// move through the E2M1 grid in one direction as t grows (t_k = alpha (Delta* beta_k), the reciprocal, the product
// and the rounding are all monotone, in binary32 too), and while t_k <= s every |code| lies at or above the one
// nearest to |w|/s, so each further step up moves away from w; for t_k >= s the mirror image.  The best factor
// for s is therefore the last one below s (A) or the first one above it (B) -- 4 pairs of the paper's 202.
// What binary32 rounding can change is covered by a certificate.  A factor beyond A that gives other codes moves
// at least one code across a rounding threshold m (>= 0.25, codes >= 0.5 apart), and |w| <= m t_A up to the rounding
// of the product, so its exact error exceeds that of A by at least 2 s^2 (0.5)(0.25)(s - t_A)/s = s (s - t_A) / 4; a
// computed error is within 18 units of 2^-24 of the exact one (all terms non-negative).  If that rise exceeds the
// rounding of both sides -- s (|s - t_A| - 2^-21 s) > kFarSideRounding error, the 2^-21 for reciprocal and product --, no factor beyond A can compute to a value as small as A's, and factors with A's codes
// have A's error.  Otherwise (s within about 1e-5 of t_A: one block in a thousand per side, or magnitudes at
// which squares leave the normal range) the walk goes one factor further out and asks again, to the end of the
// grid if need be: the result never depends on the shortcut.
// "First pair wins a tie" (factors ascending, then the candidates in their order): between pairs of different
// codes the smaller factor is the earlier one; pairs of the same codes belong to the same run of factors, and the
// candidate tried first keeps the tie.
// Needs an ascending factor table (checked on the host) and the reciprocal's range (FAST).
// Mostly bound by vector issue (the vector units are busy for 70 % of an iteration's launch): 489 instructions per block and
// iteration with two candidates, where forming the codes of all 101 factors and the errors of those at which a block's codes
// change took 8 500; 941 with three.  One decoder layer (seven tensors, 1.93e8 bf16 weights, 3 iterations): 7.65 -> 0.72 ms a
// call; with three candidates on 4096 x 4096 fp32: 0.96 -> 0.17 ms, 0.135 in one launch.
struct FactorGrid {
    const float *table;          // LDS, n factors, ascending
    int n;
    float lo, index_per_beta;
};

// what one factor gives for the stored scale s: the codes and their error
__device__ __forceinline__ float factor_error(const float w[16], float t, float s, uint32_t nib[2])
{
    float q[16];
    nib[0] = any_word();
    nib[1] = any_word();
    assign_codes_rcp<true>(w, t, nib, q);
    return block_error(w, q, s);
}

// The first factor with the smallest error for one stored scale s.  base_index: factor index per unit of s.
__device__ __forceinline__ float best_factor(const float w[16], float alpha, float delta_star, float base_index,
                                             const FactorGrid &grid, float s, uint32_t nib[2], int &k)
{
    // where s lies in the grid; any error of this estimate is met by the walk
    const float at = __builtin_fmaf(s, base_index, -grid.lo * grid.index_per_beta);
    const int ka = (int)__builtin_amdgcn_fmed3f(at, 0.0f, (float)(grid.n - 2));
    const float ta = alpha * (delta_star * grid.table[ka]), tb = alpha * (delta_star * grid.table[ka + 1]);
    uint32_t nib_b[2];
    float err = factor_error(w, ta, s, nib);
    const float err_b = factor_error(w, tb, s, nib_b);
    // s (|s - t| - 2^-21 s) / kRounding > error: see above; s - t is negative where the estimate was off
    const float per_error = s * (1.0f / kFarSideRounding16), slack = s * (0x1p-21f * per_error);
    const bool far_a = __builtin_fmaf(s - ta, per_error, -slack) > err;
    const bool far_b = __builtin_fmaf(tb - s, per_error, -slack) > err_b;
    k = ka;
    const bool take_b = err_b < err;             // the smaller factor keeps a tie
    err = take_b ? err_b : err;
    nib[0] = take_b ? nib_b[0] : nib[0];
    nib[1] = take_b ? nib_b[1] : nib[1];
    k = take_b ? ka + 1 : ka;
    if (__builtin_amdgcn_ballot_w64(!(far_a && far_b)) != 0ull) {
        int lo = ka, hi = ka + 1;
        bool down = !far_a && lo > 0, up = !far_b && hi < grid.n - 1;
        while (__builtin_amdgcn_ballot_w64(down || up) != 0ull) {
            if (down || up) {
                const int kk = down ? --lo : ++hi;
                const float t = alpha * (delta_star * grid.table[kk]);
                const float e = factor_error(w, t, s, nib_b);
                const bool far = __builtin_fmaf(down ? s - t : t - s, per_error, -slack) > e;
                if (e < err || (e == err && kk < k)) { err = e; k = kk; nib[0] = nib_b[0]; nib[1] = nib_b[1]; }
                if (down) down = !far && lo > 0;
                else up = !far && hi < grid.n - 1;
            }
        }
    }
    return err;
}

__device__ __forceinline__ void joint_search_nearest(const float w[16], float alpha, float delta_star, const FactorGrid &grid,
                                                     bool bracket, int c0, int radius, float &best_err, int &best_code,
                                                     uint32_t best_nib[2])
{
    const float base_index = __builtin_amdgcn_rcpf(alpha * delta_star) * grid.index_per_beta;
    int best_k;
    best_code = c0;
    best_err = best_factor(w, alpha, delta_star, base_index, grid, alpha * e4m3_value_of(c0), best_nib, best_k);
    auto next = [&](int code) {
        uint32_t nib[2];
        int k;
        const float err = best_factor(w, alpha, delta_star, base_index, grid, alpha * e4m3_value_of(code), nib, k);
        bool win = err < best_err;
        if (__builtin_amdgcn_ballot_w64(err == best_err) != 0ull) {
            asm volatile("");                    // rare: kept out of the straight line
            win = win || (err == best_err && k < best_k && (nib[0] != best_nib[0] || nib[1] != best_nib[1]));
        }
        best_err = win ? err : best_err;
        best_code = win ? code : best_code;
        best_k = win ? k : best_k;
        best_nib[0] = win ? nib[0] : best_nib[0];
        best_nib[1] = win ? nib[1] : best_nib[1];
    };
    // a code clamped into [0x01, 0x7E] repeats an earlier candidate
    if (bracket) {
        next(min(c0 + 1, (int)kE4M3Max));
    } else {
#pragma unroll 1
        for (int c = 1; c <= 2 * radius; ++c) {
            const int o = (c + 1) >> 1;
            next((c & 1) ? max(c0 - o, (int)kE4M3Min) : min(c0 + o, (int)kE4M3Max));
        }
    }
}

// the Eq. 1-2 state of a block: a, b, the scale's value, the error and the ratio for Eq. 6 (keep_scale: -Delta0, the
// search centre of the arm that leaves the closed-form stage out)
__device__ __forceinline__ void init_block(const float w[16], const GlobalScale &g, bool keep_scale, float &a, float &b, float &delta0,
                                           float &err, float &rho)
{
    float q[16];
    uint32_t nib[2], c0;
    block_init(w, g, c0, delta0, nib, q);
    block_sums(w, q, a, b);
    err = block_error(w, q, g.alpha0 * delta0);
    rho = keep_scale ? -delta0 : block_ratio(a, b, delta0, g.fast);
}

// What the workgroups of one tensor share in k_iter_rest: cleared by k_iter_init, at the end of the partial sums, where a tensor
// of fewer partials leaves room.  (at most kRestShares shares: deal_shares)
constexpr uint32_t kRestShares = 2048, kRestStopped = 0xFFFFFFFFu;
constexpr uint32_t kRestLooks = 64;       // looks for the next iteration, about 1 us each, between two for shares that nobody has taken
struct RestWords {
    uint64_t next[16][16];                // the iteration to carry out next (0: the launch's first) or kRestStopped; its global scale in the upper
                                          // half.  Copies: a workgroup reads the one of its number
    uint32_t taken[kRestShares];          // of a share: one more than the last iteration for which it has been taken
};
constexpr int kRestPartials = kMaxPartials - (int)(sizeof(RestWords) / sizeof(double));
__host__ __device__ inline bool has_rest_words(uint32_t n_chunks) { return n_chunks <= (uint32_t)kRestPartials; }
__device__ __forceinline__ RestWords &rest_words(const Task &t)
{
    return *reinterpret_cast<RestWords *>(t.part + 2 * kMaxPartials + kRestPartials);
}

// The Eq. 1-2 state of Algorithm 1 (Delta^q = Delta^d = Delta0) for the iterated
// path: per block the ratio a/b for Eq. 6 and the error of that state; per tensor
// the sums of Eq. 5 (-> the global scale of iteration 0) and the error before any
// iteration.
template <int DT>
__global__ __launch_bounds__(kWG) void k_iter_init(const Batch batch)
{
    __shared__ float4 s_blocks[kStage * kWG];
    __shared__ double s_wave[3][4];
    __shared__ double s_stack[3][32];
    __shared__ uint32_t s_last;
    double *s_tree = reinterpret_cast<double *>(s_blocks);      // trees_of_partials, after the last group
    static_assert(sizeof(float4) * kStage >= sizeof(double), "s_tree fits s_blocks");

    uint32_t lwg;
    const Task t = batch.t[find_task(batch, lwg)];
    const uint32_t tid = threadIdx.x;
    const uint32_t amax_bits = t.ctrl->amax_bits;
    const bool degenerate = amax_bits == 0u || amax_bits >= 0x7F800000u;
    const GlobalScale gs(amax_bits);
    const float alpha0 = gs.alpha0;

    StagedTree<> tree{s_blocks, s_wave, s_stack};
    const uint32_t T = t.tiles_per_wg < (uint32_t)kStage ? t.tiles_per_wg : (uint32_t)kStage;   // power of two
    for (uint32_t chunk = lwg; chunk < t.n_chunks; chunk += t.n_wg) {
        const uint32_t tile0 = chunk * t.tiles_per_wg;
        for (uint32_t kg = 0; kg < t.tiles_per_wg; kg += T) {
            for (uint32_t kk = 0; kk < T; ++kk) {
                const uint32_t i = (tile0 + kg + kk) * kWG + tid;
                float a = 0.0f, b = 0.0f, delta0 = 0.0f, err = 0.0f;
                if (i < t.nblk) {
                    float rho = 0.0f;
                    if (!degenerate) {
                        float w[16];
                        load_block<DT>(t.w, block_offset(t, i), w);
                        init_block(w, gs, batch.arm == SOAR_METHOD_DSS_ONLY, a, b, delta0, err, rho);
                    }
                    t.rho[i] = rho;
                }
                tree.stage(kk, a, b, delta0, err);
            }
            tree.close(kg / T, T);
        }
        if (tid == 0) {
            publish(t.part + chunk, tree.wg[0]);
            publish(t.part + kMaxPartials + chunk, tree.wg[1]);
            publish(t.part + 2 * kMaxPartials + chunk, tree.wg[2]);
        }
    }
    uint32_t *counters = t.counters + 1 * kSlots * kSlotStride;
    if (tid == 0) s_last = arrive_is_last(counters, &t.ctrl->top[1], t.n_wg, lwg) ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    if (has_rest_words(t.n_chunks))
        for (uint32_t k = tid; k < sizeof(RestWords) / 4; k += kWG) reinterpret_cast<uint32_t *>(&rest_words(t))[k] = 0u;
    double NME[3];
    trees_of_partials<3>(t.part, t.n_chunks, s_tree, &s_stack[0][0], NME);
    const double N = NME[0], M = NME[1], E = NME[2];
    if (tid == 0) {
        t.ctrl->alpha0 = alpha0;
        // the global scale of iteration 0: Eq. 5, or unchanged when the closed-form stage is left out
        t.ctrl->alpha1 = (M > 0.0 && batch.arm != SOAR_METHOD_DSS_ONLY) ? (float)(N / M) : alpha0;
        t.ctrl->N = N;
        t.ctrl->M = M;
        t.ctrl->prev_sse = E;
        t.ctrl->stopped = 0u;
        if (!degenerate && t.trace) t.trace[0] = E;
    }
    reset_counters(counters, &t.ctrl->top[1]);
}

// What an iteration leaves of one block: codes and stored scale, their error, their sums a and b with the scale's
// value d (the Eq. 5 terms of the next iteration), and the ratio a/b (or -d) for the next Eq. 6.
struct BlockState {
    uint32_t nib[2], code;
    float a, b, d, err, rho;
};

// Scales and weights so far from the ends of the binary32 range that neither the reciprocals nor the squares of the
// nearest-factor search leave it (factors within 2^-20 .. 2^20: the host): alpha Delta* is about the block's ratio, stored
// scales are alpha times [2^-9, 448].
__device__ __forceinline__ bool scales_in_range(float alpha, uint32_t amax_bits)
{
    return alpha > 0x1p-35f && alpha < 0x1p50f && f_of(amax_bits) < 0x1p60f;
}

constexpr int kChangesMinBeta = 4;       // fewer factors: evaluating every pair is no more work than forming the codes first

// every ratio of the wave is near one, or stands for a stored scale (negative)
__device__ __forceinline__ bool all_near_one(float rho)
{
    return __builtin_amdgcn_ballot_w64(rho >= 0.0f && !near_one(rho)) == 0ull;
}

// what the joint search of one tensor needs beside the block
struct JointSearch {
    FactorGrid grid;
    float alpha, inv_alpha;
    int radius;
    bool bracket, dss_only;      // dss_only: rho always carries -Delta^d, the search centre
    bool in_range;               // scales_in_range; everything else takes joint_search_changes
    bool every_pair;             // joint_search: SOAR_SEARCH_FULL, grids of fewer than kChangesMinBeta factors
    __device__ __forceinline__ void set_alpha(float alpha_, uint32_t amax_bits)
    {
        alpha = alpha_;
        inv_alpha = 1.0f / alpha_;
        in_range = scales_in_range(alpha_, amax_bits);
    }
};

template <bool NEAREST>
__device__ __forceinline__ void iterate_block(const float w[16], float rho, const JointSearch &js, BlockState &x)
{
    float q[16];
    int code;
    if (NEAREST && __builtin_expect(js.in_range && all_near_one(rho), 1)) {
        const float delta_star = (rho < 0.0f) ? -rho : div_midrange(rho, js.alpha, js.inv_alpha);
        const int c0 = js.bracket ? e4m3_floor_code(delta_star) : (int)e4m3_project(delta_star);
        joint_search_nearest(w, js.alpha, delta_star, js.grid, js.bracket, c0, js.radius, x.err, code, x.nib);
        code_sums(w, x.nib, x.a, x.b);
        x.d = e4m3_value_of(code);
        const float ratio = div_midrange(x.a, x.b, rcp_midrange(x.b));
        x.rho = (x.b == 0.0f || js.dss_only) ? -x.d : ratio;
    } else {
        const float delta_star = (rho < 0.0f) ? -rho : rho / js.alpha;
        const int c0 = js.bracket ? e4m3_floor_code(delta_star) : (int)e4m3_project(delta_star);
        // the reciprocal shortcut holds while the biased exponent of the scale stays in [1, 252];
        // the scales of a block lie between those of the first and the last factor (to within
        // rounding of the grid), which are asked to keep one binade of distance from both ends
        const float s_first = js.alpha * (delta_star * js.grid.table[0]);
        const float s_final = js.alpha * (delta_star * js.grid.table[js.grid.n - 1]);
        const bool mid = ((__float_as_uint(s_first) >> 23) - 2u) < 250u && ((__float_as_uint(s_final) >> 23) - 2u) < 250u;
        const bool fast = __builtin_amdgcn_ballot_w64(!mid) == 0ull;
        if (NEAREST || !js.every_pair) {
            if (fast)
                joint_search_changes<true>(w, js.alpha, delta_star, js.grid.table, js.grid.n, js.bracket, c0, js.radius, x.err, code, x.nib, q);
            else
                joint_search_changes<false>(w, js.alpha, delta_star, js.grid.table, js.grid.n, js.bracket, c0, js.radius, x.err, code, x.nib, q);
        } else if (fast) {
            joint_search<true, 4>(w, js.alpha, delta_star, js.grid.table, js.grid.n, js.bracket, c0, js.radius, x.err, code, x.nib, q);
        } else {
            joint_search<false, 4>(w, js.alpha, delta_star, js.grid.table, js.grid.n, js.bracket, c0, js.radius, x.err, code, x.nib, q);
        }
        block_sums(w, q, x.a, x.b);
        x.d = e4m3_value_of(code);
        x.rho = (x.b == 0.0f || js.dss_only) ? -x.d : x.a / x.b;
    }
    x.code = (uint32_t)code;
}

// the same for the closed-form arm: the projected scale assigns the codes and is stored (fast: alpha and the block's
// ratio are near one, see scales_in_range; stored scales are alpha times [2^-9, 448])
__device__ __forceinline__ void closed_form_block(const float w[16], float rho, float alpha, float inv_alpha, bool fast, BlockState &x)
{
    float q[16];
    const float delta_star = (rho < 0.0f) ? -rho : quotient(rho, alpha, inv_alpha, fast);          // Eq. 6
    x.code = e4m3_project(delta_star);
    x.d = e4m3_value_of((int)x.code);
    const float sd = alpha * x.d;
    assign_codes(w, sd, fast, x.nib, q);
    block_sums(w, q, x.a, x.b);
    x.err = block_error(w, q, sd);
    x.rho = block_ratio(x.a, x.b, x.d, fast);
}

// a block of an all-zero tensor: smallest scale, zero codes carrying the sign
__device__ __forceinline__ void zero_block(const float w[16], BlockState &x)
{
    x.nib[0] = fp4x8(w);
    x.nib[1] = fp4x8(w + 8);
    x.code = kE4M3Min;
    x.a = x.b = x.d = x.err = x.rho = 0.0f;
}

__device__ __forceinline__ void store_block(const Task &t, uint32_t i, const BlockState &x)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 packed = {x.nib[0], x.nib[1]};
    __builtin_nontemporal_store(packed, reinterpret_cast<u32x2 *>(t.codes) + i);
    __builtin_nontemporal_store((uint8_t)x.code, t.scales + i);
}

// One store of a tensor-wide result.  AGENT: performed at the memory side, where the launch itself goes on to use it (k_iter_rest).
template <bool AGENT, typename T>
__device__ __forceinline__ void put(T *p, T v)
{
    if constexpr (AGENT) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// What the last workgroup of a tensor does after iteration `it` (one lane): the outputs that describe the
// tensor, the early-stop decision and the global scale the next iteration starts from (Eq. 5).  Returned: those two as RestWords::next has
// them, which is the only place for them in k_iter_rest (its workgroups read the control words as the launches before left them).
template <bool AGENT = false>
__device__ __forceinline__ uint64_t finish_iteration(const Batch &batch, const Task &t, int it, double N, double M, double cur, float alpha,
                                                 bool degenerate, bool allzero, bool dss_only)
{
    if (degenerate) {
        *t.gscale = allzero ? 1.0f : __builtin_nanf("");
        if (t.sse) *t.sse = allzero ? 0.0 : __builtin_nan("");
        if (t.status) *t.status = allzero ? SOAR_STATUS_ALLZERO : SOAR_STATUS_NONFINITE;
        if (t.iters_run) *t.iters_run = 0;
    } else {
        const double prev = AGENT ? __hip_atomic_load(&t.ctrl->prev_sse, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : t.ctrl->prev_sse;
        put<AGENT>(t.gscale, alpha);
        if (t.sse) put<AGENT>(t.sse, cur);
        if (t.status) put<AGENT>(t.status, (int32_t)0);
        if (t.iters_run) put<AGENT>(t.iters_run, (int32_t)(it + 1));
        if (t.trace) put<AGENT>(t.trace + it + 1, cur);
        const bool stop = batch.early_stop_rel > 0.0f && (prev - cur) < (double)batch.early_stop_rel * prev;
        const float next = (M > 0.0 && !dss_only) ? (float)(N / M) : alpha;                // Eq. 5 for the next iteration
        put<AGENT>(&t.ctrl->prev_sse, cur);
        if constexpr (!AGENT) {
            t.ctrl->stopped = stop ? 1u : 0u;
            t.ctrl->alpha1 = next;
            t.ctrl->N = N;
            t.ctrl->M = M;
        }
        return (uint64_t)__float_as_uint(next) << 32 | (stop ? kRestStopped : (uint32_t)(it + 1));
    }
    return kRestStopped;
}

// One iteration of Algorithm 1.  On entry ctrl->alpha1 holds the Eq. 5 global
// scale for the current codes and stored scales and rho[i] the block ratio a/b
// (Eq. 6 is rho / alpha).  Per block: the joint search of Sec. 3.3 over
// (factor beta ascending) x (stored-scale candidates in their order), keeping
// the first pair with the smallest binary32 error; the block's codes, stored
// scale, and -- because the codes of the winning pair ARE the codes the next
// iteration starts from -- the next a/b and Eq. 5 terms.  Per tensor: the error
// after this iteration (exact adjacent-pair tree, so that the early-stop test
// is reproducible), the stop flag and the next global scale.
// A tensor whose stop flag is set is skipped by every later launch.
// Five waves per SIMD: six spill (737 against 740 us on the decoder layer, 175 against 169 on the fp32 matrix), eight
// spill a tenth of the registers (929, 199).
// NEAREST: the pairs that can win are found without walking the grid (joint_search_nearest, see nearest_search);
// otherwise the codes of every factor are formed and errors where they change (joint_search_changes), or every pair is
// evaluated (joint_search).
// bf16: a lane's next block is on its way into LDS while it searches this one, and the results of a block are stored when the
// next one has been taken out: a wait for loads also waits for the stores before them, and both are a whole search old by then. The
// ratio is read beside the weights, not after them.  One decoder layer 722 -> 703 us, 12288 x 4096 243 -> 237.  fp32 has no
// LDS left for five workgroups with four tiles staged, and with two it is slower (929 -> 944; four workgroups 941): there the nearest-factor search
// reads the ratio first (929 -> 924).  The other searches take longer for a schedule in fewer registers that the compiler finds where the ratio
// or the results are variables of the whole loop: every pair of 4096 x 4096 fp32, three iterations, 990 us, as below 959.  On bf16 the look-ahead
// costs them a wave of five per SIMD and gains all the same (985 -> 949).
template <int DT, bool NEAREST>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(NEAREST ? 5 : 4, 8))) void k_iter(const Batch batch)
{
    __shared__ float4 s_blocks[kStage * kWG];
    __shared__ double s_wave[3][4];
    __shared__ double s_stack[3][32];
    __shared__ uint32_t s_last;
    double *s_tree = reinterpret_cast<double *>(s_blocks);      // trees_of_partials, after the last group
    constexpr bool kAhead = DT == SOAR_BF16;
    __shared__ u32x4 s_next[kAhead ? kWG * BlockStream::kP : 1];
    extern __shared__ __align__(16) unsigned char s_dyn[];      // the factor table, n_beta floats
    float *s_beta = reinterpret_cast<float *>(s_dyn);

    uint32_t lwg;
    const Task t = batch.t[find_task(batch, lwg)];
    const uint32_t tid = threadIdx.x;
    const uint32_t amax_bits = t.ctrl->amax_bits;
    const bool allzero = amax_bits == 0u;
    const bool degenerate = allzero || amax_bits >= 0x7F800000u;
    if (degenerate ? batch.iter_t != 0 : t.ctrl->stopped != 0u) return;     // uniform over the tensor's workgroups

    const int n_beta = batch.n_beta;
    for (int k = (int)tid; k < n_beta; k += kWG) s_beta[k] = beta_factor(k, n_beta, batch.beta_lo, batch.beta_hi);
    __syncthreads();

    const float alpha = t.ctrl->alpha1;
    const bool dss_only = batch.arm == SOAR_METHOD_DSS_ONLY;
    JointSearch js{{s_beta, n_beta, batch.beta_lo, batch.index_per_beta}, 0.0f, 0.0f, batch.radius,
                   batch.dd_mode == SOAR_DD_BRACKET, dss_only, false, batch.full_search != 0 || n_beta < kChangesMinBeta};
    js.set_alpha(alpha, amax_bits);

    StagedTree<> tree{s_blocks, s_wave, s_stack};
    const uint32_t T = t.tiles_per_wg < (uint32_t)kStage ? t.tiles_per_wg : (uint32_t)kStage;   // power of two
    const uint32_t blocks = amax_bits < 0x7F800000u ? t.nblk : 0u;
    const BlockStream stream{s_next + (kAhead ? (tid >> 6) * (64 * BlockStream::kP) : 0u)};
    float next_rho = 0.0f;
    auto fetch = [&](uint32_t tile) {
        const uint32_t i = tile * kWG + tid;
        if (i < blocks) {
            stream.fetch(t.w, block_offset(t, i));
            next_rho = t.rho[i];
        }
    };
    BlockState x;
    uint32_t done = blocks;              // the block whose results x holds, not yet stored
    auto store = [&]() {
        if (done < blocks) {
            store_block(t, done, x);
            t.rho[done] = x.rho;
        }
    };
    if constexpr (kAhead) fetch(lwg * t.tiles_per_wg);
    for (uint32_t chunk = lwg; chunk < t.n_chunks; chunk += t.n_wg) {
        const uint32_t tile0 = chunk * t.tiles_per_wg;
        for (uint32_t kg = 0; kg < t.tiles_per_wg; kg += T) {
            for (uint32_t kk = 0; kk < T; ++kk) {
                const uint32_t i = (tile0 + kg + kk) * kWG + tid;
                if constexpr (kAhead) {
                    float w[16];
                    stream.take(w);
                    const float rho = next_rho;
                    store();
                    const uint32_t at = kg + kk + 1u;
                    const uint32_t next_chunk = at < t.tiles_per_wg ? chunk : chunk + t.n_wg;
                    if (next_chunk < t.n_chunks) fetch(next_chunk * t.tiles_per_wg + (at < t.tiles_per_wg ? at : 0u));
                    x.a = x.b = x.d = x.err = 0.0f;
                    done = i;
                    if (i < blocks) {
                        if (allzero) zero_block(w, x);
                        else iterate_block<NEAREST>(w, rho, js, x);
                    }
                    tree.stage(kk, x.a, x.b, x.d, x.err);
                } else {
                    BlockState y;
                    y.a = y.b = y.d = y.err = 0.0f;
                    if (i < t.nblk && amax_bits < 0x7F800000u) {
                        float w[16], rho = 0.0f;
                        if constexpr (NEAREST) rho = t.rho[i];
                        load_block<DT>(t.w, block_offset(t, i), w);
                        if (allzero) {
                            zero_block(w, y);
                        } else {
                            if constexpr (!NEAREST) rho = t.rho[i];
                            iterate_block<NEAREST>(w, rho, js, y);
                            t.rho[i] = y.rho;
                        }
                        store_block(t, i, y);
                    }
                    tree.stage(kk, y.a, y.b, y.d, y.err);
                }
            }
            tree.close(kg / T, T);
        }
        if (tid == 0) {
            publish(t.part + chunk, tree.wg[0]);
            publish(t.part + kMaxPartials + chunk, tree.wg[1]);
            publish(t.part + 2 * kMaxPartials + chunk, tree.wg[2]);
        }
    }
    if constexpr (kAhead) store();
    uint32_t *counters = t.counters + 2 * kSlots * kSlotStride;
    if (tid == 0) s_last = arrive_is_last(counters, &t.ctrl->top[2], t.n_wg, lwg) ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    double NME[3];
    trees_of_partials<3>(t.part, t.n_chunks, s_tree, &s_stack[0][0], NME);
    const double N = NME[0], M = NME[1], cur = NME[2];
    if (tid == 0) finish_iteration(batch, t, batch.iter_t, N, M, cur, alpha, degenerate, allzero, dss_only);
    reset_counters(counters, &t.ctrl->top[2]);
}

// One iteration of the closed-form arm of the component study (Sec. 3.2 alone): no search.  Per block the
// projected scale E4M3(Delta*) assigns the codes AND is stored; the codes' a/b and Eq. 5 terms are formed
// for the next iteration as in k_iter, and the tensor is finished by finish_iteration.  The kernel is bound
// by memory (weights and ratio read, ratio, codes and scale written), so it is built like k_stats: several
// consecutive tiles per workgroup, the three sums through the staged tree, streaming stores for the outputs
// (the weights and the ratio are read again by the next iteration and stay in the last-level cache).
// (held to 64 registers: eight waves per SIMD hide the loads of this memory-bound kernel)
template <int DT>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(8))) void k_cjso(const Batch batch)
{
    __shared__ float4 s_blocks[kStage * kWG];
    __shared__ double s_wave[3][4];
    __shared__ double s_stack[3][32];
    __shared__ uint32_t s_last;
    double *s_tree = reinterpret_cast<double *>(s_blocks);      // trees_of_partials, after the last group

    uint32_t lwg;
    const Task t = batch.t[find_task(batch, lwg)];
    const uint32_t tid = threadIdx.x;
    const uint32_t amax_bits = t.ctrl->amax_bits;
    const bool allzero = amax_bits == 0u;
    const bool degenerate = allzero || amax_bits >= 0x7F800000u;
    if (degenerate ? batch.iter_t != 0 : t.ctrl->stopped != 0u) return;     // uniform over the tensor's workgroups
    const float alpha = t.ctrl->alpha1, inv_alpha = 1.0f / alpha;
    const bool fast = scales_in_range(alpha, amax_bits);

    StagedTree<> tree{s_blocks, s_wave, s_stack};
    const uint32_t T = t.tiles_per_wg < (uint32_t)kStage ? t.tiles_per_wg : (uint32_t)kStage;   // power of two
    for (uint32_t chunk = lwg; chunk < t.n_chunks; chunk += t.n_wg) {
        const uint32_t tile0 = chunk * t.tiles_per_wg;
        for (uint32_t kg = 0; kg < t.tiles_per_wg; kg += T) {
            for (uint32_t kk = 0; kk < T; ++kk) {
                const uint32_t i = (tile0 + kg + kk) * kWG + tid;
                BlockState x;
                x.a = x.b = x.d = x.err = 0.0f;
                if (i < t.nblk && amax_bits < 0x7F800000u) {
                    float w[16];
                    load_block<DT>(t.w, block_offset(t, i), w);
                    if (allzero) {
                        zero_block(w, x);
                    } else {
                        const float rho = t.rho[i];
                        closed_form_block(w, rho, alpha, inv_alpha, fast && all_near_one(rho), x);
                        t.rho[i] = x.rho;
                    }
                    store_block(t, i, x);
                }
                tree.stage(kk, x.a, x.b, x.d, x.err);
            }
            tree.close(kg / T, T);
        }
        if (tid == 0) {
            publish(t.part + chunk, tree.wg[0]);
            publish(t.part + kMaxPartials + chunk, tree.wg[1]);
            publish(t.part + 2 * kMaxPartials + chunk, tree.wg[2]);
        }
    }
    uint32_t *counters = t.counters + 2 * kSlots * kSlotStride;
    if (tid == 0) s_last = arrive_is_last(counters, &t.ctrl->top[2], t.n_wg, lwg) ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    double NME[3];
    trees_of_partials<3>(t.part, t.n_chunks, s_tree, &s_stack[0][0], NME);
    const double N = NME[0], M = NME[1], cur = NME[2];
    if (tid == 0) finish_iteration(batch, t, batch.iter_t, N, M, cur, alpha, degenerate, allzero, false);
    reset_counters(counters, &t.ctrl->top[2]);
}

// The iterations from batch.iter_t on in one launch: most tensors have stopped by then, and a launch that finds its tensors stopped
// takes 2.4 us on the GPU and 4 to 5 on the host.  Nothing here depends on which workgroups are on the GPU: an iteration has a share
// for every workgroup (what a workgroup of k_iter does); each takes its own, whoever has one carries it out without waiting for
// anybody, and only a workgroup that has none waits -- for the ones that hold them, which run, and it looks now and then for shares
// whose workgroups are not there and carries those out as well.  So a share and the one before it on the same blocks may belong to
// different compute dies: ratios, codes, scales and the tensor's results are read and written at the memory side, and a share is
// counted as done when its stores have been performed there.
// Three of fifteen iterations do work (a launch for each / one for all after the fourth): 12288 x 4096 240 / 219 us, a layer of hidden 512 108 / 74,
// the closed-form arm there 108 / 64.  All of them do (early_stop_rel 1e-30): four matrices of 2 million weights 253 / 226 us, two of 17 million
// 664 / 640, one of 50 million 407 / 382, the closed-form arm there 393 / 378.  With one counter that hands the shares out, which is served in 12 ns a
// workgroup, and the stop flag and the scale read from the same line by all, those took 276, 760, 416 and 521.
enum class Iterate { CLOSED_FORM, NEAREST, OTHER };
template <int DT, Iterate KIND>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_iter_rest(const Batch batch, int iters)
{
    __shared__ float4 s_blocks[kStage * kWG];
    __shared__ double s_wave[3][4];
    __shared__ double s_stack[3][32];
    __shared__ uint32_t s_last, s_share, s_it;
    __shared__ uint64_t s_next;
    __shared__ float s_alpha;
    double *s_tree = reinterpret_cast<double *>(s_blocks);      // trees_of_partials, after the last group
    extern __shared__ __align__(16) unsigned char s_dyn[];      // the factor table, n_beta floats
    float *s_beta = reinterpret_cast<float *>(s_dyn);
    auto get = [](auto *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };

    uint32_t lwg;
    const Task t = batch.t[find_task(batch, lwg)];
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t amax_bits = t.ctrl->amax_bits;
    if (amax_bits == 0u || amax_bits >= 0x7F800000u) return;    // finished by the first iteration
    if (t.ctrl->stopped) return;                                // by a launch before: this one does not write it
    RestWords &rest = rest_words(t);
    const bool dss_only = batch.arm == SOAR_METHOD_DSS_ONLY;
    JointSearch js{{s_beta, batch.n_beta, batch.beta_lo, batch.index_per_beta}, 0.0f, 0.0f, batch.radius,
                   batch.dd_mode == SOAR_DD_BRACKET, dss_only, false, batch.full_search != 0 || batch.n_beta < kChangesMinBeta};
    // wave 0: takes a share of iteration `it` if it is left (the same in every lane)
    auto take = [&](uint32_t share, uint32_t it) -> bool {
        uint32_t before = 0u;
        if (lane == 0) before = __hip_atomic_fetch_max(&rest.taken[share], it + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)before) <= it;
    };

    bool filled = false, helping = false;    // helping: some workgroups were not there before
    const float first_alpha = t.ctrl->alpha1;
    for (uint32_t asked = 0u;;) {            // one more than the last iteration of which this workgroup has asked for its share
        if (tid < 64u) {
            uint32_t it, share = lwg;
            float alpha;
            for (uint32_t looks = helping ? kRestLooks - 1u : 0u;; ++looks) {
                const uint64_t next = get(&rest.next[lwg % 16u][0]);
                it = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)next);
                alpha = f_of((uint32_t)(next >> 32));
                if (it == 0u) {
                    it = (uint32_t)batch.iter_t;
                    alpha = first_alpha;
                }
                if (it >= (uint32_t)iters) break;
                if (it >= asked) {
                    asked = it + 1u;
                    share = lwg;
                    if (take(share, it)) break;
                } else if (looks % kRestLooks == kRestLooks - 1u) {
                    bool found = false;
                    // 64 at a time, every workgroup from a place of its own on and another one of those that are left
                    uint32_t me = lane;
                    asm volatile("" : "+v"(me));     // what is computed from it is not kept in registers through the search
                    const uint32_t start = lwg * 0x9E3779B1u % t.n_wg;
                    for (uint32_t first = 0; first < t.n_wg && !found;) {
                        const uint32_t at = (start + first + me) % t.n_wg;
                        const bool is_left = first + me < t.n_wg && get(&rest.taken[at]) <= it;
                        const uint64_t left = __builtin_amdgcn_ballot_w64(is_left);
                        if (left == 0ull) {
                            first += 64u;
                            continue;
                        }
                        const uint32_t rank = (uint32_t)__builtin_popcountll(left & ((1ull << me) - 1ull));
                        const uint64_t mine = __builtin_amdgcn_ballot_w64(is_left && rank == lwg % (uint32_t)__builtin_popcountll(left));
                        share = (uint32_t)__builtin_amdgcn_readlane((int)at, (int)__builtin_ctzll(mine));
                        found = take(share, it);     // (where another one was faster, it is no longer left)
                    }
                    helping = helping || found;
                    if (found) break;
                }
                __builtin_amdgcn_s_sleep(16);
            }
            if (tid == 0) {
                s_it = it;
                s_share = share;
                s_alpha = alpha;
            }
        }
        __syncthreads();
        const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_it);
        const uint32_t share = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_share);
        const float alpha = f_of((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(s_alpha)));
        if (it >= (uint32_t)iters) return;
        if constexpr (KIND != Iterate::CLOSED_FORM)
            for (int k = filled ? batch.n_beta : (int)tid; k < batch.n_beta; k += kWG) s_beta[k] = beta_factor(k, batch.n_beta, batch.beta_lo, batch.beta_hi);
        __syncthreads();                     // the factors; and what this workgroup has been told has been read
        filled = true;
        js.set_alpha(alpha, amax_bits);
        StagedTree<> tree{s_blocks, s_wave, s_stack};
        const uint32_t T = t.tiles_per_wg < (uint32_t)kStage ? t.tiles_per_wg : (uint32_t)kStage;   // power of two
        for (uint32_t chunk = share; chunk < t.n_chunks; chunk += t.n_wg) {
            for (uint32_t kg = 0; kg < t.tiles_per_wg; kg += T) {
                for (uint32_t kk = 0; kk < T; ++kk) {
                    const uint32_t i = (chunk * t.tiles_per_wg + kg + kk) * kWG + tid;
                    BlockState x;
                    x.a = x.b = x.d = x.err = 0.0f;
                    if (i < t.nblk) {
                        const float rho = get(t.rho + i);
                        float w[16];
                        load_block<DT>(t.w, block_offset(t, i), w);
                        if constexpr (KIND == Iterate::CLOSED_FORM)
                            closed_form_block(w, rho, alpha, js.inv_alpha, js.in_range && all_near_one(rho), x);
                        else
                            iterate_block<KIND == Iterate::NEAREST>(w, rho, js, x);
                        put<true>(t.rho + i, x.rho);
                        put<true>(reinterpret_cast<uint64_t *>(t.codes) + i, (uint64_t)x.nib[1] << 32 | x.nib[0]);
                        put<true>(t.scales + i, (uint8_t)x.code);
                    }
                    tree.stage(kk, x.a, x.b, x.d, x.err);
                }
                tree.close(kg / T, T);
            }
            if (tid == 0) {
                publish(t.part + chunk, tree.wg[0]);
                publish(t.part + kMaxPartials + chunk, tree.wg[1]);
                publish(t.part + 2 * kMaxPartials + chunk, tree.wg[2]);
            }
        }
        wait_then_read();                                   // every wave: its stores have been performed
        __syncthreads();
        uint32_t *counters = t.counters + 2 * kSlots * kSlotStride;
        if (tid == 0) s_last = arrive_is_last(counters, &t.ctrl->top[2], t.n_wg, share) ? 1u : 0u;
        __syncthreads();
        if (s_last) {
            double NME[3];
            trees_of_partials<3>(t.part, t.n_chunks, s_tree, &s_stack[0][0], NME);
            if (tid == 0) s_next = finish_iteration<true>(batch, t, (int)it, NME[0], NME[1], NME[2], alpha, false, false, dss_only);
            if (tid < kSlots) put<true>(counters + tid * kSlotStride, 0u);
            if (tid == 0) put<true>(&t.ctrl->top[2], 0u);
            wait_then_read();
            __syncthreads();
            uint32_t copy = tid;
            asm volatile("" : "+v"(copy));   // its address is not kept in registers from before the search
            if (copy < 16u) put<true>(&rest.next[copy][0], s_next);
        }
    }
}

}  // namespace
