// MXFP4 (blocks of 32, E8M0 scale; OCP Microscaling Formats v1.0), plain conversion or with the
// decoupled scale search of Sec. 3.3 carried over to it (Sec. 4.3): k_mx.
#pragma once
#include "soar_device.hpp"
#include "soar_iterated.hpp"      // TileTree, FactorGrid
#include "soar_once.hpp"

namespace {

// Blocks of 32 elements with an E8M0 scale byte (OCP Microscaling Formats v1.0), plain
// conversion or with the decoupled scale search of Sec. 3.3 carried over to it (Sec. 4.3,
// "DSS on MXFP4").  One lane owns one block of 64 (bf16) or 128 (fp32) bytes.
// There is no tensor-wide scale, so this is a single pass; the only tensor-wide result is the
// error sum (exact adjacent-pair tree, as in the iterated path).
struct MxTask {
    const void *w;
    uint8_t  *codes, *scales;
    double   *sse;
    int32_t  *status;
    int64_t  ld;
    uint32_t bpr;            // 32-element blocks per row
    uint32_t nblk;
    uint32_t tiles_per_wg;
    uint32_t contiguous;
    uint32_t wg_begin;       // first workgroup of the grid that works on this tensor
    uint32_t n_wg;
    Ctrl     *ctrl;          // amax_bits is used as the "saw a non-finite value" flag
    uint32_t *counters;
    double   *part;
    int32_t  n_beta, radius;
    float    beta_lo, beta_hi;
    float    index_per_beta;
};

// What k_mx does with a block.  NEAREST: the factors that can win are found without walking the grid (mx_search_nearest,
// see nearest_search); CHANGES: codes of every factor, errors where they change (mx_search_changes); EVERY: all factors
// (mx_search: single_pass, grids of fewer than kChangesMinBeta factors)
enum class Mx { PLAIN, EVERY, CHANGES, NEAREST };

struct MxBatch {
    MxTask   t[kGroupMax];
    uint32_t n;
    uint32_t once;           // one tensor of at most kOnceMaxWG workgroups: finished by once_sum, no counters
    OnceArgs once_args;
};

// 2^(e-127) for an E8M0 code e in [0, 254]; e = 0 is the binary32 subnormal 2^-127
__device__ __forceinline__ float e8m0_value(int e) { return f_of(e > 0 ? (uint32_t)e << 23 : 0x00400000u); }

__device__ __forceinline__ void mx_assign_rcp(const float w[32], float r, uint32_t nib[4], float q[32])
{
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = w[8 * h + j] * r;
        uint32_t v = nib[h];
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[0], x[1], 1.0f, 0);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[2], x[3], 1.0f, 1);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[4], x[5], 1.0f, 2);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[6], x[7], 1.0f, 3);
        nib[h] = v;
        fp4x8_values(v, q + 8 * h);
    }
}

template <bool FAST>
__device__ __forceinline__ void mx_assign(const float w[32], float scale, uint32_t nib[4], float q[32])
{
    mx_assign_rcp(w, FAST ? rcp_midrange(scale) : 1.0f / scale, nib, q);
}

// Eq. 8 with alpha = 1 over the 32 elements: one ascending chain of fused operations
__device__ __forceinline__ float mx_block_error(const float w[32], const float q[32], float s)
{
    const float ns = -s;
    float err = 0.0f;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        float e = __builtin_fmaf(q[j], ns, w[j]);
        err = __builtin_fmaf(e, e, err);
    }
    return err;
}

// candidate number c of the search order 0,-1,+1,-2,...; a code outside [0, 254] is clamped onto an
// already evaluated candidate of the same factor and can then never win
__device__ __forceinline__ int mx_candidate(int e0, int c)
{
    const int o = (c + 1) >> 1;
    return (c & 1) ? max(e0 - o, 0) : min(e0 + o, 254);
}

// Least Eq. 8 error over the stored codes e0-K..e0+K for fixed element codes q.  For fixed codes the
// exact error is a parabola in the scale, f(x) = A - 2Bx + Cx^2 with B = sum w q, C = sum q^2 and
// minimiser x* = B/C, and f(2x) < f(x) exactly when x* > 1.5 x: the power of two nearest to x* in
// that sense, clamped to the window, is the winner, and only its error chain is evaluated -- provided
// that x* stays clear of the two decision points next to it by a margin far above the rounding error
// of the computed B/C, and that the exact rise to either neighbour, C x |3x - 2x*|, exceeds the
// worst-case rounding error of the binary32 chains (34 ulp relative, all terms non-negative) by a
// wide factor; candidates further out lie higher still (the bound grows with the rise).  Where that
// cannot be shown for some lane of the wave, the other candidates are evaluated too, as the definition
// says: the result never depends on the shortcut.
__device__ __forceinline__ float mx_window_min(const float w[32], const float q[32], int e0, int radius)
{
    bool sure = false;
    float m = 0.0f;
    int cw = e0;
    {
        float B = 0.0f, C = 0.0f;
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            B = __builtin_fmaf(w[j], q[j], B);
            C = __builtin_fmaf(q[j], q[j], C);
        }
        const int lo = max(e0 - radius, 0), hi = min(e0 + radius, 254);
        const float xstar = B * __builtin_amdgcn_rcpf(C);
        // 0.75 * 2^(c-127) < x* <= 1.5 * 2^(c-127)  <=>  c = biased exponent of x* * 4/3 (approximately: checked below)
        cw = (int)(__float_as_uint(xstar * 1.33333337f) >> 23);
        cw = min(max(cw, lo), hi);
        const float xw = e8m0_value(cw);
        m = mx_block_error(w, q, xw);
        // magnitudes at which squares underflow, or overflow, are left to the full evaluation
        sure = C > 0.0f && B > 0x1p-100f && m > 0x1p-100f && m < 0x1p100f && xstar < 0x1p100f && cw >= 2 && cw <= 252;
        const float clear = 0x1p-14f * xstar;       // the computed x* is within 2^-18.8 of the exact one
        if (cw > lo) {
            const float x = 0.5f * xw;
            const float g = 2.0f * xstar - 3.0f * x;
            const float rise = C * x * g;
            sure = sure && g > clear && 0.8f * rise > 0x1p-16f * (m + rise);
        }
        if (cw < hi) {
            const float g = 3.0f * xw - 2.0f * xstar;
            const float rise = C * xw * g;
            sure = sure && g > clear && 0.8f * rise > 0x1p-16f * (m + rise);
        }
    }
    if (__builtin_amdgcn_ballot_w64(!sure) != 0ull) {
        // the 2K other codes of the window (cw is one of them; a code clamped onto [0, 254] repeats another)
        for (int t = 0; t < 2 * radius; ++t) {
            int c = e0 - radius + t;
            c += c >= cw ? 1 : 0;
            m = fminf(m, mx_block_error(w, q, e8m0_value(min(max(c, 0), 254))));
        }
    }
    return m;
}

template <bool FAST>
__device__ __forceinline__ void mx_search(const float w[32], int e0, const float *s_beta, int n_beta, int radius,
                                          float &best_err, int &best_code, uint32_t best_nib[4], float q[32])
{
    const float x0 = e8m0_value(e0);
    uint32_t nib[4] = {0u, 0u, 0u, 0u};
    float best = __builtin_inff();
    float best_beta = s_beta[0];
    for (int kb = 0; kb < n_beta; ++kb) {
        const float bk = s_beta[kb];
        mx_assign<FAST>(w, x0 * bk, nib, q);
        const float m = mx_window_min(w, q, e0, radius);
        best_beta = (m < best) ? bk : best_beta;             // strictly better only: the first factor keeps a tie
        best = fminf(best, m);
    }
    // the winning factor once more: its codes, and the first stored code that reaches its least error
    best_nib[0] = best_nib[1] = best_nib[2] = best_nib[3] = 0u;
    mx_assign<FAST>(w, x0 * best_beta, best_nib, q);
    best_code = e0;
    best_err = mx_block_error(w, q, x0);
    for (int c = 1; c <= 2 * radius; ++c) {
        const int code = mx_candidate(e0, c);
        const float e = mx_block_error(w, q, e8m0_value(code));
        if (e < best_err) { best_err = e; best_code = code; }
    }
}

template <bool FAST>
__device__ __forceinline__ void mx_codes_only(const float w[32], float scale, uint32_t nib[4])
{
    const float r = FAST ? rcp_midrange(scale) : 1.0f / scale;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = w[8 * h + j] * r;
        uint32_t v = nib[h];
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[0], x[1], 1.0f, 0);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[2], x[3], 1.0f, 1);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[4], x[5], 1.0f, 2);
        v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, x[6], x[7], 1.0f, 3);
        nib[h] = v;
    }
}

// mx_search in two passes, as joint_search_changes: codes of every factor first, errors only where this block's change;
// one window minimum per change, whatever the radius
template <bool FAST>
__device__ __forceinline__ void mx_search_changes(const float w[32], int e0, const float *s_beta, int n_beta, int radius,
                                                  float &best_err, int &best_code, uint32_t best_nib[4], float q[32])
{
    const float x0 = e8m0_value(e0);
    uint32_t nib[4] = {0u, 0u, 0u, 0u}, even[4] = {0u, 0u, 0u, 0u}, odd[4] = {0u, 0u, 0u, 0u};
    auto differ = [&]() { return ((even[0] ^ odd[0]) | (even[1] ^ odd[1]) | (even[2] ^ odd[2]) | (even[3] ^ odd[3])) != 0u; };
    float best = __builtin_inff();
    float best_beta = s_beta[0];
    for (int base = 0; base < n_beta; base += kStretch) {
        ChangeSet set;
        for (int first = base; first < min(n_beta, base + kStretch); first += 32) {
            uint32_t word = first == 0 ? 1u : 0u;
            for (int k = 0; k < min(n_beta - first, 32); k += 2) {
                mx_codes_only<FAST>(w, x0 * s_beta[first + k], even);
                word |= differ() ? 1u << k : 0u;
                if (first + k + 1 == n_beta) break;
                mx_codes_only<FAST>(w, x0 * s_beta[first + k + 1], odd);
                word |= differ() ? 2u << k : 0u;
            }
            set.push(word);
        }
        set.settle();
        while (__builtin_amdgcn_ballot_w64(!set.empty()) != 0ull) {
            if (!set.empty()) {
                const float bk = s_beta[base + set.pop()];
                mx_assign<FAST>(w, x0 * bk, nib, q);
                const float m = mx_window_min(w, q, e0, radius);
                best_beta = (m < best) ? bk : best_beta;
                best = fminf(best, m);
            }
        }
    }
    best_nib[0] = best_nib[1] = best_nib[2] = best_nib[3] = 0u;
    mx_assign<FAST>(w, x0 * best_beta, best_nib, q);
    best_code = e0;
    best_err = mx_block_error(w, q, x0);
    for (int c = 1; c <= 2 * radius; ++c) {
        const int code = mx_candidate(e0, c);
        const float e = mx_block_error(w, q, e8m0_value(code));
        if (e < best_err) { best_err = e; best_code = code; }
    }
}

// mx_search without walking the factor grid: joint_search_nearest's argument, with the power of two X0 in the place
// of alpha Delta* -- so which factors enclose a candidate scale is the same for every block of the launch.  Bound by vector issue.
// One decoder layer (1.93e8 bf16 weights, the paper's grid, K = 1): all 303 pairs 3.70 ms a call, the two factors around every
// candidate (six pairs) 0.208, the three that are left below 0.132.
__device__ __forceinline__ float mx_factor_error(const float w[32], float t, float s, uint32_t nib[4])
{
    float q[32];
#pragma unroll
    for (int h = 0; h < 4; ++h) nib[h] = any_word();
    mx_assign<true>(w, t, nib, q);
    return mx_block_error(w, q, s);
}

// best_factor for one stored scale s = ratio * x0; `wanted`: the lane takes part.
// A factor that IS the ratio (the default grid holds 0.5 and 1) assigns the codes nearest to w / s: with them the exact error is
// the least for s, and a larger factor can at best tie.  On bf16 weights (GRID16) binary32 does not change that: w / s is a bf16
// number y, the codes another factor moves from q to q' lie across a midpoint m of the E2M1 grid, and either y = m -- the
// residual only changes its sign, computed errors are equal, the smaller factor keeps the tie -- or |y - m| is a whole unit of y's last
// place, at least 2^-10, and the error rises by 2 |q - q'| |y - m| s^2 >= 2^-10 s^2: more than the rounding of two errors (34 units of
// 2^-24 each) below 200 s^2.  So nothing above such a factor is evaluated; the factor below it is, because of the ties.
constexpr float kEqualFactorError = 200.0f;      // of s^2
template <bool GRID16>
__device__ __forceinline__ float mx_best_factor(const float w[32], float x0, float ratio, const FactorGrid &grid, float s, bool wanted,
                                                uint32_t nib[4], int &k)
{
    const int last = grid.n - 1;
    const float at = (ratio - grid.lo) * grid.index_per_beta;
    // one factor where s lies beyond an end of the grid, else the two around it
    int lo = (int)__builtin_amdgcn_fmed3f(at, 0.0f, (float)last);
    int hi = at < 0.0f ? lo : min(lo + 1, last);
    if (grid.table[lo] == ratio) {               // the upper of the two, or the only one
        hi = lo;
        lo = max(lo - 1, 0);
    }
    const float per_error = s * (1.0f / kFarSideRounding32), slack = s * (0x1p-21f * per_error);
    auto excluded = [&](float distance, float e) { return __builtin_fmaf(distance, per_error, -slack) > e; };
    auto nothing_above = [&](float t, float e) { return excluded(t - s, e) || (GRID16 && t == s && e < kEqualFactorError * (s * s)); };
    const float ta = x0 * grid.table[lo];
    float err = mx_factor_error(w, ta, s, nib);
    k = lo;
    bool down = wanted && lo > 0 && !excluded(s - ta, err), up = wanted && hi < last;
    uint32_t nib_b[4];
    if (__builtin_amdgcn_ballot_w64(wanted && hi != lo) != 0ull) {
        const float tb = x0 * grid.table[hi];    // once more the same where there is only one
        const float err_b = mx_factor_error(w, tb, s, nib_b);
        up = up && !nothing_above(tb, err_b);
        const bool take_b = err_b < err;         // the smaller factor keeps a tie
        err = take_b ? err_b : err;
        k = take_b ? hi : lo;
#pragma unroll
        for (int h = 0; h < 4; ++h) nib[h] = take_b ? nib_b[h] : nib[h];
    } else {
        up = up && !nothing_above(ta, err);
    }
    while (__builtin_amdgcn_ballot_w64(down || up) != 0ull) {
        if (down || up) {
            const int kk = down ? --lo : ++hi;
            const float t = x0 * grid.table[kk];
            const float e = mx_factor_error(w, t, s, nib_b);
            const bool far = excluded(down ? s - t : t - s, e);
            if (e < err || (e == err && kk < k)) {
                err = e;
                k = kk;
#pragma unroll
                for (int h = 0; h < 4; ++h) nib[h] = nib_b[h];
            }
            if (down) down = !far && lo > 0;
            else up = !far && hi < last;
        }
    }
    return err;
}

// The candidates of one distance from X0, X0 2^-o and X0 2^o, are asked of different blocks, so that one evaluation with a
// scale of its own per lane usually serves both:
//  - X0 2^-o is left out where the largest weight alone, which its codes cannot reach, makes an error above the best so far
//    (a rounding of 34 units of 2^-24 is allowed for);
//  - X0 2^o is left out for bf16 weights whose block ends at or below 6 X0, if the grid holds the factor 1: up to 6 X0 every point of
//    its grid is a point of X0's, so the codes nearest under X0 are at least as good, by 2^-10 X0^2 or more unless all residuals
//    are equal up to sign (see mx_best_factor; the error under X0 is at most 32 X0^2), and in that tie X0 comes first: for the largest
//    weight, 4 X0 or more, to take a code of 3.5 or less -- as it has to under X0 2^o -- the factor must exceed 1.
// Pairs evaluated per block of the default grid: three (50 and 49 for X0, one for either side), where the two around every candidate
// and the one beyond an equal factor were six.
constexpr float kMissMargin = 0.9999f;
template <bool GRID16>
__device__ __forceinline__ void mx_search_nearest(const float w[32], float bmax, int e0, const FactorGrid &grid, int radius,
                                                  float &best_err, int &best_code, uint32_t best_nib[4])
{
    const float x0 = e8m0_value(e0);
    int best_k;
    best_code = e0;
    best_err = mx_best_factor<GRID16>(w, x0, 1.0f, grid, x0, true, best_nib, best_k);
    const int at_one = (int)__builtin_amdgcn_fmed3f((1.0f - grid.lo) * grid.index_per_beta, 0.0f, (float)(grid.n - 1));
    const bool holds_one = grid.table[at_one] == 1.0f || grid.table[min(at_one + 1, grid.n - 1)] == 1.0f;
    const bool no_larger = GRID16 && holds_one && bmax <= 6.0f * x0;
    auto candidate = [&](int code, float ratio, bool wanted) {
        uint32_t nib[4];
        int k;
        const float err = mx_best_factor<GRID16>(w, x0, ratio, grid, ratio * x0, wanted, nib, k);
        bool win = wanted && err < best_err;
        const bool tie = wanted && err == best_err && k < best_k;
        if (__builtin_amdgcn_ballot_w64(tie) != 0ull)
            win = win || (tie && (nib[0] != best_nib[0] || nib[1] != best_nib[1] || nib[2] != best_nib[2] || nib[3] != best_nib[3]));
        best_err = win ? err : best_err;
        best_code = win ? code : best_code;
        best_k = win ? k : best_k;
#pragma unroll
        for (int h = 0; h < 4; ++h) best_nib[h] = win ? nib[h] : best_nib[h];
    };
    // e0 and the radius are such (k_mx, mx_nearest_pays) that no candidate leaves the range of the stored codes
#pragma unroll 1
    for (int o = 1; o <= radius; ++o) {
        const float below = f_of((uint32_t)(127 - o) << 23), above = f_of((uint32_t)(127 + o) << 23);
        const float miss = fmaxf(__builtin_fmaf(below * x0, -6.0f, bmax), 0.0f);
        bool lower = !(kMissMargin * (miss * miss) > best_err), upper = !no_larger;
        // the lower one first, in a round of its own where a block asks for both
        while (__builtin_amdgcn_ballot_w64(lower || upper) != 0ull) {
            candidate(lower ? e0 - o : e0 + o, lower ? below : above, lower || upper);
            upper = upper && lower;
            lower = false;
        }
    }
}

// TileTree<1> at a fraction of the cross-lane work and the barriers: terms of up to kStage consecutive tiles are staged in LDS, a lane
// folds adjacent ones, and one wave tree finishes the group (as StagedTree does for three sums).
struct StagedSum {
    double *s_terms;             // [kStage * kWG]
    double (*s_wave)[4];
    double (*s_stack)[32];
    double wg = 0.0;
    // tile kk of a group of T tiles (a power of two)
    __device__ __forceinline__ void stage(uint32_t kk, double term) { s_terms[kk * kWG + threadIdx.x] = term; }
    // group `k` of the workgroup
    __device__ __forceinline__ void close(uint32_t k, uint32_t T)
    {
        __syncthreads();
        const double *x = s_terms + threadIdx.x * T;
        double v = x[0];
        if (T >= 2) v = v + x[1];
        if (T == 4) v = v + (x[2] + x[3]);
        v = wave_pair_tree(v);
        if ((threadIdx.x & 63) == 0) s_wave[0][threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            double y = (s_wave[0][0] + s_wave[0][1]) + (s_wave[0][2] + s_wave[0][3]);
            uint32_t lvl = 0;
            while ((k >> lvl) & 1u) { y = s_stack[0][lvl] + y; ++lvl; }
            s_stack[0][lvl] = wg = y;
        }
    }
};

// STAGED: the nearest-factor search where a workgroup has several tiles: one decoder layer 136 -> 130 us, 6000 tiles of fp32 57.8 -> 55.8, 20000
// of them 193 -> 176.  With one tile there is nothing to fold, and the same kernel is slower than one without the staging (3094 tiles of bf16 24.9 us / 24.0, 4000
// 29.2 / 28.2); so are the searches that walk the grid (3094 tiles 577 / 571 us, 12000 2002 / 1982) and the plain conversion (up to 7 %).
// (held to four waves per SIMD: left to itself the compiler takes three for the staged sum)
template <int DT, Mx MODE, bool STAGED>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(STAGED ? 4 : 1))) void k_mx(const MxBatch batch)
{
    constexpr bool DSS = MODE != Mx::PLAIN;
    __shared__ double s_wave[1][4];
    __shared__ double s_stack[1][32];
    __shared__ double s_tree[kWG];
    __shared__ uint32_t s_last;
    constexpr int kP = pieces_per_block<DT, 32>();
    __shared__ u32x4 s_x[(DSS || DT != SOAR_BF16) ? 1 : kWG * kP];   // load_wave_blocks: one region per wave
    extern __shared__ __align__(16) unsigned char s_dyn_mx[];      // the factor table
    float *s_beta = reinterpret_cast<float *>(s_dyn_mx);

    const uint32_t tid = threadIdx.x;
    uint32_t which = 0;
    for (uint32_t j = 1; j < batch.n; ++j)
        if (blockIdx.x >= batch.t[j].wg_begin) which = j;
    const MxTask t = batch.t[which];
    const uint32_t lwg = blockIdx.x - t.wg_begin;
    const int n_beta = DSS ? t.n_beta : 0;
    for (int k = (int)tid; k < n_beta; k += kWG) s_beta[k] = beta_factor(k, n_beta, t.beta_lo, t.beta_hi);
    __syncthreads();

    const FactorGrid grid{s_beta, n_beta, t.beta_lo, t.index_per_beta};
    TileTree<1> tree{s_wave, s_stack};
    __shared__ double s_terms[STAGED ? kStage * kWG : 1];
    StagedSum staged{s_terms, s_wave, s_stack};
    const uint32_t T = t.tiles_per_wg < (uint32_t)kStage ? t.tiles_per_wg : (uint32_t)kStage;   // power of two
    uint64_t epoch = 0;
    if (batch.once && t.n_wg > 1u) epoch = __hip_atomic_load(&t.ctrl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool nonfinite = false;
    const uint32_t tile0 = lwg * t.tiles_per_wg;
    for (uint32_t k = 0; k < t.tiles_per_wg; ++k) {
        const uint32_t i = (tile0 + k) * kWG + tid;
        double term[1] = {0.0};
        float w[32];
        // the plain conversion is bound by the reads: packed rows go through the coalescing exchange
        const bool exchanged = !DSS && DT == SOAR_BF16 && t.contiguous;
        if constexpr (!DSS && DT == SOAR_BF16) {
            if (exchanged) load_wave_blocks<DT, 32, true>(t.w, i - (tid & 63u), t.nblk, s_x + (tid >> 6) * (64 * kP), w);
        }
        if (i < t.nblk) {
            float q[32];
            uint32_t nib[4] = {0u, 0u, 0u, 0u};
            if (!exchanged) {
                size_t off;
                if (t.contiguous) {
                    off = (size_t)i * 32;
                } else {
                    const uint32_t row = i / t.bpr;
                    off = (size_t)row * (size_t)t.ld + (size_t)(i - row * t.bpr) * 32;
                }
                // ordinary loads: a lane's four or eight loads share cache lines, which streaming loads would drop
                load_block<DT, false>(t.w, off, w);
                load_block<DT, false>(t.w, off + 16, w + 16);
            }
            uint32_t mbits = 0u;
#pragma unroll
            for (int j = 0; j < 32; ++j) mbits = max(mbits, __float_as_uint(w[j]) & 0x7FFFFFFFu);
            nonfinite = nonfinite || mbits >= 0x7F800000u;
            const float bmax = f_of(mbits);
            // bmax = m 2^ex with m in [0.5, 1): floor(log2 bmax) = ex - 1; the largest E2M1 value is 1.5 * 2^2
            const int ex = __builtin_amdgcn_frexp_expf(bmax);
            const int e0 = mbits == 0u ? 127 : min(max(ex - 1 - 2, -127), 127) + 127;
            int code = e0;
            float err;
            if constexpr (!DSS) {
                const float x0 = e8m0_value(e0);
                mx_assign_rcp(w, e8m0_value(254 - e0), nib, q);        // 1 / X0, exact for every code
                err = mx_block_error(w, q, x0);
            } else {
                // far enough from the ends of the binary32 range for the nearest-factor search (factors within
                // 2^-20 .. 2^20: the host)?  Elsewhere the reciprocal shortcut needs the scales X0 beta_k to stay within
                // biased exponents [1, 252].
                const bool near = (uint32_t)(e0 - 67) < 120u;
                if (MODE == Mx::NEAREST && __builtin_amdgcn_ballot_w64(!near) == 0ull) {
                    mx_search_nearest<DT == SOAR_BF16>(w, bmax, e0, grid, t.radius, err, code, nib);
                } else {
                    const float s_first = e8m0_value(e0) * s_beta[0], s_final = e8m0_value(e0) * s_beta[n_beta - 1];
                    const bool mid = ((__float_as_uint(s_first) >> 23) - 2u) < 250u && ((__float_as_uint(s_final) >> 23) - 2u) < 250u;
                    const bool fast = __builtin_amdgcn_ballot_w64(!mid) == 0ull;
                    if constexpr (MODE == Mx::EVERY) {
                        if (fast) mx_search<true>(w, e0, s_beta, n_beta, t.radius, err, code, nib, q);
                        else mx_search<false>(w, e0, s_beta, n_beta, t.radius, err, code, nib, q);
                    } else {
                        if (fast) mx_search_changes<true>(w, e0, s_beta, n_beta, t.radius, err, code, nib, q);
                        else mx_search_changes<false>(w, e0, s_beta, n_beta, t.radius, err, code, nib, q);
                    }
                }
            }
            term[0] = (double)err;
            u32x4 packed = {nib[0], nib[1], nib[2], nib[3]};
            __builtin_nontemporal_store(packed, reinterpret_cast<u32x4 *>(t.codes) + i);
            __builtin_nontemporal_store((uint8_t)code, t.scales + i);
        }
        if constexpr (STAGED) {
            staged.stage(k & (T - 1u), term[0]);
            if ((k & (T - 1u)) == T - 1u) staged.close(k / T, T);
        } else {
            tree.add_tile(k, term);
        }
    }
    if constexpr (STAGED) tree.wg[0] = staged.wg;
    if (batch.once) {
        bool flag = __syncthreads_or(nonfinite ? 1 : 0) != 0;
        if (tid >= 64u) return;
        double total = readlane_f64(tree.wg[0], 0);
        if (once_sum(reinterpret_cast<uint64_t *>(t.part) + kOnceWords, &t.ctrl->epoch, epoch, batch.once_args.nonce, lwg, t.n_wg, total,
                     flag) && tid == 0) {
            if (t.sse) *t.sse = total;
            if (t.status) *t.status = flag ? SOAR_STATUS_NONFINITE : 0;
        }
        return;
    }
    if (nonfinite) {
        __hip_atomic_fetch_or(&t.ctrl->amax_bits, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);        // performed before this wave reaches the barrier below
    }
    uint32_t *counters = t.counters;
    if (tid == 0) {
        publish(t.part + lwg, tree.wg[0]);
        s_last = 0u;
    }
    __syncthreads();          // every lane's flag update has been issued before lane 0 counts the workgroup in
    if (tid == 0) s_last = arrive_is_last(counters, &t.ctrl->top[0], t.n_wg, lwg) ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    double total;
    trees_of_partials<1>(t.part, t.n_wg, s_tree, &s_stack[0][0], &total);
    if (tid == 0) {
        const uint32_t flag = __hip_atomic_load(&t.ctrl->amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t.sse) *t.sse = total;
        if (t.status) *t.status = flag ? SOAR_STATUS_NONFINITE : 0;
        t.ctrl->amax_bits = 0u;
    }
    reset_counters(counters, &t.ctrl->top[0]);
}

}  // namespace
