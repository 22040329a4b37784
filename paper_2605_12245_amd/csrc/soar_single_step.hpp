// The single-step path (Algorithm 1 with T = 1, beta = {1}): k_init, k_absmax (Eq. 1), k_stats
// (Eq. 1-2, 5) and k_search (Eq. 6, 8, packing); k_search also serves the plain conversion of Sec. 3.1.
#pragma once
#include "soar_crossing.hpp"
#include "soar_device.hpp"

namespace {

// clears the control words, arrival counters and partial maxima of every slot, except the epoch: a captured one-launch
// call takes its token from a nonce that its replays share and from the epoch, which must not return to an earlier value
// while words with that token lie in the workspace
constexpr int kInitSplit = 8;             // workgroups per slot
constexpr uint32_t kEpochPiece = offsetof(Ctrl, epoch) / 16;
static_assert(kZeroedBytes % 16 == 0, "control region is cleared with 16-byte stores");
static_assert(offsetof(Ctrl, epoch) % 16 == 8 && kSlotBytes % 16 == 0, "the epoch is the second half of its piece");
__global__ __launch_bounds__(kWG) void k_init(char *slots_base)
{
    uint4 *p = reinterpret_cast<uint4 *>(slots_base + (size_t)(blockIdx.x / kInitSplit) * kSlotBytes);
    for (uint32_t k = (blockIdx.x % kInitSplit) * kWG + threadIdx.x; k < kZeroedBytes / 16; k += kInitSplit * kWG)
        if (k == kEpochPiece) *reinterpret_cast<uint2 *>(p + k) = make_uint2(0u, 0u);
        else p[k] = make_uint4(0u, 0u, 0u, 0u);
}

// max |w| over a tensor.  |bits| of finite floats order like the values; NaN
// and Inf patterns are larger than every finite one, so they surface in the max.
// For bf16 the running maximum stays packed (two 16-bit magnitudes per register,
// packed integer max) and is unpacked once per lane; for fp32 it is a plain max.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b)
{
    u16x2 x, y;
    __builtin_memcpy(&x, &a, 4);
    __builtin_memcpy(&y, &b, 4);
    x = __builtin_elementwise_max(x, y);
    uint32_t r;
    __builtin_memcpy(&r, &x, 4);
    return r;
}

template <int DT>
__device__ __forceinline__ uint32_t absmax_accumulate(uint32_t m, uint4 v)
{
    if constexpr (DT == SOAR_BF16) {
        const uint32_t k = 0x7FFF7FFFu;
        return pk_max_u16(pk_max_u16(m, pk_max_u16(v.x & k, v.y & k)), pk_max_u16(v.z & k, v.w & k));
    } else {
        const uint32_t k = 0x7FFFFFFFu;
        return max(max(m, max(v.x & k, v.y & k)), max(v.z & k, v.w & k));
    }
}

template <int DT>
__global__ __launch_bounds__(kWG) void k_absmax(const Batch batch)
{
    __shared__ uint32_t s_wave[4];
    __shared__ uint32_t s_last;
    uint32_t lwg;
    const Task t = batch.t[find_task(batch, &Task::absmax, lwg)];
    const Shape sh = t.absmax;
    const uint32_t tid = threadIdx.x;
    constexpr int kChunks = DT == SOAR_BF16 ? 2 : 4;      // 16-byte pieces per block

    // tiles are dealt round-robin over the tensor's workgroups, so that at any moment
    // the workgroups in flight sweep one contiguous window of memory
    uint32_t m = 0;
    for (uint32_t k = 0; k < sh.tiles_per_wg; ++k) {
        const uint32_t i = (k * sh.n_wg + lwg) * kWG + tid;
        if (i >= t.nblk) break;
        const size_t off = block_offset(t, i) * (DT == SOAR_BF16 ? 2 : 4);
        const char *p = static_cast<const char *>(t.w) + off;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const u32x4 v = load16<kStreamAbsmax>(p + 16 * c);
            m = absmax_accumulate<DT>(m, make_uint4(v.x, v.y, v.z, v.w));
        }
    }
    if constexpr (DT == SOAR_BF16) m = max(m & 0xFFFFu, m >> 16) << 16;
    m = wave_max_u32(m);
    if ((tid & 63) == 0) s_wave[tid >> 6] = m;
    __syncthreads();
    uint32_t *counters = t.counters;                       // kernel 0
    if (tid == 0) {
        m = max(max(s_wave[0], s_wave[1]), max(s_wave[2], s_wave[3]));
        const uint32_t ns = sh.n_wg < (uint32_t)kSlots ? sh.n_wg : (uint32_t)kSlots;
        // arrive_is_last waits for this read-modify-write to complete before it counts the workgroup in
        __hip_atomic_fetch_max(t.slot_max + (lwg % ns) * kSlotStride, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = arrive_is_last(counters, &t.ctrl->top[0], sh.n_wg, lwg) ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    if (tid < 64) {
        uint32_t v = tid < kSlots ? __hip_atomic_load(t.slot_max + tid * kSlotStride, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT)
                                  : 0u;
        v = wave_max_u32(v);
        if (tid == 0) t.ctrl->amax_bits = v;
    }
    __syncthreads();
    if (tid < kSlots) t.slot_max[tid * kSlotStride] = 0u;
    reset_counters(counters, &t.ctrl->top[0]);
}

// Eq. 1-2 per block and the two tensor-wide sums of Eq. 5.  The per-block terms
// of kStage consecutive tiles are staged in LDS; lane t then folds the kStage
// adjacent terms t*kStage.. in registers and one wave tree finishes the group,
// which is the same adjacent-pair tree at a fraction of the cross-lane work.
template <int DT>
__global__ __launch_bounds__(kWG) void k_stats(const Batch batch)
{
    __shared__ double2 s_terms[kStage * kWG];
    __shared__ double s_wave[2][4];
    __shared__ double s_stack[2][32];
    __shared__ double s_tree[kWG];
    __shared__ uint32_t s_last;

    uint32_t lwg;
    const Task t = batch.t[find_task(batch, lwg)];
    // backwards through the tensor: what the maximum read last is still in the last-level cache, and the search begins with what
    // this pass reads last (28672 x 8192 bf16, 470 MB: 300.5 -> 296.6 us, fp32 579 -> 575; tensors the cache holds: no change)
    lwg = t.n_wg - 1u - lwg;
    const uint32_t tid = threadIdx.x;
    const uint32_t amax_bits = t.ctrl->amax_bits;
    const bool degenerate = amax_bits == 0u || amax_bits >= 0x7F800000u;
    const GlobalScale gs(amax_bits);
    const float alpha0 = gs.alpha0;

    double wgN = 0.0, wgM = 0.0;
    const uint32_t tile0 = lwg * t.tiles_per_wg;
    const uint32_t T = t.tiles_per_wg < (uint32_t)kStage ? t.tiles_per_wg : (uint32_t)kStage;   // power of two
    for (uint32_t kg = 0; kg < t.tiles_per_wg; kg += T) {
        for (uint32_t kk = 0; kk < T; ++kk) {
            const uint32_t i = (tile0 + kg + kk) * kWG + tid;
            double tN = 0.0, tM = 0.0;
            if (i < t.nblk && !degenerate) {
                float w[16], q[16];
                uint32_t nib[2], c0;
                float delta0, a, b;
                load_block<DT, kStreamStats>(t.w, block_offset(t, i), w);
                block_init(w, gs, c0, delta0, nib, q);
                block_sums(w, q, a, b);
                tN = (double)a * (double)delta0;
                tM = ((double)b * (double)delta0) * (double)delta0;
            }
            s_terms[kk * kWG + tid] = make_double2(tN, tM);
        }
        __syncthreads();
        double vN, vM;
        {
            double2 t0 = s_terms[tid * T];
            vN = t0.x; vM = t0.y;
            if (T >= 2) {
                double2 t1 = s_terms[tid * T + 1];
                vN = vN + t1.x; vM = vM + t1.y;
            }
            if (T == 4) {
                double2 t2 = s_terms[tid * T + 2], t3 = s_terms[tid * T + 3];
                vN = vN + (t2.x + t3.x); vM = vM + (t2.y + t3.y);
            }
        }
        vN = wave_pair_tree(vN);
        vM = wave_pair_tree(vM);
        if ((tid & 63) == 0) { s_wave[0][tid >> 6] = vN; s_wave[1][tid >> 6] = vM; }
        __syncthreads();
        if (tid == 0) {
            // group sum, then binary-counter stack: group k closes every level whose bit of k is set
            vN = (s_wave[0][0] + s_wave[0][1]) + (s_wave[0][2] + s_wave[0][3]);
            vM = (s_wave[1][0] + s_wave[1][1]) + (s_wave[1][2] + s_wave[1][3]);
            const uint32_t k = kg / T;
            uint32_t lvl = 0;
            while ((k >> lvl) & 1u) {
                vN = s_stack[0][lvl] + vN;
                vM = s_stack[1][lvl] + vM;
                ++lvl;
            }
            s_stack[0][lvl] = vN;
            s_stack[1][lvl] = vM;
            wgN = vN; wgM = vM;          // after the last group: the sum of all tiles
        }
    }
    double *partN = t.part, *partM = t.part + kMaxPartials;
    uint32_t *counters = t.counters + 1 * kSlots * kSlotStride;
    if (tid == 0) {
        publish(partN + lwg, wgN);
        publish(partM + lwg, wgM);
        s_last = arrive_is_last(counters, &t.ctrl->top[1], t.n_wg, lwg) ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    // last workgroup of the tensor: finish the trees and apply Eq. 5
    double NM[2];
    trees_of_partials<2>(t.part, t.n_wg, s_tree, &s_stack[0][0], NM);
    const double N = NM[0], M = NM[1];
    if (tid == 0) {
        float alpha1 = (M > 0.0) ? (float)(N / M) : alpha0;
        if (amax_bits == 0u) alpha1 = 1.0f;
        t.ctrl->alpha0 = alpha0;
        t.ctrl->alpha1 = alpha1;
        t.ctrl->N = N;
        t.ctrl->M = M;
        *t.gscale = alpha1;
    }
    reset_counters(counters, &t.ctrl->top[1]);
}

// Exhaustive form of the Eq. 8 search: candidates centre, -1, +1, -2, +2, ...;
// a later one wins only if strictly better.  A code outside [0x01, 0x7E] is
// clamped onto an already evaluated candidate and can then never win.
__device__ __forceinline__ void search_full(const float w[16], const float q[16], float alpha1, int centre,
                                            int radius, int &best, float &best_err)
{
    best = centre;
    best_err = block_error(w, q, alpha1 * e4m3_value_of(centre));
    for (int o = 1; o <= radius; ++o) {
        int cm = max(centre - o, (int)kE4M3Min);
        float em = block_error(w, q, alpha1 * e4m3_value_of(cm));
        if (em < best_err) { best_err = em; best = cm; }
        int cp = min(centre + o, (int)kE4M3Max);
        float ep = block_error(w, q, alpha1 * e4m3_value_of(cp));
        if (ep < best_err) { best_err = ep; best = cp; }
    }
}

// position of a candidate in the search order 0,-1,+1,-2,+2,...
__device__ __forceinline__ int search_rank(int code, int centre)
{
    const int o = code - centre;
    return o < 0 ? -2 * o - 1 : 2 * o;
}

// Certified short form of the same search.  For fixed codes the exact block
// error is a parabola in s = alpha*d, f(s) = A - 2Bs + Cs^2, with minimiser
// s* = B/C (B = sum w q, C = sum q^2).  The two window candidates that bracket
// s* are compared by the parabola, and the winner -- both, where that leaves a doubt -- is evaluated with the very same binary32
// chain as the exhaustive search; it is the exhaustive winner provided that
//   (i)  the bracket really encloses s* (checked with a margin far above the
//        rounding error of the computed B/C), so that f rises monotonically
//        through every other candidate on either side, and
//   (ii) that rise, at least C*h^2 with h the E4M3 spacing (>= s/16), exceeds the
//        worst-case rounding error of the binary32 evaluation (18 ulp relative,
//        all terms being non-negative), so no unevaluated candidate can compute
//        to a value as small as the winner's.
// Where only one side of the bracket fails (i) -- s* within the margin of a candidate -- the next
// candidate on that side is evaluated as well and (i) is asked of the three.
// Returns false when a condition cannot be shown; the caller then runs the
// exhaustive search, so the result never depends on this shortcut.
// One error chain instead of two, with the projections by conversion (e4m3_project), whole calls: 4096 x 4096 in one launch 23.8 -> 23.2 us, 5003 x 3120
// fp32 29.1 -> 28.6, 28672 x 8192, whose search is bound by its vector instructions, 291 -> 282; batches of cached tensors, which are not: no change.
__device__ __forceinline__ bool search_certified(const float w[16], const float q[16], float alpha1,
                                                 float inv_alpha1, int centre, int radius, int &best,
                                                 float &best_err)
{
    float B, C;
    block_sums(w, q, B, C);
    const int wmin = max(centre - radius, (int)kE4M3Min);
    const int wmax = min(centre + radius, (int)kE4M3Max);
    const float sstar = B * __builtin_amdgcn_rcpf(C);
    const float dstar = sstar * inv_alpha1;
    // largest E4M3 code whose value does not exceed dstar (approximately; (i) checks)
    const int lo_n = (int)(__float_as_uint(dstar) >> 20) - (120 << 3);
    const int lo_s = (int)(dstar * 512.0f);
    const int lo = dstar >= 0x1p-6f ? lo_n : lo_s;
    const int ka = min(max(lo, wmin), wmax);
    const int kb = min(max(lo + 1, wmin), wmax);
    const float sa = alpha1 * e4m3_value_of(ka);
    const float sb = alpha1 * e4m3_value_of(kb);
    // ka <= kb <= ka + 1.  f(sb) - f(sa) = C (sb - sa) (sa + sb - 2 s*): its sign names the winner, and where its size leaves no doubt
    // only the winner's error is evaluated (in doubt: one block in ten thousand).  The margins are four times what rounding can
    // do: 2^-18 s* to 2 s*, 2 * 18 * 2^-24 of the error to the difference of two computed ones.
    const float past = __builtin_fmaf(2.0f, sstar, -(sa + sb));
    bool b_wins = past > 0.0f;
    best_err = block_error(w, q, b_wins ? sb : sa);
    const float apart = (C * (sb - sa)) * __builtin_fmaf(-0x1p-16f, sstar, fabsf(past));
    const bool sure = ka == kb || apart > 0x1p-17f * best_err;
    if (__builtin_amdgcn_ballot_w64(!sure) != 0ull) {
        // in the order 0,-1,+1,-2,+2,... the upper of two adjacent codes comes first exactly when the lower one lies below the centre
        const float fa = block_error(w, q, sa), fb = block_error(w, q, sb);
        b_wins = (fb < fa) || (fb == fa && ka < centre);
        best_err = b_wins ? fb : fa;
    }
    best = b_wins ? kb : ka;
    const bool left_ok = (ka == wmin) || (sa * (1.0f + 0x1p-17f) <= sstar);
    const bool right_ok = (kb == wmax) || (sb * (1.0f - 0x1p-17f) >= sstar);
    bool enclosed = left_ok && right_ok;
    if (left_ok != right_ok) {
        // s* sits within the margin of one of the two candidates (about two blocks in ten thousand), so that
        // side of the bracket is in doubt: the next candidate on that side, a whole E4M3 step further out,
        // settles it -- the three enclose s* if it lies clear of s* in its turn.  Its rank in the search
        // order decides ties as in the exhaustive loop.
        const int ke = left_ok ? kb + 1 : ka - 1;            // inside the window: the side in doubt is not at its edge
        const float se = alpha1 * e4m3_value_of(ke);
        const float fe = block_error(w, q, se);
        enclosed = left_ok ? (ke == wmax) || (se * (1.0f - 0x1p-17f) >= sstar)
                           : (ke == wmin) || (se * (1.0f + 0x1p-17f) <= sstar);
        if (fe < best_err || (fe == best_err && search_rank(ke, centre) < search_rank(best, centre))) {
            best = ke;
            best_err = fe;
        }
    }
    const bool margin_ok = best_err < 512.0f * (C * (sa * sa));
    const bool range_ok = (B > 0x1p-100f) && (best_err > 0x1p-100f) && (C > 0.0f);
    return enclosed && margin_ok && range_ok;
}

// Diagnostics (off unless the host asks): how often the certified search had to hand over to the
// exhaustive one.  stats[0] blocks searched, [1] blocks that fell back, [2] wave steps (one block per lane),
// [3] wave steps in which at least one lane fell back (the whole wave then waits for the exhaustive loop).
__device__ __forceinline__ void count_search(unsigned long long *stats, bool certified)
{
    const unsigned long long active = __builtin_amdgcn_ballot_w64(true);
    const unsigned long long fell = __builtin_amdgcn_ballot_w64(!certified);
    if ((threadIdx.x & 63u) == (uint32_t)__builtin_ctzll(active)) {
        atomicAdd(stats + 0, (unsigned long long)__builtin_popcountll(active));
        atomicAdd(stats + 1, (unsigned long long)__builtin_popcountll(fell));
        atomicAdd(stats + 2, 1ull);
        atomicAdd(stats + 3, fell != 0ull ? 1ull : 0ull);
    }
}

// Eq. 6 and the new assignment; returns the projection of Delta* (fast: GlobalScale::fast, and alpha1 near one as well)
__device__ __forceinline__ int new_codes(const float w[16], float rho, float alpha1, float inv_alpha1, bool fast, uint32_t nib[2],
                                         float q[16])
{
    const float delta_star = (rho < 0.0f) ? -rho : quotient(rho, alpha1, inv_alpha1, fast);
    assign_codes(w, alpha1 * delta_star, fast, nib, q);
    return (int)e4m3_project(delta_star);
}

// Eq. 6, projection, new assignment, Eq. 8 search, packing, error sum.
// METHOD RTN emits the Eq. 1-2 state instead.
// Each block's a/b is formed again: a hundred instructions where the statistics would leave it in memory, 4 bytes a block written and read.  Carried /
// formed again: four decoder layers 863 / 830 us, one 256 / 246, four of hidden 2048 248 / 239, 12288 x 4096 75 / 73, 28672 x 8192
// 299 / 285, 36 layers 7.13 / 7.04 ms.
// (bf16: held to 64 registers, eight waves per SIMD; left to itself the compiler takes 83 for a shorter schedule and loses more in
// occupancy than it gains)
template <int DT, int METHOD>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(DT == SOAR_BF16 ? 8 : 4))) void k_search(const Batch batch)
{
    __shared__ double s_wave[4];
    __shared__ double s_tree[kWG];
    __shared__ double s_stack[16];
    __shared__ uint32_t s_last;
    // The coalescing exchange pays where the reads bound the kernel: binary32 input (64 bytes per lane)
    // and the plain conversion.  The bf16 search is as much bound by its arithmetic and gains nothing.
    constexpr bool kExchange = DT == SOAR_FP32 || METHOD == SOAR_METHOD_RTN;
    constexpr int kP = pieces_per_block<DT, 16>();
    __shared__ u32x4 s_x[kExchange ? kWG * kP : 1];    // load_wave_blocks: one region per wave

    uint32_t lwg;
    const Task t = batch.t[find_task(batch, &Task::search, lwg)];
    const Shape sh = t.search;
    const uint32_t tid = threadIdx.x;
    const int radius = batch.radius;
    const bool full_search = batch.full_search != 0;
    // a supplied maximum that is unusable is read as NaN: the arithmetic below stays defined,
    // the outputs are unspecified and the status says why
    bool bad_amax = false;
    uint32_t amax_bits = t.ctrl->amax_bits;
    if (METHOD == SOAR_METHOD_RTN && t.amax_in) {
        const float given = *t.amax_in;
        bad_amax = !(given > 0.0f) || __float_as_uint(given) >= 0x7F800000u;
        amax_bits = bad_amax ? 0x7FC00000u : __float_as_uint(given);
    }
    const bool allzero = amax_bits == 0u;
    const GlobalScale gs(amax_bits, METHOD == SOAR_METHOD_SOAR || !t.amax_in);
    const float alpha0 = gs.alpha0;
    const float alpha1 = (METHOD == SOAR_METHOD_SOAR) ? t.ctrl->alpha1 : alpha0;
    const float inv_alpha1 = 1.0f / alpha1;
    const bool fast = gs.fast && near_one(alpha1);

    // tiles dealt round-robin over the tensor's workgroups (see k_absmax)
    double sse = 0.0;
    for (uint32_t k = 0; k < sh.tiles_per_wg; ++k) {
        const uint32_t i = (k * sh.n_wg + lwg) * kWG + tid;
        float w[16], q[16];
        uint32_t nib[2];
        if (kExchange && t.contiguous) {
            // packed rows: the wave reads its 64 blocks coalesced (all of its lanes take part)
            const uint32_t wave_first = i - (tid & 63u);
            if (wave_first >= t.nblk) break;
            load_wave_blocks<DT, 16, kStreamSearch>(t.w, wave_first, t.nblk, s_x + (tid >> 6) * (64 * kP), w);
            if (i >= t.nblk) break;
        } else {
            if (i >= t.nblk) break;
            load_block<DT, kStreamSearch>(t.w, block_offset(t, i), w);
        }
        uint32_t out_code;
        float out_err;
        if (allzero) {
            // every weight is +-0: smallest scale, zero codes carrying the sign
            float x[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) x[j] = w[j];
            nib[0] = fp4x8(x);
            nib[1] = fp4x8(x + 8);
            out_code = kE4M3Min;
            out_err = 0.0f;
        } else if constexpr (METHOD == SOAR_METHOD_RTN) {
            uint32_t c0;
            float delta0;
            block_init(w, gs, c0, delta0, nib, q);
            out_code = c0;
            out_err = block_error(w, q, alpha0 * delta0);
        } else {
            float rho = 0.0f;                                                       // a / b >= 0, or -Delta0 where b == 0
            if (amax_bits < 0x7F800000u) {
                uint32_t c0;
                float delta0, a, b;
                block_init(w, gs, c0, delta0, nib, q);
                block_sums(w, q, a, b);
                rho = block_ratio(a, b, delta0, gs.fast);
            }
            const int centre = new_codes(w, rho, alpha1, inv_alpha1, fast, nib, q);
            int best;
            float best_err;
            bool done = false;
            if (!full_search) {
                done = search_certified(w, q, alpha1, inv_alpha1, centre, radius, best, best_err);
                if (batch.search_stats) count_search(batch.search_stats, done);
            }
            if (!done) search_full(w, q, alpha1, centre, radius, best, best_err);
            out_code = (uint32_t)best;
            out_err = best_err;
        }
        {
            // streaming stores: the outputs are not read again by this path
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            u32x2 packed = {nib[0], nib[1]};
            __builtin_nontemporal_store(packed, reinterpret_cast<u32x2 *>(t.codes) + i);
            __builtin_nontemporal_store((uint8_t)out_code, t.scales + i);
        }
        sse += (double)out_err;
    }
    // error sum: fixed order for a given launch shape
    sse = wave_pair_tree(sse);
    if ((tid & 63) == 0) s_wave[tid >> 6] = sse;
    __syncthreads();
    double *partS = t.part + 2 * kMaxPartials;
    uint32_t *counters = t.counters + 2 * kSlots * kSlotStride;
    if (tid == 0) {
        publish(partS + lwg, (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]));
        s_last = arrive_is_last(counters, &t.ctrl->top[2], sh.n_wg, lwg) ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    double total;
    trees_of_partials<1>(partS, sh.n_wg, s_tree, s_stack, &total);
    if (tid == 0) {
        if (t.sse) *t.sse = total;
        if (t.status)
            *t.status = bad_amax ? SOAR_STATUS_BAD_AMAX
                                 : (amax_bits >= 0x7F800000u ? SOAR_STATUS_NONFINITE : 0) | (allzero ? SOAR_STATUS_ALLZERO : 0);
        if (METHOD == SOAR_METHOD_RTN) *t.gscale = allzero ? 1.0f : alpha0;
    }
    reset_counters(counters, &t.ctrl->top[2]);
}

// ------------------------------------------------------------------ one launch, the tensor resident on chip
// A tensor handed over alone pays, on the three-pass path, four dependent launches whose ramp and tail
// dominate below a few hundred MiB, and reads its weights three times.  k_resident does the whole
// single-step path in ONE launch of at most one workgroup per compute unit: every lane loads its (up to
// kResMaxPer) blocks once and keeps them in registers as loaded; the two tensor-wide results (the Eq. 1
// maximum, the Eq. 5 sums) cross the grid through words in the workspace; the search then runs from the
// registers.  The weights are read once (2 + 9/16 bytes per bf16 weight instead of 6 + 9/16).
//
// Workgroup g owns the L * R consecutive blocks from g * L * R on (an aligned power of two, so its partial
// sums are nodes of the adjacent-pair tree) and a wave 64 R consecutive ones, in "packets" of up to 128
// bytes of weights per lane: a lane owns ADJACENT blocks (4 bf16 or 2 fp32 blocks per packet; with four
// fp32 blocks per lane a wave's range is two packets).  So the first levels of the tree are additions in
// registers, one DPP wave tree covers a packet of the whole wave, the L/64 wave sums, in block order, go
// through the wave tree once more, and a lane's scale bytes and code bytes leave in one or two stores.
// Packed rows are read through the coalescing wave exchange (load_wave_pieces).  Across workgroups the tree continues over groups of
// consecutive workgroups (one wave tree, a workgroup per lane) and then over the groups (cross_sums).  Same arithmetic, same trees
// as the three-pass path: identical bytes.
constexpr int kResMaxPer = 4;             // blocks per lane, at most

// The crossing words inside Task::part
struct ResidentWords {
    uint64_t max[kMaxEnd];
    SumWords<2> nm;
    uint64_t err[3 * kResMaxWG];
};
static_assert(sizeof(ResidentWords) <= kPartialsBytes, "layout of the crossing words");

struct ResidentArgs {
    int32_t  radius, full_search;
    uint64_t nonce;                       // new for every call
    uint64_t wait_ticks;                  // in ticks of the wall clock: k_resident, bound of the waits of a workgroup together;
                                          // k_iter_resident and k_resident_batch, of its wait for the grid to arrive
    unsigned long long *search_stats;     // null, or the diagnostic counters of count_search
};

// BATCH: workgroup g of the G that work on one tensor of a batch (k_resident_batch, which finishes every tensor: false, all outputs
// unwritten, where this one has to be done again); otherwise the launch is one tensor's.
template <int DT, int METHOD, int L, int R, bool BATCH>
__device__ __forceinline__ bool resident_body(const Task &t, const ResidentArgs &args, ResidentWords *batch_words = nullptr, uint32_t batch_g = 0u,
                                              uint32_t batch_G = 0u, uint64_t *crowded = nullptr)
{
    static_assert(L == 256 || L == 1024, "workgroup of 4 or 16 waves");
    static_assert(R == 1 || R == 2 || R == 4, "blocks per lane");
    constexpr int kWaves = L / 64;
    constexpr int kParts = kWaves;                           // wave sums of a workgroup, in block order
    constexpr int kP = pieces_per_block<DT, 16>();
    constexpr int kX = R * kP <= 8 ? R : 8 / kP;             // adjacent blocks of a lane in one packet (<= 128 bytes)
    constexpr int kPackets = R / kX;                         // 1 or 2
    constexpr int kXP = kX * kP;                             // 16-byte pieces of a lane per packet: 2, 4 or 8
    static_assert(kPackets == 1 || kPackets == 2, "packets of a wave");
    __shared__ u32x4 s_x[kWaves * 64 * kXP];                 // load_wave_pieces: one region per wave
    // first crossing: bf16 maxima have 15 significant bits (sign cleared, low half zero), fp32 ones 31
    constexpr int kMaxBits = DT == SOAR_BF16 ? 15 : 31;
    __shared__ uint32_t s_max[kWaves];
    __shared__ double s_part[3][kParts];
    __shared__ uint64_t s_cross[kSumDirect * SumWords<2>::kW];
    __shared__ float s_alpha1;
    __shared__ uint32_t s_amax, s_gone;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t wave_first = ((BATCH ? batch_g : blockIdx.x) * (uint32_t)L + wave * 64u) * (uint32_t)R;   // first block of this wave
    // block k (0 .. R-1) of this lane: packet k / kX of the wave, there the lane's kX adjacent blocks
    auto blk = [&](int k) -> uint32_t {
        return wave_first + (uint32_t)(k / kX) * (64u * kX) + lane * (uint32_t)kX + (uint32_t)(k % kX);
    };
    uint64_t *epoch_p = &t.ctrl->epoch;

    ResidentGrid grid;
    grid.g = BATCH ? batch_g : blockIdx.x;
    grid.G = BATCH ? batch_G : gridDim.x;
    grid.tok = grid.base = BATCH ? args.nonce : 0;
    grid.t0 = 0;
    grid.ticks = args.wait_ticks;
    ResidentWords &words = *(BATCH ? batch_words : reinterpret_cast<ResidentWords *>(t.part));
    grid.words = words.max;
    uint64_t epoch = 0;
    if (!BATCH && grid.G > 1u) {
        epoch = __hip_atomic_load(epoch_p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        grid.tok = grid.base = args.nonce ^ (epoch * kResOdd);
        grid.t0 = (uint64_t)wall_clock64();
    }
    // a tensor of this batch has waited in vain already
    bool no_room = false;
    if constexpr (BATCH) no_room = __hip_atomic_load(crowded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == grid.base;
    // one lane: leave the launch and tell the others -- whoever gathers this workgroup's words, now or at a
    // later crossing, finds the complemented token in the first of them
    auto give_up = [&]() {
        const uint64_t gone = ~grid.tok << kResSumBits;
        leave_max(grid, ~grid.tok << kMaxBits);
        leave_sums(grid, words.nm, gone);
        if constexpr (!BATCH) {
            __hip_atomic_store(words.err + grid.g, gone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // any change of the epoch will do for the next launch
            __hip_atomic_fetch_add(epoch_p, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (t.status) *t.status = SOAR_STATUS_GAVE_UP;
        }
    };

    // ---- the blocks of this lane, as loaded; Eq. 1 maximum
    u32x4 raw[R][kP];
    uint32_t m = 0;
    if (t.contiguous) {
        // packed rows: the wave reads each packet's range in coalesced 16-byte pieces (all of its lanes take part)
#pragma unroll
        for (int pk = 0; pk < kPackets; ++pk) {
            const uint32_t first = wave_first + (uint32_t)pk * (64u * kX);
            const uint32_t have = first < t.nblk ? min(64u * kX, t.nblk - first) * (uint32_t)kP : 0u;
            u32x4 v[kXP];
            load_wave_pieces<kXP, true>(static_cast<const u32x4 *>(t.w) + (size_t)first * kP, have, s_x + wave * (64 * kXP), v);
#pragma unroll
            for (int q = 0; q < kXP; ++q) raw[pk * kX + q / kP][q % kP] = v[q];
        }
    } else {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const uint32_t i = blk(k);
#pragma unroll
            for (int p = 0; p < kP; ++p) raw[k][p] = u32x4{0u, 0u, 0u, 0u};
            if (i < t.nblk) {
                const char *src = static_cast<const char *>(t.w) + block_offset(t, i) * (DT == SOAR_BF16 ? 2 : 4);
#pragma unroll
                for (int p = 0; p < kP; ++p) raw[k][p] = load16<false>(src + 16 * p);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
        for (int p = 0; p < kP; ++p)
            m = absmax_accumulate<DT>(m, make_uint4(raw[k][p].x, raw[k][p].y, raw[k][p].z, raw[k][p].w));
    if constexpr (DT == SOAR_BF16) m = max(m & 0xFFFFu, m >> 16) << 16;
    m = wave_max_u32(m);
    if (lane == 0) s_max[wave] = m;
    __syncthreads();
    if (wave == 0) {
        uint32_t amax = wave_max_u32(lane < (uint32_t)kWaves ? s_max[lane] : 0u);
        bool ok = true;
        if (grid.G > 1u) {
            uint32_t value = DT == SOAR_BF16 ? amax >> 16 : amax;
            if constexpr (BATCH) grid.t0 = (uint64_t)wall_clock64();
            ok = !no_room && cross_max<kMaxBits>(grid, value);
            amax = DT == SOAR_BF16 ? value << 16 : value;
            if (lane == 0) {
                if (!ok) give_up();
                if (BATCH && !ok) __hip_atomic_store(crowded, grid.base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (!BATCH && ok && grid.g == 0u)    // every workgroup has read the epoch by now: the next launch gets a new token
                    __hip_atomic_store(epoch_p, epoch + 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (lane == 0) { s_amax = amax; s_gone = ok ? 0u : 1u; }
    }
    __syncthreads();
    if (s_gone) return false;
    // from here on every workgroup is running, and either goes on or has given up and said so at this crossing's words and the next
    // one's: the waits end by themselves, and nobody gives up for any other reason than that somebody has
    if constexpr (BATCH) grid.ticks = ~0ull;
    const uint32_t amax_bits = s_amax;
    const bool allzero = amax_bits == 0u;
    const bool degenerate = allzero || amax_bits >= 0x7F800000u;
    const GlobalScale gs(amax_bits);
    const float alpha0 = gs.alpha0;

    auto widen = [&](int k, float w[16]) {
        if constexpr (DT == SOAR_BF16) {
#pragma unroll
            for (int p = 0; p < kP; ++p) {
                const uint32_t u[4] = {raw[k][p].x, raw[k][p].y, raw[k][p].z, raw[k][p].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    w[8 * p + 2 * e] = f_of(u[e] << 16);
                    w[8 * p + 2 * e + 1] = f_of(u[e] & 0xFFFF0000u);
                }
            }
        } else {
#pragma unroll
            for (int p = 0; p < kP; ++p) {
                w[4 * p] = f_of(raw[k][p].x); w[4 * p + 1] = f_of(raw[k][p].y);
                w[4 * p + 2] = f_of(raw[k][p].z); w[4 * p + 3] = f_of(raw[k][p].w);
            }
        }
    };
    // one binary64 term per block of the lane: the adjacent-pair tree over the lane's blocks of a packet in
    // registers, over the packet with the wave tree, over the packets; the wave sum goes to its place in block order
    auto wave_sum_to_lds = [&](int which, const double term[R]) {
        double v[kPackets];
#pragma unroll
        for (int pk = 0; pk < kPackets; ++pk) {
            const double *x = term + pk * kX;
            double f;
            if constexpr (kX == 1) f = x[0];
            else if constexpr (kX == 2) f = x[0] + x[1];
            else f = (x[0] + x[1]) + (x[2] + x[3]);
            v[pk] = wave_pair_tree(f);
        }
        if (lane == 0) s_part[which][wave] = kPackets == 1 ? v[0] : v[0] + v[kPackets - 1];
    };
    // wave 0, after a barrier: the sum over the workgroup's blocks
    auto workgroup_sum = [&](int which) -> double {
        return wave_pair_tree(lane < (uint32_t)kParts ? s_part[which][lane] : 0.0);
    };

    // ---- Eq. 1-2 state and Eq. 5
    float alpha1 = alpha0;
    float rho[R];
#pragma unroll
    for (int k = 0; k < R; ++k) rho[k] = 0.0f;
    if constexpr (METHOD == SOAR_METHOD_SOAR) {
        if (!degenerate) {                                   // uniform over the grid
            double tN[R], tM[R];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                tN[k] = tM[k] = 0.0;
                if (blk(k) < t.nblk) {
                    float w[16];
                    uint32_t nib[2], c0;
                    float delta0, a, b;
                    widen(k, w);
                    block_init(w, gs, c0, delta0, nib);
                    code_sums(w, nib, a, b);
                    rho[k] = block_ratio(a, b, delta0, gs.fast);
                    tN[k] = (double)a * (double)delta0;
                    tM[k] = ((double)b * (double)delta0) * (double)delta0;
                }
            }
            wave_sum_to_lds(0, tN);
            wave_sum_to_lds(1, tM);
            __syncthreads();
            if (wave == 0) {
                double NM[2] = {workgroup_sum(0), workgroup_sum(1)};
                bool ok = true;
                if (grid.G > 1u) {
                    ok = cross_sums<2>(grid, words.nm, s_cross, NM);
                    if (!ok && lane == 0) give_up();
                }
                if (lane == 0) {
                    s_alpha1 = (NM[1] > 0.0) ? (float)(NM[0] / NM[1]) : alpha0;
                    s_gone = ok ? 0u : 1u;
                }
            }
            __syncthreads();
            if (s_gone) return false;
            alpha1 = s_alpha1;
        } else {
            if constexpr (BATCH) {
                // nobody may finish here while others have given up: a crossing (of no sums) tells
                if (wave == 0) {
                    double none[2] = {0.0, 0.0};
                    bool ok = true;
                    if (grid.G > 1u) {
                        ok = cross_sums<2>(grid, words.nm, s_cross, none);
                        if (!ok && lane == 0) give_up();
                    }
                    if (lane == 0) s_gone = ok ? 0u : 1u;
                }
                __syncthreads();
                if (s_gone) return false;
            }
            if (allzero) alpha1 = 1.0f;
        }
        if ((BATCH ? batch_g : blockIdx.x) == 0u && tid == 0) *t.gscale = alpha1;
    }
    const float inv_alpha1 = 1.0f / alpha1;
    const bool fast = gs.fast && near_one(alpha1);
    const bool full_search = args.full_search != 0;

    // ---- Eq. 6, new assignment, Eq. 8 search (k_search, per block); the lane's bytes leave together
    double terr[R];
    uint32_t nibs[R][2], codes4 = 0u;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        terr[k] = 0.0;
        nibs[k][0] = nibs[k][1] = 0u;
        if (blk(k) < t.nblk) {
            float w[16], q[16];
            uint32_t out_code;
            float out_err;
            widen(k, w);
            if (allzero) {
                float x[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) x[j] = w[j];
                nibs[k][0] = fp4x8(x);
                nibs[k][1] = fp4x8(x + 8);
                out_code = kE4M3Min;
                out_err = 0.0f;
            } else if constexpr (METHOD == SOAR_METHOD_RTN) {
                uint32_t c0;
                float delta0;
                block_init(w, gs, c0, delta0, nibs[k], q);
                out_code = c0;
                out_err = block_error(w, q, alpha0 * delta0);
            } else {
                const int centre = new_codes(w, rho[k], alpha1, inv_alpha1, fast, nibs[k], q);
                int best;
                float best_err;
                bool done = false;
                if (!full_search) {
                    done = search_certified(w, q, alpha1, inv_alpha1, centre, args.radius, best, best_err);
                    if (args.search_stats) count_search(args.search_stats, done);
                }
                if (!done) search_full(w, q, alpha1, centre, args.radius, best, best_err);
                out_code = (uint32_t)best;
                out_err = best_err;
            }
            codes4 |= out_code << (8 * k);
            terr[k] = (double)out_err;
        }
    }
#pragma unroll
    for (int pk = 0; pk < kPackets; ++pk) {
        // streaming stores (the outputs are not read again here).  A packet with all its kX blocks present and
        // the output addresses aligned for it: the 8 kX code bytes in 16-byte pieces, the kX scale bytes in one piece.
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const uint32_t b0 = blk(pk * kX);
        const bool whole = b0 + (uint32_t)kX <= t.nblk;
        uint8_t *cp = t.codes + (size_t)b0 * 8;
        uint8_t *sp = t.scales + b0;
        const uint32_t (*nb)[2] = nibs + pk * kX;
        const uint32_t sc = codes4 >> (8 * pk * kX);
        if (kX >= 2 && whole && (reinterpret_cast<uintptr_t>(t.codes) & 15u) == 0u) {
#pragma unroll
            for (int k = 0; k < kX; k += 2)
                __builtin_nontemporal_store(u32x4{nb[k][0], nb[k][1], nb[k + (kX >= 2 ? 1 : 0)][0], nb[k + (kX >= 2 ? 1 : 0)][1]},
                                            reinterpret_cast<u32x4 *>(cp) + k / 2);
        } else {
#pragma unroll
            for (int k = 0; k < kX; ++k)
                if (b0 + (uint32_t)k < t.nblk)
                    __builtin_nontemporal_store(u32x2{nb[k][0], nb[k][1]}, reinterpret_cast<u32x2 *>(cp) + k);
        }
        if (kX == 4 && whole && (reinterpret_cast<uintptr_t>(t.scales) & 3u) == 0u) {
            __builtin_nontemporal_store(sc, reinterpret_cast<uint32_t *>(sp));
        } else if (kX == 2 && whole && (reinterpret_cast<uintptr_t>(t.scales) & 1u) == 0u) {
            __builtin_nontemporal_store((uint16_t)sc, reinterpret_cast<uint16_t *>(sp));
        } else {
#pragma unroll
            for (int k = 0; k < kX; ++k)
                if (b0 + (uint32_t)k < t.nblk) __builtin_nontemporal_store((uint8_t)(sc >> (8 * k)), sp + k);
        }
    }
    wave_sum_to_lds(2, terr);
    __syncthreads();
    if (wave != 0) return true;
    // ---- error sum and status: workgroup 0 collects
    double total = workgroup_sum(2);
    bool ok = true;
    if (grid.G > 1u) {
        if (t.sse) publish_sum(grid, words.err, total);
        if (grid.g != 0u) return true;
        if (t.sse) ok = collect_sum(grid, words.err, total);
    }
    if (lane == 0) {
        if (!BATCH && !ok) {
            give_up();
            return true;
        }
        if (t.sse) *t.sse = total;
        if (t.status) *t.status = (amax_bits >= 0x7F800000u ? SOAR_STATUS_NONFINITE : 0) | (allzero ? SOAR_STATUS_ALLZERO : 0);
        if (METHOD == SOAR_METHOD_RTN) *t.gscale = allzero ? 1.0f : alpha0;
    }
    return true;
}

template <int DT, int METHOD, int L, int R>
__global__ __launch_bounds__(L) void k_resident(const Task t, const ResidentArgs args)
{
    resident_body<DT, METHOD, L, R, false>(t, args);
}

// ------------------------------------------------------------------ one launch, a batch of small tensors
// A call with a few small tensors pays four launches that keep a fraction of the GPU busy; together they fit the registers of
// the GPU as one tensor does.  k_resident_batch gives every tensor its workgroups (all of one shape, at most one per compute unit
// in all), its own crossing words and its own token; tensors do not wait for one another.  The call always finishes, as it does
// with several launches, at the speed of the compute units that it gets: where the workgroups of a tensor do not arrive together within the
// bound, those that run do it together, share by share (finish_together); the tensors after it then do not wait.  On a stream of 64 compute units,
// 15 million weights in five tensors: 0.50 ms a call, several launches 0.09 (waiting 2 s a tensor, which its last workgroup then did alone: 4.0 s).
// Whole calls, several launches / one: a layer of hidden 256 (seven matrices) 21.8 / 9.4 us, four of them 70 / 11, four of hidden 512 in fp32 105 / 22.7,
// one of hidden 1024 34 / 20.6, of 1120 (99 % of the places) 38.5 / 20.5.
constexpr int kResidentTensors = 40;
constexpr int kWordsPerSlot = 5;          // tensors whose crossing words lie side by side in the partial sums of one slot
// What the workgroups of one tensor share once they have given up: of every share, the last phase for which it has been taken and the last one in which
// it has been carried out (phase_token), and what it gives.
struct TogetherWords {
    uint64_t taken[kResMaxWG], done[kResMaxWG];
    uint64_t max[kResMaxWG], sums[3][kResMaxWG];
};
struct BatchWords {
    ResidentWords cross;
    TogetherWords together;
    uint64_t crowded;                     // the first tensor's serves all: the token once the workgroups of some tensor have not come together
};
static_assert(kWordsPerSlot * sizeof(BatchWords) <= kPartialsBytes && kResidentTensors <= kWordsPerSlot * kGroupMax && kResidentTensors <= 64,
              "layout of the crossing words");

struct ResidentTensor {
    const void *w;
    uint8_t  *codes, *scales;
    float    *gscale;
    double   *sse;
    int32_t  *status;
    int64_t  ld;
    uint32_t bpr, nblk, wg_begin, n_wg;
};
struct ResidentBatch {
    ResidentTensor t[kResidentTensors];
    char    *slots;                       // the workspace
    uint32_t n;
    uint32_t tell;                        // status bit of a call that gave up and was finished all the same
    ResidentArgs r;
};
static_assert(sizeof(ResidentBatch) <= 4096, "kernel arguments");

// The single-step path of one tensor by those of its workgroups that are on the GPU, all of which have given up: the same trees, the
// same bytes.  Each of the three phases -- maximum, sums, search -- has the G shares that the workgroups would have had; a workgroup takes its own
// first and then others that nobody has taken, carries them out without waiting for anybody, and waits only when none is left, for the ones that
// hold them: they run.  One that comes late finds what is left, or nothing.  Every share has words of its own: with counters that hand them
// out and count them back the call measured below took 0.77 ms.
__device__ __forceinline__ uint64_t phase_token(uint64_t token, uint32_t phase) { return token + (phase + 1u) * kResOdd; }

template <int DT, int L, int R>
__device__ __forceinline__ void finish_together(const Task &t, const ResidentArgs &args, TogetherWords &words, uint32_t g, uint32_t G, uint32_t tell)
{
    constexpr int kWaves = L / 64;
    __shared__ double s_part[2][kWaves], s_sums[2];
    __shared__ uint32_t s_max[kWaves], s_share;
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));         // nothing computed from it is carried here in registers from before
    const uint32_t lane = tid & 63u, wave = tid >> 6;
    const uint64_t token = args.nonce;
    auto load = [&](uint32_t i, float w[16]) { load_block<DT>(t.w, block_offset(t, i), w); };
    auto put = [&](uint64_t *p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto get = [&](const uint64_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // a word of taken or done: this phase's, or a later one's
    auto reached = [&](uint64_t seen, uint32_t phase) -> bool {
        bool yes = false;
        for (uint32_t p = phase; p < 3u; ++p) yes = yes || seen == phase_token(token, p);
        return yes;
    };
    // every lane: a share of this phase that has now been taken for this workgroup, G where none is left
    auto next = [&](uint32_t phase) -> uint32_t {
        __syncthreads();
        if (wave == 0) {
            uint32_t share = G;
            bool mine = false;
            for (uint32_t first = 0; first < G && !mine;) {          // 64 shares at a time, the own one first
                const uint32_t at = first + lane < G ? (g + first + lane) % G : G;
                uint64_t seen = at < G ? get(words.taken + at) : 0ull;
                const uint64_t left = __builtin_amdgcn_ballot_w64(at < G && !reached(seen, phase));
                if (left == 0ull) {
                    first += 64u;
                    continue;
                }
                // (where another workgroup was faster, look again: that share is no longer left)
                const bool chosen = lane == (uint32_t)__builtin_ctzll(left);
                bool won = false;
                if (chosen)
                    won = __hip_atomic_compare_exchange_strong(words.taken + at, &seen, phase_token(token, phase), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                mine = __builtin_amdgcn_ballot_w64(won) != 0ull;
                share = (uint32_t)__builtin_amdgcn_readlane((int)at, __builtin_ctzll(left));
            }
            if (lane == 0) s_share = mine ? share : G;
        }
        __syncthreads();
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)s_share);
    };
    // one lane, whose stores of the share's results come before
    auto carried_out = [&](uint32_t phase, uint32_t share) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        put(words.done + share, phase_token(token, phase));
    };
    // wave 0: have all shares of a phase been carried out?
    auto complete = [&](uint32_t phase) -> bool {
        bool yes = true;
        for (uint32_t k = lane; k < G; k += 64u) yes = yes && reached(get(words.done + k), phase);
        return __builtin_amdgcn_ballot_w64(!yes) == 0ull;
    };
    auto all_done = [&](uint32_t phase) {
        if (wave == 0)
            while (!complete(phase)) __builtin_amdgcn_s_sleep(32);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    };
    // tile k of a share of two sums, in workgroup order; s_sums holds them after the last one, for lane 0
    auto add_tile = [&](uint32_t k, double x, double y) {
        x = wave_pair_tree(x);
        y = wave_pair_tree(y);
        __syncthreads();
        if (lane == 0) { s_part[0][wave] = x; s_part[1][wave] = y; }
        __syncthreads();
        if (wave == 0) {
            __shared__ double s_stack[2][3];
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                double v = wave_pair_tree(lane < (uint32_t)kWaves ? s_part[n][lane] : 0.0);
                if (lane == 0) {
                    uint32_t lvl = 0;
                    while ((k >> lvl) & 1u) { v = s_stack[n][lvl] + v; ++lvl; }
                    s_stack[n][lvl] = s_sums[n] = v;
                }
            }
        }
    };
    // wave 0: the tree over the shares
    auto sum_of = [&](const uint64_t *part) -> double {
        double v[kResMaxWG / 64];
#pragma unroll
        for (int k = 0; k < kResMaxWG / 64; ++k)
            v[k] = wave_pair_tree(lane + 64u * k < G ? __longlong_as_double((long long)get(part + lane + 64u * k)) : 0.0);
        static_assert(kResMaxWG == 256, "the tree over the groups of 64 is written out");
        return (v[0] + v[1]) + (v[2] + v[3]);
    };

    for (uint32_t share; (share = next(0u)) < G;) {
        uint32_t m = 0;
#pragma unroll 1
        for (uint32_t k = 0; k < (uint32_t)R; ++k) {
            const uint32_t i = (share * R + k) * (uint32_t)L + tid;
            if (i < t.nblk) {
                float w[16];
                load(i, w);
#pragma unroll
                for (int j = 0; j < 16; ++j) m = max(m, __float_as_uint(w[j]) & 0x7FFFFFFFu);
            }
        }
        m = wave_max_u32(m);
        if (lane == 0) s_max[wave] = m;
        __syncthreads();
        m = wave_max_u32(lane < (uint32_t)kWaves ? s_max[lane] : 0u);
        if (tid == 0) {
            put(words.max + share, m);
            carried_out(0u, share);
        }
    }
    all_done(0u);
    uint32_t amax_bits = 0;
    for (uint32_t k = lane; k < G; k += 64u) amax_bits = max(amax_bits, (uint32_t)get(words.max + k));
    amax_bits = wave_max_u32(amax_bits);
    const bool allzero = amax_bits == 0u, degenerate = allzero || amax_bits >= 0x7F800000u;
    const GlobalScale gs(amax_bits);
    auto ratio = [&](const float w[16], float &a, float &b, float &delta0) {
        uint32_t nib[2], c0;
        block_init(w, gs, c0, delta0, nib);
        code_sums(w, nib, a, b);
        return block_ratio(a, b, delta0, gs.fast);
    };
    float alpha1 = allzero ? 1.0f : gs.alpha0;
    if (!degenerate) {
        for (uint32_t share; (share = next(1u)) < G;) {
#pragma unroll 1
            for (uint32_t k = 0; k < (uint32_t)R; ++k) {
                const uint32_t i = (share * R + k) * (uint32_t)L + tid;
                float a = 0.0f, b = 0.0f, delta0 = 0.0f;
                if (i < t.nblk) {
                    float w[16];
                    load(i, w);
                    ratio(w, a, b, delta0);
                }
                add_tile(k, (double)a * (double)delta0, ((double)b * (double)delta0) * (double)delta0);
            }
            if (tid == 0) {
                for (int n = 0; n < 2; ++n) put(words.sums[n] + share, (uint64_t)__double_as_longlong(s_sums[n]));
                carried_out(1u, share);
            }
        }
        all_done(1u);
        if (wave == 0) {
            const double N = sum_of(words.sums[0]), M = sum_of(words.sums[1]);
            if (lane == 0) { s_sums[0] = N; s_sums[1] = M; }
        }
        __syncthreads();
        if (s_sums[1] > 0.0) alpha1 = (float)(s_sums[0] / s_sums[1]);
    }
    const float inv_alpha1 = 1.0f / alpha1;
    const bool fast = gs.fast && near_one(alpha1);
    for (uint32_t share; (share = next(2u)) < G;) {
#pragma unroll 1
        for (uint32_t k = 0; k < (uint32_t)R; ++k) {
            const uint32_t i = (share * R + k) * (uint32_t)L + tid;
            float err = 0.0f;
            if (i < t.nblk) {
                float w[16], q[16];
                uint32_t nib[2];
                int best = (int)kE4M3Min;
                load(i, w);
                if (allzero) {
                    nib[0] = fp4x8(w);
                    nib[1] = fp4x8(w + 8);
                } else {
                    float a, b, delta0;
                    const int centre = new_codes(w, degenerate ? 0.0f : ratio(w, a, b, delta0), alpha1, inv_alpha1, fast, nib, q);
                    if (args.full_search || !search_certified(w, q, alpha1, inv_alpha1, centre, args.radius, best, err))
                        search_full(w, q, alpha1, centre, args.radius, best, err);
                }
                __builtin_nontemporal_store((uint64_t)nib[1] << 32 | nib[0], reinterpret_cast<uint64_t *>(t.codes) + i);
                __builtin_nontemporal_store((uint8_t)best, t.scales + i);
            }
            add_tile(k, (double)err, 0.0);
        }
        if (tid == 0) {
            put(words.sums[2] + share, (uint64_t)__double_as_longlong(s_sums[0]));
            carried_out(2u, share);
        }
    }
    // the workgroup whose share was the last finds all of them carried out; others that do write the same
    wait_then_read();
    if (wave == 0 && complete(2u)) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const double total = sum_of(words.sums[2]);
        if (lane == 0) {
            *t.gscale = alpha1;
            if (t.sse) *t.sse = total;
            if (t.status) *t.status = (int32_t)tell | (amax_bits >= 0x7F800000u ? SOAR_STATUS_NONFINITE : 0) | (allzero ? SOAR_STATUS_ALLZERO : 0);
        }
    }
}

template <int DT, int L, int R>
__global__ __launch_bounds__(L) void k_resident_batch(const ResidentBatch batch)
{
    const uint32_t lane = threadIdx.x & 63u;
    // which tensor: the last one that begins at or before this workgroup
    const uint32_t begin = lane < batch.n ? batch.t[lane].wg_begin : 0xFFFFFFFFu;
    const uint32_t which = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(begin <= blockIdx.x)) - 1u;
    const ResidentTensor &x = batch.t[which];
    auto words_of = [&](uint32_t k) -> BatchWords & {
        return reinterpret_cast<BatchWords *>(batch.slots + (size_t)(k / kWordsPerSlot) * kSlotBytes + kZeroedBytes)[k % kWordsPerSlot];
    };
    BatchWords &words = words_of(which), &first = words_of(0);
    Task t;
    t.w = x.w;
    t.codes = x.codes;
    t.scales = x.scales;
    t.gscale = x.gscale;
    t.sse = x.sse;
    t.status = x.status;
    t.ld = x.ld;
    t.bpr = x.bpr;
    t.nblk = x.nblk;
    t.contiguous = x.ld == (int64_t)x.bpr * 16 ? 1u : 0u;
    t.ctrl = nullptr;
    const bool finished = resident_body<DT, SOAR_METHOD_SOAR, L, R, true>(t, batch.r, &words.cross, blockIdx.x - x.wg_begin, x.n_wg,
                                                                                    &first.crowded);
    // Given up, here or elsewhere, before any output was written.  One value for the workgroup, and nothing that is carried past this
    // point: otherwise the code below comes to lie between a lane's blocks and their search and takes registers of theirs to scratch memory.
    if (__builtin_amdgcn_readfirstlane(finished ? 0 : 1) != 0) finish_together<DT, L, R>(t, batch.r, words.together, blockIdx.x - x.wg_begin, x.n_wg, batch.tell);
}

}  // namespace
