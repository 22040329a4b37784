// The iterated path of one tensor handed over alone, in one launch: k_iter_resident.
#pragma once
#include "soar_iterated.hpp"
#include "soar_single_step.hpp"      // ResidentArgs

namespace {

// A tensor handed over alone pays, on the launch-per-iteration path, 18 dependent launches for the paper's 15
// iterations, 12 of them idle after the usual stop at the third; below some ten million weights they, and not the
// search, are what a call takes.  k_iter_resident does the whole path -- Eq. 1 maximum, Eq. 1-2 state, the iterations
// until the stop -- in ONE launch of at most one workgroup per compute unit.  Workgroup g owns the R * L consecutive
// blocks from g * R * L on, as R tiles of one block per lane (R a power of two, so its sums are nodes of the
// adjacent-pair tree); it re-reads them in every iteration, from the L2 or the last-level cache, and keeps its
// blocks' ratios in the workspace, where only the lane that wrote one reads it.  The tensor-wide sums cross the grid
// as in k_resident (tokens, no counters, bounded waits), three binary64 values a crossing; every workgroup forms the
// next global scale and the stop decision for itself from the same bits.
// Words of consecutive crossings alternate between two buffers: a workgroup publishes crossing c + 2 only after it has
// gathered c + 1, for which every workgroup had published, and had therefore gathered c.  Each crossing has a token of
// its own; the complement of the launch's token says at any of them that its writer has given up.  The launch's token
// is the call's nonce alone, without the epoch: calls being captured do not come here, and a workgroup that starts after
// others have given up has to recognise their words.
// The one wait that may not end is the first: the GPU may hold the rest of the grid back, behind another process's or
// stream's kernels or a mask of compute units.  It is bounded by wait_ticks, from where the workgroup has read its blocks and
// begins to wait.  A workgroup whose time is up tells the others, which then leave as well, at the first crossing or -- those
// that found the first complete -- at the second; whoever leaves counts itself out, and the last to do so does the whole
// tensor alone: all blocks are then its own R * G tiles (G rounded up to a power of two), the same tree, no crossings.  So a
// call always finishes, as it does with a launch per iteration.  Beyond the first crossing every workgroup is running and the
// waits last as long as the slowest one's share; their bound (later_ticks) is there for a machine that has stopped working.
// 1024 x 4096 bf16, paper settings: 72-88 -> 41 us a call (loads 2, maximum 4, state 3, sums 4, an iteration 5-6 and
// its crossing 4 us); 4096 x 4096 fp32, search-only arm: 169 -> 135 us, 32 of them an iteration's search.
// The crossing words inside Task::part (where other kernels' words may lie: theirs carry other tokens)
struct IterResidentWords {
    uint64_t max[kMaxEnd];
    SumWords<3> sums[2];                  // of alternating crossings
    uint64_t left;                        // how many workgroups have given up
};
static_assert(sizeof(IterResidentWords) <= kPartialsBytes, "layout of the crossing words");

// One lane of a workgroup that gives up: the number of workgroups that have, this one included.  The word may hold
// anything before the launch's first: the count stands beside 48 bits of the token.  An exchange fails only where
// another workgroup's has succeeded, so the loop ends.
__device__ __forceinline__ uint32_t count_out(uint64_t *word, uint64_t token)
{
    uint64_t seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), next;
    do next = token << 16 | ((seen >> 16 == (token << 16) >> 16 ? seen & 0xFFFFull : 0ull) + 1ull);
    while (!__hip_atomic_compare_exchange_strong(word, &seen, next, __ATOMIC_ACQ_REL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return (uint32_t)(next & 0xFFFFull);
}

constexpr int kIterResMaxBeta = 2048;     // factor table in LDS
constexpr int kIterResMaxTiles = 16;      // R

struct IterResidentArgs {
    ResidentArgs r;
    int32_t  iters, n_beta, bracket, arm;
    float    beta_lo, beta_hi, index_per_beta, early_stop_rel;
    uint32_t tiles;                       // R
    uint32_t tell;                        // status of a call that gave up and was finished all the same
    uint64_t later_ticks;                 // bound of every wait after the first crossing
};

// CLOSED_FORM: the arm without a search; otherwise the nearest-factor search (the host sends the others elsewhere)
template <int DT, int L, bool CLOSED_FORM>
__global__ __launch_bounds__(L) void k_iter_resident(const Task t, const IterResidentArgs args)
{
    static_assert(L == 256 || L == 1024, "workgroup of 4 or 16 waves");
    constexpr int kWaves = L / 64;
    constexpr int kP = pieces_per_block<DT, 16>();
    constexpr int kMaxBits = DT == SOAR_BF16 ? 15 : 31;
    __shared__ float4 s_blocks[kStage * L];
    __shared__ double s_wave[3][kWaves];
    __shared__ double s_stack[3][32];
    __shared__ float s_beta[CLOSED_FORM ? 1 : kIterResMaxBeta];
    __shared__ uint64_t s_cross[kSumDirect * SumWords<3>::kW];
    __shared__ uint32_t s_max[kWaves];
    __shared__ uint32_t s_amax, s_gone, s_stop;
    __shared__ float s_alpha;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const bool keep_scale = args.arm == SOAR_METHOD_DSS_ONLY;

    ResidentGrid grid;
    grid.g = blockIdx.x;
    grid.G = gridDim.x;
    grid.tok = grid.base = args.r.nonce;
    grid.t0 = 0;
    grid.ticks = args.r.wait_ticks;
    IterResidentWords &words = *reinterpret_cast<IterResidentWords *>(t.part);
    grid.words = words.max;
    uint32_t R = args.tiles, told = 0u;
    // one lane: leave the launch and tell the others, at whichever crossing they are
    auto give_up = [&]() {
        leave_max(grid, ~grid.base << kMaxBits);
        for (uint32_t b = 0; b < 2; ++b) leave_sums(grid, words.sums[b], ~grid.base << kResSumBits);
        if (t.status) *t.status = SOAR_STATUS_GAVE_UP;
        if (t.iters_run) *t.iters_run = 0;
    };
    // every lane of a workgroup that has given up: true in the last one to leave, which finds itself the only workgroup
    // of a launch over the whole tensor, with everybody's stores performed before its own
    auto last_to_leave = [&]() -> bool {
        __threadfence();
        __syncthreads();
        if (tid == 0) s_stop = count_out(&words.left, grid.base) == grid.G ? 1u : 0u;
        __syncthreads();
        if (s_stop == 0u) return false;
        __threadfence();
        while (R < args.tiles * grid.G) R <<= 1;
        grid.g = 0u;
        grid.G = 1u;
        told = args.tell;
        __syncthreads();                  // s_stop is written again
        return true;
    };
    // wave 0, every workgroup: the sums of crossing c over the grid
    auto cross = [&](uint32_t c, double v[3]) -> bool {
        if (grid.G == 1u) return true;
        grid.tok = grid.base ^ ((uint64_t)(c + 1u) * 0xBF58476D1CE4E5B9ull);
        grid.t0 = (uint64_t)wall_clock64();
        grid.ticks = args.later_ticks;
        return cross_sums<3>(grid, words.sums[c & 1u], s_cross, v);
    };

    if constexpr (!CLOSED_FORM)
        for (int k = (int)tid; k < args.n_beta; k += L) s_beta[k] = beta_factor(k, args.n_beta, args.beta_lo, args.beta_hi);

    for (;;) {       // once; a second time in the workgroup that finishes for a grid that has given up
        const uint32_t first = grid.g * R * (uint32_t)L + tid;   // this lane's block of tile 0
        // ---- Eq. 1 maximum
        uint32_t m = 0;
#pragma unroll 4
        for (uint32_t k = 0; k < R; ++k) {
            const uint32_t i = first + k * (uint32_t)L;
            if (i >= t.nblk) break;
            const char *p = static_cast<const char *>(t.w) + block_offset(t, i) * (DT == SOAR_BF16 ? 2 : 4);
#pragma unroll
            for (int c = 0; c < kP; ++c) {
                const u32x4 v = load16<false>(p + 16 * c);
                m = absmax_accumulate<DT>(m, make_uint4(v.x, v.y, v.z, v.w));
            }
        }
        if constexpr (DT == SOAR_BF16) m = max(m & 0xFFFFu, m >> 16) << 16;
        m = wave_max_u32(m);
        if (lane == 0) s_max[wave] = m;
        __syncthreads();
        if (wave == 0) {
            uint32_t amax = wave_max_u32(lane < (uint32_t)kWaves ? s_max[lane] : 0u);
            bool ok = true;
            if (grid.G > 1u) {
                uint32_t value = DT == SOAR_BF16 ? amax >> 16 : amax;
                grid.t0 = (uint64_t)wall_clock64();
                ok = cross_max<kMaxBits>(grid, value);
                amax = DT == SOAR_BF16 ? value << 16 : value;
                if (lane == 0 && !ok) give_up();
            }
            if (lane == 0) { s_amax = amax; s_gone = ok ? 0u : 1u; }
        }
        __syncthreads();
        if (s_gone) {
            if (last_to_leave()) continue;
            return;
        }
        const uint32_t amax_bits = s_amax;
        const bool allzero = amax_bits == 0u, nonfinite = amax_bits >= 0x7F800000u;
        if (allzero || nonfinite) {                              // uniform over the grid
            // nobody may finish here while others have given up: a crossing (of no sums) tells
            if (wave == 0) {
                double v[3] = {0.0, 0.0, 0.0};
                const bool ok = cross(0u, v);
                if (lane == 0) {
                    if (!ok) give_up();
                    s_gone = ok ? 0u : 1u;
                }
            }
            __syncthreads();
            if (s_gone) {
                if (last_to_leave()) continue;
                return;
            }
            if (allzero) {
                for (uint32_t k = 0; k < R; ++k) {
                    const uint32_t i = first + k * (uint32_t)L;
                    if (i >= t.nblk) break;
                    float w[16];
                    BlockState x;
                    load_block<DT>(t.w, block_offset(t, i), w);
                    zero_block(w, x);
                    store_block(t, i, x);
                }
            }
            if (grid.g == 0u && tid == 0) {
                *t.gscale = allzero ? 1.0f : __builtin_nanf("");
                if (t.sse) *t.sse = allzero ? 0.0 : __builtin_nan("");
                if (t.status) *t.status = (allzero ? SOAR_STATUS_ALLZERO : SOAR_STATUS_NONFINITE) | (int32_t)told;
                if (t.iters_run) *t.iters_run = 0;
            }
            return;
        }

        // ---- Eq. 1-2 state; the scale of iteration 0 (Eq. 5, unless the closed-form stage is left out)
        const GlobalScale gs(amax_bits);
        const float alpha0 = gs.alpha0;
        const uint32_t T = R < (uint32_t)kStage ? R : (uint32_t)kStage;
        double prev = 0.0;                                       // wave 0: the error before the iteration now running
        {
            StagedTree<L> tree{s_blocks, s_wave, s_stack};
            for (uint32_t kg = 0; kg < R; kg += T) {
                for (uint32_t kk = 0; kk < T; ++kk) {
                    const uint32_t i = first + (kg + kk) * (uint32_t)L;
                    float a = 0.0f, b = 0.0f, delta0 = 0.0f, err = 0.0f;
                    if (i < t.nblk) {
                        float w[16], rho;
                        load_block<DT>(t.w, block_offset(t, i), w);
                        init_block(w, gs, keep_scale, a, b, delta0, err, rho);
                        t.rho[i] = rho;
                    }
                    tree.stage(kk, a, b, delta0, err);
                }
                tree.close(kg / T, T);
            }
            if (wave == 0) {
                double v[3] = {tree.wg[0], tree.wg[1], tree.wg[2]};          // lane 0's
                const bool ok = cross(0u, v);
                if (lane == 0) {
                    if (!ok) give_up();
                    s_gone = ok ? 0u : 1u;
                    s_alpha = (v[1] > 0.0 && !keep_scale) ? (float)(v[0] / v[1]) : alpha0;
                    if (ok && grid.g == 0u && t.trace) t.trace[0] = v[2];
                }
                prev = v[2];
            }
        }
        __syncthreads();
        if (s_gone) {
            if (last_to_leave()) continue;
            return;
        }

        // ---- the iterations
        JointSearch js{{s_beta, args.n_beta, args.beta_lo, args.index_per_beta}, 0.0f, 0.0f, args.r.radius, args.bracket != 0, keep_scale, false, false};
        for (uint32_t it = 0; it < (uint32_t)args.iters; ++it) {
            const float alpha = s_alpha;
            js.set_alpha(alpha, amax_bits);
            StagedTree<L> tree{s_blocks, s_wave, s_stack};
            for (uint32_t kg = 0; kg < R; kg += T) {
                for (uint32_t kk = 0; kk < T; ++kk) {
                    const uint32_t i = first + (kg + kk) * (uint32_t)L;
                    BlockState x;
                    x.a = x.b = x.d = x.err = 0.0f;
                    if (i < t.nblk) {
                        float w[16];
                        load_block<DT>(t.w, block_offset(t, i), w);
                        const float rho = t.rho[i];
                        if constexpr (CLOSED_FORM)
                            closed_form_block(w, rho, alpha, js.inv_alpha, js.in_range && all_near_one(rho), x);
                        else
                            iterate_block<true>(w, rho, js, x);
                        t.rho[i] = x.rho;
                        store_block(t, i, x);
                    }
                    tree.stage(kk, x.a, x.b, x.d, x.err);
                }
                tree.close(kg / T, T);
            }
            if (wave == 0) {
                double v[3] = {tree.wg[0], tree.wg[1], tree.wg[2]};
                const bool ok = cross(it + 1u, v);
                const double cur = v[2];
                const bool stop = args.early_stop_rel > 0.0f && (prev - cur) < (double)args.early_stop_rel * prev;
                prev = cur;
                if (lane == 0) {
                    if (!ok) give_up();
                    s_gone = ok ? 0u : 1u;
                    s_stop = stop ? 1u : 0u;
                    s_alpha = (v[1] > 0.0 && !keep_scale) ? (float)(v[0] / v[1]) : alpha;      // Eq. 5 for the next iteration
                    if (ok && grid.g == 0u) {
                        if (t.trace) t.trace[it + 1u] = cur;
                        if (stop || it + 1u == (uint32_t)args.iters) {
                            *t.gscale = alpha;
                            if (t.sse) *t.sse = cur;
                            if (t.status) *t.status = (int32_t)told;
                            if (t.iters_run) *t.iters_run = (int32_t)(it + 1u);
                        }
                    }
                }
            }
            __syncthreads();
            if (s_gone || s_stop) return;
        }
        return;
    }
}

}  // namespace
