// The last step of a launch that finishes a tensor-wide sum without counters: small one-pass conversions (plain NVFP4
// with a supplied maximum, MXFP4) handed over alone need no launch that clears control words first.
#pragma once
#include "soar_single_step.hpp"      // tokens, crossing words

namespace {

constexpr uint32_t kOnceMaxWG = 256;
constexpr uint32_t kOnceWords = 40960;               // place inside the slot's partial sums: 3 kinds of kOnceMaxWG words
static_assert(kOnceWords + 3 * kOnceMaxWG <= 3 * kMaxPartials, "layout of the words");

// What a launch needs to know: the token is nonce ^ epoch * odd as in k_resident.  The nonce is new for every call, and
// captured calls do not come here, so no token is used twice.
struct OnceArgs {
    uint64_t nonce;
};

// Wave 0, all lanes, of every workgroup (g of G <= kOnceMaxWG): publish this workgroup's sum and flag with the launch's
// token, wait until that has been performed, read everybody's words ONCE, and report whether all were there; then `v` is
// the adjacent-pair tree over the workgroups and `flag` the union.  Nobody waits for anybody: of two workgroups the one
// whose publication completes later reads both, so at least one sees all G -- several may, with the same result, and
// then write the same values.
__device__ __forceinline__ bool once_sum(uint64_t *words, uint64_t *epoch_p, uint64_t epoch, uint64_t nonce, uint32_t g, uint32_t G,
                                         double &v, bool &flag)
{
    constexpr int P = kResSumBits, K = kOnceMaxWG / 64;
    const uint32_t lane = threadIdx.x & 63u;
    if (G == 1u) return true;
    const uint64_t tok = nonce ^ (epoch * kResOdd), want = (tok << P) >> P;
    uint64_t mine[3];
    resident_split(v, mine);
    mine[2] |= (uint64_t)(flag ? 1u : 0u) << (P - 1);                    // 20 bits of the sum in this word
    const uint64_t x = lane == 0u ? mine[0] : lane == 1u ? mine[1] : mine[2];
    if (lane < 3u)
        __hip_atomic_store(words + lane * kOnceMaxWG + g, (tok << P) | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_then_read();
    uint64_t w[K][3];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int n = 0; n < 3; ++n)
            w[k][n] = lane + 64u * k < G ? __hip_atomic_load(words + n * kOnceMaxWG + lane + 64u * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                         : want << P;
    __builtin_amdgcn_sched_barrier(0);
    bool missing = false, any = false;
    double s[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        uint64_t pay[3];
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            missing = missing | ((w[k][n] >> P) != want);
            pay[n] = w[k][n] & ((1ull << P) - 1ull);
        }
        any = any | ((pay[2] >> (P - 1)) != 0ull);
        pay[2] &= (1ull << (P - 1)) - 1ull;
        s[k] = resident_join(pay);
    }
    if (__builtin_amdgcn_ballot_w64(missing) != 0ull) return false;
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = wave_pair_tree(s[k]);
    static_assert(K == 4, "the tree over the groups of 64 is written out");
    v = (s[0] + s[1]) + (s[2] + s[3]);
    flag = __builtin_amdgcn_ballot_w64(any) != 0ull;
    if (lane == 0) __hip_atomic_store(epoch_p, epoch + 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Plain NVFP4 of one tensor with its maximum supplied (k_search<., RTN> otherwise), one launch instead of two: bound by
// the latency of a launch, a trip to memory for the weights and two for the sum (16 x 4096 bf16: 8.2 -> 4.6 us).
template <int DT>
__global__ __launch_bounds__(kWG) void k_rtn_once(const Task t, const OnceArgs args)
{
    constexpr int kP = pieces_per_block<DT, 16>();
    __shared__ u32x4 s_x[kWG * kP];                    // load_wave_blocks: one region per wave
    __shared__ double s_wave[4];
    const uint32_t tid = threadIdx.x, g = blockIdx.x, G = gridDim.x;
    uint64_t epoch = 0;
    if (G > 1u) epoch = __hip_atomic_load(&t.ctrl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const float given = *t.amax_in;
    const bool bad_amax = !(given > 0.0f) || __float_as_uint(given) >= 0x7F800000u;
    const GlobalScale gs(bad_amax ? 0x7FC00000u : __float_as_uint(given), false);
    double sse = 0.0;
    for (uint32_t k = 0; k < t.tiles_per_wg; ++k) {
        const uint32_t i = (g * t.tiles_per_wg + k) * kWG + tid, wave_first = i - (tid & 63u);
        if (wave_first >= t.nblk) break;
        float w[16], q[16];
        if (t.contiguous) load_wave_blocks<DT, 16, true>(t.w, wave_first, t.nblk, s_x + (tid >> 6) * (64 * kP), w);
        if (i >= t.nblk) break;
        if (!t.contiguous) load_block<DT, true>(t.w, block_offset(t, i), w);
        uint32_t c0, nib[2];
        float delta0;
        block_init(w, gs, c0, delta0, nib, q);
        sse += (double)block_error(w, q, gs.alpha0 * delta0);
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 packed = {nib[0], nib[1]};
        __builtin_nontemporal_store(packed, reinterpret_cast<u32x2 *>(t.codes) + i);
        __builtin_nontemporal_store((uint8_t)c0, t.scales + i);
    }
    sse = wave_pair_tree(sse);
    if ((tid & 63u) == 0u) s_wave[tid >> 6] = sse;
    __syncthreads();
    if (tid >= 64u) return;
    double total = (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
    bool flag = false;
    // whoever has seen all G words: by then every workgroup has read the supplied maximum, so a caller may have the global
    // scale (or the sum, or the status) written where the maximum lies, as on the path with counters
    if (once_sum(reinterpret_cast<uint64_t *>(t.part) + kOnceWords, &t.ctrl->epoch, epoch, args.nonce, g, G, total, flag) && tid == 0) {
        *t.gscale = gs.alpha0;
        if (t.sse) *t.sse = total;
        if (t.status) *t.status = bad_amax ? SOAR_STATUS_BAD_AMAX : 0;
    }
}

}  // namespace
