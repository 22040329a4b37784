// How a tensor-wide result crosses the grid inside one launch: words with tokens, gathered in one trip through memory or two.
// Used by the one-launch kernels (k_resident, k_iter_resident) and, for the token and the thirds of a sum, by once_sum.
#pragma once
#include "soar_device.hpp"

namespace {

// Crossing the grid.  All workgroups of the launch must be on the machine at the same time (the host
// launches at most one per compute unit and takes the three-pass path otherwise).  A trip through memory
// from one workgroup to another takes about 1.4 us on this part, and 256 workgroups that each read all
// 256 results queue for several microseconds more, so:
//  - there is no counter and no separate "ready" flag, hence no word that has to be cleared beforehand and
//    no second trip for the value: every word a workgroup publishes (an agent-scope atomic store) carries
//    the launch's TOKEN beside its payload, and a reader accepts a word only with that token.  A binary64
//    sum travels as three words of 22 payload bits and 42 token bits; the first crossing's word holds the
//    bf16 / fp32 maximum in 15 / 31 bits beside 49 / 33 token bits.  The token is `nonce ^ epoch * odd`:
//    the nonce comes from the host (new for every call), the epoch from the workspace, advanced by the
//    launch itself once every workgroup has read it (workgroup 0, after the first crossing), so that a
//    replayed HIP graph -- same kernel arguments -- still sees a new token every time.  Memory the library
//    never wrote matches a token field with probability 2^-42 (2^-33) per word;
//  - a few workgroups read each other's words directly (one trip: up to 16 for a maximum, up to 64 for sums); above that the first
//    workgroup of every group gathers its group and publishes the group's result in copies, and everybody gathers
//    the group results (two trips, little traffic); the error sum, which only workgroup 0 needs, is gathered by
//    workgroup 0 alone in one trip.
// Every wait is BOUNDED: a workgroup whose time is up publishes the complemented token in its words (so
// that the others leave at once instead of waiting out the limit), sets SOAR_STATUS_GAVE_UP and returns;
// every wave of the grid then reaches its end.
constexpr int kResMaxWG = 256;            // workgroups of one launch, at most
constexpr uint64_t kResOdd = 0x9E3779B97F4A7C15ull;
constexpr int kResSumBits = 22;           // payload bits of a word that carries a third of a binary64 value

// what wave 0 of a workgroup needs for its crossings
struct ResidentGrid {
    uint32_t g, G;
    uint64_t tok, base, t0, ticks;        // token of the crossing and of the launch
    uint64_t *words;                      // Task::part
};

// The bound of a wait: the wall clock (100 MHz on this part), and -- should that clock ever stand still -- a
// number of polling rounds that takes several times as long (a round is at least one trip to memory).
__device__ __forceinline__ bool resident_time_is_up(const ResidentGrid &r, uint64_t round)
{
    return (uint64_t)wall_clock64() - r.t0 > r.ticks || round > 1024ull + r.ticks / 8ull;
}

__device__ __forceinline__ void resident_split(double v, uint64_t pay[3])
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    pay[0] = b & ((1ull << kResSumBits) - 1ull);
    pay[1] = (b >> kResSumBits) & ((1ull << kResSumBits) - 1ull);
    pay[2] = b >> (2 * kResSumBits);
}

__device__ __forceinline__ double resident_join(const uint64_t pay[3])
{
    return __longlong_as_double((long long)(pay[0] | pay[1] << kResSumBits | pay[2] << (2 * kResSumBits)));
}

// Wave 0, all lanes: wait until the `count` (at most 64) words from `src` on carry the token; lane l then holds the payload of
// word l (zero from `count` on).  False when somebody has given up (a word with the complemented token) or the time is up.
template <int PBITS>
__device__ __forceinline__ bool gather_max(const ResidentGrid &r, const uint64_t *src, uint32_t count, uint32_t &value)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t want = (r.tok << PBITS) >> PBITS, gone_field = (~r.base << PBITS) >> PBITS;
    for (uint64_t round = 0;; ++round) {
        const uint64_t x = lane < count ? __hip_atomic_load(src + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : want << PBITS;
        const uint64_t field = x >> PBITS;
        value = (uint32_t)(x & ((1ull << PBITS) - 1ull));
        if (__builtin_amdgcn_ballot_w64(field == gone_field) != 0ull) return false;
        if (__builtin_amdgcn_ballot_w64(field != want) == 0ull) return true;
        if (resident_time_is_up(r, round)) return false;
    }
}

// Places inside Task::part, in 8-byte words, of the maxima: one word per workgroup, then one per group of 64 in kMaxCopies copies
// kMaxStride apart: every workgroup polls the second level, and a few lines polled by 250 workgroups at once queue at their
// memory channel (the publisher's stores behind them); a reader polls the copy of its own number modulo their count.
constexpr uint32_t kMaxGroup = 64, kMaxDirect = 16, kMaxCopies = 8, kMaxStride = 544;      // 17 * 256 bytes
constexpr uint32_t kMaxLevel1 = 0, kMaxLevel2 = 512, kMaxEnd = kMaxLevel2 + kMaxCopies * kMaxStride;
static_assert(kMaxLevel1 + kResMaxWG <= kMaxLevel2 && kMaxGroup * kMaxGroup >= (uint32_t)kResMaxWG, "layout of the maxima");

// Wave 0, all lanes, every workgroup: the maximum of `value` over the grid (uniform on return).
template <int PBITS>
__device__ __forceinline__ bool cross_max(const ResidentGrid &r, uint32_t &value)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t grp = r.g / kMaxGroup, groups = (r.G + kMaxGroup - 1u) / kMaxGroup;
    uint64_t *level1 = r.words + kMaxLevel1, *level2 = r.words + kMaxLevel2;
    auto put = [&](uint64_t *p) { __hip_atomic_store(p, (r.tok << PBITS) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (lane == 0) put(level1 + r.g);
    if (r.G > kMaxDirect) {
        if (r.g % kMaxGroup == 0u) {
            if (!gather_max<PBITS>(r, level1 + grp * kMaxGroup, min(kMaxGroup, r.G - grp * kMaxGroup), value)) return false;
            value = wave_max_u32(value);
            if (lane < kMaxCopies) put(level2 + lane * kMaxStride + grp);
        }
        if (!gather_max<PBITS>(r, level2 + (r.g % kMaxCopies) * kMaxStride, groups, value)) return false;
    } else if (!gather_max<PBITS>(r, level1, r.G, value)) {
        return false;
    }
    value = wave_max_u32(value);
    return true;
}

// one lane of a workgroup that gives up: its words among the maxima
__device__ __forceinline__ void leave_max(const ResidentGrid &r, uint64_t gone)
{
    auto put = [&](uint32_t at) { __hip_atomic_store(r.words + at, gone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    put(kMaxLevel1 + r.g);
    if (r.g % kMaxGroup == 0u)
        for (uint32_t c = 0; c < kMaxCopies; ++c) put(kMaxLevel2 + c * kMaxStride + r.g / kMaxGroup);
}

// The sums of NV binary64 values.  A workgroup's words lie side by side, and a wave reads them as they lie, one word per lane: reads
// past the L2 are served line by line, and a gather by kinds of word -- nine loads of 64 words 2 KB apart -- took 3 to
// 4 us a hop where this takes 1.6 to 2.  Up to 64 workgroups read each other's words directly, in one trip (paper settings, five
// crossings: 30 workgroups 39.2 -> 33.4 us a call, 40 workgroups 31.9 -> 29.2); above that the first of every 16 gathers its group
// and publishes the group's sums in copies, two trips with little traffic: all 256 workgroups reading all words, 16 waves
// each, took 49 us where two trips take 43.
constexpr uint32_t kSumGroup = 16, kSumDirect = 64;      // workgroups per group (and groups, at most)
constexpr uint32_t kSumCopies = 7;                       // of a group's sums: 7 * 9 words are one store instruction
constexpr uint32_t kSumStride = 160;                     // words between copies
static_assert(kSumGroup * kSumGroup >= (uint32_t)kResMaxWG && kSumGroup * 9u <= kSumStride && kSumCopies * 9u <= 64u, "layout of the sums");
template <int NV>
struct SumWords {
    static constexpr uint32_t kW = 3 * NV;
    uint64_t level1[kResMaxWG * kW];
    uint64_t level2[kSumCopies * kSumStride];
};

// the lane, for code between two searches: what is computed from it is not carried through them in registers
__device__ __forceinline__ uint32_t lane_here()
{
    uint32_t lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));
    return lane;
}

// Wave 0, all lanes: wait until the `count` entries from `src` on carry the token; lane e then holds the values of entry e
// (zeros from `count` on).  lds: MOST entries.
template <int NV, uint32_t MOST>
__device__ __forceinline__ bool gather_sums(const ResidentGrid &r, const uint64_t *src, uint32_t count, uint64_t *lds, double v[NV])
{
    constexpr int P = kResSumBits;
    constexpr uint32_t kW = 3 * NV, kLoads = (MOST * kW + 63) / 64;
    const uint32_t lane = lane_here(), n = count * kW;
    const uint64_t want = (r.tok << P) >> P, gone_field = (~r.base << P) >> P;
    uint64_t x[kLoads];
    for (uint64_t round = 0;; ++round) {
        // all loads of a round first, whatever the registers: one trip to memory a round, not one per word
#pragma unroll
        for (uint32_t k = 0; k < kLoads; ++k)
            x[k] = lane + 64u * k < n ? __hip_atomic_load(src + lane + 64u * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : want << P;
        __builtin_amdgcn_sched_barrier(0);
        bool pending = false, gone = false;
#pragma unroll
        for (uint32_t k = 0; k < kLoads; ++k) {
            const uint64_t field = x[k] >> P;
            gone = gone | (field == gone_field);
            pending = pending | (field != want);
        }
        if (__builtin_amdgcn_ballot_w64(gone) != 0ull) return false;
        if (__builtin_amdgcn_ballot_w64(pending) == 0ull) break;
        if (resident_time_is_up(r, round)) return false;
    }
#pragma unroll
    for (uint32_t k = 0; k < kLoads; ++k)
        if (lane + 64u * k < MOST * kW) lds[lane + 64u * k] = x[k] & ((1ull << P) - 1ull);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint64_t *mine = lds + min(lane, MOST - 1u) * kW;
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = lane < count ? resident_join(mine + 3 * j) : 0.0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return true;
}

// Wave 0, all lanes: entry `e` of `copies` copies, a word per lane, from NV values (uniform; by value: an array would be indexed in
// scratch memory)
template <int NV>
__device__ __forceinline__ void publish_sums(const ResidentGrid &r, uint64_t *dst, uint32_t e, uint32_t copies, double v0, double v1, double v2)
{
    constexpr uint32_t kW = 3 * NV;
    const uint32_t lane = lane_here(), copy = lane / kW, w = lane - copy * kW;
    const uint32_t value = w / 3u, third = w - value * 3u;
    uint64_t b = (uint64_t)__double_as_longlong(v0);
    if (NV > 1) b = value == 1u ? (uint64_t)__double_as_longlong(v1) : b;
    if (NV > 2) b = value == 2u ? (uint64_t)__double_as_longlong(v2) : b;
    const uint64_t x = (b >> (third * (uint32_t)kResSumBits)) & ((1ull << kResSumBits) - 1ull);
    if (copy < copies)
        __hip_atomic_store(dst + copy * kSumStride + e * kW + w, (r.tok << kResSumBits) | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave 0, all lanes, every workgroup: the adjacent-pair tree sums of NV binary64 values (lane 0's on entry; one set per workgroup,
// in workgroup order, zero-padded) over the grid; uniform on return.  lds: kSumDirect entries.
template <int NV>
__device__ __forceinline__ bool cross_sums(const ResidentGrid &r, SumWords<NV> &words, uint64_t *lds, double v[NV])
{
    constexpr uint32_t kW = SumWords<NV>::kW;
    auto tree = [&]() {
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] = wave_pair_tree(v[j]);
    };
    auto publish = [&](uint64_t *dst, uint32_t e, uint32_t copies) {
        publish_sums<NV>(r, dst, e, copies, v[0], v[NV > 1 ? 1 : 0], v[NV > 2 ? 2 : 0]);
    };
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = readlane_f64(v[j], 0);
    publish(words.level1, r.g, 1u);
    if (r.G > kSumDirect) {
        const uint32_t grp = r.g / kSumGroup, groups = (r.G + kSumGroup - 1u) / kSumGroup;
        if (r.g % kSumGroup == 0u) {
            if (!gather_sums<NV, kSumGroup>(r, words.level1 + grp * kSumGroup * kW, min(kSumGroup, r.G - grp * kSumGroup), lds, v)) return false;
            tree();
            publish(words.level2, grp, kSumCopies);
        }
        if (!gather_sums<NV, kSumGroup>(r, words.level2 + (r.g % kSumCopies) * kSumStride, groups, lds, v)) return false;
    } else if (r.G > kSumDirect / 2u) {
        if (!gather_sums<NV, kSumDirect>(r, words.level1, r.G, lds, v)) return false;
    } else if (!gather_sums<NV, kSumDirect / 2u>(r, words.level1, r.G, lds, v)) {
        return false;
    }
    tree();
    return true;
}

// one lane of a workgroup that gives up: its words among the sums
template <int NV>
__device__ __forceinline__ void leave_sums(const ResidentGrid &r, SumWords<NV> &words, uint64_t gone)
{
    auto put = [&](uint64_t *p) { __hip_atomic_store(p, gone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    put(words.level1 + r.g * SumWords<NV>::kW);
    if (r.g % kSumGroup == 0u)
        for (uint32_t c = 0; c < kSumCopies; ++c) put(words.level2 + c * kSumStride + r.g / kSumGroup * SumWords<NV>::kW);
}

// Wave 0, all lanes: the sum of ONE value, wanted by workgroup 0 only, which gathers all workgroups in one trip
// (lane l holds workgroups l, l + 64, ...: the tree of 64 is a wave tree, the rest follows); three words per workgroup, by kinds
__device__ __forceinline__ void publish_sum(const ResidentGrid &r, uint64_t *dst, double v)
{
    uint64_t pay[3];
    resident_split(v, pay);
    if ((threadIdx.x & 63u) == 0)
#pragma unroll
        for (int w = 0; w < 3; ++w)
            __hip_atomic_store(dst + w * kResMaxWG + r.g, (r.tok << kResSumBits) | pay[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool collect_sum(const ResidentGrid &r, const uint64_t *src, double &v)
{
    constexpr int P = kResSumBits, K = kResMaxWG / 64;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t want = (r.tok << P) >> P, gone_field = (~r.base << P) >> P;
    uint64_t x[K][3];
    for (uint64_t round = 0;; ++round) {
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int w = 0; w < 3; ++w)
                x[k][w] = lane + 64u * k < r.G ? __hip_atomic_load(src + w * kResMaxWG + lane + 64u * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                               : want << P;
        __builtin_amdgcn_sched_barrier(0);
        bool pending = false, gone = false;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int w = 0; w < 3; ++w) {
                const uint64_t field = x[k][w] >> P;
                gone = gone | (field == gone_field);
                pending = pending | (field != want);
            }
        if (__builtin_amdgcn_ballot_w64(gone) != 0ull) return false;
        if (__builtin_amdgcn_ballot_w64(pending) == 0ull) break;
        if (resident_time_is_up(r, round)) return false;
    }
    double s[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int w = 0; w < 3; ++w) x[k][w] &= (1ull << P) - 1ull;
        s[k] = wave_pair_tree(resident_join(x[k]));
    }
    static_assert(K == 4, "the tree over the groups of 64 is written out");
    v = (s[0] + s[1]) + (s[2] + s[3]);
    return true;
}

}  // namespace
