// Selection of the K largest 64-bit keys held in registers, by a workgroup (rerank) or by one
// wavefront (draft expansion).
//
// A key is (monotone image of an fp32 value) << 32 | ~index, so the larger key wins under
// "value descending, index ascending"; key 0 means "no element".
//
// Method: find a threshold tau that at least K elements reach, cheaply and without looking at
// every element pair; compact the elements >= tau into LDS (ballot + prefix count); rank those
// survivors exactly by counting larger keys with broadcast LDS reads.  Every step is exact; the
// threshold only limits how much is ranked.  Data with huge runs of equal values makes
// everything survive and is ranked by the same code in a slower loop.
#pragma once

#include "radar_device.h"

namespace radar {

constexpr int kTopkThreads = 256;
constexpr int kTopkWaves = kTopkThreads / kWave;
constexpr int kTopkMaxK = 64;
constexpr int kTopkMaxEPT = 16;

struct TopkSmem {
    alignas(16) uint64_t surv[kTopkThreads * kTopkMaxEPT + 32];   // compacted survivors (+32: grouped reads past the end)
    uint64_t top[kTopkMaxK];                          // result, best first; 0 where fewer than K exist
    alignas(16) uint32_t lmax[kTopkThreads / 2 + 4];  // largest value of each pair of lanes, a gap between the halves
    uint32_t tau;
    int count;                                        // number of survivors
};
constexpr int kTopkCleared = 512;                     // survivors' slots that are cleared beforehand

// Workgroup version, 256 lanes, 1 <= K <= 64, EPT <= 16 keys per lane.  tau = the K-th largest of the 128 maxima of
// pairs of lanes; the two lanes of a pair count half of the others each, and so they do when the survivors (about
// 1.4 K) are ranked.  (256 lane maxima leave fewer survivors, 1.15 K, but ranking them is 2000 cycles of comparisons
// where this is 500: a rerank of 710 candidates 5.6 us and now, with the arguments in registers at the start and depths by
// doubling, 4.0; 4096 candidates 8.2 and 5.4.)  keys[e] == 0 marks an absent element.  All 256 threads must call this (it synchronises the workgroup).  On
// return s.top[0..K) is valid for every thread.
template <int EPT>
__device__ __forceinline__ void block_topk(const uint64_t (&keys)[EPT], int K, TopkSmem &s) {
    const int tid = threadIdx.x, lane = lane_id();
    constexpr int kPairs = kTopkThreads / 2, kHalf = kPairs / 2;

    uint32_t tmax = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) tmax = max(tmax, uint32_t(keys[e] >> 32));
    tmax = max(tmax, dpp_u32<0xB1>(tmax));
    const int pair = tid >> 1, half = tid & 1;
    if (half == 0) s.lmax[pair < kHalf ? pair : pair + 4] = tmax;
    if (tid == 0) { s.count = 0; s.tau = 0xffffffffu; }
    if (tid < kTopkMaxK) s.top[tid] = 0;
    for (int i = tid; i < kTopkCleared; i += kTopkThreads) s.surv[i] = 0;
    __syncthreads();

    // ---- tau: smallest pair maximum that fewer than K pair maxima exceed
    {
        const uint32_t *const theirs = s.lmax + half * (kHalf + 4);
        uint32_t larger = 0;
#pragma unroll
        for (int j = 0; j < kHalf; j += 16) {                     // broadcast reads, 16 values in flight
            uint32_t v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = theirs[j + u];
#pragma unroll
            for (int u = 0; u < 16; ++u) larger += (v[u] > tmax) ? 1 : 0;
        }
        larger += dpp_u32<0xB1>(larger);
        uint32_t c = larger < (uint32_t)K ? tmax : 0xffffffffu;
        c = min(c, dpp_u32<0xB1>(c));
        c = min(c, dpp_u32<0x4E>(c));
        c = min(c, dpp_u32<0x141>(c));
        c = min(c, dpp_u32<0x140>(c));
        const uint32_t wmin = min(min(readlane_u32(c, 0), readlane_u32(c, 16)), min(readlane_u32(c, 32), readlane_u32(c, 48)));
        if (lane == 0) atomicMin(&s.tau, wmin);
    }
    __syncthreads();
    const uint32_t tau = max(s.tau, 1u);                          // >= 1 so that absent keys (0) never pass

    // ---- compaction: count, reserve a range per wavefront, write
    int cnt = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) cnt += __popcll(__ballot(uint32_t(keys[e] >> 32) >= tau));
    int base = 0;
    if (lane == 0 && cnt > 0) base = atomicAdd(&s.count, cnt);
    base = (int)readlane_u32((uint32_t)base, 0);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const bool keep = uint32_t(keys[e] >> 32) >= tau;
        const uint64_t m = __ballot(keep);
        if (m) {
            if (keep) s.surv[base + lanes_below(m)] = keys[e];
            base += __popcll(m);
        }
    }
    __syncthreads();
    const int n = s.count;
    if (n > kTopkCleared - 32) {                                  // long runs of equal values
        if (tid < 32) s.surv[n + tid] = 0;                        // padding for the grouped reads
        __syncthreads();
    }

    // ---- exact ranks among the n survivors, two lanes each: every other two of the survivors
    for (int i = pair; i - pair < n; i += kPairs) {
        const uint64_t key = s.surv[min(i, n - 1)];
        uint32_t rank = 0;
        for (int j = 2 * half; j < n; j += 32) {
            uint64_t kj[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) kj[u] = s.surv[j + (u >> 1) * 4 + (u & 1)];
#pragma unroll
            for (int u = 0; u < 16; ++u) rank += (kj[u] > key) ? 1 : 0;
        }
        rank += dpp_u32<0xB1>(rank);
        if (half == 0 && i < n && rank < (uint32_t)K) s.top[rank] = key;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// The same selection inside ONE wavefront, without workgroup barriers: the K <= 16 largest of the 64 * EPL keys its
// lanes hold.  These keys have 63 bits (the index keeps 31), so that a difference of two has its sign in bit 63.
//
// How things are compared here: a vector compare leaves its result in scalar registers, and the instruction that counts it has to
// wait for that (four issue slots in all, in a lone wavefront, whose every slot is on the critical path); a subtraction leaves
// it in the sign bit, and one alignbit appends that bit to a mask, whose ones are counted at the end: two slots, no wait.
// Values that are only grouped by a threshold are compared without their lowest bit, which leaves room for the sign; what the
// threshold promises still holds.
__device__ __forceinline__ uint64_t pick_key(float x, uint32_t idx) { return (uint64_t)ord_of(x) << 31 | (~idx & 0x7fffffffu); }
__device__ __forceinline__ uint32_t pick_index(uint64_t key) { return ~(uint32_t)key & 0x7fffffffu; }
__device__ __forceinline__ float pick_value(uint64_t key) { return float_of_ord((uint32_t)(key >> 31)); }

__device__ __forceinline__ uint32_t append_sign(uint32_t mask, uint32_t v) { return __builtin_amdgcn_alignbit(mask, v, 31); }   // mask << 1 | v >> 31

// K-th largest (K <= 16) of 32 values below 2^31, of which every lane passes number lane % 32; the result is the same in
// every lane.  Rows 0 and 1 of the wavefront count what is not smaller among values 0-15, rows 2 and 3 (which
// hold the same values again) among 16-31, by row rotations of the complements: g + ~c is negative if c >= g.
// (An addition: subtracting a rotated operand came out with the other sign, v_subrev_u32 with a DPP operand.)
template <int ROR>
__device__ __forceinline__ void mark_not_smaller(uint32_t nc, uint32_t g, uint32_t &mask) {
    if constexpr (ROR < 16) {
        mask = append_sign(mask, g + dpp_u32<0x120 + ROR>(nc));                 // row_ror
        mark_not_smaller<ROR + 1>(nc, g, mask);
    }
}
__device__ __forceinline__ uint32_t kth_of_32(uint32_t g, int K) {
    const auto ab = __builtin_amdgcn_permlane16_swap(g, g, false, false);       // values 0-15, values 16-31 in every row
    const uint32_t nc = ~(lane_id() < 32 ? ab[0] : ab[1]);
    uint32_t mask = append_sign(0, g + nc);
    mark_not_smaller<1>(nc, g, mask);
    const uint32_t n1 = (uint32_t)__popc(mask);
    const auto n = __builtin_amdgcn_permlane32_swap(n1, n1, false, false);
    uint32_t k = n[0] + n[1] >= (uint32_t)K ? g : 0;               // what at least K values reach; the largest of that
    k = max(k, dpp_u32<0xB1>(k));
    k = max(k, dpp_u32<0x4E>(k));
    k = max(k, dpp_u32<0x141>(k));
    k = max(k, dpp_u32<0x140>(k));
    const auto m = __builtin_amdgcn_permlane16_swap(k, k, false, false);
    return max(m[0], m[1]);
}
// The same for the maxima of groups of floats: a threshold that at least K of them reach (at least -inf, whose image is odd).
__device__ __forceinline__ float kth_threshold(float g, int K) { return float_of_ord(max(kth_of_32(ord_of(g) >> 1, K) << 1, 0x007fffffu)); }

constexpr int kPickMost = 512;                    // survivors that can be ranked
constexpr int kPickPad = 8;                       // entries that they may be padded by, where they are more than 32
struct WaveTopkSmem {
    alignas(16) uint64_t surv[kPickMost + kWave]; // complements of the survivors
    uint64_t top[16];
};

struct Picked { uint64_t key; int rank; };        // a lane's key and how many are larger; rank kNoRank: none
constexpr int kNoRank = 1 << 20;

template <int PARTS>                              // up to 64 / PARTS survivors: each is compared in PARTS lanes
__device__ __forceinline__ Picked rank_among_few(const uint64_t *surv, int n) {
    constexpr int kMost = kWave / PARTS, kEach = kMost / PARTS;
    const int lane = lane_id(), i = lane & (kMost - 1), part = lane / kMost;
    Picked p;
    p.key = ~surv[i];
    uint64_t t[kEach];
#pragma unroll
    for (int u = 0; u < kEach; ++u) t[u] = surv[part * kEach + u];
    uint32_t larger = 0;                          // (and the key itself, once)
#pragma unroll
    for (int u = 0; u < kEach; ++u) larger = append_sign(larger, (uint32_t)((p.key + t[u]) >> 32));
    uint32_t c = (uint32_t)__popc(larger);
    if (PARTS == 4) { const auto a = __builtin_amdgcn_permlane16_swap(c, c, false, false); c = a[0] + a[1]; }
    const auto b = __builtin_amdgcn_permlane32_swap(c, c, false, false);
    c = b[0] + b[1];
    p.rank = lane < n && lane < kMost ? (int)c - 1 : kNoRank;
    return p;
}

// The n survivors whose complements are in surv (room for 48 of them, and for kPickPad more), ranked: every one of the K largest is in one lane.
__device__ __forceinline__ Picked rank_survivors(uint64_t *surv, uint64_t *top, int n, int K) {
    const int lane = lane_id();
    if (lane < (n <= 32 ? 16 : kPickPad)) surv[n + lane] = ~0ull;
    wave_lds_sync();
    if (n <= 16) return rank_among_few<4>(surv, n);
    if (n <= 32) return rank_among_few<2>(surv, n);
    if (lane < 16) top[lane] = 0;
    wave_lds_sync();
    for (int i0 = 0; i0 < n; i0 += kWave) {       // one pass unless many values are equal
        const int i = i0 + lane;
        const uint64_t key = ~surv[min(i, n - 1)];
        int rank = -1;
        for (int j = 0; j < n; j += 8) {          // broadcast reads (every lane reads the same keys), eight in flight
            uint64_t t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = surv[j + u];
            uint32_t larger = 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) larger = append_sign(larger, (uint32_t)((key + t[u]) >> 32));
            rank += __popc(larger);
        }
        if (i < n && rank < K) top[rank] = key;
    }
    wave_lds_sync();
    Picked p;
    p.key = top[lane & 15];
    p.rank = lane < K && p.key != 0 ? lane : kNoRank;
    wave_lds_sync();
    return p;
}

// The K largest keys (0: none) and their ranks, each in some lane.  Threshold: the K-th largest of the maxima of the 32 pairs of lanes, so at
// least K keys pass where there are as many, and of keys in no particular order 1.2 K to 1.4 K.  (Of the maxima of the 16 quads 1.5 K,
// and all of them for K = 16.)  Survivors are compacted into the wavefront's private scratch.  Callers on different wavefronts pass different
// scratch; all 64 lanes must call.  between() runs once the keys are in LDS and their registers free.
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <int EPL, typename Between = Nothing>
__device__ __forceinline__ Picked wave_pick(const uint64_t (&keys)[EPL], int K, WaveTopkSmem &s, Between &&between = Between()) {
    static_assert(EPL * kWave + kPickPad <= kPickMost, "scratch too small");
    const int lane = lane_id();
    uint32_t tmax = 0;
#pragma unroll
    for (int e = 0; e < EPL; ++e) tmax = max(tmax, uint32_t(keys[e] >> 32));
    tmax = max(tmax, dpp_u32<0xB1>(tmax));
    tmax = (lane & 1) == (lane >> 5) ? tmax : 0;  // even lanes of one half of the wavefront, odd lanes of the other ...
    const auto h = __builtin_amdgcn_permlane32_swap(tmax, tmax, false, false);
    const uint32_t tau = max(kth_of_32(max(h[0], h[1]), K), 1u);   // ... so that both halves hold all 32 (never 0: absent keys do not pass)

    // No branches: what does not pass goes to the scratch's last slot, which no survivor reaches.
    int n = 0;                                    // survivors so far (wave-uniform)
    uint64_t m[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) m[e] = __ballot(uint32_t(keys[e] >> 32) >= tau);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const int at = n + lanes_below(m[e]);
        s.surv[uint32_t(keys[e] >> 32) >= tau ? at : kPickMost] = ~keys[e];
        n += __popcll(m[e]);
    }
    between();
    return rank_survivors(s.surv, s.top, n, K);
}

// A selection as a key of the next one: the keys picked so far in the lanes that hold them.
__device__ __forceinline__ uint64_t carried(const Picked &p, int K) { return p.rank < K ? p.key : 0; }

}  // namespace radar
