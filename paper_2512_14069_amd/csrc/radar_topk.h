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
// The same selection inside ONE wavefront, without workgroup barriers: K <= 16 largest of the
// 64 * EPL keys its lanes hold.  The 16 quads of the wavefront are the groups (tau = K-th
// largest quad maximum, so at least K keys pass; callers spread their keys over the quads, or
// few quads hold anything and tau filters little), survivors are compacted into the
// wavefront's private LDS scratch and ranked exactly.  Returns the r-th largest key in lane r
// (r < 16; 0 where fewer exist, and in lanes >= 16).  Callers on different wavefronts pass
// different scratch; all 64 lanes must call.
constexpr int kWaveTopkMaxEPL = 9;

template <int ROR>
__device__ __forceinline__ void count_larger(uint32_t g, int &larger) {
    if constexpr (ROR < 16) {
        larger += dpp_u32<0x120 + ROR>(g) > g ? 1 : 0;              // row_ror
        count_larger<ROR + 1>(g, larger);
    }
}

// Threshold for a selection of the K <= 16 largest values held by the lanes of one wavefront
// (v = largest value of the lane, 0 if it holds none): the K-th largest of the 16 quad maxima.
// At least K values are >= the result (one per quad that reaches it), and unlike the smallest
// quad maximum it does not collapse when a few quads happen to hold only small values.
// Never 0, so that absent entries (0) fail the test "value >= threshold".
// All 16 maxima are brought into every 16-lane row by row swaps (lane 4 i + r of a row receives the
// maximum of row r's quad i) and ranked there by rotations: vector instructions throughout, where sixteen
// lane reads cross to the scalar side and back.
__device__ __forceinline__ uint32_t quad_threshold(uint32_t v, int K) {
    uint32_t g = v;
    g = max(g, dpp_u32<0xB1>(g));
    g = max(g, dpp_u32<0x4E>(g));                 // quad maximum in every lane of the quad
    const int lane = lane_id();
    g = (lane & 3) == (lane >> 4) ? g : 0;
    const auto a = __builtin_amdgcn_permlane16_swap(g, g, false, false);        // rows 0 0 2 2, rows 1 1 3 3
    g = max(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(g, g, false, false);
    g = max(b[0], b[1]);
    int larger = 0;                               // quads whose maximum is strictly larger than this lane's
    count_larger<1>(g, larger);
    uint32_t c = larger < K ? g : 0xffffffffu;    // the K largest quad maxima (and their ties) stay
    c = min(c, dpp_u32<0xB1>(c));
    c = min(c, dpp_u32<0x4E>(c));
    c = min(c, dpp_u32<0x141>(c));
    c = min(c, dpp_u32<0x140>(c));                // smallest of them; the same in every row
    return max(c, 1u);
}

// K-th largest (K <= 16) of 32 values, of which every lane passes number lane % 32; the result is the same in
// every lane.  Rows 0 and 1 of the wavefront count what is larger among values 0-15, rows 2 and 3 (which
// hold the same values again) among 16-31, by row rotations.
template <int ROR>
__device__ __forceinline__ void count_larger_of(uint32_t c, uint32_t g, int &larger) {
    if constexpr (ROR < 16) {
        larger += dpp_u32<0x120 + ROR>(c) > g ? 1 : 0;              // row_ror
        count_larger_of<ROR + 1>(c, g, larger);
    }
}
__device__ __forceinline__ uint32_t kth_of_32(uint32_t g, int K) {
    const auto ab = __builtin_amdgcn_permlane16_swap(g, g, false, false);       // values 0-15, values 16-31 in every row
    const uint32_t c = lane_id() < 32 ? ab[0] : ab[1];
    int larger = c > g ? 1 : 0;
    count_larger_of<1>(c, g, larger);
    const auto n = __builtin_amdgcn_permlane32_swap((uint32_t)larger, (uint32_t)larger, false, false);
    uint32_t k = n[0] + n[1] < (uint32_t)K ? g : 0xffffffffu;      // the K largest (and their ties) stay
    k = min(k, dpp_u32<0xB1>(k));
    k = min(k, dpp_u32<0x4E>(k));
    k = min(k, dpp_u32<0x141>(k));
    k = min(k, dpp_u32<0x140>(k));
    const auto m = __builtin_amdgcn_permlane16_swap(k, k, false, false);
    return min(m[0], m[1]);
}

struct WaveTopkSmem {
    uint64_t surv[kWave * kWaveTopkMaxEPL + 8];   // +8: the ranking reads keys eight at a time
    uint64_t top[16];
};

// between() runs once the keys are in LDS and their registers free.
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <int EPL, typename Between = Nothing>
__device__ __forceinline__ uint64_t wave_topk(const uint64_t (&keys)[EPL], int K, WaveTopkSmem &s, Between &&between = Between()) {
    static_assert(EPL <= kWaveTopkMaxEPL, "scratch too small");
    const int lane = lane_id();
    uint32_t tmax = 0;
#pragma unroll
    for (int e = 0; e < EPL; ++e) tmax = max(tmax, uint32_t(keys[e] >> 32));
    const uint32_t tau = quad_threshold(tmax, K);

    int n = 0;                                    // survivors so far (wave-uniform)
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const bool keep = uint32_t(keys[e] >> 32) >= tau;
        const uint64_t m = __ballot(keep);
        if (keep) s.surv[n + lanes_below(m)] = keys[e];
        n += __popcll(m);
    }
    if (lane < 8) s.surv[n + lane] = 0;           // padding for the grouped reads
    if (lane < 16) s.top[lane] = 0;
    between();
    wave_lds_sync();
    for (int i0 = 0; i0 < n; i0 += kWave) {       // one pass unless nearly everything survived
        const int i = i0 + lane;
        const uint64_t key = s.surv[min(i, n - 1)];
        int rank = 0;
        for (int j = 0; j < n; j += 8) {          // broadcast reads (every lane reads the same keys),
            uint64_t kj[8];                       // eight in flight so that their latencies overlap
#pragma unroll
            for (int u = 0; u < 8; ++u) kj[u] = s.surv[j + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) rank += (kj[u] > key) ? 1 : 0;
        }
        if (i < n && rank < K) s.top[rank] = key;
    }
    wave_lds_sync();
    const uint64_t r = s.top[lane & 15];
    wave_lds_sync();                              // scratch may be reused right after the return
    return lane < 16 ? r : 0;
}

constexpr int kWaveListSlots = 32;               // a wavefront's list in LDS

// Lists of 16 slots, at least K of them used unless the chunk is shorter, in any order and from the first on (slot i: list
// i / 16), taken 64 slots per step: which slot a lane takes at step e.  Lanes rotate by 4 per step, so a lane
// meets slots of different places and every quad of lanes holds used slots.
__device__ __forceinline__ int topk_slot_of(int e) {
    return e * kWave + ((lane_id() + 4 * e) & (kWave - 1));
}

}  // namespace radar
