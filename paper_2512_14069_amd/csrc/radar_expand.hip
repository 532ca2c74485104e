// Draft-tree expansion and rerank for RADAR's drafting loop (App. A.1, Sec. 2.3,
// Sec. 4.2 Eq. 3), as single-launch HIP kernels for gfx950.
//
// radar_draft_expand: grid (chunks of 4096, 8192 or 16384 logits, frontier rows).
// Every workgroup streams its chunk once from HBM with 16-byte loads (the whole
// step is one read of F*V*4 bytes), keeps its 4, 8 or 16 values per lane in registers,
// and leaves (a list with the chunk's top-k keys in any order, chunk max, chunk sum of exp) in the workspace.
// Counters (one for a call of few workgroups; else one per row, then one per call) single
// out the workgroup that comes last, which takes the others' words as they arrive (each says itself that
// it is there) and merges every row, one wavefront per row
// (top-k of the chunk lists, log-sum-exp in fp64, cumulative scores, pool
// append), and picks the next frontier.  There is no second launch and no
// host round trip.  radar_draft_expand_policy lets the same workgroup go on to
// the prediction model's step on the k confidences it has just produced
// (Sec. 4.2), so the continue / stop decision costs no launch of its own.
// radar_draft_expand_batch adds a grid dimension: one such call per sequence,
// B sequences in one launch, each with its own arrays, counters and last workgroup.
#include <algorithm>
#include <mutex>

#include "radar_topk.h"
#include "radar_policy.h"
#include "radar_host.h"

namespace radar {

constexpr int kExpThreads = 1024;
constexpr int kExpWaves = kExpThreads / kWave;
constexpr int kExpMinEPT = 4;                         // logits per lane: 4, 8 or 16 (chosen per call)
constexpr int kExpMaxChunks = 256;                    // V <= 1,048,576
constexpr int kCounterStride = 32;                    // arrival counters sit 128 B apart: fetch-adds on one
                                                      // cache line serialise at roughly 10 ns each
constexpr size_t kCounterBytes = 16384;               // leading counter block of the workspace
constexpr float kLog2eF = 1.4426950408889634f;
constexpr int kStreamers = 4;                         // wavefronts of a workgroup that stream
constexpr int kDumpCap = 32;                          // hot lanes of one of them (largest logit reaches the threshold) whose logits go through LDS
constexpr int kFastCap = 512;                         // chunk candidates ranked by the short path; more (runs of equal values) rank per wavefront
constexpr int kFewChunks = 16;                        // rows of so many chunks are merged the short way (expand_finish)
constexpr int kFrontierBlock = 128;                   // candidates that are looked at together for the frontier
constexpr int kRound = 256;                           // workgroups of the single launch that run at once, one per CU
constexpr int64_t kStreamMinLogits = 4 << 20;         // batched calls over rows of less than a streaming workgroup's width stream from here on

// What the workgroups of a single launch hand over vouches for itself: the reader looks until every word is there.  A key there
// and a sum have bit 63 set (what the two-launch form leaves does not), a maximum has 1 in its upper half; the reader clears what it has
// read, and nothing else that a workspace can hold looks like that.  An empty slot of a list is a mark without a key.
constexpr uint64_t kThere = uint64_t(1) << 63;
constexpr size_t kGateOffset = 12288, kStreamGateOffset = 14336;   // the prediction model's w_hh h (of which no value is 0 in a single launch), in the counter block
static_assert((1 + RADAR_F_MAX) * kCounterStride * sizeof(unsigned int) <= kGateOffset && kGateOffset + 4 * kPolH * sizeof(float) <= kStreamGateOffset &&
              kStreamGateOffset + 4 * kPolH * sizeof(float) <= kCounterBytes, "counter block");
// (A workspace is cleared as a whole before its first use: what an uncleared one holds can look like a word.)
constexpr unsigned int kPollLimit = 1u << 22;         // looks (0.5 us and more each) at what is on its way, unless a second call uses the workspace at the same time

// what a launch carries beside the expansion itself: nothing; a batch or a cycle state; a prediction model, too
enum { kExpPlain, kExpExt, kExpPolicy };

struct ExpandArgs {
    const float *logits;
    const float *parent_scores;
    const int32_t *parent_pool_idx;
    int32_t *cand_tokens;
    float *cand_scores;
    int32_t *frontier_pool_idx;
    int32_t *frontier_tokens;
    float *frontier_scores;
    float *frontier_conf;
    int32_t *pool_tokens;
    float *pool_scores;
    int32_t *pool_parents;
    int F, V, k, nchunks, pool_count;
    int pool_capacity;          // length of one sequence's pool arrays (their stride in a batched call)
    unsigned int *counters;     // [0] rows finished, [(1+f) * kCounterStride] chunks of row f finished
    uint64_t *part_keys;        // [F][nchunks][RADAR_K_MAX] in any order, 0 where a chunk has fewer
    uint64_t *part_lm;          // [F][nchunks][2] sum of exp(x - m) over the chunk, and its maximum m in the lower half
    PolicyArgs pol;             // prediction model run by the last workgroup when has_policy != 0
    float *gate_pre;            // [4H] w_hh h of that model, computed by the first workgroups of the launch
    radar_cycle_state *cycle;   // device-side state of the drafting cycle, or null: when set, pool_count above is
                                // only the largest value the state's own count may have
    int has_policy, pol_has_state;
};

struct alignas(16) ExpandSmem {
    WaveTopkSmem wtk[kExpWaves];                  // one scratch per wavefront
    uint64_t wlist[kStreamers * RADAR_K_MAX];     // the streaming wavefronts' best (many ties only)
    float gmax[8 * kStreamers];                   // maxima of the 8-lane groups of the streaming wavefronts
    double wave_l[kStreamers];                    // sum of exp(x - chunk maximum) over each streaming wavefront
    float cmax;                                   // the maximum
    unsigned int nsurv;                           // candidates of the chunk that reached the threshold
    unsigned int ndump[kStreamers];               // lanes of each streaming wavefront whose largest logit reached it
    float tau;                                    // the threshold
    unsigned char dump_lane[kStreamers][kDumpCap];   // which lane left each block of logits
    // last workgroup only: candidate c = f * k + r (row f, rank r in it)
    float cand_sc[RADAR_F_MAX * 16];
    int cand_tok[RADAR_F_MAX * 16];
    alignas(16) uint64_t cand_key[RADAR_F_MAX * 16];
    PolicySmem pol;
    int last;                                     // this workgroup finishes the call
};

__device__ __forceinline__ bool word_there(uint64_t w) { return (int64_t)w < 0; }                   // a key's or a sum's
__device__ __forceinline__ bool max_there(uint64_t w) { return (uint32_t)(w >> 32) == 1u; }
__device__ __forceinline__ uint64_t key_of_word(uint64_t w) { return w & ~kThere; }
__device__ __forceinline__ double sum_of_word(uint64_t w) { return __longlong_as_double((long long)(w & ~kThere)); }   // (sums are not negative)
__device__ __forceinline__ float max_of_word(uint64_t w) { return __uint_as_float((uint32_t)w); }

// A key that passes any threshold, whatever the value's bits: the two lowest images belong to NaNs and have no bit in a key's upper half.
__device__ __forceinline__ uint64_t key_of_any(float x, uint32_t idx) { return (uint64_t)max(ord_of(x), 2u) << 31 | (~idx & 0x7fffffffu); }

// Entry `at` of the next frontier is candidate c.  conf_lds, when given, also receives the confidence.
__device__ __forceinline__ void put_frontier(const ExpandArgs &a, const ExpandSmem &s, int at, int c, float *conf_lds) {
    const float sc = s.cand_sc[c];
    a.frontier_pool_idx[at] = a.pool_count + c;
    a.frontier_tokens[at] = s.cand_tok[c];
    a.frontier_scores[at] = sc;
    const float conf = expf(sc);
    a.frontier_conf[at] = conf;
    if (conf_lds) conf_lds[at] = conf;
}

// Next frontier: the k largest of n candidates by cumulative score (candidate index breaks ties), by one wavefront; where they are MANY every
// wavefront calls.  s.cand_key holds zeros from n on.  (By the whole workgroup, each candidate's larger ones counted in parts of the list, it was
// bound by LDS: a broadcast read takes as long as any other, 0.4 us of them for 100 candidates.)
template <bool MANY>                                               // more than kFrontierBlock of them
__device__ __forceinline__ void pick_frontier(const ExpandArgs &a, ExpandSmem &s, int n, float *conf_lds) {
    const int lane = lane_id(), w = wave_id();
    Picked p = {0, kNoRank};
    auto key = [&](int i) { return s.cand_key[i + (lane >> 1) + 32 * (lane & 1)]; };     // (the lanes of a pair far apart: a row's candidates are sorted)
    if constexpr (MANY) {
        // 256 to a wavefront (by 128, 256 candidates were two selections, 0.6 us more); of more than that the best of each are put together.
        uint64_t kk[4];
        if (w * 4 * kWave < n) {
#pragma unroll
            for (int e = 0; e < 4; ++e) kk[e] = key((w * 4 + e) * kWave);
            p = wave_pick<4>(kk, a.k, s.wtk[w]);
        }
        if (n > 4 * kWave) {
            static_assert(RADAR_F_MAX * 16 <= kStreamers * 4 * kWave, "a list for each wavefront that takes part");
            if (w < kStreamers && lane < RADAR_K_MAX) s.wlist[w * RADAR_K_MAX + lane] = 0;
            wave_lds_sync();
            if (w * 4 * kWave < n && p.rank < a.k) s.wlist[w * RADAR_K_MAX + p.rank] = p.key;
            __syncthreads();
            if (w == 0) {
                const uint64_t best[2] = {s.wlist[lane], 0};
                p = wave_pick<2>(best, a.k, s.wtk[0]);
            }
        }
        if (w != 0) return;
    } else {
        const uint64_t kk[2] = {key(0), key(kWave)};
        p = wave_pick<2>(kk, a.k, s.wtk[0]);
    }
    if (p.rank < a.k) put_frontier(a, s, p.rank, (int)pick_index(p.key), conf_lds);
}

// Sequence bz of a batched call: every array of the call, the workspace parts and the cycle states
// have a leading batch dimension; after this the workgroup sees its own sequence only.
__device__ __forceinline__ void sequence_view(ExpandArgs &a, int bz) {
    const size_t b = (size_t)bz, fk = (size_t)a.F * a.k, fc = (size_t)a.F * a.nchunks;
    a.logits += b * a.F * a.V;
    a.parent_scores += b * a.F; a.parent_pool_idx += b * a.F;
    a.cand_tokens += b * fk; a.cand_scores += b * fk;
    a.frontier_pool_idx += b * a.k; a.frontier_tokens += b * a.k;
    a.frontier_scores += b * a.k; a.frontier_conf += b * a.k;
    a.pool_tokens += b * a.pool_capacity; a.pool_scores += b * a.pool_capacity; a.pool_parents += b * a.pool_capacity;
    a.counters += b * (kCounterBytes / sizeof(unsigned int));
    a.part_keys += b * fc * RADAR_K_MAX; a.part_lm += b * fc * 2;
    a.gate_pre += b * (kCounterBytes / sizeof(float));
    if (a.cycle) a.cycle += b;
}

// What the last workgroup of a sequence's call does once every chunk list and partial sum of the
// sequence is in the workspace (all 1024 lanes must call): rows are merged, candidates scored and
// pooled, the next frontier chosen; with a prediction model its step follows, with a cycle state
// its update.  `a` is already the sequence's own view of the call (bz = its index in the batch).
// settle() is called once the first loads are on their way and says whether the call is made at all (a
// batched call learns here that the sequence's cycle has stopped, and its pool count).
// hidden(row) returns row `row` of w_hh h (complete before the call; only used with a prediction
// model that has a state).
// POLL: what the other workgroups hand over may still be on its way (all of them have begun, and wait for nobody), and is cleared
// once it has been read.  Without, it is all there.
template <int MODE, bool POLL, bool GENERAL, typename Settle, typename Hidden>
__device__ __forceinline__ void expand_finish(ExpandArgs &a, ExpandSmem &s, int bz, radar_cycle_state *cycle,
                                              bool cycle_first, Settle &&settle, Hidden &&hidden) {
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int K = a.k, n = a.F * K;
    const bool few = !GENERAL || a.nchunks <= kFewChunks;                      // (V <= 131072 at 8 logits per lane)
    const int nslot = a.nchunks * RADAR_K_MAX;
    if (tid >= n) s.cand_key[tid] = 0;
    if (MODE == kExpPolicy && tid < RADAR_K_MAX) s.pol.in[kPolH + tid] = 0.f;

    // One wavefront per row (rows w, w+16, ...):
    // top-k of the row's chunk lists, log-sum-exp of the row, cumulative scores, pool append.
    // A look at 256 slots of the lists, four per lane and two to a load (device scope, as load_shared_result's; slots past the lists read 0),
    // and one at the chunks' sums.  What is waited for here is requests: with loads of one slot a call took 8.1 us, 7.9 with two, ten
    // rows of 32000 7.5 and 7.3.  A further look asks only for what the one before did not see.
    uint64_t w2[3][2];
    float pscore = 0.f;
    int ppool = 0;
    const int sum_at = (few ? (lane & 15) : lane) * 16;            // up to 16 chunks: every 16-lane row of the wavefront takes all
    auto look = [&](int fr, int c0, int e) {
        const int urow = __builtin_amdgcn_readfirstlane(fr);
        const auto from = e == 2 ? __builtin_amdgcn_make_buffer_rsrc(a.part_lm + (size_t)urow * a.nchunks * 2, 0, a.nchunks * 16, 0x00027000)
                                 : __builtin_amdgcn_make_buffer_rsrc(a.part_keys + (size_t)urow * nslot, 0, nslot * (int)sizeof(uint64_t), 0x00027000);
        const int at = e == 0 ? c0 * 8 + lane * 16 : e == 1 ? c0 * 8 + kWave * 16 + ((lane + 4) & (kWave - 1)) * 16 : c0 * 16 + sum_at;
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(from, at, 0, 16);
        w2[e][0] = (uint64_t)v[0] | (uint64_t)v[1] << 32;
        w2[e][1] = (uint64_t)v[2] | (uint64_t)v[3] << 32;
    };
    auto all_there = [&](int fr, int c0, bool keys, bool sums) {
        if (!POLL) return;
#pragma unroll 1
        for (unsigned int looks = 0; looks < kPollLimit; ++looks) {
            bool missing[3];
            missing[0] = keys && !(word_there(w2[0][0]) && word_there(w2[0][1])) && c0 + lane * 2 < nslot;
            missing[1] = keys && !(word_there(w2[1][0]) && word_there(w2[1][1])) && c0 + kWave * 2 + ((lane + 4) & (kWave - 1)) * 2 < nslot;
            missing[2] = sums && !(word_there(w2[2][0]) && max_there(w2[2][1])) && c0 + (sum_at >> 4) < a.nchunks;
            if (__ballot(missing[0] || missing[1] || missing[2]) == 0) return;
            asm volatile("" ::: "memory");                         // (else the loads are the ones before)
#pragma unroll
            for (int e = 0; e < 3; ++e) if (missing[e]) look(fr, c0, e);
        }
        // Given up (the call's words were overwritten from elsewhere): the row's scores are NaN, and nothing found in their place is taken for a token.
        pscore = __builtin_nanf("");
#pragma unroll
        for (int e = 0; e < 4; ++e) w2[e >> 1][e & 1] = lane * 4 + e < a.V ? key_of_any(pscore, uint32_t(lane * 4 + e)) : 0;
    };
    auto merge_row = [&](int fr, auto &&between) {
        float ml = sum_at < a.nchunks * 16 ? max_of_word(w2[2][1]) : -INFINITY;
        double ll = sum_of_word(w2[2][0]);
#pragma unroll 1
        for (int c = kWave; GENERAL && c < a.nchunks; c += kWave) {           // V > 262144 only
            look(fr, c, 2);
            all_there(fr, c, false, true);
            if (c + lane < a.nchunks) {
                const float m2 = max_of_word(w2[2][1]), mn = fmaxf(ml, m2);
                if (mn > -INFINITY)
                    ll = ll * (double)__builtin_amdgcn_exp2f((ml - mn) * kLog2eF) + sum_of_word(w2[2][0]) * (double)__builtin_amdgcn_exp2f((m2 - mn) * kLog2eF);
                ml = mn;
            }
        }
        // Maximum and sum inside each 16-lane row by DPP steps alone (no lane reads: those cost a
        // scalar round trip each); fixed order of addition.  In one line with the selection, whose
        // chain of dependent steps leaves room for this one.
        float M = ml;
        M = fmaxf(M, dpp_f32<0xB1>(M));
        M = fmaxf(M, dpp_f32<0x4E>(M));
        M = fmaxf(M, dpp_f32<0x141>(M));
        M = fmaxf(M, dpp_f32<0x140>(M));
        if (!few) M = fmaxf(fmaxf(readlane_f32(M, 0), readlane_f32(M, 16)), fmaxf(readlane_f32(M, 32), readlane_f32(M, 48)));
        double L = ml > -INFINITY ? ll * (double)__builtin_amdgcn_exp2f((ml - M) * kLog2eF) : 0.0;
        auto add = [](double x, uint64_t moved) { return x + __longlong_as_double((long long)moved); };
        L = add(L, dpp_u64<0xB1>((uint64_t)__double_as_longlong(L)));
        L = add(L, dpp_u64<0x4E>((uint64_t)__double_as_longlong(L)));
        L = add(L, dpp_u64<0x141>((uint64_t)__double_as_longlong(L)));
        L = add(L, dpp_u64<0x140>((uint64_t)__double_as_longlong(L)));
        if (!few) L = (readlane_f64(L, 0) + readlane_f64(L, 16)) + (readlane_f64(L, 32) + readlane_f64(L, 48));
        // log in fp32 (1 ulp of a value below 14: 1e-6, a tenth of the tolerance on log-probabilities); the
        // fp64 routine costs 0.3 us on this serial path
        const double lse = (double)M + (double)logf((float)L);
        Picked top;
        uint64_t kk[GENERAL ? 5 : 4];
        auto take = [&] {
#pragma unroll
            for (int e = 0; e < 4; ++e) kk[e] = key_of_word(w2[e >> 1][e & 1]);
        };
        take();
        if constexpr (GENERAL) {
            kk[4] = 0;
#pragma unroll 1
            for (int c0 = 4 * kWave;; c0 += 4 * kWave) {           // the selection so far rides along
                if (c0 < nslot) { look(fr, c0, 0); look(fr, c0, 1); }
                top = wave_pick<5>(kk, K, s.wtk[w]);
                if (c0 >= nslot) break;
                kk[4] = carried(top, K);
                all_there(fr, c0, true, false);
                take();
            }
        } else {
            top = wave_pick<4>(kk, K, s.wtk[w], between);
        }
        if (top.rank < K) {
            const int tok = (int)pick_index(top.key);
            const double logp = (double)pick_value(top.key) - lse;
            const float cum = (float)((double)pscore + logp);
            const int c = fr * K + top.rank;
            s.cand_sc[c] = cum;
            s.cand_tok[c] = tok;
            s.cand_key[c] = key_of_any(cum, uint32_t(c));
            a.cand_tokens[c] = tok;
            a.cand_scores[c] = cum;
            a.pool_tokens[a.pool_count + c] = tok;
            a.pool_scores[a.pool_count + c] = cum;
            a.pool_parents[a.pool_count + c] = ppool;
        }
    };
    auto look_at_row = [&](int fr) {
        look(fr, 0, 0); look(fr, 0, 1); look(fr, 0, 2);
        pscore = a.parent_scores[fr];
        ppool = a.parent_pool_idx[fr];
    };
    if (w < a.F) look_at_row(w);
    if (!settle()) return;
    // The prediction model's operands are requested by every wavefront as its row's lists have been read, or its rows are done, and
    // arrive while the row is ranked and the frontier is chosen.  (Requested with the lists they hold those up: 2 % of a cycle.
    // Requested after the row they came 0.75 us after it: a cycle of eight calls of 10 rows 124.4 us, then 120.2; four calls of 4 rows 48.1 and 46.6.)
    PolicyRegs pr;
    auto fetch = [&] {
        if constexpr (MODE == kExpPolicy) {
            policy_fetch_head(a.pol, pr);
            policy_fetch_rest<true>(a.pol, bz, a.pol_has_state != 0, pr, hidden);
        }
    };
    if constexpr (GENERAL) {
#pragma unroll 1
        for (int fr = w; fr < a.F; fr += kExpWaves) {
            if (fr != w) look_at_row(fr);
            all_there(fr, 0, true, true);
            merge_row(fr, [] {});
        }
        fetch();
    } else if (w < a.F) {
        all_there(w, 0, true, true);
        merge_row(w, fetch);
    } else {
        fetch();
    }
    __syncthreads();
    float *const conf = MODE == kExpPolicy ? &s.pol.in[kPolH] : nullptr;
    if (GENERAL || w == 0) pick_frontier<GENERAL>(a, s, n, conf);
    auto advance = [&](int action) {                               // by one lane
        if (!cycle) return;
        cycle->pool_count = a.pool_count + n;
        cycle->steps_done = cycle_first ? 1 : cycle->steps_done + 1;
        if (action >= 0 || cycle_first) cycle->last_action = action;
        if (action == 0) cycle->stopped = 1;
        else if (cycle_first) cycle->stopped = 0;
    };
    if constexpr (MODE == kExpPolicy) {
        if (POLL && a.pol_has_state && w >= kPolWaves / 2)          // this lane's row of w_hh h
            for (unsigned int looks = 0; __float_as_uint(pr.hid) == 0; ++looks) pr.hid = looks < kPollLimit ? hidden(policy_gate_row()) : __builtin_nanf("");
        // ---- prediction-model step on the new frontier's confidences
        __syncthreads();
        policy_decide<true>(a.pol, bz, a.pol_has_state != 0, s.pol, pr, hidden, advance);
    } else {
        if (tid == 0) advance(-1);
    }
    if constexpr (POLL) {
        // Everything that was handed over has been read: clear it, written through like the words themselves.  By wavefronts that have
        // nothing else to do at the end, and where nothing loads any more (a wait for loads is one for these stores, too: 0.5 us
        // of a call with the prediction model).
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 zeros = {0, 0, 0, 0};
        const int idle = kExpThreads - kWave, from = MODE == kExpPolicy ? tid : tid - kWave, nlist = a.F * nslot * (int)sizeof(uint64_t), nsum = a.F * a.nchunks * 16;
        const auto lists = __builtin_amdgcn_make_buffer_rsrc(a.part_keys, 0, nlist, 0x00027000);
        const auto sums = __builtin_amdgcn_make_buffer_rsrc(a.part_lm, 0, nsum, 0x00027000);
        if (from >= 0 && from < idle) {
            for (int i = from * 16; i < nlist; i += idle * 16) __builtin_amdgcn_raw_buffer_store_b128(zeros, lists, i, 0, 16);
            for (int i = from * 16; i < nsum; i += idle * 16) __builtin_amdgcn_raw_buffer_store_b128(zeros, sums, i, 0, 16);
            if (MODE == kExpPolicy && a.pol_has_state && from < 4 * kPolH) store_shared_result(&a.gate_pre[from], 0.f);
        }
    }
}

// MODE: the plain expansion is compiled without any code for batches, cycle states or the prediction model.
// GENERAL: any number of chunks, rows and candidates at the call's end (launch_expand).
// A call is a chain of dependent stages, none of which is bound by bandwidth: F = 10, V = 128256, k = 10 takes 6.1 us per call on warm logits.
// (With lists announced by tickets once their stores were acknowledged 7.9; then 7.1, until the selections compared by sign bits and ranked what
// passes in parts, radar_topk.h: ten rows of 128257 with k = 16 12.2 -> 9.1, of 200000 16.8 -> 9.0.)  Lists longer than 16 slots need no ranking at
// all, but the last workgroup's loads are slow (from beyond its L2, 37 bytes per ns): 24 slots cost it 0.4 us, records of 32 0.7.
// The leading arguments are what the stream waits for; they are in registers when the kernel starts (0.25 us).
//
// Up to how many workgroups all count on one counter: they wait for each other there, some 10 ns each, but the last one is
// spared a second counter's round trip (by row first, then the rows).  Over 100 calls of 1 ... 10 rows, V = 32001 ... 400001, all on one counter costs
// 2-8 % where they are more (80 of 81 ... 256 workgroups), up to 96 or up to 48 is the same within 0.5 %.
constexpr int kDirectArrivals = 96;

struct ExpandKernArgs {                    // the argument segment of expand_kernel
    const float *logits;
    int F, V, k, nchunks, pool_count;
    radar_cycle_state *cycle;
    uint64_t *part_keys;
    unsigned int *counters;
    ExpandArgs a;
};
typedef ArgBlock<ExpandArgs> LateArgs;
__device__ __forceinline__ LateArgs late_args() { return args_from_here<ExpandArgs>(offsetof(ExpandKernArgs, a)); }
// What a call's end needs of them.
template <int MODE>
__device__ __forceinline__ ExpandArgs finish_args() {
    const LateArgs p = late_args();
    ExpandArgs a;
    a.parent_scores = p->parent_scores; a.parent_pool_idx = p->parent_pool_idx; a.cand_tokens = p->cand_tokens; a.cand_scores = p->cand_scores;
    a.frontier_pool_idx = p->frontier_pool_idx; a.frontier_tokens = p->frontier_tokens; a.frontier_scores = p->frontier_scores; a.frontier_conf = p->frontier_conf;
    a.pool_tokens = p->pool_tokens; a.pool_scores = p->pool_scores; a.pool_parents = p->pool_parents; a.pool_capacity = p->pool_capacity;
    a.part_lm = p->part_lm;
    if constexpr (MODE == kExpPolicy) {
        a.gate_pre = p->gate_pre; a.pol_has_state = p->pol_has_state;
        a.pol.w_ih = p->pol.w_ih; a.pol.w_hh = p->pol.w_hh; a.pol.b_ih = p->pol.b_ih; a.pol.b_hh = p->pol.b_hh;
        a.pol.w1 = p->pol.w1; a.pol.b1 = p->pol.b1; a.pol.w2 = p->pol.w2; a.pol.b2 = p->pol.b2;
        a.pol.h_in = p->pol.h_in; a.pol.c_in = p->pol.c_in; a.pol.uniforms = p->pol.uniforms; a.pol.h_out = p->pol.h_out; a.pol.c_out = p->pol.c_out;
        a.pol.logits = p->pol.logits; a.pol.probs = p->pol.probs; a.pol.action = p->pol.action; a.pol.k = p->pol.k; a.pol.M = p->pol.M;
    }
    return a;
}

template <bool VEC4, int EPT, int MODE, bool GENERAL>
__global__ __launch_bounds__(kExpThreads, 1) void expand_kernel(const float *logits, int F, int V, int k, int nchunks, int pool_count,
                                                                radar_cycle_state *cycle_, uint64_t *part_keys, unsigned int *counters,
                                                                ExpandArgs) {
    constexpr bool EXT = MODE != kExpPlain;
    struct { const float *logits; int F, V, k, nchunks, pool_count; radar_cycle_state *cycle; uint64_t *part_keys; unsigned int *counters; } a =
        {logits, F, V, k, nchunks, pool_count, cycle_, part_keys, counters};
    static_assert(EPT == 4 || EPT == 8 || EPT == 16, "EPT");
    static_assert(kFastCap <= kPickMost && kExpWaves == 16 && kStreamers == 4, "candidate list inside the selection scratch");
    constexpr int kChunk = kExpThreads * EPT;
    __shared__ ExpandSmem s;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int f = blockIdx.y, chunk = blockIdx.x;
    const int bz = EXT ? (int)blockIdx.z : 0;
    if (EXT && bz != 0) {                                // sequence bz's part of what the stream needs
        a.logits += (size_t)bz * F * V;
        a.counters += (size_t)bz * (kCounterBytes / sizeof(unsigned int));
        a.part_keys += (size_t)bz * F * nchunks * RADAR_K_MAX;
        if (a.cycle) a.cycle += bz;
    }
    radar_cycle_state *const cycle = EXT ? a.cycle : nullptr;
    // The first draft call of a cycle (the host says so: the largest count the state may hold is 0)
    // never reads the state; its last workgroup writes all of it.
    const bool cycle_first = cycle != nullptr && a.pool_count == 0;
    if (cycle && !cycle_first) {
        // A drafting cycle that has stopped skips its remaining draft calls: every workgroup leaves
        // before touching anything.  (The state is only written by the last workgroup of a launch,
        // after every other workgroup has handed over its results, i.e. long after this read.)
        const int pc = cycle->pool_count;
        if (cycle->stopped != 0 || pc < 0 || pc > a.pool_count) return;
        a.pool_count = pc;
    }
    const float *row = a.logits + (size_t)f * a.V;
    const int base = chunk * kChunk;
    const int K = a.k;
    // Who finishes the call: the workgroup that is counted last.  The others are running by then, or done, and wait for nobody, so it may wait
    // for what they hand over.  One lane of a wavefront that does not stream counts, beside the stream; few workgroups when their logits are
    // there (counted at the start, one row of V = 200000 7.14 us, so 6.74; counted beside the candidates 6.93).
    const bool direct = a.F * a.nchunks <= kDirectArrivals, counting = w == kExpWaves - 1 && lane == 0;
    unsigned int before = 0;
    if (counting && !direct) before = __hip_atomic_fetch_add(&a.counters[(1 + f) * kCounterStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- stream the chunk.  Only the first four wavefronts (one per SIMD) stream and select: a
    // 64-wide vector instruction occupies its SIMD for four cycles whichever wavefront issues it, so
    // four wavefronts with 4 * EPT logits per lane do the per-logit work in the same time as sixteen
    // with EPT each, and what a wavefront does once (reductions, threshold, list bookkeeping) is
    // done four times per workgroup instead of sixteen.  The other wavefronts only serve the end of
    // the call (one row each, the prediction model).  NE/4 x (256 lanes x 16 B) coalesced loads, all
    // issued before anything is computed from them (out-of-range lanes read a valid address and are
    // masked).
    constexpr int kSLanes = kStreamers * kWave;
    constexpr int NE = EPT * (kExpThreads / kSLanes);              // logits per streaming lane
    const bool streamer = w < kStreamers;
    const bool tail = base + kChunk > a.V;                         // the row ends inside this chunk
    float x[NE];
    if (streamer) {
        __builtin_amdgcn_s_setprio(3);                             // the others wait for these four
        float4 raw[NE / 4];
        if (VEC4) {
#pragma unroll
            for (int g = 0; g < NE / 4; ++g) {
                const int idx0 = base + g * (kSLanes * 4) + tid * 4;
                raw[g] = *reinterpret_cast<const float4 *>(row + (idx0 < a.V ? idx0 : 0));
            }
        } else if (a.V >= 4) {
#pragma unroll
            for (int g = 0; g < NE / 4; ++g) raw[g] = load4_of_row(row, base + g * (kSLanes * 4) + tid * 4, a.V);
        } else {
#pragma unroll
            for (int g = 0; g < NE / 4; ++g) raw[g] = load4_of_short_row(row, a.V);
        }
#pragma unroll
        for (int g = 0; g < NE / 4; ++g) {
            x[4 * g + 0] = raw[g].x; x[4 * g + 1] = raw[g].y; x[4 * g + 2] = raw[g].z; x[4 * g + 3] = raw[g].w;
        }
        if (tail) {
            if (!VEC4) place_row_end<NE / 4>([&](int g, int j) -> float & { return x[4 * g + j]; }, base + tid * 4, kSLanes * 4, a.V);
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int idx = base + (e >> 2) * (kSLanes * 4) + tid * 4 + (e & 3);
                x[e] = idx < a.V ? x[e] : -INFINITY;
            }
        }
    }
    // The prediction model's input-free part (w_hh h) is shared out over the workgroups of the
    // launch: its loads travel with the logits', and what is made of them, after the selection, is
    // handed to the last workgroup through the workspace like the chunk partials.  By the wavefronts that
    // do not stream.
    HiddenRows<2, 2 * (kExpWaves - kStreamers)> hrows;
    bool hidden_rows = false;
    PolicyArgs pol;
    float *gate_pre = nullptr;
    if (MODE == kExpPolicy && !streamer) {
        const LateArgs la = late_args();
        hidden_rows = la->pol_has_state != 0;
        pol.w_hh = la->pol.w_hh;
        pol.h_in = la->pol.h_in;
        gate_pre = la->gate_pre + (size_t)bz * (kCounterBytes / sizeof(float));
        if (hidden_rows) hrows.load(pol, bz, blockIdx.y * nchunks + blockIdx.x, nchunks * F, tid / 32 - 2 * kStreamers);
    }

    // ---- the threshold of the chunk's top-k: the k-th largest of the maxima of the 32 eight-lane groups of the
    // streaming wavefronts.  At least k logits of the chunk reach it (one per group whose maximum does), and on
    // untied data 1.2 k (k = 10) to 1.4 k (k = 16).  Everything here is a chain of latencies (a ballot whose
    // count a scalar instruction needs costs ~30 cycles, a lane read with a compare ~40, an LDS round trip
    // ~120), so every streaming wavefront finds the threshold by itself, in vector registers, and the
    // exponentials wait until the other wavefronts have something to do beside them.
    float lmax = -INFINITY;                                        // the lane's largest logit
    if (streamer) {
        lmax = x[0];
#pragma unroll
        for (int e = 1; e < NE; ++e) lmax = fmaxf(lmax, x[e]);
        float gm = lmax;
        gm = fmaxf(gm, dpp_f32<0xB1>(gm));
        gm = fmaxf(gm, dpp_f32<0x4E>(gm));
        gm = fmaxf(gm, dpp_f32<0x141>(gm));                        // every lane: the maximum of its eight lanes
        if ((lane & 7) == 0) s.gmax[w * 8 + (lane >> 3)] = gm;
    }
    if (tid == 0) s.nsurv = 0;
    __syncthreads();
    // Lanes whose largest logit reaches the threshold (about 1.2 k of the 256) leave all their logits
    // in LDS; only those are compared one by one afterwards.
    float *const dump = reinterpret_cast<float *>(&s.wtk[1]);      // [kStreamers][kDumpCap][NE], inside the selection scratch
    uint64_t *const surv = s.wtk[0].surv;                          // complements; room for kFastCap + kPickPad
    static_assert(kStreamers * kDumpCap * NE * sizeof(float) <= (kExpWaves - 1) * sizeof(WaveTopkSmem), "dump inside the scratch");
    float cm = 0.f;                                                // chunk maximum (streamers)
    if (streamer) {
        const float g32 = s.gmax[lane & 31];
        const float tau = kth_threshold(g32, K);
        const bool hot = lmax >= tau && base + tid * 4 < a.V;      // (a lane wholly past the row holds -inf only)
        const uint64_t hm = __ballot(hot);
        if (hot) {
            const int at = lanes_below(hm);
            if (at < kDumpCap) {
                float4 *d4 = reinterpret_cast<float4 *>(dump + (size_t)(w * kDumpCap + at) * NE);
#pragma unroll
                for (int g = 0; g < NE / 4; ++g) d4[g] = make_float4(x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]);
                s.dump_lane[w][at] = (unsigned char)lane;
            }
        }
        if (lane == 0) s.ndump[w] = (unsigned int)__popcll(hm);
        if (tid == 0) s.tau = tau;
        cm = fmaxf(g32, dpp_f32<0xB1>(g32));
        cm = fmaxf(cm, dpp_f32<0x4E>(cm));
        cm = fmaxf(cm, dpp_f32<0x141>(cm));
        cm = fmaxf(cm, dpp_f32<0x140>(cm));
        const auto c2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(cm), __float_as_uint(cm), false, false);
        cm = fmaxf(__uint_as_float(c2[0]), __uint_as_float(c2[1]));
    } else {
        if (counting && direct) before = __hip_atomic_fetch_add(&a.counters[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // The arguments that only the call's end needs are brought close by now: read by the last workgroup when it
        // gets there, each cache line of them would be a round trip of its own (0.3 us).
        const auto la = (const __attribute__((address_space(4))) int *)late_args();
        static_assert(sizeof(ExpandArgs) > 4 * 64 && sizeof(ExpandArgs) <= 5 * 64, "cache lines of the arguments");
        asm volatile("" :: "s"(la[0]), "s"(la[16]), "s"(la[32]), "s"(la[48]), "s"(la[64]));
        if (counting && !direct)                                   // the last one of the row counts the row
            before = before == (unsigned int)(a.nchunks - 1) ? __hip_atomic_fetch_add(&a.counters[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0u;
    }
    __syncthreads();
    if (streamer) {
        // ---- sum of exp(x - chunk maximum): fp32 exponentials; a lane adds its terms in fp32 chains of at most eight, as the
        // streaming kernel does, the rest is fp64 in a fixed order.
        // (x - cm) first: folding the scale into one fused multiply-add would round cm * log2(e), an
        // absolute error in the exponent that grows with |cm|.
        constexpr int kChains = NE > 32 ? NE / 8 : 4;
        float tl[kChains] = {};
        if (cm > -INFINITY) {
#pragma unroll
            for (int e = 0; e < NE; ++e) tl[e % kChains] += __builtin_amdgcn_exp2f((x[e] - cm) * kLog2eF);
        }
        double ll = ((double)tl[0] + (double)tl[1]) + ((double)tl[2] + (double)tl[3]);
        if constexpr (kChains == 8) ll += ((double)tl[4] + (double)tl[5]) + ((double)tl[6] + (double)tl[7]);
        const double wl = wave_sum_f64(ll);
        if (lane == 0) s.wave_l[w] = wl;
        if (tid == 0) s.cmax = cm;
        __builtin_amdgcn_s_setprio(0);
    } else {
        // ---- Meanwhile the logits of the hot lanes against the threshold, three wavefronts to each streaming one: a
        // lane takes one logit of one block; what passes is a candidate (their order is immaterial).
        constexpr int kReaders = (kExpWaves - kStreamers) / kStreamers;
        constexpr int kPerWave = NE <= kWave ? kWave / NE : 1;     // blocks a wavefront takes at a time
        const int from = w % kStreamers, ndump = (int)s.ndump[from];
        const float tau_f = s.tau;
        if (ndump > kDumpCap) {                                    // long runs of equal values
            if (w < 2 * kStreamers && lane == 0) atomicAdd(&s.nsurv, kFastCap + 1u);
        } else {
            for (int d0 = (w / kStreamers - 1) * kPerWave; d0 < ndump; d0 += kReaders * kPerWave) {
#pragma unroll
                for (int e1 = 0; e1 < NE; e1 += kWave) {           // (one round unless a lane streams more than 64 logits)
                    const int d = d0 + (NE <= kWave ? lane / NE : 0);
                    const int e = NE <= kWave ? lane % NE : e1 + lane;
                    const int slot = from * kDumpCap + min(d, ndump - 1);
                    const float v = dump[(size_t)slot * NE + e];
                    const int src = from * kWave + (int)(&s.dump_lane[0][0])[slot];
                    const int idx = base + (e >> 2) * (kSLanes * 4) + src * 4 + (e & 3);
                    const uint64_t m = __ballot(d < ndump && v >= tau_f && idx < a.V);
                    if (m != 0) {
                        int at = 0;
                        if (lane == 0) at = (int)atomicAdd(&s.nsurv, (unsigned int)__popcll(m));
                        at = (int)readlane_u32((uint32_t)at, 0) + lanes_below(m);
                        if (((m >> lane) & 1) && at < kFastCap) surv[at] = ~pick_key(v, uint32_t(idx));
                    }
                }
            }
        }
        if (counting) s.last = before == (unsigned int)((direct ? a.F * a.nchunks : a.F) - 1);
    }
    __syncthreads();
    const size_t pslot = (size_t)f * a.nchunks + chunk;
    uint64_t *const list = a.part_keys + pslot * RADAR_K_MAX;
    const int nsurv = (int)s.nsurv;
    if (nsurv > kFastCap || nsurv < min(K, a.V - base)) {
        // Long runs of equal values (more candidates than the list holds), or NaNs (fewer than the chunk has to give, so that a
        // row would not have K of them): every streaming wavefront
        // ranks its own logits exactly, four per lane at a time with the selection so far riding
        // along, then one wavefront the four selections.  The logits are read again (a rolled loop
        // over registers would index them dynamically); this path only runs on heavily tied rows and rows of NaN, which rank by their bits here.
        if (streamer) {
            if (lane < RADAR_K_MAX) s.wlist[w * RADAR_K_MAX + lane] = 0;
            uint64_t k5[5] = {0, 0, 0, 0, 0};
#pragma unroll 1
            for (int g = 0; g <= NE / 4; ++g) {
                if (g == NE / 4) {
                    __syncthreads();
                    if (w != 0) break;
                    k5[0] = s.wlist[lane];
                    k5[1] = k5[2] = k5[3] = k5[4] = 0;
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int idx = base + g * (kSLanes * 4) + tid * 4 + u;
                        const float v = row[min(idx, a.V - 1)];
                        k5[u] = idx < a.V ? key_of_any(v, uint32_t(idx)) : 0;
                    }
                }
                const Picked p = wave_pick<5>(k5, K, s.wtk[w]);
                k5[4] = carried(p, K);
                uint64_t *const best = s.wlist + w * RADAR_K_MAX;
                if (g >= NE / 4 - 1 && p.rank < K) best[p.rank] = p.key;
            }
        } else {
            __syncthreads();
        }
        if (w == 0) {
            wave_lds_sync();
            if (lane < RADAR_K_MAX) store_shared_result(list + lane, (lane < K ? s.wlist[lane] : 0) | kThere);
        }
    } else if (w == 0 && nsurv <= RADAR_K_MAX) {
        // the candidates as they are: the finishing workgroup ranks them with the other chunks'
        if (lane < RADAR_K_MAX) store_shared_result(list + lane, lane < nsurv ? ~surv[lane] | kThere : kThere);
    } else if (w == 0) {
        // more candidates than slots (k = 10: one chunk in a hundred; k above 12: most): the k best of them
        const Picked p = rank_survivors(surv, s.wtk[0].top, nsurv, K);
        if (p.rank < K) store_shared_result(list + p.rank, p.key | kThere);          // ranks are distinct
        if (lane >= K && lane < RADAR_K_MAX) store_shared_result(list + lane, kThere);
    }
    if (w == 1) {
        double l = 0.0;                                            // fixed order of addition
#pragma unroll
        for (int i = 0; i < kStreamers; ++i) l += s.wave_l[i];
        uint64_t *const part_lm = late_args()->part_lm + (size_t)bz * F * nchunks * 2;
        if (lane < 2)
            store_shared_result(&part_lm[pslot * 2 + lane], lane == 0 ? (uint64_t)__double_as_longlong(l) | kThere : uint64_t(1) << 32 | __float_as_uint(s.cmax));
    }
    // (Here, because nothing waits for it soon: before the candidates it held up their barrier by 0.6 us, in a call of few workgroups, which
    // have more rows each, by 1.2.)
    if (hidden_rows) hrows.finish(pol, bz, [&](int r, float v) { store_shared_result(&gate_pre[r], __float_as_uint(v) == 0 ? -0.f : v); });
    if (!s.last) return;
    if (tid <= a.F) store_shared_result(&a.counters[tid * kCounterStride], 0u);      // (all have counted)

    // ================= the workgroup that finishes the call
    ExpandArgs fin = finish_args<MODE>();
    fin.logits = logits; fin.F = F; fin.V = V; fin.k = k; fin.nchunks = nchunks; fin.cycle = cycle_; fin.part_keys = part_keys; fin.counters = counters;
    if (EXT && bz != 0) sequence_view(fin, bz);
    fin.pool_count = a.pool_count;
    expand_finish<MODE, true, GENERAL>(fin, s, bz, cycle, cycle_first, [] { return true; },
                        [&](int row) { return load_shared_result(&fin.gate_pre[row]); });
}

// ------------------------------------------------------------------ rerank
struct RerankArgs {
    const int32_t *pool_tokens;
    const float *pool_scores;
    const int32_t *pool_parents;
    int pool_count, N, root_token;
    const radar_cycle_state *cycle;   // or null; when set, pool_count is the state's, clamped to the value above
    const int32_t *root_tokens;       // batched call: one root token per sequence (else null: root_token)
    int pool_capacity;                // batched call: stride of the pool arrays
    int32_t *tree_tokens;
    int32_t *tree_parents;
    float *tree_scores;
    int32_t *tree_depth;
    int32_t *tree_pool_idx;
    int32_t *n_nodes_out;
};

constexpr int kRerankStaged = 4 * kTopkThreads;       // pools up to this size are copied to LDS whole

struct RerankSmem {
    TopkSmem topk;
    int16_t node_of[RADAR_POOL_MAX];     // pool index -> node number, -1 if dropped
    // small pools: tokens, parents and scores ride along with the first loads, so that the kept
    // entries are read from LDS instead of a second round trip to memory
    int32_t tok[kRerankStaged], par[kRerankStaged];
    float sc[kRerankStaged];
};

template <int EPT>                       // pool entries per lane: 4 (pools up to 1024) or 16
__global__ __launch_bounds__(kTopkThreads) void rerank_kernel(const float *pool_scores, const int32_t *pool_tokens, const int32_t *pool_parents,
                                                              const radar_cycle_state *cycle, int pool_count, int N, int pool_capacity, int root_token, RerankArgs a) {
    a.pool_scores = pool_scores; a.pool_tokens = pool_tokens; a.pool_parents = pool_parents; a.cycle = cycle;
    a.pool_count = pool_count; a.N = N; a.pool_capacity = pool_capacity; a.root_token = root_token;
    __shared__ RerankSmem s;
    const int tid = threadIdx.x;
    if (blockIdx.x != 0) {                               // sequence b of a batched call: every array has a leading batch dimension
        const size_t b = blockIdx.x, n1 = (size_t)a.N + 1;
        a.pool_tokens += b * a.pool_capacity; a.pool_scores += b * a.pool_capacity; a.pool_parents += b * a.pool_capacity;
        a.tree_tokens += b * n1; a.tree_parents += b * n1; a.tree_scores += b * n1;
        a.tree_depth += b * n1; a.tree_pool_idx += b * n1;
        a.n_nodes_out += b;
        if (a.cycle) a.cycle += b;
    }
    // All loads first, one round trip.  A cycle's own count comes with them where the pool is known to reach to the
    // host's (a batched call's capacity), else before them: the host's count only bounds the state's then.
    const bool late_count = a.cycle != nullptr && a.pool_capacity > 0;
    if (a.cycle && !late_count) a.pool_count = min(max(a.cycle->pool_count, 0), a.pool_count);
    constexpr bool kStaged = EPT * kTopkThreads <= kRerankStaged;
    uint64_t keys[EPT];
    float sc0[EPT];
    int tk[EPT], pr[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = max(0, min(tid + e * kTopkThreads, a.pool_count - 1));
        sc0[e] = a.pool_scores[i];
        if constexpr (kStaged) { tk[e] = a.pool_tokens[i]; pr[e] = a.pool_parents[i]; }
    }
    if (a.root_tokens) a.root_token = a.root_tokens[blockIdx.x];
    if (late_count) a.pool_count = min(max(a.cycle->pool_count, 0), a.pool_count);
    const int keep = min(a.N, a.pool_count);
    asm volatile("" :: "s"(a.tree_tokens), "s"(a.n_nodes_out));
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = tid + e * kTopkThreads;
        keys[e] = (i < a.pool_count) ? make_key(sc0[e], uint32_t(i)) : 0;
        if constexpr (kStaged) { s.sc[i] = sc0[e]; s.tok[i] = tk[e]; s.par[i] = pr[e]; }
    }
    for (int i = tid; i < a.pool_count; i += kTopkThreads) s.node_of[i] = -1;
    if (keep > 0) block_topk<EPT>(keys, keep, s.topk);
    else __syncthreads();

    int my_pool = -1;
    if (tid >= 1 && tid <= keep) {
        const uint64_t key = s.topk.top[tid - 1];
        my_pool = (int)key_index(key);
        if (key == 0 || my_pool < 0 || my_pool >= a.pool_count) my_pool = 0;   // only reachable with NaN scores
        s.node_of[my_pool] = (int16_t)tid;
    }
    __syncthreads();
    if (tid >= kWave) return;                            // the tree has at most 64 nodes: one per lane of one wavefront
    int tok = -1, par = -1, pidx = -1;
    float sc = 0.f;
    if (tid == 0) { tok = a.root_token; }
    else if (tid <= keep) {
        tok = kStaged ? s.tok[my_pool] : a.pool_tokens[my_pool];
        sc = kStaged ? s.sc[my_pool] : a.pool_scores[my_pool];
        pidx = my_pool;
        const int pp = kStaged ? s.par[my_pool] : a.pool_parents[my_pool];
        if (pp < 0) par = 0;
        else if (pp < a.pool_count && s.node_of[pp] >= 0 && s.node_of[pp] < tid) par = s.node_of[pp];
        else par = -2;
    }
    // Depths by doubling: an ancestor's distance to its own ancestor is added until all have reached the root, or a
    // node without a parent in the tree (which has depth 0, and so have all below it).
    int up = par >= 0 ? par : tid, depth = par >= 0 ? 1 : 0, lost = par == -2 ? 1 : 0;
    for (int r = 1; r < RADAR_T_MAX; r *= 2) {
        const int there = __shfl(up | depth << 8 | lost << 16, up);
        const bool moved = (there & 0xff) != up;
        depth += there >> 8 & 0xff;
        lost |= there >> 16;
        up = there & 0xff;
        if (__ballot(moved) == 0) break;
    }
    if (tid <= a.N) {
        a.tree_tokens[tid] = tok;
        a.tree_parents[tid] = par;
        a.tree_scores[tid] = sc;
        a.tree_pool_idx[tid] = pidx;
        a.tree_depth[tid] = lost ? 0 : depth;
    }
    if (tid == 0) *a.n_nodes_out = 1 + keep;
}

// ------------------------------------------------------------------ large batches: stream, then finish
// For many sequences per call the single launch above is bound by what every workgroup does around
// its share of the stream (one workgroup per CU, hand-over and ticket per chunk).  Two launches
// instead: a streaming kernel of small workgroups (several per CU, out of step with each other)
// without tickets or hand-over, each of which leaves one top-k list, maximum and sum of exponentials per
// 8192 logits in the workspace, then one workgroup per sequence that does what the last workgroup of the single
// launch does.  (Per 4096 logits the stream paid for its barriers and bookkeeping twice as often, and rows of more than
// 65536 logits were merged the long way: F = 10, V = 128256, 4 / 16 / 64 sequences 12.1 / 21.7 / 61.7 us, now 10.6 /
// 20.3 / 59.5, the last 5.5 TB/s.)
constexpr int kStreamThreads = 256;
constexpr int kStreamWaves = kStreamThreads / kWave;
constexpr int kStreamEPT = 32;                                     // logits per lane
constexpr int kStreamChunk = kStreamThreads * kStreamEPT;

// true: the sequence's cycle has stopped (or its state is out of range) and the call leaves it alone
__device__ __forceinline__ bool cycle_skips(const radar_cycle_state *st, int pool_count_max, int *pool_count) {
    if (st == nullptr || pool_count_max == 0) return false;        // no cycle, or its first call
    const int pc = st->pool_count;
    if (st->stopped != 0 || pc < 0 || pc > pool_count_max) return true;
    *pool_count = pc;
    return false;
}

// Lanes of a wavefront whose logits go through LDS.  With k = 16 a chunk has 22 of them on average and one wavefront in some thousands more
// than sixteen, which costs the call the exact ranking.
constexpr int kStreamHot = 24;
constexpr int kStreamCap = 128;                                    // candidates of a chunk; more (runs of equal values) rank per wavefront

struct StreamFast {
    alignas(16) float dump[kStreamWaves][kStreamHot * kStreamEPT];
    alignas(16) uint64_t surv[kStreamCap + kPickPad];              // complements
    uint64_t top[16];
    unsigned char lane_of[kStreamWaves][kStreamHot];
};

template <bool VEC4>
__global__ __launch_bounds__(kStreamThreads, 8) void expand_stream_kernel(const float *logits, int F, int V, int k, int nchunks, int pool_count,
                                                                         radar_cycle_state *cycle, int has_policy, int pol_has_state, ExpandArgs a) {
    a.logits = logits; a.F = F; a.V = V; a.k = k; a.nchunks = nchunks; a.pool_count = pool_count; a.cycle = cycle;
    a.has_policy = has_policy; a.pol_has_state = pol_has_state;
    constexpr int EPT = kStreamEPT;
    __shared__ union {
        StreamFast fast;
        struct {
            WaveTopkSmem wtk[kStreamWaves];
            uint64_t wlist[kStreamWaves * RADAR_K_MAX];
        } ties;
    } s;
    __shared__ float gmax[8 * kStreamWaves];                       // maxima of the 32 eight-lane groups
    __shared__ double wave_l[kStreamWaves];
    __shared__ unsigned int nsurv;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int row = blockIdx.y;                                    // sequence * F + frontier row
    int unused;
    if (cycle_skips(a.cycle ? a.cycle + row / a.F : nullptr, a.pool_count, &unused)) return;   // the whole workgroup
    // EPT logits per lane, four at a time and all wavefronts side by side: where a row ends inside the chunk,
    // every wavefront still has some of it
    const int base = blockIdx.x * kStreamChunk;
    const float *rowp = a.logits + (size_t)row * a.V;
    const int K = a.k;
    float4 raw[EPT / 4];
#pragma unroll
    for (int g = 0; g < EPT / 4; ++g) {
        const int idx0 = base + g * (kStreamThreads * 4) + tid * 4;
        raw[g] = VEC4 ? *reinterpret_cast<const float4 *>(rowp + (idx0 < a.V ? idx0 : 0)) : load4_of_row(rowp, idx0, a.V);   // (V >= 64)
    }
    float x[EPT];
#pragma unroll
    for (int g = 0; g < EPT / 4; ++g) {
        x[4 * g + 0] = raw[g].x; x[4 * g + 1] = raw[g].y; x[4 * g + 2] = raw[g].z; x[4 * g + 3] = raw[g].w;
    }
    if (base + kStreamChunk > a.V) {                               // the row's last chunk only
        if (!VEC4) place_row_end<EPT / 4>([&](int g, int j) -> float & { return x[4 * g + j]; }, base + tid * 4, kStreamThreads * 4, a.V);
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int idx = base + (e >> 2) * (kStreamThreads * 4) + tid * 4 + (e & 3);
            x[e] = idx < a.V ? x[e] : -INFINITY;
        }
    }
    // ---- the maxima of the 32 eight-lane groups: the chunk's maximum, and as threshold of its top-k their k-th largest (at least k logits of the
    // chunk reach it, one per group whose maximum does; on untied data 1.2 k to 1.4 k. Of sixteen groups the 16th largest is the smallest, which lets
    // the whole chunk through: 64 sequences of 16 rows, V = 32000, k = 16 took 57 us instead of 30.)
    float tm = x[0];
#pragma unroll
    for (int e = 1; e < EPT; ++e) tm = fmaxf(tm, x[e]);
    float gm = tm;
    gm = fmaxf(gm, dpp_f32<0xB1>(gm));
    gm = fmaxf(gm, dpp_f32<0x4E>(gm));
    gm = fmaxf(gm, dpp_f32<0x141>(gm));
    if ((lane & 7) == 0) gmax[w * 8 + (lane >> 3)] = gm;
    if (threadIdx.x == 0) nsurv = 0;
    __syncthreads();
    const float g32 = gmax[lane & 31];
    float cm = g32;
    cm = fmaxf(cm, dpp_f32<0xB1>(cm));
    cm = fmaxf(cm, dpp_f32<0x4E>(cm));
    cm = fmaxf(cm, dpp_f32<0x141>(cm));
    cm = fmaxf(cm, dpp_f32<0x140>(cm));
    const auto c2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(cm), __float_as_uint(cm), false, false);
    cm = fmaxf(__uint_as_float(c2[0]), __uint_as_float(c2[1]));
    float tl[4] = {0.f, 0.f, 0.f, 0.f};                            // four fp32 chains of eight terms, fp64 from there on
    if (cm > -INFINITY) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) tl[e & 3] += __builtin_amdgcn_exp2f((x[e] - cm) * kLog2eF);
    }
    const double wl = wave_sum_f64(((double)tl[0] + (double)tl[1]) + ((double)tl[2] + (double)tl[3]));
    if (lane == 0) wave_l[w] = wl;
    const float tau = kth_threshold(g32, K);

    // ---- Lanes whose largest logit reaches the threshold (1.2 k to 1.4 k of the 256) leave all their logits in
    // LDS; their wavefront compares those one per lane and appends what passes to the chunk's list.  (A
    // threshold per wavefront and a comparison of every logit with it were 150 instructions, a sixth of the time.)
    const bool hot = tm >= tau && base + tid * 4 < a.V;           // (a lane wholly past the row holds -inf only)
    const uint64_t hm = __ballot(hot);
    const int nhot = __popcll(hm);
    if (nhot > kStreamHot) {
        if (lane == 0) atomicAdd(&nsurv, kStreamCap + 1u);         // long runs of equal values
    } else if (nhot > 0) {
        float *const dump = s.fast.dump[w];
        if (hot) {
            const int at = lanes_below(hm);
            float4 *d4 = reinterpret_cast<float4 *>(dump + at * EPT);
#pragma unroll
            for (int g = 0; g < EPT / 4; ++g) d4[g] = make_float4(x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]);
            s.fast.lane_of[w][at] = (unsigned char)lane;
        }
        wave_lds_sync();
        for (int d0 = 0; d0 < nhot; d0 += kWave / EPT) {           // two or four lanes' logits at a time
            const int d = d0 + lane / EPT, e = lane % EPT;
            const bool live = d < nhot;
            const float v = dump[min(d, nhot - 1) * EPT + e];
            const int idx = base + (e >> 2) * (kStreamThreads * 4) + (w * kWave + (int)s.fast.lane_of[w][min(d, nhot - 1)]) * 4 + (e & 3);
            const uint64_t m = __ballot(live && v >= tau && idx < a.V);
            if (m != 0) {
                int at = 0;
                if (lane == 0) at = (int)atomicAdd(&nsurv, (unsigned int)__popcll(m));
                at = (int)readlane_u32((uint32_t)at, 0) + lanes_below(m);
                if (((m >> lane) & 1) && at < kStreamCap) s.fast.surv[at] = ~pick_key(v, uint32_t(idx));
            }
        }
    }
    __syncthreads();
    const size_t slot = (size_t)row * a.nchunks + blockIdx.x;
    const int n = (int)nsurv;
    if (n > kStreamCap || n < min(K, a.V - base)) {
        // Long runs of equal values, or NaNs: every wavefront ranks its own logits exactly, then one ranks the four lists.
        __syncthreads();                                           // the short path's LDS is overlaid
        if (lane < RADAR_K_MAX) s.ties.wlist[w * RADAR_K_MAX + lane] = 0;
        uint64_t k5[5] = {0, 0, 0, 0, 0};
#pragma unroll 1
        for (int g = 0; g <= EPT / 4; ++g) {
            if (g == EPT / 4) {
                __syncthreads();
                if (w != 0) break;
                k5[0] = s.ties.wlist[lane];
                k5[1] = k5[2] = k5[3] = k5[4] = 0;
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {                      // (read again: a rolled loop would index the registers dynamically)
                    const int idx = base + g * (kStreamThreads * 4) + tid * 4 + u;
                    const float v = rowp[min(idx, a.V - 1)];
                    k5[u] = idx < a.V ? key_of_any(v, uint32_t(idx)) : 0;
                }
            }
            const Picked p = wave_pick<5>(k5, K, s.ties.wtk[w]);
            k5[4] = carried(p, K);
            if (g >= EPT / 4 - 1 && p.rank < K) s.ties.wlist[w * RADAR_K_MAX + p.rank] = p.key;
        }
        if (w == 0) {
            wave_lds_sync();
            if (lane < RADAR_K_MAX) a.part_keys[slot * RADAR_K_MAX + lane] = lane < K ? s.ties.wlist[lane] : 0;
        }
    } else if (w == 0 && n <= RADAR_K_MAX) {
        // the candidates as they are: the finishing workgroup ranks them with the other chunks'
        if (lane < RADAR_K_MAX) a.part_keys[slot * RADAR_K_MAX + lane] = lane < n ? ~s.fast.surv[lane] : 0;
    } else if (w == 0) {
        // more than that: the k best
        const Picked p = rank_survivors(s.fast.surv, s.fast.top, n, K);
        if (p.rank < K) a.part_keys[slot * RADAR_K_MAX + p.rank] = p.key;
        if (lane >= K && lane < RADAR_K_MAX) a.part_keys[slot * RADAR_K_MAX + lane] = 0;
    }
    if (w == 1 && lane == 0) {                                     // fixed order of addition
        double l = 0.0;
#pragma unroll
        for (int i = 0; i < kStreamWaves; ++i) l += wave_l[i];
        a.part_lm[slot * 2] = (uint64_t)__double_as_longlong(l) & ~kThere;
        a.part_lm[slot * 2 + 1] = __float_as_uint(cm);
    }
    // The prediction model's input-free part (w_hh h) of this row's sequence is shared out over the sequence's workgroups, as the single launch does;
    // the finish kernel reads it.  Here, because in front of the logits it held them up by a round trip (V = 128256, 16 sequences of ten rows, eight
    // calls 147.2 us, now 146.0; 30 of four rows, six calls 91.4 and 88.3).  By the two wavefronts that have no list to write, one or two rows a
    // lane; where a sequence has few workgroups, hence more rows for each, by all four (40 sequences of ten rows of 8190, six calls 79 us, by two
    // 82).
    if (a.has_policy && a.pol_has_state) {
        const int bz = row / a.F, part = (row - bz * a.F) * gridDim.x + blockIdx.x, parts = a.F * gridDim.x;
        float *const gate = a.gate_pre + (size_t)bz * (kCounterBytes / sizeof(float));
        auto rows = [&](auto hrows, int hwave) {
            hrows.load(a.pol, bz, part, parts, hwave);
            hrows.finish(a.pol, bz, [&](int r, float v) { gate[r] = v; });
        };
        if (parts < 64) rows(HiddenRows<4, 2 * kStreamWaves>{}, tid / 32);
        else if (w >= kStreamWaves / 2) rows(HiddenRows<2, kStreamWaves>{}, tid / 32 - kStreamWaves);
    }
}

// one workgroup per sequence, after expand_stream_kernel
template <int MODE, bool GENERAL>
__global__ __launch_bounds__(kExpThreads, 1) void expand_finish_kernel(uint64_t *part_keys, uint64_t *part_lm, int F, int nchunks,
                                                                       int k, int pool_count, radar_cycle_state *cycle_, ExpandArgs a) {
    a.part_keys = part_keys; a.part_lm = part_lm;
    a.F = F; a.nchunks = nchunks; a.k = k; a.pool_count = pool_count; a.cycle = cycle_;
    __shared__ ExpandSmem s;
    const int bz = blockIdx.x;
    if (bz != 0) sequence_view(a, bz);
    radar_cycle_state *const cycle = a.cycle;
    const bool cycle_first = cycle != nullptr && a.pool_count == 0;
    // (the prediction model's input-free part was left in the workspace by the streaming kernel)
    expand_finish<MODE, false, GENERAL>(a, s, bz, cycle, cycle_first, [&] { return !cycle_skips(cycle, a.pool_count, &a.pool_count); },
                        [&](int row) { return a.gate_pre[row]; });
}

}  // namespace radar

using namespace radar;

// Logits per lane: the fewest (shortest critical path per workgroup) that keep the launch at one
// workgroup per CU and a row at as many chunks as are merged the short way, as far as there are such (a call over one row
// of V = 128256 in 16 chunks takes 7.0 us, of V = 262144 in 16 instead of 64 chunks 7.0 instead of 8.0); launches too
// large for that take the most, i.e. the fewest workgroups.
static int plan_expand_ept(int F, int V) {
    for (const int most : {kFewChunks, kExpMaxChunks})
        for (int ept = kExpMinEPT; ept <= 16; ept *= 2) {
            const int64_t chunk = (int64_t)kExpThreads * ept, nchunks = ((int64_t)V + chunk - 1) / chunk;
            if (F * nchunks <= kRound && nchunks <= most) return ept;
        }
    return 16;
}

// Workspace of a call over B sequences: [B] counter blocks, [B][F][chunks] chunk lists, then [B][F][chunks] sums and maxima: kPartBytes for
// each chunk of the call's plan.  The size that callers are given goes by 4096 logits (the smallest chunk of any plan) at kSizedBytes each, and
// kSpareBytes per sequence; callers keep it and the call without a workspace is limited by it, so it stays as it is.  It covers every layout:
//   - chunks of 4096 are planned for at most kRound workgroups, which take 4 bytes each out of the spare ones;
//   - larger ones are at most two for three of 4096 where a row has several, and one per row out of the spare bytes where it has one.
constexpr size_t kPartBytes = (RADAR_K_MAX + 2) * sizeof(uint64_t), kSizedBytes = 140, kSpareBytes = 2048;
static_assert(kRound * (kPartBytes - kSizedBytes) <= kSpareBytes && RADAR_F_MAX * (kPartBytes - kSizedBytes) <= kSpareBytes &&
              2 * kPartBytes <= 3 * kSizedBytes && kStreamChunk >= 2 * kExpThreads * kExpMinEPT, "every layout inside the workspace");

static size_t expand_workspace_bytes(const radar_expand_desc *d, size_t B) {
    if (!d || d->F < 1 || d->V < 1 || B < 1) return 0;
    const size_t per_chunk = (size_t)kExpThreads * kExpMinEPT;
    const size_t nchunks = ((size_t)d->V + per_chunk - 1) / per_chunk;
    auto round_up = [](size_t bytes) { return (bytes + 255) & ~size_t(255); };
    return round_up(B * kCounterBytes + B * d->F * nchunks * kSizedBytes) + round_up(B * kSpareBytes);
}

extern "C" size_t radar_draft_expand_workspace_bytes(const radar_expand_desc *d) { return expand_workspace_bytes(d, 1); }

extern "C" size_t radar_draft_expand_batch_workspace_bytes(const radar_expand_desc *d, int32_t B) {
    return B < 1 ? 0 : expand_workspace_bytes(d, (size_t)B);
}

namespace radar { radar_status policy_args_from(const radar_policy_params *pp, PolicyArgs *out); }

static radar_status launch_expand(const float *logits, const float *parent_scores,
                                  const int32_t *parent_pool_idx, int32_t *cand_tokens, float *cand_scores,
                                  int32_t *frontier_pool_idx, int32_t *frontier_tokens,
                                  float *frontier_scores, float *frontier_conf, int32_t *pool_tokens,
                                  float *pool_scores, int32_t *pool_parents, const radar_expand_desc *d,
                                  const PolicyArgs *pol, radar_cycle_state *cycle, int B, void *workspace,
                                  size_t workspace_bytes, void *stream_, bool check_only = false) {
    if (!d || !logits || !parent_scores || !parent_pool_idx || !cand_tokens || !cand_scores || !frontier_pool_idx ||
        !frontier_tokens || !frontier_scores || !frontier_conf || !pool_tokens || !pool_scores || !pool_parents ||
        !workspace)
        return RADAR_INVALID_ARG;
    if (d->F < 1 || d->V < 1 || d->k < 1 || d->k > d->V || d->pool_count < 0 ||
        (int64_t)d->pool_count + (int64_t)d->F * d->k > (int64_t)d->pool_capacity)
        return RADAR_INVALID_ARG;
    if (B < 1) return RADAR_INVALID_ARG;
    if (B > 65535) return RADAR_UNSUPPORTED_SHAPE;
    const bool vec4 = (d->V % 4 == 0) && (((uintptr_t)logits & 15) == 0);
    const int ept = plan_expand_ept((int)std::min<int64_t>((int64_t)d->F * B, 1 << 20), d->V);
    // Batches whose single launch would take more than one round of the chip stream.  In one round the single launch is the faster one at any size
    // (ten rows of V = 128256, three sequences 7.1 us per call, streamed 9.0; four rows of 8190, 64 sequences 4.9 and 7.2), the second round starts
    // behind the whole first (eight rows of 50257: 320 workgroups 10.5 and 9.7, 480 13.4 and 11.1).  Where sequences may have stopped, which the host
    // does not know, the line is a quarter of a round further out: 300 workgroups of which some leave at once 0.91 ... 1.07 of the streamed time, 384
    // 1.09 ... 0.86.
    const int64_t groups = (int64_t)B * d->F * (((int64_t)d->V + kExpThreads * ept - 1) / (kExpThreads * ept));
    const int64_t line = cycle != nullptr && d->pool_count > 0 ? kRound + kRound / 4 : kRound;
    const bool stream = B > 1 && (int64_t)B * d->F <= 65535 &&
                        (d->V >= kStreamThreads * 4 ? groups > line : (int64_t)B * d->F * d->V >= kStreamMinLogits);
    const int64_t chunk = stream ? kStreamChunk : (int64_t)kExpThreads * ept;
    const int64_t nchunks = ((int64_t)d->V + chunk - 1) / chunk;
    if (d->F > RADAR_F_MAX || d->k > RADAR_K_MAX || nchunks > kExpMaxChunks) return RADAR_UNSUPPORTED_SHAPE;
    const size_t cbytes = (size_t)B * kCounterBytes, nslots = (size_t)B * d->F * nchunks;
    if (workspace_bytes < expand_workspace_bytes(d, (size_t)B) || workspace_bytes < cbytes + nslots * kPartBytes) return RADAR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)workspace & 255) != 0) return RADAR_INVALID_ARG;
    if (check_only) return RADAR_OK;                               // every argument is acceptable; nothing launched

    ExpandArgs a;
    a.logits = logits; a.parent_scores = parent_scores; a.parent_pool_idx = parent_pool_idx;
    a.cand_tokens = cand_tokens; a.cand_scores = cand_scores;
    a.frontier_pool_idx = frontier_pool_idx; a.frontier_tokens = frontier_tokens;
    a.frontier_scores = frontier_scores; a.frontier_conf = frontier_conf;
    a.pool_tokens = pool_tokens; a.pool_scores = pool_scores; a.pool_parents = pool_parents;
    a.F = d->F; a.V = d->V; a.k = d->k; a.nchunks = (int)nchunks; a.pool_count = d->pool_count;
    a.pool_capacity = d->pool_capacity;
    char *ws = static_cast<char *>(workspace);
    a.counters = reinterpret_cast<unsigned int *>(ws);
    a.part_keys = reinterpret_cast<uint64_t *>(ws + cbytes);
    a.part_lm = a.part_keys + nslots * RADAR_K_MAX;
    a.gate_pre = reinterpret_cast<float *>(ws + (stream ? kStreamGateOffset : kGateOffset));
    a.cycle = cycle;
    a.pol = pol ? *pol : PolicyArgs{};
    a.has_policy = pol ? 1 : 0;
    a.pol_has_state = (pol && pol->h_in) ? 1 : 0;

    // Most calls' ends are one row per wavefront, one look at its lists and one at the candidates; the code for more would cost them 2-7 % (a cycle of the
    // 8B shape 97 us without, 105 with: registers and fetches of instructions), so it has kernels of its own.
    const bool general = nchunks > kFewChunks || d->F > kExpWaves || d->F * d->k > kFrontierBlock;
    const dim3 grid((unsigned)nchunks, (unsigned)d->F, (unsigned)B), block(kExpThreads);
    hipStream_t st = static_cast<hipStream_t>(stream_);
    hipError_t e;
    if (stream) {
        const dim3 sgrid((unsigned)nchunks, (unsigned)(B * d->F));
        auto go = [&](auto kernel) {
            return launch("expand_stream", kernel, sgrid, dim3(kStreamThreads), 0, st, a.logits, a.F, a.V, a.k, a.nchunks, a.pool_count, a.cycle, a.has_policy,
                          a.pol_has_state, a);
        };
        e = vec4 ? go(expand_stream_kernel<true>) : go(expand_stream_kernel<false>);
        if (e != hipSuccess) return RADAR_HIP_ERROR;
        auto fin = [&](auto kernel) {
            return launch("expand_finish", kernel, dim3((unsigned)B), block, 0, st, a.part_keys, a.part_lm, a.F, a.nchunks, a.k, a.pool_count, a.cycle, a);
        };
        if (general) e = pol ? fin(expand_finish_kernel<kExpPolicy, true>) : fin(expand_finish_kernel<kExpExt, true>);
        else         e = pol ? fin(expand_finish_kernel<kExpPolicy, false>) : fin(expand_finish_kernel<kExpExt, false>);
        return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
    }
    const bool ext = cycle != nullptr || B > 1;
    auto go = [&](auto kernel) {
        return launch("expand", kernel, grid, block, 0, st, a.logits, a.F, a.V, a.k, a.nchunks, a.pool_count, a.cycle, a.part_keys, a.counters, a);
    };
#define RADAR_EXPAND_LAUNCH(V4, E) \
    (general ? (pol ? go(expand_kernel<V4, E, kExpPolicy, true>) : go(expand_kernel<V4, E, kExpExt, true>)) \
             : (pol ? go(expand_kernel<V4, E, kExpPolicy, false>) : ext ? go(expand_kernel<V4, E, kExpExt, false>) : go(expand_kernel<V4, E, kExpPlain, false>)))
    if (ept == 4)      e = vec4 ? RADAR_EXPAND_LAUNCH(true, 4) : RADAR_EXPAND_LAUNCH(false, 4);
    else if (ept == 8) e = vec4 ? RADAR_EXPAND_LAUNCH(true, 8) : RADAR_EXPAND_LAUNCH(false, 8);
    else               e = vec4 ? RADAR_EXPAND_LAUNCH(true, 16) : RADAR_EXPAND_LAUNCH(false, 16);
#undef RADAR_EXPAND_LAUNCH
    return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
}

extern "C" radar_status radar_draft_expand(const float *logits, const float *parent_scores,
                                           const int32_t *parent_pool_idx, int32_t *cand_tokens, float *cand_scores,
                                           int32_t *frontier_pool_idx, int32_t *frontier_tokens,
                                           float *frontier_scores, float *frontier_conf, int32_t *pool_tokens,
                                           float *pool_scores, int32_t *pool_parents, const radar_expand_desc *d,
                                           void *workspace, size_t workspace_bytes, void *stream) {
    return launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                         frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores, pool_parents, d,
                         nullptr, nullptr, 1, workspace, workspace_bytes, stream);
}

// ------------------------------------------------------------------ the entry point that allocates nothing
// For callers that cannot call hipMalloc (code under HIP graph capture, tight serving loops,
// harnesses that forbid it): radar_draft_expand with its workspace in a device array of this
// library instead of a caller-owned buffer.  The array lives in every GPU the library runs on
// until the process ends; its device address is looked up once per device.
static __device__ __align__(256) unsigned char scratch[RADAR_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kScratchMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kScratchMaxDevices];      // device address of `scratch` on each device; null until looked up

__global__ void scratch_clear_kernel(uint4 *p, size_t n16) {
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x) p[i] = z;
}

// The current device's copy of `scratch` (in host code the array's name is only a handle for the
// lookup, never an address).  The first call on a device also clears the array on `stream`: the
// arrival counters at its head must start at zero, and every call leaves them at zero.
radar_status static_scratch(hipStream_t stream, void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return RADAR_HIP_ERROR;
    if (dev < 0 || dev >= kScratchMaxDevices) return RADAR_UNSUPPORTED_SHAPE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return RADAR_HIP_ERROR;
        if (((uintptr_t)ptr & 255) != 0) return RADAR_HIP_ERROR;
        hipLaunchKernelGGL(scratch_clear_kernel, dim3(64), dim3(256), 0, stream, static_cast<uint4 *>(ptr),
                           (size_t)RADAR_NOALLOC_SCRATCH_BYTES / 16);
        if (hipGetLastError() != hipSuccess) return RADAR_HIP_ERROR;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return RADAR_OK;
}
}  // namespace

extern "C" radar_status radar_draft_expand_noalloc(const float *logits, const float *parent_scores,
                                                   const int32_t *parent_pool_idx, int32_t *cand_tokens,
                                                   float *cand_scores, int32_t *frontier_pool_idx,
                                                   int32_t *frontier_tokens, float *frontier_scores,
                                                   float *frontier_conf, int32_t *pool_tokens, float *pool_scores,
                                                   int32_t *pool_parents, const radar_expand_desc *d, void *stream) {
    if (!d || d->F < 1 || d->V < 1) return RADAR_INVALID_ARG;
    const size_t need = expand_workspace_bytes(d, 1);
    if (need == 0 || need > (size_t)RADAR_NOALLOC_SCRATCH_BYTES) return RADAR_UNSUPPORTED_SHAPE;   // F * V beyond the array
    // arguments first (against a stand-in for the array's address), so that an error launches nothing
    radar_status st = launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                                    frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores,
                                    pool_parents, d, nullptr, nullptr, 1, reinterpret_cast<void *>(uintptr_t(256)),
                                    (size_t)RADAR_NOALLOC_SCRATCH_BYTES, stream, true);
    if (st != RADAR_OK) return st;
    void *ws = nullptr;
    st = static_scratch(static_cast<hipStream_t>(stream), &ws);
    if (st != RADAR_OK) return st;
    return launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                         frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores, pool_parents, d,
                         nullptr, nullptr, 1, ws, (size_t)RADAR_NOALLOC_SCRATCH_BYTES, stream);
}

extern "C" radar_status radar_draft_expand_policy(const float *logits, const float *parent_scores,
                                                  const int32_t *parent_pool_idx, int32_t *cand_tokens,
                                                  float *cand_scores, int32_t *frontier_pool_idx,
                                                  int32_t *frontier_tokens, float *frontier_scores,
                                                  float *frontier_conf, int32_t *pool_tokens, float *pool_scores,
                                                  int32_t *pool_parents, const radar_expand_desc *d,
                                                  const radar_policy_params *params, const radar_policy_io *io,
                                                  void *workspace, size_t workspace_bytes, void *stream) {
    PolicyArgs pa;
    const radar_status st = policy_args_from(params, &pa);
    if (st != RADAR_OK) return st;
    if (!d || !io || !io->h_out || !io->c_out || !io->logits || !io->probs || !io->action) return RADAR_INVALID_ARG;
    if ((io->h_in == nullptr) != (io->c_in == nullptr) || ((uintptr_t)io->h_in & 15) != 0) return RADAR_INVALID_ARG;
    if (params->k != d->k) return RADAR_INVALID_ARG;               // the model reads exactly the k confidences
    pa.h_in = io->h_in; pa.c_in = io->c_in; pa.uniforms = io->uniform;
    pa.h_out = io->h_out; pa.c_out = io->c_out; pa.logits = io->logits; pa.probs = io->probs; pa.action = io->action;
    return launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                         frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores, pool_parents, d,
                         &pa, nullptr, 1, workspace, workspace_bytes, stream);
}

// fill kernel for the cycle state (a graph may not hold a memset node)
__global__ void cycle_begin_kernel(radar_cycle_state *st) {
    if (threadIdx.x == 0) { st->stopped = 0; st->pool_count = 0; st->steps_done = 0; st->last_action = -1; }
}

extern "C" radar_status radar_cycle_begin(radar_cycle_state *state, void *stream) {
    if (!state) return RADAR_INVALID_ARG;
    const hipError_t e = launch("cycle_begin", cycle_begin_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), state);
    return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
}

extern "C" radar_status radar_draft_expand_cycle(const float *logits, const float *parent_scores,
                                                 const int32_t *parent_pool_idx, int32_t *cand_tokens,
                                                 float *cand_scores, int32_t *frontier_pool_idx,
                                                 int32_t *frontier_tokens, float *frontier_scores,
                                                 float *frontier_conf, int32_t *pool_tokens, float *pool_scores,
                                                 int32_t *pool_parents, const radar_expand_desc *d,
                                                 const radar_policy_params *params, const radar_policy_io *io,
                                                 radar_cycle_state *state, void *workspace, size_t workspace_bytes,
                                                 void *stream) {
    if (!state || !d) return RADAR_INVALID_ARG;
    if (!params) {
        if (io) return RADAR_INVALID_ARG;
        return launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                             frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores, pool_parents, d,
                             nullptr, state, 1, workspace, workspace_bytes, stream);
    }
    PolicyArgs pa;
    const radar_status st = policy_args_from(params, &pa);
    if (st != RADAR_OK) return st;
    if (!io || !io->h_out || !io->c_out || !io->logits || !io->probs || !io->action) return RADAR_INVALID_ARG;
    if ((io->h_in == nullptr) != (io->c_in == nullptr) || ((uintptr_t)io->h_in & 15) != 0) return RADAR_INVALID_ARG;
    if (params->k != d->k) return RADAR_INVALID_ARG;
    pa.h_in = io->h_in; pa.c_in = io->c_in; pa.uniforms = io->uniform;
    pa.h_out = io->h_out; pa.c_out = io->c_out; pa.logits = io->logits; pa.probs = io->probs; pa.action = io->action;
    return launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                         frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores, pool_parents, d,
                         &pa, state, 1, workspace, workspace_bytes, stream);
}

extern "C" radar_status radar_draft_expand_batch(const float *logits, const float *parent_scores,
                                                 const int32_t *parent_pool_idx, int32_t *cand_tokens,
                                                 float *cand_scores, int32_t *frontier_pool_idx,
                                                 int32_t *frontier_tokens, float *frontier_scores,
                                                 float *frontier_conf, int32_t *pool_tokens, float *pool_scores,
                                                 int32_t *pool_parents, const radar_expand_desc *d, int32_t B,
                                                 const radar_policy_params *params, const radar_policy_io *io,
                                                 radar_cycle_state *states, void *workspace, size_t workspace_bytes,
                                                 void *stream) {
    if (!d) return RADAR_INVALID_ARG;
    if (!params) {
        if (io) return RADAR_INVALID_ARG;
        return launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                             frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores, pool_parents, d,
                             nullptr, states, B, workspace, workspace_bytes, stream);
    }
    PolicyArgs pa;
    const radar_status st = policy_args_from(params, &pa);
    if (st != RADAR_OK) return st;
    if (!io || !io->h_out || !io->c_out || !io->logits || !io->probs || !io->action) return RADAR_INVALID_ARG;
    if ((io->h_in == nullptr) != (io->c_in == nullptr) || ((uintptr_t)io->h_in & 15) != 0) return RADAR_INVALID_ARG;
    if (params->k != d->k) return RADAR_INVALID_ARG;
    pa.h_in = io->h_in; pa.c_in = io->c_in; pa.uniforms = io->uniform;
    pa.h_out = io->h_out; pa.c_out = io->c_out; pa.logits = io->logits; pa.probs = io->probs; pa.action = io->action;
    return launch_expand(logits, parent_scores, parent_pool_idx, cand_tokens, cand_scores, frontier_pool_idx,
                         frontier_tokens, frontier_scores, frontier_conf, pool_tokens, pool_scores, pool_parents, d,
                         &pa, states, B, workspace, workspace_bytes, stream);
}

extern "C" size_t radar_draft_rerank_workspace_bytes(int32_t pool_count, int32_t N) {
    (void)pool_count; (void)N;
    return 256;   // rerank keeps everything in LDS; a minimal workspace keeps the calling convention uniform
}

static radar_status launch_rerank(const int32_t *pool_tokens, const float *pool_scores, const int32_t *pool_parents,
                                  int32_t pool_count, const radar_cycle_state *cycle, int32_t N, int32_t root_token,
                                  int32_t *tree_tokens, int32_t *tree_parents, float *tree_scores,
                                  int32_t *tree_depth, int32_t *tree_pool_idx, int32_t *n_nodes_out, void *stream,
                                  int32_t B = 1, const int32_t *root_tokens = nullptr, int32_t pool_capacity = 0) {
    if (!pool_tokens || !pool_scores || !pool_parents || !tree_tokens || !tree_parents || !tree_scores ||
        !tree_depth || !tree_pool_idx || !n_nodes_out)
        return RADAR_INVALID_ARG;
    if (pool_count < 0 || N < 0) return RADAR_INVALID_ARG;
    if (pool_count > RADAR_POOL_MAX || N >= RADAR_T_MAX) return RADAR_UNSUPPORTED_SHAPE;
    if (B < 1 || (B > 1 && pool_capacity < pool_count)) return RADAR_INVALID_ARG;
    RerankArgs a;
    a.root_tokens = root_tokens; a.pool_capacity = pool_capacity;
    a.pool_tokens = pool_tokens; a.pool_scores = pool_scores; a.pool_parents = pool_parents;
    a.pool_count = pool_count; a.N = N; a.root_token = root_token; a.cycle = cycle;
    a.tree_tokens = tree_tokens; a.tree_parents = tree_parents; a.tree_scores = tree_scores;
    a.tree_depth = tree_depth; a.tree_pool_idx = tree_pool_idx; a.n_nodes_out = n_nodes_out;
    auto go = [&](auto kernel) {
        return launch("rerank", kernel, dim3((unsigned)B), dim3(kTopkThreads), 0, static_cast<hipStream_t>(stream), a.pool_scores, a.pool_tokens,
                      a.pool_parents, a.cycle, a.pool_count, a.N, a.pool_capacity, a.root_token, a);
    };
    const hipError_t e = pool_count <= 4 * kTopkThreads
        ? go(rerank_kernel<4>)
        : go(rerank_kernel<16>);
    return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
}

extern "C" radar_status radar_draft_rerank(const int32_t *pool_tokens, const float *pool_scores,
                                           const int32_t *pool_parents, int32_t pool_count, int32_t N,
                                           int32_t root_token, int32_t *tree_tokens, int32_t *tree_parents,
                                           float *tree_scores, int32_t *tree_depth, int32_t *tree_pool_idx,
                                           int32_t *n_nodes_out, void *workspace, size_t workspace_bytes,
                                           void *stream) {
    (void)workspace; (void)workspace_bytes;
    return launch_rerank(pool_tokens, pool_scores, pool_parents, pool_count, nullptr, N, root_token, tree_tokens,
                         tree_parents, tree_scores, tree_depth, tree_pool_idx, n_nodes_out, stream);
}

extern "C" radar_status radar_draft_rerank_cycle(const int32_t *pool_tokens, const float *pool_scores,
                                                 const int32_t *pool_parents, const radar_cycle_state *state,
                                                 int32_t pool_count_max, int32_t N, int32_t root_token,
                                                 int32_t *tree_tokens, int32_t *tree_parents, float *tree_scores,
                                                 int32_t *tree_depth, int32_t *tree_pool_idx, int32_t *n_nodes_out,
                                                 void *workspace, size_t workspace_bytes, void *stream) {
    (void)workspace; (void)workspace_bytes;
    if (!state) return RADAR_INVALID_ARG;
    return launch_rerank(pool_tokens, pool_scores, pool_parents, pool_count_max, state, N, root_token, tree_tokens,
                         tree_parents, tree_scores, tree_depth, tree_pool_idx, n_nodes_out, stream);
}

extern "C" radar_status radar_draft_rerank_batch(const int32_t *pool_tokens, const float *pool_scores,
                                                 const int32_t *pool_parents, const radar_cycle_state *states,
                                                 int32_t pool_count, int32_t pool_capacity, int32_t B, int32_t N,
                                                 const int32_t *root_tokens, int32_t *tree_tokens,
                                                 int32_t *tree_parents, float *tree_scores, int32_t *tree_depth,
                                                 int32_t *tree_pool_idx, int32_t *n_nodes_out, void *workspace,
                                                 size_t workspace_bytes, void *stream) {
    (void)workspace; (void)workspace_bytes;
    if (!root_tokens || B < 1 || pool_capacity < 0 || pool_count > pool_capacity) return RADAR_INVALID_ARG;
    if (B > 65535) return RADAR_UNSUPPORTED_SHAPE;
    return launch_rerank(pool_tokens, pool_scores, pool_parents, pool_count, states, N, 0, tree_tokens, tree_parents,
                         tree_scores, tree_depth, tree_pool_idx, n_nodes_out, stream, B, root_tokens, pool_capacity);
}
