// Verification walk of RADAR's speculative-sampling cycle (Sec. 3, Eq. 1-2; tree
// form per Sec. 4.3, Eq. 11-13) as one HIP launch for gfx950.
//
// Phase 1, grid (blocks of the vocabulary, sequences, tree rows): one streaming
// read of target logits.  Every wavefront owns NB x 1024 consecutive logits and
// leaves, per 1024, their arg-max key or, in sampling mode, (max, sum exp) of the
// temperature-scaled values; nothing is combined inside a workgroup.  Phase 2: the
// workgroup whose arrival ticket is the last of its ROW merges that row's partials
// in one wavefront and turns the sums into masses relative to the row maximum.
// Phase 3, the walk, starts with the root row's completion and is carried on by
// whichever row completes next on the path: a completed row marks itself done, a
// walk that arrives at a row marks it reached, and the one that finds the other's
// mark goes on (the two marks are one atomic OR each, so exactly one does).
// Nobody waits.  One wavefront, one lane per node: sibling sets come from ballots,
// everything the walk compares sits in registers and is passed between lanes by
// lane reads or DPP scans.  The residual draw scans the 1024-logit masses across
// lanes and then re-reads one such block (4 KB).
//
// Only rows on the accepted path decide anything, and most rows of a batch are
// known to be off it long before their turn in the stream: the walk publishes the
// node it has arrived at, and a workgroup whose row does not descend from it leaves
// its logits unread.  Rows go through the grid level by level over all sequences
// (trees are numbered from the root), so that the roots' decisions come first.
// What bounds a call is then the chain of decisions and the starting of workgroups, not
// the logits' bytes: 61 rows of V = 128256, 16 sequences, paths of 0, 1, 2, 4 and 8 nodes 17.9, 23.2,
// 24.6, 30.7 and 36.9 us greedy and 23.2, 26.7, 28.3, 33.4 and 41.6 sampled (129 when every row is
// read); one sequence 7.1 ... 7.6 and 9.2 ... 13.2 us (one set of logits replayed; with logits that are in no
// cache 18.1 ... 44.1 and 23.3 ... 46.9, one sequence 9.9 ... 10.4 and 12.1 ... 15.6).  In a large launch the
// workgroups behind the roots' rows hold back until the roots are decided (below).
#include <algorithm>

#include "radar_device.h"
#include "radar_host.h"

namespace radar {

constexpr int kAccThreads = 256;
constexpr int kAccWaves = kAccThreads / kWave;
constexpr int kAccEPT = 16;
constexpr int kAccSub = kWave * kAccEPT;              // 1024 logits per wavefront = one partial
constexpr int kAccChunk = kAccThreads * kAccEPT;      // logits per workgroup
constexpr int kAccMaxSubs = 4096;                     // V <= 4,194,304
constexpr int kAccCounterStride = 16;   // counters 64 B apart (same-line fetch-adds serialise)
constexpr int64_t kAccManyBlocks = 49152;
constexpr int64_t kAccWalkLast = 3072;  // greedy launches up to this many workgroups leave the walk to the last row
constexpr int kAccUnchecked = 1024;     // workgroups the chip starts first: nothing is decided yet when they do
constexpr int kAccPolls = 3;            // how often a waiting workgroup looks (1 us apart)
constexpr int kAccWaitNodes = 8;        // trees of fewer nodes never wait (launch_accept)
constexpr float kAccLog2e = 1.4426950408889634f;
constexpr unsigned int kAccDone = 1u << 30, kAccReached = 1u << 29;   // marks beside a row's count of arrivals
constexpr int kAccEnded = RADAR_T_MAX;  // "node arrived at" once the walk has ended
constexpr int kAccDistribution = 2;     // internal mode: acceptance-length distribution instead of a walk

struct AcceptArgs {
    const float *logits;
    const int32_t *tokens;
    const int32_t *parents;
    const int32_t *n_nodes;
    const float *uniforms;
    int32_t *accept_len;
    int32_t *accept_path;
    int32_t *bonus;
    double *dist;               // mode kAccDistribution: [B][D_max+1]
    int B, T, V, D_max, nwg, nsub;   // nwg workgroups and nsub 1024-logit blocks per row
    int check_from;             // workgroups from this number on ask whether their row can still be on the path
    int wait;                   // (units of 10 ns) those of them that start with the launch wait so long for the roots' decisions:
    int wait_until, wait_nodes; // those before this number, of trees of so many nodes
    int exact_scale;            // 1/temperature is exactly representable in fp32
    float inv_temp_f;
    double inv_temp;
    unsigned int *counters;     // [(b*T + r) * stride] workgroups of a row and its marks, [(B*T + b) * stride] finished rows
                                // of a sequence, [(B*T + B + b) * stride] node its walk has arrived at (0: the root)
    uint64_t *row_key;          // [B][T] greedy: arg-max key of the row
    uint64_t *row_lm;           // [B][T][2] sampling: sum of exp(y - M), y = logit / temperature, and M, the row's maximum, in the lower half
    uint64_t *part_key;         // [B][T][nsub] greedy: arg-max key of the block
    uint64_t *part_lm;          // [B][T][nsub][2] sampling: sum of exp(y - m) over the block and its reference maximum m; once the row is merged
                                //              the first is the sum of exp(y - M) over the block
};

struct AcceptSmem {
    unsigned int ticket;
    int row_arg[RADAR_T_MAX];                     // rows whose results this wavefront holds
    float row_M[RADAR_T_MAX];
    double row_L[RADAR_T_MAX];
    int rej_tok[RADAR_T_MAX];
    float rej_x[RADAR_T_MAX];                     // their logits
    int internal[RADAR_T_MAX];                    // distribution: nodes with children,
    unsigned long long kid_mask[RADAR_T_MAX], depth_mask[RADAR_T_MAX];   // the children of each node, the nodes at each depth
    double rej_e[RADAR_T_MAX];                    // what each rejected token carries, and the block it lies in
    int rej_sub[RADAR_T_MAX];
    unsigned int rej_bits[kWave];                 // pass (b): which of a lane's 16 tokens are rejected ones
    union alignas(16) {
        unsigned char seen[4096];                 // sibling tokens, hashed
        float mass[kAccSub];                      // pass (b): the block's exponentials
    };
};

// exp(x / temperature - ref) for one logit.  The exponent difference is rounded to
// fp32 once (an fp32 FMA does that when the scale is exact in fp32, else it is formed in fp64);
// the exponential itself is the fp32 one.  The sums that use it are kept in fp64.
template <bool EXACT>
__device__ __forceinline__ float scaled_exp(float x, const AcceptArgs &a, float ref) {
    if (EXACT) return __builtin_amdgcn_exp2f(__builtin_fmaf(x, a.inv_temp_f, -ref) * kAccLog2e);
    return expf((float)((double)x * a.inv_temp - (double)ref));
}

// 16 logits per lane of one 1024-logit block: lane l takes [16 * l, 16 * l + 16) when CONTIG (pass
// (b) needs token order inside a lane), else 4 x (64 lanes x 16 B) interleaved (widest requests).
template <bool VEC4, bool CONTIG>
__device__ __forceinline__ void load_block(const float *row, int i_block, int V, float (&x)[kAccEPT], int (&first)[kAccEPT / 4]) {
    const int lane = lane_id();
    float4 raw[kAccEPT / 4];
#pragma unroll
    for (int g = 0; g < kAccEPT / 4; ++g) {
        const int i = i_block + (CONTIG ? lane * kAccEPT + 4 * g : g * (kWave * 4) + lane * 4);
        first[g] = i;
        // branch-free: out-of-range lanes read a valid address and are masked afterwards
        if (VEC4) raw[g] = *reinterpret_cast<const float4 *>(row + (i < V ? i : 0));
    }
    if (!VEC4 && V >= 4) {
#pragma unroll
        for (int g = 0; g < kAccEPT / 4; ++g) raw[g] = load4_of_row(row, first[g], V);
    } else if (!VEC4) {
#pragma unroll
        for (int g = 0; g < kAccEPT / 4; ++g) raw[g] = load4_of_short_row(row, V);
    }
#pragma unroll
    for (int g = 0; g < kAccEPT / 4; ++g) { x[4 * g] = raw[g].x; x[4 * g + 1] = raw[g].y; x[4 * g + 2] = raw[g].z; x[4 * g + 3] = raw[g].w; }
    if (i_block + kAccSub > V) {                              // wave-uniform: only a row's last block needs masking
        if (!VEC4) place_row_end<kAccEPT / 4>([&](int g, int j) -> float & { return x[4 * g + j]; }, first[0], CONTIG ? 4 : kWave * 4, V);
#pragma unroll
        for (int e = 0; e < kAccEPT; ++e) x[e] = (first[e / 4] + (e & 3) < V) ? x[e] : -INFINITY;
    }
}

// One OR / addition on a counter by lane 0; every lane of the wavefront gets the value before it.
__device__ __forceinline__ unsigned int wave_fetch_or(unsigned int *p, unsigned int v) {
    unsigned int old = 0;
    if (lane_id() == 0) old = __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return readlane_u32(old, 0);
}
__device__ __forceinline__ unsigned int wave_fetch_add(unsigned int *p, unsigned int v) {
    unsigned int old = 0;
    if (lane_id() == 0) old = __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return readlane_u32(old, 0);
}

// A sum and a maximum side by side: handed over by two lanes in one request, taken in one (device scope, as load_shared_result's; entries past
// the n behind `from` read zeros, and `from` is the same in every lane).  As two arrays, of 8 and of 4 bytes,
// 61 rows of V = 128256 took 11.33 us, as pairs 11.08; 9 trees of 5 nodes, V = 45299, 9.41 and 9.00; two of 16, V = 51757, 8.58 and 8.27.
struct SumMax { double l; float m; };
__device__ __forceinline__ void store_sum_max(uint64_t *to, double l, float m) {        // by lanes 0 and 1
    const int lane = lane_id();
    if (lane < 2) store_shared_result(to + lane, lane == 0 ? (uint64_t)__double_as_longlong(l) : (uint64_t)__float_as_uint(m));
}
__device__ __forceinline__ SumMax load_sum_max(const uint64_t *from, int n, int i) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(from), 0, n * 16, 0x00027000), i * 16, 0, 16);
    return {__longlong_as_double((long long)((uint64_t)v[1] << 32 | v[0])), __uint_as_float(v[2])};
}
__device__ __forceinline__ double load_sum(const uint64_t *from) { return __longlong_as_double((long long)load_shared_result(from)); }

// NB: 1024-logit blocks per wavefront, all requested at once
// LAST: the walk is left to the last row of the sequence (greedy only).
// A sampled walk and the distribution ask for nobody's arg-max; with the keys found, stored, fetched and merged all the same a sampled call
// over 9 trees of 5 nodes, V = 45299, took 9.78 us instead of 9.41, two of 16, V = 51757, 9.08 instead of 8.58, the distribution of 11 trees
// of V = 128256 18.68 instead of 17.45 (before sums and maxima were pairs).
// The sampled kernel fits into 72 registers so, seven wavefronts per SIMD, but six are the better number: with more the other rows'
// logits are in front of the root's in the memory's queue, with fewer too little is in flight.  Over 40 shapes (1, 4, 8, 16 sequences of 61 rows,
// V = 32000 and 128256, paths of 0 ... 8 nodes; the workgroups that wait are as many as fit) seven, five and four take 1.004, 1.023 and 1.076 times
// as long as six on replayed logits, 1.014, 1.008 and 1.045 on logits that are in no cache.  One by one they differ: of V = 128256, 16 trees whose
// root is the end 22.9 us with six, 21.2 with seven, 29.8 with four; 8 trees with paths of two nodes 21.9, 23.1, 22.8.
template <int MODE, bool LAST, bool VEC4, int NB>
__global__ __launch_bounds__(kAccThreads) __attribute__((amdgpu_waves_per_eu(1, MODE == RADAR_ACCEPT_SAMPLE ? 6 : 8))) void accept_kernel(AcceptArgs a) {
    __shared__ AcceptSmem s;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int b = blockIdx.y, r = blockIdx.z;
    constexpr bool sampling = MODE != RADAR_ACCEPT_GREEDY;      // row statistics are needed
    // A root's row is there whatever the number of nodes, and everything waits for it: its logits are asked for first, the number of nodes
    // beside the tree's arrays (61 rows of V = 128256 11.08 us, so 10.90; the distribution of 11 trees 17.33 and 17.19).  Greedy roots have
    // nothing to do meanwhile (16 trees 18.6 us, so 18.9).  That the arrays are then read at clamped places, and not where there is a node, is so that
    // they need not wait for the number of nodes; alone it changes nothing (1.00 over the 40 shapes above).
    const bool root_first = sampling && r == 0;
    auto node_count = [&] { return max(1, min(a.n_nodes ? a.n_nodes[b] : a.T, a.T)); };
    int nn = 1;
    if (!root_first) {
        nn = node_count();
        if (r >= nn) return;
    }
    constexpr bool distribution = MODE == kAccDistribution;
    const float *row = a.logits + ((size_t)b * a.T + r) * a.V;
    const int sub0 = (blockIdx.x * kAccWaves + w) * NB;      // this wavefront's first 1024-logit block
    unsigned int *const words = a.counters + (size_t)b * a.T * kAccCounterStride;          // of this sequence's rows
    unsigned int *const seq_counter = &a.counters[((size_t)a.B * a.T + b) * kAccCounterStride];
    unsigned int *const arrived_at = &a.counters[((size_t)a.B * a.T + a.B + b) * kAccCounterStride];

    // ---------------- is the row needed?  The distribution reads the rows of nodes that have children (a
    // leaf keeps whatever reaches it).  A walk reads the rows it arrives at, and those below the node it has
    // arrived at so far may still be among them.  (The wavefronts of a workgroup, and the workgroups of a
    // row, may see the walk at different nodes: one that finds the row off the path is right, the walk
    // only moves down, and then nobody will ask for the row's results.)
    bool needed = true;
    const unsigned int number = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    if (!root_first && (distribution || (!LAST && number >= (unsigned int)a.check_from))) {
        unsigned int at = 0;
        if (!distribution && (int)number < a.wait_until && nn >= a.wait_nodes) {
            // By the clock, not by anything another workgroup does: whatever happens elsewhere, this ends.
            const uint64_t t0 = wall_clock64();
            for (int k = 0; k < kAccPolls && at == 0; ++k) {
                for (int i = 0; i < 400 && wall_clock64() - t0 < (uint64_t)(a.wait + 100 * k); ++i) __builtin_amdgcn_s_sleep(8);
                at = load_shared_result(arrived_at);
            }
        } else if (!distribution) {
            at = load_shared_result(arrived_at);
        }
        int par = lane < nn ? a.parents[(size_t)b * a.T + lane] : -1;
        par = par < lane ? par : -1;
        if (distribution) {
            if (__ballot(par == r) == 0ull) return;
        } else {
            const int cur = (int)readlane_u32(at, 0);
            int x = r;
            while (x > cur) x = (int)readlane_u32((uint32_t)par, x);        // strictly decreasing
            needed = x == cur;
        }
    }

    // ---------------- phase 1: per-wavefront arg-max (and scaled max / sum-exp)
    if (needed && sub0 < a.nsub) {
        float x[NB][kAccEPT];
        int first[NB][kAccEPT / 4];
#pragma unroll
        for (int i = 0; i < NB; ++i) load_block<VEC4, false>(row, (sub0 + i) * kAccSub, a.V, x[i], first[i]);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            // Largest logit of the block first (lane, then wavefront); only the lanes that hold it look for
            // its position, lowest index first (-0.0 equals +0.0 here, as in the key order).
            float tmx = x[i][0];
#pragma unroll
            for (int e = 1; e < kAccEPT; ++e) tmx = fmaxf(tmx, x[i][e]);
            const float wmx = wave_max_f32(tmx);
            const size_t pslot = ((size_t)b * a.T + r) * a.nsub + sub0 + i;
            const bool live = NB == 1 || sub0 + i < a.nsub;       // wave-uniform
            if (sampling) {
                // 1 / temperature > 0 and rounding is monotone, so the largest scaled logit is the scaled largest
                const float wm = wmx * a.inv_temp_f;
                double tl = 0.0;
                if (wm > -INFINITY) {
                    if (a.exact_scale) {
#pragma unroll
                        for (int e = 0; e < kAccEPT; ++e) tl += (double)scaled_exp<true>(x[i][e], a, wm);
                    } else {
#pragma unroll
                        for (int e = 0; e < kAccEPT; ++e) tl += (double)scaled_exp<false>(x[i][e], a, wm);
                    }
                }
                const double wl = wave_sum_f64(tl);
                if (live) store_sum_max(&a.part_lm[2 * pslot], wl, wm);
            }
            if constexpr (!sampling) {
                uint32_t bi = 0xffffffffu;
                if (tmx == wmx) {
#pragma unroll
                    for (int e = kAccEPT - 1; e >= 0; --e) bi = (x[i][e] == wmx) ? uint32_t(first[i][e / 4] + (e & 3)) : bi;
                }
                bi = ~wave_max_u32(~bi);                          // lowest index over the wavefront
                const uint64_t best = bi < (uint32_t)a.V ? make_key(wmx, bi) : 0;
                if (lane == 0 && live) store_shared_result(&a.part_key[pslot], best);
            }
        }
    }
    // What the walk needs to know of the tree is fetched beside the stream's last results: behind the ticket it was a round
    // trip before the gather of the tokens' logits could be asked for.
    const int c = lane;
    int p = -1, t = -1;
    float uc = 0.f, ubonus = 0.f;
    if (w == 0) {
        if (root_first) nn = node_count();
        if constexpr (sampling) {
            const size_t at = (size_t)b * a.T + min(c, a.T - 1);
            p = a.parents[at];
            t = a.tokens[at];
            if (c >= nn) p = t = -1;
        } else if (c < nn) {
            p = a.parents[(size_t)b * a.T + c];
            t = a.tokens[(size_t)b * a.T + c];
        }
        if (MODE == RADAR_ACCEPT_SAMPLE) {
            const float *u = a.uniforms + (size_t)b * (a.T + 1);
            uc = u[min(c, a.T)];
            ubonus = u[a.T];
        }
    }
    const bool tree_ok = (c > 0 && c < nn && p >= 0 && p < c);
    if ((publish_then_ticket(&words[r * kAccCounterStride], &s.ticket) & (kAccReached - 1)) != (unsigned int)(a.nwg - 1)) return;
    if (w != 0) return;                                      // one wavefront does the rest

    // A row is finished once whoever completed it has nothing more to do for it; the last row of the sequence
    // leaves the counters clean for the next call (every workgroup has arrived by then, and the walk
    // has ended: its steps are taken by rows not finished yet).
    auto finish_row = [&](unsigned int before) {
        if (before != (unsigned int)(nn - 1)) return;
        if (lane < nn) store_shared_result(&words[lane * kAccCounterStride], 0u);
        if (lane == 0) { store_shared_result(seq_counter, 0u); store_shared_result(arrived_at, 0u); }
    };
    if (!needed) { finish_row(wave_fetch_add(seq_counter, 1u)); return; }

    // ---------------- phase 2: last workgroup of row r -- merge the row's partials.
    // The logits that only the walk needs (lane c is tree node c) are asked for together with the partials.
    float xg = 0.f;
    uint64_t kb = 0;
    float M;
    double L, mass_[2] = {0.0, 0.0};                         // this row's first 128 block masses
    {
        if (sampling && tree_ok && t >= 0 && t < a.V) xg = a.logits[((size_t)b * a.T + p) * a.V + t];
        const size_t p0 = ((size_t)b * a.T + r) * a.nsub;
        uint64_t *const pairs = a.part_lm + 2 * p0;
        // the first 128 partials (all of them up to V = 131072) are taken in one round trip
        float m_[2];
        double l_[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c0 = i * kWave + lane;
            const int cc = min(c0, a.nsub - 1);                  // branch-free: clamp, load, mask
            m_[i] = -INFINITY; l_[i] = 0.0;
            if constexpr (!sampling) {
                const uint64_t k2 = load_shared_result(&a.part_key[p0 + cc]);
                kb = max_u64(kb, c0 < a.nsub ? k2 : 0);
            } else {
                const SumMax v = load_sum_max(pairs, a.nsub, cc);
                if (c0 < a.nsub) { m_[i] = v.m; l_[i] = v.l; }
            }
        }
        float mmax = fmaxf(m_[0], m_[1]);
        for (int c0 = 2 * kWave + lane; c0 < a.nsub; c0 += kWave) {
            if (!sampling) kb = max_u64(kb, load_shared_result(&a.part_key[p0 + c0]));
            else mmax = fmaxf(mmax, load_sum_max(pairs, a.nsub, c0).m);
        }
        if constexpr (!sampling) kb = wave_max_u64(kb);
        M = wave_max_f32(mmax);
        double lsum = 0.0;
        if (sampling) {
            // each block's mass relative to the row maximum: summed for the row, and left in the first half
            // of the block's pair for the residual draw
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int c0 = i * kWave + lane;
                mass_[i] = m_[i] > -INFINITY ? l_[i] * exp((double)m_[i] - (double)M) : 0.0;
                if (c0 < a.nsub) store_shared_result(&pairs[2 * c0], (uint64_t)__double_as_longlong(mass_[i]));
                lsum += mass_[i];
            }
            for (int c0 = 2 * kWave + lane; c0 < a.nsub; c0 += kWave) {
                const SumMax v = load_sum_max(pairs, a.nsub, c0);
                const double mass = v.m > -INFINITY ? v.l * exp((double)v.m - (double)M) : 0.0;
                store_shared_result(&pairs[2 * c0], (uint64_t)__double_as_longlong(mass));
                lsum += mass;
            }
        }
        L = wave_sum_f64(lsum);
        const size_t rs = (size_t)b * a.T + r;
        if constexpr (sampling) store_sum_max(&a.row_lm[2 * rs], L, M);
        if (lane == 0) {
            if constexpr (!sampling) store_shared_result(&a.row_key[rs], kb);
            if (distribution || LAST) store_shared_result(&words[r * kAccCounterStride], 0u);   // leave the row's counter clean
        }
    }

    if (distribution) {
        // the last of the rows with children (and the root's) goes on
        s.internal[lane] = lane == 0;
        wave_lds_sync();
        if (tree_ok) s.internal[p] = 1;
        wave_lds_sync();
        const bool inner = s.internal[lane] != 0;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (wave_fetch_add(seq_counter, 1u) != (unsigned int)(__popcll(__ballot(inner)) - 1)) return;
        if (lane == 0) store_shared_result(seq_counter, 0u);
        asm volatile("" ::: "memory");
        if (inner) {
            const SumMax v = load_sum_max(a.row_lm + 2 * (size_t)b * a.T, nn, c);
            s.row_M[c] = v.m;
            s.row_L[c] = v.l;
        }
        wave_lds_sync();
        double pc = 0.0;                                     // probability of each node's token under its parent's row
        if (tree_ok && t >= 0 && t < a.V) pc = exp((double)xg * a.inv_temp - (double)s.row_M[p]) / s.row_L[p];
        // Sec. 4.3, Eq. 11-13, one lane per node.
        // Children of each node as a bit mask; the sums below run over the bits, in node order.
        s.kid_mask[lane] = 0;
        s.rej_tok[lane] = t;
        wave_lds_sync();
        if (tree_ok) atomicOr(&s.kid_mask[p], 1ull << lane);
        wave_lds_sync();
        bool dup = false;                                    // same token as an earlier sibling: never reached
        for (unsigned long long m = tree_ok ? s.kid_mask[p] & ((1ull << lane) - 1) : 0ull; m; m &= m - 1)
            dup = dup || s.rej_tok[__ffsll((long long)m) - 1] == t;
        if (dup) pc = 0.0;
        // depth and reach level by level: a lane whose parent is settled takes depth(parent) + 1 and
        // reach(parent) * its own probability (two lane gathers); as many rounds as the tree is deep.
        // Nodes with a broken parent count as settled with depth 0 and reach 0.
        int depth = 0;
        double reach = c == 0 ? 1.0 : 0.0, kids = 0.0;       // mass that arrives here / that goes on to children
        bool settled = !tree_ok;                             // the root and everything outside the tree
        for (int round = 0; round < nn; ++round) {
            if (__ballot(!settled) == 0ull) break;
            const int src = max(p, 0);
            const int pd = __shfl(depth, src);
            const bool ps = __shfl((int)settled, src) != 0;
            const double pr = __longlong_as_double(__shfl((long long)__double_as_longlong(reach), src));
            if (!settled && ps) {
                depth = pd + 1;
                if (depth > a.D_max) pc = 0.0;               // cut: nothing is handed below D_max
                reach = pr * pc;
                settled = true;
            }
        }
        s.rej_e[lane] = pc;
        s.depth_mask[lane] = 0;
        wave_lds_sync();
        for (unsigned long long m = s.kid_mask[lane]; m; m &= m - 1) kids += s.rej_e[__ffsll((long long)m) - 1];   // children's mass per parent
        double stay = 1.0 - kids;
        stay = stay > 0.0 ? stay : 0.0;
        const double pstop = (c < nn && depth <= a.D_max) ? reach * stay : 0.0;
        wave_lds_sync();
        s.rej_e[lane] = pstop;
        if (c < nn && pstop > 0.0) atomicOr(&s.depth_mask[depth], 1ull << lane);
        wave_lds_sync();
        double acc = 0.0;
        for (unsigned long long m = s.depth_mask[lane]; m; m &= m - 1) acc += s.rej_e[__ffsll((long long)m) - 1];
        for (int d = lane; d <= a.D_max; d += kWave) a.dist[(size_t)b * (a.D_max + 1) + d] = d == lane ? acc : 0.0;
        return;
    }

    // ---------------- phase 3: this row is done; if the walk has arrived here already (it starts at the root), go on with it
    if (LAST) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (wave_fetch_add(seq_counter, 1u) != (unsigned int)(nn - 1)) return;
        if (lane == 0) store_shared_result(seq_counter, 0u);
    } else if (r > 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if ((wave_fetch_or(&words[r * kAccCounterStride], kAccDone) & kAccReached) == 0u) {
            finish_row(wave_fetch_add(seq_counter, 1u));
            return;
        }
    }
    uint64_t have = 0;                                       // rows whose results are in s.row_*
    bool match = false;                                      // greedy: the token is its parent's row's arg-max
    double pc = 0.0;                                         // sampled: probability of the token under its parent's row
    // the results of the rows whose lanes say so, and what follows from them for their children
    auto take_rows = [&](bool take, bool own) {
        asm volatile("" ::: "memory");                       // (after the marks)
        if (take) {
            if constexpr (!sampling) {
                const uint64_t key = own ? kb : load_shared_result(&a.row_key[(size_t)b * a.T + lane]);
                s.row_arg[lane] = (int)key_index(key);
            } else {
                SumMax v = {L, M};
                if (!own) v = load_sum_max(a.row_lm + 2 * (size_t)b * a.T, a.T, lane);
                s.row_M[lane] = v.m;
                s.row_L[lane] = v.l;
            }
        }
        const uint64_t fresh = __ballot(take);
        have |= fresh;
        wave_lds_sync();
        if (tree_ok && ((fresh >> p) & 1)) {
            if (!sampling) match = s.row_arg[p] == t;
            else if (t >= 0 && t < a.V) pc = exp((double)xg * a.inv_temp - (double)s.row_M[p]) / s.row_L[p];   // (no logarithm on the way)
        }
    };
    const int up = tree_ok ? p : -1;
    int cur = 0, len = 0, mypath = 0;                        // lane i keeps path[i]
    if (LAST) {
        take_rows(lane < nn, false);
    } else {
        take_rows(lane == r, true);
        cur = r;
        for (int x = r; x > 0; x = (int)readlane_u32((uint32_t)up, x)) ++len;
        int d = len;
        for (int x = r; x > 0; x = (int)readlane_u32((uint32_t)up, x), --d)
            if (lane == d) mypath = x;
    }
    double R = 0.0;
    int nrej = 0, rejtok = -1;                               // lane j keeps the j-th rejected token and its logit
    float rejx = 0.f;
    for (;;) {
        uint64_t kids = (len < a.D_max) ? __ballot(tree_ok && p == cur) : 0ull;
        R = 0.0; nrej = 0;
        int next = -1;
        if (!sampling) {
            kids &= __ballot(match);
            if (kids) next = __ffsll((long long)kids) - 1;
        } else if (__popcll(kids) > 4) {
            // wide level: all children at once.  A child is reached only if every earlier sibling was
            // rejected, so its residual is the sum of the earlier siblings' probabilities.
            const bool kid = (kids >> lane) & 1;
            // same token as an earlier sibling?  Tokens are hashed into a byte table; a lane that does
            // not read its own number back shares a bucket, and only then are tokens compared.
            const uint32_t h = ((uint32_t)t * 2654435761u) >> 20;
            if (kid) s.seen[h] = (unsigned char)lane;
            wave_lds_sync();
            const bool shared = kid && s.seen[h] != (unsigned char)lane;
            wave_lds_sync();
            bool dup = false;
            if (__ballot(shared)) {
                for (uint64_t m = kids; m; m &= m - 1) {
                    const int cc = __ffsll((long long)m) - 1;
                    const int tcc = (int)readlane_u32((uint32_t)t, cc);
                    dup = dup || (kid && lane > cc && t == tcc);
                }
            }
            const bool live = kid && !dup;
            const double mine = live ? pc : 0.0;
            const double before = wave_scan_f64(mine) - mine;
            const uint64_t acc = __ballot(live && (double)uc * (1.0 - before) < pc);
            uint64_t rejected = __ballot(live);
            if (acc) {
                next = __ffsll((long long)acc) - 1;
                rejected &= (1ull << next) - 1;
            }
            nrej = __popcll(rejected);
            R = nrej ? readlane_f64(before + mine, 63 - __clzll((long long)rejected)) : 0.0;
            // lane j takes the token of the j-th rejected child
            if ((rejected >> lane) & 1) {
                s.rej_tok[lanes_below(rejected)] = t;
                s.rej_x[lanes_below(rejected)] = xg;
            }
            wave_lds_sync();
            rejtok = lane < nrej ? s.rej_tok[lane] : -1;
            rejx = s.rej_x[lane];
            wave_lds_sync();
        } else {
            while (kids) {
                const int cc = __ffsll((long long)kids) - 1;
                kids &= kids - 1;
                const int tcc = (int)readlane_u32((uint32_t)t, cc);
                if (__ballot(lane < nrej && rejtok == tcc)) continue;   // same token as an earlier sibling
                const double pcc = readlane_f64(pc, cc);
                const float ucc = readlane_f32(uc, cc);
                if ((double)ucc * (1.0 - R) < pcc) { next = cc; break; }
                R += pcc;
                const float xcc = readlane_f32(xg, cc);
                if (lane == nrej) { rejtok = tcc; rejx = xcc; }
                ++nrej;
            }
        }
        if (next < 0) break;
        cur = next;
        ++len;
        if (lane == len) mypath = cur;
        if (LAST) continue;
        if (lane == 0) store_shared_result(arrived_at, (unsigned int)cur);
        if ((have >> cur) & 1) continue;
        // The next row's results: if it is not done yet, whoever completes it finds the mark and goes on.
        // Otherwise every row that is done by now is fetched, and the walk continues in registers.
        const unsigned int seen = wave_fetch_or(&words[cur * kAccCounterStride], kAccReached);
        const unsigned int word = load_shared_result(&words[min(lane, nn - 1) * kAccCounterStride]);
        if ((seen & kAccDone) == 0u) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            finish_row(wave_fetch_add(seq_counter, 1u));
            return;
        }
        take_rows((lane == cur || (lane < nn && (word & kAccDone) != 0u)) && !((have >> lane) & 1), false);
    }
    if (lane == 0 && !LAST) store_shared_result(arrived_at, (unsigned int)kAccEnded);
    if (c <= a.D_max) a.accept_path[(size_t)b * (a.D_max + 1) + c] = (c <= len) ? mypath : -1;
    if (lane == 0) a.accept_len[b] = len;
    if (!sampling) {
        if (lane == 0) a.bonus[b] = s.row_arg[cur];
        if (LAST) return;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        finish_row(wave_fetch_add(seq_counter, 1u));
        return;
    }

    // ---- residual draw, (a): the 1024-logit block that holds the target mass
    M = s.row_M[cur];
    L = s.row_L[cur];
    const size_t p0 = ((size_t)b * a.T + cur) * a.nsub;
    const float *xr = a.logits + ((size_t)b * a.T + cur) * a.V;
    // masses of the first 128 blocks (a row this wavefront has just merged still has them in registers)
    double mass0 = mass_[0], mass1 = mass_[1];
    if (cur != r) {
        mass0 = (lane < a.nsub) ? load_sum(&a.part_lm[2 * (p0 + lane)]) : 0.0;
        mass1 = (kWave + lane < a.nsub) ? load_sum(&a.part_lm[2 * (p0 + kWave + lane)]) : 0.0;
    }
    {   // what the rejected children's tokens carry (the same arithmetic as pass (b) uses)
        float xj = -INFINITY;
        int sj = -1;
        if (lane < nrej && rejtok >= 0 && rejtok < a.V) {
            xj = rejx;
            sj = rejtok / kAccSub;
        }
        s.rej_e[lane] = sj < 0 ? 0.0 : (double)(a.exact_scale ? scaled_exp<true>(xj, a, M) : scaled_exp<false>(xj, a, M));
        s.rej_sub[lane] = sj;
        wave_lds_sync();
    }
    const double target = (double)ubonus * (1.0 - R) * L;
    double before = 0.0;                                     // mass of the blocks before this group of 64
    int pick = -1, lastc = -1;
    double resid = 0.0;
    // what the blocks' masses are without the rejected tokens; two groups of 64 blocks at a time
    for (int c0 = 0; c0 < a.nsub && pick < 0; c0 += 2 * kWave) {
        double mass[2] = {mass0, mass1};
        if (c0 > 0) {
#pragma unroll
            for (int i = 0; i < 2; ++i) mass[i] = (c0 + i * kWave + lane < a.nsub) ? load_sum(&a.part_lm[2 * (p0 + c0 + i * kWave + lane)]) : 0.0;
        }
        for (int j0 = 0; j0 < nrej; j0 += 8) {                // broadcast LDS reads, eight in flight; entries
#pragma unroll                                                 // past nrej name no block
            for (int j = j0; j < j0 + 8; ++j) {
                const double e = s.rej_e[j];                 // read unconditionally: no branch per entry
                const int sub = s.rej_sub[j] - c0;
                mass[0] -= (sub == lane) ? e : 0.0;
                mass[1] -= (sub == kWave + lane) ? e : 0.0;
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int cs = c0 + i * kWave + lane;
            const double m = mass[i] > 0.0 ? mass[i] : 0.0;
            const double incl = before + wave_scan_f64(m);
            const uint64_t hit = __ballot(cs < a.nsub && incl > target);
            const uint64_t pos = __ballot(cs < a.nsub && m > 0.0);
            if (pick < 0) {
                if (pos) lastc = c0 + i * kWave + 63 - __clzll((long long)pos);
                if (hit) {
                    const int hl = __ffsll((long long)hit) - 1;
                    pick = c0 + i * kWave + hl;
                    resid = target - (readlane_f64(incl, hl) - readlane_f64(m, hl));
                }
                before = readlane_f64(incl, kWave - 1);
            }
        }
    }
    if (pick < 0) {                                          // rounding pushed the target past the total:
        pick = lastc >= 0 ? lastc : 0;                       // the last token with mass is taken
        resid = INFINITY;
    }

    // ---- residual draw, (b): inside the chosen block every lane owns 16 consecutive tokens
    s.rej_bits[lane] = 0;
    wave_lds_sync();
    if (lane < nrej && rejtok >= 0 && rejtok / kAccSub == pick) {
        const int off = rejtok - pick * kAccSub;
        atomicOr(&s.rej_bits[off / kAccEPT], 1u << (off % kAccEPT));
    }
    // The block is asked for first, then this row counted (everything else asked for has been used by now, and the stores are
    // acknowledged while the block is on its way); the count is looked at when the token is out.
    float xv[kAccEPT];
    int first[kAccEPT / 4];
    load_block<VEC4, true>(xr, pick * kAccSub, a.V, xv, first);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    unsigned int rows_before = 0;
    if (lane == 0) rows_before = __hip_atomic_fetch_add(seq_counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wave_lds_sync();
    const unsigned int rejected = s.rej_bits[lane];
    const int i0 = pick * kAccSub + lane * kAccEPT;
    // (Every lane adds up its sixteen exponentials and leaves them in LDS, from where the sixteen of the lane that the target
    // falls into are taken one per lane.)
    if (a.exact_scale) {
#pragma unroll
        for (int e = 0; e < kAccEPT; ++e) xv[e] = scaled_exp<true>(xv[e], a, M);
    } else {
#pragma unroll
        for (int e = 0; e < kAccEPT; ++e) xv[e] = scaled_exp<false>(xv[e], a, M);
    }
    double sum = 0.0;
    int lastpos = -1;
#pragma unroll
    for (int e = 0; e < kAccEPT; ++e) {
        xv[e] = (i0 + e < a.V && !((rejected >> e) & 1)) ? xv[e] : 0.f;
        sum += (double)xv[e];
        if (xv[e] > 0.f) lastpos = i0 + e;
    }
#pragma unroll
    for (int g = 0; g < kAccEPT / 4; ++g)
        reinterpret_cast<float4 *>(s.mass)[lane * (kAccEPT / 4) + g] = make_float4(xv[4 * g], xv[4 * g + 1], xv[4 * g + 2], xv[4 * g + 3]);
    wave_lds_sync();
    const double incl = wave_scan_f64(sum);
    const uint64_t hit = __ballot(incl > resid);
    int bonus = (int)wave_max_u32((uint32_t)(lastpos + 1)) - 1;          // last token of the block with mass
    if (hit) {
        const int owner = __ffsll((long long)hit) - 1;
        const float pe = lane < kAccEPT ? s.mass[owner * kAccEPT + lane] : 0.f;
        const double cdf = (readlane_f64(incl, owner) - readlane_f64(sum, owner)) + wave_scan_f64((double)pe);
        const uint64_t with_mass = __ballot(pe > 0.f), past = with_mass & __ballot(cdf > resid);
        // (rounding may leave none past the target: the owner's last token with mass)
        const int e = past ? __ffsll((long long)past) - 1 : with_mass ? 63 - __clzll((long long)with_mass) : -1;
        if (e >= 0) bonus = pick * kAccSub + owner * kAccEPT + e;
    }
    if (lane == 0) a.bonus[b] = bonus;
    finish_row(readlane_u32(rows_before, 0));
}

__global__ void validate_tree_kernel(const int32_t *parents, const int32_t *n_nodes, int B, int T, int32_t *bad) {
    __shared__ int count;
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < B * T; i += blockDim.x) {
        const int b = i / T, n = i % T;
        int nn = n_nodes ? n_nodes[b] : T;
        nn = max(1, min(nn, T));
        if (n < nn) {
            const int p = parents[i];
            const bool ok = (n == 0) ? (p == -1) : (p >= 0 && p < n);
            if (!ok) atomicAdd(&count, 1);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) *bad = count;
}

}  // namespace radar

using namespace radar;

// Workspace layout: arrival counters (one 64-byte slot per row and per sequence), row results,
// per-wavefront partials.  Returns the total size; fills the pointers when `ws` is given.
static size_t accept_layout(int B, int T, size_t nsub, char *ws, AcceptArgs *a) {
    const size_t rows = (size_t)B * T, slots = rows * nsub;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~size_t(255); return o; };
    const size_t o_cnt = take((rows + 2 * (size_t)B) * kAccCounterStride * sizeof(unsigned int));
    // Keys (greedy) or pairs (sampling) of the rows, then of the blocks, in the same places; the size is one that callers keep, so what was
    // there for each row and block (20 bytes) stays.
    const size_t o_row = take(rows * sizeof(uint64_t));
    take(rows * sizeof(uint64_t));
    take(rows * sizeof(float));
    const size_t o_part = take(slots * sizeof(uint64_t));
    take(slots * sizeof(uint64_t));
    take(slots * sizeof(float));
    if (ws) {
        a->counters = reinterpret_cast<unsigned int *>(ws + o_cnt);
        a->row_key = a->row_lm = reinterpret_cast<uint64_t *>(ws + o_row);
        a->part_key = a->part_lm = reinterpret_cast<uint64_t *>(ws + o_part);
    }
    return off;
}

extern "C" size_t radar_verify_accept_workspace_bytes(const radar_accept_desc *d) {
    if (!d || d->B < 1 || d->T_max < 1 || d->V < 1) return 0;
    const size_t nsub = ((size_t)d->V + kAccSub - 1) / kAccSub;
    return accept_layout(d->B, d->T_max, nsub, nullptr, nullptr);
}

template <int MODE, bool LAST>
static hipError_t launch_mode(const char *name, bool vec4, int nb, dim3 grid, dim3 block, hipStream_t st, const AcceptArgs &a) {
    if (nb == 1)
        return vec4 ? launch(name, accept_kernel<MODE, LAST, true, 1>, grid, block, 0, st, a) : launch(name, accept_kernel<MODE, LAST, false, 1>, grid, block, 0, st, a);
    return vec4 ? launch(name, accept_kernel<MODE, LAST, true, 2>, grid, block, 0, st, a) : launch(name, accept_kernel<MODE, LAST, false, 2>, grid, block, 0, st, a);
}

static radar_status launch_accept(const float *target_logits, const int32_t *draft_tokens, const int32_t *parents,
                                  const int32_t *n_nodes, const float *uniforms, int32_t *accept_len,
                                  int32_t *accept_path, int32_t *bonus_token, double *dist, int mode,
                                  const radar_accept_desc *d, void *workspace, size_t workspace_bytes, void *stream) {
    if (d->B < 1 || d->T_max < 1 || d->V < 1 || d->D_max < 0) return RADAR_INVALID_ARG;
    if (mode != RADAR_ACCEPT_GREEDY && !(d->temperature > 0.0f)) return RADAR_INVALID_ARG;
    const int64_t nsub = ((int64_t)d->V + kAccSub - 1) / kAccSub;
    // Blocks per wavefront: one gives the most wavefronts and the shortest chain for each; launches of many rounds
    // take two, half the workgroups to start, to be told that their row is not needed and to count.  61 rows of
    // V = 128256, sampled, paths of two nodes: 4 sequences 17.4 us with one and 22.1 with two, 8 sequences 25.1 and 21.9, 16
    // sequences 39.1 and 27.9 (four took 30 % longer than two: fewer bytes in flight for the rows that are needed).
    const int nb = (int64_t)d->B * d->T_max * nsub >= kAccManyBlocks ? 2 : 1;
    const int64_t nwg = (nsub + kAccWaves * nb - 1) / (kAccWaves * nb);
    if (d->T_max > RADAR_T_MAX || d->D_max >= RADAR_T_MAX || d->B > 65535 || nsub > kAccMaxSubs)
        return RADAR_UNSUPPORTED_SHAPE;
    if (workspace_bytes < radar_verify_accept_workspace_bytes(d)) return RADAR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)workspace & 255) != 0) return RADAR_INVALID_ARG;

    AcceptArgs a;
    a.logits = target_logits; a.tokens = draft_tokens; a.parents = parents; a.n_nodes = n_nodes; a.uniforms = uniforms;
    a.accept_len = accept_len; a.accept_path = accept_path; a.bonus = bonus_token; a.dist = dist;
    a.B = d->B; a.T = d->T_max; a.V = d->V; a.D_max = d->D_max;
    a.nsub = (int)nsub; a.nwg = (int)nwg;
    a.inv_temp = mode != RADAR_ACCEPT_GREEDY ? 1.0 / (double)d->temperature : 1.0;
    a.inv_temp_f = (float)a.inv_temp;
    a.exact_scale = ((double)a.inv_temp_f == a.inv_temp) ? 1 : 0;
    accept_layout(d->B, d->T_max, (size_t)nsub, static_cast<char *>(workspace), &a);
    // Large launches: the roots' rows are read first and alone, the workgroups behind them wait for the roots' decisions (the
    // memory's queue is first come, first served: 2048 workgroups that read at once are 64 MB ahead of the roots' results, whose
    // rows were complete after 9.5 us instead of 6.7).  Greedy 2.5 us, sampled 4.5 (its decisions are later; 3.5 and 4.0 take the same, 5.5
    // one per cent more).  Those wait that start with the launch, by their number (rows past the end of a tree count too): eight workgroups
    // per CU of the greedy kernel, six of the sampled one, which is what the chip holds.  Ending at 1792 in greedy launches is slower (16 sequences of 61 rows,
    // V = 128256, paths of 0, 2 and 8 nodes 18.1, 26.7, 39.6 us; 17.8, 24.7, 36.9 at 2048).
    // Looking once before the wait changes nothing (1 %); with every workgroup waiting until the roots are decided V = 1048576 gains
    // 4-9 % (4 sequences 46.6, 56.1, 96.8 -> 44.8, 52.7, 88.2) and V = 128256 loses as much (16 sequences 17.4, 24.6, 35.3 -> 19.2, 25.6, 35.9).
    // us without / with the wait, trees of 61 rows, paths of 0, 2 and 8 nodes: greedy, V = 128256, 4 sequences 14.4 / 11.4, 16.6 / 16.3, 21.6 / 19.8;
    // 16 sequences 23.6 / 17.5, 27.4 / 24.6, 39.6 / 35.0; V = 1048576, 4 sequences 50.3 / 47.7, 59.0 / 56.3, 99 / 96.5; sampled, V = 128256, 8
    // sequences 20.6 / 15.5, 23.8 / 21.9, 33.1 / 30.5; 16 sequences 28.0 / 22.9, 31.4 / 27.9, 45.0 / 40.7.  Smaller launches lose
    // by it (sampled, V = 128256, 4 sequences 15.4 / 15.0, 17.4 / 18.9, 24.5 / 25.3; V = 32000, 16 sequences 15.9 / 16.0, 17.7 / 19.5, 25.2 / 27.0;
    // greedy, 8 sequences of V = 32000 10.3 / 10.7).
    // So do small trees in a launch that is large by T_max alone, once the path leaves the root (16 trees of 6 nodes, T_max = 64, paths of
    // 0, 2 and 5 nodes: greedy, V = 32000 6.0 / 7.2, 7.5 / 11.2, 8.0 / 11.6; 0, 2 and 4 nodes, sampled, V = 128256 13.3 / 10.3, 15.6 / 19.1, 16.9 / 20.2).  Only trees
    // wait with which the launch would be half a large one if all were like them; reading the others' sizes is not worth it
    // (every workgroup starts later then: 16 x 61 rows 17.5 -> 22.4).  16 trees of 12 nodes, T_max = 64, paths of 0, 2 and 4 nodes, greedy,
    // V = 32000 8.7 / 7.6, 9.5 / 12.3, 10.5 / 12.7, of 24 nodes 12.6 / 8.5, 13.3 / 12.6, 13.6 / 13.1.  With a whole large one instead of half, batches of
    // unlike trees lose: 16 of 2 to 60 nodes (377 rows), sampled, V = 128256, paths of 0, 1 and 2 nodes 15.7, 23.3, 25.7 us when all wait, 15.6, 22.3, 24.7
    // with half, 17.3, 22.5, 25.4 with a whole.
    const int64_t blocks = (int64_t)d->B * d->T_max * nsub;
    const bool wait = mode == RADAR_ACCEPT_GREEDY ? blocks >= kAccManyBlocks / 2 : mode == RADAR_ACCEPT_SAMPLE && blocks >= kAccManyBlocks;
    a.check_from = wait ? (int)(d->B * nwg) : kAccUnchecked;
    a.wait = mode == RADAR_ACCEPT_GREEDY ? 250 : 450;
    a.wait_until = wait ? (mode == RADAR_ACCEPT_GREEDY ? 2048 : 1536) : 0;
    a.wait_nodes = (int)std::max<int64_t>(kAccWaitNodes, (mode == RADAR_ACCEPT_GREEDY ? kAccManyBlocks / 4 : kAccManyBlocks / 2) / (d->B * nsub));
    // A greedy walk is shortest at the end of the launch, in registers over all rows' results, as long as the launch
    // is not much more than the chip holds at once (one sequence of 16 rows, V = 32000: 5.6 us against 7.1; two of
    // 61 rows, V = 128256, 3904 workgroups: 13.9 against 13.3).  A sampled one is not: its exponentials and the
    // draw's block masses are better taken as the rows end (61 rows, V = 128256, when this was decided: 14.3 us at the end, 12.9 on the way).
    const bool last = mode == RADAR_ACCEPT_GREEDY && (int64_t)d->B * d->T_max * nwg <= kAccWalkLast;

    const dim3 grid((unsigned)nwg, (unsigned)d->B, (unsigned)d->T_max), block(kAccThreads);
    const bool vec4 = (d->V % 4 == 0) && (((uintptr_t)target_logits & 15) == 0);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const char *name = mode == kAccDistribution ? "accept_length_distribution" : "accept";
    const auto go = mode == kAccDistribution ? launch_mode<kAccDistribution, false>
                    : mode == RADAR_ACCEPT_SAMPLE ? launch_mode<RADAR_ACCEPT_SAMPLE, false>
                                                  : (last ? launch_mode<RADAR_ACCEPT_GREEDY, true> : launch_mode<RADAR_ACCEPT_GREEDY, false>);
    const hipError_t e = go(name, vec4, nb, grid, block, st, a);
    return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
}

extern "C" radar_status radar_verify_accept(const float *target_logits, const int32_t *draft_tokens,
                                            const int32_t *parents, const int32_t *n_nodes, const float *uniforms,
                                            int32_t *accept_len, int32_t *accept_path, int32_t *bonus_token,
                                            const radar_accept_desc *d, void *workspace, size_t workspace_bytes,
                                            void *stream) {
    if (!d || !target_logits || !draft_tokens || !parents || !accept_len || !accept_path || !bonus_token || !workspace)
        return RADAR_INVALID_ARG;
    if (d->mode != RADAR_ACCEPT_GREEDY && d->mode != RADAR_ACCEPT_SAMPLE) return RADAR_INVALID_ARG;
    if (d->mode == RADAR_ACCEPT_SAMPLE && !uniforms) return RADAR_INVALID_ARG;
    return launch_accept(target_logits, draft_tokens, parents, n_nodes, uniforms, accept_len, accept_path, bonus_token,
                         nullptr, d->mode, d, workspace, workspace_bytes, stream);
}

extern "C" radar_status radar_accept_length_distribution(const float *target_logits, const int32_t *draft_tokens,
                                                         const int32_t *parents, const int32_t *n_nodes, double *dist,
                                                         const radar_accept_desc *d, void *workspace,
                                                         size_t workspace_bytes, void *stream) {
    if (!d || !target_logits || !draft_tokens || !parents || !dist || !workspace) return RADAR_INVALID_ARG;
    return launch_accept(target_logits, draft_tokens, parents, n_nodes, nullptr, nullptr, nullptr, nullptr, dist,
                         kAccDistribution, d, workspace, workspace_bytes, stream);
}

extern "C" radar_status radar_debug_validate_tree(const int32_t *parents, const int32_t *n_nodes, int32_t B,
                                                  int32_t T_max, int32_t *bad_count_out, void *stream) {
    if (!parents || !bad_count_out || B < 1 || T_max < 1) return RADAR_INVALID_ARG;
    const hipError_t e = launch("validate_tree", validate_tree_kernel, dim3(1), dim3(256), 0,
                                static_cast<hipStream_t>(stream), parents, n_nodes, (int)B, (int)T_max, bad_count_out);
    return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
}
