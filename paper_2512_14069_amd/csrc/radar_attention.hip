// Tree-verify attention for RADAR's target pass (Sec. 1: the draft tree is serialized
// and verified with masked attention in one LLM pass; Sec. 3), hand-written for
// gfx950: bf16 MFMA 32x32x16, 64-wide wavefronts, KV tiles staged through LDS.
//
// Inside a wavefront everything is kept transposed: S^T = K Q^T (keys x queries)
// and O^T = V^T P^T (head-dim x queries).  With the MFMA accumulator layout a lane
// then owns ONE query column: its softmax statistics need no cross-lane traffic
// beyond one exchange with lane^32, the rescaling factor is lane-local, and the
// exponentiated scores already sit in the register order the next MFMA wants as
// its B operand (the key order inside a 16-key step is permuted consistently for
// P^T and V^T, which a contraction does not care about).  The running output is
// rescaled only when some lane's maximum has risen past its reference by a factor of 256.
//
// The ancestor mask is never materialised in memory: a wavefront finds the ancestor
// sets of all rows by doubling over parents[], and each lane keeps its query row's as one
// 64-bit word; a tile that lies entirely in the prefix skips masking altogether.
//
// Work decomposition.  A workgroup of eight wavefronts owns (sequence, KV head,
// range of cache rows, block of eight (query head, 32 tree rows) units); each
// wavefront is one unit, and all eight share every K/V tile through LDS, so KV
// comes from HBM once per group of heads.  Two wavefronts per SIMD let one
// wavefront's MFMAs run underneath the other's softmax arithmetic.  Tiles are
// double-buffered in LDS (one barrier per tile) and the next tile's global loads
// are in flight during the arithmetic.  Ranges of cache rows are merged from partials
// (fp16 pairs scaled per row, plus maximum, sum and scale in fp32) by a small second kernel.  Short
// ranges: how many to cut is decided on the host from a cost model that counts whole rounds of
// resident workgroups and the partial traffic.  Long ranges: the workgroups read the lengths and
// deal the batch's cache rows out among themselves, so that a batch of unlike sequences keeps every
// CU busy to the end.  Short contexts: one launch, a workgroup per unit over all rows, merged in LDS.
#include "radar_device.h"
#include <algorithm>
#include <type_traits>
#include "radar_host.h"

namespace radar {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));     // a 16-byte load/store unit kept in registers
typedef float float3u __attribute__((ext_vector_type(3), aligned(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

constexpr int kAttnThreads = 256;
constexpr int kAttnWaves = 4;
constexpr int kKT = 64;                    // cache rows per LDS tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMaxSlack = 8.0f;          // how far a row's maximum may pass its reference (log2 units; tile_softmax)
constexpr float kNegBig = -1.0e30f;        // finite stand-in for "no score yet" (log2 units)

// (Each kernel takes what its first loads wait for as leading scalar arguments beside this: those are in registers when it
// starts, the rest is a round trip of 0.25 us.)
struct AttnArgs {
    const __bf16 *q, *k, *v;
    const int32_t *parents, *ctx_lens, *n_nodes;
    __bf16 *out;
    float *lse;
    int B, T, Hq, Hkv, G, S, kps, max_splits, n_ublk, nqb;   // nqb 32-row blocks per head, n_ublk workgroups per KV range
    int64_t q_sb, q_st, q_sh, kv_sb, kv_sh, kv_ss, o_sb, o_st, o_sh;
    float scale_log2;                      // softmax scale * log2(e), > 0
    uint32_t shares_inv;                   // ceil(2^32 / shares)
    int per_unit;                          // shares / (B * Hkv)
    int shares;                            // > 0: the rows are dealt out on the device, to so many workgroups per unit block
    uint64_t *part_o;                      // [slot][n_ublk * 8][D/8][32][8]: partial outputs, fp16, scaled per row
    uint64_t *unit_tab;                    // [B][Hkv] dealt-out rows: first slot (low half) and number of a head's partials (high half)
    float *part_ml;                        // [slot][n_ublk * 8][32][3]: running maximum (log2 units), sum, and the scale of part_o
};

// Byte offset of the 16-byte chunk `chunk` of cache row `key` in a K tile.  The chunks of a row are
// XOR-swizzled with the row number so that the sixteen lanes of one pass of a 16-byte operand read
// (sixteen consecutive rows, the same chunk) cover all 64 banks: 16 distinct chunk slots at D = 128
// (256-byte rows), 8 slots times the two rows of a 256-byte bank period at D = 64.
template <int D>
__device__ __forceinline__ int ks_swz(int key) {
    constexpr int CH = D / 8;
    return (key >> (CH == 16 ? 0 : 1)) & (CH - 1);
}
template <int D>
__device__ __forceinline__ int ks_off(int key, int chunk) { return key * (D * 2) + ((chunk ^ ks_swz<D>(key)) << 4); }
// byte offset of element (d, pos) of a transposed V tile; pos = permuted key slot.
// 16-byte groups of a row are XOR-swizzled so that both the transposing writes
// (lanes differ in d/8) and the operand reads (lanes differ in d) spread over banks.
__device__ __forceinline__ int vt_off(int d, int pos) {
    const int f = (d ^ (d >> 3)) & 7;
    return d * (kKT * 2) + ((((pos >> 3) ^ f) & 7) << 4) + ((pos & 7) << 1);
}
// slot of key kappa (0..63) inside a tile: bits 2 and 3 swapped, so that the 8 values a
// lane holds in accumulator registers [8s, 8s+8) line up with MFMA k-slots [8*g2, 8*g2+8).
__device__ __forceinline__ int key_slot(int kappa) {
    return (kappa & ~12) | ((kappa & 4) << 1) | ((kappa & 8) >> 1);
}

// byte offset of 16-byte chunk `chunk` of row `row` in a row-major V tile that is read by transposing
// LDS reads: one pass of such a read (32 lanes) touches 64 consecutive bytes of four consecutive rows,
// and rows 256 bytes apart would meet in the same banks; the row's two low bits (128-byte rows: the second) move its
// 64-byte windows apart.  (8 rows + 8 keeps the swizzle: the second read of a pair differs by a constant.)
template <int D>
__device__ __forceinline__ int vs_swz(int row) { return D == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2; }
template <int D>
__device__ __forceinline__ int vs_off(int row, int chunk) { return row * (D * 2) + ((chunk ^ vs_swz<D>(row)) << 4); }

// What loads that write LDS directly read for V rows past the end: a masked row's probability is 0, and 0 * Inf would be NaN.
// (Clearing the rows in LDS afterwards cost a call over 272 rows 2 %.)
__device__ __attribute__((aligned(16))) const uint32_t kZeroChunk[4] = {0, 0, 0, 0};

// Rows of the prefix: at most the cache's, so that the tree's rows can be added in 32 bits for any content of
// ctx_lens (a length near 2^31 would wrap, and the sequence seem empty to one kernel and not to the next).
// Where the prefix fills the cache nothing is left for the tree, as before.  Negative: no such sequence.
__device__ __forceinline__ int prefix_rows(const AttnArgs &a, int b) { return min(a.ctx_lens[b], a.S); }                     // b: per lane
__device__ __forceinline__ int prefix_rows_of(const AttnArgs &a, int b) { return min(uniform_word(a.ctx_lens, b), a.S); }    // b: the workgroup's

// v = keep ? v : 0 without a branch (a select after a load tempts the compiler into a
// conditional load, and conditional loads into register arrays wreck register allocation)
__device__ __forceinline__ void and_mask(u32x4 &v, bool keep) {
    v &= 0u - (uint32_t)keep;
}

// Ancestor word of this lane's tree row (bit a set <=> a is the row or an ancestor of it), lane = row; p: the
// row's parent.  Valid and in bounds for any content: a parent counts only if it is an earlier row.  By
// doubling: after r rounds a lane holds the 2^r nearest ancestors (itself included) and the next one's
// number, so a tree of depth 8 takes four rounds of lane gathers (walking up through LDS took eight dependent reads
// and a barrier; a chain of 60 rows 3 us).  All lanes call.
__device__ __forceinline__ uint64_t ancestor_words(int p, int nn) {
    const int lane = lane_id();
    uint32_t lo = lane < 32 ? 1u << lane : 0u, hi = lane < 32 ? 0u : 1u << (lane - 32);
    p = (lane < nn && p < lane) ? p : -1;
    while (__ballot(p >= 0) != 0ull) {
        const int src = max(p, 0);
        const uint32_t l2 = (uint32_t)__shfl((int)lo, src), h2 = (uint32_t)__shfl((int)hi, src);
        const int p2 = __shfl(p, src);
        if (p >= 0) { lo |= l2; hi |= h2; p = p2; }
    }
    return (uint64_t)hi << 32 | lo;
}
// the word of row i, whose lane it is; rows past the tree have none
__device__ __forceinline__ uint64_t ancestor_word_of(uint64_t words, int i, int nn) {
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)words, i), hi = (uint32_t)__shfl((int)(uint32_t)(words >> 32), i);
    return i < nn ? (uint64_t)hi << 32 | lo : 0ull;
}

// One wavefront, one tile of SUBS x 32 rows that sits in LDS, in three phases: scores into
// `sacc` (register r of sub-tile `sub` is row 32*sub + 8*(r/4) + 4*g2 + r%4), masked online softmax
// from `sacc` into the bf16 operand `pk` (rescaling the output accumulators when the maximum moved far),
// and the update of the transposed output accumulators, from a transposed V tile (vt_off) or, with
// VTR, from a row-major one (vs_off) through transposing LDS reads.
// The lane's query operands are passed in registers (qop: row j32 of the block, d = 16*st + 8*g2
// .. +8; 32 VGPRs at D = 128): every LDS byte not read matters here, the eight wavefronts of a
// workgroup already read each K and V tile eight times over.  K operands are read from LDS four
// MFMAs before they are needed and the two score sub-tiles (the four output blocks) take turns, so
// that consecutive MFMAs are independent and none starts by waiting for LDS.
//   t0        cache row of the tile's first key;  L = prefix length;  kend = end of this range
//   first     true if the accumulators are still zero (no rescaling needed)
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef const __attribute__((address_space(3))) u32x4 *lds_u32x4;

// kaddr(k): where step k's K operand sits in LDS (sub-tile k % SUBS, 16-byte chunk 2 * (k / SUBS) + g2 of row j32)
template <int D, int SUBS, typename KAddr>
__device__ __forceinline__ void tile_scores(KAddr kaddr, const bf16x8 (&qop)[D / 16], floatx16 (&sacc)[SUBS]) {
    constexpr int KSTEPS = D / 16, NS = SUBS * KSTEPS, kAhead = 4;
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[sub][r] = 0.f;
    auto kread = [&](int k) { return *kaddr(k); };
    u32x4 kf[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) kf[k] = kread(k);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const u32x4 cur = kf[k % kAhead];
        if (k + kAhead < NS) kf[k % kAhead] = kread(k + kAhead);
        sacc[k % SUBS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, cur), qop[k / SUBS], sacc[k % SUBS], 0, 0, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);          // the order written above, for the scheduler
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (k + kAhead < NS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
}

template <int D, int SUBS>
__device__ __forceinline__ void tile_softmax(floatx16 (&sacc)[SUBS], floatx16 (&oacc)[D / 32][1], float &m_run, float &l_run,
                                           uint64_t anc, int t0, int L, int kend, bool first, float scale_log2, float slack,
                                           bf16x8 (&pk)[SUBS][2]) {
    constexpr int DB = D / 32, ROWS = 32 * SUBS;
    const int g2 = lane_id() >> 5;
    if ((t0 + ROWS > L) || (t0 + ROWS > kend)) {                     // wave-uniform; prefix tiles skip it
        const int pre = L - t0;                                      // prefix keys in this tile (may be <= 0 or >= 64)
        uint64_t allow = pre >= 64 ? ~0ull : (pre > 0 ? ((1ull << pre) - 1) : 0ull);
        if (pre > -64 && pre < 64) allow |= pre >= 0 ? (anc << pre) : (anc >> (-pre));
        const int len = kend - t0;
        if (len < 64) allow &= len > 0 ? ((1ull << len) - 1) : 0ull;
        allow >>= 4 * g2;
        const uint32_t aw[2] = {(uint32_t)allow, (uint32_t)(allow >> 32)};
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sacc[sub][r] = ((aw[sub] >> (8 * (r >> 2) + (r & 3))) & 1u) ? sacc[sub][r] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[sub][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // The reference the exponentials are taken against follows the maximum only when that has risen by
    // more than 8 (a factor of 256 in a probability): the maxima of 32 rows keep moving a little in most
    // tiles, and each move would cost rescaling the accumulators, a sixth of a tile's vector instructions.
    // Probabilities keep their eight bits and sums their fp32, but a row's largest probability is no longer
    // exactly 1: against 64 bits the output is off by 2.24e-3 (2-norm, N(0,1) scores, 2048 rows) instead of
    // 2.15e-3, by 1.86e-3 instead of 1.68e-3 with scores four times as wide, both mostly the output's own
    // rounding to bf16.  Time with / without the slack: 2048 rows 14.5 / 14.7 us, ragged 16 79.4 / 81.2,
    // 4 x 16384 rows with 64 heads 148.5 / 155.8.  (Short contexts in one launch take no slack: a wavefront has few steps.)
    const float mt = mx * scale_log2;                                // scale_log2 > 0; -inf stays -inf
    const float m_new = mt > m_run + slack ? mt : m_run;
    if (!first && __any(m_new != m_run)) {                           // wave-uniform
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][0][r] *= alpha;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    m_run = m_new;
    float rs = 0.f;
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[sub][r], scale_log2, -m_new));
            rs += p;
            pk[sub][r >> 3][r & 7] = (__bf16)p;
        }
    l_run += rs;
}

// vaddr(k, hi): VTR = false: where step k's V^T operand sits (16 bytes; hi unused); VTR = true: the 8-byte
// piece this lane names for the first (hi = 0) or second (hi = 1) transposing read of step k
template <int D, int SUBS, bool VTR, typename VAddr>
__device__ __forceinline__ void tile_pv(VAddr vaddr, const bf16x8 (&pk)[SUBS][2], floatx16 (&oacc)[D / 32][1]) {
    constexpr int DB = D / 32, NP = 2 * SUBS * DB, kAhead = 4;
    // V^T operand straight from the row-major tile, by two transposing LDS reads.  In each block of 16
    // lanes, lane 4j+q names an 8-byte piece (row kv0+j, elements 4q..4q+3 of the block's 16) and lane l
    // receives element l%4 of the pieces named by lanes 4j + l/4, j = 0..3: its own d for four
    // consecutive rows.  Rows 16ss + 4g2 .. +4 fill k-slots 8g2 .. 8g2+3 and the rows eight further on
    // fill 8g2+4 .. 8g2+7, which is where the P operand has them.
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    typedef bf16x4_t __attribute__((address_space(3))) *lds_b64;
    auto vread = [&](int k) {
        if constexpr (!VTR) {
            return __builtin_bit_cast(bf16x8, *(lds_u32x4)vaddr(k, 0));
        } else {
            const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b64)vaddr(k, 0));
            const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b64)vaddr(k, 1));
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    bf16x8 vf[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) vf[k] = vread(k);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const bf16x8 cur = vf[k % kAhead];
        if (k + kAhead < NP) vf[k % kAhead] = vread(k + kAhead);
        const int db = k % DB, ss = k / DB;
        oacc[db][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, pk[ss >> 1][ss & 1], oacc[db][0], 0, 0, 0);
    }
}

// ===================================================================== group-share kernel
// 512 lanes: eight wavefronts, two per SIMD, so that one wavefront's MFMAs run underneath the
// other's softmax arithmetic.  A wavefront is one (query head, block of 32 tree rows); the eight of
// a workgroup share every K/V tile through LDS.
constexpr int kGsThreads = 512;
constexpr int kGsWaves = kGsThreads / kWave;

// Staging of one 64-row K/V tile by the 512 lanes of the workgroup, no request made twice and the
// same work for every wavefront (a wavefront that staged more than the others would reach the tile's
// barrier after them, and everybody would wait for it): every lane fetches 16-byte chunks of K rows
// (two at D = 128) and one V item = one chunk of two consecutive cache rows, which it interleaves
// into the transposed tile with 4-byte LDS writes.  Branch-free loads: rows past the range re-read
// the last valid row; V is zeroed on its way into LDS (0 * anything must stay 0; masking right
// after the load would make the wavefront wait for its own loads), K is masked by the softmax.
template <int D>
struct GsTileRegs {
    static constexpr int CH = D / 8;                                       // 16-byte chunks per row
    static constexpr int KL = kKT * CH / 512;                              // K chunks per lane: 2 at D = 128, 1 at D = 64
    static constexpr int VITEMS = CH * (kKT / 2);                          // (chunk, row pair) items: 512 at D = 128, 256 at D = 64
    u32x4 k[KL], v[2];
};

// (One straight line of loads, no separate path for tiles that need no clamping: wherever loads sit
// under a condition the compiler cannot tell how many are in flight at the store, and waits for all
// of them, the tile after next included.)
template <int D>
__device__ __forceinline__ void gs_load_tile(GsTileRegs<D> &g, const __bf16 *kbase, const __bf16 *vbase, int kv_ss,
                                             int t0, int kend, int tid) {
    constexpr int CH = GsTileRegs<D>::CH;
    const int item = min(tid, GsTileRegs<D>::VITEMS - 1);
    const int ch = item % CH, kp = item / CH;
#pragma unroll
    for (int i = 0; i < GsTileRegs<D>::KL; ++i) {
        const int c = i * 512 + tid;
        const int kpos = min(t0 + c / CH, kend - 1);
        g.k[i] = *reinterpret_cast<const u32x4 *>(kbase + (uint32_t)(kpos * kv_ss + (c % CH) * 8));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int kpos = min(t0 + 2 * kp + i, kend - 1);
        g.v[i] = *reinterpret_cast<const u32x4 *>(vbase + (uint32_t)(kpos * kv_ss + ch * 8));
    }
}

// t0, kend: the tile's first cache row and the end of the range, as given to gs_load_tile
template <int D>
__device__ __forceinline__ void gs_store_tile(const GsTileRegs<D> &g, unsigned char *Ks, unsigned char *Vt, int t0, int kend,
                                              int tid) {
    constexpr int CH = GsTileRegs<D>::CH;
#pragma unroll
    for (int i = 0; i < GsTileRegs<D>::KL; ++i) {
        const int c = i * 512 + tid;
        *reinterpret_cast<u32x4 *>(Ks + ks_off<D>(c / CH, c % CH)) = g.k[i];
    }
    if (tid < GsTileRegs<D>::VITEMS) {
        const int ch = tid % CH, kp = tid / CH;
        u32x4 v0 = g.v[0], v1 = g.v[1];
        if (t0 + kKT > kend) {                                             // wave-uniform: a range's last tile only
            and_mask(v0, t0 + 2 * kp < kend);
            and_mask(v1, t0 + 2 * kp + 1 < kend);
        }
        const int pos0 = key_slot(2 * kp);                                 // even; the pair's second row sits next to it
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            // elements 2*e2 (low halves) and 2*e2+1 (high halves) of the two rows
            const uint32_t lo = (v0[e2] & 0xffffu) | (v1[e2] << 16);
            const uint32_t hi = (v0[e2] >> 16) | (v1[e2] & 0xffff0000u);
            *reinterpret_cast<uint32_t *>(Vt + vt_off(ch * 8 + 2 * e2, pos0)) = lo;
            *reinterpret_cast<uint32_t *>(Vt + vt_off(ch * 8 + 2 * e2 + 1, pos0)) = hi;
        }
    }
}

// x * scl and y * scl as fp16, rounded once each (v_fma_mixlo and mixhi: seen together they would be two products and a conversion).
__device__ __forceinline__ uint32_t two_halves(float x, float y, float scl) {
    _Float16 lo = (_Float16)(x * scl);
    asm("" : "+v"(lo));
    return __builtin_bit_cast(uint32_t, half2v{lo, (_Float16)(y * scl)});
}

// End of a group-share kernel: a lane owns query i; its accumulator registers O(db, r) hold
// d = 32*db + 8*(r/4) + 4*g2 + r%4 of the transposed output.
// direct: this wavefront saw all of its rows' keys; otherwise its result is partial number `entry`.
template <int D, typename Acc>
__device__ __forceinline__ void gs_finish(const AttnArgs &a, Acc O, float m_run, float l_run, int b, int h, int i, int nn,
                                          bool direct, int entry) {
    constexpr int DB = D / 32;
    const int g2 = lane_id() >> 5;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (direct) {
        if (i >= a.T) return;
        __bf16 *orow = a.out + (size_t)b * a.o_sb + (size_t)i * a.o_st + (size_t)h * a.o_sh;
        const float inv = (i < nn && l_tot > 0.f) ? 1.0f / l_tot : 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                bf16x4 o4;
#pragma unroll
                for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(i < nn ? O(db, 4 * r4 + e) * inv : 0.f);
                *reinterpret_cast<bf16x4 *>(orow + 32 * db + 8 * r4 + 4 * g2) = o4;
            }
        if (a.lse && g2 == 0)
            a.lse[((size_t)b * a.T + i) * a.Hq + h] = (i < nn) ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : 0.f;
    } else {
        // Partial result of this key range: the row's output normalised by its own l and by the row's largest magnitude, as fp16 -- [D/8][32 rows][8
        // d], so that a wavefront's 16-byte stores cover 1024 contiguous bytes and the merge reads 16 bytes per lane -- plus (m, l, magnitude) of a
        // row next to each other in fp32.  The partials of all ranges together outweigh the K/V bytes, and writing them is what the tail of this
        // kernel waits for; halving them costs 2^-11 of the row's largest element in precision, an eighth of the bf16 rounding of the final output.
        // Written through: nothing is left dirty in L2 for the end of the kernel.
        // Two lanes share a row: the halves of two blocks of eight d change places, and each of the lanes stores 16 bytes of one.
        const int j32 = i & 31, slot = __builtin_amdgcn_readfirstlane(entry);
        const auto po = __builtin_amdgcn_make_buffer_rsrc(a.part_o + (size_t)slot * (D / 4 * 32), 0, D * 64, 0x00027000);
        const auto pml = __builtin_amdgcn_make_buffer_rsrc(a.part_ml + (size_t)slot * 96, 0, 96 * (int)sizeof(float), 0x00027000);
        const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
        float top[4] = {0.f, 0.f, 0.f, 0.f};                     // (one chain of maxima would be serial)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) top[r >> 2] = fmaxf(top[r >> 2], fabsf(O(db, r)));
        float amax = fmaxf(fmaxf(top[0], top[1]), fmaxf(top[2], top[3]));
        amax = fmaxf(amax, __shfl_xor(amax, 32)) * inv;          // both halves of the row's d range
        const float mag = amax > 0.f && amax < 3.0e38f ? amax : 1.f;
        const float scl = inv / mag;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int pair = 0; pair < 2; ++pair) {               // d = 32 * db + 16 * pair + 8 * (first or second) + 4 * g2 + 0..3
                uint32_t first[2], second[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    first[e] = two_halves(O(db, 8 * pair + 2 * e), O(db, 8 * pair + 2 * e + 1), scl);
                    second[e] = two_halves(O(db, 8 * pair + 4 + 2 * e), O(db, 8 * pair + 5 + 2 * e), scl);
                }
                const auto s0 = __builtin_amdgcn_permlane32_swap(first[0], second[0], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(first[1], second[1], false, false);
                const u32x4 eight = {s0[0], s1[0], s0[1], s1[1]};
                __builtin_amdgcn_raw_buffer_store_b128(eight, po, ((4 * db + 2 * pair + g2) * 32 + j32) * 16, 0, 16);
            }
        const u32x3 ml = {__builtin_bit_cast(uint32_t, m_run), __builtin_bit_cast(uint32_t, l_tot), __builtin_bit_cast(uint32_t, mag)};
        if (g2 == 0) __builtin_amdgcn_raw_buffer_store_b96(ml, pml, j32 * 12, 0, 16);
    }
}

struct GsKernArgs { const __bf16 *k, *v; int64_t kv_sb, kv_sh; int kv_ss, kps, S, blocks; const __bf16 *q; AttnArgs a; };
// blocks: n_ublk in the lower half, nqb in the upper
template <int D, bool DEEP>
__global__ __launch_bounds__(kGsThreads) void tree_attn_gs_kernel(const __bf16 *k_, const __bf16 *v_, int64_t kv_sb, int64_t kv_sh, int kv_ss_, int kps,
                                                                 int S, int blocks, const __bf16 *q_, AttnArgs) {
    constexpr int DB = D / 32;              // 32-row blocks of O^T

    constexpr int TILE = 2 * kKT * D * 2;   // one K tile ([64][D] bf16, swizzled) + one V^T tile ([D][64], swizzled)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int sp = blockIdx.x;
    // The blocks of units that share a range of cache rows are ranges x KV heads apart in workgroup number:
    // a multiple of eight with eight KV heads, and consecutive numbers go to consecutive XCDs, so the
    // blocks meet in one XCD's L2 and their rows come from HBM once.
    const int n_ublk = blocks & 0xffff, nqb = blocks >> 16, hk = blockIdx.y;
    int b = blockIdx.z, ublk = 0;
    if (n_ublk > 1) { b = blockIdx.z / n_ublk; ublk = blockIdx.z - b * n_ublk; }      // (a division is 30 dependent instructions before the first load)
    const int kbeg = sp * kps;                            // < S: the grid has ceil(S / kps) ranges

    const int u = ublk * kGsWaves + w;                    // (head within the group, block of 32 rows)
    const int g = u >> (nqb - 1), qb = u & (nqb - 1);
    const int j32 = lane & 31, g2 = lane >> 5;
    const int i = 32 * qb + j32;                          // this lane's tree row

    const __bf16 *kbase = k_ + (size_t)b * kv_sb + (size_t)hk * kv_sh;
    const __bf16 *vbase = v_ + (size_t)b * kv_sb + (size_t)hk * kv_sh;
    const int kv_ss = kv_ss_;                // 32-bit offsets inside one head's cache (checked on the host)

    // The first tile and the query rows are requested before the sequence's context length and tree size are known (two dependent scalar loads, most
    // of a microsecond in a cold start): rows are clamped to the cache the caller described instead of to the end of the range.  Whatever rows past
    // that end hold is never used: their scores are masked by selection and their V rows zeroed on the way into LDS, both from the range's real end
    // below.
    // DEEP (ranges of many tiles): staging runs two tiles ahead through two register sets, which hides HBM latency better but doubles the loop's
    // code; short ranges keep the compact one-ahead loop (their time goes into a cold start, where code size counts).
    // A range of two tiles asks for both at once (asked for after the first had come, the second was consumed 1.25 us after it: 32 heads over 2048
    // rows 13.5 us for the call, 12.6 with this and the shorter ways to the first loads here and in the merge); with more of them the first would
    // wait for the second's bytes (16 heads on 8 x 2 over 750 rows 10.7 -> 11.5).
    GsTileRegs<D> regs0, regs1;
    gs_load_tile<D>(regs0, kbase, vbase, kv_ss, kbeg, S, tid);
    const bool both = !DEEP && kps > kKT && kps <= 2 * kKT;
    if (both) gs_load_tile<D>(regs1, kbase, vbase, kv_ss, kbeg + kKT, S, tid);
    // The other arguments from here on (with two divisions they held up the first tile's loads by half a microsecond).
    AttnArgs a;
    {
        const ArgBlock<AttnArgs> p = args_from_here<AttnArgs>(offsetof(GsKernArgs, a));
        a.q_sb = p->q_sb; a.q_st = p->q_st; a.q_sh = p->q_sh; a.T = p->T; a.G = p->G; a.Hq = p->Hq; a.Hkv = p->Hkv; a.max_splits = p->max_splits;
        a.ctx_lens = p->ctx_lens; a.n_nodes = p->n_nodes; a.parents = p->parents; a.scale_log2 = p->scale_log2;
        a.out = p->out; a.lse = p->lse; a.o_sb = p->o_sb; a.o_st = p->o_st; a.o_sh = p->o_sh; a.part_o = p->part_o; a.part_ml = p->part_ml;
        a.S = S; a.kps = kps; a.n_ublk = n_ublk; a.q = q_;
    }
    const bool active = g < a.G;
    const int h = hk * a.G + (active ? g : 0);
    // this lane's query operands, kept in registers for the whole kernel: row i, d = 16*st + 8*g2 .. +8
    bf16x8 qop[D / 16];
    {
        const __bf16 *qrow = a.q + (size_t)b * a.q_sb + (size_t)h * a.q_sh + (uint32_t)(min(i, a.T - 1) * (int)a.q_st);
#pragma unroll
        for (int st = 0; st < D / 16; ++st) {
            u32x4 raw = *reinterpret_cast<const u32x4 *>(qrow + 16 * st + 8 * g2);
            and_mask(raw, active && i < a.T);
            qop[st] = __builtin_bit_cast(bf16x8, raw);
        }
    }
    const int L = prefix_rows_of(a, b);
    int nn = a.n_nodes ? uniform_word(a.n_nodes, b) : a.T;
    nn = max(1, min(nn, a.T));
    const int total = min(L + nn, a.S);                  // never read past the cache the caller described
    if (L < 0 || kbeg >= total) return;
    const int kend = min(total, kbeg + a.kps);
    const int nsplit = (total + a.kps - 1) / a.kps;
    const int ntiles = (kend - kbeg + kKT - 1) / kKT;
    if (DEEP) gs_load_tile<D>(regs1, kbase, vbase, kv_ss, kbeg + kKT, kend, tid);
    const int parent = a.parents[(size_t)b * a.T + min(lane, nn - 1)];
    gs_store_tile<D>(regs0, smem, smem + TILE / 2, kbeg, kend, tid);
    if (both && ntiles > 1) gs_store_tile<D>(regs1, smem + TILE, smem + TILE + TILE / 2, kbeg + kKT, kend, tid);
    __syncthreads();
    if (DEEP) gs_load_tile<D>(regs0, kbase, vbase, kv_ss, kbeg + 2 * kKT, kend, tid);
    else if (!both && ntiles > 1) gs_load_tile<D>(regs0, kbase, vbase, kv_ss, kbeg + kKT, kend, tid);
    uint64_t anc[1];
    anc[0] = kend > L ? ancestor_word_of(ancestor_words(parent, nn), i, nn) : 0ull;

    floatx16 oacc[DB][1];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][0][r] = 0.f;
    float m_run[1] = {kNegBig}, l_run[1] = {0.f};

    // Two tile buffers in LDS: while tile t is consumed from one, every wavefront drops its share of
    // tile t+1 into the other as soon as it is done with t.  One barrier per tile: it publishes tile
    // t+1 and tells that nobody reads tile t any more.
    auto step = [&](int t, GsTileRegs<D> &next_regs, int ahead) {
        unsigned char *cur = smem + (t & 1) * TILE, *nxt = smem + ((t + 1) & 1) * TILE;
        if (active) {
            floatx16 sacc[2];
            bf16x8 pk[2][2];
            const unsigned char *Vt = cur + TILE / 2;
            tile_scores<D, 2>([&](int k) { return (lds_u32x4)(cur + ks_off<D>(32 * (k & 1) + j32, 2 * (k >> 1) + g2)); }, qop, sacc);
            tile_softmax<D, 2>(sacc, oacc, m_run[0], l_run[0], anc[0], kbeg + t * kKT, L, kend, t == 0, a.scale_log2, kMaxSlack, pk);
            tile_pv<D, 2, false>([&](int k, int) { return (const lds_byte *)(Vt + vt_off(32 * (k % DB) + j32, 16 * (k / DB) + 8 * g2)); },
                              pk, oacc);
        }
        if (both) return;                                 // (there already)
        if (t + 1 < ntiles) {
            gs_store_tile<D>(next_regs, nxt, nxt + TILE / 2, kbeg + (t + 1) * kKT, kend, tid);
            __syncthreads();
        }
        // Two tiles ahead, the loads are issued whether or not the range still has such a tile (rows past
        // its end re-read its last row): only if every step issues the same loads does the compiler
        // know how many are in flight when a set is stored, and wait for that set alone.
        if (DEEP || t + ahead < ntiles) gs_load_tile<D>(next_regs, kbase, vbase, kv_ss, kbeg + (t + ahead) * kKT, kend, tid);
    };
    if (DEEP) {                                           // unrolled by two: odd tiles travel through regs1, even ones through regs0
        int t = 0;
        for (; t + 1 < ntiles; t += 2) {
            step(t, regs1, 3);
            step(t + 1, regs0, 3);
        }
        if (t < ntiles) step(t, regs1, 3);
    } else {
        for (int t = 0; t < ntiles; ++t) step(t, regs0, 2);
    }
    if (!active) return;
    gs_finish<D>(a, [&](int db, int r) { return oacc[db][0][r]; }, m_run[0], l_run[0], b, h, i, nn, nsplit == 1,
                 (((b * a.Hkv + hk) * a.max_splits + sp) * a.n_ublk + ublk) * kGsWaves + w);
}

// ===================================================================== dealing the rows out on the device
// The work of a launch over long ranges is one line of pairs of tiles: sequence by sequence, KV head by
// KV head, pair by pair, each with the time it takes.  It is cut into equal shares, one per workgroup,
// wherever the cuts fall; a workgroup takes the pieces of its share one after the other and leaves a
// partial result for each.  With a range of rows per workgroup fixed on the host by the longest
// sequence, a batch lasts as long as that sequence's ranges while the workgroups of the others have
// long left: 16 sequences of 700 ... 8192 rows (8 KV heads, 4 query heads each) took 121 us that way and
// take 80 us this way, 11 of them in the merge of their 380 pieces; what is left of the imbalance is the
// granule of a pair (4.5 us with the whole chip at work).
// All of it in units of an eighth of a full tile.
constexpr int kTileCost = 8;               // a tile for eight units
constexpr int kTileCostLight = 5;          // for at most half as many: the loads stay
constexpr int kUnitCost = 20;               // query rows, ancestor words and partials of a unit's first piece
constexpr int kFlatMaxB = kWave;           // one lane per sequence

struct FlatPlan {                          // lane = sequence
    int L, nn, pairs, cost, start, len;    // cost: of a tile; start: where the sequence's KV heads begin on the line, len each
    int total, share, unit;                // of the line; what a unit costs besides its tiles; the same in every lane
};

// Blocks of 32 rows that a sequence's tree fills; whether its units are at most half of what the workgroups
// hold; and, where those are then in half of the workgroups, that the other half takes the second half
// of every piece's rows.  (Inside one workgroup the idle wavefronts are left idle: having them take every
// second tile was no faster, the loads bound such a tile, and doubled the partials: 1-15 % slower.)
__device__ __forceinline__ int flat_row_blocks(const AttnArgs &a, int nn) { return nn <= 32 ? 1 : a.nqb; }
__device__ __forceinline__ bool flat_light(const AttnArgs &a, int nn) { return a.G * flat_row_blocks(a, nn) * 2 <= kGsWaves * a.n_ublk; }
__device__ __forceinline__ bool flat_shared(const AttnArgs &a, int nn) {
    return (a.n_ublk & 1) == 0 && a.G * flat_row_blocks(a, nn) * 2 == kGsWaves * a.n_ublk;
}

__device__ __forceinline__ FlatPlan flat_plan(const AttnArgs &a) {
    FlatPlan f;
    const int lane = lane_id(), b = min(lane, a.B - 1);
    f.L = prefix_rows(a, b);
    f.nn = a.n_nodes ? a.n_nodes[b] : a.T;
    f.nn = max(1, min(f.nn, a.T));
    const int rows = min(f.L + f.nn, a.S);
    const int tiles = (lane < a.B && f.L >= 0) ? (rows + kKT - 1) / kKT : 0;
    f.pairs = (tiles + 1) / 2;
    f.cost = flat_light(a, f.nn) && (a.n_ublk == 1 || flat_shared(a, f.nn)) ? kTileCostLight : kTileCost;
    f.unit = kUnitCost;
    f.len = tiles > 0 ? kUnitCost + tiles * f.cost : 0;
    const uint32_t mine = (uint32_t)(f.len * a.Hkv);
    const uint32_t incl = wave_scan_u32(mine);
    f.start = (int)(incl - mine);
    f.total = (int)readlane_u32(incl, kWave - 1);
    // Every piece of a unit costs writing and merging a partial, about 0.3 of a tile's time; with p pairs
    // per unit and s pairs per piece, s + 0.15 p / s is least at s = sqrt(0.15 p).
    const int most = (int)wave_max_u32((uint32_t)f.pairs);
    const int tile = __ballot(f.pairs == most && f.cost == kTileCostLight) != 0 ? kTileCostLight : kTileCost;
    const float merge = tile == kTileCost || a.n_ublk == 1 ? 0.15f : 0.3f;       // (two partials where keys are shared)
    const int least = max(2 * tile * (int)(__builtin_amdgcn_sqrtf(merge * (float)most) + 0.5f), kUnitCost + 2 * kTileCost);
    // total / shares rounded up (exactly so below 2^24; never less)
    f.share = max((int)__umulhi((uint32_t)(f.total + a.shares - 1), a.shares_inv), least);
    // Equal sequences: whole pieces, as long as they are not longer than a share with one more beginning in it.
    const int len0 = (int)readlane_u32((uint32_t)f.len, 0) - kUnitCost;
    if (a.per_unit > 0 && __ballot(lane < a.B && f.len - kUnitCost != len0) == 0 && len0 > 0) {
        const int whole = max((len0 + a.per_unit - 1) / a.per_unit, least);
        if (whole <= f.share + kUnitCost) {
            f.share = whole;
            f.unit = 0;
            f.len = lane < a.B ? (len0 + whole - 1) / whole * whole : 0;
            f.start = lane * a.Hkv * f.len;
            f.total = a.B * a.Hkv * (int)readlane_u32((uint32_t)f.len, 0);
        }
    }
    return f;
}

struct FlatUnit { int b, hk, start, pairs, cost, len, unit; };     // one sequence's KV head on the line

__device__ __forceinline__ FlatUnit flat_unit(const AttnArgs &a, const FlatPlan &f, int pos) {
    const uint64_t before = __ballot(f.len > 0 && f.start <= pos);
    FlatUnit u;
    u.unit = f.unit;
    u.b = 63 - __clzll((long long)before);
    const int base = (int)readlane_u32((uint32_t)f.start, u.b);
    u.len = (int)readlane_u32((uint32_t)f.len, u.b);
    u.pairs = (int)readlane_u32((uint32_t)f.pairs, u.b);
    u.cost = (int)readlane_u32((uint32_t)f.cost, u.b);
    u.hk = __popcll(__ballot(lane_id() < a.Hkv && base + lane_id() * u.len <= pos)) - 1;    // at most 64 KV heads
    u.start = base + u.hk * u.len;
    return u;
}
// The share that holds a pair's middle (its first tile's end: the second may be missing) takes it; the
// unit's own cost goes with its first pair.
__device__ __forceinline__ int flat_middle(const FlatUnit &u, int j) { return u.start + u.unit + (2 * j + 1) * u.cost - 1; }
// first pair whose middle is not before pos
__device__ __forceinline__ int flat_pair_at(const FlatUnit &u, int pos) {
    const uint32_t x = (uint32_t)max(pos - flat_middle(u, 0), 0);
    const uint32_t j = u.cost == kTileCost ? (x + 2 * kTileCost - 1) / (2 * kTileCost) : (x + 2 * kTileCostLight - 1) / (2 * kTileCostLight);
    return min(u.pairs, (int)j);
}

// ===================================================================== group-share kernel, long ranges
// The same decomposition with tiles that reach LDS without passing through registers: every wavefront
// issues four loads per tile that write LDS directly (1 KB each: four rows of K or V; a lane's 16 bytes
// land at the instruction's LDS base + 16 * lane, so the swizzle is applied by choosing which chunk of
// the row the lane fetches), a pair of tiles ahead of the pair being consumed, four tile buffers.  V
// stays row-major and is transposed by the LDS reads that fetch the operands.  No staging registers,
// no vector instructions for the transposition, one barrier per pair of tiles.  Rows past the end
// of a range re-read its last row in K, whose scores are masked, and are zeros in V.
constexpr int kLdBufs = 4;
// Ranges of so many tiles take it.  At eight the compact one-ahead loop still wins (16 sequences of up to 900
// rows 20.3 us against 22.0), at nine the long-range kernel (8 of up to 2000 rows 26.6 against 28.6).
// At D = 64 the choice is between one and two tiles ahead.  With one workgroup per CU two ahead gain 1 % at nine
// tiles and 3 % from sixteen on (one layer of 32 heads, 2048 rows in ranges of 9, 16 and 32 tiles: 17.2, 24.9 and 42.9 us
// against 17.4, 25.6 and 44.3); where workgroups are several rounds they lose 1-5 % at nine (32 sequences of 2048 rows
// 30.4 against 29.0), are even at sixteen and gain 2-4 % at 32.  The library's own ranges of nine tiles or more: 1-4 % gained.
constexpr int kLongTiles = 9;

// A lane's share of a tile: two chunks of K and two of V.  Wavefront w loads the row groups 2w and
// 2w + 1 (four rows, 1 KB each); the lane's 16 bytes land at the group's LDS base + 16 * lane, i.e. in
// slot lane % 16 of row 4 * group + lane / 16, so it fetches the chunk that the swizzle puts there.
// The byte offsets inside a tile are fixed for the kernel's lifetime.
struct LdLane {
    uint32_t offk[2], offv[2];        // from the tile's first row, rows kv_ss elements apart
};

template <int D>
__device__ __forceinline__ LdLane ld_lane_offsets(int kv_ss, int w, int lane) {
    static_assert(D == 128, "1 KB per instruction = four 256-byte rows");
    LdLane o;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = 4 * (2 * w + i) + (lane >> 4), slot = lane & 15;
        o.offk[i] = (uint32_t)(row * kv_ss) * 2 + (uint32_t)((slot ^ (row & 15)) << 4);          // inverse of ks_off's swizzle
        o.offv[i] = (uint32_t)(row * kv_ss) * 2 + (uint32_t)((slot ^ ((row & 3) << 2)) << 4);    // inverse of vs_off's
    }
    return o;
}

// One load of 16 bytes a lane that writes LDS directly, 1 KB from the byte address lds on (the same in every lane), from base + off
// or from the lane's own address.
// Issued as assembly: told about loads that write LDS, the compiler waits for all of them before the
// next LDS read it cannot tell apart from their targets, which would undo the run-ahead; the waits for
// these loads are the explicit ones in the kernels' loops.  (m0 is a reserved register: the compiler
// sets it right before each of its own uses and warns about the clobber.)  The load takes its LDS address from m0, which has to have been
// written one wait state before; inside assembly nobody but this adds it.
__device__ __forceinline__ void load_to_lds(uint32_t lds, const __bf16 *base, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void load_to_lds(uint32_t lds, const __bf16 *src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(src) : "memory", "m0");
}

// Issues this wavefront's four loads of the tile whose first cache row is t0 into the buffer `buf`.
// A tile inside the range
// takes a scalar base and the lane's fixed offsets, no vector arithmetic; a tile that reaches past the
// end of the range clamps every row to the range's last one in K and reads zeros in V.
template <int D>
__device__ __forceinline__ void ld_issue_tile(unsigned char *buf, const __bf16 *kbase, const __bf16 *vbase, int kv_ss, int t0,
                                              int kend, int w, int lane, const LdLane &o) {
    // (the wavefront's number is the same in every lane, which the compiler cannot see: the LDS bases below have to be scalars)
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)buf + (uint32_t)w * 2048);
    if (t0 + kKT <= kend) {                                          // wave-uniform
        // (the tile bases are the same in every lane; passed through readfirstlane so that they are scalars
        // for the assembly below whatever the compiler knows about their uniformity)
        auto scalar_ptr = [](const __bf16 *p) {
            const uint64_t v = (uint64_t)(uintptr_t)p;
            const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
            return (const __bf16 *)(uintptr_t)(((uint64_t)hi << 32) | lo);
        };
        const __bf16 *kt = scalar_ptr(kbase + (uint32_t)(t0 * kv_ss)), *vt = scalar_ptr(vbase + (uint32_t)(t0 * kv_ss));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t ldsk = lds0 + i * 1024, ldsv = ldsk + kKT * D * 2;
            load_to_lds(ldsk, kt, o.offk[i]);
            load_to_lds(ldsv, vt, o.offv[i]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = 4 * (2 * w + i) + (lane >> 4), slot = lane & 15;
            const uint32_t rowoff = (uint32_t)(min(t0 + row, max(kend, 1) - 1) * kv_ss);
            const __bf16 *gk = kbase + rowoff + ((slot ^ (row & 15)) << 3);
            const __bf16 *gv = t0 + row < kend ? vbase + rowoff + ((slot ^ ((row & 3) << 2)) << 3) : (const __bf16 *)kZeroChunk;
            const uint32_t ldsk = lds0 + i * 1024, ldsv = ldsk + kKT * D * 2;
            load_to_lds(ldsk, gk);
            load_to_lds(ldsv, gv);
        }
    }
}

// FLAT: the rows are dealt out on the device; otherwise one fixed range of kps rows per workgroup.
template <int D, bool FLAT>
__global__ __launch_bounds__(kGsThreads) void tree_attn_ld_kernel(const int32_t *ctx_lens, const int32_t *n_nodes, int T, int S, int B, int Hkv, int G,
                                                                 int n_ublk, int nqb, int shares, uint32_t shares_inv, int per_unit, AttnArgs a) {
    a.ctx_lens = ctx_lens; a.n_nodes = n_nodes; a.T = T; a.S = S; a.B = B; a.Hkv = Hkv; a.G = G;
    a.n_ublk = n_ublk; a.nqb = nqb; a.shares = shares; a.shares_inv = shares_inv; a.per_unit = per_unit;
    constexpr int DB = D / 32;
    constexpr int TILE = 2 * kKT * D * 2;   // one K tile ([64][D] bf16, swizzled) + one V tile (row-major, swizzled)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int j32 = lane & 31, g2 = lane >> 5;
    const int kv_ss = (int)a.kv_ss;          // 32-bit offsets inside one head's cache (checked on the host)
    // The blocks of units that share a range of cache rows are a multiple of eight apart in workgroup
    // number (256 / n_ublk shares; ranges x KV heads with eight KV heads), and consecutive numbers go to
    // consecutive XCDs, so the blocks meet in one XCD's L2 and their rows come from HBM once.
    const int ublk = FLAT ? (int)blockIdx.z : (int)(blockIdx.z % a.n_ublk);

    // a piece: tiles [t0, t1) of one sequence's KV head
    struct Piece {
        int b, hk, L, nn, kend;               // kend: end of the rows that count
        int t0, t1, slot;
        bool direct;
    };
    FlatPlan f;
    int pos = 0, end = 0;                     // what is left of this workgroup's share
    auto next_piece = [&](Piece &p) -> bool { // the first piece of [pos, end); all values the same in every lane
        while (pos < end) {
            const FlatUnit u = flat_unit(a, f, pos);
            const int j0 = flat_pair_at(u, pos), j1 = flat_pair_at(u, end);
            const bool whole = j0 == 0 && j1 == u.pairs;
            pos = u.start + u.len;
            if (j0 >= j1) continue;
            p.b = u.b; p.hk = u.hk;
            p.L = (int)readlane_u32((uint32_t)f.L, u.b);
            p.nn = (int)readlane_u32((uint32_t)f.nn, u.b);
            p.kend = min(p.L + p.nn, a.S);                    // never read past the cache the caller described
            p.t0 = 2 * j0;
            p.t1 = min(2 * j1, (p.kend + kKT - 1) / kKT);
            p.slot = (int)blockIdx.x + u.b * a.Hkv + u.hk;
            p.direct = whole && !flat_shared(a, p.nn) && flat_row_blocks(a, p.nn) == a.nqb;
            if (j0 == 0 && ublk == 0 && tid == 0) {           // for the merge (whose time is short; it does not plan again)
                const int pieces = flat_middle(u, u.pairs - 1) / f.share - (int)blockIdx.x + 1;
                a.unit_tab[u.b * a.Hkv + u.hk] = (uint64_t)(uint32_t)p.slot | (uint64_t)(uint32_t)(p.direct ? 0 : pieces) << 32;
            }
            return true;
        }
        return false;
    };
    Piece pc;
    if constexpr (FLAT) {
        f = flat_plan(a);
        pos = (int)blockIdx.x * f.share;
        end = min(pos + f.share, f.total);
        if (!next_piece(pc)) return;
    } else {
        const int sp = blockIdx.x;
        pc.b = blockIdx.z / a.n_ublk; pc.hk = blockIdx.y;
        pc.L = prefix_rows(a, pc.b);
        pc.nn = a.n_nodes ? a.n_nodes[pc.b] : a.T;
        pc.nn = max(1, min(pc.nn, a.T));
        const int total = min(pc.L + pc.nn, a.S);
        if (pc.L < 0 || sp * a.kps >= total) return;
        pc.kend = min(total, (sp + 1) * a.kps);
        pc.t0 = sp * (a.kps / kKT);
        pc.t1 = (pc.kend + kKT - 1) / kKT;
        pc.slot = (pc.b * a.Hkv + pc.hk) * a.max_splits + sp;
        pc.direct = total <= a.kps;
    }
    // Shared keys with the units in half of the workgroups: the other half takes the second half of the
    // piece's pairs (and, where there is one pair only, the same rows with none of them allowed).
    auto own_half = [&](Piece &p) {
        if (!FLAT || !flat_shared(a, p.nn)) return;
        const int mid = p.t0 + ((p.t1 - p.t0 + 3) / 4) * 2;
        if (2 * ublk < a.n_ublk) p.t1 = min(p.t1, mid);
        else if (mid < p.t1) p.t0 = mid;
        else p.L = p.nn = p.kend = 0;
    };
    // where the loads are, one pair ahead of the arithmetic
    const __bf16 *kb, *vb;
    int lt, lt1, lend;                                    // next tile, the piece's end, the end of the rows that count
    auto load_from = [&](const Piece &p) {
        const size_t at = (size_t)p.b * a.kv_sb + (size_t)p.hk * a.kv_sh;
        kb = a.k + at; vb = a.v + at;
        lt = p.t0; lt1 = p.t1; lend = p.kend;
    };

    // the first two tiles are requested before anything else: the query rows below are consumed as soon as
    // they arrive, and loads issued behind that wait would start a memory round trip late
    const LdLane ldo = ld_lane_offsets<D>(kv_ss, w, lane);
    own_half(pc);
    load_from(pc);
    ld_issue_tile<D>(smem, kb, vb, kv_ss, lt * kKT, lend, w, lane, ldo);
    ld_issue_tile<D>(smem + TILE, kb, vb, kv_ss, lt * kKT + kKT, lend, w, lane, ldo);
    lt += 2;

    // Operand addresses: a lane's are the same in every tile up to the tile's place in LDS, so they are
    // kept in registers (eight for K: the XOR swizzle is not additive in the chunk; four for V) and the
    // sub-tile, the step inside the tile and the second tile of a pair are instruction offsets; only the
    // pair's own 64 KB step is added, once per pair.  (Recomputed per tile, as the compiler does when
    // handed a tile pointer, they were a quarter of the loop's vector instructions.)
    const lds_byte *ka[D / 16], *va[DB];
    {
        const lds_byte *base = (const lds_byte *)smem;
#pragma unroll
        for (int st = 0; st < D / 16; ++st) ka[st] = base + ks_off<D>(j32, 2 * st + g2);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int d0 = 32 * db + (j32 & 16) + 4 * (lane & 3), kv0 = 4 * g2 + ((lane >> 2) & 3);
            va[db] = base + TILE / 2 + vs_off<D>(kv0, d0 >> 3) + (d0 & 7) * 2;
        }
    }
    int half = 0;                                         // the current pair sits in buffers 2*half, 2*half + 1

    for (;;) {
        // which unit this wavefront is: (head within the group, block of 32 rows), and which keys of the piece
        const int nqb = FLAT ? flat_row_blocks(a, pc.nn) : a.nqb, units = a.G * nqb;
        int u = ublk * kGsWaves + w;
        const int entry = (pc.slot * a.n_ublk + ublk) * kGsWaves + w;
        bool active = u < units;
        if (FLAT && flat_shared(a, pc.nn)) {
            active = u < 2 * units;
            if (u >= units) u -= units;
        }
        const int g = u / nqb, qb = u % nqb;
        const int h = pc.hk * a.G + (active ? g : 0);
        const int i = 32 * qb + j32;                      // this lane's tree row
        const int L = pc.L, nn = pc.nn, kend = pc.kend;

        const int parent = a.parents[(size_t)pc.b * a.T + min(lane, max(nn, 1) - 1)];
        bf16x8 qop[D / 16];                               // row i, d = 16*st + 8*g2 .. +8, for the whole piece
        {
            const __bf16 *qrow = a.q + (size_t)pc.b * a.q_sb + (size_t)h * a.q_sh + (uint32_t)(min(i, a.T - 1) * (int)a.q_st);
#pragma unroll
            for (int st = 0; st < D / 16; ++st) {
                u32x4 raw = *reinterpret_cast<const u32x4 *>(qrow + 16 * st + 8 * g2);
                and_mask(raw, active && i < a.T);
                qop[st] = __builtin_bit_cast(bf16x8, raw);
            }
        }
        Piece nx;
        bool more = false;
        if constexpr (FLAT) {
            more = next_piece(nx);
            if (more) own_half(nx);
        }
        // the next piece's query rows and parents: brought close by, not kept (a row is two cache lines)
        uint32_t touched = 0;
        if (FLAT && more) {
            const int nq = flat_row_blocks(a, nx.nn);
            int v = ublk * kGsWaves + w;
            if (v >= a.G * nq) v -= a.G * nq;
            const int row = min(32 * (v % nq) + j32, a.T - 1), hd = nx.hk * a.G + min(v / nq, a.G - 1);
            touched = *reinterpret_cast<const uint32_t *>(a.q + (size_t)nx.b * a.q_sb + (size_t)hd * a.q_sh +
                                                          (uint32_t)(row * (int)a.q_st + (D / 2) * g2));
            touched ^= (uint32_t)a.parents[(size_t)nx.b * a.T + min(lane, a.T - 1)];
        }
        uint64_t anc[1];
        anc[0] = kend > L ? ancestor_word_of(ancestor_words(parent, nn), i, nn) : 0ull;

        floatx16 oacc[DB][1];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][0][r] = 0.f;
        float m_run[1] = {kNegBig}, l_run[1] = {0.f};

        // Tiles are taken in pairs, four buffers: while the pair (t, t+1) is consumed from two of them the
        // loads of the next pair (the next piece's first, at the end of one) arrive in the other two.
        // One barrier per pair: it publishes the pair (every wavefront has waited for its own loads) and
        // tells that nobody reads the previous pair any more, whose buffers the loads issued right after
        // it overwrite.  (Not __syncthreads(): nothing here needs its fence.)
        // The two wavefronts of a SIMD (w and w + 4) are favoured in turn, one in the first tile of a pair
        // and the other in the second.  Left alone, the older wavefront wins the arbitration in every
        // tile and finishes it a third ahead of the other; taking turns measured 3-4 % faster at 16 K
        // cached rows.  (A barrier per pair without the priorities is slower than one per tile, and
        // priorities with a barrier per tile change nothing.)
        floatx16 sacc[2];
        bf16x8 pk[2][2];
        auto run_tile = [&](auto second, int t0) {
            constexpr int TOFF = decltype(second)::value ? TILE : 0;
            // sub-tile k % 2: 32 rows on, the same swizzle (32 is a multiple of 16)
            tile_scores<D, 2>([&](int k) { return (lds_u32x4)(ka[k >> 1] + TOFF + (k & 1) * (32 * D * 2)); }, qop, sacc);
            tile_softmax<D, 2>(sacc, oacc, m_run[0], l_run[0], anc[0], t0, L, kend, false, a.scale_log2, kMaxSlack, pk);   // (zeros rescaled once: no second copy of the loop for the first pair)
            // step k: output block k % DB, rows 16 * (k / DB) on (a multiple of 4: the same swizzle), hi: 8 rows on
            tile_pv<D, 2, true>([&](int k, int hi) { return va[k % DB] + TOFF + (k / DB) * (16 * D * 2) + hi * (8 * D * 2); }, pk, oacc);
        };
        const int fav = w < kGsWaves / 2 ? 1 : 0;
        for (int t = pc.t0; t < pc.t1; t += 2) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (FLAT && lt >= lt1 && more) load_from(nx);            // (past the last piece: its last rows once more)
            ld_issue_tile<D>(smem + (2 - 2 * half) * TILE, kb, vb, kv_ss, lt * kKT, lend, w, lane, ldo);
            ld_issue_tile<D>(smem + (3 - 2 * half) * TILE, kb, vb, kv_ss, lt * kKT + kKT, lend, w, lane, ldo);
            lt += 2;
            if (active) {
                if (fav) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0);
                run_tile(std::false_type{}, t * kKT);
                if (fav) __builtin_amdgcn_s_setprio(0); else __builtin_amdgcn_s_setprio(1);
                if (t + 1 < pc.t1) run_tile(std::true_type{}, (t + 1) * kKT);
            }
            const int step = half ? -2 * TILE : 2 * TILE;            // the next pair sits in the other two buffers
#pragma unroll
            for (int st = 0; st < D / 16; ++st) ka[st] += step;
#pragma unroll
            for (int db = 0; db < DB; ++db) va[db] += step;
            half ^= 1;
        }
        asm volatile("" :: "v"(touched));
        __builtin_amdgcn_s_setprio(0);
        if (!more) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may still be on its way into LDS at the end
        if (active) gs_finish<D>(a, [&](int db, int r) { return oacc[db][0][r]; }, m_run[0], l_run[0], pc.b, h, i, nn, pc.direct, entry);
        if (!more) return;
        pc = nx;
    }
}

// ===================================================================== one launch, short contexts
// A call over a few hundred rows is two launches of about four dependent round trips each; what it computes would take
// a microsecond.  Here a workgroup takes one unit (query head, block of 32 tree rows) over all rows, its eight
// wavefronts 32 rows each in turn, and merges their results in LDS: one launch, no partials in memory.  A
// wavefront stages its own rows straight into its own part of LDS and waits for nobody until the merge.  The
// price is that every unit's CU reads all of its KV head's rows: what bounds it is that CU's port, about 1 us per
// 64 KB, after 5 us of launch and round trips (32 heads, D = 128: 260 rows 8.3 us, 540 rows 9.9; with ranges
// and a merge 10.7 and 11.2.  One layer of 4 heads with D = 64 over 272 rows 6.0 instead of 7.8).
constexpr int kOneRows = 32;                             // cache rows of a wavefront's step
constexpr int kInvShift = 20;                            // a KV head's number times its sequence's share of 2^20

struct OneKernArgs { const __bf16 *k, *v; const int32_t *ctx_lens, *n_nodes; int64_t kv_sb, kv_sh; int first; uint32_t second; AttnArgs a; };
// first, second: what is needed first; EIGHTS: the KV heads and their share of 2^20, else the rows of the cache and their stride
template <int D, bool EIGHTS>
__global__ __launch_bounds__(kGsThreads) void tree_attn_one_kernel(const __bf16 *k_, const __bf16 *v_, const int32_t *ctx_lens, const int32_t *n_nodes,
                                                                  int64_t kv_sb, int64_t kv_sh, int first, uint32_t second, AttnArgs) {
    constexpr int DB = D / 32, ROW = D * 2, SUB = kOneRows * ROW;           // bytes of a row, of a step's K or V rows
    constexpr int LOADS = SUB / 1024, RPL = 1024 / ROW, CPR = ROW / 16;     // 1 KB loads; rows of one; 16-byte chunks of a row
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float *const s_m = reinterpret_cast<float *>(smem + kGsWaves * 2 * SUB), *const s_l = s_m + kGsWaves * 32;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int j32 = lane & 31, g2 = lane >> 5;
    // Which workgroups share a KV head's rows, and whether they share an XCD: plan_attention.
    int b = blockIdx.z, hk = blockIdx.x;
    if (EIGHTS) {
        const int number = 8 * b + hk;                   // the batch's KV heads, counted through
        b = (int)((uint32_t)number * second >> kInvShift);
        hk = number - b * first;
    }
    const ArgBlock<AttnArgs> early = args_from_here<AttnArgs>(offsetof(OneKernArgs, a));
    if (EIGHTS && b >= early->B) return;
    const int S = EIGHTS ? early->S : first;
    const int kv_ss = EIGHTS ? (int)early->kv_ss : (int)second;        // 32-bit offsets inside one head's cache (checked on the host)
    const int32_t ctx = uniform_word(ctx_lens, b), nodes = n_nodes ? uniform_word(n_nodes, b) : RADAR_T_MAX;
    const __bf16 *const kbase = k_ + (size_t)b * kv_sb + (size_t)hk * kv_sh;
    const __bf16 *const vbase = v_ + (size_t)b * kv_sb + (size_t)hk * kv_sh;

    // This wavefront's rows of a step: K [32][D], then V [32][D], both row-major with their own swizzle (ks_off, vs_off); a
    // lane's 16 bytes land at the load's LDS base + 16 * lane, so it fetches the chunk that belongs there.  Rows past
    // the end re-read the last one in K, whose scores are masked, and are zeros in V.
    unsigned char *const mine = smem + w * 2 * SUB;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)mine);
    // Whole steps: a scalar base per load and the lane's offset in it, which repeats after 16 rows of K and is one for all of V.
    const int lrow = lane / CPR, slot = lane % CPR;
    uint32_t offk[16 / RPL], offv = (uint32_t)(lrow * kv_ss) * 2 + (uint32_t)((slot ^ vs_swz<D>(lrow)) << 4);
#pragma unroll
    for (int i = 0; i < 16 / RPL; ++i) offk[i] = (uint32_t)(lrow * kv_ss) * 2 + (uint32_t)((slot ^ ks_swz<D>(RPL * i + lrow)) << 4);
    auto issue = [&](const __bf16 *base, auto is_v, int sub, int total) {
        constexpr bool V = decltype(is_v)::value;
        const int row0 = __builtin_amdgcn_readfirstlane(sub * kOneRows);
        if (row0 + kOneRows <= total) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const __bf16 *const src = base + (uint32_t)((row0 + RPL * i) * kv_ss);
                const uint32_t dst = lds0 + (V ? SUB : 0) + i * 1024;
                load_to_lds(dst, src, V ? offv : offk[i % (16 / RPL)]);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int row = RPL * i + lrow, at = row0 + row;
            const int chunk = V ? slot ^ vs_swz<D>(row) : slot ^ ks_swz<D>(row);
            const __bf16 *src = base + (uint32_t)(min(at, total - 1) * kv_ss) + chunk * 8;
            if (V) src = at < total ? src : (const __bf16 *)kZeroChunk;
            const uint32_t dst = lds0 + (V ? SUB : 0) + i * 1024;
            load_to_lds(dst, src);
        }
    };
    constexpr std::false_type kK{};
    constexpr std::true_type kV{};
    // The first rows of K are asked for before the sequence's lengths are there: rows past its end, of the cache that the caller described, are
    // masked by the softmax.  (V's have to be zeros, which takes the lengths.)
    if (w * kOneRows < S) issue(kbase, kK, w, S);
    AttnArgs a;
    {
        const ArgBlock<AttnArgs> p = args_from_here<AttnArgs>(offsetof(OneKernArgs, a));
        a.T = p->T; a.G = p->G; a.Hq = p->Hq; a.nqb = p->nqb; a.q = p->q; a.q_sb = p->q_sb; a.q_st = p->q_st; a.q_sh = p->q_sh; a.parents = p->parents;
        a.scale_log2 = p->scale_log2; a.out = p->out; a.lse = p->lse; a.o_sb = p->o_sb; a.o_st = p->o_st; a.o_sh = p->o_sh;
    }
    const int unit = blockIdx.y, qb = unit & (a.nqb - 1), h = hk * a.G + (unit >> (a.nqb - 1));
    const int L = min(ctx, S);                           // (prefix_rows)
    const int nn = max(1, min(nodes, a.T));
    const int total = min(L + nn, S);                    // never read past the cache the caller described
    if (L < 0 || total < 1) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); return; }     // (nothing may still be on its way into LDS at the end)
    const int nsub = (total + kOneRows - 1) / kOneRows, nact = min(nsub, kGsWaves);
    const int i = 32 * qb + j32;                         // this lane's tree row
    bf16x8 qop[D / 16];                                  // its query operands: d = 16*st + 8*g2 .. +8
    floatx16 oacc[DB][1];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][0][r] = 0.f;
    float m_run = kNegBig, l_run = 0.f;
    if (w < nact) {
        issue(vbase, kV, w, total);
        const __bf16 *qrow = a.q + (size_t)b * a.q_sb + (size_t)h * a.q_sh + (uint32_t)(min(i, a.T - 1) * (int)a.q_st);
#pragma unroll
        for (int st = 0; st < D / 16; ++st) {
            u32x4 raw = *reinterpret_cast<const u32x4 *>(qrow + 16 * st + 8 * g2);
            and_mask(raw, i < a.T);
            qop[st] = __builtin_bit_cast(bf16x8, raw);
        }
        uint64_t anc = 0;
        // (only wavefronts that meet rows of the tree need the ancestors: the last steps')
        const int last = w + (nsub - 1 - w) / kGsWaves * kGsWaves;
        if (last * kOneRows + kOneRows > L)
            anc = ancestor_word_of(ancestor_words(a.parents[(size_t)b * a.T + min(lane, nn - 1)], nn), i, nn);
        const lds_byte *const kl = (const lds_byte *)mine, *const vl = kl + SUB;
#pragma unroll
        for (int st = 0; st < D / 16; ++st) asm volatile("" : "+v"(qop[st]));       // (they have landed, and with them the first K and V: no waits for them in the loop)
        for (int sub = w; sub < nsub; sub += kGsWaves) {
            const bool more = sub + kGsWaves < nsub;
            floatx16 sacc[1];
            bf16x8 pk[1][2];
            // K has landed when no more than V's loads are under way, which are issued after it and land in order; V when K's next ones are left.
            if (sub == w) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" : : "n"(LOADS) : "memory");
            tile_scores<D, 1>([&](int k) { return (lds_u32x4)(kl + ks_off<D>(j32, 2 * k + g2)); }, qop, sacc);
            if (more) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // the K rows have been read: the next may land there
                issue(kbase, kK, sub + kGsWaves, total);
            }
            tile_softmax<D, 1>(sacc, oacc, m_run, l_run, anc, sub * kOneRows, L, total, sub == w, a.scale_log2, 0.f, pk);
            if (more) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(LOADS) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            tile_pv<D, 1, true>([&](int k, int hi) {
                const int d0 = 32 * (k % DB) + (j32 & 16) + 4 * (lane & 3), kv0 = 4 * g2 + ((lane >> 2) & 3);
                return vl + vs_off<D>(kv0, d0 >> 3) + (d0 & 7) * 2 + (k / DB) * (16 * ROW) + hi * (8 * ROW);   // (8 rows on: the same swizzle)
            }, pk, oacc);
            if (more) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                issue(vbase, kV, sub + kGsWaves, total);
            }
        }
        const float l_tot = l_run + __shfl_xor(l_run, 32);
        if (g2 == 0) { s_m[w * 32 + j32] = m_run; s_l[w * 32 + j32] = l_tot; }
    }
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // (rows asked for in vain have landed, too)
    __syncthreads();                                     // every wavefront is done with its rows; maxima and sums are in LDS
    float *const s_o = reinterpret_cast<float *>(smem);  // [wavefront][d][32], over the rows
    if (w < nact) {
        float M = kNegBig;
        for (int v = 0; v < nact; ++v) M = fmaxf(M, s_m[v * 32 + j32]);
        const float scl = __builtin_amdgcn_exp2f(m_run - M);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) s_o[(w * D + 32 * db + 8 * (r >> 2) + 4 * g2 + (r & 3)) * 32 + j32] = oacc[db][0][r] * scl;
    }
    __syncthreads();
    const int row = tid & 31, d8 = tid >> 5, ti = 32 * qb + row;            // eight outputs of one row
    if (d8 * 8 >= D || ti >= a.T) return;
    const bool live = ti < nn;
    float M = kNegBig, l = 0.f, acc[8];
    for (int v = 0; v < nact; ++v) M = fmaxf(M, s_m[v * 32 + row]);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    for (int v = 0; v < nact; ++v) {
        l += s_l[v * 32 + row] * __builtin_amdgcn_exp2f(s_m[v * 32 + row] - M);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += s_o[(v * D + d8 * 8 + e) * 32 + row];
    }
    const float inv = (live && l > 0.f) ? 1.0f / l : 0.f;
    bf16x8 o8;
#pragma unroll
    for (int e = 0; e < 8; ++e) o8[e] = (__bf16)(live ? acc[e] * inv : 0.f);             // rows past the tree are zeroed
    *reinterpret_cast<bf16x8 *>(a.out + (size_t)b * a.o_sb + (size_t)ti * a.o_st + (size_t)h * a.o_sh + d8 * 8) = o8;
    if (a.lse && d8 == 0) a.lse[((size_t)b * a.T + ti) * a.Hq + h] = live ? (M + __builtin_amdgcn_logf(l)) * kLn2 : 0.f;
}

// Merges the group-share kernels' partials.  A workgroup takes one (sequence, query head, 32-wide slice
// of the head dimension): lane = (8 consecutive d, tree row i), rows rounded up to 16, 32 or 64, so that a
// small tree's rows sit in few wavefronts (four rows, 48 partials: 31 us for the call with 64 lanes per
// d, 22 with 16).  The time is that of dependent rounds of loads, so a lane asks for NB partials at once, or for
// as many as there are, two or in steps of four (12 sequences of 64 heads, a head's rows in one or two pieces: 55.0 us for the call with four,
// 54.3 with two; 17 of them in rounds of 8, 8 and 1, which the compiler made five rounds to save
// registers: 16.0 us for a call over 2048 rows, 15.0 in one), and weighs them by their common maximum.  Where the rows
// are dealt out on the device into sixteen shares or more per KV head, two groups
// of lanes take every other partial and meet in LDS (3 heads of 16000 rows 26.5 -> 24.8 us; with 11 pieces it costs
// 0.1 us more than it gives, and four groups cost more than two nearly everywhere: a workgroup of 1024 lanes starts
// late).  Ranges cut on the host are merged by one group, however many they are.
// CUT: ranges cut on the host.  The lengths come first (before them, as many partials as the grid had ranges would be 0.2 us slower where
// there are that many, and 1.1 to 1.5 where the sequence is short); the arguments that only the end needs are read there.
// heads: KV heads in the lower half, query heads of each in the upper; blocks: n_ublk and nqb likewise.  Not CUT: kps is unit_tab's offset from part_ml.
struct MergeKernArgs { const uint64_t *part_o; const float *part_ml; const int32_t *ctx_lens, *n_nodes; int T, kps, S, max_splits; uint32_t heads; int blocks; AttnArgs a; };
constexpr int kMergeSlice = 32;                          // of the head's D
template <int D, int E, int NB, bool CUT>
__global__ __launch_bounds__(kAttnThreads * E) void tree_attn_merge_kernel(const uint64_t *part_o, const float *part_ml, const int32_t *ctx_lens, const int32_t *n_nodes,
                                                                          int T, int kps, int S, int max_splits, uint32_t heads, int blocks, AttnArgs) {
    constexpr int DQ = 8, SL = kMergeSlice, SLICES = D / SL, kGroup = kAttnThreads;        // floats per lane; lanes of a group
    static_assert(kGroup == RADAR_T_MAX * (SL / DQ), "a lane for each row and eight of a slice");
    __shared__ float red[E > 1 ? E - 1 : 1][10][kGroup];
    const int slice = blockIdx.x % SLICES, g = blockIdx.x / SLICES, hk = blockIdx.y, b = blockIdx.z;
    const int G = heads >> 16, Hkv = heads & 0xffff, h = hk * G + g, n_ublk = blocks & 0xffff;
    int slot0 = (b * Hkv + hk) * max_splits, count = max_splits, nqb = blocks >> 16, shared = 0;   // partials of this head's KV head: consecutive slots, each once or twice
    int nn = T;
    {
        const int L = min(uniform_word(ctx_lens, b), S);    // (prefix_rows)
        if (n_nodes) nn = uniform_word(n_nodes, b);
        nn = max(1, min(nn, T));
        if (L < 0) return;
        if constexpr (CUT) {
            count = (min(L + nn, S) + kps - 1) / kps;
            if (count <= 1) return;                         // the workgroup wrote the result itself
        } else {
            AttnArgs f;                                     // what flat_row_blocks and flat_shared ask for
            f.G = G; f.nqb = nqb; f.n_ublk = n_ublk;
            const int32_t *const tab = reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(part_ml) + kps);   // (unit_tab)
            slot0 = uniform_word(tab, 2 * (b * Hkv + hk));
            count = uniform_word(tab, 2 * (b * Hkv + hk) + 1);
            if (count == 0) return;
            nqb = flat_row_blocks(f, nn);
            shared = flat_shared(f, nn) ? 1 : 0;
            count <<= shared;
        }
    }

    const int tg = threadIdx.x & (kGroup - 1), eg = E > 1 ? (int)threadIdx.x / kGroup : 0;
    const int rbits = T > 32 ? 6 : T > 16 ? 5 : 4;
    const int i = tg & ((1 << rbits) - 1), part = tg >> rbits;          // query row, which 8 of the slice
    if (E == 1 && part >= SL / DQ) return;
    const bool live = i < nn && part < SL / DQ;
    const int d0 = slice * SL + part * DQ;
    const int units = G * nqb, j32 = i & 31;
    // an entry's address: a uniform part, kept in scalar registers, and the lane's offset in the entries of its block
    const int entry0 = slot0 * n_ublk * kGsWaves + g * nqb;
    const uint32_t block = nqb == 1 ? 0 : i >> 5;
    const uint32_t lane_ml = block * 96 + j32 * 3, lane_o = block * (D / 4 * 32) + ((d0 >> 3) * 32 + j32) * 2;
    auto entry_of = [&](int n) { return (size_t)__builtin_amdgcn_readfirstlane(entry0 + (n >> shared) * n_ublk * kGsWaves + ((n & shared) ? units : 0)); };
    float M = kNegBig, lsum = 0.f;
    float acc[DQ];
#pragma unroll
    for (int d = 0; d < DQ; ++d) acc[d] = 0.f;
    auto take = [&](auto batch, int s0) __attribute__((always_inline)) {   // so many partials at a time, their loads in flight together
        constexpr int N = decltype(batch)::value;
        float m[N], l[N], mag[N];
        u32x4 o[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const size_t en = entry_of(min(s0 + j * E, count - 1));
            const float3u ml = *reinterpret_cast<const float3u *>(part_ml + en * 96 + lane_ml);
            m[j] = ml[0]; l[j] = ml[1]; mag[j] = ml[2];
            o[j] = *reinterpret_cast<const u32x4 *>(part_o + en * (size_t)(D / 4 * 32) + lane_o);
        }
        if constexpr (NB > 8) __builtin_amdgcn_sched_barrier(0);    // (else loads follow the arithmetic, to save registers)
        float Mn = M;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if (s0 + j * E >= count) m[j] = kNegBig;
            Mn = fmaxf(Mn, m[j]);
        }
        const float aold = __builtin_amdgcn_exp2f(M - Mn);
        M = Mn;
        lsum *= aold;
#pragma unroll
        for (int d = 0; d < DQ; ++d) acc[d] *= aold;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float wl = s0 + j * E < count ? __builtin_amdgcn_exp2f(m[j] - Mn) * l[j] : 0.f;
            lsum += wl;
            const float wo = wl * mag[j];                     // the stored rows are o / (l x magnitude)
#pragma unroll
            for (int d = 0; d < DQ / 2; ++d) {
                acc[2 * d] = fmaf(wo, (float)__builtin_bit_cast(_Float16, (uint16_t)(o[j][d] & 0xffffu)), acc[2 * d]);
                acc[2 * d + 1] = fmaf(wo, (float)__builtin_bit_cast(_Float16, (uint16_t)(o[j][d] >> 16)), acc[2 * d + 1]);
            }
        }
    };
    auto take_all = [&](auto batch) __attribute__((always_inline)) {
        constexpr int N = decltype(batch)::value;
        for (int s0 = eg; s0 < count; s0 += N * E) take(batch, s0);
    };
    if (live) {
        const int each = (count + E - 1) / E;
        if (each <= 2) take_all(std::integral_constant<int, 2>{});
        else if (NB == 4 || each <= 4) take_all(std::integral_constant<int, 4>{});
        else if (NB == 8 || each <= 8) take_all(std::integral_constant<int, 8>{});
        else if (each <= 12 || (each > NB && each <= 24)) take_all(std::integral_constant<int, 12>{});      // (two rounds: even ones)
        else if (each <= 16 || (each > NB && each <= 32)) take_all(std::integral_constant<int, 16>{});
        else take_all(std::integral_constant<int, NB>{});
        // What is asked for beyond the last partial is that one again, with no weight.  Where it holds an infinity 0 * Inf has made the
        // row NaN: its partials are added up again one by one.  (The check is 0.06 us of a call over 2048 rows, 13.40 -> 13.46; masking them 0.3.)
        float any = acc[0] + acc[1];
#pragma unroll
        for (int d = 2; d < DQ; ++d) any += acc[d];
        if (__builtin_expect(__any(any != any), 0)) {
            M = kNegBig;
            lsum = 0.f;
#pragma unroll
            for (int d = 0; d < DQ; ++d) acc[d] = 0.f;
            take_all(std::integral_constant<int, 1>{});
        }
    }
    if constexpr (E > 1) {
        if (live && eg > 0) {
            red[eg - 1][0][tg] = M;
            red[eg - 1][1][tg] = lsum;
#pragma unroll
            for (int d = 0; d < DQ; ++d) red[eg - 1][2 + d][tg] = acc[d];
        }
        __syncthreads();
        if (eg > 0) return;
        if (live) {
#pragma unroll
            for (int e = 0; e < E - 1; ++e) {
                const float m = red[e][0][tg], Mn = fmaxf(M, m);
                const float aold = __builtin_amdgcn_exp2f(M - Mn), wnew = __builtin_amdgcn_exp2f(m - Mn);
                lsum = lsum * aold + red[e][1][tg] * wnew;
#pragma unroll
                for (int d = 0; d < DQ; ++d) acc[d] = acc[d] * aold + red[e][2 + d][tg] * wnew;
                M = Mn;
            }
        }
    }
    if (i >= T || part >= SL / DQ) return;
    const ArgBlock<AttnArgs> a = args_from_here<AttnArgs>(offsetof(MergeKernArgs, a));
    __bf16 *const orow = a->out + (size_t)b * a->o_sb + (size_t)i * a->o_st + (size_t)h * a->o_sh + d0;
    float *const lse = a->lse;
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    bf16x8 o8;
#pragma unroll
    for (int e = 0; e < 8; ++e) o8[e] = (__bf16)(live ? acc[e] * inv : 0.f);      // rows past the tree are zeroed
    *reinterpret_cast<bf16x8 *>(orow) = o8;
    if (lse && slice == 0 && part == 0) lse[((size_t)b * T + i) * (Hkv * G) + h] = live ? (M + __builtin_amdgcn_logf(lsum)) * kLn2 : 0.f;
}

// ------------------------------------------------------------------ host-side planning
struct AttnPlan {
    int kps, max_splits, n_ublk, nqb, shares;
    bool one, by_eights;                                   // one launch, no ranges; its KV heads taken eight at a time
    size_t off_part_o, off_part_ml, off_tab, bytes;
};

static int unit_blocks(const radar_attn_desc *d, int nqb) { return (d->Hq / d->Hkv * nqb + kGsWaves - 1) / kGsWaves; }

// Number of key ranges: the one that minimises a small cost model, in units of one tile of
// one workgroup (1.45 us): rounds of 256 resident workgroups x (tiles per range +
// 3 for prologue and epilogue), plus what the merge of the ranges costs: the launch, and every
// range's partials written and read again.  Counting whole rounds matters: 576 workgroups take
// as long as 768.  What a range costs grows with the bytes of its partials (with 0.08 for any, 1300 rows of 32 heads were cut
// into 22 ranges of one tile, 15.4 us; 11 of two take 13.7).  Over 753 calls of 900 ... 6500 rows, each timed with one to
// eight tiles per range, this choice is 1.1 % slower than the best one in the geometric mean; 0.08 for any is 1.7 %.
static long range_count(const radar_attn_desc *d, int nqb) {
    const double per_range = std::max(0.078, 0.045 + 4e-7 * (double)d->B * d->Hq * d->T_max * d->D);
    const long units = (long)d->B * d->Hkv * unit_blocks(d, nqb);
    const long tiles_all = ((long)d->S_max + kKT - 1) / kKT;
    double best = 1e30;
    long best_ns = 1;
    for (long ns = 1; ns <= 64 && ns <= tiles_all; ++ns) {
        const long tiles = (tiles_all + ns - 1) / ns;
        const long rounds = (units * ns + 255) / 256;
        const double cost = (double)rounds * (double)(tiles + 3) + (ns > 1 ? 1.2 + per_range * (double)ns : 0.0);
        if (cost < best) { best = cost; best_ns = ns; }
    }
    return best_ns;
}

// Up to how many cache rows a call is one launch of whole units (tree_attn_one_kernel): as long as the units are no more than the chip holds at once
// (one per CU with D = 128, two with D = 64), to where a unit's CU takes as long to read all rows as ranges and their merge take.  That is later the
// more units there are, because ranges then wait for each other, and earlier where a KV head has at most four: half of a range's wavefronts are idle
// then, and it takes a tile the faster.
// Both sides measured for 633 combinations of batch, heads and tree at ten contexts of 150 ... 1850 rows; one launch / ranges in us, at D = 128, 60
// tree rows: 32 heads 8.3 / 10.7 over 260 rows, 9.9 / 11.2 over 540, 11.6 / 12.1 over 820, 13.1 / 13.1 over 1050; 64 heads 10.3 / 13.6 over 620, 13.1
// / 15.2 over 1050, 14.8 / 16.2 over 1360, 17.5 / 17.4 over 1560; four sequences of 32 heads 10.6 / 15.2 over 540, 17.5 / 19.5 over 1560; 16 heads on
// 8 KV heads 8.6 / 9.3 over 360, 9.8 / 9.9 over 540; 16 tree rows, 32 heads 8.0 / 8.6 over 316, 9.2 / 8.6 over 496, three sequences 9.6 / 10.3 over
// 626.
// D = 64, 8 heads on 4: 8.1 / 8.6 over 820, 9.1 / 8.5 over 960; 16 on 4 over 1000 rows, 60 tree rows, one / four / eight sequences 9.4 / 9.8, 9.8 /
// 11.0, 10.2 / 15.3; eight of 16 heads 8.6 / 11.8 over 820, 11.7 / 18.3 over 1560.
// Two units of at most 32 tree rows per CU (D = 64, more than 256) take longer over a row: 16 tree rows, 32 sequences of 16 heads on 2 10.3 / 11.1
// over 640, 13.0 / 12.8 over 900; 64 of 8 on 8 22.3 / 35.1 over 900, 33.0 / 52.2 over 1600; 32 of 12 on 3 13.7 / 15.6 over 1100, 17.7 / 18.5 over
// 1600.
// Over all of these the better side is missed by 0.8 % in the geometric mean, as by a line between the two sides' estimated times.  Trees just past
// 32 rows in ragged batches would have it earlier (33 tree rows, three sequences of 32 heads, the longest 1533 16.8 / 14.7), in even ones not (four
// of 32 heads over 1400 15.6 / 16.9, eight of 8 on 8 with D = 64 over 1600 11.2 / 13.4), and the host does not know which they are.
//
// Where there are many KV heads one launch is the better side for longer.  What it takes is the longest sequence's rows, whatever
// the others have; ranges go by the largest share of a range, or (dealt out, D = 128) by all rows.  So the lines lie where no batch loses, a
// single long sequence among short ones included.  One launch / ranges over 10800 calls: even batches, lengths spread from an eighth up,
// every second or only one sequence long and the others a 16th or a 500th.
//   D = 128, worst batch: 68 ... 192 KV heads 0.74 ... 1.01 up to 1900 rows, 0.99 ... 1.07 over 2000; more of them 0.97 over 1300, 1.08 over
//   1900 (256, one query head each, stay dealt out); 64 to 67 from 1.08 over 1200 to 0.92 over 1300, level on average.  Groups of five and
//   more in 192 units: 40 and more KV heads 0.90 ... 1.01 up to 1400 rows, 24 ... 36 1.07 ... 1.13 over 1200.
//   D = 64: a workgroup of a range takes four times as long over a row, so with 60 KV heads and more one long sequence loses only where the
//   ranges are more than four: five 1.03 over 3015 rows, 1.39 over 12000, seven 1.21 over 10600; up to 2660 rows 0.92. Up to four ranges
//   0.63 ... 0.94 up to 12000 rows (1.14 over 16640); with more units than CUs, of 96 and more KV heads, 0.67 ... 0.91 up to 8000, 1.2 over 12000;
//   256 and more 0.58 ... 0.84 at any length.  48 KV heads 0.86 ... 1.01 up to 2660 rows, 1.08 over 4000; 32 with 224 units and more 0.80 ... 0.97 over
//   1900, 1.04 over 2300.
// (*ranges: the number of ranges, where the line goes by it.)
static int one_launch_rows(const radar_attn_desc *d, int nqb, long *ranges) {
    const long units = (long)d->B * d->Hq * nqb, kv_heads = (long)d->B * d->Hkv;
    const int G = d->Hq / d->Hkv;
    if (d->D == 64) {
        if (units > 512) return 0;
        if (kv_heads >= (units <= 256 ? 60 : 96)) {
            if (d->S_max > 2660) *ranges = range_count(d, nqb);
            return *ranges > 4 ? 2660 : kv_heads >= 256 ? INT32_MAX : units <= 256 ? 12000 : 8000;
        }
        if (units <= 256 && kv_heads >= 48) return 2660;
        if (units <= 256 && units >= 224 && kv_heads >= 32) return 1900;
        if (units > 256 && nqb == 1) return G <= 4 ? 1600 : 832;
        if (units >= 128) return nqb == 1 && G >= 4 && units < 192 ? 1300 : 1600;
        return G * nqb <= 4 || nqb == 1 ? 832 : 1024;
    }
    if (units > 256) return 0;
    if (kv_heads >= 68 && kv_heads < 256) return kv_heads <= 192 ? 1850 : 1300;
    if (units >= 192 && kv_heads >= 40 && nqb == 1 && G > 4) return 1400;
    if (G * nqb <= 4) return units >= 96 ? 800 : units >= 64 && nqb == 2 ? 700 : 384;
    if (nqb == 2 && units >= 64) return units >= 192 ? 1600 : units >= 128 ? 1400 : 900;
    return units >= 192 ? 1100 : units >= 96 ? 800 : 640;
}

// The units of a KV head read the same rows.  Workgroups go to the eight XCDs in turn, and where grid x is the KV head and Hkv a
// multiple of eight, a head's are all on one, whose L2 then holds the rows for them (32 heads x 3 sequences over 572 rows
// 13.9 -> 10.7 us).  With another Hkv they are on two, four or eight XCDs, each of which fetches the rows: that
// is as good while the L2s (32 MB together) hold all of it.  From 28 MB on the batch's KV heads are taken eight at a
// time instead, if every XCD gets as few units as its CUs can take (one each, or two with D = 64 if there are more units than CUs);
// elsewhere the call goes in ranges from 42 MB on.  Over 900 rows, us, grid x the KV head / by eights (finding the head costs 0.15): D = 64, 60
// tree rows, 8 sequences of 8 heads on 4 (15 MB) 9.3 / 9.5, 16 (29 MB) 9.9 / 9.8, 32 (59 MB) 16.0 / 14.2, 32 of 4 on one (59 MB)
// 13.8 / 9.8, 64 (118 MB) 22.0 / 13.5 (in ranges 16.1); D = 128, 16 tree rows, 32 of 8 on one (118 MB) 22.6 / 13.0 (14.8).  More units than
// CUs on an XCD, 16 tree rows: D = 64, 18 of 14 heads on 2 (33 MB) 9.7 / 12.0 (11.3), D = 128 over 900 rows (66 MB) 16.2 and 15.0 in
// ranges, 36 of 7 on one (116 MB) 22.9 and 17.3.
static bool one_launch_by_eights_fits(const radar_attn_desc *d, int nqb) {
    const int64_t heads = (int64_t)d->B * d->Hkv, units = (int64_t)(d->Hq / d->Hkv) * nqb;
    return (heads + 7) / 8 * units <= (d->D == 64 && heads * units > 256 ? 64 : 32);
}
static int64_t one_launch_fetches(const radar_attn_desc *d, int nqb) {          // megabytes, with grid x the KV head
    const int64_t xcds = d->Hkv % 8 == 0 ? 1 : d->Hkv % 4 == 0 ? 2 : d->Hkv % 2 == 0 ? 4 : 8, units = (int64_t)(d->Hq / d->Hkv) * nqb;
    return (int64_t)d->B * d->Hkv * d->S_max * d->D * 4 * std::min(xcds, units) / 1000000;
}

static AttnPlan plan_attention(const radar_attn_desc *d) {
    AttnPlan p;
    p.nqb = d->T_max <= 32 ? 1 : 2;
    p.n_ublk = unit_blocks(d, p.nqb);
    long kps = d->keys_per_split;
    long ranges = 0;
    p.one = kps <= 0 && d->S_max <= one_launch_rows(d, p.nqb, &ranges);
    p.by_eights = p.one && d->Hkv % 8 != 0 && one_launch_fetches(d, p.nqb) >= 28;
    if (p.by_eights && !one_launch_by_eights_fits(d, p.nqb)) {
        p.by_eights = false;
        p.one = one_launch_fetches(d, p.nqb) < 42;
    }
    if (p.one) kps = ((long)d->S_max + kKT - 1) / kKT * kKT;
    if (kps <= 0) {
        if (ranges == 0) ranges = range_count(d, p.nqb);
        const long tiles_all = ((long)d->S_max + kKT - 1) / kKT;
        kps = (tiles_all + ranges - 1) / ranges * kKT;
    }
    p.kps = (int)kps;
    p.max_splits = (int)(((long)d->S_max + kps - 1) / kps);
    // Long ranges are dealt out on the device, one share per CU and unit block, unless the caller fixed them.
    // (A lane per sequence and per KV head; positions on the line and partial numbers stay within 32 bits.  Beyond that the
    // workgroups are many rounds, and the hardware's dispatch evens them out.)
    p.shares = 0;
    const long pairs = ((long)d->S_max + 2 * kKT - 1) / (2 * kKT), heads = (long)d->B * d->Hkv;
    if (!p.one && d->keys_per_split == 0 && kps >= kLongTiles * kKT && d->D == 128 && d->B <= kFlatMaxB && d->Hkv <= kWave && p.n_ublk <= 16 &&
        heads * (2 * pairs * kTileCost + kUnitCost) < (1l << 30))
        p.shares = 256 / p.n_ublk;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~size_t(255); return o; };
    take(256);                                             // never empty: callers always pass a workspace
    // shares and KV heads cut the same line: a piece's slot is the sum of its share's and its head's number
    const size_t slots = p.shares > 0 ? (size_t)(p.shares + heads) : p.max_splits > 1 ? (size_t)heads * p.max_splits : 0;
    const size_t entries = slots * p.n_ublk * kGsWaves;
    p.off_part_o = take(entries * 32 * (d->D / 2) * sizeof(uint32_t));
    p.off_part_ml = take(entries * 96 * sizeof(float));
    p.off_tab = take(p.shares > 0 ? heads * sizeof(uint64_t) : 0);
    p.bytes = off;
    return p;
}

}  // namespace radar

using namespace radar;

static radar_status check_attn_desc(const radar_attn_desc *d) {
    if (!d) return RADAR_INVALID_ARG;
    if (d->B < 1 || d->T_max < 1 || d->Hq < 1 || d->Hkv < 1 || d->S_max < 1 || d->Hq % d->Hkv != 0)
        return RADAR_INVALID_ARG;
    if (d->keys_per_split < 0 || d->keys_per_split % kKT != 0) return RADAR_INVALID_ARG;
    if (d->softmax_scale < 0.f) return RADAR_INVALID_ARG;
    if ((d->D != 64 && d->D != 128) || d->T_max > RADAR_T_MAX) return RADAR_UNSUPPORTED_SHAPE;
    if (d->B > 65535 || d->Hq > 65535) return RADAR_UNSUPPORTED_SHAPE;
    return RADAR_OK;
}

extern "C" size_t radar_tree_attention_workspace_bytes(const radar_attn_desc *d) {
    if (check_attn_desc(d) != RADAR_OK) return 0;
    return plan_attention(d).bytes;
}

template <int D>
constexpr int gs_smem_bytes() { return 2 * (2 * kKT * D * 2); }

template <int D, bool FLAT>
static hipError_t launch_ld(const AttnArgs &a, dim3 grid, hipStream_t s) {
    constexpr int bytes = kLdBufs * (2 * kKT * D * 2);
    static const hipError_t configured = hipFuncSetAttribute(reinterpret_cast<const void *>(&tree_attn_ld_kernel<D, FLAT>),
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (configured != hipSuccess) return configured;
    return launch("tree_attn_group_share", tree_attn_ld_kernel<D, FLAT>, grid, dim3(kGsThreads), bytes, s, a.ctx_lens, a.n_nodes, a.T, a.S, a.B, a.Hkv, a.G,
                  a.n_ublk, a.nqb, a.shares, a.shares_inv, a.per_unit, a);
}

template <int D, bool DEEP>
static hipError_t launch_gs(const AttnArgs &a, dim3 grid, hipStream_t s) {
    // the dynamic LDS limit is raised once per instantiation (a function-local static is initialised
    // exactly once, also when several threads launch at the same time)
    static const hipError_t configured = hipFuncSetAttribute(reinterpret_cast<const void *>(&tree_attn_gs_kernel<D, DEEP>),
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, gs_smem_bytes<D>());
    if (configured != hipSuccess) return configured;
    return launch("tree_attn_group_share", tree_attn_gs_kernel<D, DEEP>, grid, dim3(kGsThreads), gs_smem_bytes<D>(), s, a.k, a.v, a.kv_sb, a.kv_sh,
                  (int)a.kv_ss, a.kps, a.S, a.n_ublk | a.nqb << 16, a.q, a);
}

template <int D, bool EIGHTS>
static hipError_t launch_one(const AttnArgs &a, hipStream_t s) {
    const int heads = a.B * a.Hkv;                         // at most the 512 units of one launch: exact with the share rounded up
    const dim3 grid((unsigned)(EIGHTS ? 8 : a.Hkv), (unsigned)(a.G * a.nqb), (unsigned)(EIGHTS ? (heads + 7) / 8 : a.B));
    const uint32_t inv = ((1u << kInvShift) + a.Hkv - 1) / a.Hkv;
    constexpr int bytes = kGsWaves * (2 * kOneRows * D * 2 + 2 * 32 * (int)sizeof(float));
    static const hipError_t configured = hipFuncSetAttribute(reinterpret_cast<const void *>(&tree_attn_one_kernel<D, EIGHTS>),
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (configured != hipSuccess) return configured;
    return launch("tree_attn_one", tree_attn_one_kernel<D, EIGHTS>, grid, dim3(kGsThreads), bytes, s, a.k, a.v, a.ctx_lens, a.n_nodes, a.kv_sb, a.kv_sh,
                  EIGHTS ? a.Hkv : a.S, EIGHTS ? inv : (uint32_t)a.kv_ss, a);
}

extern "C" radar_status radar_tree_attention(const void *q, const void *k_cache, const void *v_cache,
                                             const int32_t *parents, const int32_t *ctx_lens, const int32_t *n_nodes,
                                             void *out, float *lse_out, const radar_attn_desc *d, void *workspace,
                                             size_t workspace_bytes, void *stream) {
    if (!q || !k_cache || !v_cache || !parents || !ctx_lens || !out || !workspace) return RADAR_INVALID_ARG;
    radar_status st = check_attn_desc(d);
    if (st != RADAR_OK) return st;
    const AttnPlan p = plan_attention(d);
    if (workspace_bytes < p.bytes) return RADAR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)workspace & 255) != 0) return RADAR_INVALID_ARG;

    AttnArgs a;
    a.q = static_cast<const __bf16 *>(q); a.k = static_cast<const __bf16 *>(k_cache);
    a.v = static_cast<const __bf16 *>(v_cache);
    a.parents = parents; a.ctx_lens = ctx_lens; a.n_nodes = n_nodes;
    a.out = static_cast<__bf16 *>(out); a.lse = lse_out;
    a.B = d->B; a.T = d->T_max; a.Hq = d->Hq; a.Hkv = d->Hkv; a.G = d->Hq / d->Hkv; a.S = d->S_max;
    a.kps = p.kps; a.max_splits = p.max_splits; a.n_ublk = p.n_ublk; a.nqb = p.nqb; a.shares = p.shares;
    a.shares_inv = p.shares > 0 ? (uint32_t)(((uint64_t(1) << 32) + p.shares - 1) / p.shares) : 0;
    const int64_t D = d->D;
    a.q_sh = d->q_stride_h ? d->q_stride_h : D;
    a.q_st = d->q_stride_t ? d->q_stride_t : D * d->Hq;
    a.q_sb = d->q_stride_b ? d->q_stride_b : D * d->Hq * d->T_max;
    a.kv_ss = d->kv_stride_s ? d->kv_stride_s : D;
    a.kv_sh = d->kv_stride_h ? d->kv_stride_h : D * d->S_max;
    a.kv_sb = d->kv_stride_b ? d->kv_stride_b : D * d->S_max * d->Hkv;
    a.o_sh = d->out_stride_h ? d->out_stride_h : D;
    a.o_st = d->out_stride_t ? d->out_stride_t : D * d->Hq;
    a.o_sb = d->out_stride_b ? d->out_stride_b : D * d->Hq * d->T_max;
    // 16-byte alignment of every row the kernels touch with vector accesses
    const uintptr_t al = (uintptr_t)q | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)out;
    const int64_t strides = a.q_sh | a.q_st | a.q_sb | a.kv_ss | a.kv_sh | a.kv_sb | a.o_sh | a.o_st | a.o_sb;
    if ((al & 15) != 0 || (strides & 7) != 0) return RADAR_INVALID_ARG;
    // the kernels address rows inside one head's cache / one head's queries with 32-bit offsets
    if (a.kv_ss <= 0 || a.q_st <= 0 || a.kv_ss * (int64_t)d->S_max >= (int64_t(1) << 31) ||
        a.q_st * (int64_t)d->T_max >= (int64_t(1) << 31))
        return RADAR_UNSUPPORTED_SHAPE;
    const float scale = d->softmax_scale != 0.f ? d->softmax_scale : 1.0f / sqrtf((float)d->D);
    a.scale_log2 = scale * kLog2e;
    char *ws = static_cast<char *>(workspace);
    a.part_o = reinterpret_cast<uint64_t *>(ws + p.off_part_o);
    a.part_ml = reinterpret_cast<float *>(ws + p.off_part_ml);
    a.per_unit = p.shares / (d->B * d->Hkv);
    a.unit_tab = reinterpret_cast<uint64_t *>(ws + p.off_tab);

    hipStream_t s = static_cast<hipStream_t>(stream);
    if ((long)a.B * a.n_ublk > 65535) return RADAR_UNSUPPORTED_SHAPE;
    if (p.one) {
        const hipError_t e = p.by_eights ? (d->D == 128 ? launch_one<128, true>(a, s) : launch_one<64, true>(a, s))
                                         : (d->D == 128 ? launch_one<128, false>(a, s) : launch_one<64, false>(a, s));
        return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
    }
    const dim3 grid = p.shares > 0 ? dim3((unsigned)p.shares, 1, (unsigned)p.n_ublk)
                                   : dim3((unsigned)a.max_splits, (unsigned)a.Hkv, (unsigned)(a.B * a.n_ublk));
    {
        hipError_t e;
        if (p.shares > 0)     e = launch_ld<128, true>(a, grid, s);
        else if (p.kps >= kLongTiles * kKT) e = d->D == 128 ? launch_ld<128, false>(a, grid, s) : launch_gs<64, true>(a, grid, s);
        else                  e = d->D == 128 ? launch_gs<128, false>(a, grid, s) : launch_gs<64, false>(a, grid, s);
        if (e != hipSuccess) return RADAR_HIP_ERROR;
    }
    if (a.max_splits > 1 || p.shares > 0) {
        const bool many = p.shares >= 16l * d->B * d->Hkv;          // sixteen shares per KV head or more (dealt-out rows only: D = 128)
        // Many partials at once take registers that a launch of more wavefronts needs to have all of them on the chip: up to 640
        // (40 heads of 60 rows, 160 of 16 rows).  One sequence of 2048 rows: 32 heads 16.0 -> 15.0 us (8 -> 18 partials at
        // a time), 16 tree rows 11.7 -> 10.6, 8 heads on 2 13.7 -> 12.4, D = 64 on 4 10.6 -> 9.5; with 48 or 64 heads
        // 3000 rows would go from 17.6 to 17.8 and from 19.4 to 19.9.
        const bool wide = (long)d->D / 32 * a.Hq * a.B * (d->T_max > 32 ? 4 : d->T_max > 16 ? 2 : 1) <= 640;
        const dim3 mgrid((unsigned)(d->D / kMergeSlice * a.G), (unsigned)a.Hkv, (unsigned)a.B);
        auto go = [&](auto kernel, int groups) {
            return launch("tree_attn_merge", kernel, mgrid, dim3((unsigned)(kAttnThreads * groups)), 0, s, a.part_o, a.part_ml, a.ctx_lens, a.n_nodes, a.T,
                          p.shares > 0 ? (int)(p.off_tab - p.off_part_ml) : a.kps, a.S, a.max_splits, (uint32_t)a.Hkv | (uint32_t)a.G << 16, a.n_ublk | a.nqb << 16, a);
        };
        const hipError_t e = d->D == 64 ? (wide ? go(tree_attn_merge_kernel<64, 1, 18, true>, 1) : go(tree_attn_merge_kernel<64, 1, 8, true>, 1))
                           : p.shares == 0 ? (wide ? go(tree_attn_merge_kernel<128, 1, 18, true>, 1) : go(tree_attn_merge_kernel<128, 1, 8, true>, 1))
                           : many       ? (wide ? go(tree_attn_merge_kernel<128, 2, 18, false>, 2) : go(tree_attn_merge_kernel<128, 2, 4, false>, 2))
                                        : (wide ? go(tree_attn_merge_kernel<128, 1, 18, false>, 1) : go(tree_attn_merge_kernel<128, 1, 8, false>, 1));
        if (e != hipSuccess) return RADAR_HIP_ERROR;
    }
    return RADAR_OK;
}
