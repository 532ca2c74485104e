// radar_verify_accept_q: verification with draft distributions (Sec. 3, Eq. 1-2), for trees
// whose tokens were drawn from the draft model's distributions.
//
// One launch.  The walk is sequential by nature (Eq. 1 is applied child by child, Eq. 2 changes the
// distribution every later test sees), and it visits few rows: the target rows on the accepted path and
// the draft rows of the children it tests.  Only those are read.  (Taking every row's normaliser first,
// with the whole chip, read 62 MB at 61 + 61 rows of V = 128256 and was 17 of a call's 42 us; the walk
// that followed read its rows again.)
//
// The walk of a sequence is shared by up to 32 workgroups, each of which holds a slice of the rows at hand
// in registers; after every row and every rejection they meet and exchange a few numbers each.  What
// bounds a call is that chain: rows from HBM (about 2 us, requested one node ahead) and a meeting (about
// 1.5 us) per node and per rejection.  Slices that do not fit into registers are walked over in laps.  Where
// there are more sequences than pairs of workgroups, where a row fits one workgroup's first float4,
// and where workgroups of a sequence could not meet or the caller wants none that wait, one workgroup walks alone:
// every rejection is then a vocabulary-wide pass that turns the unnormalised residual u into max(0, u - W q)
// (W = sum u), keeps it in a workspace row and leaves sums per 256 tokens in LDS, from which the bonus token is
// found.  Where such a call has few rows, the whole chip takes their statistics in a launch before it.
#include <type_traits>

#include "radar_device.h"
#include "radar_host.h"

namespace radar {

constexpr int kAqWaves = 8;                           // wavefronts that hold the vocabulary
constexpr int kAqStream = kAqWaves * kWave;
constexpr int kAqThreads = kAqStream + kWave;         // and one that meets the other workgroups and decides
constexpr int kAqLone = 1024;                         // a lone walk that was launched as one: more loads in flight
constexpr int kAqMaxV = 1 << 20;
constexpr int kAqGran = 4 * kWave;                    // tokens per partial sum in the lone walk (one wavefront x 16 B)
constexpr int kAqMaxGran = kAqMaxV / kAqGran;         // 4096
constexpr int kAqChunk = 16384;                       // tokens per workgroup of the statistics launch
constexpr int kCoG = 32;                              // most workgroups per sequence
constexpr int kCoR = 8;                               // most float4 per lane that a row's slice may take in registers
constexpr int kCoLapR = 4;                            // and what is taken at a time where a slice is longer
constexpr int kCoCtl = 32;                            // uints per sequence in the control block: leave counter, abort flag at 8, 16
constexpr int kCoWords = 4;                           // 8-byte words a workgroup brings to a meeting

struct AqArgs {
    const float *target;        // [B][T][V]
    const float *draft;         // [B][Tq][V]
    const int32_t *q_rows;      // [B][T] or null
    const int32_t *tokens, *parents, *n_nodes;
    const float *uniforms;      // [B][T+1]
    int32_t *accept_len, *accept_path, *bonus;
    int B, T, Tq, V, D_max;
    double inv_t, inv_td;
    float *part_m;              // statistics launch: [B*T + B*Tq][nchunks] maximum per chunk
    double *part_l;             // and its sum of exponentials
    int nchunks;
    float *ubuf;                // [B][V] unnormalised residual of the node being verified (lone walk, long slices)
    int co_laps;                // long slices: how often R float4 per lane go into one
    unsigned int *co_ctl;       // [B][32]
    uint64_t *co_words;         // [B][2][32][4] what the workgroups brought to the last two meetings
    uint64_t *co_sib;           // [B][2][64] residual at the tokens of untried children
    unsigned int co_spin_limit; // polls of a meeting before a workgroup gives up
};

// exp((x - m) * inv_temp) with the difference formed in fp64, rounded to fp32 once, and the fp32
// hardware exponential; the sums that use it are fp64.
__device__ __forceinline__ double exp_rel(float x, float m, double inv_temp) {
    return (double)__expf((float)(((double)x - (double)m) * inv_temp));
}

// the same in fp32 throughout (relative error about 1e-7 per unit of |x - m| * inv_temp)
__device__ __forceinline__ float exp_rel_f32(float x, float m, float inv_temp) { return __expf((x - m) * inv_temp); }

// a value that is the same in every lane (read from LDS, say), kept in a scalar register
__device__ __forceinline__ int uniform_of(int v) { return __builtin_amdgcn_readfirstlane(v); }

// sum over the workgroup of N threads of one double per thread, fixed order; every thread gets it
template <int N>
__device__ __forceinline__ double block_sum_f64(double v, double *wred) {
    const double ws = wave_sum_f64(v);
    __syncthreads();
    if (lane_id() == 0) wred[wave_id()] = ws;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < N / kWave; ++i) t += wred[i];
    return t;
}

// ------------------------------------------------------------------------ walk by one workgroup
struct AqSmem {
    double gsum[kAqMaxGran];     // residual mass per 256 tokens (of the last pass)
    double wred[kAqLone / kWave];
    float wmax[kAqLone / kWave];
    double px[kWave];            // per node: residual at its token under its parent
    float qx[kWave];             // draft logit of its token
    int par[kWave], tok[kWave], qrow[kWave];
    float uni[kWave + 1];
    double W;                    // mass of the residual
    unsigned long long kids;     // untried children of the current node
    int cur, len, next, have_u;
    int chunk;                   // where the bonus token lies, and the mass in front of it
    double before;
};

// maximum of a row and sum of exp((x - maximum) * inv) (all threads call it): row number `id` of the call, from the
// statistics launch if there was one, else from the row itself
template <bool VEC4, int N, bool PARTS>
__device__ __forceinline__ void row_stats(const AqArgs &a, AqSmem &s, const float *row, int id, double inv, float *m_out, double *l_out) {
    const int tid = threadIdx.x;
    float m = -INFINITY;
    double l = 0.0;
    if constexpr (PARTS) {                                           // at most 64 chunks, one per lane, in every wavefront
        const bool has = lane_id() < a.nchunks;
        const size_t at = (size_t)id * a.nchunks + min(lane_id(), a.nchunks - 1);
        const float mc = has ? a.part_m[at] : -INFINITY;
        const double lc = a.part_l[at];
        m = wave_max_f32(mc);
        *m_out = m;
        *l_out = wave_sum_f64(mc > -INFINITY ? lc * exp(((double)mc - (double)m) * inv) : 0.0);
        return;
    }
    for (int pass = 0; pass < 2; ++pass) {
        if (VEC4) {
#pragma unroll 4
            for (int i = tid * 4; i < a.V; i += N * 4) {
                const float4 v = *reinterpret_cast<const float4 *>(row + i);
                if (pass == 0) m = fmaxf(fmaxf(fmaxf(m, v.x), fmaxf(v.y, v.z)), v.w);
                else l += (exp_rel(v.x, m, inv) + exp_rel(v.y, m, inv)) + (exp_rel(v.z, m, inv) + exp_rel(v.w, m, inv));
            }
        } else {
#pragma unroll 4
            for (int i = tid; i < a.V; i += N) {
                if (pass == 0) m = fmaxf(m, row[i]);
                else l += exp_rel(row[i], m, inv);
            }
        }
        if (pass == 0) {
            m = wave_max_f32(m);
            __syncthreads();
            if (lane_id() == 0) s.wmax[wave_id()] = m;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < N / kWave; ++i) m = fmaxf(m, s.wmax[i]);
        }
    }
    *m_out = m;
    *l_out = block_sum_f64<N>(l, s.wred);
}

// One pass over tokens [lo, hi) of sequence b (lo a multiple of 256):
//   u(i) = have_u ? ubuf[i] : softmax(target row)[i];   u(i) <- max(0, u(i) - W * q(i)) when q is given;
// u is written to ubuf (as fp32), its sums per 256 tokens to s.gsum[(i - lo) / 256]; returns the total
// of the stored values.  All threads call it.
template <bool VEC4, int N>
__device__ __forceinline__ double residual_pass(const AqArgs &a, AqSmem &s, int b, const float *prow, float pm, double pinv_l,
                                                const float *qrow, float qm, double qinv_l, double W, int lo, int hi) {
    const int tid = threadIdx.x, lane = lane_id();
    float *ub = a.ubuf + (size_t)b * a.V;
    const int ngran = (hi - lo + kAqGran - 1) / kAqGran;
    const float it_f = (float)a.inv_t, itd_f = (float)a.inv_td, pinv_l_f = (float)pinv_l, qinv_l_f = (float)qinv_l, W_f = (float)W;
    constexpr int U = VEC4 ? 4 : 3;                                  // steps of 4 N tokens whose loads are in flight together (word by word a fourth spills)
    for (int base0 = lo + tid * 4; base0 - lane * 4 < hi; base0 += U * N * 4) {
        float u4[U][4], q4[U][4];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int base = base0 + k * N * 4;
            if (VEC4) {                                              // V % 4 == 0: a float4 is all in or all out
                const int i0 = base < hi ? base : lo;                // out of range: any legal address, masked below
                const float4 v = *reinterpret_cast<const float4 *>((prow ? prow : ub) + i0);
                u4[k][0] = v.x; u4[k][1] = v.y; u4[k][2] = v.z; u4[k][3] = v.w;
                if (qrow) {
                    const float4 y = *reinterpret_cast<const float4 *>(qrow + i0);
                    q4[k][0] = y.x; q4[k][1] = y.y; q4[k][2] = y.z; q4[k][3] = y.w;
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = min(base + j, hi - 1);
                    u4[k][j] = (prow ? prow : ub)[i];
                    if (qrow) q4[k][j] = qrow[i];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int base = base0 + k * N * 4;
            if (base - lane * 4 >= hi) break;                        // wave-uniform
            // fp32 per token (one workgroup's vector ALUs, not its memory path, bound this loop), fp64 sums
            float out[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float u = prow ? exp_rel_f32(u4[k][j], pm, it_f) * pinv_l_f : u4[k][j];
                if (qrow) u = fmaxf(0.f, fmaf(-W_f, exp_rel_f32(q4[k][j], qm, itd_f) * qinv_l_f, u));
                out[j] = (base + j < hi) ? u : 0.f;
            }
            double sum = ((double)out[0] + (double)out[1]) + ((double)out[2] + (double)out[3]);
            if (VEC4) {
                if (base < hi) *reinterpret_cast<float4 *>(ub + base) = make_float4(out[0], out[1], out[2], out[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (base + j < hi) ub[base + j] = out[j];
            }
            sum = wave_sum_f64(sum);
            if (lane == 0) s.gsum[(base - lo) / kAqGran] = sum;
        }
    }
    __syncthreads();
    double part = 0.0;
    for (int g = tid; g < ngran; g += N) part += s.gsum[g];
    return block_sum_f64<N>(part, s.wred);
}

// Inverse CDF by wavefront 0: first token i in [lo, hi) with before0 + sum_{lo..i} u > target, or, if
// the sums never get there (rounding), the last token with u > 0; -1 if there is none.  The sums per
// 256 tokens are in s.gsum, u itself in ubuf.  Returns the token to every lane of wavefront 0.
template <bool VEC4>
__device__ __forceinline__ int pick_token(const AqArgs &a, AqSmem &s, int b, double before0, double target, int lo, int hi) {
    const int lane = lane_id();
    const float *ub = a.ubuf + (size_t)b * a.V;
    const int ngran = (hi - lo + kAqGran - 1) / kAqGran;
    const int per = (ngran + kWave - 1) / kWave;
    // each lane owns `per` consecutive granules
    double mine = 0.0;
    int last_pos = -1;
    for (int g = lane * per; g < min((lane + 1) * per, ngran); ++g) {
        mine += s.gsum[g];
        if (s.gsum[g] > 0.0) last_pos = g;
    }
    const double incl = wave_scan_f64(mine);
    const uint64_t cross = __ballot(before0 + incl > target);
    int g_pick;
    double before;
    if (cross != 0) {
        const int owner = __ffsll((long long)cross) - 1;
        // the owner walks its granules
        int g_loc = -1;
        double acc = before0 + incl - mine, bef = acc;
        for (int g = lane * per; g < min((lane + 1) * per, ngran); ++g) {
            if (g_loc < 0) {
                bef = acc;
                acc += s.gsum[g];
                if (acc > target) g_loc = g;
            }
        }
        if (g_loc < 0) {                                             // the lane's own running sum was rounded differently: its last granule
            g_loc = min((lane + 1) * per, ngran) - 1;
            bef = acc - s.gsum[g_loc];
        }
        g_pick = __shfl(g_loc, owner);
        before = readlane_f64(bef, owner);
    } else {
        // no crossing: the last granule with mass
        int lp = last_pos;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) lp = max(lp, __shfl_xor(lp, off));
        if (lp < 0) return -1;
        g_pick = lp;
        before = -1.0;                                               // marks "take the last positive token"
    }
    // the 256 tokens of the granule, 4 per lane in token order
    const int i0 = lo + g_pick * kAqGran + lane * 4;
    double v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (i0 + j < hi) ? (double)ub[i0 + j] : 0.0;
    if (before < 0.0) {
        int lastj = -1;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (v[j] > 0.0) lastj = i0 + j;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) lastj = max(lastj, __shfl_xor(lastj, off));
        return lastj;
    }
    const double lsum = (v[0] + v[1]) + (v[2] + v[3]);
    const double linc = wave_scan_f64(lsum);
    const uint64_t c2 = __ballot(before + linc > target);
    if (c2 == 0) {                                                   // the granule's own sum was rounded differently: its last positive token
        int lastj = -1;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (v[j] > 0.0) lastj = i0 + j;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) lastj = max(lastj, __shfl_xor(lastj, off));
        return lastj;
    }
    const int owner2 = __ffsll((long long)c2) - 1;
    double acc = before + linc - lsum;
    int pick = -1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        acc += v[j];
        if (pick < 0 && acc > target) pick = i0 + j;
    }
    return __shfl(pick, owner2);
}

// The whole walk of sequence b by one workgroup of N threads (all of them call it).
template <bool VEC4, int N, bool PARTS>
__device__ __forceinline__ void walk_single(const AqArgs &a, AqSmem &s, int b) {
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int nn = a.n_nodes ? min(max(a.n_nodes[b], 0), a.T) : a.T;
    int32_t *path = a.accept_path + (size_t)b * (a.D_max + 1);
    for (int d = tid; d <= a.D_max; d += N) path[d] = d == 0 && nn >= 1 ? 0 : -1;
    if (nn < 1) {
        if (tid == 0) { a.accept_len[b] = 0; a.bonus[b] = -1; }
        return;
    }
    if (tid < kWave) {
        const bool live = tid < nn;
        s.par[tid] = live ? a.parents[(size_t)b * a.T + tid] : -2;
        s.tok[tid] = live ? a.tokens[(size_t)b * a.T + tid] : -1;
        s.qrow[tid] = !live ? -1 : a.q_rows ? a.q_rows[(size_t)b * a.T + tid] : tid;
        s.uni[tid] = tid <= a.T ? a.uniforms[(size_t)b * (a.T + 1) + tid] : 0.f;
        if (tid == 0) { s.uni[kWave] = a.T == kWave ? a.uniforms[(size_t)b * (a.T + 1) + kWave] : 0.f; s.cur = 0; s.len = 0; }
    }
    __syncthreads();

    for (;;) {                                                       // one iteration per visited node; at most T of them
        const int cur = s.cur, len = s.len;
        const float *prow = a.target + ((size_t)b * a.T + cur) * a.V;
        float pm, qm = 0.f;
        double pl, ql = 1.0;
        int q_have = -1;                                             // the draft row whose statistics are at hand
        row_stats<VEC4, N, PARTS>(a, s, prow, b * a.T + cur, a.inv_t, &pm, &pl);
        const double pinv_l = 1.0 / pl;
        // ---- children of cur (ascending node index) and, for each, p(token) and its draft logit
        if (w == 0) {
            const int x = s.tok[lane], qr = s.qrow[lane];
            const bool kid = lane > cur && lane < nn && s.par[lane] == cur && len < a.D_max && x >= 0 && x < a.V && qr >= 0 && qr < a.Tq;
            if (kid) {
                s.px[lane] = exp_rel(prow[x], pm, a.inv_t) * pinv_l;
                s.qx[lane] = a.draft[((size_t)b * a.Tq + qr) * a.V + x];
            }
            const unsigned long long kids = __ballot(kid);
            if (lane == 0) { s.kids = kids; s.W = 1.0; s.have_u = 0; s.next = -1; }
        }
        __syncthreads();
        // ---- Eq. 1 child by child; Eq. 2 after every rejection
        while (s.kids != 0 && s.next < 0 && s.W > 0.0) {
            const int c = __ffsll((long long)s.kids) - 1, qr = s.qrow[c];
            const float *qrow = a.draft + ((size_t)b * a.Tq + qr) * a.V;
            if (qr != q_have) { row_stats<VEC4, N, PARTS>(a, s, qrow, a.B * a.T + b * a.Tq + qr, a.inv_td, &qm, &ql); q_have = qr; }
            const double W = s.W;
            const bool accept = (double)s.uni[c] * W * (exp_rel(s.qx[c], qm, a.inv_td) / ql) < s.px[c];
            __syncthreads();                                         // everyone has read the state of this test
            if (accept) {
                if (tid == 0) s.next = c;
            } else {
                const double total = residual_pass<VEC4, N>(a, s, b, s.have_u ? nullptr : prow, pm, pinv_l, qrow, qm, 1.0 / ql, W, 0, a.V);
                // the residual at the tokens of the children still to be tried (written by this workgroup)
                const unsigned long long rest = s.kids & ~(1ull << c);
                if (w == 0 && ((rest >> lane) & 1)) s.px[lane] = (double)a.ubuf[(size_t)b * a.V + s.tok[lane]];
                __syncthreads();
                if (tid == 0) { s.kids = rest; s.W = total; s.have_u = 1; }
            }
            __syncthreads();
        }
        if (s.next >= 0) {
            if (tid == 0) {
                const int c = s.next;
                s.cur = c;
                s.len = len + 1;
                path[len + 1] = c;
            }
            __syncthreads();
            continue;
        }
        // ---- bonus token from the residual (or from p itself when nothing was rejected, or when
        // the residual vanished)
        double W = s.W, before0 = 0.0;
        int lo = 0, hi = a.V;
        const bool use_u = s.have_u && W > 0.0;
        __syncthreads();
        if (PARTS && !use_u) {
            // the chunk that the token lies in, from the row's partials; u = p is then made on that chunk only
            W = 1.0;
            if (w == 0) {
                const float mc = lane < a.nchunks ? a.part_m[((size_t)b * a.T + cur) * a.nchunks + lane] : -INFINITY;
                // (a chunk counts if its largest probability is above zero in fp32, in which u is made: others have no token to find)
                const bool any = mc > -INFINITY && exp_rel_f32(mc, pm, (float)a.inv_t) * (float)pinv_l > 0.f;
                const double mass = any ? a.part_l[((size_t)b * a.T + cur) * a.nchunks + lane] * exp(((double)mc - (double)pm) * a.inv_t) * pinv_l : 0.0;
                const double incl = wave_scan_f64(mass);
                const uint64_t cross = __ballot(lane < a.nchunks && incl > (double)s.uni[a.T]), has = __ballot(mass > 0.0);
                const int ch = cross ? __ffsll((long long)cross) - 1 : has ? 63 - __clzll((long long)has) : 0;
                const double bef = readlane_f64(incl - mass, ch);
                if (lane == 0) { s.chunk = ch; s.before = bef; }
            }
            __syncthreads();
            lo = s.chunk * kAqChunk;
            hi = min(a.V, lo + kAqChunk);
            before0 = s.before;
        }
        if (!use_u) {
            const double mass = residual_pass<VEC4, N>(a, s, b, prow, pm, pinv_l, nullptr, 0.f, 0.0, 0.0, lo, hi);
            if (!PARTS) W = mass;
        }
        if (w == 0) {
            const int pick = pick_token<VEC4>(a, s, b, before0, (double)s.uni[a.T] * W, lo, hi);
            if (lane == 0) {
                a.bonus[b] = pick;
                a.accept_len[b] = len;
            }
        }
        return;
    }
}

// Statistics of every row that a lone walk may visit, taken by the whole chip beforehand: one workgroup per 16384
// logits of a row leaves its maximum and sum; the walk merges a row's when it gets there.  (Where that
// pays: aq_take_statistics.)
template <bool VEC4>
__global__ __launch_bounds__(kAqStream) void accept_q_stats_kernel(AqArgs a) {
    __shared__ float wm[kAqWaves];
    __shared__ double wl[kAqWaves];
    const int tid = threadIdx.x, lane = lane_id(), id = blockIdx.y, lo = blockIdx.x * kAqChunk;
    const bool is_target = id < a.B * a.T;
    const int b = is_target ? id / a.T : (id - a.B * a.T) / a.Tq, r = is_target ? id % a.T : (id - a.B * a.T) % a.Tq;
    const int nn = a.n_nodes ? min(max(a.n_nodes[b], 0), a.T) : a.T;
    if (is_target) {
        if (r >= nn) return;
    } else {                                                         // the rows of live nodes other than the root
        const int qr = lane >= 1 && lane < nn ? (a.q_rows ? a.q_rows[(size_t)b * a.T + lane] : lane) : -1;
        if (__ballot(qr == r) == 0) return;
    }
    const float *row = is_target ? a.target + (size_t)id * a.V : a.draft + (size_t)(id - a.B * a.T) * a.V;
    const double inv = is_target ? a.inv_t : a.inv_td;
    constexpr int R = kAqChunk / (kAqStream * 4);
    float x[R][4], m = -INFINITY;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int i0 = lo + (k * kAqStream + tid) * 4;
        const float4 v = VEC4 ? *reinterpret_cast<const float4 *>(row + (i0 < a.V ? i0 : 0)) : load4_of_row(row, i0, a.V);   // (V >= 12288)
        x[k][0] = v.x; x[k][1] = v.y; x[k][2] = v.z; x[k][3] = v.w;
    }
    if (!VEC4) place_row_end<R>([&](int k, int j) -> float & { return x[k][j]; }, lo + tid * 4, kAqStream * 4, a.V);
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[k][j] = lo + (k * kAqStream + tid) * 4 + j < a.V ? x[k][j] : -INFINITY;
            m = fmaxf(m, x[k][j]);
        }
    m = wave_max_f32(m);
    if (lane == 0) wm[wave_id()] = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kAqWaves; ++i) m = fmaxf(m, wm[i]);
    double l = 0.0;
    if (m > -INFINITY) {
#pragma unroll
        for (int k = 0; k < R; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) l += inv == 1.0 ? (double)exp_rel_f32(x[k][j], m, 1.f) : exp_rel(x[k][j], m, inv);   // (the same value)
    }
    l = wave_sum_f64(l);
    if (lane == 0) wl[wave_id()] = l;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < kAqWaves; ++i) t += wl[i];
        a.part_m[(size_t)id * a.nchunks + blockIdx.x] = m;
        a.part_l[(size_t)id * a.nchunks + blockIdx.x] = t;
    }
}

template <bool VEC4, bool PARTS>
__global__ __launch_bounds__(kAqLone) void accept_q_walk_kernel(AqArgs a) {
    __shared__ AqSmem s;
    walk_single<VEC4, kAqLone, PARTS>(a, s, blockIdx.x);
}

// ------------------------------------------------------------------- walk by several workgroups
// G workgroups per sequence; workgroup g holds tokens [g * slice, (g + 1) * slice) of the rows at hand in
// the registers of eight wavefronts (R float4 per lane and row): the current node's target row, which
// becomes the residual at the first rejection, the draft row of the child being tested, and, one node
// ahead, the rows that will be asked for if that child is accepted.  The ninth wavefront does everything
// that is said and decided: it merges the wavefronts' results, meets the other workgroups and tests the
// next child.  (It loads no rows: a wavefront's loads return in order, and a poll would wait for them.)
// While it does, the others take the statistics of the rows one node ahead: an accepted first child's meeting
// begins with the decision.  (Taken after it, a node cost 3.6 us where it costs 2.6 now; in a call of one sequence,
// V = 128256, a meeting's words are 1.1 us on their way, merging them and deciding takes 0.7, rows that are not
// ahead 0.75 + their load.  Calls of one / four sequences that replay one tree 28.3 / 31.0 -> 26.4 / 26.7 us, over twelve / four trees in
// turn (their rows cold) 20.8 / 28.1 -> 20.0 / 26.7.  Rows too
// long to be held one ahead gain from the two rows' chains side by side: 16 / 32 sequences 61.2 / 79.5 -> 57.1 / 72.0.  Having the last of the
// eight merge their results at once (18.0 instead of 17.6) and two polls in flight (2 % slower) were taken out again.)
//
// Every workgroup takes the same decisions from the same numbers, added in the same order.  At a meeting
// a workgroup stores two or four 8-byte words, each with the meeting's number in its low byte, and polls
// all workgroups' words until they carry that number: the values need no counter to vouch for them, no
// acknowledgement is awaited and nothing is fetched afterwards.  Two sets of words alternate; one is
// written again only after everyone has read the set after it.
// The wait is bounded: a workgroup that gives up (the workgroups of a sequence were not all resident,
// which the host avoids by keeping G * B within the chip) raises the sequence's abort flag, everyone
// leaves, and the last one to leave redoes the sequence alone.
enum { kCoAccept, kCoReject, kCoBonusP, kCoBonusU, kCoAbort };

struct CoSmem {
    // statistics and children's logits: of the node at hand, and of the one that is next if its first child is accepted
    float wm[2][2][kAqWaves];    // per wavefront: maximum and sum of exponentials of its part of the target / draft row
    double wl[2][2][kAqWaves];
    double wsum[kAqWaves];       // residual mass of its part
    float gx[2][kWave], gq[2][kWave];   // per child of the node: target and draft logit of its token
    float pm, pinv_l, qm, qinv_l, W;
    uint64_t order[2];           // command and node of the last two decisions: the next may be taken while one is read
    int gave_up;
    int owner, take_last, pick, wlast[kAqWaves];
    double before, goal;
    double wtot[2][kCoR][kAqWaves];
    int last, redo;
};

union CoLds {
    CoSmem s;
    AqSmem alone;
};

// A double travels whole: its low byte, which the meeting's number replaces in the first word of a pair, sits
// above that number in the second, whose upper half is free for a float.
__device__ __forceinline__ uint64_t word_of_f64(double v, unsigned int tag) { return ((uint64_t)__double_as_longlong(v) & ~0xffull) | tag; }
__device__ __forceinline__ uint64_t word_of_rest(double v, float m, unsigned int tag) {
    return ((uint64_t)__float_as_uint(m) << 32) | (((uint64_t)__double_as_longlong(v) & 0xffull) << 8) | tag;
}
__device__ __forceinline__ double f64_of_words(uint64_t w, uint64_t rest) { return __longlong_as_double((long long)((w & ~0xffull) | ((rest >> 8) & 0xffull))); }
__device__ __forceinline__ uint64_t word_of_f32(float v, unsigned int tag) { return ((uint64_t)__float_as_uint(v) << 32) | tag; }
__device__ __forceinline__ float f32_of_word(uint64_t w) { return __uint_as_float((uint32_t)(w >> 32)); }

// LAPS: slices longer than eight float4 per lane (large batches, V beyond 32 * 16384) are walked over in laps of R
// float4 per lane: rows are read from memory as often as they are needed (one read for the statistics, one per
// rejection), and the residual is kept in the workspace.  What bounds it is one CU's path to memory, some 64 KB/us.
template <bool VEC4, int R, bool LAPS>
__global__ __launch_bounds__(kAqThreads) void accept_q_coop_kernel(const int32_t *parents, const int32_t *tokens, const int32_t *q_rows, const int32_t *n_nodes,
                                                                    const float *target_rows, int T, int V, int D_max, AqArgs a) {
    a.parents = parents; a.tokens = tokens; a.q_rows = q_rows; a.n_nodes = n_nodes; a.target = target_rows; a.T = T; a.V = V; a.D_max = D_max;
    __shared__ CoLds lds;
    CoSmem &s = lds.s;
    const int tid = threadIdx.x, lane = lane_id(), w = uniform_of(wave_id());
    const bool control = w == kAqWaves;
    const int g = blockIdx.x, G = gridDim.x, b = blockIdx.y;
    constexpr int lap_tokens = R * kAqStream * 4;
    const int laps = LAPS ? a.co_laps : 1, slice = laps * lap_tokens, lo = g * slice;
    const int nn = a.n_nodes ? min(max(a.n_nodes[b], 0), a.T) : a.T;
    unsigned int *ctl = a.co_ctl + (size_t)b * kCoCtl;
    uint64_t *words = a.co_words + (size_t)b * 2 * kCoG * kCoWords;
    uint64_t *sibs = a.co_sib + (size_t)b * 2 * kWave;
    int32_t *path = a.accept_path + (size_t)b * (a.D_max + 1);
    const float *target = a.target + (size_t)b * a.T * a.V, *draft = a.draft + (size_t)b * a.Tq * a.V;

    // this lane's tokens: float4 r of a lap covers lo + lap * lap_tokens + (r * 512 + tid) * 4 .. + 3
    // (made anew for every row: the offsets and end-of-row masks of 4 R tokens are not worth keeping through the walk)
    auto first_token = [&](int lap) { int i = lo + lap * lap_tokens + tid * 4; asm volatile("" : "+v"(i)); return i; };
    auto load_row = [&](const float *row, float (&x)[R][4], int lap = 0) {
        const int at = first_token(lap);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i0 = at + r * kAqStream * 4;
            const float4 v = VEC4 ? *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(row) + (uint32_t)(i0 < a.V ? i0 : 0) * 4u)
                                  : load4_of_row(row, i0, a.V);    // (V > 2048 here)
            x[r][0] = v.x; x[r][1] = v.y; x[r][2] = v.z; x[r][3] = v.w;
        }
    };
    constexpr bool kAhead = R <= 2 && !LAPS;              // rows are requested one node ahead (wider slices have no registers left)
    float nx[kAhead ? R : 1][4], nq[kAhead ? R : 1][4], ngx = 0.f, ngq = 0.f;   // one ahead; its children's logits (wavefront 0)
    // the tree, one node per lane, in every wavefront
    const bool live = lane < nn;
    const int nl = min(lane, a.T - 1);
    int par = a.parents[(size_t)b * a.T + nl], tok = a.tokens[(size_t)b * a.T + nl];
    int qrow = a.q_rows ? a.q_rows[(size_t)b * a.T + nl] : lane;
    const float uni = control ? a.uniforms[(size_t)b * (a.T + 1) + min(lane, a.T)] : 0.f;
    const float uni_bonus = control ? a.uniforms[(size_t)b * (a.T + 1) + a.T] : 0.f;
    if constexpr (kAhead) if (!control) load_row(target, nx);     // the root's row does not wait for the tree
    __builtin_amdgcn_sched_barrier(0);
    if (!live) { par = -2; tok = -1; qrow = -1; }
    const bool usable = live && tok >= 0 && tok < a.V && qrow >= 0 && qrow < a.Tq;
    auto kids_of = [&](int node, int depth) -> uint64_t {
        return depth < a.D_max ? __ballot(usable && lane > node && par == node) : 0ull;
    };
    auto first_of = [](uint64_t m) { return __ffsll((long long)m) - 1; };
    auto qrow_of = [&](int node) { return (int)readlane_u32((uint32_t)qrow, node); };

    // Outputs are written through (agent-scope stores): should the sequence be redone by another
    // workgroup, on another die, no older copy of them may linger in this die's L2 to be written back later.
    if (g == 0) for (int d = tid; d <= a.D_max; d += kAqThreads) store_shared_result(&path[d], d == 0 && nn >= 1 ? 0 : -1);
    if (nn < 1) {                                         // nobody meets on this path
        if (g == 0 && tid == 0) { store_shared_result(&a.accept_len[b], 0); store_shared_result(&a.bonus[b], -1); }
        return;
    }

    const float it_f = (float)a.inv_t, itd_f = (float)a.inv_td;
    // tokens past the vocabulary (at the end of the last slice only) are -inf from here on: no mass in a row, none in
    // a residual (a residual read back: 0)
    auto settle = [&](float (&x)[R][4], int lap = 0, float none = -INFINITY) {
        if (lo + (lap + 1) * lap_tokens <= a.V) return;
        const int at = first_token(lap);
        if (!VEC4) place_row_end<R>([&](int r, int j) -> float & { return x[r][j]; }, at, kAqStream * 4, a.V);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[r][j] = at + r * kAqStream * 4 + j < a.V ? x[r][j] : none;
    };
    // maximum over the wavefront's tokens and this lane's sum of exponentials
    auto lane_stats = [&](const float (&x)[R][4], double inv, double *l_out) -> float {
        float m = -INFINITY;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) m = fmaxf(m, x[r][j]);
        m = wave_max_f32(m);
        double l = 0.0;
        if (m > -INFINITY) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
#pragma unroll
                for (int j = 0; j < 4; ++j) l += inv == 1.0 ? (double)exp_rel_f32(x[r][j], m, 1.f) : exp_rel(x[r][j], m, inv);   // (the same value)
            }
        }
        *l_out = l;
        return m;
    };
    int at = 0;                                           // which of the two statistics is the current node's
    auto put_stats = [&](float m, double l, int which, int buf) {
        l = wave_sum_f64(l);
        if (lane == 0) { s.wm[buf][which][w] = m; s.wl[buf][which][w] = l; }
    };
    auto wave_stats = [&](const float (&x)[R][4], double inv, int which, int buf) {
        double l;
        const float m = lane_stats(x, inv, &l);
        put_stats(m, l, which, buf);
    };
    // wave_stats of a target row and a draft row, their chains of dependent steps side by side
    auto both_stats = [&](const float (&x)[R][4], const float (&y)[R][4], int buf) {
        float mx = -INFINITY, my = -INFINITY;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) { mx = fmaxf(mx, x[r][j]); my = fmaxf(my, y[r][j]); }
        mx = wave_max_f32(mx);
        my = wave_max_f32(my);
        const float rx = mx > -INFINITY ? mx : 0.f, ry = my > -INFINITY ? my : 0.f;   // (nothing but -inf: a sum of 0)
        double lx = 0.0, ly = 0.0;
        if (a.inv_t == 1.0 && a.inv_td == 1.0) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    lx += (double)exp_rel_f32(x[r][j], rx, 1.f);
                    ly += (double)exp_rel_f32(y[r][j], ry, 1.f);
                }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    lx += exp_rel(x[r][j], rx, a.inv_t);
                    ly += exp_rel(y[r][j], ry, a.inv_td);
                }
        }
        lx = wave_sum_f64(lx);
        ly = wave_sum_f64(ly);
        if (lane == 0) { s.wm[buf][0][w] = mx; s.wl[buf][0][w] = lx; s.wm[buf][1][w] = my; s.wl[buf][1][w] = ly; }
    };
    auto lane_mass = [&](const float (&u)[R][4]) {
        double t = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) t += ((double)u[r][0] + (double)u[r][1]) + ((double)u[r][2] + (double)u[r][3]);
        return t;
    };
    auto put_mass = [&](double t) {
        t = wave_sum_f64(t);
        if (lane == 0) s.wsum[w] = t;
    };
    // logits -> probabilities, given the row's maximum and 1 / sum
    auto to_probs = [&](float (&x)[R][4], float m, float inv, float inv_l) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[r][j] = exp_rel_f32(x[r][j], m, inv) * inv_l;
    };
    // Eq. 2: u <- max(0, u - W q)
    auto subtract = [&](float (&u)[R][4], const float (&q)[R][4], float W) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) u[r][j] = fmaxf(0.f, fmaf(-W, q[r][j], u[r][j]));
    };
    // the same over a slice of several laps: each lap's sum is brought to the maximum so far
    auto long_stats = [&](const float *row, double inv, int which) {
        float m = -INFINITY;
        double l = 0.0;
        for (int lap = 0; lap < laps; ++lap) {
            float y[R][4];
            load_row(row, y, lap);
            settle(y, lap);
            double l1;
            const float m1 = lane_stats(y, inv, &l1);
            if (m1 > m) {                                 // (the same in every lane of the wavefront)
                l = (m > -INFINITY ? l * exp(((double)m - (double)m1) * inv) : 0.0) + l1;
                m = m1;
            } else if (m1 > -INFINITY) {
                l += m1 == m ? l1 : l1 * exp(((double)m1 - (double)m) * inv);
            }
        }
        put_stats(m, l, which, at);
    };
    float *ub = a.ubuf + (size_t)b * a.V;                 // long slices: the residual; a lane reads back what it wrote
    auto store_residual = [&](const float (&u)[R][4], int lap) {
        // written through: should the sequence be redone on another die, no older copy may be written back over it
        const int at = first_token(lap);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i0 = at + r * kAqStream * 4;
            if (VEC4) {
                if (i0 < a.V) {
#pragma unroll
                    for (int j = 0; j < 4; j += 2)
                        store_shared_result(reinterpret_cast<uint64_t *>(ub + i0 + j),
                                            (uint64_t)__float_as_uint(u[r][j]) | (uint64_t)__float_as_uint(u[r][j + 1]) << 32);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (i0 + j < a.V) store_shared_result(&ub[i0 + j], u[r][j]);
            }
        }
    };

    // ---- streaming wavefronts' state
    float x[R][4], q[R][4];                               // target row (logits; after a rejection the residual), draft row
    bool q_ready = false;                                 // q holds probabilities (else logits)
    auto look_ahead = [&](int node, int depth) -> uint64_t {
        const uint64_t k = kids_of(node, depth);
        if constexpr (kAhead) {
            if (depth > 0) load_row(target + (size_t)node * a.V, nx);
            if (k != 0) load_row(draft + (size_t)qrow_of(first_of(k)) * a.V, nq);
        }
        if (w == 0 && ((k >> lane) & 1)) {
            ngx = target[(size_t)node * a.V + tok];
            ngq = draft[(size_t)qrow * a.V + tok];
        }
        return k;
    };
    auto put_logits = [&](int buf) { if (w == 0) { s.gx[buf][lane] = ngx; s.gq[buf][lane] = ngq; } };
    // Statistics of the rows that were requested one node ahead, taken while the control wavefront meets the others about
    // the node at hand: if the child is accepted its meeting begins at once (k: its children).
    auto stage = [&](uint64_t k, int buf) {
        if constexpr (kAhead) {
            settle(nx);
            if (k != 0) {
                settle(nq);
                both_stats(nx, nq, buf);
            } else {
                wave_stats(nx, a.inv_t, 0, buf);
            }
            put_logits(buf);
        }
    };
    unsigned int meetings = 0;                            // so far
    // the residual at the tokens of the children still to be tried: the lanes that hold them publish it
    auto publish = [&](const float (&u)[R][4], uint64_t kids, int lap) {
        for (uint64_t m = kids; m != 0; m &= m - 1) {
            const int c2 = first_of(m);
            const int off = (int)readlane_u32((uint32_t)tok, c2) - (lo + lap * lap_tokens);
            if (off >= 0 && off < lap_tokens && ((off >> 2) & (kAqStream - 1)) == tid) {
                const int r2 = off / (kAqStream * 4), j2 = off & 3;      // float4 index, element
                float val = 0.f;
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (r == r2 && j == j2) val = u[r][j];
                store_shared_result(&sibs[(meetings & 1) * kWave + c2], word_of_f32(val, meetings % 255 + 1));
            }
        }
    };
    // ---- the control wavefront's state (the same in all of its lanes unless said otherwise)
    double W = 1.0, pl = 1.0, ql = 1.0, px = 0.0, qx = 0.0, psum = 0.0;      // px, qx: lane = node; psum: lane = workgroup
    float pm = 0.f, qm = 0.f;

    // Maximum and sum of exponentials over the eight wavefronts (lanes 0-7 the target row's, 32-39 the draft
    // row's), then over the workgroups (lane, lane - 32 = workgroup).  m: -inf where a lane has none.
    // at_max(Mp, Mq) runs once the maxima are known, beside the sums.
    auto half_merge = [&](float m, double l, double inv, auto &&at_max, float *mo, double *lo_) {
        float M = m;
        M = fmaxf(M, dpp_f32<0xB1>(M));
        M = fmaxf(M, dpp_f32<0x4E>(M));
        M = fmaxf(M, dpp_f32<0x141>(M));
        M = fmaxf(M, dpp_f32<0x140>(M));                  // every lane: the maximum of its 16-lane row
        const float Mp = fmaxf(readlane_f32(M, 0), readlane_f32(M, 16)), Mq = fmaxf(readlane_f32(M, 32), readlane_f32(M, 48));
        M = lane < 32 ? Mp : Mq;
        at_max(Mp, Mq);
        double t = m > -INFINITY ? l * exp(((double)m - (double)M) * inv) : 0.0;
        auto add = [](double v, uint64_t moved) { return v + __longlong_as_double((long long)moved); };
        t = add(t, dpp_u64<0xB1>((uint64_t)__double_as_longlong(t)));
        t = add(t, dpp_u64<0x4E>((uint64_t)__double_as_longlong(t)));
        t = add(t, dpp_u64<0x141>((uint64_t)__double_as_longlong(t)));
        t = add(t, dpp_u64<0x140>((uint64_t)__double_as_longlong(t)));
        const double Lp = readlane_f64(t, 0) + readlane_f64(t, 16), Lq = readlane_f64(t, 32) + readlane_f64(t, 48);
        *mo = M;
        *lo_ = lane < 32 ? Lp : Lq;
    };
    const double inv_half = lane < 32 ? a.inv_t : a.inv_td;
    // One meeting.  with_p / with_q: statistics of a target / draft row are exchanged; with_u: residual masses;
    // rest: children whose tokens' residuals their owners publish.  false: somebody gave up.
    auto meet = [&](bool with_p, bool with_q, bool with_u, uint64_t rest) -> bool {
        const unsigned int set = meetings & 1, tag = meetings % 255 + 1;
        uint64_t *mine = words + ((size_t)set * kCoG + g) * kCoWords;
        if (with_p || with_q) {
            const int which = lane >> 5, i = lane & 31;
            const bool has = i < kAqWaves && (which ? with_q : with_p);
            const float m0 = s.wm[at][which][i & (kAqWaves - 1)];
            const double l0 = s.wl[at][which][i & (kAqWaves - 1)];
            float m;
            double l;
            half_merge(has ? m0 : -INFINITY, has ? l0 : 0.0, inv_half, [](float, float) {}, &m, &l);
            if (i == 0 && (which ? with_q : with_p)) {
                store_shared_result(&mine[2 * which], word_of_f64(l, tag));
                store_shared_result(&mine[2 * which + 1], word_of_rest(l, m, tag));
            }
        }
        if (with_u) {
            double t = 0.0;
#pragma unroll
            for (int i = 0; i < kAqWaves; ++i) t += s.wsum[i];
            if (lane == 0) {
                store_shared_result(&mine[0], word_of_f64(t, tag));
                store_shared_result(&mine[1], word_of_rest(t, 0.f, tag));
            }
        }
        const float gx = s.gx[at][lane], gq = s.gq[at][lane];
        int from = lane & 31;
        const int which = lane >> 5;
        asm volatile("" : "+v"(from));                    // addresses made here and not kept through the walk
        const uint64_t *theirs = words + ((size_t)set * kCoG + min(from, G - 1)) * kCoWords + 2 * which;
        const bool has_theirs = from < G && (which ? with_q : (with_p || with_u));
        const bool sib = (rest >> lane) & 1;
        struct Poll { uint64_t a0, a1, as; unsigned int given_up; };
        auto look = [&](Poll &p) {
            p.a0 = load_shared_result(&theirs[0]);
            p.a1 = load_shared_result(&theirs[1]);
            p.as = load_shared_result(&sibs[set * kWave + lane]);
            p.given_up = load_shared_result(&ctl[16]);
        };
        auto there = [&](const Poll &p) {
            const bool ok = (!has_theirs || ((p.a0 & 0xff) == tag && (p.a1 & 0xff) == tag)) && (!sib || (p.as & 0xff) == tag);
            return __ballot(!ok) == 0;
        };
        Poll p;
        for (unsigned int spins = 0;;) {
            look(p);
            if (there(p)) break;
            if (++spins > a.co_spin_limit || p.given_up != 0u) {
                if (lane == 0) store_shared_result(&ctl[16], 1u);
                return false;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        const uint64_t a0 = p.a0, a1 = p.a1, as = p.as;
        if (with_p || with_q) {
            float m;
            double l;
            const bool row = from < G && (which ? with_q : with_p);
            double ex = 0.0, eq = 0.0;                    // this child's numerators
            half_merge(row ? f32_of_word(a1) : -INFINITY, row ? f64_of_words(a0, a1) : 0.0, inv_half, [&](float Mp, float Mq) {
                ex = exp_rel(gx, Mp, a.inv_t);
                eq = exp_rel(gq, Mq, a.inv_td);
            }, &m, &l);
            if (with_p) { pm = readlane_f32(m, 0); pl = readlane_f64(l, 0); px = ex * (1.0 / pl); }
            if (with_q) { qm = readlane_f32(m, 32); ql = readlane_f64(l, 32); qx = eq / ql; }
        }
        if (with_u) {
            psum = lane < G ? f64_of_words(a0, a1) : 0.0;
            W = wave_sum_f64(psum);
        }
        if (sib) px = (double)f32_of_word(as);
        return true;
    };
    // Eq. 1 for the next child (px, qx: used at the child's lane).  What a meeting about rows has changed is passed on
    // to the streaming wavefronts.
    auto decide = [&](uint64_t kids, bool was_rejected, bool new_p, bool new_q) {
        int cmd = was_rejected && W > 0.0 ? kCoBonusU : kCoBonusP, arg = -1;
        if (kids != 0 && W > 0.0) {
            arg = first_of(kids);
            const uint64_t yes = __ballot((double)uni * W * qx < px);
            cmd = (yes >> arg) & 1 ? kCoAccept : kCoReject;
        }
        if (lane == 0) {
            s.order[meetings & 1] = (uint64_t)(uint32_t)arg << 32 | (uint32_t)cmd;
            s.W = (float)W;
            if (new_p) { s.pm = pm; s.pinv_l = (float)(1.0 / pl); }
            if (new_q) { s.qm = qm; s.qinv_l = (float)(1.0 / ql); }
        }
    };
    auto give_up = [&]() { if (lane == 0) { s.order[meetings & 1] = kCoAbort; s.gave_up = 1; } };
    int cur = 0, len = 0, cmd = kCoAbort, arg = 0;
    // The decision of the last meeting, after the barrier that follows it.  What a decision leaves in LDS beside this is read before
    // a barrier that the control wavefront passes before its next decision, but nothing holds that one back after an acceptance.
    auto read_order = [&]() {
        const uint64_t o = s.order[(meetings - 1) & 1];
        cmd = uniform_of((int)(uint32_t)o);
        arg = uniform_of((int)(uint32_t)(o >> 32));
    };

    // The control wavefront and the streaming ones run loops of their own with the same barriers, command by
    // command: the registers of a row and the state of the tests are never held by the same code.  (In one loop, with
    // a row's addresses and end-of-row masks kept through the walk as well, eight float4 per lane spilled 69 registers,
    // 154 without 16-byte loads: 24 sequences of V = 128256 70 us and now 54, 20 of 128257 110 and 72.)
    bool rejected = false;
    if (tid == 0) s.gave_up = 0;
    if (control) {
        for (;;) {                                        // one iteration per visited node
            uint64_t kids = kids_of(cur, len);
            rejected = false;
            if (!kAhead || len == 0) __syncthreads();
            if (meet(true, kids != 0, false, 0)) {
                W = 1.0;
                decide(kids, false, true, kids != 0);
            } else {
                give_up();
            }
            ++meetings;
            __syncthreads();
            for (read_order(); cmd == kCoReject; read_order()) {
                kids &= ~(1ull << arg);
                const bool other_q = kids != 0 && qrow_of(first_of(kids)) != qrow_of(arg);
                rejected = true;
                __syncthreads();
                if (meet(false, other_q, true, kids)) decide(kids, true, false, other_q);
                else give_up();
                ++meetings;
                __syncthreads();
            }
            if (cmd != kCoAccept) break;
            cur = arg;
            ++len;
            at ^= 1;
        }
    } else {
        const uint64_t k0 = look_ahead(0, 0);
        stage(k0, 0);
        for (;;) {
            uint64_t kids = kids_of(cur, len);
            rejected = false;
            const float *prow = target + (size_t)cur * a.V;
            if constexpr (kAhead) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int j = 0; j < 4; ++j) { x[r][j] = nx[r][j]; q[r][j] = nq[r][j]; }
                q_ready = false;
                if (len == 0) __syncthreads();
            } else {
                put_logits(at);
                if constexpr (LAPS) {
                    long_stats(prow, a.inv_t, 0);
                    if (kids != 0) long_stats(draft + (size_t)qrow_of(first_of(kids)) * a.V, a.inv_td, 1);
                } else {
                    load_row(prow, x);
                    if (kids != 0) load_row(draft + (size_t)qrow_of(first_of(kids)) * a.V, q);
                    q_ready = false;
                    settle(x);
                    if (kids != 0) {
                        settle(q);
                        both_stats(x, q, at);
                    } else {
                        wave_stats(x, a.inv_t, 0, at);
                    }
                }
                __syncthreads();
            }
            if (kids != 0) stage(look_ahead(first_of(kids), len + 1), at ^ 1);
            ++meetings;
            __syncthreads();
            for (read_order(); cmd == kCoReject; read_order()) {
                // Eq. 2, then the next child (whose draft row may be another one)
                const int c = arg;
                kids &= ~(1ull << c);
                const int next = kids != 0 ? first_of(kids) : -1;
                const bool other_q = next >= 0 && qrow_of(next) != qrow_of(c);
                const float m_p = s.pm, il_p = s.pinv_l, m_q = s.qm, il_q = s.qinv_l, W_f = s.W;
                if constexpr (LAPS) {
                    double mass = 0.0;
                    for (int lap = 0; lap < laps; ++lap) {
                        load_row(rejected ? ub : prow, x, lap);
                        load_row(draft + (size_t)qrow_of(c) * a.V, q, lap);
                        settle(x, lap, rejected ? 0.f : -INFINITY);
                        settle(q, lap);
                        if (!rejected) to_probs(x, m_p, it_f, il_p);
                        to_probs(q, m_q, itd_f, il_q);
                        subtract(x, q, W_f);
                        store_residual(x, lap);
                        publish(x, kids, lap);
                        mass += lane_mass(x);
                    }
                    put_mass(mass);
                    if (other_q) long_stats(draft + (size_t)qrow_of(next) * a.V, a.inv_td, 1);
                } else {
                    if (!q_ready) to_probs(q, m_q, itd_f, il_q);
                    if (!rejected) to_probs(x, m_p, it_f, il_p);
                    subtract(x, q, W_f);
                    q_ready = !other_q;
                    if (other_q) load_row(draft + (size_t)qrow_of(next) * a.V, q);
                    publish(x, kids, 0);
                    put_mass(lane_mass(x));
                    if (other_q) { settle(q); wave_stats(q, a.inv_td, 1, at); }
                }
                rejected = true;
                __syncthreads();
                if (next >= 0) stage(look_ahead(next, len + 1), at ^ 1);
                ++meetings;
                __syncthreads();
            }
            if (cmd != kCoAccept) break;
            cur = arg;
            ++len;
            at ^= 1;
            if (g == 0 && tid == 0) store_shared_result(&path[len], cur);
        }
    }

    // ---- bonus token, from the residual, or from p where nothing was rejected or the residual vanished
    auto probs_of = [&](int lap) {                        // x: the current node's probabilities
        load_row(target + (size_t)cur * a.V, x, lap);
        settle(x, lap);
        to_probs(x, s.pm, it_f, s.pinv_l);
    };
    if (cmd == kCoBonusP) {
        if (!control) {
            double mass = 0.0;
            if constexpr (LAPS) {
                for (int lap = 0; lap < laps; ++lap) { probs_of(lap); mass += lane_mass(x); }
            } else {
                if (rejected) probs_of(0);                // the residual vanished
                else to_probs(x, s.pm, it_f, s.pinv_l);
                mass = lane_mass(x);
            }
            put_mass(mass);
        }
        __syncthreads();
        if (control && !meet(false, false, true, 0)) give_up();
    }
    if (cmd != kCoAbort) {
        if (control) {
            const double goal = (double)uni_bonus * W, incl = wave_scan_f64(psum);
            const uint64_t over = __ballot(lane < G && incl > goal), mass = __ballot(psum > 0.0);
            const int owner = over ? first_of(over) : mass ? 63 - __clzll((long long)mass) : -1;
            if (lane == 0) {
                s.owner = owner; s.take_last = over == 0; s.goal = goal;
                s.pick = 0x7fffffff;
                if (g == 0) store_shared_result(&a.accept_len[b], len);
                if (g == 0 && owner < 0) store_shared_result(&a.bonus[b], -1);
            }
            const double before = incl - psum;
            if (lane == max(owner, 0)) s.before = before;
        }
        __syncthreads();
        if (s.gave_up == 0 && g == s.owner) {
            // token order inside the slice: lap, float4 row r, then thread, then element
            double run = s.before;
            int lastp = -1;
            for (int lap = 0; lap < laps; ++lap) {
                double linc[R], lsum[R];
                double (&wtot)[kCoR][kAqWaves] = s.wtot[lap & 1];
                if (!control) {
                    if (LAPS) {
                        if (cmd == kCoBonusP) probs_of(lap);
                        else { load_row(ub, x, lap); settle(x, lap, 0.f); }
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        lsum[r] = ((double)x[r][0] + (double)x[r][1]) + ((double)x[r][2] + (double)x[r][3]);
                        linc[r] = wave_scan_f64(lsum[r]);
                        if (lane == kWave - 1) wtot[r][w] = linc[r];
                    }
                }
                __syncthreads();
                if (!control) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        double wbefore = run;
#pragma unroll
                        for (int i = 0; i < kAqWaves; ++i) {
                            if (i < w) wbefore += wtot[r][i];
                            run += wtot[r][i];
                        }
                        const int i0 = lo + lap * lap_tokens + (r * kAqStream + tid) * 4;
                        double acc = wbefore + linc[r] - lsum[r];
                        int pick = -1;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            if (x[r][j] > 0.f) lastp = i0 + j;
                            acc += (double)x[r][j];
                            if (pick < 0 && acc > s.goal) pick = i0 + j;
                        }
                        if (pick >= 0 && !s.take_last) atomicMin(&s.pick, pick);
                    }
                }
            }
            if (!control) {
                lastp = (int)wave_max_u32((uint32_t)(lastp + 1)) - 1;
                if (lane == 0) s.wlast[w] = lastp;
            }
            __syncthreads();
            if (tid == 0) {
                int lp = -1;
#pragma unroll
                for (int i = 0; i < kAqWaves; ++i) lp = max(lp, s.wlast[i]);
                store_shared_result(&a.bonus[b], s.pick != 0x7fffffff ? s.pick : lp);
            }
        }
    }

    // ---- leave: every workgroup of the sequence ends here.  The last one clears what the next call's
    // meetings start from, and redoes the sequence if anybody gave up on the way (all their stores are
    // complete by then).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        const unsigned int before = __hip_atomic_fetch_add(&ctl[8], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s.last = before == (unsigned int)(G - 1);
        s.redo = s.last ? (int)load_shared_result(&ctl[16]) : 0;
    }
    __syncthreads();
    if (!s.last) return;
    const bool redo = s.redo != 0;
    for (int i = tid; i < 2 * kCoG * kCoWords; i += kAqThreads) store_shared_result(&words[i], (uint64_t)0);
    for (int i = tid; i < 2 * kWave; i += kAqThreads) store_shared_result(&sibs[i], (uint64_t)0);
    if (tid == 0) {
        store_shared_result(&ctl[8], 0u);
        store_shared_result(&ctl[16], 0u);
    }
    if (!redo) return;
    __syncthreads();
    walk_single<VEC4, kAqThreads, false>(a, lds.alone, b);
}

}  // namespace radar

using namespace radar;

// How many workgroups of the shared walk the current device can hold at once: the
// occupancy the runtime reports for the kernel times the number of CUs (queried once; 0 if the
// queries fail, which selects the single-workgroup walk).
static int aq_resident_capacity() {
    static const int capacity = [] {
        int dev = 0, per_cu = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(&accept_q_coop_kernel<true, kCoR, false>),
                                                         kAqThreads, 0) != hipSuccess)
            return 0;
        return per_cu * prop.multiProcessorCount;
    }();
    return capacity;
}

// Workgroups per sequence (G), float4 per lane (R) and laps of the walk; G = 1 means the single-workgroup
// walk.  The G * B workgroups of the shared walk meet after every row, which only makes progress
// while all of them are resident, so their number stays within what the device holds at once (on a
// GPU that other work shares, the bounded wait turns a missing workgroup into the fall-back).
// Slices that fit eight float4 per lane stay in registers, longer ones are walked over in laps: a sequence left to
// one workgroup gets 64 KB/us (one sequence of V = 1048576: 3013 us alone, 124 in laps; 40 of V = 128256: 399 and 126).
static void aq_coop_plan(const radar_accept_q_desc *d, int *G, int *R, int *laps) {
    *G = 1; *R = 1; *laps = 1;
    const int cap = aq_resident_capacity();
    if (d->walk_spin_limit < 0 || cap < 2 || d->B > cap / 2) return;
    const int gcap = cap / d->B < kCoG ? cap / d->B : kCoG;
    const int per_wg = kAqStream * 4;
    const int need = ((d->V + per_wg - 1) / per_wg + gcap - 1) / gcap;     // float4 per lane needed with gcap workgroups
    int r = 1, n = 1;
    if (need > kCoR) { r = kCoLapR; n = (need + r - 1) / r; }
    else while (r < need) r *= 2;                                         // compiled for 1, 2, 4 and 8
    const int g = (d->V + per_wg * r * n - 1) / (per_wg * r * n);
    if (g < 2) return;                                                    // one workgroup would cover it anyway
    *G = g; *R = r; *laps = n;
}

// Whether a lone walk's rows have their statistics taken beforehand.  Inside the walk a row costs its workgroup two
// passes at 64 KB/us, however many sequences walk beside it; beforehand every row of the call costs the chip one pass,
// and a launch.  Measured (us, inside / beforehand): one sequence, 122 rows, V = 8192 12.3 / 14.9, 16000 21.9 / 20.5,
// 32000 23.5 / 15.8, 128256 184 / 146, 1048576 1022 / 714; 488 rows of 128256 217 / 200, 732 264 / 289, 1464 261 / 338;
// 976 rows of 32000, which the memory-side cache holds, 126 / 105, of 128256 270 / 304; 2240 of 32000 76 / 89.
static bool aq_take_statistics(const radar_accept_q_desc *d) {
    const int64_t rows = (int64_t)d->B * ((int64_t)d->T_max + d->Tq);
    return d->V >= 12288 && (rows <= 600 || (rows <= 1000 && rows * d->V <= (int64_t(1) << 26)));
}

static int aq_chunks(const radar_accept_q_desc *d) { return (d->V + kAqChunk - 1) / kAqChunk; }

extern "C" size_t radar_verify_accept_q_workspace_bytes(const radar_accept_q_desc *d) {
    if (!d || d->B < 1 || d->T_max < 1 || d->Tq < 1 || d->V < 1) return 0;
    size_t bytes = ((size_t)d->B * d->V * sizeof(float) + 255) & ~size_t(255);
    bytes += ((size_t)d->B * kCoCtl * sizeof(unsigned int) + 255) & ~size_t(255);
    bytes += ((size_t)d->B * 2 * kCoG * kCoWords * sizeof(uint64_t) + 255) & ~size_t(255);
    bytes += ((size_t)d->B * 2 * kWave * sizeof(uint64_t) + 255) & ~size_t(255);
    if (aq_take_statistics(d)) {
        const size_t parts = (size_t)d->B * ((size_t)d->T_max + d->Tq) * aq_chunks(d);
        bytes += (parts * sizeof(float) + 255) & ~size_t(255);
        bytes += (parts * sizeof(double) + 255) & ~size_t(255);
    }
    return bytes;
}

extern "C" radar_status radar_verify_accept_q(const float *target_logits, const float *draft_logits, const int32_t *q_rows,
                                              const int32_t *draft_tokens, const int32_t *parents, const int32_t *n_nodes,
                                              const float *uniforms, int32_t *accept_len, int32_t *accept_path,
                                              int32_t *bonus_token, const radar_accept_q_desc *d, void *workspace,
                                              size_t workspace_bytes, void *stream) {
    if (!d || !target_logits || !draft_logits || !draft_tokens || !parents || !uniforms || !accept_len || !accept_path ||
        !bonus_token || !workspace)
        return RADAR_INVALID_ARG;
    if (d->B < 1 || d->T_max < 1 || d->Tq < 1 || d->V < 1 || d->D_max < 0 || !(d->temperature > 0.f) ||
        !(d->draft_temperature > 0.f))
        return RADAR_INVALID_ARG;
    if (!q_rows && d->Tq != d->T_max) return RADAR_INVALID_ARG;
    if (d->T_max > RADAR_T_MAX || d->D_max >= RADAR_T_MAX || d->V > kAqMaxV) return RADAR_UNSUPPORTED_SHAPE;
    if ((int64_t)d->B * ((int64_t)d->T_max + d->Tq) > 65535) return RADAR_UNSUPPORTED_SHAPE;
    if (workspace_bytes < radar_verify_accept_q_workspace_bytes(d)) return RADAR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)workspace & 255) != 0) return RADAR_INVALID_ARG;

    AqArgs a{};
    a.target = target_logits; a.draft = draft_logits; a.q_rows = q_rows;
    a.tokens = draft_tokens; a.parents = parents; a.n_nodes = n_nodes; a.uniforms = uniforms;
    a.accept_len = accept_len; a.accept_path = accept_path; a.bonus = bonus_token;
    a.B = d->B; a.T = d->T_max; a.Tq = d->Tq; a.V = d->V; a.D_max = d->D_max;
    a.inv_t = 1.0 / (double)d->temperature; a.inv_td = 1.0 / (double)d->draft_temperature;
    char *ws = static_cast<char *>(workspace);
    auto take = [&](size_t bytes) { char *p = ws; ws += (bytes + 255) & ~size_t(255); return p; };
    a.co_ctl = reinterpret_cast<unsigned int *>(take((size_t)d->B * kCoCtl * sizeof(unsigned int)));
    a.co_words = reinterpret_cast<uint64_t *>(take((size_t)d->B * 2 * kCoG * kCoWords * sizeof(uint64_t)));
    a.co_sib = reinterpret_cast<uint64_t *>(take((size_t)d->B * 2 * kWave * sizeof(uint64_t)));
    a.ubuf = reinterpret_cast<float *>(take((size_t)d->B * d->V * sizeof(float)));
    int G = 1, R = 1;
    aq_coop_plan(d, &G, &R, &a.co_laps);
    // default: 256 polls of about 0.5 us (an atomic load and a short sleep): the workgroups of a walk reach a
    // meeting within microseconds of each other, so 100 us without progress means one of them is not running;
    // a lap more takes them some 3 us more
    a.co_spin_limit = d->walk_spin_limit > 0 ? (unsigned int)d->walk_spin_limit : 256u + 16u * (unsigned int)(a.co_laps - 1);

    const bool vec4 = (d->V % 4 == 0) && (((uintptr_t)target_logits & 15) == 0) && (((uintptr_t)draft_logits & 15) == 0);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((unsigned)G, (unsigned)d->B), block(kAqThreads);
    hipError_t e;
    if (G == 1) {
        const bool parts = aq_take_statistics(d);
        if (parts) {
            const size_t rows = (size_t)d->B * ((size_t)d->T_max + d->Tq);
            a.nchunks = aq_chunks(d);
            a.part_m = reinterpret_cast<float *>(take(rows * a.nchunks * sizeof(float)));
            a.part_l = reinterpret_cast<double *>(take(rows * a.nchunks * sizeof(double)));
            const dim3 all((unsigned)a.nchunks, (unsigned)rows);
            e = vec4 ? launch("accept_q_stats", accept_q_stats_kernel<true>, all, dim3(kAqStream), 0, st, a)
                     : launch("accept_q_stats", accept_q_stats_kernel<false>, all, dim3(kAqStream), 0, st, a);
            if (e != hipSuccess) return RADAR_HIP_ERROR;
        }
        auto go = [&](auto has) {
            constexpr bool P = decltype(has)::value;
            return vec4 ? launch("accept_q_walk", accept_q_walk_kernel<true, P>, dim3((unsigned)d->B), dim3(kAqLone), 0, st, a)
                        : launch("accept_q_walk", accept_q_walk_kernel<false, P>, dim3((unsigned)d->B), dim3(kAqLone), 0, st, a);
        };
        e = parts ? go(std::true_type{}) : go(std::false_type{});
    } else {
        auto go = [&](auto r, auto laps) {
            constexpr int RR = decltype(r)::value;
            constexpr bool LL = decltype(laps)::value;
            return vec4 ? launch("accept_q_walk_shared", accept_q_coop_kernel<true, RR, LL>, grid, block, 0, st, a.parents, a.tokens, a.q_rows,
                                 a.n_nodes, a.target, a.T, a.V, a.D_max, a)
                        : launch("accept_q_walk_shared", accept_q_coop_kernel<false, RR, LL>, grid, block, 0, st, a.parents, a.tokens, a.q_rows,
                                 a.n_nodes, a.target, a.T, a.V, a.D_max, a);
        };
        using std::integral_constant;
        using std::false_type;
        e = a.co_laps > 1 ? go(integral_constant<int, kCoLapR>{}, std::true_type{})
          : R == 1 ? go(integral_constant<int, 1>{}, false_type{}) : R == 2 ? go(integral_constant<int, 2>{}, false_type{})
          : R == 4 ? go(integral_constant<int, 4>{}, false_type{}) : go(integral_constant<int, 8>{}, false_type{});
    }
    return e == hipSuccess ? RADAR_OK : RADAR_HIP_ERROR;
}
