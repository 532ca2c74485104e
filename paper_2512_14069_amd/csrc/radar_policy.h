// One call of RADAR's prediction model (Sec. 4.2; architecture per App. A.3) as a
// workgroup-wide device routine: LSTM cell over the k frontier confidences, the new
// hidden vector joined with those inputs, two-layer perceptron, softmax over
// {0 = stop, 1 = continue}.
//
// The routine is written for one workgroup of 1024 threads (16 wavefronts) per state and
// is used twice: by the stand-alone kernel behind radar_policy_step and as the tail of the
// expansion kernel's last workgroup, where the confidences are still in LDS.
//
// The work is 4H x (H + k) + M x (H + k) multiply-adds on fp32 weights that sit in L2
// between calls (about 350 KB at H = M = 128, k = 10): a chain of latencies.  So every operand is
// asked for before the inputs exist and waits in registers (policy_fetch_*), and what follows the
// inputs is laid out for few and short steps: the gates of a unit sit in one quad of lanes and a
// head row's 138 products in eight lanes, so that both meet by DPP moves of a few cycles (lane
// shuffles through LDS cost 130 each; sixteen in a row were a microsecond).  Fused into the
// expansion at V = 128256, k = 10: inputs to action 4.2 us before, 1.6 us so.
#pragma once

#include "radar_device.h"

namespace radar {

constexpr int kPolThreads = 1024;
constexpr int kPolWaves = kPolThreads / kWave;       // 16
constexpr int kPolH = 128;                           // LSTM hidden size (App. A.3)
constexpr int kPolMMax = 128;                        // largest hidden size of the head
constexpr int kPolHeadLanes = 8;                     // lanes that share a row of the head
// Columns each of them takes: 4 l .. 4 l + 3 of every 32 of h', then l and l + 8 of x.
constexpr int kPolHeadQuads = kPolH / (4 * kPolHeadLanes), kPolHeadTail = RADAR_K_MAX / kPolHeadLanes;
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));     // rows of any length: 16-byte loads from 4-byte addresses
static_assert(kPolMMax * kPolHeadLanes == kPolThreads && 4 * kPolH * 2 == kPolThreads, "one thread per share of a head row, half of them one gate each");

struct PolicyArgs {
    const float *w_ih, *w_hh, *b_ih, *b_hh, *w1, *b1, *w2, *b2;
    const float *h_in, *c_in;       // [B][H] or null = zero state
    const float *uniforms;          // [B] or null = argmax action
    float *h_out, *c_out;           // [B][H]
    float *logits, *probs;          // [B][2]
    int32_t *action;                // [B]
    int k, M;
};

struct alignas(16) PolicySmem {
    float in[kPolH + RADAR_K_MAX];  // [h'; x]: the new hidden vector, the k confidences, zeros
    float z[kPolMMax];
    float gate[4 * kPolH];          // w_hh h (stand-alone kernel; the fused path keeps it in global memory)
};

// What a thread holds of the model: half of the threads one gate row (four gates of a unit in a quad of
// lanes), all of them an eighth of a head row, the last wavefront the last layer.
struct PolicyRegs {
    float4u wih[RADAR_K_MAX / 4];
    float b_ih, b_hh, c_prev, hid;
    float4u w1[kPolHeadQuads];
    float w1x[kPolHeadTail], b1;
    float w2[2][2], b2[2], uni;
};

// The value of lane ^ OFF, by DPP moves (through LDS it takes 130 cycles; 8, 4, 2 or 1 stay inside a row of 16 lanes).
template <int OFF>
__device__ __forceinline__ float lane_xor(float v) {
    static_assert(OFF == 8 || OFF == 4 || OFF == 2 || OFF == 1, "inside a row");
    if constexpr (OFF == 8) return dpp_f32<0x128>(v);                // row_ror:8
    if constexpr (OFF == 2) return dpp_f32<0x4E>(v);
    if constexpr (OFF == 1) return dpp_f32<0xB1>(v);
    const int from_above = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x104, 0xF, 0x5, false);           // row_shl:4 into lanes 0-3 and 8-11
    return __int_as_float(__builtin_amdgcn_update_dpp(from_above, __float_as_int(v), 0x114, 0xF, 0xA, false));  // row_shr:4 into the others
}

// v[0..N) per lane -> sums over groups of lanes.  One step with lane distance OFF halves the
// number of values a lane carries: lanes whose bit OFF is set keep the upper half.
template <int N, int OFF>
__device__ __forceinline__ void fold_step(float *v, int lane) {
    const bool up = (lane & OFF) != 0;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        if constexpr (OFF == 16) {                                   // rows 0 and 2 keep v[i], rows 1 and 3 the other
            const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + N / 2]), false, false);
            v[i] = __uint_as_float(a[0]) + __uint_as_float(a[1]);
        } else {
            const float send = up ? v[i] : v[i + N / 2];
            const float keep = up ? v[i + N / 2] : v[i];
            v[i] = keep + lane_xor<OFF>(send);
        }
    }
}

// Logistic function and tanh from the hardware exponential and reciprocal (a few 1e-7 of
// absolute error; both saturate cleanly for large arguments of either sign).
__device__ __forceinline__ float fast_sigmoid(float a) { return __frcp_rn(1.f + __expf(-a)); }
__device__ __forceinline__ float fast_tanh(float a) { return 1.f - 2.f * __frcp_rn(1.f + __expf(2.f * a)); }

// The part of the gate pre-activations that needs no input: rows of w_hh times h_in.  A row is
// 128 floats = one 32-lane half-wavefront x 16 bytes.  The calling workgroup is part `part` of
// `parts` that share the 4H rows; its HW half-wavefronts that take part (number hwave) take rows
// (part + parts * i) * HW + hwave for i = 0, 1, ... in batches of NR (2, 4 or 16) rows per lane.  load()
// asks for the first batch; finish() folds it and goes through what is left, all loads of a batch
// issued before its sums are folded.  store(row, value) is called by one lane per row.
template <int NR, int HW>
struct HiddenRows {
    static_assert(NR == 2 || NR == 4 || NR == 16, "NR");
    static constexpr int rows = 4 * kPolH;
    float4 h4, wv[NR];
    int part, parts, hwave;

    __device__ __forceinline__ void batch(const PolicyArgs &p, int i0) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int row = min((part + parts * (i0 + i)) * HW + hwave, rows - 1);      // clamped: stays a legal read
            wv[i] = *reinterpret_cast<const float4 *>(p.w_hh + (size_t)row * kPolH + 4 * (threadIdx.x % 32));
        }
    }
    __device__ __forceinline__ void load(const PolicyArgs &p, int b, int part_, int parts_, int hwave_) {
        part = part_; parts = parts_; hwave = hwave_;
        if (part * HW >= rows) return;
        h4 = *reinterpret_cast<const float4 *>(p.h_in + (size_t)b * kPolH + 4 * (threadIdx.x % 32));
        batch(p, 0);
    }
    template <typename Store>
    __device__ __forceinline__ void finish(const PolicyArgs &p, int b, Store &&store) {
        const int lane = threadIdx.x % kWave;
        for (int i0 = 0; (part + parts * i0) * HW < rows; i0 += NR) {
            if (i0 > 0) batch(p, i0);
            float v[NR];
#pragma unroll
            for (int i = 0; i < NR; ++i) v[i] = fmaf(wv[i].x, h4.x, fmaf(wv[i].y, h4.y, fmaf(wv[i].z, h4.z, wv[i].w * h4.w)));
            int mine;                                                // which of the NR rows this lane ends up with
            if constexpr (NR == 16) {
                fold_step<16, 16>(v, lane);
                fold_step<8, 8>(v, lane);
                fold_step<4, 4>(v, lane);
                fold_step<2, 2>(v, lane);
                v[0] += lane_xor<1>(v[0]);
                mine = ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
            } else if constexpr (NR == 4) {
                fold_step<4, 16>(v, lane);
                fold_step<2, 8>(v, lane);
                v[0] += lane_xor<4>(v[0]);
                v[0] += lane_xor<2>(v[0]);
                v[0] += lane_xor<1>(v[0]);
                mine = ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
            } else {
                fold_step<2, 16>(v, lane);
                v[0] += lane_xor<8>(v[0]);
                v[0] += lane_xor<4>(v[0]);
                v[0] += lane_xor<2>(v[0]);
                v[0] += lane_xor<1>(v[0]);
                mine = (lane >> 4) & 1;
            }
            const int row = (part + parts * (i0 + mine)) * HW + hwave;
            const bool writer = (lane & (NR == 16 ? 1 : NR == 4 ? 7 : 15)) == 0;
            if (writer && row < rows) store(row, v[0]);
        }
    }
};

// Which of the 4H gate rows a thread of the upper half of the workgroup holds.
__device__ __forceinline__ int policy_gate_row() { return (threadIdx.x & 3) * kPolH + (((int)threadIdx.x - kPolThreads / 2) >> 2); }

// Request what the step for state b will need, the head's rows (policy_fetch_head) and the rest, by the
// kPolThreads threads of one workgroup; nothing waits here.  Every load is from a clamped, valid address, taken or not (rows and columns that do not
// exist are discarded where the values are used); only which kind of load a wavefront makes depends on
// its number.  hidden(row): (w_hh h)[row]; with EARLY a value in global memory, complete before the call,
// otherwise it is read by policy_decide (a value this workgroup wrote to LDS).
__device__ __forceinline__ void policy_fetch_head(const PolicyArgs &p, PolicyRegs &r) {
    const int tid = threadIdx.x, cols = kPolH + p.k, row = min(tid / kPolHeadLanes, p.M - 1);
    const float *src = p.w1 + (size_t)row * cols;
    const int l = tid % kPolHeadLanes;
#pragma unroll
    for (int j = 0; j < kPolHeadQuads; ++j) r.w1[j] = *reinterpret_cast<const float4u *>(src + 4 * (l + kPolHeadLanes * j));
#pragma unroll
    for (int j = 0; j < kPolHeadTail; ++j) r.w1x[j] = src[min(kPolH + l + kPolHeadLanes * j, cols - 1)];
    r.b1 = p.b1[row];
}
template <bool EARLY, typename Hidden>
__device__ __forceinline__ void policy_fetch_rest(const PolicyArgs &p, int b, bool has_state, PolicyRegs &r, Hidden &&hidden) {
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    if (w >= kPolWaves / 2) {
        const int unit = (tid - kPolThreads / 2) >> 2, row = policy_gate_row();
        const float *src = p.w_ih + (size_t)row * p.k;
#pragma unroll
        for (int i4 = 0; i4 < RADAR_K_MAX; i4 += 4) {                // (the conditions are the same in every lane)
            if (i4 + 4 <= p.k) r.wih[i4 / 4] = *reinterpret_cast<const float4u *>(src + i4);
            else if (i4 < p.k) {
#pragma unroll
                for (int i = 0; i < 4; ++i) r.wih[i4 / 4][i] = src[min(i4 + i, p.k - 1)];
            }
        }
        r.b_ih = p.b_ih[row];
        r.b_hh = p.b_hh[row];
        r.c_prev = (has_state ? p.c_in + (size_t)b * kPolH : p.b_ih)[unit];
        if (EARLY) r.hid = hidden(row);
        if (w == kPolWaves - 1) {
            const int l0 = min(lane, p.M - 1), l1 = min(lane + 64, p.M - 1);
            r.w2[0][0] = p.w2[l0]; r.w2[0][1] = p.w2[l1];
            r.w2[1][0] = p.w2[p.M + l0]; r.w2[1][1] = p.w2[p.M + l1];
            r.b2[0] = p.b2[0]; r.b2[1] = p.b2[1];
            r.uni = *(p.uniforms ? p.uniforms + b : p.b2);
        }
    }
}

// The step itself, once the k confidences are in s.in[kPolH ..] (zeros up to RADAR_K_MAX) and a barrier has
// passed since; every thread must call it (it contains barriers).  h_out / c_out may be the arrays
// h_in / c_in.  decided(action) is called by the one lane that has just written the outputs.
template <bool EARLY, typename Hidden, typename Decided>
__device__ __forceinline__ void policy_decide(const PolicyArgs &p, int b, bool has_state, PolicySmem &s, const PolicyRegs &r,
                                              Hidden &&hidden, Decided &&decided) {
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    // ---- cell update: every lane finishes one gate (input part, biases, activation; tanh of the
    // candidate gate as 2 sigm(2a) - 1 so that all lanes run the same code), then the four gates of
    // a unit meet in their quad's first lane
    if (w >= kPolWaves / 2) {
        const int gate = tid & 3, unit = (tid - kPolThreads / 2) >> 2;
        float pre = r.b_ih + r.b_hh;
        if (has_state) pre += EARLY ? r.hid : hidden(gate * kPolH + unit);
#pragma unroll
        for (int i4 = 0; i4 < RADAR_K_MAX; i4 += 4) {
            if (i4 >= p.k) break;
            const float4 in = *reinterpret_cast<const float4 *>(&s.in[kPolH + i4]);
            pre = fmaf(r.wih[i4 / 4].x, in.x, pre);
            if (i4 + 1 < p.k) pre = fmaf(r.wih[i4 / 4].y, in.y, pre);
            if (i4 + 2 < p.k) pre = fmaf(r.wih[i4 / 4].z, in.z, pre);
            if (i4 + 3 < p.k) pre = fmaf(r.wih[i4 / 4].w, in.w, pre);
        }
        const bool cand = gate == 2;
        const float sg = fast_sigmoid(cand ? 2.f * pre : pre);
        const float act = cand ? 2.f * sg - 1.f : sg;
        const float fg = dpp_f32<0x55>(act), gg = dpp_f32<0xAA>(act), og = dpp_f32<0xFF>(act);     // lanes 1, 2, 3 of the quad
        if (gate == 0) {
            const float cn = fmaf(fg, has_state ? r.c_prev : 0.f, act * gg);
            const float hn = og * fast_tanh(cn);
            s.in[unit] = hn;
            p.c_out[(size_t)b * kPolH + unit] = cn;
            p.h_out[(size_t)b * kPolH + unit] = hn;
        }
    }
    __syncthreads();

    // ---- first layer of the head on [h'; x], ReLU: eight lanes per row
    {
        const int cols = kPolH + p.k, l = tid % kPolHeadLanes, row = tid / kPolHeadLanes;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < kPolHeadQuads; ++j) {
            const float4 in = *reinterpret_cast<const float4 *>(&s.in[4 * (l + kPolHeadLanes * j)]);
            v[0] = fmaf(r.w1[j].x, in.x, v[0]); v[1] = fmaf(r.w1[j].y, in.y, v[1]);
            v[2] = fmaf(r.w1[j].z, in.z, v[2]); v[3] = fmaf(r.w1[j].w, in.w, v[3]);
        }
#pragma unroll
        for (int j = 0; j < kPolHeadTail; ++j) {
            const int col = kPolH + l + kPolHeadLanes * j;
            v[j & 3] = fmaf(col < cols ? r.w1x[j] : 0.f, s.in[col], v[j & 3]);
        }
        float sum = (v[0] + v[1]) + (v[2] + v[3]);
        sum += dpp_f32<0xB1>(sum);
        sum += dpp_f32<0x4E>(sum);
        sum += dpp_f32<0x141>(sum);                                  // the other quad of the eight lanes
        if (l == 0 && row < p.M) s.z[row] = fmaxf(sum + r.b1, 0.f);
    }
    __syncthreads();

    // ---- two logits, softmax, action
    if (w == kPolWaves - 1) {
        const float z0 = lane < p.M ? s.z[lane] : 0.f;
        const float z1 = lane + 64 < p.M ? s.z[lane + 64] : 0.f;
        const float l0 = wave_sum_f32(fmaf(r.w2[0][0], z0, r.w2[0][1] * z1)) + r.b2[0];
        const float l1 = wave_sum_f32(fmaf(r.w2[1][0], z0, r.w2[1][1] * z1)) + r.b2[1];
        if (lane == 0) {
            const float p1 = __frcp_rn(1.f + __expf(l0 - l1));
            const float p0 = __frcp_rn(1.f + __expf(l1 - l0));
            p.logits[2 * b] = l0;
            p.logits[2 * b + 1] = l1;
            p.probs[2 * b] = p0;
            p.probs[2 * b + 1] = p1;
            const int act = p.uniforms ? (r.uni < p1 ? 1 : 0) : (l1 > l0 ? 1 : 0);
            p.action[b] = act;
            decided(act);
        }
    }
}

}  // namespace radar
