// Policy updates and inference of fp32 vector networks (Algorithm 1 of the paper, batched).
//
// The networks here are small (layers of at most 512 units), so a pass is not bound by arithmetic but by the
// number of dependent kernels (about 2.4 us each before the first instruction runs) and by memory
// latency inside each of them.  An update is therefore two launches, three on long batches:
//
//   f32_rows    one block per 4 NR transitions: all layers of all forward passes, the TD target (or the
//               clipped objective), and the input gradients back to the first hidden layer.  Activations
//               and gradients of the block's rows live in LDS; only what the weight gradients need (layer inputs
//               of s, output gradients) is written to memory.
//   f32_update  one block per tile of a weight matrix: its gradient over the whole batch, then Adam on the
//               tile, the weight copy the forward pass reads, and the target network where it is due.
//   f32_adam    where update_plan cuts a long batch into slices: their sum, and everything behind it.
//
// f32_rows multiplies with v_mfma_f32_4x4x1_16b_f32: sixteen independent 4 x 4 products per instruction,
// the A operand (4 rows x 1) broadcast to all of them, so one instruction is 4 rows x 64 features x one k at
// the full fp32 matrix rate (136 TFLOP/s measured on the bare instruction).  Rows come in groups of four, not
// 16 or 32: a batch of 512 spreads over 128 blocks without padding.
//
// What bounds the kernel is the stream of weights from the L2 into a CU, each read once per block (41 - 46 bytes per clock where a
// layer is wide), and everything between two layers, which a nearly empty chip cannot hide: with two waves per SIMD an instruction costs
// 5 - 10 clocks, so 150 of them between two layers cost as much as a 64 KB layer.  Hence, in the forward pass:
//   - The weight copy is [k / 4][features][4]: a lane's 16-byte load is four k of one feature, and a wave is given fewer features and more
//     of k side by side (64 / q features, q parts) until eight waves cover the layer.  A wave then ends with whole sums after at most
//     two lane exchanges, writes the activations and meets one barrier; slices of k over the waves, added through LDS, took two barriers
//     and 1.5 - 2 times a 64-wide layer's products.
//   - The layers' shapes come worked out by the host, loads take a scalar base and lane offsets that do not change within a layer, and
//     the head is apart from the loop over the hidden layers: weights loaded ahead across a barrier may not meet a register copy there.
//   - A load that finds nothing is not issued at all: it would still take its 16 clocks on the way back.
// Rows of the objective stay in registers (one lane per output).  The backward pass reads the parameters as stored.  There eight waves split a
// matrix into groups of 64 columns x slices of rows, the slices added through LDS; sixteen rows (NR = 4) are as wide as
// v_mfma_f32_16x16x4_f32, whose sums need neither slices nor exchanges.
// Against partial sums of every layer in LDS, loads of four features per lane and 1.2 times the arguments, us per call of the whole update:
// 4-64-64-2 at 32 rows 21.9 -> 18.9, 128-256-256-18 at 512 41.1 -> 37.2, on-policy 4-256-256-3 at 4096 54.6 -> 47.8.
#include "tj_mlp_f32.h"
#include "tj_mlp_plan.h"
#include <math.h>
#include <algorithm>
#include <type_traits>

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 load16(buf_rsrc r, uint32_t at, int base)
{
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, base, 0));
}

constexpr int kWaves = tjplan::kF32Waves, kThreads = 64 * kWaves;   // f32_rows: two waves per SIMD, 256 registers each
constexpr size_t kLdsMax = tjplan::kF32Lds;
typedef tjplan::F32Lds RowsLds;

__host__ __device__ inline int up(int x, int a) { return (x + a - 1) / a * a; }

// A layer's forward pass as the kernel reads it.  Scalar arithmetic is on every wave's critical path: what the host can work out, it does.
struct Forward {
    const float *w0, *w1;        // w1: the target network's (Q-learner; elsewhere never used)
    uint32_t bytes;              // of a weight copy
    int pitch, lq, wstep, xstep; // bytes of a step of 16 q k: in the copy, in an activation row
    int KS, bias, cols;          // slices; the layer's biases in LDS, bytes; 16 tiles
    uint32_t wave[tjplan::kF32Waves];   // tile | slice << 8 | steps << 16
};

Forward make_forward(const TjF32Layer &y, bool head, int bias)
{
    const tjplan::F32Forward p = tjplan::f32_forward(y.in, y.out, head);
    Forward d;
    d.w0 = y.WT; d.w1 = y.WT_tg;
    d.bytes = (uint32_t)(y.kp * y.ldn * sizeof(float));
    d.pitch = p.pitch; d.lq = p.lq;
    d.wstep = (64 << p.lq) * p.pitch;
    d.xstep = 64 << p.lq;
    d.KS = p.KS; d.bias = 4 * bias; d.cols = 16 * p.tiles;
    for (int w = 0; w < tjplan::kF32Waves; ++w) {
        const tjplan::F32Wave x = tjplan::f32_wave(p, w);
        d.wave[w] = (uint32_t)x.tile | (uint32_t)x.ks << 8 | (uint32_t)x.n << 16;
    }
    return d;
}

struct Phase : tjplan::F32Phase {
    const float *w;
    int cols;
    uint32_t rF;              // u / F = u * rF >> 16 (u < 4096, F <= 16)
};

// What else the kernel wants of a layer.  The arguments are kept short: the host writes them, and every block waits for them to arrive.
struct RowsLayer {
    float *X, *dZ;
    int in, ldx, lddz, ldn;
};

struct RowsArgs {
    TjRowsCall a;
    RowsLds o;
    const float *bias, *bias_tg, *head_W;
    int A, n_bias, head_slices, kp;    // head outputs; kp: columns of the first layer's input rows
    RowsLayer lay[TJ_MAX_LAYERS];
    Forward fwd[TJ_MAX_LAYERS];
    Phase bwd[TJ_MAX_LAYERS];          // bwd[l]: gradient wrt layer l's input
};

Phase make_phase(const float *w, int pitch, int rows, int cols)
{
    Phase p;
    static_cast<tjplan::F32Phase &>(p) = tjplan::f32_phase(pitch, rows, cols);
    p.w = w; p.cols = cols; p.rF = 65535u / (uint32_t)p.F + 1u;
    return p;
}

// KIND: TJ_ROWS_DQN (three passes, backward), TJ_ROWS_PPO (one pass, backward), TJ_ROWS_ACT (forward only; `mode`
// says what is done with the head outputs)
template <int KIND, int NR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, KIND == TJ_ROWS_ACT && NR == 2 ? 4 : 2))) void f32_rows(const RowsArgs args, const int mode)
{
    constexpr bool DQN = KIND == TJ_ROWS_DQN, BACK = KIND != TJ_ROWS_ACT;
    constexpr int R = 4 * NR;                       // transitions per block
    constexpr int NG = DQN ? 3 * NR : NR;           // row groups: s | s' online | s' target
    constexpr int NON = DQN ? 2 * NR : NR;          // ... of the online network
    const TjRowsCall &a = args.a;
    const RowsLayer *const lay = args.lay;
    {   // the argument block is read all over the kernel: its cache lines are fetched together, once
        uint32_t t = 0;
#pragma unroll
        for (size_t i = 0; i < sizeof(args); i += 64) t ^= ((const uint32_t *)&args)[i / 4];
        asm volatile("" ::"s"(t));
    }
    extern __shared__ __align__(16) float lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = a.L, j0 = blockIdx.x * R;
    const RowsLds &o = args.o;
    const int P = o.pitch;
    float *const keep = lds + o.keep, *const pp = lds + o.pp, *const part = lds + o.part, *const dzb = lds + o.dz;
    auto kept = [&](int l) { return keep + (BACK ? l : l & 1) * R * P; };
    float *const bs = lds + o.bias, *const sm = lds + o.small;
    const int last = L - 1, A = args.A;

    // ---- forward: this wave's part of a layer, a tile of 64 / q features x every KS-th step of 16 q k.  A load is 16 bytes per
    // lane, four k of its own feature; lane part h of q takes chunk h of a step (16 k).  Weights come in two sets of one step, both loaded
    // ahead of the layer that uses them.
    struct Mine {
        const float *w0, *w1;
        uint32_t bytes, at[4];             // lane's bytes from a step's start, per load
        int n, w_at, wstep, x_at, xstep;   // steps; the first one's offset and the distance, in the copy and in a row
        int lq, f, part;                   // f: this lane's feature
    };
    const uint32_t quarter = lane >> 4;
    auto mine = [&](const Forward &p) {
        Mine m;
        const uint32_t w = p.wave[wave];
        const int ks = (int)(w >> 8 & 255u);
        m.lq = p.lq; m.n = (int)(w >> 16);
        m.w_at = ks * p.wstep; m.wstep = p.KS * p.wstep;
        m.x_at = ks * p.xstep; m.xstep = p.KS * p.xstep;
        m.w0 = p.w0; m.w1 = p.w1; m.bytes = p.bytes;
        m.part = tjplan::f32_part(lane, p.lq);
        m.f = tjplan::f32_feature(lane, (int)(w & 255u), p.lq);
#pragma unroll
        for (int b = 0; b < 4; ++b) m.at[b] = 4u * tjplan::f32_weight_at(m.part, b, m.f, p.pitch);
        return m;
    };
    f32x4 wa[2][4], wb[2][4];
    auto fetch = [&](auto set, const Mine &p, int i) {
        constexpr int s = decltype(set)::value;
        if (i >= p.n) return;   // a load that finds nothing would still take its turn on the way back
        const int at = p.w_at + i * p.wstep;
        const buf_rsrc r0 = buf_of(p.w0, (int)p.bytes), r1 = buf_of(p.w1, (int)p.bytes);
#pragma unroll
        for (int b = 0; b < 4; ++b) wa[s][b] = load16(r0, p.at[b], at);
        if constexpr (DQN) {
#pragma unroll
            for (int b = 0; b < 4; ++b) wb[s][b] = load16(r1, p.at[b], at);
        }
        __builtin_amdgcn_sched_barrier(0);   // issued here, not where the registers run short
    };
    const std::integral_constant<int, 0> set0;
    const std::integral_constant<int, 1> set1;

    // ---- backward: chunks of 16 rows of the matrix as stored, [n][k]; load b of one takes row 4 b + q in lane quarter q, columns 4 c .. 4 c + 3
    // (c = lane % 16) of the wave's 64.  One set is loaded ahead of the phase that uses it.  The last group's columns may run past the
    // matrix: zeros or the next row's, features that nobody reads.
    struct Back {             // this wave's part of a phase
        const float *w;
        int pitch, rows, nk, F, KS, f, ks;
        uint32_t rF, row[4];
    };
    auto back = [&](const Phase &p) {
        Back m;
        m.w = p.w; m.pitch = p.pitch; m.rows = p.rows; m.nk = p.nk; m.F = p.F; m.KS = p.KS; m.rF = p.rF;
        m.ks = (int)((uint32_t)wave * p.rF >> 16);
        m.f = wave - m.ks * p.F;
#pragma unroll
        for (int b = 0; b < 4; ++b) m.row[b] = tjplan::f32_row_at(lane, b, p.pitch);
        return m;
    };
    auto active = [&](const Back &p) { return p.ks < p.KS && p.ks < p.nk; };
    auto load_chunk = [&](f32x4 (&w)[4], const Back &p, int c, bool have) {
        const buf_rsrc r = buf_of(p.w, have ? 4 * p.rows * p.pitch : 0);
        const int at = have ? 4 * (int)tjplan::f32_chunk_at(c, p.pitch) : 0;
        const uint32_t last_row = tjplan::f32_last_row_at(c, p.rows, p.pitch);
#pragma unroll
        for (int b = 0; b < 4; ++b) w[b] = load16(r, 4u * tjplan::f32_lane_at(p.row[b], last_row, lane, p.f), at);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto load_first = [&](const Back &p, bool have) { load_chunk(wa[0], p, tjplan::f32_first_chunk(p.ks, p.nk), have && active(p)); };
    // this wave's chunks of a phase; mul(set, chunk) multiplies a set.  The last round is apart: a loop that loads in
    // every round has no wait that covers more than it must.
    auto chunks = [&](const Back &p, auto &&mul) {
        int c = p.ks;
        for (; c + 2 * p.KS < p.nk; c += 2 * p.KS) {
            load_chunk(wa[1], p, c + p.KS, true);
            mul(wa[0], c);
            load_chunk(wa[0], p, c + 2 * p.KS, true);
            mul(wa[1], c + p.KS);
        }
        if (c + p.KS < p.nk) {
            load_chunk(wa[1], p, c + p.KS, true);
            mul(wa[0], c);
            mul(wa[1], c + p.KS);
        } else {
            mul(wa[0], c);
        }
    };
    // ---- backward of sixteen rows (NR = 4); its places are tjplan::f32_back16_*
    struct Back16 { const float *w; int bytes, pitch, steps, tiles; };
    auto back16 = [&](const Phase &p) { return Back16{p.w, 4 * p.rows * p.pitch, 4 * p.pitch, tjplan::f32_back16_steps(p.rows), tjplan::f32_back16_tiles(p.cols)}; };
    auto load_step = [&](f32x4 (&w)[4], const Back16 &p, int tile, int s) {
        const buf_rsrc r = buf_of(p.w, p.bytes);
        const int at = tjplan::f32_back16_at((int)quarter, lane & 15, tile, s, p.pitch);   // past the end in the lane's part: a scalar part must not be
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, at + tjplan::f32_back16_row(j) * p.pitch, 0, 0));
            w[j / 2][j % 2 * 2] = v[0]; w[j / 2][j % 2 * 2 + 1] = v[1];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto back_of = [&](const Phase &p) {
        if constexpr (NR == 4) return back16(p);
        else return back(p);
    };
    auto back_first = [&](const auto &p, bool have) {
        if constexpr (NR == 4) { if (have && wave < p.tiles) load_step(wa[0], p, wave, 0); }
        else load_first(p, have);
    };
    // Sums over the wave's parts: x = {low half of x, low half of y} + {high half of x, high half of y}, and the same
    // for the odd and even quarters of a half.
    auto add_halves = [](float x, float y) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    auto add_quarters = [](float x, float y) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    // Partial sums of a backward phase in LDS: [wave][group][position][4 rows].  acc[e] holds, for the rows n of this lane quarter,
    // feature 4 c + e; two exchanges add the quarters, after which lane (q, c) has feature 4 c + q.  Its position is the lane.
    auto put_part = [&](f32x4 (&acc)[4], int g) {
        f32x4 s;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            s[i] = add_quarters(add_halves(acc[0][i], acc[2][i]), add_halves(acc[1][i], acc[3][i]));
        ((f32x4 *)part)[(wave * NR + g) * 64 + lane] = s;
    };
    // ... and their sum, in slice order, for group g, features 64 f ..; lane = position
    auto get_part = [&](const Back &p, int g, int f) {
        const f32x4 *src = (const f32x4 *)part + (f * NR + g) * 64 + lane;
        const int step = p.F * NR * 64, n = min(p.KS, p.nk);
        f32x4 s = src[0];
        for (int k = 1; k < n; k += 3) {
            f32x4 p[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) p[i] = src[min(k + i, n - 1) * step];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (k + i < n) s += p[i];
        }
        return s;
    };
    const int fpos = 4 * (lane & 15) + (int)quarter;   // feature at position `lane`

    Mine ph = mine(args.fwd[0]);
    fetch(set0, ph, 0);
    fetch(set1, ph, 1);

    // ---- the block's inputs: observation rows, the head weights of the actions taken, biases.  Everything that leads to an address
    // is asked for first, then what lies there, then it is stored: two latencies in all.
    constexpr int RW = (R + kWaves - 1) / kWaves;   // transitions per wave in the objective
    int act_w[RW];
    float rew_w[RW], nd_w[RW], olp_w[RW], adv_w[RW], ret_w[RW];
    {
        const int D = lay[0].in, kp = args.kp, in_h = lay[last].in;
        constexpr int NO = (DQN ? 2 : 1) * R, NOW = (NO + kWaves - 1) / kWaves;
        buf_rsrc src[NOW], head_w[RW];
        uint32_t idx[NOW];
        int aj[RW];
#pragma unroll
        for (int i = 0; i < NOW; ++i) {
            const int r = min(wave + kWaves * i, NO - 1), j = min(j0 + (DQN ? r % R : r), a.B - 1);
            idx[i] = a.rows ? a.rows[j] : (uint32_t)j;
        }
        if (DQN)   // the actions' rows are fetched by the waves from the last one on
#pragma unroll
            for (int i = 0; i < RW; ++i) aj[i] = a.action[min(j0 + min(kWaves - 1 - wave + kWaves * i, R - 1), a.B - 1)];
        // what this wave's rows of the objective need, long before it is used
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int j = min(j0 + wave + i * kWaves, a.B - 1);
            if (DQN) { act_w[i] = a.action[j]; rew_w[i] = a.reward[j]; nd_w[i] = a.done[j] ? 0.f : 1.f; }
            if (KIND == TJ_ROWS_PPO) {
                act_w[i] = a.action[j];
                olp_w[i] = a.old_logp[j]; adv_w[i] = a.adv[j]; ret_w[i] = a.ret[j];
            }
        }
        const int nb = args.n_bias;
        const buf_rsrc b_on = buf_of(args.bias, 4 * nb), b_tg = buf_of(args.bias_tg, DQN ? 4 * nb : 0);
        float b[2], bt[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            b[i] = load4(b_on, 4 * (tid + i * kThreads));
            if (DQN) bt[i] = load4(b_tg, 4 * (tid + i * kThreads));
        }
#pragma unroll
        for (int i = 0; i < NOW; ++i) {
            const int r = wave + kWaves * i;
            const uint32_t row = __builtin_amdgcn_readfirstlane(a.rows ? min(idx[i], a.n_rows - 1u) : idx[i]);
            src[i] = buf_of((!DQN || r < R ? a.obs : a.next_obs) + (size_t)row * D, r < NO ? 4 * D : 0);
        }
        if (DQN && L >= 2)
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                const int aw = __builtin_amdgcn_readfirstlane(min(max(aj[i], 0), A - 1));
                head_w[i] = buf_of(args.head_W + (size_t)aw * in_h, kWaves - 1 - wave + kWaves * i < R ? 4 * in_h : 0);
            }
        const int width = max(kp, DQN && L >= 2 ? in_h : 0);
        for (int c0 = 0; c0 < width; c0 += 128) {   // columns past a row are zeros
            float x[NOW][2], y[RW][2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
#pragma unroll
                for (int i = 0; i < NOW; ++i) x[i][e] = load4(src[i], 4 * (c0 + 64 * e + lane));
                if (DQN && L >= 2)
#pragma unroll
                    for (int i = 0; i < RW; ++i) y[i][e] = load4(head_w[i], 4 * (c0 + 64 * e + lane));
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int c = c0 + 64 * e;
                if (c >= width) break;
#pragma unroll
                for (int i = 0; i < NOW; ++i) {
                    const int r = wave + kWaves * i;
                    if (r < NO) (r < R ? keep + r * P : pp + (r - R) * P)[c + lane] = x[i][e];
                }
                if (DQN && L >= 2)
#pragma unroll
                    for (int i = 0; i < RW; ++i) {
                        const int r = kWaves - 1 - wave + kWaves * i;
                        if (r < R) lds[o.wa + r * P + c + lane] = y[i][e];
                    }
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (tid + i * kThreads < nb) {
                bs[tid + i * kThreads] = b[i];
                if (DQN) bs[nb + tid + i * kThreads] = bt[i];
            }
        for (int i = tid + 2 * kThreads; i < nb; i += kThreads) {
            bs[i] = args.bias[i];
            if (DQN) bs[nb + i] = args.bias_tg[i];
        }
    }
    block_sync();

    // A operand: row lane % 4 of a group, four k from 4 (lane / 4 % 4) on of this lane part's chunk
    const int arow = (lane & 3) * P + 4 * ((lane >> 2) & 3);

    // row r of layer l's input, for the weight gradients
    auto store_input = [&](int l, int r) {
        if (j0 + r >= a.B) return;
        float *const x = lay[l].X + (size_t)(j0 + r) * lay[l].ldx;
        for (int c = 4 * lane; c < lay[l].in; c += 256) *(f32x4 *)(x + c) = *(const f32x4 *)(keep + (l * R + r) * P + c);
    };

    // ---- forward
    f32x4 acc[NG];
    // this wave's part of layer l, and the first loads of the next one (`first(set)`), in flight across the barrier behind it
    auto contract = [&](int l, const Mine &m, auto &&first) {
        // rows of this layer's input, group g
        const float *xs = kept(l), *xn = pp + (l & 1) * 2 * R * P, *xt = l == 0 ? xn : xn + R * P;
        const int x_at = 4 * (arow + 16 * m.part) + m.x_at;
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto mul = [&](const f32x4 (&w)[4], const f32x4 (&wt)[4], int i) {
            f32x4 x[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const float *base = g < NR ? xs + 4 * g * P : g < NON ? xn + 4 * (g - NR) * P : xt + 4 * (g - NON) * P;
                x[g] = *(const f32x4 *)((const uint8_t *)base + x_at + i * m.xstep);
            }
#define TJ_STEP(b)                                                                                                    \
    _Pragma("unroll") for (int e = 0; e < 4; ++e) _Pragma("unroll") for (int g = 0; g < NG; ++g) acc[g] =             \
        __builtin_amdgcn_mfma_f32_4x4x1f32(x[g][e], g < NON ? w[b][e] : wt[b][e], acc[g], 2, b, 0);
            TJ_STEP(0) TJ_STEP(1) TJ_STEP(2) TJ_STEP(3)
#undef TJ_STEP
        };
        int i = 0;
        for (; i + 2 < m.n; i += 2) {
            mul(wa[0], wb[0], i);
            fetch(set0, m, i + 2);
            mul(wa[1], wb[1], i + 1);
            fetch(set1, m, i + 3);
        }
        if (i < m.n) mul(wa[0], wb[0], i);
        first(set0);
        if constexpr (BACK && NR > 1)
            for (int r = wave; r < R; r += kWaves) store_input(l, r);
        if (i + 1 < m.n) mul(wa[1], wb[1], i + 1);
        first(set1);
    };
    // the lane parts' sums: 4 / q rows are left in a lane, from r0 = part << (2 - lq) on
    auto add_halves_of = [&]() {
#pragma unroll
        for (int g = 0; g < NG; ++g) { acc[g][0] = add_halves(acc[g][0], acc[g][2]); acc[g][1] = add_halves(acc[g][1], acc[g][3]); }
    };
    auto add_quarters_of = [&]() {
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g][0] = add_quarters(acc[g][0], acc[g][1]);
    };
    for (int l = 0; l < last; ++l) {
        const Mine nx = mine(args.fwd[l + 1]);
        const int bias = args.fwd[l].bias;
        const float b0 = *(const float *)((const uint8_t *)bs + bias + 4 * ph.f);
        const float b1 = DQN ? *(const float *)((const uint8_t *)(bs + args.n_bias) + bias + 4 * ph.f) : 0.f;
        contract(l, ph, [&](auto set) { fetch(set, nx, decltype(set)::value); });
        if (ph.n > 0) {
            const int to = (ph.part << (2 - ph.lq)) * P + ph.f;
            float *const ds = kept(l + 1) + to, *const dn = pp + ((l + 1) & 1) * 2 * R * P + to;
            auto put_row = [&](int e) {
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    (g < NR ? ds + (4 * g + e) * P : dn + (4 * (g - NR) + e) * P)[0] = fmaxf(acc[g][e] + (g < NON ? b0 : b1), 0.f);
            };
            if (ph.lq > 0) add_halves_of();
            if (ph.lq > 1) add_quarters_of();
            put_row(0);
            if (ph.lq < 2) put_row(1);
            if (ph.lq == 0) { put_row(2); put_row(3); }
        }
        block_sync();
        ph = nx;
    }
    // the head's slices of k: [slice][row][cols]
    const int cols = args.fwd[last].cols;
    const int top = DQN ? L - 2 : L - 1;   // first layer whose input gradient is a contraction; the Q-learner's head's is none
    auto bk = back_of(args.bwd[max(top, 0)]);
    contract(last, ph, [&](auto set) {
        if (BACK && decltype(set)::value == 0) back_first(bk, top >= 1);
    });
    if (ph.n > 0) {
        add_halves_of();
        add_quarters_of();
        float *const to = part + ((args.fwd[last].wave[wave] >> 8 & 255u) * NG * 4 + ph.part) * cols + ph.f;
#pragma unroll
        for (int g = 0; g < NG; ++g) to[4 * g * cols] = acc[g][0];
    }
    block_sync();

    // Head output `lane` of transition `row` under every pass, by one wave: the slices in order, then the bias.
    struct Out { float z[NG / NR]; };
    auto head_out = [&](int row) {
        const int w = cols, n = args.head_slices, ob = args.n_bias - lay[last].ldn + lane;
        const float *src = part + row * w + min(lane, w - 1);
        Out out;
        float p[NG / NR][4];
#pragma unroll
        for (int pass = 0; pass < NG / NR; ++pass)
#pragma unroll
            for (int k = 0; k < 4; ++k) p[pass][k] = src[(min(k, n - 1) * NG * 4 + pass * R) * w];
#pragma unroll
        for (int pass = 0; pass < NG / NR; ++pass) {
            float s = p[pass][0];
#pragma unroll
            for (int k = 1; k < 4; ++k)
                if (k < n) s += p[pass][k];
            s += bs[(pass == 2 ? args.n_bias : 0) + ob];
            out.z[pass] = s;
            const int j = j0 + row;
            if (BACK && lane < A && j < a.B) a.Q[((size_t)pass * a.B + j) * a.ldq + lane] = s;
        }
        return out;
    };
    if constexpr (KIND == TJ_ROWS_ACT) {   // one wave per row, one lane per head output
        for (int row = wave; row < R && j0 + row < a.B; row += kWaves) act_row(a, mode, j0 + row, A, head_out(row).z[0]);
        return;
    }

    // one group of rows leaves four waves without a transition: they store the inputs meanwhile
    if (NR == 1 && wave >= 4)
        for (int l = 0; l < L; ++l) store_input(l, wave - 4);

    // ---- the objective: one wave per transition, one lane per head output
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        const int row = wave + q * kWaves;
        if (row >= R) break;
        const bool valid = j0 + row < a.B;
        const Out out = head_out(row);
        act_w[q] = __builtin_amdgcn_readfirstlane(min(max(act_w[q], 0), A - (DQN ? 1 : 2)));
        if constexpr (DQN) {
            const TdRow t = td_row(a, A, out.z[0], out.z[1], out.z[2], act_w[q], rew_w[q], nd_w[q], valid);
            if (lane == 0) {
                sm[row] = t.loss;
                sm[16 + row] = t.g;
                if (valid) a.astar[j0 + row] = t.best;
            }
            if (valid) lay[last].dZ[(size_t)(j0 + row) * lay[last].lddz + lane] = lane == act_w[q] ? t.g : 0.f;
        } else {
            const PpoRow t = ppo_row(a, A - 1, out.z[0], act_w[q], olp_w[q], adv_w[q], ret_w[q], valid);
            if (lane == 0) {
                sm[row] = t.pi;
                sm[16 + row] = t.v;
                sm[32 + row] = t.H;
            }
            dzb[row * o.dzp + lane] = t.g;
            if (valid) lay[last].dZ[(size_t)(j0 + row) * lay[last].lddz + lane] = t.g;
        }
    }
    block_sync();
    // ---- input gradients.  dZ of layer l - 1 = relu'(X_l) (dZ_l W_l)
    int cur = 0;
    auto put = [&](int l, int g, int col, f32x4 s, int buf) {   // layer l's input gradient, rows of group g
        const RowsLayer &b = lay[l - 1];
        const int in = lay[l].in, j = j0 + 4 * g;
        const float *x = keep + (l * R + 4 * g) * P + col;
        float *dst = dzb + (buf * R + 4 * g) * P + col, *z = b.dZ + (size_t)j * b.lddz + col;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = col < in && x[i * P] > 0.f ? s[i] : 0.f;
            dst[i * P] = v;
            if (j + i < a.B) z[i * b.lddz] = v;
        }
    };
    if (DQN && L >= 2) {   // the head's: one non-zero per row of dL/dQ, no contraction
        const int F = (lay[last].in + 63) / 64;
        for (int u = wave; u < NR * F; u += kWaves) {
            const int g = NR == 1 ? 0 : u / F, col = (u - g * F) * 64 + lane;
            f32x4 s;
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = sm[16 + 4 * g + i] * lds[o.wa + (4 * g + i) * P + col];
            put(last, g, col, s, 0);
        }
        block_sync();
    }
    // A operand: row lane % 4 of a group, row n of a chunk as the loads have it
    const int brow = (lane & 3) * P + 4 * ((lane >> 2) & 3) + (int)quarter;
    if constexpr (NR == 4) {
        const int r = lane & 15;
        for (int l = top; l >= 1; --l) {
            const float *const src = dzb + cur * R * o.dzp + r * o.dzp + tjplan::f32_back16_dz((int)quarter, 0);
            float *const dst = dzb + (cur ^ 1) * R * o.dzp + r * o.dzp;
            const Back16 nx = back16(args.bwd[max(l - 1, 1)]);
            const int in = lay[l].in, ldz = lay[l - 1].lddz;
            float *const z = lay[l - 1].dZ + (size_t)(j0 + r) * ldz;
            if (wave >= bk.tiles) back_first(nx, l > 1);
            for (int tile = wave; tile < bk.tiles; tile += kWaves) {
                f32x4 ab[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
                auto mul = [&](const f32x4 (&w)[4], int st) {
                    const f32x4 v[2] = {*(const f32x4 *)(src + 32 * st), *(const f32x4 *)(src + 32 * st + 16)};
#pragma unroll
                    for (int j = 0; j < 8; ++j)
#pragma unroll
                        for (int e = 0; e < 2; ++e)
                            ab[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j / 2][j % 2 * 2 + e], v[j / 4][j % 4], ab[e], 0, 0, 0);
                };
                int st = 0;
                for (; st + 2 < bk.steps; st += 2) {
                    load_step(wa[1], bk, tile, st + 1);
                    mul(wa[0], st);
                    load_step(wa[0], bk, tile, st + 2);
                    mul(wa[1], st + 1);
                }
                if (st + 1 < bk.steps) {
                    load_step(wa[1], bk, tile, st + 1);
                    mul(wa[0], st);
                    mul(wa[1], st + 1);
                } else {
                    mul(wa[0], st);
                }
                if (tile + kWaves < bk.tiles) load_step(wa[0], bk, tile + kWaves, 0);
                else back_first(nx, l > 1);
                // columns c .. c + 7 of row r: element 2 i + e is register i of operand e
                const int c = tjplan::f32_back16_col((int)quarter, tile);
                const float *const x = keep + (l * R + r) * P + c;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 m = *(const f32x4 *)(x + 4 * h);
                    f32x4 v;
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = c + 4 * h + u < in && m[u] > 0.f ? ab[u % 2][2 * h + u / 2] : 0.f;
                    *(f32x4 *)(dst + c + 4 * h) = v;
                    if (j0 + r < a.B) *(f32x4 *)(z + c + 4 * h) = v;
                }
            }
            block_sync();
            cur ^= 1;
            bk = nx;
        }
    } else {
        for (int l = top; l >= 1; --l) {
            const float *src = dzb + cur * R * P;
            const Back nx = back(args.bwd[max(l - 1, 1)]);
            f32x4 ab[NR][4];
            if (active(bk)) {
#pragma unroll
                for (int g = 0; g < NR; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) ab[g][e] = f32x4{0.f, 0.f, 0.f, 0.f};
                chunks(bk, [&](const f32x4 (&w)[4], int c) {
                    float ax[NR];
#pragma unroll
                    for (int g = 0; g < NR; ++g) ax[g] = src[4 * g * P + brow + 16 * c];
#define TJ_STEP(b)                                                                                            \
        _Pragma("unroll") for (int e = 0; e < 4; ++e) _Pragma("unroll") for (int g = 0; g < NR; ++g) ab[g][e] =   \
            __builtin_amdgcn_mfma_f32_4x4x1f32(ax[g], w[b][e], ab[g][e], 2, b, 0);
                    TJ_STEP(0) TJ_STEP(1) TJ_STEP(2) TJ_STEP(3)
#undef TJ_STEP
                });
            }
            load_first(nx, l > 1);
            if (active(bk)) {
#pragma unroll
                for (int g = 0; g < NR; ++g) put_part(ab[g], g);
            }
            block_sync();
            const int F = bk.F;
            for (int u = wave; u < NR * F; u += kWaves) {
                const int g = (int)((uint32_t)u * bk.rF >> 16), f = u - g * F;
                put(l, g, f * 64 + fpos, get_part(bk, g, f), cur ^ 1);
            }
            block_sync();
            cur ^= 1;
            bk = nx;
        }
    }

    if (wave == 0) {   // the block's sums, in a fixed order
        if (DQN) {
            const float s = wave_sum(lane < R ? sm[lane] : 0.f);
            if (lane == 0) a.loss_part[blockIdx.x] = s;
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const float s = wave_sum(lane < R ? sm[16 * q + lane] : 0.f);
                if (lane == 0) a.loss_part[(size_t)blockIdx.x * 4 + q] = s;
            }
        }
    }
}

// ---------------------------------------------------------------- weights

// dW[n][k] = sum_m dZ[m][n] X[m][k] over the whole batch, and Adam on it.  Both operands have m as their slow index,
// which is what the fp32 MFMA wants (16x16x4: lane (q, n) holds element n of row q), so they come straight from
// memory.  A block of sixteen waves takes a tile of dW, 64 or 16 columns wide on either side.  On a side of 64 a
// wave works on 32 columns: an 8-byte load per lane is four rows x 32 columns, and its component e is an operand
// of 16 columns (2 n + e).  The waves that remain split the rows; their sums meet in LDS.
//   16 x 16 tiles: everything about a weight happens in one block, sixteen waves deep: for short batches, where
//     the kernel is a chain of latencies (4.3 us on the smallest network, 8.5 us for 0.1 M weights x 512 rows).
//   64 x 64 tiles: four times less operand traffic per weight, which bounds long batches; the batch is cut into
//     S slices so that the tiles fill the chip, and f32_adam adds them.  (One launch in which the block that
//     arrives last at a tile's counter adds the slices took 25 us instead of 9 + 7 on 67 k weights x 4096 rows: the
//     coherent stores, the counter and the few blocks that finish cost more than a launch.)
struct UpdatePlan {
    int begin[TJ_MAX_LAYERS + 1];   // first tile of every layer
    int tn[TJ_MAX_LAYERS], tk[TJ_MAX_LAYERS], nk[TJ_MAX_LAYERS];   // tile sides (64 or 16), tiles along k
    int wide, S, rows;              // 64-wide tiles; slices of the batch, rows of one (a multiple of 16)
};

constexpr int kUThreads = 1024, kUWaves = 16;
constexpr int kLongBatch = 2048;   // rows

template <int TN, int TK>
__device__ __forceinline__ void update_tile(const TjF32Update &a, const UpdatePlan &plan, const int l, const int t,
                                            const int z, float *lds)
{
    constexpr int QN = TN == 64 ? 2 : 1, QK = TK == 64 ? 2 : 1, NQ = QN * QK;   // waves side by side
    constexpr int EN = QN, EK = QK, NP = EN * EK;   // operands per side of a wave, operand pairs
    constexpr int RG = kUWaves / NQ;                // row groups
    constexpr int NV = RG == 4 ? 4 : 1;             // weights per thread in the end
    constexpr int U = 8;                            // steps of four rows whose loads are in flight together
    typedef float vecN __attribute__((ext_vector_type(EN)));
    typedef float vecK __attribute__((ext_vector_type(EK)));
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = wave % NQ, rg = wave / NQ;
    const TjF32Layer &y = a.lay[l];
    const int nkt = plan.nk[l];
    const int k0 = (t % nkt) * TK, n0 = (t / nkt) * TN;
    const int nw = n0 + 32 * (wq % QN), kw = k0 + 32 * (wq / QN);   // this wave's corner
    const bool with_bias = k0 == 0;

    // Once the row groups are added, this thread owns accumulator register r of operand pair v0 (and of the others
    // where NV = 4): row n = nw + EN (4 q + r) + i, column k = kw + EK c16 + j of pair (i, j).
    const int r_own = rg & 3, v0 = NV == 4 ? 0 : rg >> 2;
    const bool owner = rg < 4 * NP;
    auto n_of = [&](int v) { return nw + EN * (4 * q + r_own) + v / EK; };
    auto k_of = [&](int v) { return kw + EK * c16 + v % EK; };
    // db[n0 + w 32 + EN c + i]: thread 32 w + 16 i + c, from the waves of the first column half
    const int nb = n0 + 32 * (tid >> 5) + EN * (tid & 15) + (EN == 2 ? (tid >> 4) & 1 : 0);
    const bool bias_thread = with_bias && tid < TN && nb < y.out;

    const int m0 = z * plan.rows, m1 = min(a.B, m0 + plan.rows);
    const int per = ((m1 - m0 + 4 * RG - 1) / (4 * RG)) * 4;      // rows per group
    const int w0 = m0 + rg * per, w1 = min(m1, w0 + per);
    const float *pz = y.dZ + nw + EN * c16, *px = y.X + kw + EK * c16;
    f32x4 acc[EN][EK];
#pragma unroll
    for (int i = 0; i < EN; ++i)
#pragma unroll
        for (int j = 0; j < EK; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum[EN];
#pragma unroll
    for (int i = 0; i < EN; ++i) bsum[i] = 0.f;
    if constexpr (NQ == 4) {
        // Four waves want every row: the block brings stages of 64 rows x (64 + 64) columns into LDS (16-byte direct
        // loads, two buffers) instead of each wave its own columns.  A row's two 128-byte halves are exchanged
        // in odd rows, so that the two rows a 32-lane read touches lie in different banks.
        typedef __attribute__((address_space(3))) uint8_t *lds_u8;
        uint8_t *const buf = (uint8_t *)lds;
        const int n_stage = m1 > m0 ? (m1 - m0 + 63) / 64 : 0;
        auto dma16 = [](const float *src, uint8_t *dst) {
            const uint32_t at = (uint32_t)(uintptr_t)(lds_u8)dst;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(src) : "memory");
        };
        const int piece = (lane & 15) ^ ((q & 1) << 3);
        auto issue = [&](int st) {   // each wave four rows of both operands; rows past the batch repeat the last one
            const size_t row = (size_t)min(m0 + 64 * st + 4 * wave + q, a.B - 1);
            uint8_t *dst = buf + (st & 1) * 32768 + wave * 1024;
            dma16(y.dZ + row * y.lddz + n0 + 4 * piece, dst);
            dma16(y.X + row * y.ldx + k0 + 4 * piece, dst + 16384);
        };
        if (n_stage > 0) issue(0);
        for (int st = 0; st < n_stage; ++st) {
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");   // stage st is here, stage st - 1 has been read
            if (st + 1 < n_stage) issue(st + 1);
            const uint8_t *base = buf + (st & 1) * 32768 + (16 * rg + q) * 256 + c16 * 8;
            const uint8_t *bz = base + 128 * ((wq % QN) ^ (q & 1)), *bx = base + 16384 + 128 * ((wq / QN) ^ (q & 1));
            vecN zr[4];
            vecK xr[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { zr[u] = *(const vecN *)(bz + 1024 * u); xr[u] = *(const vecK *)(bx + 1024 * u); }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = m0 + 64 * st + 16 * rg + 4 * u + q < m1;
#pragma unroll
                for (int i = 0; i < EN; ++i) {
                    const float zv = in ? zr[u][i] : 0.f;
                    bsum[i] += zv;
#pragma unroll
                    for (int j = 0; j < EK; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(zv, xr[u][j], acc[i][j], 0, 0, 0);
                }
            }
        }
        __syncthreads();   // the stages have been read: their memory takes the sums
    } else {
        for (int m = w0; m < w1; m += 4 * U) {
            vecN zr[U];
            vecK xr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t rr = (uint32_t)min(m + 4 * u + q, w1 - 1);
                zr[u] = *(const vecN *)(pz + rr * (uint32_t)y.lddz);
                xr[u] = *(const vecK *)(px + rr * (uint32_t)y.ldx);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (m + 4 * u >= w1) break;
                const bool in = m + 4 * u + q < w1;
#pragma unroll
                for (int i = 0; i < EN; ++i) {
                    const float zv = in ? zr[u][i] : 0.f;
                    bsum[i] += zv;
#pragma unroll
                    for (int j = 0; j < EK; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(zv, xr[u][j], acc[i][j], 0, 0, 0);
                }
            }
        }
    }
    // the owned weights' optimizer state
    AdamState s[NV], sb = {0.f, 0.f, 0.f};
    auto load_state = [&]() {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int n = n_of(v0 + v), k = k_of(v0 + v);
            s[v] = {0.f, 0.f, 0.f};
            if (owner && n < y.out && k < y.in) {
                const size_t at = (size_t)n * y.in + k;
                s[v] = {y.W[at], a.m[y.w_off + at], a.v[y.w_off + at]};
            }
        }
        if (bias_thread) sb = {y.bias[nb], a.m[y.b_off + nb], a.v[y.b_off + nb]};
    };
    if (plan.S == 1) load_state();   // in flight during the exchange below

    // ---- the row groups' sums through LDS, in group order: [wave][register][operand pair][lane]
    float *red = lds, *redb = lds + kUWaves * 4 * NP * 64;
#pragma unroll
    for (int i = 0; i < EN; ++i) {
#pragma unroll
        for (int j = 0; j < EK; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[((wave * 4 + r) * NP + i * EK + j) * 64 + lane] = acc[i][j][r];
        if (with_bias && wq < QN) redb[((rg * QN + wq) * EN + i) * 64 + lane] = bsum[i];
    }
    __syncthreads();
    float g[NV], gb = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        g[v] = 0.f;
        if (owner)
            for (int w = 0; w < RG; ++w) g[v] += red[(((w * NQ + wq) * 4 + r_own) * NP + v0 + v) * 64 + lane];
    }
    if (bias_thread) {
        for (int w = 0; w < RG; ++w)
#pragma unroll
            for (int p = 0; p < 4; ++p)
                gb += redb[((w * QN + (tid >> 5)) * EN + (EN == 2 ? (tid >> 4) & 1 : 0)) * 64 + 16 * p + (tid & 15)];
    }

    if (plan.S > 1) {   // a slice of the gradient, in the order of the parameters
        float *out = a.slices + (size_t)z * a.slice_stride;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int n = n_of(v0 + v), k = k_of(v0 + v);
            if (owner && n < y.out && k < y.in) out[y.w_off + (size_t)n * y.in + k] = g[v];
        }
        if (bias_thread) out[y.b_off + nb] = gb;
        return;
    }

    // ---- Adam, and what follows the weights: the copy of the forward pass, [k / 4][n][4], through LDS [k][n]
    constexpr int TP = TN + 1;
    __syncthreads();   // the sums have been read
    if (owner) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int n = n_of(v0 + v), k = k_of(v0 + v);
            const AdamState x = adam(a, s[v], g[v]);
            lds[(k - k0) * TP + n - n0] = x.th;
            if (n < y.out && k < y.in) {
                const size_t at = (size_t)n * y.in + k, off = y.w_off + at;
                y.W[at] = x.th; a.m[off] = x.m; a.v[off] = x.v; a.g[off] = g[v];
                if (a.sync_target) y.W_tg[at] = x.th;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < (TN * TK + kUThreads - 1) / kUThreads; ++i) {
        const int e = tid + i * kUThreads, kk = e / (4 * TN) * 4 + e % 4, nn = e / 4 % TN;
        if (kk < TK && k0 + kk < y.in && n0 + nn < y.out) {
            const size_t at = tjplan::f32_copy_at(n0 + nn, k0 + kk, y.ldn);
            const float th = lds[kk * TP + nn];
            y.WT[at] = th;
            if (a.sync_target) y.WT_tg[at] = th;
        }
    }
    if (bias_thread) {
        const AdamState x = adam(a, sb, gb);
        y.bias[nb] = y.BP[nb] = x.th; a.m[y.b_off + nb] = x.m; a.v[y.b_off + nb] = x.v; a.g[y.b_off + nb] = gb;
        if (a.sync_target) y.bias_tg[nb] = y.BP_tg[nb] = x.th;
    }
}

template <bool WIDE>
__global__ __launch_bounds__(kUThreads) void f32_update(const TjF32Update a, const UpdatePlan plan)
{
    {
        uint32_t t = 0;
#pragma unroll
        for (size_t i = 0; i < sizeof(a); i += 64) t ^= ((const uint32_t *)&a)[i / 4];
        asm volatile("" ::"s"(t));
    }
    __shared__ __align__(16) float lds[WIDE ? kUWaves * 4 * 4 * 64 + kUWaves * 2 * 64 : kUWaves * 4 * 64 + kUWaves * 64];
    const int n_block = gridDim.x - (plan.S == 1 ? 1 : 0);
    if ((int)blockIdx.x == n_block) { step_stats<kUThreads>(a, lds); return; }   // the last block of the update's last launch
    // An XCD (id % 8) takes a run of the slice-major order: it reads few slices' rows.
    const int per_xcd = n_block / 8, id = WIDE ? (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int n_tile = plan.begin[a.L], z = WIDE ? id / n_tile : 0, tile = id - z * n_tile;
    if (z >= plan.S) return;
    int l = 0;
    while (l + 1 < a.L && tile >= plan.begin[l + 1]) ++l;
    const int t = tile - plan.begin[l];
    if constexpr (!WIDE) {
        update_tile<16, 16>(a, plan, l, t, z, lds);
    } else if (plan.tn[l] == 64) {
        if (plan.tk[l] == 64) update_tile<64, 64>(a, plan, l, t, z, lds);
        else update_tile<64, 16>(a, plan, l, t, z, lds);
    } else {
        if (plan.tk[l] == 64) update_tile<16, 64>(a, plan, l, t, z, lds);
        else update_tile<16, 16>(a, plan, l, t, z, lds);
    }
}

struct F32Cast { TjF32Layer lay[TJ_MAX_LAYERS]; int online; };

// Second half of an update whose gradient came in slices: their sum in slice order, Adam, the copy of the forward pass.  A
// block owns 16 x 32 weights, a thread two of them; every load is issued before the first use.
constexpr int kAdamN = 16, kAdamK = 32;

__global__ __launch_bounds__(256) void f32_adam(const TjF32Update a, const UpdatePlan plan)
{
    __shared__ float tile[kAdamK][kAdamN + 1];
    const int tid = threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) { step_stats<256>(a, &tile[0][0]); return; }
    int l = 0;
    while (l + 1 < a.L && (int)blockIdx.x >= plan.begin[l + 1]) ++l;
    const TjF32Layer &y = a.lay[l];
    const int t = (int)blockIdx.x - plan.begin[l], k0 = (t % plan.nk[l]) * kAdamK, n0 = (t / plan.nk[l]) * kAdamN;
    const int k = k0 + (tid & 31), r = tid >> 5;
    size_t at[3];
    bool in[3];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int n = n0 + r + 8 * v;
        in[v] = n < y.out && k < y.in;
        at[v] = in[v] ? y.w_off + (size_t)n * y.in + k : y.w_off;
    }
    const int nb = n0 + tid;
    in[2] = k0 == 0 && tid < kAdamN && nb < y.out;
    at[2] = in[2] ? y.b_off + nb : y.w_off;
    float *theta = y.W - y.w_off, *theta_tg = y.W_tg - y.w_off;   // the flat vectors
    AdamState s[3];
    float g[3];
#pragma unroll
    for (int v = 0; v < 3; ++v) {
        s[v] = {theta[at[v]], a.m[at[v]], a.v[at[v]]};
        g[v] = a.slices[at[v]];
    }
    for (int z = 1; z < plan.S; z += 8) {
        float p[8][3];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int v = 0; v < 3; ++v) p[u][v] = a.slices[(size_t)min(z + u, plan.S - 1) * a.slice_stride + at[v]];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (z + u >= plan.S) break;
#pragma unroll
            for (int v = 0; v < 3; ++v) g[v] += p[u][v];
        }
    }
#pragma unroll
    for (int v = 0; v < 3; ++v) {
        const AdamState x = adam(a, s[v], g[v]);
        if (v < 2) tile[tid & 31][r + 8 * v] = x.th;
        if (in[v]) {
            theta[at[v]] = x.th; a.m[at[v]] = x.m; a.v[at[v]] = x.v; a.g[at[v]] = g[v];
            if (a.sync_target) theta_tg[at[v]] = x.th;
            if (v == 2) {
                y.BP[nb] = x.th;
                if (a.sync_target) y.BP_tg[nb] = x.th;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int kk = (tid >> 6) * 4 + (tid & 3) + 16 * v, nn = (tid >> 2) & 15;
        if (k0 + kk < y.in && n0 + nn < y.out) {
            const size_t to = tjplan::f32_copy_at(n0 + nn, k0 + kk, y.ldn);
            y.WT[to] = tile[kk][nn];
            if (a.sync_target) y.WT_tg[to] = tile[kk][nn];
        }
    }
}

// The copies that the forward pass reads, from the master parameters (creation and set_state only): a layer per blockIdx.y.
__global__ __launch_bounds__(256) void f32_cast(const F32Cast a)
{
    const TjF32Layer &y = a.lay[blockIdx.y];
    const float *W = a.online ? y.W : y.W_tg, *b = a.online ? y.bias : y.bias_tg;
    float *WT = a.online ? y.WT : y.WT_tg, *BP = a.online ? y.BP : y.BP_tg;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < (size_t)y.in * y.out; e += (size_t)gridDim.x * 256)
        WT[tjplan::f32_copy_at((int)(e / y.in), (int)(e % y.in), y.ldn)] = W[e];
    if (blockIdx.x == 0)
        for (int n = threadIdx.x; n < y.out; n += 256) BP[n] = b[n];
}

// Tiles of every layer, tn x tk wide.
int plan_tiles(int L, const TjF32Layer *lay, UpdatePlan &p)
{
    int n = 0;
    for (int l = 0; l < L; ++l) {
        p.begin[l] = n;
        p.nk[l] = (lay[l].in + p.tk[l] - 1) / p.tk[l];
        n += p.nk[l] * ((lay[l].out + p.tn[l] - 1) / p.tn[l]);
    }
    p.begin[L] = n;
    return n;
}

// 16 x 16 tiles while their operand traffic (128 bytes per tile and row, at the 24 bytes per clock and CU that 4-byte
// loads reach) stays below what a second launch costs; then 64-wide tiles and as many slices of the batch as
// one round of blocks holds.  A network of few tiles never has that traffic, but its few blocks are a chain as long as
// the batch: past kLongBatch rows the slices are worth the launch for every network (on-policy updates, us with whole columns :
// sliced; 4-64-64-2 at 2048 rows 33 : 33, 4096 49 : 40, 8192 85 : 60; 4-16-2 at 2048 28 : 28, 4096 42 : 30, 32768 254 : 101).
int update_plan(int L, const TjF32Layer *lay, int B, UpdatePlan &p)
{
    for (int l = 0; l < L; ++l) p.tn[l] = p.tk[l] = 16;
    int n = plan_tiles(L, lay, p);
    p.S = 1;
    p.wide = (size_t)n * B > 400000 || B > kLongBatch;
    if (p.wide) {
        for (int l = 0; l < L; ++l) {
            p.tn[l] = lay[l].out > 32 ? 64 : 16;
            p.tk[l] = lay[l].in > 32 ? 64 : 16;
        }
        n = plan_tiles(L, lay, p);
        p.S = std::max(1, std::min(std::min(kF32MaxSlices, 256 / n), B / 128));
    }
    p.rows = up((B + p.S - 1) / p.S, 16);
    return n;
}

int rows_nr(const TjF32Rows &a, int mode)
{
    return tjplan::f32_groups(a.L, a.lay, a.B, mode == TJ_ROWS_DQN, mode == TJ_ROWS_DQN || mode == TJ_ROWS_PPO);
}

template <int KIND, int NR> int launch_rows(const TjF32Rows &a, int mode, hipStream_t st)
{
    const bool dqn = KIND == TJ_ROWS_DQN, back = KIND != TJ_ROWS_ACT;
    const RowsLds o = tjplan::f32_lds(a.L, a.lay, NR, dqn, back);
    static bool attr_set = false;   // idempotent: a race sets it twice
    if (!attr_set) {
        TJ_HIP_TRY(hipFuncSetAttribute((const void *)f32_rows<KIND, NR>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kLdsMax));
        attr_set = true;
    }
    RowsArgs r;
    r.a = a;
    r.o = o;
    r.bias = a.lay[0].BP; r.bias_tg = a.lay[0].BP_tg; r.head_W = a.lay[a.L - 1].W;
    r.A = a.lay[a.L - 1].out;
    r.kp = a.lay[0].kp;
    r.n_bias = 0;
    for (int l = 0; l < a.L; ++l) {
        const TjF32Layer &y = a.lay[l];
        r.lay[l] = {y.X, y.dZ, y.in, y.ldx, y.lddz, y.ldn};
        r.fwd[l] = make_forward(y, l == a.L - 1, r.n_bias);
        r.bwd[l] = make_phase(y.W, y.in, y.out, y.in);
        r.n_bias += y.ldn;
    }
    const tjplan::F32Forward head = tjplan::f32_forward(a.lay[a.L - 1].in, a.lay[a.L - 1].out, true);
    r.head_slices = std::min(head.KS, head.steps);
    f32_rows<KIND, NR><<<(a.B + 4 * NR - 1) / (4 * NR), kThreads, o.total * sizeof(float), st>>>(r, mode);
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}

}  // namespace

bool tj_f32_fits(int L, const int *in, const int *out, int passes, int max_batch) { return tjplan::f32_fits(L, in, out, passes, max_batch); }

int tj_f32_blocks(const TjF32Rows &a, int mode)
{
    const int nr = rows_nr(a, mode);
    return (a.B + 4 * nr - 1) / (4 * nr);
}

int tj_f32_rows(const TjF32Rows &a, int mode, hipStream_t st)
{
    if (a.B < 1 || a.L < 1 || a.L > TJ_MAX_LAYERS) return TJ_ERR_SHAPE;
    const int nr = rows_nr(a, mode);
    if (mode == TJ_ROWS_DQN) return nr == 1 ? launch_rows<TJ_ROWS_DQN, 1>(a, mode, st) : launch_rows<TJ_ROWS_DQN, 2>(a, mode, st);
    if (mode == TJ_ROWS_PPO)
        return nr == 1 ? launch_rows<TJ_ROWS_PPO, 1>(a, mode, st)
                       : nr == 2 ? launch_rows<TJ_ROWS_PPO, 2>(a, mode, st) : launch_rows<TJ_ROWS_PPO, 4>(a, mode, st);
    return nr == 1 ? launch_rows<TJ_ROWS_ACT, 1>(a, mode, st)
                   : nr == 2 ? launch_rows<TJ_ROWS_ACT, 2>(a, mode, st) : launch_rows<TJ_ROWS_ACT, 4>(a, mode, st);
}

int tj_f32_slices(int L, const TjF32Layer *lay, int B)
{
    UpdatePlan p;
    update_plan(L, lay, B, p);
    return p.S > 1 ? p.S : 0;   // a smaller batch has no more of them
}

int tj_f32_update(const TjF32Update &a, hipStream_t st)
{
    if (a.B < 1 || a.L < 1 || a.L > TJ_MAX_LAYERS) return TJ_ERR_SHAPE;
    UpdatePlan p;
    const int n = update_plan(a.L, a.lay, a.B, p);
    const int stats = p.S == 1;   // one block more for the step's statistics
    if (p.wide) f32_update<true><<<up(n * p.S, 8) + stats, kUThreads, 0, st>>>(a, p);
    else f32_update<false><<<n + stats, kUThreads, 0, st>>>(a, p);
    if (p.S > 1) {
        for (int l = 0; l < a.L; ++l) { p.tn[l] = kAdamN; p.tk[l] = kAdamK; }
        const int n_adam = plan_tiles(a.L, a.lay, p);
        f32_adam<<<n_adam + 1, 256, 0, st>>>(a, p);
    }
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}

void tj_f32_copy_shape(TjF32Layer &y, bool head)
{
    const tjplan::F32Forward p = tjplan::f32_forward(y.in, y.out, head);
    y.kp = (16 << p.lq) * p.steps;
    y.ldn = p.pitch;
}

size_t tj_f32_copy_at(const TjF32Layer &y, int n, int k) { return tjplan::f32_copy_at(n, k, y.ldn); }

int tj_f32_cast(int L, const TjF32Layer *lay, bool online, hipStream_t st)
{
    F32Cast a;
    size_t most = 0;
    for (int l = 0; l < TJ_MAX_LAYERS; ++l) {
        a.lay[l] = lay[l < L ? l : 0];
        most = std::max(most, (size_t)a.lay[l].in * a.lay[l].out);
    }
    a.online = online;
    f32_cast<<<dim3((unsigned)((most + 255) / 256), L), 256, 0, st>>>(a);
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}
