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
//               tile, the transposed copy the forward pass reads, and the target network where it is due.
//   f32_adam    where update_plan cuts a long batch into slices: their sum, and everything behind it.
//
// f32_rows multiplies with v_mfma_f32_4x4x1_16b_f32: sixteen independent 4 x 4 products per instruction,
// the A operand (4 rows x 1) broadcast to all of them, so one instruction is 4 rows x 64 features x one k at
// the full fp32 matrix rate (136 TFLOP/s measured on the bare instruction).  Rows come in groups of four, not
// 16 or 32: a batch of 512 spreads over 128 blocks without padding.  What bounds the kernel is the stream of
// weights from the L2 into a CU: each is read once per block, from a matrix with the features contiguous (the
// transposed copy in the forward pass, the parameters as stored in the backward pass), by 16-byte loads whose
// 16-lane quarters take 64 features of four consecutive k (4-byte loads, one k each, moved 24 bytes per clock
// and CU).  The instruction's broadcast is limited to a quarter of the wave, so each quarter multiplies its own
// k; the quarters are added by lane swaps at the end of a layer.  Eight waves split a layer into groups of 64
// features x slices of k; the slices are added through LDS in slice order.  Weight loads do not depend on activations, so a wave has its first loads of the next
// layer in flight across the barriers between two layers.
#include "tj_mlp_f32.h"
#include "tj_mlp_plan.h"
#include <math.h>
#include <algorithm>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) uint8_t *gbytes;
typedef const __attribute__((address_space(1))) __attribute__((aligned(4))) f32x4 *gf32x4;

constexpr int kWaves = tjplan::kF32Waves, kThreads = 64 * kWaves;   // f32_rows: two waves per SIMD, 256 registers each
constexpr size_t kLdsMax = 160 * 1024;

__host__ __device__ inline int up(int x, int a) { return (x + a - 1) / a * a; }

// LDS layout of f32_rows in floats.  Activation rows are `pitch` floats apart, pitch % 64 == 16: the four
// rows x 16 k of an A operand fall on 64 distinct banks.
struct RowsLds {
    int pitch, keep, pp, part, dz, wa, qs, bias, small, total;
};

RowsLds rows_lds(int L, const TjF32Layer *lay, int nr, bool dqn, bool backward)
{
    RowsLds o;
    int w = 0, nb = 0, waves = 0;   // waves: those with a part of some phase
    for (int l = 0; l < L; ++l) {
        waves = std::max(waves, tjplan::f32_part_waves(tjplan::f32_phase(lay[l].ldn, lay[l].kp, lay[l].ldn)));
        if (backward && l) waves = std::max(waves, tjplan::f32_part_waves(tjplan::f32_phase(lay[l].in, lay[l].out, lay[l].in)));
        w = lay[l].kp > w ? lay[l].kp : w;
        if (l + 1 < L) w = lay[l].ldn > w ? lay[l].ldn : w;
        nb += lay[l].ldn;
    }
    o.pitch = up(w, 64) + 16;
    const int R = 4 * nr, NG = dqn ? 3 * nr : nr;
    int at = 0;
    o.keep = at; at += (backward ? L : std::min(L, 2)) * R * o.pitch;   // input rows of every layer, s; acting: two layers in turn
    o.pp = at; at += dqn ? 2 * 2 * R * o.pitch : 0;     // s' (online), s' (target), two layers in turn
    o.part = at; at += waves * 2 * NG * 256;            // the k slices of one layer
    o.dz = at; at += backward ? 2 * R * o.pitch : 0;    // output gradients, two layers in turn
    o.wa = at; at += dqn ? R * o.pitch : 0;             // head weights of the actions taken
    o.qs = at; at += 4 * NG * 64;                       // head outputs
    o.bias = at; at += nb * (dqn ? 2 : 1);
    o.small = at; at += 64;                             // per row: loss terms, gradient
    o.total = at;
    return o;
}

struct Phase : tjplan::F32Phase {
    const float *w0, *w1;     // w1: the target network's (forward of the Q-learner; elsewhere never used)
    uint32_t rF;              // u / F = u * rF >> 16 (u < 4096, F <= 16)
};

struct RowsArgs {
    TjF32Rows a;
    RowsLds o;
    Phase fwd[TJ_MAX_LAYERS], bwd[TJ_MAX_LAYERS];   // bwd[l]: gradient wrt layer l's input
    int n_bias;
};

Phase make_phase(const float *w0, const float *w1, int pitch, int rows, int cols)
{
    Phase p;
    static_cast<tjplan::F32Phase &>(p) = tjplan::f32_phase(pitch, rows, cols);
    p.w0 = w0; p.w1 = w1; p.rF = 65535u / (uint32_t)p.F + 1u;
    return p;
}

template <bool V> struct Two { static constexpr bool value = V; };   // both networks' weights, or one's

// KIND: TJ_ROWS_DQN (three passes, backward), TJ_ROWS_PPO (one pass, backward), TJ_ROWS_ACT (forward only; `mode`
// says what is done with the head outputs)
template <int KIND, int NR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, KIND == TJ_ROWS_ACT && NR == 2 ? 4 : 2))) void f32_rows(const RowsArgs args, const int mode)
{
    constexpr bool DQN = KIND == TJ_ROWS_DQN, BACK = KIND != TJ_ROWS_ACT;
    constexpr int R = 4 * NR;                       // transitions per block
    constexpr int NG = DQN ? 3 * NR : NR;           // row groups: s | s' online | s' target
    constexpr int NON = DQN ? 2 * NR : NR;          // ... of the online network
    const TjF32Rows &a = args.a;
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
    float *const qs = lds + o.qs, *const bs = lds + o.bias, *const sm = lds + o.small;
    const int last = L - 1, A = a.lay[last].out;

    // A chunk is 16 k; load b of it takes k = 4 b + q in lane quarter q, features 4 n .. 4 n + 3 (n = lane % 16) of the
    // wave's 64.  Weights come in two sets of one chunk, set 0 loaded ahead of the phase that uses it.  In the backward
    // pass the last group's columns may run past the matrix into the parameters behind it: features that nobody reads.
    struct Mine {             // this wave's part of a phase
        const float *w0, *w1;
        int pitch, rows, nk, F, KS, f, ks;
        uint32_t rF, row[4];
    };
    const uint32_t quarter = lane >> 4;
    auto mine = [&](const Phase &p) {
        Mine m;
        m.w0 = p.w0; m.w1 = p.w1; m.pitch = p.pitch; m.rows = p.rows; m.nk = p.nk; m.F = p.F; m.KS = p.KS; m.rF = p.rF;
        m.ks = (int)((uint32_t)wave * p.rF >> 16);
        m.f = wave - m.ks * p.F;
#pragma unroll
        for (int b = 0; b < 4; ++b) m.row[b] = tjplan::f32_row_at(lane, b, p.pitch);
        return m;
    };
    auto active = [](const Mine &p) { return p.ks < p.KS && p.ks < p.nk; };
    auto load = [&](f32x4 (&w)[4], const float *base, const Mine &p, int c) {
        gbytes rows = (gbytes)(uintptr_t)(base + tjplan::f32_chunk_at(c, p.pitch));
        asm("" : "+s"(rows));                // wave-uniform: the scalar base of the loads
        const uint32_t last_row = tjplan::f32_last_row_at(c, p.rows, p.pitch);
#pragma unroll
        for (int b = 0; b < 4; ++b) w[b] = *(gf32x4)(rows + 4u * tjplan::f32_lane_at(p.row[b], last_row, lane, p.f));
        __builtin_amdgcn_sched_barrier(0);   // issued here, not where the registers run short
    };
    f32x4 wa[2][4], wb[2][4];
    auto load_first = [&](const Mine &p, auto two) {
        const int c = tjplan::f32_first_chunk(p.ks, p.nk);
        load(wa[0], p.w0, p, c);
        if constexpr (decltype(two)::value) load(wb[0], p.w1, p, c);
    };
    // this wave's chunks of a phase; mul(set, chunk) multiplies a set.  The last round is apart: a loop that loads in
    // every round has no wait that covers more than it must.
    auto chunks = [&](const Mine &p, auto two_nets, auto &&mul) {
        constexpr bool two = decltype(two_nets)::value;
        int c = p.ks;
        for (; c + 2 * p.KS < p.nk; c += 2 * p.KS) {
            load(wa[1], p.w0, p, c + p.KS);
            if constexpr (two) load(wb[1], p.w1, p, c + p.KS);
            mul(wa[0], wb[0], c);
            load(wa[0], p.w0, p, c + 2 * p.KS);
            if constexpr (two) load(wb[0], p.w1, p, c + 2 * p.KS);
            mul(wa[1], wb[1], c + p.KS);
        }
        if (c + p.KS < p.nk) {
            load(wa[1], p.w0, p, c + p.KS);
            if constexpr (two) load(wb[1], p.w1, p, c + p.KS);
            mul(wa[0], wb[0], c);
            mul(wa[1], wb[1], c + p.KS);
        } else {
            mul(wa[0], wb[0], c);
        }
    };
    // Partial sums of a layer in LDS: [wave][2][group][position][4 rows], two per wave.  acc[e] holds, for the k of this
    // lane quarter, feature 4 n + e; one exchange of wave halves adds quarters q and q + 2, after which lane
    // (q, n) has features 4 n + e + 2 (q / 2), e < 2, of slice q % 2.  Feature 4 n + e lies at position 16 e + n: writes
    // and reads touch consecutive 16-byte pieces.
    auto put_part = [&](f32x4 (&acc)[4], int g, int ng) {
        f32x4 *dst = (f32x4 *)part + (((wave * 2 + (quarter & 1)) * ng + g) * 64 + 32 * (quarter >> 1) + (lane & 15));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            f32x4 s;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[e][i]), __float_as_uint(acc[e + 2][i]), false, false);
                s[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            }
            dst[16 * e] = s;
        }
    };
    // ... and their sum, in slice order, for group g, features 64 f ..; lane = position
    auto get_part = [&](const Mine &p, int g, int ng, int f) {
        const f32x4 *src = (const f32x4 *)part + ((f * 2 * ng + g) * 64 + lane);
        const int step = p.F * 2 * ng * 64, n = min(p.KS, p.nk);
        f32x4 s = src[0] + src[ng * 64];
        for (int k = 1; k < n; ++k) { src += step; s += src[0] + src[ng * 64]; }
        return s;
    };
    const int fpos = 4 * (lane & 15) + (lane >> 4);   // feature at position `lane`

    Mine ph = mine(args.fwd[0]);
    load_first(ph, Two<DQN>{});

    // ---- the block's inputs: biases, observation rows, the head weights of the actions taken
    {
        for (int i = tid; i < args.n_bias; i += kThreads) {
            const float b = a.bias[i], bt = DQN ? a.bias_tg[i] : 0.f;
            bs[i] = b;
            if (DQN) bs[args.n_bias + i] = bt;
        }
        const int D = a.lay[0].in, kp = a.lay[0].kp;
        constexpr int NO = (DQN ? 2 : 1) * R;
        for (int r = wave; r < NO; r += kWaves) {
            const int jr = DQN ? r % R : r, j = min(j0 + jr, a.B - 1);
            const size_t srow = a.rows ? (size_t)min(a.rows[j], a.n_rows - 1u) : (size_t)j;
            const float *src = (r < R ? a.obs : a.next_obs) + srow * D;
            float *dst = r < R ? keep + r * P : pp + (r - R) * P;
            float *x0 = BACK && r < R && j0 + jr < a.B ? a.lay[0].X + (size_t)j * a.lay[0].ldx : nullptr;
            for (int c0 = 0; c0 < kp; c0 += 256) {
                float x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = c0 + 64 * q + lane;
                    x[q] = c < D ? src[c] : 0.f;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = c0 + 64 * q + lane;
                    if (c < kp) dst[c] = x[q];
                    if (x0 && c < D) x0[c] = x[q];
                }
            }
        }
        if (DQN && L >= 2) {
            const int in = a.lay[last].in;
            for (int r = kWaves - 1 - wave; r < R; r += kWaves) {
                const int act = a.action[min(j0 + r, a.B - 1)], aj = min(max(act, 0), A - 1);
                const float *src = a.lay[last].W + (size_t)aj * in;
                for (int c = lane; c < in; c += 64) lds[o.wa + r * P + c] = src[c];
            }
        }
    }
    // what this wave's rows of the objective need, long before it is used
    constexpr int RW = (R + kWaves - 1) / kWaves;
    int act_w[RW];
    float rew_w[RW], nd_w[RW], olp_w[RW], adv_w[RW], ret_w[RW];
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        const int j = min(j0 + wave + q * kWaves, a.B - 1);
        if (DQN) { act_w[q] = min(max(a.action[j], 0), A - 1); rew_w[q] = a.reward[j]; nd_w[q] = a.done[j] ? 0.f : 1.f; }
        if (KIND == TJ_ROWS_PPO) {
            act_w[q] = min(max(a.action[j], 0), A - 2);
            olp_w[q] = a.old_logp[j]; adv_w[q] = a.adv[j]; ret_w[q] = a.ret[j];
        }
    }
    block_sync();

    // A operand: row lane % 4 of a group, k of a chunk as the loads above have it
    const int arow = (lane & 3) * P + 4 * ((lane >> 2) & 3) + (int)quarter;
    f32x4 acc[NG][4];

    // ---- forward
    int boff = 0;
    for (int l = 0; l < L; ++l) {
        // rows of this layer's input, group g
        const float *xs = kept(l), *xn = pp + (l & 1) * 2 * R * P, *xt = l == 0 ? xn : xn + R * P;
        Mine nx = ph;
        if (l + 1 < L) nx = mine(args.fwd[l + 1]);
        else if (BACK && (DQN ? L - 2 : L - 1) >= 1) nx = mine(args.bwd[DQN ? L - 2 : L - 1]);   // the Q-learner's head gradient is no contraction
        if (active(ph)) {
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[g][e] = f32x4{0.f, 0.f, 0.f, 0.f};
            chunks(ph, Two<DQN>{}, [&](const f32x4 (&w)[4], const f32x4 (&wt)[4], int c) {
                float ax[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const float *base = g < NR ? xs + 4 * g * P : g < NON ? xn + 4 * (g - NR) * P : xt + 4 * (g - NON) * P;
                    ax[g] = base[arow + 16 * c];
                }
#define TJ_STEP(b)                                                                                                    \
    _Pragma("unroll") for (int e = 0; e < 4; ++e) _Pragma("unroll") for (int g = 0; g < NG; ++g) acc[g][e] =          \
        __builtin_amdgcn_mfma_f32_4x4x1f32(ax[g], g < NON ? w[b][e] : wt[b][e], acc[g][e], 2, b, 0);
                TJ_STEP(0) TJ_STEP(1) TJ_STEP(2) TJ_STEP(3)
#undef TJ_STEP
            });
        }
        load_first(nx, Two<DQN>{});   // in flight across the barriers; nobody's if nothing follows
        if (active(ph)) {
#pragma unroll
            for (int g = 0; g < NG; ++g) put_part(acc[g], g, NG);
        }
        block_sync();
        const int F = ph.F;
        for (int u = wave; u < NG * F; u += kWaves) {
            const int g = (int)((uint32_t)u * ph.rF >> 16), f = u - g * F, col = f * 64 + fpos;
            const float b = bs[(g < NON ? boff : args.n_bias + boff) + col];
            f32x4 s = get_part(ph, g, NG, f) + b;
            if (l < last) {
                float *dst = g < NR ? kept(l + 1) + 4 * g * P + col : pp + (((l + 1) & 1) * 2 * R + 4 * (g - NR)) * P + col;
#pragma unroll
                for (int i = 0; i < 4; ++i) { s[i] = fmaxf(s[i], 0.f); dst[i * P] = s[i]; }
                if (BACK && g < NR) {
                    const int j = j0 + 4 * g, ldx = a.lay[l + 1].ldx;
                    float *x = a.lay[l + 1].X + (size_t)j * ldx + col;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (j + i < a.B) x[i * ldx] = s[i];
                }
            } else {
                const int gr = DQN ? g % NR : g, pass = DQN ? g / NR : 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    qs[(4 * g + i) * 64 + fpos] = s[i];
                    const int j = j0 + 4 * gr + i;
                    if (BACK && fpos < A && j < a.B) a.Q[((size_t)pass * a.B + j) * a.ldq + fpos] = s[i];
                }
            }
        }
        block_sync();
        boff += a.lay[l].ldn;
        ph = nx;
    }

    if constexpr (KIND == TJ_ROWS_ACT) {   // one wave per row, one lane per head output
        for (int row = wave; row < R && j0 + row < a.B; row += kWaves) {
            act_row(a, mode, j0 + row, A, qs + row * 64);
        }
        return;
    }

    // ---- the objective: one wave per transition, one lane per head output
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        const int row = wave + q * kWaves;
        if (row >= R) break;
        const bool valid = j0 + row < a.B;
        if constexpr (DQN) {
            const TdRow t = td_row(a, A, qs + row * 64, qs + (R + row) * 64, qs + (2 * R + row) * 64, act_w[q], rew_w[q], nd_w[q], valid);
            if (lane == 0) {
                sm[row] = t.loss;
                sm[16 + row] = t.g;
                if (valid) a.astar[j0 + row] = t.best;
            }
            if (valid) a.lay[last].dZ[(size_t)(j0 + row) * a.lay[last].lddz + lane] = lane == act_w[q] ? t.g : 0.f;
        } else {
            const PpoRow t = ppo_row(a, A - 1, qs + row * 64, act_w[q], olp_w[q], adv_w[q], ret_w[q], valid);
            if (lane == 0) {
                sm[row] = t.pi;
                sm[16 + row] = t.v;
                sm[32 + row] = t.H;
            }
            dzb[row * P + lane] = t.g;
            if (valid) a.lay[last].dZ[(size_t)(j0 + row) * a.lay[last].lddz + lane] = t.g;
        }
    }
    block_sync();
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

    // ---- input gradients.  dZ of layer l - 1 = relu'(X_l) (dZ_l W_l)
    int cur = 0;
    auto put = [&](int l, int g, int col, f32x4 s, int buf) {   // layer l's input gradient, rows of group g
        const TjF32Layer &b = a.lay[l - 1];
        const int in = a.lay[l].in, j = j0 + 4 * g;
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
        const int F = (a.lay[last].in + 63) / 64;
        for (int u = wave; u < NR * F; u += kWaves) {
            const int g = NR == 1 ? 0 : u / F, col = (u - g * F) * 64 + lane;
            f32x4 s;
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = sm[16 + 4 * g + i] * lds[o.wa + (4 * g + i) * P + col];
            put(last, g, col, s, 0);
        }
        block_sync();
    }
    for (int l = DQN ? L - 2 : L - 1; l >= 1; --l) {
        const float *src = dzb + cur * R * P;
        Mine nx = ph;
        if (l - 1 >= 1) nx = mine(args.bwd[l - 1]);
        f32x4 ab[NR][4];
        if (active(ph)) {
#pragma unroll
            for (int g = 0; g < NR; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) ab[g][e] = f32x4{0.f, 0.f, 0.f, 0.f};
            chunks(ph, Two<false>{}, [&](const f32x4 (&w)[4], const f32x4 (&)[4], int c) {
                float ax[NR];
#pragma unroll
                for (int g = 0; g < NR; ++g) ax[g] = src[4 * g * P + arow + 16 * c];
#define TJ_STEP(b)                                                                                            \
    _Pragma("unroll") for (int e = 0; e < 4; ++e) _Pragma("unroll") for (int g = 0; g < NR; ++g) ab[g][e] =   \
        __builtin_amdgcn_mfma_f32_4x4x1f32(ax[g], w[b][e], ab[g][e], 2, b, 0);
                TJ_STEP(0) TJ_STEP(1) TJ_STEP(2) TJ_STEP(3)
#undef TJ_STEP
            });
        }
        if (l > 1) load_first(nx, Two<false>{});
        if (active(ph)) {
#pragma unroll
            for (int g = 0; g < NR; ++g) put_part(ab[g], g, NR);
        }
        block_sync();
        const int F = ph.F;
        for (int u = wave; u < NR * F; u += kWaves) {
            const int g = (int)((uint32_t)u * ph.rF >> 16), f = u - g * F;
            put(l, g, f * 64 + fpos, get_part(ph, g, NR, f), cur ^ 1);
        }
        block_sync();
        cur ^= 1;
        ph = nx;
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

    // ---- Adam, and what follows the weights: the transposed copy through LDS [k][n], features contiguous
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
        const int e = tid + i * kUThreads, kk = e / TN, nn = e % TN;
        if (kk < TK && k0 + kk < y.in && n0 + nn < y.out) {
            const size_t at = (size_t)(k0 + kk) * y.ldn + n0 + nn;
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

// Second half of an update whose gradient came in slices: their sum in slice order, Adam, the transposed copy.  A
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
        const int kk = (tid >> 4) + 16 * v, nn = tid & 15;
        if (k0 + kk < y.in && n0 + nn < y.out) {
            const size_t to = (size_t)(k0 + kk) * y.ldn + n0 + nn;
            y.WT[to] = tile[kk][nn];
            if (a.sync_target) y.WT_tg[to] = tile[kk][nn];
        }
    }
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

// Groups of four rows per block: the fewest that need no second round of blocks on the chip, or the most that LDS holds.  The
// Q-learner's second group fits where rows are narrow or the layers short enough that not all waves have partial sums
// (us with one group : two; 4-64-64-2 at 2048 rows 37 : 31, 8192 101 : 76; 16-32-5 8192 66 : 50).
// Acting on rows of at most kActPaired floats stays at two groups, whose blocks find place in pairs on a CU: one hides the other's
// latency.  On wider rows the weights, read once per block, weigh more (us for 32768 rows, two groups : four; 4-64-64-3 51 : 61,
// 128-256-256-19 121 : 134, 64-384-384-7 187 : 206, 128-512-512-19 294 : 286, 256-512-512-512-33 547 : 499).
constexpr int kActPaired = 384 + 16;

int rows_nr(const TjF32Rows &a, int mode)
{
    const bool dqn = mode == TJ_ROWS_DQN, back = dqn || mode == TJ_ROWS_PPO;
    const int most = dqn ? 2 : !back && rows_lds(a.L, a.lay, 2, dqn, back).pitch <= kActPaired ? 2 : 4;
    int best = 1;
    for (int nr = 1; nr <= most; nr *= 2) {
        if (rows_lds(a.L, a.lay, nr, dqn, back).total * sizeof(float) > kLdsMax) break;
        best = nr;
        if ((a.B + 4 * nr - 1) / (4 * nr) <= 256) break;   // one round of blocks on the chip
    }
    return best;
}

template <int KIND, int NR> int launch_rows(const TjF32Rows &a, int mode, hipStream_t st)
{
    const bool dqn = KIND == TJ_ROWS_DQN, back = KIND != TJ_ROWS_ACT;
    const size_t bytes = rows_lds(a.L, a.lay, NR, dqn, back).total * sizeof(float);
    static bool attr_set = false;   // idempotent: a race sets it twice
    if (!attr_set) {
        TJ_HIP_TRY(hipFuncSetAttribute((const void *)f32_rows<KIND, NR>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kLdsMax));
        attr_set = true;
    }
    RowsArgs r;
    r.a = a;
    r.o = rows_lds(a.L, a.lay, NR, dqn, back);
    r.n_bias = 0;
    for (int l = 0; l < a.L; ++l) {
        const TjF32Layer &y = a.lay[l];
        r.fwd[l] = make_phase(y.WT, y.WT_tg, y.ldn, y.kp, y.ldn);
        r.bwd[l] = make_phase(y.W, y.W, y.in, y.out, y.in);
        r.n_bias += y.ldn;
    }
    for (int l = a.L; l < TJ_MAX_LAYERS; ++l) r.fwd[l] = r.bwd[l] = r.fwd[0];
    f32_rows<KIND, NR><<<(a.B + 4 * NR - 1) / (4 * NR), kThreads, bytes, st>>>(r, mode);
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}

}  // namespace

// Largest batch of a Q-learner that is updated here.  One group of four rows per block reads the weights of both networks for
// every four transitions, and past some batch the layered kernels, whose tiles share them, are faster (us here : there;
// 128-512-512-512-18 at 8192 rows 769 : 844, 16384 1559 : 1394; 300-500-384-500-33 757 : 773, 1515 : 1315; 128-256-256-18 at 16384
// 358 : 370, 32768 701 : 637; seven layers of 64-128 513 : 581, 1000 : 969; with two groups 16-32-5 84 : 96, 157 : 150).
constexpr int kQRows = 16384, kQRowsWide = 8192, kQWide = 256 + 16;   // the latter past rows of kQWide floats

bool tj_f32_fits(int L, const int *in, const int *out, int passes, int max_batch)
{
    if (L < 1 || L > TJ_MAX_LAYERS || in[0] > kF32MaxInput || out[L - 1] > kF32MaxOut) return false;
    TjF32Layer lay[TJ_MAX_LAYERS] = {};
    for (int l = 0; l < L; ++l) {
        if (l + 1 < L && out[l] > kF32MaxWidth) return false;
        lay[l].in = in[l]; lay[l].out = out[l];
        lay[l].kp = up(in[l], 16); lay[l].ldn = up(out[l], 64);
    }
    const RowsLds o = rows_lds(L, lay, 1, passes == 3, true);
    if (passes == 3 && max_batch > (o.pitch > kQWide ? kQRowsWide : kQRows)) return false;
    return o.total * sizeof(float) <= kLdsMax;
}

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
