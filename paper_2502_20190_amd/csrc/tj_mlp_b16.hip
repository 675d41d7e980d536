// Policy updates and inference of bf16 vector networks up to 1024 wide (Algorithm 1 of the paper, batched).
//
//   b16_rows    one block per 16 NR transitions: all layers of all forward passes, the TD target (or the clipped
//               objective) and the input gradients back to the first hidden layer, activations in LDS.
//   b16_update  one block per tile of a weight matrix: its gradient over the whole batch, then Adam on the tile and
//               the copies that follow it; long batches are cut into slices that b16_adam adds.
//
// As layer-by-layer GEMMs the 77-300-300-17 network at batch 1000 was 13 kernels of 5 to 36 us, each on 8 to 48
// blocks: 229 us with the sampling before it, 41 us now (b16_rows 21, b16_update 7).  128-512-512-512-18 at batch 4096:
// 145 -> 78 us; on-policy 128-512-512-512-19 at 32768 rows: 339 -> 229 us.  A block here has no other operand traffic than the weights, each read once: they are stored as the matrix
// instruction takes them, so that a wave's load is 4 KB of contiguous memory straight into registers, which is what a
// CU's path to the L2 moves fastest (45 - 47 bytes per clock; the kernel is bound by this stream and, on
// small networks, by the latency between layers).  The eight waves of a block split a layer by groups of 32 features; a wave
// keeps two groups of loads in flight, the first of the next layer across the barrier between two layers.
// v_mfma_f32_16x16x32_bf16: the weights are the first operand (rows = features), the transitions the second, so that a
// lane ends up with four neighbouring features of one transition: 8-byte LDS stores.
#include "tj_mlp_b16.h"
#include "tj_mlp_plan.h"
#include <algorithm>
#include <cmath>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) uint8_t *gbytes;
typedef const __attribute__((address_space(1))) u32x4 *gu32x4;
typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr size_t kLdsMax = tjplan::kB16Lds;
constexpr int kGroup = 4096;        // bytes of a weight group (32 rows x 64 contraction elements)
using tjplan::kPartPitch, tjplan::kZPitch;
typedef tjplan::B16Lds RowsLds;

__host__ __device__ inline int up(int x, int a) { return (x + a - 1) / a * a; }

__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    const bf16x2 v = {(__bf16)lo, (__bf16)hi};   // round to nearest even
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ f32x4 mma(const u32x4 &p, const u32x4 &q, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, p), __builtin_bit_cast(bf16x8, q), c, 0, 0, 0);
}

struct Phase {
    const tj_bf16 *w;
    int items, per;           // groups of 32 features (of both networks where there are two), groups per item
};

struct RowsArgs {
    TjB16Rows a;
    RowsLds o;
    Phase fwd[TJ_MAX_LAYERS], bwd[TJ_MAX_LAYERS];   // bwd[l]: gradient wrt layer l's input
    int ms;                                         // 32-row steps of the batch
};

// LDS accesses ordered across the block; global loads stay in flight (they belong to the next layer)
__device__ __forceinline__ void block_sync_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int KIND, int NR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void b16_rows(const RowsArgs args, const int mode)
{
    constexpr bool DQN = KIND == TJ_ROWS_DQN, BACK = KIND != TJ_ROWS_ACT;
    constexpr int R = 16 * NR;                      // transitions per block
    constexpr int NON = DQN ? 2 * NR : NR;          // row groups of the online network: s | s'
    constexpr int NS = 4;                           // slices of the head's contraction, per network
    const TjB16Rows &a = args.a;
    {   // the argument block is read all over the kernel: its cache lines are fetched together, once
        uint32_t t = 0;
#pragma unroll
        for (size_t i = 0; i < sizeof(args); i += 64) t ^= ((const uint32_t *)&args)[i / 4];
        asm volatile("" ::"s"(t));
    }
    extern __shared__ __align__(16) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, n16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = a.L, j0 = blockIdx.x * R, last = L - 1, A = a.lay[last].out;
    const RowsLds &o = args.o;
    const int P = o.pitch;
    float *const part = (float *)(lds + o.part), *const bs = (float *)(lds + o.bias);
    float *const sm = (float *)(lds + o.small);
    uint8_t *const dzb = lds + o.dz;
    auto keep = [&](int l) { return lds + o.keep + (BACK ? l : l & 1) * R * P; };
    auto pp = [&](int l, int net) { return lds + o.pp + ((l & 1 ? 0 : 2) + net) * R * P; };   // (0, 1) is keep(0)

    // This wave's weight groups of a phase: items wave, wave + 8, ... of `per` groups each; of the head's forward one item,
    // a slice of its contraction.
    struct Mine { gbytes p; int n, per, jump, k0, g; };
    auto mine = [&](const Phase &ph, bool head) {
        Mine m;
        m.g = 0;
        int at;
        if (head) {
            const int net = DQN ? wave >> 2 : 0, sl = wave & 3;
            m.k0 = sl * ph.per / NS;
            m.per = (sl + 1) * ph.per / NS - m.k0;
            m.n = DQN || wave < 4 ? m.per : 0;
            at = net * ph.per + m.k0;
            m.jump = 0;
        } else {
            m.k0 = 0; m.per = ph.per;
            const int items = wave < ph.items ? (ph.items - wave + kWaves - 1) / kWaves : 0;
            m.n = items * ph.per;
            at = items ? wave * ph.per : 0;
            m.jump = ((kWaves - 1) * ph.per + 1) * kGroup;
        }
        m.p = (gbytes)(uintptr_t)ph.w + (size_t)at * kGroup;
        return m;
    };
    const uint32_t lane16 = lane * 16;
    auto load = [&](u32x4 (&w)[4], Mine &m) {   // the next group, and on
        gbytes base = m.p;
        asm("" : "+s"(base));                   // wave-uniform: the scalar base of the loads
#pragma unroll
        for (int f = 0; f < 4; ++f) w[f] = *(gu32x4)(base + lane16 + 1024 * f);
        __builtin_amdgcn_sched_barrier(0);
        const bool wrap = ++m.g == m.per;
        m.g = wrap ? 0 : m.g;
        m.p += wrap ? m.jump : kGroup;
    };
    u32x4 wa[4], wb[4];
    // mul(group, position along the contraction), fin(item) after an item's last group.  The first group has been loaded
    // before; the last round is apart, so that a loop that loads in every round waits for no more than it must.
    auto stream = [&](Mine &m, auto &&mul, auto &&fin) {
        int c = 0, gc = 0, item = 0;
        auto one = [&](const u32x4 (&w)[4]) {
            mul(w, m.k0 + gc, item);
            if (++gc == m.per) { fin(item); gc = 0; ++item; }
        };
        if (m.n == 0) return;
        for (; c + 2 < m.n; c += 2) {
            load(wb, m); one(wa);
            load(wa, m); one(wb);
        }
        if (c + 1 < m.n) { load(wb, m); one(wa); one(wb); }
        else one(wa);
    };

    Mine ph = mine(args.fwd[0], L == 1);
    load(wa, ph);

    // ---- the block's inputs: observation rows, biases.  Everything that leads to an address or waits for the objective is asked for
    // first, then the rows, then they are stored: two latencies in all (the scalars' values are taken when they are needed: 21.5 -> 19.3 us
    // on 77-300-300-17 at 1000 rows).
    constexpr int RW = R / kWaves;
    int act_w[RW], done_w[RW];
    float rew_w[RW], olp_w[RW], adv_w[RW], ret_w[RW];
    {
        constexpr int NO = (DQN ? 2 : 1) * R / kWaves;   // rows per wave
        const int D = a.lay[0].in, kp = up(D, 64);
        buf_rsrc src[NO];
        uint32_t idx[NO];
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const int r = wave + kWaves * i, j = min(j0 + (DQN ? r % R : r), a.B - 1);
            idx[i] = a.rows ? a.rows[j] : (uint32_t)j;
        }
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int j = min(j0 + wave + i * kWaves, a.B - 1);
            if (BACK) act_w[i] = a.action[j];
            if (DQN) { rew_w[i] = a.reward[j]; done_w[i] = a.done[j]; }
            if (KIND == TJ_ROWS_PPO) { olp_w[i] = a.old_logp[j]; adv_w[i] = a.adv[j]; ret_w[i] = a.ret[j]; }
        }
        const int nb = DQN ? 2 * o.n_bias : o.n_bias;   // the target network's follow
        const buf_rsrc bias = buf_of(a.lay[0].BP, 4 * nb);
        float b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = load4(bias, 4 * (tid + i * kThreads));
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const int r = wave + kWaves * i;
            const uint32_t row = __builtin_amdgcn_readfirstlane(a.rows ? min(idx[i], a.n_rows - 1u) : idx[i]);
            src[i] = buf_of((!DQN || r < R ? a.obs : a.next_obs) + (size_t)row * D, 4 * D);
        }
        for (int c0 = 0; c0 < kp; c0 += 128) {   // columns past a row are zeros
            float x[NO][2];
#pragma unroll
            for (int i = 0; i < NO; ++i)
#pragma unroll
                for (int e = 0; e < 2; ++e) x[i][e] = load4(src[i], 4 * (c0 + 64 * e + lane));
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int c = c0 + 64 * e;
                if (c >= kp) break;
#pragma unroll
                for (int i = 0; i < NO; ++i) {
                    const int r = wave + kWaves * i;
                    uint8_t *dst = r < R ? keep(0) + r * P : pp(0, 0) + (r - R) * P;
                    *(tj_bf16 *)(dst + 2 * (c + lane)) = __builtin_bit_cast(tj_bf16, (__bf16)x[i][e]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (tid + i * kThreads < nb) bs[tid + i * kThreads] = b[i];
        for (int i = tid + 4 * kThreads; i < nb; i += kThreads) bs[i] = a.lay[0].BP[i];
    }
    block_sync_lds();

    // LDS rows [transition][feature] as fragments for the weight gradient: transposing reads give a lane eight
    // transitions of one feature; a block of 16 transitions is half a fragment
    auto put_frags = [&](const uint8_t *buf, int pitch, int width, tj_bf16 *F) {
        const int np = (width + 31) / 32, t = lane >> 5, h8 = (lane >> 4) & 1;
        for (int u = wave; u < NR * np; u += kWaves) {
            const int gr = NR == 1 ? 0 : u % NR, fp = u / NR, mr = blockIdx.x * NR + gr;
            if (NR > 2 && (mr >> 1) >= args.ms) continue;   // rows past the batch's last step
            const uint8_t *p = buf + (16 * gr + 8 * h8 + (n16 >> 2)) * pitch + 2 * (32 * fp + 16 * t + 4 * (n16 & 3));
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)p);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + 4 * pitch));
            const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
            const u32x4 v = {l2.x, l2.y, h2.x, h2.y};
            *(u32x4 *)(F + (((size_t)(fp * args.ms + (mr >> 1)) * 2 + t) * 64 + (2 * (mr & 1) + h8) * 16 + n16) * 8) = v;
        }
    };
    if constexpr (BACK) put_frags(keep(0), P, a.lay[0].in, a.lay[0].XF);

    // second operand: row n16 of a group, 8 contraction elements from 8 q
    const int brow = n16 * P + 16 * q;
    f32x4 acc[2][NON];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int g = 0; g < NON; ++g) acc[t][g] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();

    // ---- forward
    int boff = 0;
    for (int l = 0; l < L; ++l) {
        const bool head = l == last;
        const uint8_t *xs = keep(l) + brow, *xn = pp(l, 0) + brow, *xt = l == 0 ? xn : pp(l, 1) + brow;
        const int half = args.fwd[l].items >> (DQN ? 1 : 0);   // items of one network
        auto target = [&](int item) { return DQN && (head ? wave >= 4 : wave + kWaves * item >= half); };
        stream(ph, [&](const u32x4 (&w)[4], int kg, int item) {
            const int at = kg * 128;
            if (DQN && target(item)) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int g = 0; g < NR; ++g) {
                        const u32x4 x = *(const u32x4 *)(xt + 16 * g * P + at + 64 * s);
#pragma unroll
                        for (int t = 0; t < 2; ++t) acc[t][g] = mma(w[2 * t + s], x, acc[t][g]);
                    }
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int g = 0; g < NON; ++g) {
                        const u32x4 x = *(const u32x4 *)((g < NR ? xs + 16 * g * P : xn + 16 * (g - NR) * P) + at + 64 * s);
#pragma unroll
                        for (int t = 0; t < 2; ++t) acc[t][g] = mma(w[2 * t + s], x, acc[t][g]);
                    }
            }
        }, [&](int item) {
            const bool tg = target(item);
            if (head) {   // a slice's partial sums: [slice][row][36]; online s | s', then target
                const int sl = wave & 3;
                float *dst = part + ((tg ? NS * NON * 16 + sl * R : sl * NON * 16) + n16) * kPartPitch + 4 * q;
#pragma unroll
                for (int g = 0; g < NON; ++g)
                    if (!tg || g < NR) {
#pragma unroll
                        for (int t = 0; t < 2; ++t) *(f32x4 *)(dst + 16 * g * kPartPitch + 16 * t) = acc[t][g];
                    }
            } else {
                const int f = wave + kWaves * item - (tg ? half : 0);
                const bool pad = f == half - 1 && (half & 1);   // the next layer reads whole groups of 64
                const float *b = bs + (tg ? o.n_bias : 0) + boff + 32 * f + 4 * q;
                uint8_t *ds = keep(l + 1), *dn = pp(l + 1, 0), *dt = pp(l + 1, 1);
                const int at = n16 * P + 64 * f + 8 * q;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const f32x4 bias = *(const f32x4 *)(b + 16 * t);
#pragma unroll
                    for (int g = 0; g < NON; ++g)
                        if (!tg || g < NR) {
                            f32x4 v = acc[t][g] + bias;
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
                            uint8_t *d = (tg ? dt + 16 * g * P : g < NR ? ds + 16 * g * P : dn + 16 * (g - NR) * P) + at + 32 * t;
                            *(uint2 *)d = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
                            if (pad) *(uint2 *)(d + 64) = make_uint2(0u, 0u);
                        }
                }
            }
            clear();
        });
        if (l + 1 < L) { ph = mine(args.fwd[l + 1], l + 1 == last); load(wa, ph); }
        else if (BACK && L > 1) { ph = mine(args.bwd[last], false); load(wa, ph); }
        block_sync_lds();
        boff += up(a.lay[l].out, 32);
    }

    // Head output `lane` % 32 of transition `row` under every pass, by one wave: the slices in order, then the bias.
    constexpr int NP = DQN ? 3 : 1;
    struct Out { float z[NP]; };
    const int per = args.fwd[last].per;
    auto head_out = [&](int row) {
        const int c = lane & 31, j = j0 + row;
        const float *hb = bs + boff - 32;
        Out out;
        float p[NP][NS];
#pragma unroll
        for (int pass = 0; pass < NP; ++pass) {
            const float *src = part + (pass == 2 ? NS * NON * 16 + row : pass * R + row) * kPartPitch + c;
            const int step = (pass == 2 ? R : NON * 16) * kPartPitch;
#pragma unroll
            for (int k = 0; k < NS; ++k) p[pass][k] = src[k * step];
        }
#pragma unroll
        for (int pass = 0; pass < NP; ++pass) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < NS; ++k)
                if (k * per / NS != (k + 1) * per / NS) s += p[pass][k];
            s += hb[(pass == 2 ? o.n_bias : 0) + c];
            out.z[pass] = s;
            if (BACK && lane < A && j < a.B) a.Q[((size_t)pass * a.B + j) * a.ldq + lane] = s;
        }
        return out;
    };

    if constexpr (KIND == TJ_ROWS_ACT) {
        for (int row = wave; row < R && j0 + row < a.B; row += kWaves) act_row(a, mode, j0 + row, A, head_out(row).z[0]);
        return;
    }

    // ---- the objective: one wave per transition, one lane per head output
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int row = wave + i * kWaves;
        const bool valid = j0 + row < a.B;
        act_w[i] = __builtin_amdgcn_readfirstlane(min(max(act_w[i], 0), A - (DQN ? 1 : 2)));
        const Out out = head_out(row);
        float g;
        if constexpr (DQN) {
            const TdRow t = td_row(a, A, out.z[0], out.z[1], out.z[2], act_w[i], rew_w[i], done_w[i] ? 0.f : 1.f, valid);
            if (lane == 0) {
                sm[row] = t.loss;
                if (valid) a.astar[j0 + row] = t.best;
            }
            g = lane == act_w[i] ? t.g : 0.f;
        } else {
            const PpoRow t = ppo_row(a, A - 1, out.z[0], act_w[i], olp_w[i], adv_w[i], ret_w[i], valid);
            if (lane == 0) { sm[row] = t.pi; sm[R + row] = t.v; sm[2 * R + row] = t.H; }
            g = t.g;
        }
        *(tj_bf16 *)(dzb + row * kZPitch + 2 * lane) = __builtin_bit_cast(tj_bf16, (__bf16)g);
    }

    for (int l = 1; l < L; ++l) put_frags(keep(l), P, a.lay[l].in, a.lay[l].XF);
    block_sync_lds();
    // ---- input gradients: layer l's input rows are replaced by relu'(X_l) (dZ_l W_l)
    for (int l = last; l >= 1; --l) {
        const int pz = l == last ? kZPitch : P;
        const uint8_t *z = (l == last ? dzb : keep(l + 1)) + n16 * pz + 16 * q;
        uint8_t *const x = keep(l);
        stream(ph, [&](const u32x4 (&w)[4], int kg, int) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int g = 0; g < NR; ++g) {
                    const u32x4 v = *(const u32x4 *)(z + 16 * g * pz + kg * 128 + 64 * s);
#pragma unroll
                    for (int t = 0; t < 2; ++t) acc[t][g] = mma(w[2 * t + s], v, acc[t][g]);
                }
        }, [&](int item) {
            const int f = wave + kWaves * item;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int g = 0; g < NR; ++g) {
                    uint2 *d = (uint2 *)(x + (16 * g + n16) * P + 64 * f + 32 * t + 8 * q);
                    const uint2 m = *d;
                    auto on = [](uint32_t w, int hi) { return __uint_as_float(hi ? w & 0xFFFF0000u : w << 16) > 0.f; };
                    const f32x4 v = acc[t][g];
                    *d = make_uint2(pack2(on(m.x, 0) ? v[0] : 0.f, on(m.x, 1) ? v[1] : 0.f),
                                    pack2(on(m.y, 0) ? v[2] : 0.f, on(m.y, 1) ? v[3] : 0.f));
                }
            clear();
        });
        if (l > 1) { ph = mine(args.bwd[l - 1], false); load(wa, ph); }
        block_sync_lds();
    }
    if (wave == 0) {   // the block's sums, in a fixed order
#pragma unroll
        for (int k = 0; k < (DQN ? 1 : 3); ++k) {
            const float s = wave_sum(lane < R ? sm[R * k + lane] : 0.f);
            if (lane == 0) a.loss_part[DQN ? (size_t)blockIdx.x : (size_t)blockIdx.x * 4 + k] = s;
        }
    }
    put_frags(dzb, kZPitch, A, a.lay[last].ZF);
    for (int l = 1; l < L; ++l) put_frags(keep(l), P, a.lay[l].in, a.lay[l - 1].ZF);
}

// ---------------------------------------------------------------- weights

// dW[n][k] = sum_m dZ[m][n] X[m][k] over the batch: both operands are stored as fragments, so they go from memory
// into the matrix instruction; the waves of a block split the 32-row steps of the batch and their sums meet in LDS.
//   32 x 32 tiles, sixteen waves, Adam in the same block: short batches, where the kernel is a chain of latencies.
//   64 x 64 tiles, eight waves: half the operand traffic per weight, which bounds long batches; the batch is cut into
//     slices so that the tiles fill the chip, and b16_adam adds them.
// The bias gradient is one more product, with a fragment of ones.
using UpdatePlan = tjplan::B16Update;

__device__ __forceinline__ u32x4 frag(const tj_bf16 *F, int fp, int ms, int step, int t, int lane)
{
    return *(const u32x4 *)(F + (((size_t)fp * ms + step) * 2 + t) * 512 + lane * 8);
}

// After Adam: the copies of a 32 x 32 tile.  tile: [32 n][40] bf16, zero outside the matrix.
__device__ __forceinline__ void emit_copies(const TjB16Update &a, const TjB16Layer &y, int l, int n0, int k0,
                                            const tj_bf16 *tile, int tid)
{
    const int lane = tid & 63, t = (tid >> 6) & 1, r = lane & 15, c8 = 8 * (lane >> 4);
    if (tid < 128) {
        const u32x4 v = *(const u32x4 *)(tile + (16 * t + r) * 40 + c8);
        const size_t at = tj_b16_group_off(n0 + 16 * t + r, k0 + c8, (y.in + 63) / 64);
        *(u32x4 *)(y.WF + at) = v;
        if (a.sync_target) *(u32x4 *)(y.WF + (size_t)((y.out + 31) / 32) * ((y.in + 63) / 64) * 2048 + at) = v;
    } else if (tid < 256 && l > 0) {
        u32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = (uint32_t)tile[(c8 + 2 * e) * 40 + 16 * t + r] | (uint32_t)tile[(c8 + 2 * e + 1) * 40 + 16 * t + r] << 16;
        *(u32x4 *)(y.WB + tj_b16_group_off(k0 + 16 * t + r, n0 + c8, (y.out + 63) / 64)) = v;
    }
}

template <int TILE>
__global__ __launch_bounds__(TILE == 32 ? 1024 : 512) void b16_update(const TjB16Update a, const UpdatePlan plan)
{
    constexpr int W = TILE == 32 ? 16 : 8;          // waves
    constexpr int NT = TILE / 16;                   // 16-wide tiles per side
    constexpr int U = 2;                            // steps of a set of loads
    {
        uint32_t t = 0;
#pragma unroll
        for (size_t i = 0; i < sizeof(a); i += 64) t ^= ((const uint32_t *)&a)[i / 4];
        asm volatile("" ::"s"(t));
    }
    extern __shared__ __align__(16) float red[];    // [wave][row tile, column tile, register][lane]; bias: [wave][TILE]
    float *const redb = red + W * NT * NT * 4 * 64;
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_tile = plan.begin[a.L];
    if (TILE == 32 && (int)blockIdx.x == n_tile) { step_stats<1024>(a, red); return; }
    // An XCD (block % 8) takes a run of the slice-major order: it reads few slices' rows.
    const int id = TILE == 64 ? (int)(blockIdx.x & 7) * (int)(gridDim.x / 8) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int z = TILE == 64 ? id / n_tile : 0, tile_id = id - z * n_tile;
    if (z >= plan.S) return;
    int l = 0;
    while (l + 1 < a.L && tile_id >= plan.begin[l + 1]) ++l;
    const TjB16Layer &y = a.lay[l];
    const int t = tile_id - plan.begin[l], k0 = (t % plan.nk[l]) * TILE, n0 = (t / plan.nk[l]) * TILE;
    const bool with_bias = k0 == 0;

    f32x4 acc[NT][NT], accb[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    const int s1 = min(plan.steps, (z + 1) * plan.per);
    // a tile's second group of 32 features may lie past the layer: the last one is read again and not used
    const int zmax = (y.out - 1) / 32, xmax = (y.in - 1) / 32;
    u32x4 fa[U][2 * NT], fb[U][2 * NT];   // two sets of U steps, the next in flight while one is multiplied
    auto fetch = [&](u32x4 (&f)[U][2 * NT], int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int su = min(s + W * u, s1 - 1);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                f[u][i] = frag(y.ZF, min(n0 / 32 + i / 2, zmax), plan.steps, su, i & 1, lane);
                f[u][NT + i] = frag(y.XF, min(k0 / 32 + i / 2, xmax), plan.steps, su, i & 1, lane);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](const u32x4 (&f)[U][2 * NT], int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s + W * u >= s1) break;
#pragma unroll
            for (int i = 0; i < NT; ++i) {
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = mma(f[u][i], f[u][NT + j], acc[i][j]);
                if (with_bias) accb[i] = mma(f[u][i], ones, accb[i]);
            }
        }
    };
    int s = z * plan.per + wave;
    if (s < s1) {
        constexpr int D = W * U;
        fetch(fa, s);
        for (; s + 2 * D < s1; s += 2 * D) {
            fetch(fb, s + D); mul(fa, s);
            fetch(fa, s + 2 * D); mul(fb, s + D);
        }
        if (s + D < s1) { fetch(fb, s + D); mul(fa, s); mul(fb, s + D); }
        else mul(fa, s);
    }
    // this thread's weights: accumulator register r of tile pair (i, j): row n = n0 + 16 i + 4 q + r, column k0 + 16 j + c16
    constexpr int NV = TILE == 32 ? 1 : 8;
    auto slot = [&](int v) { return (tid >> 6) + W * v; };   // (i NT + j) 4 + r
    auto n_of = [&](int v) { return n0 + 16 * (slot(v) / 4 / NT) + 4 * q + (slot(v) & 3); };
    auto k_of = [&](int v) { return k0 + 16 * (slot(v) / 4 % NT) + c16; };
    const int nb = n0 + tid;
    const bool bias_thread = with_bias && tid < TILE && nb < y.out;
    AdamState st = {0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f};
    const bool in0 = n_of(0) < y.out && k_of(0) < y.in;
    if constexpr (TILE == 32) {   // in flight during the exchange below
        if (in0) {
            const size_t at = (size_t)n_of(0) * y.in + k_of(0);
            st = {y.W[at], a.m[y.w_off + at], a.v[y.w_off + at]};
        }
        if (bias_thread) sb = {y.bias[nb], a.m[y.b_off + nb], a.v[y.b_off + nb]};
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[((wave * NT * NT + i * NT + j) * 4 + r) * 64 + lane] = acc[i][j][r];
        if (with_bias && c16 == 0) *(f32x4 *)(redb + wave * TILE + 16 * i + 4 * q) = accb[i];
    }
    __syncthreads();
    float g[NV], gb = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        g[v] = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) g[v] += red[(w * NT * NT * 4 + slot(v)) * 64 + lane];
    }
    if (bias_thread)
        for (int w = 0; w < W; ++w) gb += redb[w * TILE + tid];

    if constexpr (TILE == 64) {   // a slice of the gradient, in the order of the parameters
        float *out = a.slices + (size_t)z * a.slice_stride;
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (n_of(v) < y.out && k_of(v) < y.in) out[y.w_off + (size_t)n_of(v) * y.in + k_of(v)] = g[v];
        if (bias_thread) out[y.b_off + nb] = gb;
    } else {
        __syncthreads();   // the sums have been read
        tj_bf16 *tile = (tj_bf16 *)red;
        const AdamState x = adam(a, st, g[0]);
        tile[(n_of(0) - n0) * 40 + k_of(0) - k0] = in0 ? __builtin_bit_cast(tj_bf16, (__bf16)x.th) : (tj_bf16)0;
        if (in0) {
            const size_t at = (size_t)n_of(0) * y.in + k_of(0), off = y.w_off + at;
            y.W[at] = x.th; a.m[off] = x.m; a.v[off] = x.v; a.g[off] = g[0];
            if (a.sync_target) y.W_tg[at] = x.th;
        }
        if (bias_thread) {
            const AdamState b = adam(a, sb, gb);
            y.bias[nb] = y.BP[nb] = b.th; a.m[y.b_off + nb] = b.m; a.v[y.b_off + nb] = b.v; a.g[y.b_off + nb] = gb;
            if (a.sync_target) y.bias_tg[nb] = y.BP_tg[nb] = b.th;
        }
        __syncthreads();
        emit_copies(a, y, l, n0, k0, tile, tid);
    }
}

// Second half of an update whose gradient came in slices: their sum in slice order, Adam, the copies.  A block owns
// 32 x 32 weights, a thread two of them; every load is issued before the first use.
__global__ __launch_bounds__(512) void b16_adam(const TjB16Update a, const UpdatePlan plan)
{
    __shared__ __align__(16) tj_bf16 tile[32 * 40];
    const int tid = threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) { step_stats<512>(a, (float *)tile); return; }
    int l = 0;
    while (l + 1 < a.L && (int)blockIdx.x >= plan.begin[l + 1]) ++l;
    const TjB16Layer &y = a.lay[l];
    const int t = (int)blockIdx.x - plan.begin[l], k0 = (t % plan.nk[l]) * 32, n0 = (t / plan.nk[l]) * 32;
    const int kl = tid & 31, nl = tid >> 5, nb = n0 + tid;
    size_t at[3];
    bool in[3];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int n = n0 + nl + 16 * v;
        in[v] = n < y.out && k0 + kl < y.in;
        at[v] = in[v] ? y.w_off + (size_t)n * y.in + k0 + kl : y.w_off;
    }
    in[2] = k0 == 0 && tid < 32 && nb < y.out;
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
        if (v < 2) tile[(nl + 16 * v) * 40 + kl] = in[v] ? __builtin_bit_cast(tj_bf16, (__bf16)x.th) : (tj_bf16)0;
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
    emit_copies(a, y, l, n0, k0, tile, tid);
}

// Fragments from the master parameters, one thread per weight (creation and set_state only).
__global__ __launch_bounds__(256) void b16_cast(const TjB16Layer y, const int online, const int with_wb)
{
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    const float *W = online ? y.W : y.W_tg, *b = online ? y.bias : y.bias_tg;
    if (e < (size_t)y.in * y.out) {
        const int n = (int)(e / y.in), k = (int)(e % y.in), kp = (y.in + 63) / 64;
        const tj_bf16 v = __builtin_bit_cast(tj_bf16, (__bf16)W[e]);
        y.WF[(online ? 0 : (size_t)((y.out + 31) / 32) * kp * 2048) + tj_b16_group_off(n, k, kp)] = v;
        if (with_wb) y.WB[tj_b16_group_off(k, n, (y.out + 63) / 64)] = v;
    }
    if (e < (size_t)y.out) (online ? y.BP : y.BP_tg)[e] = b[e];
}

int rows_nr(const TjB16Rows &a, int mode)
{
    return tjplan::b16_groups(a.L, a.lay, a.B, mode == TJ_ROWS_DQN, mode == TJ_ROWS_DQN || mode == TJ_ROWS_PPO);
}

int grid_of(int B, int nr, bool back) { return back && nr == 1 ? (B + 31) / 32 * 2 : (B + 16 * nr - 1) / (16 * nr); }

template <int KIND, int NR> int launch_rows(const TjB16Rows &a, int mode, hipStream_t st)
{
    constexpr bool dqn = KIND == TJ_ROWS_DQN, back = KIND != TJ_ROWS_ACT;
    static bool attr_set = false;   // idempotent: a race sets it twice
    if (!attr_set) {
        TJ_HIP_TRY(hipFuncSetAttribute((const void *)b16_rows<KIND, NR>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
        attr_set = true;
    }
    RowsArgs r;
    r.a = a;
    r.o = tjplan::b16_lds(a.L, a.lay, NR, dqn, back);
    r.ms = (a.B + 31) / 32;
    for (int l = 0; l < TJ_MAX_LAYERS; ++l) {
        const TjB16Layer &y = a.lay[l < a.L ? l : 0];
        r.fwd[l] = {y.WF, (y.out + 31) / 32 * (dqn ? 2 : 1), (y.in + 63) / 64};
        r.bwd[l] = {y.WB, (y.in + 31) / 32, (y.out + 63) / 64};
    }
    b16_rows<KIND, NR><<<grid_of(a.B, NR, back), kThreads, r.o.total, st>>>(r, mode);
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}

}  // namespace

bool tj_b16_fits(int L, const int *in, const int *out, int passes, int max_batch) { return tjplan::b16_fits(L, in, out, passes, max_batch); }

int tj_b16_blocks(const TjB16Rows &a, int mode)
{
    return grid_of(a.B, rows_nr(a, mode), mode == TJ_ROWS_DQN || mode == TJ_ROWS_PPO);
}

int tj_b16_rows(const TjB16Rows &a, int mode, hipStream_t st)
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

int tj_b16_slices(int L, const TjB16Layer *lay, int B) { return tjplan::b16_slices(L, lay, B); }

int tj_b16_update(const TjB16Update &a, hipStream_t st)
{
    if (a.B < 1 || a.L < 1 || a.L > TJ_MAX_LAYERS) return TJ_ERR_SHAPE;
    static bool attr_set = false;
    if (!attr_set) {
        TJ_HIP_TRY(hipFuncSetAttribute((const void *)b16_update<32>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
        TJ_HIP_TRY(hipFuncSetAttribute((const void *)b16_update<64>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
        attr_set = true;
    }
    UpdatePlan p;
    const int tile = tjplan::b16_update(a.L, a.lay, a.B, p), n = p.begin[a.L];
    if (tile == 32) {
        b16_update<32><<<n + 1, 1024, 16 * 32 * 32 * 4 + 16 * 32 * 4, st>>>(a, p);
    } else {
        b16_update<64><<<up(n * p.S, 8), 512, 8 * 64 * 64 * 4 + 8 * 64 * 4, st>>>(a, p);
        b16_adam<<<tjplan::b16_tiles(a.L, a.lay, 32, p) + 1, 512, 0, st>>>(a, p);
    }
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}

int tj_b16_cast(int L, const TjB16Layer *lay, bool online, hipStream_t st)
{
    for (int l = 0; l < L; ++l) {
        const size_t n = std::max((size_t)lay[l].in * lay[l].out, (size_t)lay[l].out);
        b16_cast<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(lay[l], online ? 1 : 0, online && l > 0);
    }
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}
