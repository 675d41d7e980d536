// What the kernels that run a whole vector network per block (tj_mlp_f32.hip, tj_mlp_b16.hip) have in common: the
// description of a call, the arithmetic of one transition's objective and of one weight's update.
#pragma once
#include "tj_common.h"
#include <math.h>

enum { TJ_ROWS_DQN = 0, TJ_ROWS_ACT = 1, TJ_ROWS_PPO = 2, TJ_ROWS_POLICY = 3, TJ_ROWS_EVAL = 4 };

// All per-row work of one call.
struct TjRowsCall {
    int L, B;
    const float *obs, *next_obs;     // rows of the first layer's input width
    const uint32_t *rows;            // optional: row j is table row min(rows[j], n_rows - 1)
    uint32_t n_rows;
    // Q-learner step
    const int32_t *action;           // also the on-policy step
    const float *reward;
    const uint8_t *done;
    float gamma, kappa;
    float *Q; int ldq;               // [3B][ldq] (on-policy step: [B][ldq]); may be null when acting
    int32_t *astar;
    float *loss_part;                // one per block; on-policy: four per block
    // on-policy step
    const float *old_logp, *adv, *ret;
    float clip, c_v, c_e;
    // acting (A = Q-network's outputs, or the policy's logits with the value behind them)
    uint32_t threshold;
    uint64_t seed;
    int32_t version;
    int32_t *action_out, *version_out;
    float *q_out, *logp_out, *value_out;   // q_out: [B][A]
};

// Everything per weight of one update.
struct TjUpdateCall {
    int L, B;
    float *m, *v, *g;                // flat, as the parameters
    float *slices;                   // gradient slices of the batch, slice_stride floats apart
    size_t slice_stride;
    float b1, b2, eps, lr1, rc2;     // lr1 = lr / (1 - b1^t), rc2 = 1 / (1 - b2^t)
    int sync_target;                 // also write the target network (parameters and copies)
    // statistics of the step, from the row kernel's per-block sums
    const float *part;
    int n_part, ppo;
    uint32_t t_next;
    tj_step_stats *stats, *stats_internal;
    float c_v, c_e;
    tj_ppo_stats *ppo_stats, *ppo_internal;
};

// A wave-uniform stretch of memory; loads at or past its end are zeros and touch nothing.
typedef __amdgpu_buffer_rsrc_t buf_rsrc;
__device__ __forceinline__ buf_rsrc buf_of(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, bytes, 0x00027000);
}
__device__ __forceinline__ float load4(buf_rsrc r, int at) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0)); }

// Orders LDS accesses across the block without waiting for global loads: those in flight belong to the next
// layer (a __syncthreads() may drain them).
__device__ __forceinline__ void block_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Reductions over the wave with lane moves that stay in the vector unit.
template <int CTRL> __device__ __forceinline__ float dpp(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
template <typename OP> __device__ __forceinline__ float wave_reduce(float v, OP op)
{
    v = op(v, dpp<0x128>(v));   // rotations by 8, 4, 2, 1 inside a row of 16 lanes
    v = op(v, dpp<0x124>(v));
    v = op(v, dpp<0x122>(v));
    v = op(v, dpp<0x121>(v));
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float wave_sum(float v) { return wave_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }
// lowest lane that holds the maximum; as a scan that starts with lane 0 and goes by ">": a NaN in lane 0 stays, others lose
__device__ __forceinline__ int wave_argmax(float v)
{
    if (__ballot(v != v) & 1) return 0;
    const unsigned long long m = __ballot(v == wave_max(v));
    return m ? __ffsll((long long)m) - 1 : 0;
}

// The value that one lane of the wave holds; `lane` is the same on all of them.
__device__ __forceinline__ float lane_value(float v, int lane) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane)); }

// The objective of transition j, by one wave with one lane per head output (lanes from A on hold anything); act is the same on all
// lanes; `valid` is false for rows past the batch.
struct TdRow { float loss, g; int best; };   // g = dL/dQ(s, action)
__device__ __forceinline__ TdRow td_row(const TjRowsCall &a, int A, float q_s, float q_next, float q_next_tg, int act, float reward, float not_done, bool valid)
{
    const int lane = threadIdx.x & 63;
    TdRow t;
    t.best = wave_argmax(lane < A ? q_next : -INFINITY);
    const float target = reward + a.gamma * not_done * lane_value(q_next_tg, t.best);
    const float d = lane_value(q_s, act) - target, ad = fabsf(d);
    t.g = valid ? fminf(fmaxf(d, -a.kappa), a.kappa) / (float)a.B : 0.f;
    t.loss = !valid ? 0.f : ad <= a.kappa ? 0.5f * d * d : a.kappa * (ad - 0.5f * a.kappa);
    return t;
}

struct PpoRow { float pi, v, H, g; };        // g: this lane's dL/dz
__device__ __forceinline__ PpoRow ppo_row(const TjRowsCall &a, int n, float zs, int act, float old_logp, float adv,
                                          float ret, bool valid)
{
    const int lane = threadIdx.x & 63;
    const float z = lane <= n ? zs : 0.f;
    const float mx = wave_max(lane < n ? z : -INFINITY);
    const float lse = mx + logf(wave_sum(lane < n ? expf(z - mx) : 0.f));
    const float lp = z - lse, pk = lane < n ? expf(lp) : 0.f;
    PpoRow r;
    r.H = wave_sum(lane < n ? -pk * lp : 0.f);
    const float rho = expf(lane_value(zs, act) - lse - old_logp);
    const float rc = fminf(fmaxf(rho, 1.f - a.clip), 1.f + a.clip);
    const float s1 = rho * adv, s2 = rc * adv;
    const bool unclipped = s1 <= s2;   // the minimum is the unclipped term: it carries the gradient
    const float verr = lane_value(zs, n) - ret, inv_b = 1.f / (float)a.B;
    r.g = 0.f;
    if (lane < n) {
        r.g = a.c_e * pk * (lp + r.H);
        if (unclipped) r.g -= adv * rho * ((lane == act ? 1.f : 0.f) - pk);
        r.g *= inv_b;
    } else if (lane == n) {
        r.g = 2.f * a.c_v * verr * inv_b;
    }
    if (!valid) r.g = 0.f;
    r.pi = valid ? -(unclipped ? s1 : s2) : 0.f;
    r.v = valid ? verr * verr : 0.f;
    if (!valid) r.H = 0.f;
    return r;
}

// What acting does with the head outputs of observation j (A of them, one per lane), by one wave.
__device__ __forceinline__ void act_row(const TjRowsCall &a, int mode, int j, int A, float zs)
{
    const int lane = threadIdx.x & 63;
    const float z = lane < A ? zs : 0.f;
    if (mode == TJ_ROWS_ACT) {
        const int best = wave_argmax(lane < A ? z : -INFINITY);
        if (a.q_out && lane < A) a.q_out[(size_t)j * A + lane] = z;
        if (lane == 0) {
            const uint64_t u = tj_splitmix64(a.seed, 2 * (uint64_t)j), v = tj_splitmix64(a.seed, 2 * (uint64_t)j + 1);
            a.action_out[j] = (uint32_t)(u >> 40) < a.threshold ? (int32_t)__umul64hi(v, (uint64_t)A) : best;
            a.version_out[j] = a.version;
        }
        return;
    }
    const int n = A - 1;              // logits, then the value
    if (a.value_out && lane == n) a.value_out[j] = z;
    if (mode == TJ_ROWS_EVAL) {
        if (a.q_out && lane < n) a.q_out[(size_t)j * n + lane] = z;
        return;
    }
    const float mx = wave_max(lane < n ? z : -INFINITY);
    const float lse = mx + logf(wave_sum(lane < n ? expf(z - mx) : 0.f));
    float cdf = lane < n ? expf(z - lse) : 0.f;
    for (int d = 1; d < n; d <<= 1) {
        const float below = __shfl_up(cdf, d, 64);
        if (lane >= d) cdf += below;
    }
    const float u = (float)(tj_splitmix64(a.seed, j) >> 40) * (1.f / 16777216.f);
    const unsigned long long past = __ballot(lane < n && cdf > u);
    const int pick = past ? __ffsll((long long)past) - 1 : n - 1;
    if (lane == pick) { a.action_out[j] = pick; a.logp_out[j] = z - lse; }
}

// Adam (bias-corrected, eps outside the square root); lr1 = lr / c1 and rc2 = 1 / c2 come rounded from double
struct AdamState { float th, m, v; };
__device__ __forceinline__ AdamState adam(const TjUpdateCall &a, AdamState s, float g)
{
    s.m = a.b1 * s.m + (1.f - a.b1) * g;
    s.v = a.b2 * s.v + (1.f - a.b2) * g * g;
    s.th -= a.lr1 * s.m / (sqrtf(s.v * a.rc2) + a.eps);
    return s;
}

// The step's statistics from the row kernel's per-block sums, in a fixed order, by a block of its own (THREADS; up to
// 2048 sums: one wave of another block's threads took 20 us for them, one latency after the other).
template <int THREADS> __device__ __forceinline__ void step_stats(const TjUpdateCall &a, float *lds)
{
    const int tid = threadIdx.x, stride = a.ppo ? 4 : 1, nq = a.ppo ? 3 : 1;
    float q[3] = {0.f, 0.f, 0.f};
    for (int b = tid; b < a.n_part; b += THREADS)
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < nq) q[i] += a.part[(size_t)b * stride + i];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        q[i] = wave_sum(q[i]);
        if ((tid & 63) == 0) lds[i * 16 + (tid >> 6)] = q[i];
    }
    __syncthreads();
    if (tid >= 64) return;
#pragma unroll
    for (int i = 0; i < 3; ++i) q[i] = wave_sum(tid < THREADS / 64 ? lds[i * 16 + tid] : 0.f);
    if (tid != 0) return;
    if (a.ppo) {
        tj_ppo_stats o;
        o.loss_pi = q[0] / (float)a.B;
        o.loss_v = q[1] / (float)a.B;
        o.entropy = q[2] / (float)a.B;
        o.loss = o.loss_pi + a.c_v * o.loss_v - a.c_e * o.entropy;
        o.step = a.t_next;
        *a.ppo_internal = o;
        if (a.ppo_stats) *a.ppo_stats = o;
    } else {
        tj_step_stats o;
        o.loss = q[0] / (float)a.B;
        o.step = a.t_next;
        *a.stats_internal = o;
        if (a.stats) *a.stats = o;
    }
}
