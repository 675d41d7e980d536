// The three convolutions of a pixel Q-network (8x8 -> 32 channels, 4x4 / 2 -> 64, 3x3 -> 64) as one kernel, straight
// from the u8 frame stacks: the forward passes of an update and the network's lower part when acting.
//
// A block per compute unit takes a run of passes (an image under one network's weights) through all three layers; what lies
// between the layers stays in LDS.  As launches of their own the layers are bound by their fixed part at small batches (10 us each
// for 256 images) and by gathered operand reads and 200 MB of activations that nobody reads again at large ones (only s under
// the online weights is needed by the backward pass).
//   first layer   32 patches x 32 channels per wave, both operands from LDS, as in tj_conv_first.hip;
//   second, third 16 x 16 x 32 MFMAs, a = 16 channels of weights, b = 16 patches out of LDS.  The weights live in registers
//                 for the whole run: a wave has 16 of the 64 channels and half of the patches (64 + 72 registers of the
//                 256 that eight waves leave each).  Every sum runs over its whole contraction in one accumulator, in the order of
//                 the gathered GEMMs (one 16 x 16 x 32 step adds in the order of two 32 x 32 x 16 steps: checked bit for bit), so
//                 that greedy actions do not move between this kernel and those.
// Rows of the activations in LDS are padded by 16 bytes: 80 and 144 bytes apart, 16 consecutive patches read 16 distinct 16-byte
// columns.  The second layer has stride 2, so its input keeps even and odd columns apart, which makes consecutive patches
// consecutive rows.
// While an image is in the second layer the next one, fetched into registers a layer ahead, is converted into the image buffer.
#include "tj_conv_planes.h"

namespace {

using namespace tjplanes;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 512, kWaves = 8;
constexpr int K1 = 8, C1 = 32, K2 = 4, S2 = 2, C2 = 64, K3 = 3, C3 = 64;   // kernels, strides, output channels
constexpr int kRounds = 4;              // 4-pixel tasks per thread and image
constexpr int kTiles2 = 3, kTiles3 = 2; // tiles of 16 patches per wave (two waves share the patches)
constexpr int kSteps2 = K2 * K2 * C1 / 32, kSteps3 = K3 * K3 * C2 / 32;   // 32-value steps of a contraction
constexpr int kRow1 = C1 * 2 + 16, kRow2 = C2 * 2 + 16;   // bytes between activation rows in LDS
constexpr int kW1Pitch = (4 * K1 * K1 + 8) * 2;           // ... between the first layer's weight rows
constexpr size_t kLdsLimit = 160 * 1024;

struct TowerPlan {
    int w1, out1, out2, bias, total;   // byte offsets in LDS (the image is at 0)
    int half1, pitch1;                       // columns per parity of the first layer's output, rows of LDS per image row
    uint32_t mg_ow1, mg_ow2, mg_ow3;         // ceil(2^32 / OW)
    int n_pass;
};

__host__ __device__ inline uint32_t magic(int d) { return (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

TowerPlan tower_plan(int H, int W, int OH1, int OW1, int OH2, int OW2, int OW3)
{
    TowerPlan p;
    p.half1 = (OW1 + S2 - 1) / S2;
    p.pitch1 = S2 * p.half1;
    int at = H * W * 8;
    p.w1 = at; at += C1 * kW1Pitch;
    p.out1 = at; at += OH1 * p.pitch1 * kRow1;
    p.out2 = at; at += OH2 * OW2 * kRow2;
    p.bias = at; at += (C1 + C2 + C3) * 4;
    p.total = at;
    p.mg_ow1 = magic(OW1); p.mg_ow2 = magic(OW2); p.mg_ow3 = magic(OW3);
    p.n_pass = 0;
    return p;
}

// Orders LDS accesses across the block; global loads (the next image) and stores stay in flight.
__device__ __forceinline__ void lds_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void conv_tower(const TjConvTowerArgs a, const TowerPlan p)
{
    extern __shared__ __align__(16) uint8_t lds[];
    uint8_t *const img = lds, *const w1 = lds + p.w1, *const out1 = lds + p.out1, *const out2 = lds + p.out2;
    float *const bias = (float *)(lds + p.bias);
    const TjConvFirstArgs &f = a.first;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5, l16 = lane & 15, q4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ct = wave & 3, rh = wave >> 2;
    const int HW = f.H * f.W, W = f.W, OHW1 = f.OH * f.OW, OHW2 = a.OH2 * a.OW2, OHW3 = a.OH3 * a.OW3;
    const int begin = (int)((long)blockIdx.x * p.n_pass / gridDim.x), end = (int)((long)(blockIdx.x + 1) * p.n_pass / gridDim.x);
    if (begin >= end) return;

    // ---- images.  Unit = 16 bytes of LDS = two pixels; the units of odd groups of 16 are exchanged in pairs, so that the 16
    // patches an operand read touches (every other unit) fall on 16 distinct units of a 256-byte line
    const int n_task = HW / 4;
    uint32_t px[kRounds][4];
    auto fetch = [&](int pass) {
        const int g = pass < 2 * f.B ? pass : pass - f.B;   // s, s', and s' again for the target network
        const bool next = g >= f.B;
        const PlaneOff off = plane_offsets(f.rows, f.planes, f.n_rows, next ? g - f.B : g, next, HW);
        const uint8_t *src = next ? f.next_obs : f.obs;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int t = tid + r * kThreads;
            if (t < n_task) {
#pragma unroll
                for (int c = 0; c < 4; ++c) px[r][c] = *(const uint32_t *)(src + off.o[c] + 4 * t);
            }
        }
    };
    auto convert = [&]() {
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int t = tid + r * kThreads;
            if (t < n_task) {
                u32x4 v[2];
#pragma unroll
                for (int q = 0; q < 4; ++q) {     // pixel 4t + q: channels 0..3
                    float x[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) x[c] = (float)((px[r][c] >> (8 * q)) & 0xFF) * f.scale;
                    v[q >> 1][2 * (q & 1)] = pack2(x[0], x[1]);
                    v[q >> 1][2 * (q & 1) + 1] = pack2(x[2], x[3]);
                }
                uint8_t *dst = img + (size_t)t * 32;
                const int swap = (t >> 3) & 1;
                *(u32x4 *)(dst + 16 * swap) = v[0];
                *(u32x4 *)(dst + 16 * (swap ^ 1)) = v[1];
            }
        }
    };

    // ---- weights of one network
    u32x4 w2[kSteps2], w3[kSteps3];
    auto load_net = [&](int net) {
        const tj_bf16 *W2 = (net ? a.W2_tg : a.W2_on) + (size_t)(16 * ct + l16) * (K2 * K2 * C1) + 8 * q4;
        const tj_bf16 *W3 = (net ? a.W3_tg : a.W3_on) + (size_t)(16 * ct + l16) * (K3 * K3 * C2) + 8 * q4;
#pragma unroll
        for (int i = 0; i < kSteps2; ++i) w2[i] = *(const u32x4 *)(W2 + 32 * i);
#pragma unroll
        for (int i = 0; i < kSteps3; ++i) w3[i] = *(const u32x4 *)(W3 + 32 * i);
        constexpr int VR = 4 * K1 * K1 / 8;   // 16-byte vectors per row of the first layer's weights
        for (int v = tid; v < C1 * VR; v += kThreads)
            *(u32x4 *)(w1 + (v / VR) * kW1Pitch + (v % VR) * 16) = *(const u32x4 *)((net ? f.W_tg : f.W_on) + (size_t)v * 8);
        if (tid < C1) bias[tid] = (net ? f.b_tg : f.b_on)[tid];
        else if (tid < C1 + C2) bias[tid] = (net ? a.b2_tg : a.b2_on)[tid - C1];
        else if (tid < C1 + C2 + C3) bias[tid] = (net ? a.b3_tg : a.b3_on)[tid - C1 - C2];
    };

    fetch(begin);
    int net = begin >= 2 * f.B;
    load_net(net);
    convert();
    if (begin + 1 < end) fetch(begin + 1);

    // where this wave's patches start in the activations of the layer below (tiles past the last patch repeat it)
    int at2[kTiles2], at3[kTiles3];
#pragma unroll
    for (int i = 0; i < kTiles2; ++i) {
        const uint32_t m = min((rh * kTiles2 + i) * 16 + l16, OHW2 - 1), oh = __umulhi(m, p.mg_ow2), ow = m - oh * a.OW2;
        at2[i] = (oh * S2 * p.pitch1 + ow) * kRow1 + 16 * q4;
    }
#pragma unroll
    for (int i = 0; i < kTiles3; ++i) {
        const uint32_t m = min((rh * kTiles3 + i) * 16 + l16, OHW3 - 1), oh = __umulhi(m, p.mg_ow3), ow = m - oh * a.OW3;
        at3[i] = (oh * a.s3 * a.OW2 + ow * a.s3) * kRow2 + 16 * q4;
    }
    auto row1 = [&](uint32_t m) -> uint8_t * {   // patch m of the first layer's output
        const uint32_t oh = __umulhi(m, p.mg_ow1), ow = m - oh * f.OW;
        return out1 + (oh * p.pitch1 + (ow & 1) * p.half1 + (ow >> 1)) * kRow1;
    };

    for (int pass = begin; pass < end; ++pass) {
        if ((pass >= 2 * f.B) != net) {   // the run goes on with the target network
            lds_sync();
            net = 1;
            load_net(net);
        }
        lds_sync();   // the image and the first layer's weights are in place; the last pass is out of out1

        // ---- first layer: image -> out1
        const int n_tile = (OHW1 + 31) / 32;
        for (int tile = wave; tile < n_tile; tile += 2 * kWaves) {   // two tiles share the weight reads
            const bool two = tile + kWaves < n_tile;
            int unit[2];
            uint8_t *dst[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint32_t m = min(32 * (tile + t * kWaves) + l32, OHW1 - 1), oh = __umulhi(m, p.mg_ow1), ow = m - oh * f.OW;
                unit[t] = (int)(oh * f.s * W + ow * f.s) / 2 + h;
                dst[t] = row1(m) + 8 * h;
            }
            f32x16 acc[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
#pragma unroll 2
            for (int kh = 0; kh < K1; ++kh) {
#pragma unroll
                for (int kw0 = 0; kw0 < K1; kw0 += 4) {   // 16 contraction values: 4 pixels x 4 channels
                    const u32x4 wv = *(const u32x4 *)(w1 + l32 * kW1Pitch + ((kh * K1 + kw0) * 4 + 8 * h) * 2);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (t == 1 && !two) continue;
                        const int u = unit[t] + (kh * W + kw0) / 2;
                        const u32x4 pv = *(const u32x4 *)(img + (u ^ ((u >> 4) & 1)) * 16);
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wv), __builtin_bit_cast(bf16x8, pv),
                                                                         acc[t], 0, 0, 0);
                    }
                }
            }
            // acc[4q + e] = channel 8q + 4h + e of a patch; tiles past the last patch repeat it, into the same place
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t == 1 && !two) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 b = *(const f32x4 *)(bias + 8 * q + 4 * h);
                    float x[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = fmaxf(acc[t][4 * q + e] + b[e], 0.f);
                    *(uint2 *)(dst[t] + 16 * q) = make_uint2(pack2(x[0], x[1]), pack2(x[2], x[3]));
                }
            }
        }
        lds_sync();

        // ---- second layer: out1 -> out2; the image buffer takes the next image
        if (pass + 1 < end) {
            convert();
            if (pass + 2 < end) fetch(pass + 2);
        }
        const bool keep = f.out && pass < f.B;
        if (keep) {
            tj_bf16 *dst = f.out + (size_t)pass * OHW1 * C1;
            for (int v = tid; v < OHW1 * 4; v += kThreads) *(u32x4 *)(dst + (size_t)v * 8) = *(const u32x4 *)(row1(v >> 2) + (v & 3) * 16);
        }
        f32x4 acc2[kTiles2];
#pragma unroll
        for (int i = 0; i < kTiles2; ++i) acc2[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < kSteps2; ++n) {   // a step is one tap of 32 channels
            const int kh = n / K2, kw = n % K2;
            const int off = (kh * p.pitch1 + (kw % S2) * p.half1 + kw / S2) * kRow1;
#pragma unroll
            for (int i = 0; i < kTiles2; ++i) {
                const u32x4 x = *(const u32x4 *)(out1 + at2[i] + off);
                acc2[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w2[n]), __builtin_bit_cast(bf16x8, x),
                                                                  acc2[i], 0, 0, 0);
            }
        }
        {   // acc[r] = channel 16 ct + 4 q4 + r of patch l16
            const f32x4 b = *(const f32x4 *)(bias + C1 + 16 * ct + 4 * q4);
#pragma unroll
            for (int i = 0; i < kTiles2; ++i) {
                const int m = (rh * kTiles2 + i) * 16 + l16;
                const f32x4 s = acc2[i] + b;
                if (m < OHW2)
                    *(uint2 *)(out2 + m * kRow2 + (16 * ct + 4 * q4) * 2) =
                        make_uint2(pack2(fmaxf(s[0], 0.f), fmaxf(s[1], 0.f)), pack2(fmaxf(s[2], 0.f), fmaxf(s[3], 0.f)));
            }
        }
        lds_sync();

        // ---- third layer: out2 -> out
        if (keep) {
            tj_bf16 *dst = a.act2 + (size_t)pass * OHW2 * C2;
            for (int v = tid; v < OHW2 * 8; v += kThreads) *(u32x4 *)(dst + (size_t)v * 8) = *(const u32x4 *)(out2 + (v >> 3) * kRow2 + (v & 7) * 16);
        }
        f32x4 acc3[kTiles3];
#pragma unroll
        for (int i = 0; i < kTiles3; ++i) acc3[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < kSteps3; ++n) {   // a step is half a tap
            const int kh = n / 2 / K3, kw = n / 2 % K3;
            const int off = (kh * a.OW2 + kw) * kRow2 + (n & 1) * 64;
#pragma unroll
            for (int i = 0; i < kTiles3; ++i) {
                const u32x4 x = *(const u32x4 *)(out2 + at3[i] + off);
                acc3[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w3[n]), __builtin_bit_cast(bf16x8, x),
                                                                  acc3[i], 0, 0, 0);
            }
        }
        const f32x4 b3 = *(const f32x4 *)(bias + C1 + C2 + 16 * ct + 4 * q4);
#pragma unroll
        for (int i = 0; i < kTiles3; ++i) {
            const int m = (rh * kTiles3 + i) * 16 + l16;
            const f32x4 s = acc3[i] + b3;
            if (m < OHW3)
                *(uint2 *)(a.out + ((size_t)pass * OHW3 + m) * C3 + 16 * ct + 4 * q4) =
                    make_uint2(pack2(fmaxf(s[0], 0.f), fmaxf(s[1], 0.f)), pack2(fmaxf(s[2], 0.f), fmaxf(s[3], 0.f)));
        }
    }
}

}  // namespace

// The kernel's layer shapes; image, activations and weights beside one another in LDS; no more patches than the waves'
// accumulators take.
bool tj_conv_tower_fits(const TjConvShape *c)
{
    const TjConvShape &x = c[0], &y = c[1], &z = c[2];
    if (!tj_conv_first_fits(x.C, x.H, x.W, x.k, x.s, x.O) || x.k != K1) return false;
    if (y.C != C1 || y.O != C2 || y.k != K2 || y.s != S2 || z.C != C2 || z.O != C3 || z.k != K3) return false;
    if (x.H * x.W > 4 * kThreads * kRounds) return false;
    if (y.OH * y.OW > 2 * kTiles2 * 16 || z.OH * z.OW > 2 * kTiles3 * 16) return false;
    if (x.OW < 2 || y.OW < 2 || z.OW < 2) return false;   // ceil(2^32 / 1) does not fit 32 bits
    return (size_t)tower_plan(x.H, x.W, x.OH, x.OW, y.OH, y.OW, z.OW).total <= kLdsLimit;
}

int tj_conv_tower(const TjConvTowerArgs &a, hipStream_t st)
{
    const TjConvFirstArgs &f = a.first;
    const TjConvShape c[3] = {{4, f.H, f.W, C1, f.k, f.s, f.OH, f.OW}, {C1, f.OH, f.OW, C2, K2, S2, a.OH2, a.OW2},
                              {C2, a.OH2, a.OW2, C3, K3, a.s3, a.OH3, a.OW3}};
    if (!f.obs || !f.W_on || !f.b_on || !a.W2_on || !a.W3_on || !a.b2_on || !a.b3_on || !a.out) return TJ_ERR_INVALID_ARG;
    if (f.next_obs && (!f.W_tg || !f.b_tg || !a.W2_tg || !a.W3_tg || !a.b2_tg || !a.b3_tg)) return TJ_ERR_INVALID_ARG;
    if (!f.out != !a.act2 || a.s3 < 1) return TJ_ERR_INVALID_ARG;
    if (f.B < 1 || f.B > 0x20000000 / 3) return TJ_ERR_SHAPE;
    for (int l = 0; l < 3; ++l)
        if (c[l].H < c[l].k || c[l].W < c[l].k || c[l].OH != (c[l].H - c[l].k) / c[l].s + 1 || c[l].OW != (c[l].W - c[l].k) / c[l].s + 1)
            return TJ_ERR_SHAPE;
    if (!tj_conv_tower_fits(c)) return TJ_ERR_SHAPE;
    if ((((uintptr_t)f.obs | (uintptr_t)f.next_obs) & 3) != 0) return TJ_ERR_INVALID_ARG;
    if ((f.rows || f.planes) && f.n_rows == 0) return TJ_ERR_INVALID_ARG;
    if (f.rows && f.planes) return TJ_ERR_INVALID_ARG;
    TowerPlan p = tower_plan(f.H, f.W, f.OH, f.OW, a.OH2, a.OW2, a.OW3);
    p.n_pass = f.next_obs ? 3 * f.B : f.B;
    TJ_HIP_TRY(hipFuncSetAttribute((const void *)conv_tower, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit));
    int dev = 0, n_cu = 256, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
        n_cu = v;
    conv_tower<<<p.n_pass < n_cu ? p.n_pass : n_cu, kThreads, p.total, st>>>(a, p);
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}
