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
// Rows of the activations in LDS are padded by 32 bytes, to 96 and 160.  A 16-byte read serves sixteen lanes at a time, not consecutive ones
// but rows 0 - 3 and 12 - 15 of one lane group of the fragment and rows 4 - 11 of the next one (8 channels on): rows an odd number of 16-byte
// units apart (80, 144 bytes) meet there and run at half rate, 6.0 against 3.2 clocks per wave read in a bare loop; rows 2 mod 4 units
// apart do not.  Writes do: 34 % of the cycles in which the LDS is busy are conflicts here (profiles/c3_gemm_counters.md), no fewer than with rows of
// 80 and 144.  By their banks, the image's pieces lie 64 bytes apart from lane to lane in conv_tower_pipe (four lanes of sixteen meet), the
// 8-byte stores of activations meet in twos at 160 bytes (not at all at 144) and in four or five at 96 (two or three at 80).
// The second layer has stride 2, so its input keeps even and odd columns apart, which makes consecutive patches
// consecutive rows.  Sixteen patches mostly end one output row and begin another: the rows of the image they read (even and odd ones
// apart as well) have a pitch that continues the sequence of columns there (tower_plan).
// While an image is in the second layer the next one, fetched into registers a layer ahead, is converted into the image buffer.
#include "tj_conv_planes.h"
#include "tj_conv_tower_plan.h"
#include <algorithm>
#include <type_traits>

namespace {

using namespace tjplanes;
using namespace tjtower;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) uint8_t *lds_ptr_t;

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
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ct = wave & 3, rh = wave >> 2;
    const int HW = f.H * f.W, W = f.W, OHW1 = f.OH * f.OW, OHW2 = a.OH2 * a.OW2, OHW3 = a.OH3 * a.OW3;
    const int begin = (int)((long)blockIdx.x * p.n_pass / gridDim.x), end = (int)((long)(blockIdx.x + 1) * p.n_pass / gridDim.x);
    if (begin >= end) return;

    // ---- images.  Unit = 16 bytes of LDS = two pixels.  Even and odd units lie apart: with a stride of four pixels the operand
    // reads of consecutive patches are consecutive units of one half, which one is fixed by the lane
    const int n_task = HW / 4;
    uint32_t px[kRounds][4];
    // Image of a pass: s, s', and s' again for the target network.  Fetches go through the run in order, and the place of the next
    // one is looked up right after the current one was issued, off the critical path.
    auto image_of = [&](int pass) { return pass < 2 * f.B ? pass : pass - f.B; };
    auto where = [&](int pass) {
        const int g = image_of(pass);
        return plane_offsets(f.rows, f.planes, f.n_rows, g < f.B ? g : g - f.B, g >= f.B, HW);
    };
    PlaneOff off = where(begin);
    auto fetch = [&](int pass, int tid) {
        const uint8_t *src = image_of(pass) >= f.B ? f.next_obs : f.obs;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int t = tid + r * kThreads;
            if (t < n_task) {
#pragma unroll
                for (int c = 0; c < 4; ++c) px[r][c] = *(const uint32_t *)(src + off.o[c] + 4 * t);
            }
        }
        if (pass + 1 < end) off = where(pass + 1);
    };
    auto convert = [&](int r, int tid) {
        {
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
                *(u32x4 *)(img + t * 16) = v[0];
                *(u32x4 *)(img + HW * 4 + t * 16) = v[1];
            }
        }
    };

    // ---- weights of one network.  The second and third layer's rows come through LDS, where between two runs nothing lives behind the
    // first layer's weights, and in front of the first image nothing in the image buffer: whole lines, each once, instead of
    // 64-byte pieces of 16 rows per load, twice.  A group is the 16 rows of one ct.
    u32x4 w2[kSteps2], w3[kSteps3];
    auto stage = [&](const tj_bf16 *src, auto row_units, int groups, uint8_t *dst, int lane) {
        constexpr int N = decltype(row_units)::value;
        const int total = groups * 16 * (N + 1);
        for (int i = wave; i < (total + 63) / 64; i += kWaves) {
            const uint32_t u = min(64 * i + lane, total - 1), row = u / (N + 1), col = min(u % (N + 1), N - 1);
            const uint32_t at = (uint32_t)(uintptr_t)(lds_ptr_t)(dst + i * 1024);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(src + (row * N + col) * 8) : "memory");
        }
    };
    auto take = [&](auto &w, const uint8_t *group, int units, int lane) {
#pragma unroll
        for (int i = 0; i < (int)(sizeof(w) / sizeof(w[0])); ++i) w[i] = *(const u32x4 *)(group + ((lane & 15) * (units + 1) + 4 * i + (lane >> 4)) * 16);
    };
    typedef std::integral_constant<int, kUnits2> Units2;
    typedef std::integral_constant<int, kUnits3> Units3;
    auto landed = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // where this wave's patches start in the activations of the layer below (tiles past the last patch repeat it)
    int at2[kTiles2], at3[kTiles3];
#pragma unroll
    for (int i = 0; i < kTiles2; ++i) {
        const uint32_t m = min((rh * kTiles2 + i) * 16 + l16, OHW2 - 1), oh = __umulhi(m, p.mg_ow2), ow = m - oh * a.OW2;
        at2[i] = oh * p.pitch1 + ow * kRow1 + 16 * q4;
    }
#pragma unroll
    for (int i = 0; i < kTiles3; ++i) {
        const uint32_t m = min((rh * kTiles3 + i) * 16 + l16, OHW3 - 1), oh = __umulhi(m, p.mg_ow3), ow = m - oh * a.OW3;
        at3[i] = oh * a.s3 * p.pitch2 + ow * a.s3 * kRow2 + 16 * q4;
    }
    auto row1 = [&](uint32_t m) -> uint8_t * {   // patch m of the first layer's output
        const uint32_t oh = __umulhi(m, p.mg_ow1), ow = m - oh * f.OW;
        return out1 + ((oh & 1) * p.rows1 + (oh >> 1)) * p.pitch1 + ((ow & 1) * p.half1 + (ow >> 1)) * kRow1;
    };
    auto row2 = [&](uint32_t m) -> uint8_t * {   // the second layer's
        const uint32_t oh = __umulhi(m, p.mg_ow2), ow = m - oh * a.OW2;
        return out2 + oh * p.pitch2 + ow * kRow2;
    };

    bool first_run = true;
    for (int pass = begin; pass < end;) {   // runs under one network's weights: one, or two where the block's passes meet the target's
    const int net = pass >= 2 * f.B, run_end = net ? end : min(end, 2 * f.B);
    int tid0 = tid;   // opaque, as in the loop below
    asm volatile("" : "+v"(tid0));
    const int lane0 = tid0 & 63;
    const tj_bf16 *const W2 = net ? a.W2_tg : a.W2_on, *const W3 = net ? a.W3_tg : a.W3_on;
    if (first_run) {
        stage(W3, Units3{}, p.groups_img, img, lane0);
        stage(W3 + p.groups_img * 16 * kUnits3 * 8, Units3{}, 4 - p.groups_img, out1 + 4 * kGroup2, lane0);
    }
    lds_sync();   // nobody reads the last run's activations, weights and biases any more
    stage(W2, Units2{}, 4, out1, lane0);
    {
        constexpr int VR = 4 * K1 * K1 / 8;   // 16-byte vectors per row of the first layer's weights
        for (int v = tid0; v < C1 * VR; v += kThreads)
            *(u32x4 *)(w1 + (v / VR) * kW1Pitch + (v % VR) * 16) = *(const u32x4 *)((net ? f.W_tg : f.W_on) + (size_t)v * 8);
        if (tid0 < C1) bias[tid0] = (net ? f.b_tg : f.b_on)[tid0];
        else if (tid0 < C1 + C2) bias[tid0] = (net ? a.b2_tg : a.b2_on)[tid0 - C1];
        else if (tid0 < C1 + C2 + C3) bias[tid0] = (net ? a.b3_tg : a.b3_on)[tid0 - C1 - C2];
    }
    if (first_run) fetch(pass, tid0);
    landed();
    take(w2, out1 + ct * kGroup2, kUnits2, lane0);
    if (first_run) {
        take(w3, ct < p.groups_img ? img + ct * kGroup3 : out1 + 4 * kGroup2 + (ct - p.groups_img) * kGroup3, kUnits3, lane0);
        lds_sync();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) convert(r, tid0);
        if (begin + 1 < end) fetch(begin + 1, tid0);
        first_run = false;
    } else {
        lds_sync();
        stage(W3, Units3{}, 4, out1, lane0);
        landed();
        take(w3, out1 + ct * kGroup3, kUnits3, lane0);
    }

    for (; pass < run_end; ++pass) {
        lds_sync();   // the image is in place; the last pass is out of out1 (the first one: every weight has been read)

        // ---- first layer: image -> out1
        const int n_tile = (OHW1 + 31) / 32;
        // opaque, so that addresses are not kept in registers (or rather in memory) from pass to pass
        int tid1 = tid;
        asm volatile("" : "+v"(tid1));
        const int lane1 = tid1 & 31, h1 = (tid1 >> 5) & 1, p16 = tid1 & 15, c4 = 16 * ct + 4 * ((tid1 >> 4) & 3);
        for (int tile = wave; tile < n_tile; tile += 2 * kWaves) {   // two tiles share the weight reads
            const bool two = tile + kWaves < n_tile;
            const uint8_t *src[2];
            uint8_t *dst[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint32_t m = min(32 * (tile + t * kWaves) + lane1, OHW1 - 1), oh = __umulhi(m, p.mg_ow1), ow = m - oh * f.OW;
                src[t] = img + h1 * HW * 4 + (oh * f.s * W + ow * f.s) * 4;
                dst[t] = row1(m) + 8 * h1;
            }
            const uint8_t *const wsrc = w1 + lane1 * kW1Pitch + 16 * h1;
            f32x16 acc[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
            // steps of 16 contraction values (4 pixels x 4 channels), the next one's operands on their way
            u32x4 wv[2], pv[2][2];
            auto read = [&](int n) {
                wv[n & 1] = *(const u32x4 *)(wsrc + n * 32);
#pragma unroll
                for (int t = 0; t < 2; ++t) pv[n & 1][t] = *(const u32x4 *)(src[t] + (n >> 1) * W * 4 + (n & 1) * 16);
            };
            read(0);
#pragma unroll
            for (int n = 0; n < 2 * K1; ++n) {
                if (n + 1 < 2 * K1) read(n + 1);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    if (t == 1 && !two) continue;
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wv[n & 1]), __builtin_bit_cast(bf16x8, pv[n & 1][t]),
                                                                     acc[t], 0, 0, 0);
                }
            }
            // acc[4q + e] = channel 8q + 4h + e of a patch; tiles past the last patch repeat it, into the same place
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t == 1 && !two) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 b = *(const f32x4 *)(bias + 8 * q + 4 * h1);
                    float x[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = fmaxf(acc[t][4 * q + e] + b[e], 0.f);
                    *(uint2 *)(dst[t] + 16 * q) = make_uint2(pack2(x[0], x[1]), pack2(x[2], x[3]));
                }
            }
        }
        lds_sync();

        // ---- second layer: out1 -> out2; the image buffer takes the next image
        const bool keep = f.out && pass < f.B;
        if (keep) {
            tj_bf16 *dst = f.out + (size_t)pass * OHW1 * C1;
            for (int v = tid1; v < OHW1 * 4; v += kThreads) *(u32x4 *)(dst + (size_t)v * 8) = *(const u32x4 *)(row1(v >> 2) + (v & 3) * 16);
        }
        f32x4 acc2[kTiles2];
#pragma unroll
        for (int i = 0; i < kTiles2; ++i) acc2[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        // a step is one tap of 32 channels; between the reads of four steps and their use a quarter of the next image is converted
        static_assert(kRounds == K2, "a round of the image per row of the kernel");
#pragma unroll
        for (int kh = 0; kh < K2; ++kh) {
            u32x4 x[K2][kTiles2];
#pragma unroll
            for (int kw = 0; kw < K2; ++kw)
#pragma unroll
                for (int i = 0; i < kTiles2; ++i)
                    x[kw][i] = *(const u32x4 *)(out1 + at2[i] + ((kh % S2) * p.rows1 + kh / S2) * p.pitch1 + ((kw % S2) * p.half1 + kw / S2) * kRow1);
            if (pass + 1 < end) convert(kh, tid1);
#pragma unroll
            for (int kw = 0; kw < K2; ++kw)
#pragma unroll
                for (int i = 0; i < kTiles2; ++i)
                    acc2[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w2[kh * K2 + kw]),
                                                                      __builtin_bit_cast(bf16x8, x[kw][i]), acc2[i], 0, 0, 0);
        }
        if (pass + 2 < end) fetch(pass + 2, tid1);
        {   // acc[r] = channel 16 ct + 4 q4 + r of patch l16
            const f32x4 b = *(const f32x4 *)(bias + C1 + c4);
#pragma unroll
            for (int i = 0; i < kTiles2; ++i) {
                const int m = (rh * kTiles2 + i) * 16 + p16;
                const f32x4 s = acc2[i] + b;
                if (m < OHW2)
                    *(uint2 *)(row2(m) + c4 * 2) =
                        make_uint2(pack2(fmaxf(s[0], 0.f), fmaxf(s[1], 0.f)), pack2(fmaxf(s[2], 0.f), fmaxf(s[3], 0.f)));
            }
        }
        lds_sync();

        // ---- third layer: out2 -> out
        if (keep) {
            tj_bf16 *dst = a.act2 + (size_t)pass * OHW2 * C2;
            for (int v = tid1; v < OHW2 * 8; v += kThreads) *(u32x4 *)(dst + (size_t)v * 8) = *(const u32x4 *)(row2(v >> 3) + (v & 7) * 16);
        }
        f32x4 acc3[kTiles3];
#pragma unroll
        for (int i = 0; i < kTiles3; ++i) acc3[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < kSteps3; ++n) {   // a step is half a tap
            const int kh = n / 2 / K3, kw = n / 2 % K3;
            const int off = kh * p.pitch2 + kw * kRow2 + (n & 1) * 64;
#pragma unroll
            for (int i = 0; i < kTiles3; ++i) {
                const u32x4 x = *(const u32x4 *)(out2 + at3[i] + off);
                acc3[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w3[n]), __builtin_bit_cast(bf16x8, x),
                                                                  acc3[i], 0, 0, 0);
            }
        }
        const f32x4 b3 = *(const f32x4 *)(bias + C1 + C2 + c4);
#pragma unroll
        for (int i = 0; i < kTiles3; ++i) {
            const int m = (rh * kTiles3 + i) * 16 + p16;
            const f32x4 s = acc3[i] + b3;
            if (m < OHW3)
                *(uint2 *)(a.out + ((size_t)pass * OHW3 + m) * C3 + c4) =
                    make_uint2(pack2(fmaxf(s[0], 0.f), fmaxf(s[1], 0.f)), pack2(fmaxf(s[2], 0.f), fmaxf(s[3], 0.f)));
        }
    }
    }
}

// ---- many passes per block: the layers of two images side by side

// The same layers, sums and results as conv_tower for blocks with several passes.  There eight waves go through the layers of one image
// together and wait for each other behind each: LDS reads, the image's conversion and the products take turns.  Here four waves (one
// per SIMD) take the first layer of an image while the other four take the second and third of the one before it:
//             first four waves                                       last four waves
//   phase 1   first layer of image i -> out1[i % 2]                  second layer of image i - 1 -> out2
//   phase 2   image i + 1 into the image buffer, i + 2 asked for     third layer of image i - 1
// with a barrier behind each phase.  The first layer's weights live in the first waves' registers (they took a third of that layer's LDS
// reads), a last wave has 16 channels of the other two layers and all patches.  What bounds it: 4350 clocks of products per SIMD and pass and
// the reads that feed them (700 KB per pass) in 10200, phase 1 about 6200 of them.  Measured, us per update of 3 x 2048 passes from a
// frame ring: 430 -> 402.  Reads further ahead change nothing, priority for either half costs 1 - 4 %, and loads of the image spread over both
// phases take 0.4 % off 24 passes per block and add 1.2 % to three.
constexpr int kHalf = kThreads / 2;
constexpr int kFetch = 2;                    // 16-pixel tasks per thread of the first four waves

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void conv_tower_pipe(const TjConvTowerArgs a, const PipePlan p)
{
    extern __shared__ __align__(16) uint8_t lds[];
    uint8_t *const img = lds, *const out2 = lds + p.out2;
    float *const bias = (float *)(lds + p.bias);
    const TjConvFirstArgs &f = a.first;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HW = f.H * f.W, W = f.W, OHW1 = f.OH * f.OW, OHW2 = a.OH2 * a.OW2, OHW3 = a.OH3 * a.OW3;
    const int begin = (int)((long)blockIdx.x * p.n_pass / gridDim.x), end = (int)((long)(blockIdx.x + 1) * p.n_pass / gridDim.x);
    if (begin >= end) return;
    auto out1 = [&](int pass) { return lds + p.out1 + (pass & 1 ? p.out1_bytes : 0); };
    auto row1 = [&](uint8_t *base, uint32_t m) -> uint8_t * {   // patch m of the first layer's output
        const uint32_t oh = __umulhi(m, p.mg_ow1), ow = m - oh * f.OW;
        return base + ((oh & 1) * p.rows1 + (oh >> 1)) * p.pitch1 + ((ow & 1) * p.half1 + (ow >> 1)) * kRow1;
    };
    auto row2 = [&](uint32_t m) -> uint8_t * {   // the second layer's
        const uint32_t oh = __umulhi(m, p.mg_ow2), ow = m - oh * a.OW2;
        return out2 + oh * p.pitch2 + ow * kRow2;
    };

    if (wave < 4) {
        // ---- images.  Unit = 16 bytes of LDS = two pixels, even and odd units apart, as in conv_tower
        typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
        typedef const __attribute__((address_space(1))) uint8_t *gbytes;
        u32x4 px[kFetch][4];
        uint32_t idx[4];
        auto image_of = [&](int pass) { return pass < 2 * f.B ? pass : pass - f.B; };
        const bool named = f.planes || f.rows;
        // What names the pass's planes, a fetch ahead of their use.  One load whatever names them (a float's bits where nothing
        // does): values that meet behind branches would be waited for there.
        auto look_up = [&](int pass) {
            const int g = image_of(pass), b = g < f.B ? g : g - f.B;
            const uint32_t *at = f.planes ? f.planes + (size_t)b * 8 + (g >= f.B ? 4 : 0) : f.rows ? f.rows + b : (const uint32_t *)f.b_on;
            const int step = f.planes ? 1 : 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) idx[c] = at[c * step];
        };
        auto fetch = [&](int pass) {
            const int g = image_of(pass), b = g < f.B ? g : g - f.B;
            const uint8_t *src = g >= f.B ? f.next_obs : f.obs;
            int t0 = tid;
            asm volatile("" : "+v"(t0));
            // the last task may begin before its turn, and threads without one repeat it: a load under a condition leaves its register
            // with two possible values, and the copy that joins them waits for it (12000 -> 10200 clocks per pass with what follows)
            const uint32_t at0 = min(16 * t0, HW - 16), at1 = min(16 * (t0 + kHalf), HW - 16);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t i = named ? min((uint32_t)__builtin_amdgcn_readfirstlane(idx[c]), f.n_rows - 1u) : (uint32_t)b;
                gbytes plane = (gbytes)(uintptr_t)(src + (f.planes ? (size_t)i : (size_t)i * 4 + c) * HW);
                asm("" : "+s"(plane));
                px[0][c] = *(const __attribute__((address_space(1))) u32x4_a4 *)(plane + at0);
                px[1][c] = *(const __attribute__((address_space(1))) u32x4_a4 *)(plane + at1);
            }
        };
        auto convert = [&]() {
            int t0 = tid;
            asm volatile("" : "+v"(t0));
#pragma unroll
            for (int r = 0; r < kFetch; ++r) {
                const int t = t0 + r * kHalf;
                if (16 * t >= HW) break;
                uint8_t *const dst = img + min(16 * t, HW - 16) * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    u32x4 v[2];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {     // a pixel, channels 0..3
                        float x[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) x[c] = (float)((px[r][c][j] >> (8 * q)) & 0xFF) * f.scale;
                        v[q >> 1][2 * (q & 1)] = pack2(x[0], x[1]);
                        v[q >> 1][2 * (q & 1) + 1] = pack2(x[2], x[3]);
                    }
                    *(u32x4 *)(dst + j * 16) = v[0];
                    *(u32x4 *)(dst + HW * 4 + j * 16) = v[1];
                }
            }
        };
        look_up(begin);
        for (int pass = begin; pass < end;) {   // runs under one network's weights
            const int net = pass >= 2 * f.B, run_end = net ? end : min(end, 2 * f.B);
            fetch(pass);
            if (pass + 1 < end) look_up(pass + 1);
            lds_sync();   // the last run is through
            constexpr int VR = 4 * K1 * K1 / 8;   // 16-byte vectors per row of the first layer's weights
            uint8_t *const w1 = lds + p.out1 + p.out1_bytes;
            for (int v = tid; v < C1 * VR; v += kHalf)
                *(u32x4 *)(w1 + (v / VR) * kW1Pitch + (v % VR) * 16) = *(const u32x4 *)((net ? f.W_tg : f.W_on) + (size_t)v * 8);
            if (tid < C1) bias[tid] = (net ? f.b_tg : f.b_on)[tid];
            else if (tid < C1 + C2) bias[tid] = (net ? a.b2_tg : a.b2_on)[tid - C1];
            else if (tid < C1 + C2 + C3) bias[tid] = (net ? a.b3_tg : a.b3_on)[tid - C1 - C2];
            convert();
            lds_sync();
            u32x4 wv[2 * K1];
#pragma unroll
            for (int n = 0; n < 2 * K1; ++n) wv[n] = *(const u32x4 *)(w1 + (tid & 31) * kW1Pitch + 16 * ((tid >> 5) & 1) + n * 32);
            lds_sync();   // the weights have been read: their memory is out1 of the odd passes
            if (pass + 1 < run_end) {
                fetch(pass + 1);
                if (pass + 2 < end) look_up(pass + 2);
            }
            for (; pass < run_end; ++pass) {
                // ---- phase 1: first layer
                int tid1 = tid;   // opaque, so that addresses are not kept in registers from pass to pass
                asm volatile("" : "+v"(tid1));
                const int lane1 = tid1 & 31, h1 = (tid1 >> 5) & 1, n_tile = (OHW1 + 31) / 32;
                uint8_t *const out = out1(pass);
                auto tiles = [&](int tile, auto count) {
                    constexpr int N = decltype(count)::value;
                    const uint8_t *src[N];
                    uint8_t *dst[N];
                    f32x16 acc[N];
#pragma unroll
                    for (int t = 0; t < N; ++t) {
                        const uint32_t m = min(32 * (tile + t * 4) + lane1, OHW1 - 1), oh = __umulhi(m, p.mg_ow1), ow = m - oh * f.OW;
                        src[t] = img + h1 * HW * 4 + (oh * f.s * W + ow * f.s) * 4;
                        dst[t] = row1(out, m) + 8 * h1;
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
                    }
                    // steps of 16 contraction values (4 pixels x 4 channels), the next ones' operands on their way
                    u32x4 pv[4][N];
                    auto read = [&](int n) {
#pragma unroll
                        for (int t = 0; t < N; ++t) pv[n & 3][t] = *(const u32x4 *)(src[t] + (n >> 1) * W * 4 + (n & 1) * 16);
                    };
                    read(0); read(1); read(2);
#pragma unroll
                    for (int n = 0; n < 2 * K1; ++n) {
                        if (n + 3 < 2 * K1) read(n + 3);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int t = 0; t < N; ++t)
                            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wv[n]), __builtin_bit_cast(bf16x8, pv[n & 3][t]),
                                                                             acc[t], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // acc[4q + e] = channel 8q + 4h + e of a patch; tiles past the last patch repeat it, into the same place
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 b = *(const f32x4 *)(bias + 8 * q + 4 * h1);
#pragma unroll
                        for (int t = 0; t < N; ++t) {
                            float x[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) x[e] = fmaxf(acc[t][4 * q + e] + b[e], 0.f);
                            *(uint2 *)(dst[t] + 16 * q) = make_uint2(pack2(x[0], x[1]), pack2(x[2], x[3]));
                        }
                    }
                };
                int tile = wave;
                for (; tile + 4 < n_tile; tile += 8) tiles(tile, std::integral_constant<int, 2>{});
                if (tile < n_tile) tiles(tile, std::integral_constant<int, 1>{});
                lds_sync();
                // ---- phase 2: the next image, and what the backward pass reads of this one
                if (pass + 1 < run_end) {
                    convert();
                    if (pass + 2 < run_end) {
                        fetch(pass + 2);
                        if (pass + 3 < end) look_up(pass + 3);
                    }
                }
                if (f.out && pass < f.B) {
                    tj_bf16 *dst = f.out + (size_t)pass * OHW1 * C1;
                    for (int v = tid1; v < OHW1 * 4; v += kHalf) *(u32x4 *)(dst + (size_t)v * 8) = *(const u32x4 *)(row1(out, v >> 2) + (v & 3) * 16);
                }
                lds_sync();
            }
            lds_sync();   // the last image's second layer
            lds_sync();   // ... and third
            if (pass < end) look_up(pass);
        }
    } else {
        const int ct = wave - 4;
        constexpr int T2 = 2 * kTiles2, T3 = 2 * kTiles3;
        constexpr int D2 = 2, D3 = 2;   // reads ahead: half steps of the second layer, steps of the third
        const int lane = tid & 63, l16 = lane & 15, q4 = lane >> 4;
        // where the patches start in the activations of the layer below (tiles past the last patch repeat it)
        int at2[T2], at3[T3];
#pragma unroll
        for (int i = 0; i < T2; ++i) {
            const uint32_t m = min(i * 16 + l16, OHW2 - 1), oh = __umulhi(m, p.mg_ow2), ow = m - oh * a.OW2;
            at2[i] = oh * p.pitch1 + ow * kRow1 + 16 * q4;
        }
#pragma unroll
        for (int i = 0; i < T3; ++i) {
            const uint32_t m = min(i * 16 + l16, OHW3 - 1), oh = __umulhi(m, p.mg_ow3), ow = m - oh * a.OW3;
            at3[i] = oh * a.s3 * p.pitch2 + ow * a.s3 * kRow2 + 16 * q4;
        }
        for (int pass = begin; pass < end;) {
            const int net = pass >= 2 * f.B, run_end = net ? end : min(end, 2 * f.B);
            u32x4 w2[kSteps2], w3[kSteps3];
            {
                const tj_bf16 *r2 = (net ? a.W2_tg : a.W2_on) + ((size_t)(16 * ct + l16) * kUnits2 + q4) * 8;
                const tj_bf16 *r3 = (net ? a.W3_tg : a.W3_on) + ((size_t)(16 * ct + l16) * kUnits3 + q4) * 8;
#pragma unroll
                for (int i = 0; i < kSteps2; ++i) w2[i] = *(const u32x4 *)(r2 + 32 * i);
#pragma unroll
                for (int i = 0; i < kSteps3; ++i) w3[i] = *(const u32x4 *)(r3 + 32 * i);
            }
            lds_sync();   // the last run is through
            lds_sync();   // the first image and the weights of the first layer are in place
            lds_sync();   // ... which have been read
            lds_sync();   // the first image's first layer
            lds_sync();   // the second image
            for (; pass < run_end; ++pass) {
                int tid1 = tid;
                asm volatile("" : "+v"(tid1));
                const int p16 = tid1 & 15, c4 = 16 * ct + 4 * ((tid1 >> 4) & 3);
                // ---- phase 1: second layer, out1 -> out2.  A step is one tap of 32 channels, the next one's reads on their way
                const uint8_t *const in = out1(pass);
                f32x4 acc2[T2];
#pragma unroll
                for (int i = 0; i < T2; ++i) acc2[i] = f32x4{0.f, 0.f, 0.f, 0.f};
                u32x4 x[D2 + 1][kTiles2];
                auto read2 = [&](int u) {   // half the tiles of step u / 2
                    const int kh = u / 2 / K2, kw = u / 2 % K2;
                    const int off = ((kh % S2) * p.rows1 + kh / S2) * p.pitch1 + ((kw % S2) * p.half1 + kw / S2) * kRow1;
#pragma unroll
                    for (int i = 0; i < kTiles2; ++i) x[u % (D2 + 1)][i] = *(const u32x4 *)(in + at2[u % 2 * kTiles2 + i] + off);
                };
#pragma unroll
                for (int u = 0; u < D2; ++u) read2(u);
#pragma unroll
                for (int u = 0; u < 2 * kSteps2; ++u) {
                    if (u + D2 < 2 * kSteps2) read2(u + D2);
                    __builtin_amdgcn_sched_barrier(0);   // left alone, the compiler reads right before each product
#pragma unroll
                    for (int i = 0; i < kTiles2; ++i) {
                        f32x4 &s = acc2[u % 2 * kTiles2 + i];
                        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w2[u / 2]), __builtin_bit_cast(bf16x8, x[u % (D2 + 1)][i]), s, 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                {   // acc[r] = channel 16 ct + 4 q4 + r of patch l16
                    const f32x4 b = *(const f32x4 *)(bias + C1 + c4);
#pragma unroll
                    for (int i = 0; i < T2; ++i) {
                        const int m = i * 16 + p16;
                        const f32x4 s = acc2[i] + b;
                        if (m < OHW2)
                            *(uint2 *)(row2(m) + c4 * 2) =
                                make_uint2(pack2(fmaxf(s[0], 0.f), fmaxf(s[1], 0.f)), pack2(fmaxf(s[2], 0.f), fmaxf(s[3], 0.f)));
                    }
                }
                lds_sync();
                // ---- phase 2: third layer, out2 -> out
                if (f.out && pass < f.B) {
                    tj_bf16 *dst = a.act2 + (size_t)pass * OHW2 * C2;
                    for (int v = tid1 - kHalf; v < OHW2 * 8; v += kHalf) *(u32x4 *)(dst + (size_t)v * 8) = *(const u32x4 *)(row2(v >> 3) + (v & 7) * 16);
                }
                f32x4 acc3[T3];
#pragma unroll
                for (int i = 0; i < T3; ++i) acc3[i] = f32x4{0.f, 0.f, 0.f, 0.f};
                u32x4 y[D3 + 1][T3];
                auto read3 = [&](int n) {   // a step is half a tap
                    const int off = n / 2 / K3 * p.pitch2 + n / 2 % K3 * kRow2 + (n & 1) * 64;
#pragma unroll
                    for (int i = 0; i < T3; ++i) y[n % (D3 + 1)][i] = *(const u32x4 *)(out2 + at3[i] + off);
                };
#pragma unroll
                for (int n = 0; n < D3; ++n) read3(n);
#pragma unroll
                for (int n = 0; n < kSteps3; ++n) {
                    if (n + D3 < kSteps3) read3(n + D3);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < T3; ++i)
                        acc3[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w3[n]), __builtin_bit_cast(bf16x8, y[n % (D3 + 1)][i]),
                                                                          acc3[i], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                const f32x4 b3 = *(const f32x4 *)(bias + C1 + C2 + c4);
#pragma unroll
                for (int i = 0; i < T3; ++i) {
                    const int m = i * 16 + p16;
                    const f32x4 s = acc3[i] + b3;
                    if (m < OHW3)
                        *(uint2 *)(a.out + ((size_t)pass * OHW3 + m) * C3 + c4) =
                            make_uint2(pack2(fmaxf(s[0], 0.f), fmaxf(s[1], 0.f)), pack2(fmaxf(s[2], 0.f), fmaxf(s[3], 0.f)));
                }
                lds_sync();
            }
        }
    }
}

}  // namespace

// The kernel's layer shapes; image, activations and weights beside one another in LDS; no more patches than the waves'
// accumulators take.
bool tj_conv_tower_fits(const TjConvShape *c)
{
    const TjConvShape &x = c[0], &y = c[1], &z = c[2];
    if (!tj_conv_first_fits(x.C, x.H, x.W, x.k, x.s, x.O) || x.k != K1 || x.s % 4 || x.W % 4) return false;
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
    PipePlan q = pipe_plan(f.H, f.W, f.OH, f.OW, a.OH2, a.OW2, a.OW3);
    if (two_images(q, p.n_pass, n_cu)) {
        q.n_pass = p.n_pass;
        TJ_HIP_TRY(hipFuncSetAttribute((const void *)conv_tower_pipe, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit));
        conv_tower_pipe<<<n_cu, kThreads, q.total, st>>>(a, q);
        return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
    }
    conv_tower<<<p.n_pass < n_cu ? p.n_pass : n_cu, kThreads, p.total, st>>>(a, p);
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}
