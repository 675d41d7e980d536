// Shapes and LDS layouts of the three convolutions in one kernel (tj_conv_tower.hip), and which of its two forms a call takes: plain host
// arithmetic without HIP, so that it can be compiled and checked on its own.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <algorithm>

namespace tjtower {

constexpr int kThreads = 512, kWaves = 8;
constexpr int K1 = 8, C1 = 32, K2 = 4, S2 = 2, C2 = 64, K3 = 3, C3 = 64;   // kernels, strides, output channels
constexpr int kRounds = 4;              // 4-pixel tasks per thread and image
constexpr int kTiles2 = 3, kTiles3 = 2; // tiles of 16 patches per wave (two waves share the patches)
constexpr int kSteps2 = K2 * K2 * C1 / 32, kSteps3 = K3 * K3 * C2 / 32;   // 32-value steps of a contraction
constexpr int kRow1 = C1 * 2 + 32, kRow2 = C2 * 2 + 32;   // bytes between activation rows in LDS
constexpr int kW1Pitch = (4 * K1 * K1 + 8) * 2;           // ... between the first layer's weight rows
constexpr int kUnits2 = 4 * kSteps2, kUnits3 = 4 * kSteps3;               // 16-byte units of a weight row of the other two,
constexpr int kGroup2 = 16 * (kUnits2 + 1) * 16, kGroup3 = 16 * (kUnits3 + 1) * 16;   // bytes of 16 such rows, a unit apart, in LDS
constexpr size_t kLdsLimit = 160 * 1024;

struct TowerPlan {
    int w1, bias, out1, out2, total;   // byte offsets in LDS (the image is at 0)
    int groups_img;                          // groups of 16 rows of the third layer's weights that the image buffer holds
    int half1, rows1;                        // columns and rows per parity of the first layer's output
    int pitch1, pitch2;                      // bytes between image rows (of one parity) of the first layer's output, of the second's
    uint32_t mg_ow1, mg_ow2, mg_ow3;         // ceil(2^32 / OW)
    int n_pass;
};

inline uint32_t magic(int d) { return (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

inline TowerPlan tower_plan(int H, int W, int OH1, int OW1, int OH2, int OW2, int OW3)
{
    TowerPlan p;
    p.half1 = (OW1 + S2 - 1) / S2;
    p.rows1 = (OH1 + S2 - 1) / S2;
    // 16 lanes read 16 consecutive patches, which end one output row and begin the next: the step to it is the step between patches
    // modulo the 16 units of the LDS banks (units of 16 bytes)
    auto pitch = [](int row_bytes, int step_bytes, int OW) {
        int u = row_bytes / 16;
        while ((u - OW * (step_bytes / 16)) % 16) ++u;
        return u * 16;
    };
    p.pitch1 = pitch(S2 * p.half1 * kRow1, kRow1, OW2);
    p.pitch2 = pitch(OW2 * kRow2, kRow2, OW3);
    int at = H * W * 8;
    p.w1 = at; at += C1 * kW1Pitch;
    p.bias = at; at += (C1 + C2 + C3) * 4;
    p.out1 = at; at += S2 * p.rows1 * p.pitch1;
    p.out2 = at; at += OH2 * p.pitch2;
    auto whole = [](int bytes) { return (bytes + 1023) / 1024 * 1024; };   // a load instruction fills a KiB
    p.groups_img = 4;
    while (whole(p.groups_img * kGroup3) > H * W * 8) --p.groups_img;
    p.total = std::max(at, p.out1 + std::max(whole(4 * kGroup3), 4 * kGroup2 + whole((4 - p.groups_img) * kGroup3)));
    p.mg_ow1 = magic(OW1); p.mg_ow2 = magic(OW2); p.mg_ow3 = magic(OW3);
    p.n_pass = 0;
    return p;
}

// Two images side by side, in blocks of many passes.
struct PipePlan {
    int bias, out1, out1_bytes, out2, total; // byte offsets in LDS (the image is at 0); two outputs of the first layer, out1_bytes apart
    int half1, rows1, pitch1, pitch2;        // as in TowerPlan
    uint32_t mg_ow1, mg_ow2, mg_ow3;
    int n_pass;
};

inline PipePlan pipe_plan(int H, int W, int OH1, int OW1, int OH2, int OW2, int OW3)
{
    const TowerPlan t = tower_plan(H, W, OH1, OW1, OH2, OW2, OW3);
    PipePlan p;
    p.half1 = t.half1; p.rows1 = t.rows1; p.pitch1 = t.pitch1; p.pitch2 = t.pitch2;
    p.mg_ow1 = t.mg_ow1; p.mg_ow2 = t.mg_ow2; p.mg_ow3 = t.mg_ow3;
    p.bias = H * W * 8;
    p.out1 = p.bias + (C1 + C2 + C3) * 4;
    p.out1_bytes = std::max(S2 * p.rows1 * p.pitch1, C1 * kW1Pitch);   // the second one takes the first layer's weights before a run
    p.out2 = p.out1 + 2 * p.out1_bytes;
    p.total = p.out2 + OH2 * p.pitch2;
    p.n_pass = 0;
    return p;
}

// Two images side by side from four passes per block on, the first and the last image being alone (us per update, one image at a time : two;
// 84 x 84: 3 passes 134.5 : 136.2, 4 148.9 : 145.8, 8 170.0 : 168.6, 12 267.0 : 255.8, 24 430 : 402; 52 x 52: 3 99 : 101, 4 107 : 107, 8 127 : 124, 12
// 147 : 143; 37 x 68: 3 96 : 98, 4 103 : 103, 8 122 : 118), if LDS holds two outputs of the first layer.
inline bool two_images(const PipePlan &q, int n_pass, int n_cu) { return n_pass >= 4 * n_cu && (size_t)q.total <= kLdsLimit; }

}  // namespace tjtower
