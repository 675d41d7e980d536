// The plans of the three convolutions in one kernel as functions that a test can call.
#include "../paper_2502_20190_amd/csrc/tj_conv_tower_plan.h"

using namespace tjtower;

static int out_side(int n, int k, int s) { return (n - k) / s + 1; }

// Whether a call of n_pass passes on n_cu compute units takes two images side by side; images H x W, strides s and s3 of the first and third layer.
extern "C" int tower_two_images(int H, int W, int s, int s3, int n_pass, int n_cu)
{
    const int OH1 = out_side(H, K1, s), OW1 = out_side(W, K1, s), OH2 = out_side(OH1, K2, S2), OW2 = out_side(OW1, K2, S2);
    return two_images(pipe_plan(H, W, OH1, OW1, OH2, OW2, out_side(OW2, K3, s3)), n_pass, n_cu);
}

// 0 if the pieces of LDS lie apart and hold what the kernel with two images puts there: the image, three biases, two outputs of the first layer
// (the second one also that layer's weights), one of the second.
extern "C" int tower_overlap(int H, int W, int s, int s3)
{
    const int OH1 = out_side(H, K1, s), OW1 = out_side(W, K1, s), OH2 = out_side(OH1, K2, S2), OW2 = out_side(OW1, K2, S2);
    const PipePlan p = pipe_plan(H, W, OH1, OW1, OH2, OW2, out_side(OW2, K3, s3));
    int last1 = 0, last2 = 0;   // ends of the last rows written
    for (int oh = 0; oh < OH1; ++oh)
        for (int ow = 0; ow < OW1; ++ow)
            last1 = std::max(last1, ((oh & 1) * p.rows1 + (oh >> 1)) * p.pitch1 + ((ow & 1) * p.half1 + (ow >> 1)) * kRow1 + 2 * C1);
    for (int oh = 0; oh < OH2; ++oh) last2 = std::max(last2, oh * p.pitch2 + (OW2 - 1) * kRow2 + 2 * C2);
    if (p.bias < H * W * 8 || p.out1 < p.bias + (C1 + C2 + C3) * 4) return 1;
    if (last1 > p.out1_bytes || C1 * kW1Pitch > p.out1_bytes) return 2;
    if (p.out2 < p.out1 + 2 * p.out1_bytes || p.out2 + last2 > p.total) return 3;
    if (p.bias % 16 || p.out1 % 16 || p.out1_bytes % 16 || p.out2 % 16 || p.pitch1 % 16 || p.pitch2 % 16) return 4;
    return 0;
}
