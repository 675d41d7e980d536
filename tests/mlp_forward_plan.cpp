// The forward plan of the fp32 row kernel as functions that a test can call.
#include "../paper_2502_20190_amd/csrc/tj_mlp_plan.h"
#include <vector>

// Walks every load of every wave of a layer.  Returns the elements from the start of the weight copy to the end of what is loaded,
// or -1 where some weight W[n][k] of the layer is not multiplied exactly once, or not with the k that its place stands for.
extern "C" long f32_forward_reach(int in, int out, int head, int *kp, int *ldn)
{
    const tjplan::F32Forward p = tjplan::f32_forward(in, out, head != 0);
    *kp = (16 << p.lq) * p.steps;
    *ldn = p.pitch;
    std::vector<int> seen((size_t)*kp * *ldn, 0);
    long most = 0;
    for (int wave = 0; wave < tjplan::kF32Waves; ++wave) {
        const tjplan::F32Wave w = tjplan::f32_wave(p, wave);
        for (int i = 0; i < w.n; ++i) {
            const int k0 = (16 << p.lq) * (w.ks + i * p.KS);
            for (int lane = 0; lane < 64; ++lane)
                for (int b = 0; b < 4; ++b) {
                    const int part = tjplan::f32_part(lane, p.lq), f = tjplan::f32_feature(lane, w.tile, p.lq);
                    const size_t at = (size_t)k0 * p.pitch + tjplan::f32_weight_at(part, b, f, p.pitch);
                    most = std::max(most, (long)at + 4);
                    for (int e = 0; e < 4; ++e) {
                        const int k = k0 + 16 * part + 4 * b + e;   // what the kernel multiplies it with
                        if (at + e != tjplan::f32_copy_at(f, k, p.pitch) || at + e >= seen.size()) return -1;
                        ++seen[at + e];
                    }
                }
        }
    }
    for (int n = 0; n < out; ++n)
        for (int k = 0; k < in; ++k)
            if (seen[tjplan::f32_copy_at(n, k, p.pitch)] != 1) return -1;
    for (int n : seen)
        if (n > 1) return -1;
    return most;
}
