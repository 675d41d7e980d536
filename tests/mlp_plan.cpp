// The plan of the whole-network kernels as functions that a test can call.
#include "../paper_2502_20190_amd/csrc/tj_mlp_plan.h"

struct Layer { int in, out; };

// Gradient slices that the arena of a learner for up to max_batch rows holds, and the most that any of its updates writes.
extern "C" void b16_slices(int L, const Layer *lay, int max_batch, int *held, int *written)
{
    *held = tjplan::b16_slices(L, lay, max_batch);
    *written = 0;
    for (int B = 1; B <= max_batch; ++B) {
        tjplan::B16Update p;
        if (tjplan::b16_update(L, lay, B, p) == 64 && p.S > *written) *written = p.S;
    }
}

// Elements from the start of a weight matrix to the end of what the row kernel of fp32 networks loads of it: every wave's first
// chunk, whether it is used or not, and the chunks it multiplies.
extern "C" long f32_reach(int pitch, int rows, int cols)
{
    const tjplan::F32Phase p = tjplan::f32_phase(pitch, rows, cols);
    long most = 0;
    auto load = [&](int chunk, int f) {
        for (int lane = 0; lane < 64; ++lane)
            for (int b = 0; b < 4; ++b)
                most = std::max(most, (long)tjplan::f32_chunk_at(chunk, pitch) + 4 +
                                          tjplan::f32_lane_at(tjplan::f32_row_at(lane, b, pitch), tjplan::f32_last_row_at(chunk, rows, pitch), lane, f));
    };
    for (int wave = 0; wave < tjplan::kF32Waves; ++wave) {
        const int ks = wave / p.F, f = wave % p.F;
        load(tjplan::f32_first_chunk(ks, p.nk), f);
        if (ks < p.KS)
            for (int c = ks; c < p.nk; c += p.KS) load(c, f);
    }
    return most;
}

// Waves that multiply in a phase (a mask), and how many of them the memory for their partial sums is laid out for.
extern "C" unsigned f32_active(int pitch, int rows, int cols, int *held)
{
    const tjplan::F32Phase p = tjplan::f32_phase(pitch, rows, cols);
    unsigned mask = 0;
    for (int wave = 0; wave < tjplan::kF32Waves; ++wave)
        if (wave / p.F < p.KS && wave / p.F < p.nk) mask |= 1u << wave;
    *held = tjplan::f32_part_waves(p);
    return mask;
}

// Rows of a block of the row kernel of fp32 networks, and whether a learner of that shape runs there.
extern "C" int f32_rows(int L, const Layer *lay, int B, int dqn, int backward) { return 4 * tjplan::f32_groups(L, lay, B, dqn, backward); }
extern "C" int f32_fits(int L, const Layer *lay, int passes, int max_batch)
{
    int in[TJ_MAX_LAYERS], out[TJ_MAX_LAYERS];
    for (int l = 0; l < L && l < TJ_MAX_LAYERS; ++l) { in[l] = lay[l].in; out[l] = lay[l].out; }
    return tjplan::f32_fits(L, in, out, passes, max_batch);
}
