// The plan of the whole-network kernels as functions that a test can call.
#include "../paper_2502_20190_amd/csrc/tj_mlp_plan.h"
#include <vector>

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

// Walks every load of the sixteen-row backward pass over a matrix [rows][cols].  Returns the columns of the gradient it multiplies, and in
// *written the columns of the result it writes, or -1 where some weight is not multiplied exactly once, meets another row's gradient or
// reaches another column's sum.
extern "C" int f32_back16_reach(int rows, int cols, int *written)
{
    const int pitch = cols, steps = tjplan::f32_back16_steps(rows), tiles = tjplan::f32_back16_tiles(cols);
    std::vector<int> seen((size_t)rows * cols, 0);
    int read = 0;
    *written = 0;
    for (int wave = 0; wave < tjplan::kF32Waves; ++wave)
        for (int tile = wave; tile < tiles; tile += tjplan::kF32Waves)
            for (int lane = 0; lane < 64; ++lane) {
                const int first = tjplan::f32_back16_col(lane >> 4, tile);
                *written = std::max(*written, first + 8);
                for (int step = 0; step < steps; ++step)
                    for (int j = 0; j < 8; ++j)
                        for (int e = 0; e < 2; ++e) {
                            const int n = tjplan::f32_back16_dz(lane >> 4, step) + tjplan::f32_back16_row(j);
                            read = std::max(read, n + 1);
                            const long at = (tjplan::f32_back16_at(lane >> 4, lane & 15, tile, step, 4 * pitch) + tjplan::f32_back16_row(j) * 4l * pitch) / 4 + e;
                            // matrix instruction: row lane % 16 of its first operand is row 4 q + i of the result, register i of quarter q; the
                            // kernel takes register i of operand e as element 2 i + e of the quarter's eight columns
                            const int m = lane & 15, k = 32 * tile + 8 * (m / 4) + 2 * (m % 4) + e;
                            if (k >= cols) continue;                       // a sum that nobody reads
                            if (n >= rows) { if (at < (long)rows * cols) return -1; continue; }   // zero, from past the end
                            if (at != (long)n * pitch + k) return -1;
                            ++seen[at];
                        }
            }
    for (int n : seen)
        if (n != 1) return -1;
    return read;
}

// Floats of LDS per group of four rows that the head's slices take, and those they have.
extern "C" int f32_head_floats(int in, int out, int *held)
{
    const tjplan::F32Forward p = tjplan::f32_forward(in, out, true);
    const Layer lay = {in, out};
    const tjplan::F32Lds o = tjplan::f32_lds(1, &lay, 1, false, true);
    *held = o.dz - o.part;
    return std::min(p.KS, p.steps) * 4 * 16 * p.tiles;
}

// Where the arrays of a network's rows end in LDS: floats between activation rows, between gradient rows.
extern "C" void f32_pitches(int L, const Layer *lay, int nr, int *row, int *gradient)
{
    const tjplan::F32Lds o = tjplan::f32_lds(L, lay, nr, false, true);
    *row = o.pitch; *gradient = o.dzp;
}

// The same of the row kernel of bf16 networks.
extern "C" int b16_rows(int L, const Layer *lay, int B, int dqn, int backward) { return 16 * tjplan::b16_groups(L, lay, B, dqn, backward); }
extern "C" int b16_fits(int L, const Layer *lay, int passes, int max_batch)
{
    int in[TJ_MAX_LAYERS], out[TJ_MAX_LAYERS];
    for (int l = 0; l < L && l < TJ_MAX_LAYERS; ++l) { in[l] = lay[l].in; out[l] = lay[l].out; }
    return tjplan::b16_fits(L, in, out, passes, max_batch);
}
