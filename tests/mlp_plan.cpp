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
