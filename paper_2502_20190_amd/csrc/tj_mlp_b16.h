// bf16 vector networks as two or three launches per update (tj_mlp_b16.hip): everything that is per transition in one
// kernel, everything that is per weight in one or two others.
#pragma once
#include "tj_mlp_rows.h"
#include "tj_gemm.h"

// A matrix operand is stored as the matrix instruction takes it: fragments of 16 rows x 32 contraction elements, 1 KB,
// lane (q, n) = row n, elements 8 q .. 8 q + 7; four of them (two row tiles x two steps) make a contiguous 4 KB group
// of 32 rows x 64 elements, the groups of 32 rows follow each other along the contraction.
__host__ __device__ inline size_t tj_b16_group_off(int row, int c, int cp)   // element (row, c), cp groups along c
{
    return ((((size_t)(row >> 5) * cp + (c >> 6)) * 4 + ((row >> 4) & 1) * 2 + ((c >> 5) & 1)) * 64 +
            ((c >> 3) & 3) * 16 + (row & 15)) * 8 + (c & 7);
}

// One layer.  Fragments of the weights: WF with the outputs as rows (forward), WB with the inputs as rows (input
// gradient; absent for the first layer).  XF, ZF: the layer's input rows of s and the gradient wrt its output,
// features as rows and transitions as the contraction, 32 features x 32 transitions per 2 KB.
struct TjB16Layer {
    int in, out;
    float *W, *bias, *W_tg, *bias_tg;   // fp32 master parameters
    tj_bf16 *WF, *WB;                   // the target network's WF follows the online one's
    float *BP, *BP_tg;                  // bias copies padded to whole groups; all layers' online ones, then all target ones, contiguous
    tj_bf16 *XF, *ZF;
    size_t w_off, b_off;                // offsets of W and bias in the flat vectors
};
inline size_t tj_b16_wf_elems(int in, int out) { return (size_t)((out + 31) / 32) * ((in + 63) / 64) * 2048; }
inline size_t tj_b16_wb_elems(int in, int out) { return (size_t)((in + 31) / 32) * ((out + 63) / 64) * 2048; }
inline size_t tj_b16_frag_elems(int width, int rows) { return (size_t)((width + 31) / 32) * ((rows + 31) / 32) * 1024; }

struct TjB16Rows : TjRowsCall {
    TjB16Layer lay[TJ_MAX_LAYERS];
};

// True if the networks of this shape run in these kernels; decides the learner's layout.
bool tj_b16_fits(int L, const int *in, const int *out, int passes, int max_batch);
// Blocks (and with them loss_part entries) of a launch for B rows; at most tj_b16_max_blocks(B).
int tj_b16_blocks(const TjB16Rows &a, int mode);
inline int tj_b16_max_blocks(int B) { return (B + 31) / 32 * 2; }
int tj_b16_rows(const TjB16Rows &a, int mode, hipStream_t st);

struct TjB16Update : TjUpdateCall {
    TjB16Layer lay[TJ_MAX_LAYERS];
};
int tj_b16_slices(int L, const TjB16Layer *lay, int B);   // most that an update of B rows or fewer writes
int tj_b16_update(const TjB16Update &a, hipStream_t st);
// Fragments and padded biases of one network from its master parameters.
int tj_b16_cast(int L, const TjB16Layer *lay, bool online, hipStream_t st);
