// fp32 vector networks as two or three launches per update (tj_mlp_f32.hip): everything that is per transition in one
// kernel, everything that is per weight in one or two others.
#pragma once
#include "tj_mlp_rows.h"

constexpr int kF32MaxSlices = 16;    // slices of the batch in the weight gradient

// One layer.  W and bias are the fp32 master parameters themselves.  WT is the weight copy that the forward pass reads,
// [kp / 4][ldn][4]: four input features k of an output feature, then the next output feature (kp and ldn from
// tj_f32_copy_shape; pads are zero).
// X [B][ldx] receives the layer's input rows of s (layer 0: a dense copy of the observations), dZ [B][lddz] the
// gradient wrt its output; both feed the weight-gradient kernel.
struct TjF32Layer {
    int in, out, kp, ldn;
    float *W, *bias, *WT;
    float *W_tg, *bias_tg, *WT_tg;   // target network (Q-learner)
    float *BP, *BP_tg;               // bias copies [ldn], pads zero; those of successive layers are contiguous
    float *X, *dZ;
    int ldx, lddz;
    size_t w_off, b_off;             // offsets of W and bias in the flat vectors
};

struct TjF32Rows : TjRowsCall {
    const TjF32Layer *lay;           // L of them, on the host
};

// True if the networks of this shape, in updates of up to max_batch rows, run in these kernels; decides the learner's layout.
bool tj_f32_fits(int L, const int *in, const int *out, int passes, int max_batch);
// Blocks (and with them loss_part entries) of a launch for B rows.
int tj_f32_blocks(const TjF32Rows &a, int mode);
int tj_f32_rows(const TjF32Rows &a, int mode, hipStream_t st);

// Weight gradients, Adam and everything that follows the master parameters.
struct TjF32Update : TjUpdateCall {
    TjF32Layer lay[TJ_MAX_LAYERS];
};
void tj_f32_copy_shape(TjF32Layer &y, bool head);                // kp and ldn of a layer, from in and out
size_t tj_f32_copy_at(const TjF32Layer &y, int n, int k);         // element of WT that is W[n][k]
int tj_f32_cast(int L, const TjF32Layer *lay, bool online, hipStream_t st);   // WT and BP of one network from its parameters
int tj_f32_slices(int L, const TjF32Layer *lay, int B);
int tj_f32_update(const TjF32Update &a, hipStream_t st);
