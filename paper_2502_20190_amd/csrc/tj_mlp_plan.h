// How the whole-network kernels (tj_mlp_f32.hip, tj_mlp_b16.hip) divide an update: plain host arithmetic without HIP, so
// that it can be compiled and checked on its own.  `Layer` is anything with the members in and out.
#pragma once
#include "../../include/tianji.h"
#include <math.h>
#include <stddef.h>
#include <algorithm>

#ifdef __HIPCC__
#define TJ_HD __host__ __device__
#else
#define TJ_HD
#endif

namespace tjplan {

// ---- the row kernel of fp32 networks
constexpr int kF32Waves = 8;

// The forward pass of a layer.  The weight copy is [k / 4][pitch][4]; a wave takes a tile of 64 / q features, its q lane
// parts a chunk of 16 k each of a step of 16 q, and every KS-th step from its slice's on.  A hidden layer has as many tiles as eight
// waves can be given and no slices, so that a wave ends with whole sums; the head, whose few outputs make few tiles, has slices
// instead, which whoever needs the outputs adds.
struct F32Forward {
    int pitch, lq, tiles, KS, steps;     // q = 1 << lq
};
inline F32Forward f32_forward(int in, int out, bool head)
{
    F32Forward p;
    p.pitch = (out + 63) / 64 * 64;
    p.lq = head || p.pitch <= 128 ? 2 : p.pitch <= 256 ? 1 : 0;
    p.tiles = head ? (out + 15) / 16 : (p.pitch << p.lq) / 64;
    p.KS = head ? std::min(4, kF32Waves / p.tiles) : 1;
    p.steps = (in + (16 << p.lq) - 1) / (16 << p.lq);
    return p;
}
// A wave's tile, slice and number of steps (wave = slice tiles + tile): steps slice, slice + KS, ... < p.steps, or none.
struct F32Wave { int tile, ks, n; };
inline F32Wave f32_wave(const F32Forward &p, int wave)
{
    F32Wave w;
    w.ks = wave / p.tiles;
    w.tile = wave - w.ks * p.tiles;
    w.n = w.ks < p.KS && w.ks < p.steps ? (p.steps - w.ks + p.KS - 1) / p.KS : 0;
    return w;
}
TJ_HD inline int f32_part(int lane, int lq) { return lane >> (6 - lq); }   // lane part
TJ_HD inline int f32_feature(int lane, int tile, int lq) { return (tile << (6 - lq)) + (lane & ((64 >> lq) - 1)); }
// Element from a step's first k on that load b takes for feature f, with the three behind it: k = 16 part + 4 b ..
TJ_HD inline unsigned f32_weight_at(int part, int b, int f, int pitch) { return (4u * part + b) * 4u * pitch + 4u * f; }
TJ_HD inline size_t f32_copy_at(int n, int k, int pitch) { return ((size_t)(k >> 2) * pitch + n) * 4 + (k & 3); }

// A phase of the backward pass: one contraction of a block's rows with a weight matrix [rows][columns] as stored, as F groups
// of 64 columns x KS slices of the nk chunks of 16 rows, one per wave.
struct F32Phase {
    int pitch, rows, nk, F, KS;     // pitch: elements between rows of the matrix
};
inline F32Phase f32_phase(int pitch, int rows, int cols)
{
    F32Phase p;
    p.pitch = pitch; p.rows = rows; p.nk = (rows + 15) / 16; p.F = (cols + 63) / 64; p.KS = kF32Waves / p.F;
    return p;
}
// Waves 0 .. n - 1 have a part of the phase (wave = ks F + f).
inline int f32_part_waves(const F32Phase &p) { return p.F * std::min(p.KS, p.nk); }
// A wave whose slice is ks multiplies chunks ks, ks + KS, ... < nk, or none (ks >= KS or ks >= nk).  Its first load goes out
// before that is decided, so it is of a chunk that exists.
TJ_HD inline int f32_first_chunk(int ks, int nk) { return ks < nk ? ks : nk - 1; }
// Element of the matrix at which load b of a chunk starts, four features wide: the chunk's part, and the lane's from the start of
// row 4 b + lane / 16 of the chunk.  Rows past the matrix meet zeros of the other operand and are its last row instead: what
// lies behind the matrix need not be finite.
TJ_HD inline unsigned f32_chunk_at(int chunk, int pitch) { return 16u * chunk * pitch; }
TJ_HD inline unsigned f32_row_at(int lane, int b, int pitch) { return (unsigned)(lane >> 4) * pitch + 4u * b * pitch; }
TJ_HD inline unsigned f32_last_row_at(int chunk, int rows, int pitch) { return (unsigned)(rows - 1 - 16 * chunk) * pitch; }
TJ_HD inline unsigned f32_lane_at(unsigned row_at, unsigned last_row_at, int lane, int f)
{
    return (row_at < last_row_at ? row_at : last_row_at) + 64u * f + 4u * (lane & 15);
}

// The backward pass of sixteen rows: v_mfma_f32_16x16x4_f32, the weights its first operand (columns of the matrix as stored), the rows the second,
// so that a wave ends with whole sums: a tile of 32 columns, every eighth one.  Load j of a step of 32 matrix rows takes row
// 16 (j / 4) + 4 q + j % 4 in lane quarter q, columns 2 c, 2 c + 1 (c = lane % 16), and multiplies them with element 16 (j / 4) + j % 4 of the lane's
// part of the gradient; columns 8 q .. 8 q + 7 of row c are the lane's sums.  What lies past the matrix is zero.
TJ_HD inline int f32_back16_steps(int rows) { return (rows + 31) / 32; }
TJ_HD inline int f32_back16_tiles(int cols) { return (cols + 31) / 32; }
TJ_HD inline int f32_back16_at(int q, int c, int tile, int step, int pitch)   // bytes to the lane's part of a step, pitch in bytes
{
    return (32 * step + 4 * q) * pitch + 128 * tile + 8 * c;
}
TJ_HD inline int f32_back16_row(int j) { return 16 * (j / 4) + j % 4; }   // load j's row from there; its element of the gradient
TJ_HD inline int f32_back16_dz(int q, int step) { return 32 * step + 4 * q; }   // the lane's part of the gradient
TJ_HD inline int f32_back16_col(int q, int tile) { return 32 * tile + 8 * q; }  // its first column of the result

// LDS layout of the row kernel in floats.  Activation rows are `pitch` floats apart, pitch % 64 == 16: the 16-byte pieces that a
// quarter of a wave reads (four rows x 16 k) cover the 64 banks once.
constexpr size_t kF32Lds = 160 * 1024;
struct F32Lds {
    int pitch, dzp, keep, pp, part, dz, wa, bias, small, total;
};
// nr groups of four rows per block; dqn: the Q-learner's three passes; backward: an update, not acting.
template <typename Layer> F32Lds f32_lds(int L, const Layer *lay, int nr, bool dqn, bool backward)
{
    F32Lds o;
    int w = 0, nb = 0, waves = 0;   // waves: those with a part of some phase of the backward pass with slices
    for (int l = 0; l < L; ++l) {
        if (backward && l && nr < 4) waves = std::max(waves, f32_part_waves(f32_phase(lay[l].in, lay[l].out, lay[l].in)));
        w = std::max(w, std::max(lay[l].in, lay[l].out));   // steps of 16, 32 or 64 inputs end within whole 64 columns
        nb += (lay[l].out + 63) / 64 * 64;
    }
    o.pitch = (w + 63) / 64 * 64 + 16;
    const int R = 4 * nr, NG = dqn ? 3 * nr : nr;
    int at = 0;
    o.keep = at; at += (backward ? L : std::min(L, 2)) * R * o.pitch;   // input rows of every layer, s; acting: two layers in turn
    o.pp = at; at += dqn ? 2 * 2 * R * o.pitch : 0;     // s' (online), s' (target), two layers in turn
    o.part = at; at += std::max(waves * nr * 256, kF32Waves * NG * 64);   // the slices of a backward phase; of the head
    // output gradients, two layers in turn; sixteen rows are read side by side, 16 bytes each: their pitch keeps them on distinct banks
    o.dzp = o.pitch + (nr == 4 ? 4 : 0);
    o.dz = at; at += backward ? 2 * R * o.dzp : 0;
    o.wa = at; at += dqn ? R * o.pitch : 0;             // head weights of the actions taken
    o.bias = at; at += nb * (dqn ? 2 : 1);
    o.small = at; at += 64;                             // per row: loss terms, gradient
    o.total = at;
    return o;
}

// Groups of four rows per block: the fewest that need no second round of blocks on the chip, or the most that LDS holds.  The
// Q-learner's second group fits unless the network is deep and wide (us per update with one group and the partial sums that kept the second
// one out : with two groups; 128-256-256-18 at 2048 rows 71.8 : 54.3, 8192 197 : 132, 64-128 x 6-8 at 2000 93.7 : 62.9, 300-384-384-384-33 at
// 4096 313 : 227).
// Acting on rows of at most kF32ActPaired floats stays at two groups, whose blocks find place in pairs on a CU: one hides the other's
// latency.  On wider rows the weights, read once per block, weigh more (us for 32768 rows, two groups : four; 4-64-64-3 51 : 61,
// 128-256-256-19 121 : 134, 64-384-384-7 187 : 206, 128-512-512-19 294 : 286, 256-512-512-512-33 547 : 499).
constexpr int kF32ActPaired = 384 + 16;
template <typename Layer> int f32_groups(int L, const Layer *lay, int B, bool dqn, bool backward)
{
    const int most = dqn ? 2 : !backward && f32_lds(L, lay, 2, dqn, backward).pitch <= kF32ActPaired ? 2 : 4;
    int best = 1;
    for (int nr = 1; nr <= most; nr *= 2) {
        if (f32_lds(L, lay, nr, dqn, backward).total * sizeof(float) > kF32Lds) break;
        best = nr;
        if ((B + 4 * nr - 1) / (4 * nr) <= 256) break;   // one round of blocks on the chip
    }
    return best;
}

// Largest batch of a Q-learner that is updated here.  One group of four rows per block reads the weights of both networks for every four
// or eight transitions, and past some batch the layered kernels, whose tiles share them, are faster (us here : there; 128-512-512-512-18 at 8192
// rows 729 : 844, 16384 1419 : 1397, 32768 2865 : 2696; 300-500-384-500-33 at 8192 702 : 772, 16384 1400 : 1313).  The lines are older than
// the present forward pass, which is the faster one past them too where layers are narrower or fewer (128-384-384-384-18 at 32768 1494 : 1831,
// 4-512-512-2 1358 : 1516, 128-256-256-18 at 65536 912 : 1233, 16-32-5 215 : 268).
constexpr int kF32QRows = 16384, kF32QRowsWide = 8192, kF32QWide = 256 + 16;   // the latter past rows of kF32QWide floats

constexpr int kF32MaxWidth = 512;    // widest layer (eight 64-feature groups)
constexpr int kF32MaxInput = 1024;   // widest observation
constexpr int kF32MaxOut = 64;       // head outputs: one lane each

// Q-learners with updates of few rows that run layer by layer.  Few blocks leave the weights' stream into each what it is: 12.3 us per MB of both
// networks' forward pass, 12.5 per MB of the backward pass (5 where 32 blocks ask for the same weights in the L2), while a layer's launches
// take 23 - 25 us (us here : there; 1024-512-18 at 8 rows 65 : 48, at 128 66 : 55, at 256 60 : 69; 512-512 x 6-18 at 32 rows 233 : 185, at 128
// 194 : 188, at 256 192 : 220; 128-512 x 4-64 at 32 138 : 127, at 128 119 : 132; 768-384-384-384-18 at 32 91 : 91).  Only networks are asked that need
// more LDS than kF32FewRowsLds, those that could not run here while the forward pass kept partial sums in LDS; the others lose 18 % of an
// update at the worst (512-512-512-512-18 at 32 rows 116 : 98) and act on 8 observations in 27 us instead of 42.
constexpr int kF32FewRows = 128;
constexpr size_t kF32FewRowsLds = 116 * 1024;
inline bool f32_few_rows(int L, const int *in, const int *out, size_t lds, int max_batch)
{
    if (max_batch > kF32FewRows || lds <= kF32FewRowsLds) return false;
    double forward = 0, backward = 0;   // MB
    for (int l = 0; l < L; ++l) {
        forward += 8e-6 * in[l] * out[l];
        if (l > 0 && l + 1 < L) backward += 4e-6 * in[l] * out[l];
    }
    return 18 + 12.3 * forward + (max_batch <= 64 ? 12.5 : 5) * backward > (23 + max_batch / 64.0) * L;
}

// On-policy learners with long updates that run layer by layer.  Where LDS holds one group of four rows, every four transitions read the
// weights of a forward and a backward pass (11.5 us per MB and round of blocks), past some batch for longer than the layered kernels take,
// whose tiles share them (us here : there; 896-256 x 7-18 at 8192 rows 599 : 788, 16384 1203 : 1014, 65536 4766 : 3344; 1024-320 x 6-18 at 16384
// 1657 : 1542; 1024-192 x 6-18 at 16384 821 : 918, 32768 1641 : 1593; 1024-128 x 6-3 at 32768 972 : 937; 896-64 x 7-18 at 65536 1410 : 1466).  Only networks
// are asked that need more LDS than kF32LongRowsLds, as above; the others lose up to 32 % of an update (1024-256 x 5-18 at 32768 2022 : 1530) and act in
// one launch instead of one per layer.
constexpr int kF32LongRows = 8192;
constexpr size_t kF32LongRowsLds = 150 * 1024;
constexpr double kF32LongRowsRead = 38e3;   // rows x MB
inline bool f32_long_rows(int L, const int *in, const int *out, size_t lds, int max_batch)
{
    if (max_batch <= kF32LongRows || lds <= kF32LongRowsLds) return false;
    double mb = 0;
    for (int l = 0; l < L; ++l) mb += (l > 0 ? 8e-6 : 4e-6) * in[l] * out[l];
    return mb * max_batch > kF32LongRowsRead;
}

// True if a learner of this shape, with updates of up to max_batch rows in `passes` forward passes (the Q-learner's three), runs in
// these kernels.
inline bool f32_fits(int L, const int *in, const int *out, int passes, int max_batch)
{
    if (L < 1 || L > TJ_MAX_LAYERS || in[0] > kF32MaxInput || out[L - 1] > kF32MaxOut) return false;
    struct { int in, out; } lay[TJ_MAX_LAYERS];
    for (int l = 0; l < L; ++l) {
        if (l + 1 < L && out[l] > kF32MaxWidth) return false;
        lay[l].in = in[l]; lay[l].out = out[l];
    }
    const F32Lds o = f32_lds(L, lay, 1, passes == 3, true);
    if (passes == 3 && max_batch > (o.pitch > kF32QWide ? kF32QRowsWide : kF32QRows)) return false;
    const size_t lds = o.total * sizeof(float);
    if (passes == 3 ? f32_few_rows(L, in, out, lds, max_batch) : f32_long_rows(L, in, out, lds, max_batch)) return false;
    return lds <= kF32Lds;
}

// ---- the row kernel of bf16 networks
constexpr size_t kB16Lds = 160 * 1024;
constexpr int kB16MaxWidth = 1024;   // widest layer and observation
constexpr int kB16MaxOut = 32;       // head outputs: one block of 32 features
constexpr int kPartPitch = 36;       // floats per row of the head's partial sums
constexpr int kZPitch = 144;         // bytes per row of dL/dQ (64 columns)

// LDS layout in bytes.  Activation rows are `pitch` bytes apart, pitch % 128 == 16: the 16-byte pieces that eight neighbouring lanes
// read fall on distinct banks.
struct B16Lds {
    int pitch, keep, pp, part, dz, bias, small, total, n_bias;
};
// nr groups of sixteen rows per block; dqn: the Q-learner's three passes; backward: an update, not acting.
template <typename Layer> B16Lds b16_lds(int L, const Layer *lay, int nr, bool dqn, bool backward)
{
    B16Lds o;
    int w = 0;
    o.n_bias = 0;
    for (int l = 0; l < L; ++l) {
        w = std::max(w, (lay[l].in + 63) / 64 * 64);
        o.n_bias += (lay[l].out + 31) / 32 * 32;
    }
    const int R = 16 * nr, ns = 4;
    o.pitch = 2 * w + 16;
    const int part = ns * (dqn ? 3 : 1) * R * kPartPitch * 4, half = dqn ? 2 * R * o.pitch : 0;
    int at = 0;
    // s' under both networks, two layers in turn; input rows of the layers, s, behind it: those of the first layer take the
    // place of s' under the target network, where the first layer has no rows of its own
    o.pp = at; at += 2 * half;
    o.keep = dqn ? at - R * o.pitch : at;
    at = o.keep + (backward ? L : std::min(L, 2)) * R * o.pitch;
    // the head's partial sums take memory that is free by then if they fit: the half of pp that the head's input does not
    // use, or the first layer's input (its fragments are written at the start)
    const bool in_pp = dqn && part <= half, in_keep = !dqn && L >= 2 && (backward || (L - 1) % 2) && part <= R * o.pitch;
    o.part = in_pp ? o.pp + ((L - 1) & 1 ? half : 0) : in_keep ? o.keep : at;
    if (!in_pp && !in_keep) at += part;
    o.dz = at; at += backward ? R * kZPitch : 0;
    o.bias = at; at += o.n_bias * (dqn ? 2 : 1) * 4;
    o.small = at; at += 3 * R * 4;
    o.total = at;
    return o;
}

// Groups of sixteen rows per block: the fewest that need no second round of blocks on the chip, or the most that LDS holds.
template <typename Layer> int b16_groups(int L, const Layer *lay, int B, bool dqn, bool backward)
{
    int best = 1;
    for (int nr = 1; nr <= (dqn ? 2 : 4); nr *= 2) {
        if ((size_t)b16_lds(L, lay, nr, dqn, backward).total > kB16Lds) break;
        best = nr;
        if ((B + 16 * nr - 1) / (16 * nr) <= 256) break;
    }
    return best;
}

// True if a learner of this shape, with updates of up to max_batch rows, runs in these kernels.
inline bool b16_fits(int L, const int *in, const int *out, int passes, int max_batch)
{
    if (L < 1 || L > TJ_MAX_LAYERS || in[0] > kB16MaxWidth || out[L - 1] > kB16MaxOut) return false;
    struct { int in, out; } lay[TJ_MAX_LAYERS];
    for (int l = 0; l < L; ++l) {
        if (l + 1 < L && out[l] > kB16MaxWidth) return false;
        lay[l].in = in[l]; lay[l].out = out[l];
    }
    const bool dqn = passes == 3;
    // The line below was measured when the kernel kept 33 floats per row and pass more in LDS.  Which networks come here follows that size
    // still, and so does the number of groups in the estimate; the launch takes what b16_groups says.  Networks that this alone keeps out are
    // mostly faster here (us here : layer by layer; double DQN 384-64 x 6-18 at 512 rows 23 : 155, 768-512-512-18 at 2048 58 : 81, 640-640 x 3-18 at 64
    // 93 : 85; on-policy 128-384 x 5-18 at 32768 283 : 490, 768-512 x 5-18 at 64 80 : 122): room to move the line, with the estimate's figures.
    auto holds = [&](int nr) { return (size_t)b16_lds(L, lay, nr, dqn, true).total + (dqn ? 3 : 1) * 16 * nr * 33 * sizeof(float) <= kB16Lds; };
    if (!holds(1)) return false;
    // Against one GEMM per layer (an update of 90 us and 820 TFLOP/s on 128-1024-1024-1024-19 at 4096 .. 32768 rows): the
    // weights every block streams (120 GB/s per CU) and 8 us per round of blocks, then the weight gradient at 400 TFLOP/s.
    // Wide networks on long batches are better off as GEMMs, whose tiles share the weights.
    double params = 0, stream = 0;   // bytes of one block
    for (int l = 0; l < L; ++l) {
        params += (double)in[l] * out[l];
        stream += 2.0 * in[l] * out[l] * (passes == 3 ? 2 : 1) + (l ? 2.0 * in[l] * out[l] : 0.0);
    }
    const int nr = holds(2) ? 2 : 1;
    const double rounds = std::max(1.0, std::ceil(max_batch / (256.0 * 16 * nr)));
    const double whole_us = rounds * (8 + stream / 0.12e6) + 15 + 2 * params * max_batch / 400e6;
    const double gemms_us = 90 + 2 * params * max_batch * (passes + 2) / 820e6;
    return whole_us <= gemms_us;
}

// ---- the weight kernel of bf16 networks

constexpr int kB16MaxSlices = 16;    // slices of the batch in the bf16 weight gradient

struct B16Update {
    int begin[TJ_MAX_LAYERS + 1];   // first tile of every layer
    int nk[TJ_MAX_LAYERS];          // tiles along k
    int S, steps, per;              // slices; 32-row steps of the batch, of a slice
};

template <typename Layer> int b16_tiles(int L, const Layer *lay, int tile, B16Update &p)
{
    int n = 0;
    for (int l = 0; l < L; ++l) {
        p.begin[l] = n;
        p.nk[l] = (lay[l].in + tile - 1) / tile;
        n += p.nk[l] * ((lay[l].out + tile - 1) / tile);
    }
    p.begin[L] = n;
    return n;
}

// 32 x 32 tiles while their operand traffic (128 bytes per tile and row) stays below what a second launch costs; then
// 64-wide tiles and the number of slices with the least estimated time: rounds of 256 blocks (one per CU) of 5 us and
// 94 ns per 32-row step, and a pass over the slices at 5 TB/s (128-512-512-512-18, 32768 rows: 96 us with one
// slice on 152 blocks).  Returns the tile side.
template <typename Layer> int b16_update(int L, const Layer *lay, int B, B16Update &p)
{
    p.steps = (B + 31) / 32;
    p.S = 1;
    p.per = p.steps;
    int n = b16_tiles(L, lay, 32, p);
    if ((size_t)n * B <= 400000) return 32;
    n = b16_tiles(L, lay, 64, p);
    float best = 0.f;
    for (int S = 1; S <= std::min(kB16MaxSlices, std::max(1, p.steps / 8)); ++S) {
        const int per = (p.steps + S - 1) / S;
        const float ns = (float)((n * S + 255) / 256) * (5000.f + 94.f * per) + (float)n * 4096 * 8 / 5000 * S;
        if (S == 1 || ns < best) { best = ns; p.S = S; p.per = per; }
    }
    return 64;
}

// Most gradient slices that an update of B rows or fewer writes.  The count follows the steps but not evenly, and only 64-wide
// tiles have any; of the batches with the same steps the longest one is the first to take them, so it speaks for all.
template <typename Layer> int b16_slices(int L, const Layer *lay, int B)
{
    int most = 0;
    for (int steps = (B + 31) / 32; steps > 0; --steps) {
        B16Update p;
        if (b16_update(L, lay, std::min(32 * steps, B), p) == 64) most = std::max(most, p.S);
    }
    return most;
}

}  // namespace tjplan
