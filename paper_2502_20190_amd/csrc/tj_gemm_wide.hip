// The large contractions of wide vector networks (hidden layers at batches of thousands): 256 x 256 tiles, one block of eight
// waves per compute unit.  Same problems, operand forms and sums as gemm_bf16_dlds (tj_gemm.hip), bit for bit where a
// result is one accumulation; tj_gemm_wide_* and the rules of tj_gemm_plan.h say which calls they take.
//
// What bounds these contractions is power: with all matrix cores busy on real data the clock falls from 2.4 to 1.5 - 1.8 GHz (the same
// kernel on zeros runs at 2.2).  A bare loop of v_mfma_f32_32x32x16_bf16 reaches 1.84 PFLOP/s on random operands, of
// v_mfma_f32_16x16x32_bf16 2.07, and every byte moved to the matrix cores takes its share too.  So: the 16 x 16 x 32
// instruction; 256 x 256 tiles, which load a quarter less than 256 x 128 per operation, and wave tiles of 128 x 64, which read a
// quarter less from LDS; and a loop in which nothing waits for long, since an idle unit still draws power:
//   - two stages of 64 contraction elements (128-byte rows) in LDS, filled by direct-to-LDS loads;
//   - operands go one step of 32 ahead into registers: a fragment is read again as soon as its four MFMAs are issued;
//   - one barrier per stage, in the middle of its second step, when the stage's last reads have returned: it says both that the
//     next stage is here (each wave has waited for its own loads) and that this stage's buffer may be filled again.
// Results are stored from LDS as whole lines.
#include "tj_gemm.h"
#include "tj_gemm_plan.h"
#include <algorithm>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
typedef __attribute__((address_space(3))) uint8_t *lds_u8;

constexpr int kThreads = 512, kTile = tjplan::kWideTile;
constexpr int kBufA = 32768, kBufB = 32768;              // one stage of either operand
constexpr int kBias = 2 * (kBufA + kBufB), kLds = kBias + kTile * 4;

enum { kForward = 0, kInputGrad = 1, kWeightGrad = 2 };   // bias and ReLU | ReLU mask | fp32 slices, column sums of Q

template <int N> struct IntC { static constexpr int value = N; };

__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ void wave_sync()   // LDS accesses of one wave, in order
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// One tile, 256 (i) x 64 * WJ (j), contraction elements [k_begin, k_begin + 64 n_stage).  Waves WI (i) x WJ (j).
// KIND kWeightGrad: both operands contraction-major; kInputGrad: P only; kForward: neither.
template <int KIND, int WJ>
__device__ __forceinline__ void tile(const TjGemmArgs<tj_bf16> &a, const TjGemmSeg<tj_bf16> &seg, const int i0, const int j0,
                                     const int z, const int sum_lo, const int sum_step, uint8_t *lds)
{
    constexpr bool TP = KIND != kForward, TQ = KIND == kWeightGrad;
    constexpr int WI = 8 / WJ, NJ = 64 * WJ;
    constexpr int FI = kTile / WI / 16, FJ = 4, LB = NJ / 64;   // fragments of a wave, load instructions of Q per wave and stage
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wj = wave % WJ, wi = wave / WJ;
    const int j_end = seg.j_end;
    const int k_begin = z * a.k_chunk, n_stage = (min(a.K, k_begin + a.k_chunk) - k_begin) / 64;

    // ---- loads.  A contraction-major operand is halves of [64 k][128 columns], 256-byte rows, vector v of row r at
    // v ^ ((r & 3) << 2) ^ ((r >> 2) & 2); the other form is 128-byte rows, vector v of row r at v ^ ((r >> 1) & 7).  Rows and columns
    // past the end repeat the last ones.
    uint32_t oA[4], oB[LB];
    auto offset = [&](int c, bool trans, int ld, int left) -> uint32_t {   // instruction c of a stage; `left` rows or columns exist
        if (trans) {
            const int row = 4 * (c & 15) + (lane >> 4), v = (lane & 15) ^ ((row & 3) << 2) ^ ((row >> 2) & 2);
            return (uint32_t)(row * ld + min((c >> 4) * 128 + v * 8, ((left + 7) & ~7) - 8)) * 2;
        }
        const int row = 8 * c + (lane >> 3), v = (lane & 7) ^ ((row >> 1) & 7);
        return (uint32_t)(min(row, left - 1) * ld + v * 8) * 2;
    };
#pragma unroll
    for (int t = 0; t < 4; ++t) oA[t] = offset(wave + 8 * t, TP, a.ldp, a.I - i0);
#pragma unroll
    for (int t = 0; t < LB; ++t) oB[t] = offset(wave + 8 * t, TQ, a.ldq, j_end - j0);
    const tj_bf16 *const bP = TP ? seg.P + (size_t)k_begin * a.ldp + i0 : seg.P + (size_t)i0 * a.ldp + k_begin;
    const tj_bf16 *const bQ = TQ ? a.Q + (size_t)k_begin * a.ldq + j0 : a.Q + (size_t)(j0 - seg.q_shift) * a.ldq + k_begin;
    const size_t stP = TP ? (size_t)64 * a.ldp : 64, stQ = TQ ? (size_t)64 * a.ldq : 64;
    // Inline assembly, so that the compiler's wait counts do not see these loads; M0 is written here and nowhere else.
    // Should the compiler keep the base in lanes of a vector register, reading it back is a vector instruction's write of a
    // scalar, which a memory instruction may read five wait states later: the move and the s_nop are six.
    auto dma = [](const tj_bf16 *base, uint32_t off, uint32_t at) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(at), "v"(off), "s"(base) : "memory");
    };
    const uint32_t l0 = (uint32_t)(uintptr_t)(lds_u8)lds + wave * 1024;
    const int k_valid = KIND == kWeightGrad && a.k_valid ? a.k_valid : a.K;
    auto issue = [&](int s, int t) {   // part t (of four) of stage s
        uint32_t off = oA[t];
        if (KIND == kWeightGrad && k_begin + (s + 1) * 64 > k_valid)   // the stage the batch ends in: no rows past the last one
            off -= max(k_begin + s * 64 + 4 * ((wave + 8 * t) & 15) + (lane >> 4) - (k_valid - 1), 0) * (uint32_t)a.ldp * 2;
        dma(bP + (size_t)s * stP, off, l0 + (s & 1) * kBufA + t * 8192);
        if (t < LB) dma(bQ + (size_t)s * stQ, oB[t < LB ? t : 0], l0 + 2 * kBufA + (s & 1) * kBufB + t * 8192);
    };

    // ---- operand fragments: 16 rows, 8 contraction elements from 8 q4 of a step of 32
    f32x4 acc[FI][FJ];
#pragma unroll
    for (int f = 0; f < FI; ++f)
#pragma unroll
        for (int g = 0; g < FJ; ++g) acc[f][g] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 pa[FI], qb[2][FJ];
    const int tr_row = 8 * q4 + (l16 >> 2);
    const int tr_off = tr_row * 256 + (((l16 & 3) >> 1) << 4) + (l16 & 1) * 8;
    const int tr_x = ((((l16 >> 2) & 3) << 2) ^ ((tr_row >> 2) & 2)) << 4;
    auto read_t = [&](const uint8_t *base, int ks, int col) {   // columns col .. + 15 of a half; rows + 4 and + 32 have the same swizzle
        const uint8_t *p = base + ks * 8192 + tr_off + ((col * 2) ^ tr_x);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + 1024));
        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
        const u32x4 v = {l2.x, l2.y, h2.x, h2.y};
        return v;
    };
    const int swz = (((l16 >> 1) & 7) ^ q4) * 16;
    const int rA = (wi * FI * 16 + l16) * 128 + swz, rB = 2 * kBufA + (wj * 64 + l16) * 128 + swz;
    auto readA = [&](int par, int ks, int f) {
        if constexpr (TP) {
            const int col = wi * FI * 16 + f * 16;
            pa[f] = read_t(lds + par * kBufA + (col >> 7) * 16384, ks, col & 127);
        } else {
            pa[f] = *(const u32x4 *)(lds + ((rA ^ (ks * 64)) + par * kBufA + f * 2048));
        }
    };
    auto readB = [&](int par, int ks, int g) {
        if constexpr (TQ) {
            const int col = wj * 64 + g * 16;
            qb[ks][g] = read_t(lds + 2 * kBufA + par * kBufB + (col >> 7) * 16384, ks, col & 127);
        } else {
            qb[ks][g] = *(const u32x4 *)(lds + ((rB ^ (ks * 64)) + par * kBufB + g * 2048));
        }
    };
    float qs[FJ];   // kWeightGrad: sums of this lane's elements of the fragments g = sum_lo, sum_lo + sum_step, ...
#pragma unroll
    for (int g = 0; g < FJ; ++g) qs[g] = 0.f;
    const bool sums = KIND == kWeightGrad && wi == 0 && sum_lo < FJ;
    auto mm = [&](int f, int ks) {
#pragma unroll
        for (int g = 0; g < FJ; ++g)
            acc[f][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pa[f]), __builtin_bit_cast(bf16x8, qb[ks][g]),
                                                                acc[f][g], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto add_sums = [&](int ks) {
        if constexpr (KIND == kWeightGrad) {
            if (sums) {
#pragma unroll
                for (int g = 0; g < FJ; ++g)
                    if (g % sum_step == sum_lo) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            qs[g] += __uint_as_float(qb[ks][g][e] << 16) + __uint_as_float(qb[ks][g][e] & 0xFFFF0000u);
                    }
            }
        }
    };
    auto stage = [&](int s, auto kind) {   // 0: with the loads of stage s + 2; 1: the last but one; 2: the last
        constexpr int S = decltype(kind)::value;
        const int par = s & 1;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < FJ; ++g) readB(par, 1, g);
        add_sums(0);
#pragma unroll
        for (int f = 0; f < FI; ++f) { mm(f, 0); readA(par, 1, f); }
        add_sums(1);
#pragma unroll
        for (int f = 0; f < FI / 2; ++f) mm(f, 1);
        if constexpr (S < 2) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < FJ; ++g) readB(par ^ 1, 0, g);
#pragma unroll
            for (int f = 0; f < FI / 2; ++f) readA(par ^ 1, 0, f);
        }
#pragma unroll
        for (int f = FI / 2; f < FI; ++f) {
            constexpr int per = 4 / (FI / 2);   // load instructions of either operand per fragment
            if constexpr (S == 0) {
#pragma unroll
                for (int u = 0; u < per; ++u) issue(s + 2, (f - FI / 2) * per + u);
            }
            mm(f, 1);
            if constexpr (S < 2) readA(par ^ 1, 0, f);
        }
    };

    float *const bias = (float *)(lds + kBias);
    if (KIND == kForward && wave < kTile / 64) {
        const uint32_t at = (uint32_t)(uintptr_t)(lds_u8)(bias + wave * 64);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(at), "v"(seg.bias + min(i0 + tid, a.I - 1)) : "memory");
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) issue(0, t);
    if (n_stage > 1) {
#pragma unroll
        for (int t = 0; t < 4; ++t) issue(1, t);
    }
    if (n_stage > 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 + LB) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int g = 0; g < FJ; ++g) readB(0, 0, g);
#pragma unroll
    for (int f = 0; f < FI; ++f) readA(0, 0, f);
    int s = 0;
    for (; s + 2 < n_stage; ++s) stage(s, IntC<0>{});
    if (n_stage > 1) stage(s++, IntC<1>{});
    stage(s, IntC<2>{});
    __syncthreads();   // the stages have been read: their memory takes the results

    // ---- acc[f][g][r]: i = i0 + 16 (wi FI + f) + 4 q4 + r, j = j0 + 64 wj + 16 g + l16
    const int ib = i0 + wi * FI * 16, jb = j0 + wj * 64;
    if constexpr (KIND == kWeightGrad) {
        if (sums) {
#pragma unroll
            for (int g = 0; g < FJ; ++g) {
                if (g % sum_step != sum_lo) continue;
                float t = qs[g] + __shfl_xor(qs[g], 16, 64);
                t += __shfl_xor(t, 32, 64);
                const int j = jb + 16 * g + l16;
                if (q4 == 0 && j < j_end) a.qsum[(size_t)z * a.qsum_zstride + j] = t;
            }
        }
        constexpr int W = FI * 16, pitch = W * 4 + 16, V = W / 4, RPI = 64 / V;   // floats and bytes of a row; rows per store
        uint8_t *scr = lds + wave * (16 * pitch);
        float *const out = a.Cf + (size_t)z * a.cf_zstride;
        const bool vectors = (((uintptr_t)out | (uintptr_t)(a.ldcf * 4)) & 15) == 0 && a.I % 4 == 0;
#pragma unroll
        for (int g = 0; g < FJ; ++g) {
            wave_sync();
#pragma unroll
            for (int f = 0; f < FI; ++f) *(f32x4 *)(scr + l16 * pitch + (f * 16 + q4 * 4) * 4) = acc[f][g];
            wave_sync();
            if (vectors) {
#pragma unroll
                for (int t = 0; t < 16 / RPI; ++t) {
                    const int r = t * RPI + lane / V, c = lane % V * 4, j = jb + 16 * g + r, i = ib + c;
                    const f32x4 v = *(const f32x4 *)(scr + r * pitch + c * 4);
                    if (j < j_end && i < a.I) *(f32x4 *)(out + (size_t)j * a.ldcf + i) = v;
                }
            } else {   // rows of any length and place: 64 neighbouring elements per store
                for (int r = 0; r < 16; ++r)
                    for (int c = lane; c < W; c += 64) {
                        const int j = jb + 16 * g + r, i = ib + c;
                        if (j < j_end && i < a.I) out[(size_t)j * a.ldcf + i] = *(const float *)(scr + r * pitch + c * 4);
                    }
            }
        }
        return;
    }
    constexpr int W = FI * 16, pitch = W * 2 + 16, V = W / 8, RPI = 64 / V;
    uint8_t *scr = lds + wave * (16 * pitch);
#pragma unroll
    for (int g = 0; g < FJ; ++g) {
        u32x4 mask[16 / RPI];
        if constexpr (KIND == kInputGrad) {
#pragma unroll
            for (int t = 0; t < 16 / RPI; ++t) {
                const int j = min(jb + 16 * g + t * RPI + lane / V, j_end - 1), i = min(ib + lane % V * 8, ((a.I + 7) & ~7) - 8);
                mask[t] = *(const u32x4 *)(a.mask + (size_t)j * a.ldmask + i);
            }
        }
        wave_sync();
#pragma unroll
        for (int f = 0; f < FI; ++f) {
            f32x4 v = acc[f][g];
            if constexpr (KIND == kForward) {
                const f32x4 b = *(const f32x4 *)(bias + wi * FI * 16 + f * 16 + q4 * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = ib + f * 16 + q4 * 4 + e < a.I ? fmaxf(v[e] + b[e], 0.f) : 0.f;   // pads stay zero
            }
            *(uint2 *)(scr + l16 * pitch + (f * 16 + q4 * 4) * 2) = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        }
        wave_sync();
#pragma unroll
        for (int t = 0; t < 16 / RPI; ++t) {
            const int r = t * RPI + lane / V, j = jb + 16 * g + r, i = ib + lane % V * 8;
            u32x4 d = *(const u32x4 *)(scr + r * pitch + lane % V * 16);
            if constexpr (KIND == kInputGrad) {   // keep where the bf16 mask value is > 0
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    d[e] &= ((int16_t)(mask[t][e] & 0xFFFFu) > 0 ? 0xFFFFu : 0u) | ((int16_t)(mask[t][e] >> 16) > 0 ? 0xFFFF0000u : 0u);
            }
            if (j < j_end && i < a.I) *(u32x4 *)(a.Ci + (size_t)j * a.ldci + i) = d;
        }
    }
}

// Tiles of a problem without a split contraction, 256 columns each; XCD (id % 8) x takes columns x, x + 8, ... and sweeps their i
// tiles, so that every L2 keeps the weights and each activation row is fetched once.
struct WidePlan {
    int tiles_i, tiles_j, seg0;   // seg0: columns of tiles of the first segment
    int whole;                    // columns of 256; those behind them are cut into halves, one round of blocks
    int n_whole;                  // blocks of the former
};

__device__ __forceinline__ bool place(int id, int tiles_i, int tiles_j, int &ti, int &tj)
{
    const int slot = id >> 3;
    ti = slot % tiles_i;
    tj = (slot / tiles_i) * 8 + (id & 7);
    return tj < tiles_j;
}

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_wide_forward(const TjGemmArgs<tj_bf16> a, const WidePlan p)
{
    extern __shared__ __align__(1024) uint8_t lds[];
    int ti, tj;
    if ((int)blockIdx.x < p.n_whole) {
        if (!place(blockIdx.x, p.tiles_i, p.whole, ti, tj)) return;
        const TjGemmSeg<tj_bf16> &seg = a.seg[tj >= p.seg0 ? 1 : 0];
        tile<kForward, 4>(a, seg, ti * kTile, seg.j_begin + (tj - (tj >= p.seg0 ? p.seg0 : 0)) * kTile, 0, 0, 1, lds);
    } else {
        if (!place((int)blockIdx.x - p.n_whole, p.tiles_i, 2 * (p.tiles_j - p.whole), ti, tj)) return;
        const int half = tj & 1;
        tj = p.whole + (tj >> 1);
        const TjGemmSeg<tj_bf16> &seg = a.seg[tj >= p.seg0 ? 1 : 0];
        const int j0 = seg.j_begin + (tj - (tj >= p.seg0 ? p.seg0 : 0)) * kTile + half * (kTile / 2);
        if (j0 >= seg.j_end) return;
        tile<kForward, 2>(a, seg, ti * kTile, j0, 0, 0, 1, lds);
    }
}

// A hidden layer's weight gradient (blocks [0, n0), a slice of a tile each) and its input gradient.
struct WidePair {
    TjGemmArgs<tj_bf16> w, x;
    int w_tiles_i, n0, sum_step;
    int x_tiles_i, x_tiles_j;
};

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_wide_pair(const WidePair p)
{
    extern __shared__ __align__(1024) uint8_t lds[];
    if ((int)blockIdx.x < p.n0) {
        const int z = blockIdx.x % p.w.n_split, t = blockIdx.x / p.w.n_split;
        const int ti = t % p.w_tiles_i, tj = t / p.w_tiles_i;
        tile<kWeightGrad, 4>(p.w, p.w.seg[0], ti * kTile, p.w.seg[0].j_begin + tj * kTile, z, ti, p.sum_step, lds);
    } else {
        int ti, tj;
        if (!place((int)blockIdx.x - p.n0, p.x_tiles_i, p.x_tiles_j, ti, tj)) return;
        tile<kInputGrad, 4>(p.x, p.x.seg[0], ti * kTile, p.x.seg[0].j_begin + tj * kTile, 0, 0, 1, lds);
    }
}

int lds_attr(const void *fn)
{
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLds) == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}

int up_div(int x, int y) { return (x + y - 1) / y; }

bool aligned16(const void *p, size_t ld_bytes) { return (((uintptr_t)p | ld_bytes) & 15) == 0; }

int vectors8(int n) { return (n + 7) & ~7; }   // columns of whole 16-byte vectors

}  // namespace

bool tj_gemm_wide_forward(const TjGemmArgs<tj_bf16> &a, hipStream_t st, int *rc)
{
    if (a.trans || a.gather.on || a.out_map.on || a.n_split != 1 || a.qsum || a.bias_j || a.mask || a.Cj || a.Cf || !a.Ci || !a.relu)
        return false;
    if (a.K % 64 || a.K < 64 || a.I < kTile || a.ldci < vectors8(a.I)) return false;
    if (!aligned16(a.Q, a.ldq * 2) || !aligned16(a.Ci, a.ldci * 2)) return false;
    WidePlan p;
    p.tiles_i = up_div(a.I, kTile);
    int cols[2] = {0, 0};
    for (int s = 0; s < a.n_seg; ++s) {
        if (!a.seg[s].bias || !aligned16(a.seg[s].P, a.ldp * 2)) return false;
        cols[s] = up_div(a.seg[s].j_end - a.seg[s].j_begin, kTile);
    }
    p.seg0 = cols[0];
    p.tiles_j = cols[0] + cols[1];
    if (!tjplan::wide_forward_pays(p.tiles_i, p.tiles_j, a.K)) return false;
    p.whole = tjplan::wide_whole_columns(p.tiles_i, p.tiles_j);
    auto blocks = [&](int cols_) { return p.tiles_i * up_div(cols_, 8) * 8; };
    p.n_whole = blocks(p.whole);
    const int n = p.n_whole + (p.whole < p.tiles_j ? blocks(2 * (p.tiles_j - p.whole)) : 0);
    if ((*rc = lds_attr((const void *)gemm_wide_forward)) != TJ_OK) return true;
    gemm_wide_forward<<<n, kThreads, kLds, st>>>(a, p);
    *rc = hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
    return true;
}

bool tj_gemm_wide_pair(const TjGemmArgs<tj_bf16> &w, const TjGemmArgs<tj_bf16> &x, hipStream_t st, int *rc)
{
    // the forms and outputs of a hidden layer
    if (w.trans != 1 || x.trans != 2 || w.n_seg != 1 || x.n_seg != 1 || w.gather.on || x.gather.on || w.out_map.on || x.out_map.on) return false;
    if (!w.Cf || w.Ci || w.Cj || w.mask || w.relu || w.bias_j || w.seg[0].bias || !w.qsum || w.seg[0].q_shift) return false;
    if (!x.Ci || x.Cf || x.Cj || !x.mask || x.relu || x.bias_j || x.seg[0].bias || x.qsum || x.n_split != 1 || x.seg[0].q_shift) return false;
    const int wj = w.seg[0].j_end - w.seg[0].j_begin, xj = x.seg[0].j_end - x.seg[0].j_begin;
    const int valid = w.k_valid ? w.k_valid : w.K;
    if (w.K % 64 || w.k_chunk % 64 || w.k_chunk < 64 || valid > w.K || w.K - valid >= 64 || w.seg[0].j_begin % 8) return false;
    if (vectors8(w.I) > w.ldp || vectors8(w.seg[0].j_end) > w.ldq) return false;
    if ((w.n_split - 1) * w.k_chunk >= w.K || x.K % 64 || x.K < 64) return false;
    if (vectors8(x.I) > x.ldp || vectors8(x.I) > x.ldci || vectors8(x.I) > x.ldmask) return false;
    if (!aligned16(w.seg[0].P, w.ldp * 2) || !aligned16(w.Q, w.ldq * 2)) return false;
    if (!aligned16(x.seg[0].P, x.ldp * 2) || !aligned16(x.Q, x.ldq * 2) || !aligned16(x.Ci, x.ldci * 2) || !aligned16(x.mask, x.ldmask * 2))
        return false;
    WidePair p;
    p.w = w; p.x = x;
    p.w_tiles_i = up_div(w.I, kTile);
    p.n0 = p.w_tiles_i * up_div(wj, kTile) * w.n_split;
    p.sum_step = p.w_tiles_i >= 4 ? 4 : p.w_tiles_i >= 2 ? 2 : 1;   // the column sums are shared by the blocks of a column
    p.x_tiles_i = up_div(x.I, kTile);
    p.x_tiles_j = up_div(xj, kTile);
    const int n1 = p.x_tiles_i * p.x_tiles_j;
    if (!tjplan::wide_pair_pays(p.n0 + n1, x.K)) return false;
    if ((*rc = lds_attr((const void *)gemm_wide_pair)) != TJ_OK) return true;
    gemm_wide_pair<<<p.n0 + p.x_tiles_i * up_div(p.x_tiles_j, 8) * 8, kThreads, kLds, st>>>(p);
    *rc = hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
    return true;
}
