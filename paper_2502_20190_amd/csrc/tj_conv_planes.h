// What the kernels that read u8 frame stacks have in common (tj_conv_first.hip, tj_conv_tower.hip).
#pragma once
#include "tj_gemm.h"

namespace tjplanes {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// round to nearest even in hardware (v_cvt_pk_bf16_f32); the inputs here are finite
__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    const f32x2_t f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

// Byte offsets of an image's four planes inside its source table: the planes of batch position b, of the
// table row an index names for it, or four planes named one by one (a frame ring's frames).  Indices
// are clamped to the table.
struct PlaneOff {
    size_t o[4];
};

__device__ __forceinline__ PlaneOff plane_offsets(const uint32_t *rows, const uint32_t *planes, const uint32_t n_rows,
                                                  const int b, const bool next, const int HW)
{
    PlaneOff p;
    if (planes) {
        const uint32_t *q = planes + (size_t)b * 8 + (next ? 4 : 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) p.o[c] = (size_t)min(q[c], n_rows - 1u) * HW;
    } else {
        const uint32_t r = rows ? min(rows[b], n_rows - 1u) : (uint32_t)b;
#pragma unroll
        for (int c = 0; c < 4; ++c) p.o[c] = ((size_t)r * 4 + c) * HW;
    }
    return p;
}

}  // namespace tjplanes
