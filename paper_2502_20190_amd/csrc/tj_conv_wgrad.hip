// The weight gradient of a convolution as a launch of its own (a convolution with a gathered input gradient has both in
// one launch, tj_gemm_conv_backward).
#include "tj_conv_wgrad.h"

namespace {

template <int NFI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
void conv_wgrad_bf16(const TjConvWgradArgs a, const int njb)
{
    __shared__ __align__(1024) uint8_t lds[tjwgrad::lds_bytes<NFI>()];
    tjwgrad::body<NFI>(a, njb, (int)blockIdx.x, lds);
}

}  // namespace

int tj_conv_wgrad(const TjConvWgradArgs &a, hipStream_t st)
{
    int njb, rc;
    unsigned nblk;
    if ((rc = tjwgrad::plan(a, njb, nblk)) != TJ_OK) return rc;
    if (a.O == 64)
        conv_wgrad_bf16<2><<<nblk, 512, 0, st>>>(a, njb);
    else
        conv_wgrad_bf16<1><<<nblk, 512, 0, st>>>(a, njb);
    return hipGetLastError() == hipSuccess ? TJ_OK : TJ_ERR_DEVICE;
}
