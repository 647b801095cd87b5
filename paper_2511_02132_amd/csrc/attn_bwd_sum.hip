// attn_bwd_sum.hip -- the launch that adds up the fp32 parts of dK and dV after the
// merged gradient launch (attn_bwd_dq.hip).  Bound by the parts it reads: 128 KiB
// per part and key block, about 4 us and 30 ns a part.
#include <hip/hip_runtime.h>

#include "attn_bwd_sum.h"
#include "attn_internal.h"

namespace attn {
namespace {

template <bool CAUSAL>
__global__ __launch_bounds__(256) void attn_bwd_sum_kernel(const BwdArgs p) {
    bwd::sum_parts<CAUSAL>(p, blockIdx.x);
}

}  // namespace

hipError_t launch_attn_bwd_sum(const BwdArgs &a, bool causal, hipStream_t stream) {
    const int grid = a.B * a.Hkv * ((a.Skv + kBwdSumRows - 1) / kBwdSumRows);
    if (causal)
        hipLaunchKernelGGL((attn_bwd_sum_kernel<true>), dim3(grid), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((attn_bwd_sum_kernel<false>), dim3(grid), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace attn
