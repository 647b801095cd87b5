// attn_bwd_sum.h -- the sum of dK's and dV's parts: device code shared by its own
// kernel (attn_bwd_sum.hip) and by the dQ launch that it can ride on
// (attn_bwd_dq.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_bwd_common.h"
#include "attn_internal.h"

namespace attn {
namespace bwd {

// dK and dV of 16 keys of (b, K/V head): the sum of the key block's fp32 parts in
// the order of the parts, for key blocks of several parts (the others are
// written already).  Thread: 8 columns of key 16 * block + tid / 16.
template <bool CAUSAL>
__device__ __forceinline__ void sum_parts(const BwdArgs &p, const int block) {
    const int blocks = (p.Skv + kBwdSumRows - 1) / kBwdSumRows;
    const int head = block / blocks;
    const int key = (block % blocks) * kBwdSumRows + (threadIdx.x >> 4);
    if (key >= p.Skv) return;
    const int n_parts = bwd_parts(p, CAUSAL, key / kBwdKeys);
    if (n_parts == 1) return;
    const int col = (threadIdx.x & 15) * 8;
    const int64_t slab = (int64_t)p.Skv * D;
    const int64_t dv_off = (int64_t)p.B * p.Hkv * p.parts * slab;
    const float *src = p.part + (int64_t)head * p.parts * slab + (int64_t)key * D + col;
    f32x4 acc[2][2] = {};   // dK, dV
    for (int i = 0; i < n_parts; ++i, src += slab)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int e = 0; e < 2; ++e) acc[x][e] += *(const f32x4 *)(src + x * dv_off + 4 * e);
    const int64_t out = ((int64_t)head * p.Skv + key) * D + col;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const float s = x == 0 ? p.scale : 1.0f;
        __bf16 *const dst = (__bf16 *)(x == 0 ? p.dk : p.dv) + out;
        const f32x8 v8 = {acc[x][0][0] * s, acc[x][0][1] * s, acc[x][0][2] * s, acc[x][0][3] * s,
                          acc[x][1][0] * s, acc[x][1][1] * s, acc[x][1][2] * s, acc[x][1][3] * s};
        *(u32x4 *)dst = __builtin_bit_cast(u32x4, __builtin_convertvector(v8, bf16x8));
    }
}

}  // namespace bwd
}  // namespace attn
