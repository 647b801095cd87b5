// attn_checks.h -- argument checks shared by the entry points of
// libattn_numa.so.  Host code only; no HIP call is made.
#pragma once

#include <cmath>
#include <cstdint>

#include "attn_internal.h"
#include "attn_numa.h"

namespace attn {

inline bool supported_d(int d) { return d == 56 || d == 64 || d == 128; }

// Shape checks shared by every entry point.  Offsets inside one head are
// 32-bit byte offsets, so a head (plus one tile of slack) must stay below 2^31.
inline int check_shape(int B, int Hq, int Hkv, int Sq, int Skv, int d) {
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || Sq <= 0 || Skv <= 0 || d <= 0) return ATTN_ERR_SHAPE;
    if (Hq % Hkv != 0) return ATTN_ERR_SHAPE;
    if (!supported_d(d)) return ATTN_ERR_UNSUPPORTED;
    const int64_t lim = INT32_MAX;
    if (((int64_t)Sq + attn::kMaxBlockM) * d * 2 > lim) return ATTN_ERR_SHAPE;
    if (((int64_t)Skv + 2 * attn::kBlockN) * d * 2 > lim) return ATTN_ERR_SHAPE;
    const int bm = attn::block_m_for(d);
    const int64_t nb = ((int64_t)Sq + bm - 1) / bm;
    if ((int64_t)B * Hq * nb > lim) return ATTN_ERR_SHAPE;
    return ATTN_OK;
}

// Base mapping in the low 4 bits, optional order flag above them.
inline bool valid_mapping(int mapping) {
    const int base = mapping & 0xf;
    const int flags = mapping & ~0xf;
    if (base < ATTN_MAP_NAIVE_BLOCK_FIRST || base > ATTN_MAP_SWIZZLED_BLOCK_FIRST) return false;
    if ((flags & ~(ATTN_ORDER_HEAVY_FIRST | ATTN_ORDER_XCD_BLOCK_MAJOR | ATTN_ORDER_PAIRED)) != 0)
        return false;
    // the block-major order inside an XCD's piece is defined for mapping 2 only
    return (flags & ATTN_ORDER_XCD_BLOCK_MAJOR) == 0 || base == ATTN_MAP_SWIZZLED_HEAD_FIRST;
}

inline bool overlaps(const void *a, int64_t a_bytes, const void *b, int64_t b_bytes) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + (uintptr_t)b_bytes && b0 < a0 + (uintptr_t)a_bytes;
}

inline int validate(const void *q, const void *k, const void *v, const void *o, int B, int Hq, int Hkv,
             int Sq, int Skv, int d, float scale, int mapping) {
    if (!q || !k || !v || !o) return ATTN_ERR_NULL;
    int rc = check_shape(B, Hq, Hkv, Sq, Skv, d);
    if (rc) return rc;
    if (!valid_mapping(mapping)) return ATTN_ERR_MAPPING;
    if (!std::isfinite(scale) || !(scale > 0.0f)) return ATTN_ERR_SCALE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15u) return ATTN_ERR_ALIGN;
    const int64_t qo_bytes = (int64_t)B * Hq * Sq * d * 2;
    const int64_t kv_bytes = (int64_t)B * Hkv * Skv * d * 2;
    if (overlaps(o, qo_bytes, q, qo_bytes) || overlaps(o, qo_bytes, k, kv_bytes) ||
        overlaps(o, qo_bytes, v, kv_bytes))
        return ATTN_ERR_ALIAS;
    return ATTN_OK;
}

// Checks of a forward's optional row statistics.
inline int validate_lse(const float *lse, const void *q, const void *k, const void *v,
                        const void *o, int B, int Hq, int Hkv, int Sq, int Skv, int d) {
    if (!lse) return ATTN_OK;
    if (((uintptr_t)lse) & 3u) return ATTN_ERR_ALIGN;
    const int64_t lse_bytes = (int64_t)B * Hq * Sq * 4;
    const int64_t qo_bytes = (int64_t)B * Hq * Sq * d * 2;
    const int64_t kv_bytes = (int64_t)B * Hkv * Skv * d * 2;
    if (overlaps(lse, lse_bytes, q, qo_bytes) || overlaps(lse, lse_bytes, k, kv_bytes) ||
        overlaps(lse, lse_bytes, v, kv_bytes) || overlaps(lse, lse_bytes, o, qo_bytes))
        return ATTN_ERR_ALIAS;
    return ATTN_OK;
}

// Records a HIP error for attn_last_hip_error() and returns ATTN_ERR_HIP
// (attn_abi.cpp).
int hip_fail(hipError_t e);

}  // namespace attn
