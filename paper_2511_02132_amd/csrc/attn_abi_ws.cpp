// attn_abi_ws.cpp -- the forward entry point that may use a caller-owned
// workspace (attn_fwd_ws) and the rule that decides when it runs the split
// kernel (attn_fwd_split.hip) instead of the ones attn_fwd runs.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "attn_checks.h"
#include "attn_internal.h"
#include "attn_numa.h"

namespace {

struct SplitPlan {
    bool use;
    int R, MB, splits, tiles_per_split;
    int64_t bytes;   // workspace
};

constexpr int kComputeUnits = 256;
// Longer runs of packed rows stay with the kernels of attn_fwd, whose output
// the persistent form repeats bitwise.
constexpr int kSplitMaxRows = 2048;

// When the split kernel runs: one workgroup per 32 packed rows, so either there
// is one such tile per K/V head (a K/V row is then copied once, in any number of
// workgroups), or all tiles run at once.  Measured against attn_fwd, in us:
//   one row tile per K/V head:
//     d 128  B 4  Hq 64 Hkv 8 Sq 1 Skv 8192    197 -> 27   (8 splits)
//     d 128  B 32 Hq 64 Hkv 8 Sq 1 Skv 8192   1450 -> 179  (1 split, 6 TB/s)
//     d 128  B 32 Hq 64 Hkv 64 Sq 8 Skv 2000   475 -> 334
//     d 64   the same                          182 -> 175
//   all tiles at once (256 of them at d 128, 512 at d 64 and 56):
//     d 128  B 1 H 32 Sq 256 Skv 1000           25 -> 12,  Skv 64  8.3 -> 5.0
//     d 64   B 1 H 16 Sq 1000 Skv 500         10.5 -> 8.2, Skv 2000 28 -> 17
//   more than that, several tiles per K/V head (each copies K and V again):
//     d 128  B 4 H 32 Sq 128 Skv 1000           27 -> 26,  Sq 256   29 -> 48
//     d 64   B 8 H 64 Sq 64 Skv 1000            25 -> 26,  Sq 128   26 -> 44
bool takes_split(int64_t heads, int64_t R, int d, int causal) {
    if (causal || R > kSplitMaxRows) return false;
    if (R <= 32) return true;
    return heads * ((R + 31) / 32) <= (d == 128 ? kComputeUnits : 2 * kComputeUnits);
}

SplitPlan plan_split(int B, int Hq, int Hkv, int Sq, int Skv, int d, int causal) {
    SplitPlan s{};
    const int64_t R = (int64_t)(Hq / Hkv) * Sq;
    if (!takes_split((int64_t)B * Hkv, R, d, causal)) return s;
    s.R = (int)R;
    s.MB = (s.R + 31) / 32;
    const int64_t units = (int64_t)B * Hkv * s.MB;
    if (units * attn::kMaxSplits > INT32_MAX) return s;
    s.use = true;
    const int tiles = (Skv + attn::kSplitKeys - 1) / attn::kSplitKeys;
    // Workgroups that run at once: one per compute unit at d = 128 (128 KiB of
    // LDS), two otherwise.
    const int slots = d == 128 ? kComputeUnits : 2 * kComputeUnits;
    double best = 0.0;
    for (int n = 1; n <= attn::kMaxSplits; ++n) {
        const int per = (tiles + n - 1) / n;
        if (n > 1 && (per < 4 || units >= slots)) break;   // a tile for every wave; units idle
        if ((int64_t)(n - 1) * per >= tiles) continue;   // the last split would be empty
        // Estimated time in us: rounds of workgroups, each a start and a walk of
        // ceil(per / 4) tiles per wave (about 1 us a tile alone, 2.6 with every
        // unit streaming), and a second launch to merge splits.  Against every
        // count from 1 to 64 measured, the count with the least estimate was
        // within 6% of the best on ten of eleven decoding shapes, 10% on one.
        const int64_t wgs = units * n;
        const int64_t rounds = (wgs + slots - 1) / slots;
        const double fill = wgs < slots ? (double)wgs / slots : 1.0;
        const double tile_us = 1.0 + 1.6 * fill;
        const double t = rounds * (3.0 + ((per + 3) / 4) * tile_us) + (n > 1 ? 4.0 : 0.0);
        if (n == 1 || t < best) {
            best = t;
            s.splits = n;
            s.tiles_per_split = per;
        }
    }
    if (s.splits > 1) s.bytes = (int64_t)B * Hq * Sq * s.splits * (d + 2) * 4;
    return s;
}

}  // namespace

extern "C" {

int64_t attn_fwd_workspace_bytes(int B, int Hq, int Hkv, int Sq, int Skv, int d, int causal) {
    const int rc = attn::check_shape(B, Hq, Hkv, Sq, Skv, d);
    if (rc) return rc;
    return plan_split(B, Hq, Hkv, Sq, Skv, d, causal).bytes;
}

int attn_fwd_ws(const void *q, const void *k, const void *v, void *o, float *lse, void *workspace,
                int64_t workspace_bytes, int B, int Hq, int Hkv, int Sq, int Skv, int d, int causal,
                float scale, int mapping) {
    int rc = attn::validate(q, k, v, o, B, Hq, Hkv, Sq, Skv, d, scale, mapping);
    if (rc) return rc;
    const SplitPlan s = plan_split(B, Hq, Hkv, Sq, Skv, d, causal);
    if (!s.use || (s.bytes > 0 && (workspace == nullptr || workspace_bytes < s.bytes)))
        return lse == nullptr
                   ? attn_fwd(q, k, v, o, B, Hq, Hkv, Sq, Skv, d, causal, scale, mapping)
                   : attn_fwd_lse(q, k, v, o, lse, B, Hq, Hkv, Sq, Skv, d, causal, scale, mapping);
    // pairs exist for head dimension 128 only, whichever kernel runs
    if ((mapping & ATTN_ORDER_PAIRED) && d != 128) return ATTN_ERR_UNSUPPORTED;
    rc = attn::validate_lse(lse, q, k, v, o, B, Hq, Hkv, Sq, Skv, d);
    if (rc) return rc;
    if (s.bytes > 0) {
        if ((uintptr_t)workspace & 15u) return ATTN_ERR_ALIGN;
        const int64_t qo = (int64_t)B * Hq * Sq * d * 2;
        const int64_t kv = (int64_t)B * Hkv * Skv * d * 2;
        const int64_t st = (int64_t)B * Hq * Sq * 4;
        if (attn::overlaps(workspace, s.bytes, q, qo) || attn::overlaps(workspace, s.bytes, k, kv) ||
            attn::overlaps(workspace, s.bytes, v, kv) || attn::overlaps(workspace, s.bytes, o, qo) ||
            (lse && attn::overlaps(workspace, s.bytes, lse, st)))
            return ATTN_ERR_ALIAS;
    }
    const int nx = attn_num_xcd();
    if (nx < 0) return nx;
    attn::SplitArgs a{};
    a.q = q;
    a.k = k;
    a.v = v;
    a.o = o;
    a.lse = lse;
    if (s.bytes > 0) {
        a.part = (float *)workspace;
        a.part_stat = a.part + (int64_t)B * Hq * Sq * s.splits * d;
    }
    a.B = B;
    a.Hkv = Hkv;
    a.R = s.R;
    a.Skv = Skv;
    a.MB = s.MB;
    a.splits = s.splits;
    a.tiles_per_split = s.tiles_per_split;
    a.mapping = mapping & 0xf;
    a.NX = nx;
    a.scale_log2 = (float)((double)scale * 1.4426950408889634073599246810019);  // log2(e)
    const hipError_t e = attn::launch_attn_fwd_split(a, d, (hipStream_t)attn_get_stream());
    return e == hipSuccess ? ATTN_OK : attn::hip_fail(e);
}

}  // extern "C"
