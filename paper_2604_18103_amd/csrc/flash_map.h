// Which query tile of which head a workgroup of the bf16 attention kernels takes.
#pragma once

#include "common.h"

namespace dash {

// Work-item -> (query tile, head) map. Workgroups are handed to the 8 XCDs round-robin
// (workgroup b runs on XCD b % 8) and each XCD has its own L2, so all workgroups of one XCD are given
// the same KV head (or as few as possible): its K/V tiles are then fetched into that L2 once and shared
// by the query heads of the group and by neighbouring query tiles. Heaviest (latest) query tiles first.
struct FaMap {
    int xcd_mode;      // 1: XCD-aware, 0: plain
    int xcds_per_g;    // XCDs serving one KV head (Hkv <= 8)
    int g_per_xcd;     // KV heads per XCD (Hkv >= 8)
    int items_per_g;   // n_qtiles * group size
};

__device__ __forceinline__ bool fa_map_block(const FaMap& mp, int bid, int n_qtiles, int Hq, int Hkv,
                                             int& qt, int& head) {
    const int group = Hq / Hkv;
    if (!mp.xcd_mode) {
        qt = n_qtiles - 1 - bid / Hq;
        head = bid % Hq;
        return true;
    }
    const int xcd = bid % 8, slot = bid / 8;
    int g, idx;
    if (mp.g_per_xcd == 1) {
        g = xcd / mp.xcds_per_g;
        idx = slot * mp.xcds_per_g + xcd % mp.xcds_per_g;
    } else {
        g = xcd * mp.g_per_xcd + slot % mp.g_per_xcd;
        idx = slot / mp.g_per_xcd;
    }
    if (idx >= mp.items_per_g) return false;
    qt = n_qtiles - 1 - idx / group;
    head = g * group + idx % group;
    return true;
}

// The map of a launch over n_qtiles query tiles, and its workgroups.
inline FaMap fa_map(int n_qtiles, int Hq, int Hkv, unsigned& blocks) {
    FaMap mp{0, 1, 1, n_qtiles * (Hq / Hkv)};
    blocks = (unsigned)n_qtiles * Hq;
    if (Hkv <= 8 && 8 % Hkv == 0) {
        mp.xcd_mode = 1;
        mp.xcds_per_g = 8 / Hkv;
        blocks = 8u * (unsigned)((mp.items_per_g + mp.xcds_per_g - 1) / mp.xcds_per_g);
    } else if (Hkv % 8 == 0) {
        mp.xcd_mode = 1;
        mp.g_per_xcd = Hkv / 8;
        blocks = 8u * (unsigned)(mp.items_per_g * mp.g_per_xcd);
    }
    return mp;
}

}  // namespace dash
