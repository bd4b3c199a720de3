// Which query tile of which head a workgroup of the bf16 attention kernels takes.
#pragma once

#include "common.h"
#include "staging_addr.h"

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
    int units, later;  // fa_item_of; with the XCD map of one XCD
};

__device__ __forceinline__ bool fa_map_block(const FaMap& mp, int bid, int n_qtiles, int Hq, int Hkv,
                                             int& qt, int& head) {
    const int group = Hq / Hkv;
    if (!mp.xcd_mode) {
        const int item = fa_item_of(bid, mp.later, mp.units);
        qt = n_qtiles - 1 - item / Hq;
        head = item % Hq;
        return true;
    }
    const int xcd = bid % 8, slot = fa_item_of(bid / 8, mp.later, mp.units);
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

// The map of a launch over n_qtiles query tiles, and its workgroups, which start heaviest first (fa_map_later: but for the few
// that fa_launch_later has wait).
inline FaMap fa_map(int n_qtiles, int Hq, int Hkv, unsigned& blocks) {
    FaMap mp{0, 1, 1, n_qtiles * (Hq / Hkv), 0, 0};
    const int slots = fa_slots(n_qtiles, Hq, Hkv);
    mp.xcd_mode = fa_xcd_map(Hkv);
    if (mp.xcd_mode && Hkv <= 8) mp.xcds_per_g = 8 / Hkv;
    else if (mp.xcd_mode) mp.g_per_xcd = Hkv / 8;
    blocks = mp.xcd_mode ? 8u * (unsigned)slots : (unsigned)slots;
    return mp;
}

// The same where a launch's workgroups run one at a time on each of `cu` units and rows get longer from tile to tile.
inline FaMap fa_map_later(int n_qtiles, int Hq, int Hkv, int head_dim, int groups, int cu, unsigned& blocks) {
    FaMap mp = fa_map(n_qtiles, Hq, Hkv, blocks);
    mp.units = mp.xcd_mode ? cu / 8 : cu;
    mp.later = fa_launch_later(n_qtiles, Hq, Hkv, head_dim, groups, cu);
    return mp;
}

}  // namespace dash
