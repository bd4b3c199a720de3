// TopK's selection by one workgroup: the cut between the rows that are kept and the others, found on keys in registers. Shared by the
// decision kernels and the one-launch score + decision + compaction kernel.
#pragma once

#include "common.h"
#include "score_rows.h"

namespace dash {

// Key under which TopK ranks a score: the order-preserving key, or its complement when the rows with the
// LOWEST scores are to be kept (the direction control of Sec. 5.4).
__device__ __forceinline__ uint32_t rank_key(float f, int keep_low) {
    const uint32_t k = order_key(f);
    return keep_low ? ~k : k;
}

constexpr int kSelectThreads = 1024;
constexpr int kSelectBins = 2048;   // histogram bins of one radix pass (11-bit digits)
constexpr int kSelectBatch = 16;    // scores a thread has in flight per load batch
// Copies of the histogram, one per lane % kHistCopies: adds of one wave instruction to the same LDS word are done one
// after the other, and keys that crowd into a few bins make a pass several times longer: in the first pass over top digits (longer
// inputs; sign, exponent and two mantissa bits, where the relative scores of one layer may span only an octave or two), with ties and
// with neighbours behind an outlier in any. Two copies cost the widely spread case 5 % and take a third off the crowded ones; four
// cost more than they return.
constexpr int kHistCopies = 2;

constexpr int kListMax = 64;  // so many keys left in a bin are ranked by counting (one wave); more take another pass
struct SelectShared {
    int hist[kSelectBins][kHistCopies];  // the copies of a bin side by side: in different LDS banks
    uint32_t list[kListMax];
    uint2 least[kSelectThreads / kWave];
    int n_list;
    int wave_tot[kSelectThreads / kWave];
    uint32_t prefix;
    int remaining, ties;
};

__device__ __forceinline__ void clear_hist(SelectShared& sh) {
    int* h = &sh.hist[0][0];
    for (int b = threadIdx.x; b < kHistCopies * kSelectBins; b += kSelectThreads) h[b] = 0;
}

__device__ __forceinline__ void hist_add(SelectShared& sh, uint32_t digit) {
    atomicAdd(&sh.hist[digit][threadIdx.x % kHistCopies], 1);
}

// After a pass has filled sh.hist (and a barrier): the bin that holds the remaining-th largest key, i.e. the largest
// b with (keys in bins >= b) >= remaining; updates prefix and remaining (uniform) and leaves the bin's count in
// sh.ties. Thread t owns bins 2t and 2t + 1; suffix sums over the threads of a wave by shuffles, over the waves
// through LDS. Called by all kSelectThreads threads; ends with a barrier after which sh.hist may be cleared.
__device__ __forceinline__ void select_bin(SelectShared& sh, int shift, uint32_t& prefix, int& remaining) {
    constexpr int kWaves = kSelectThreads / kWave;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    int h0 = 0, h1 = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) {
        h0 += sh.hist[2 * tid][c];
        h1 += sh.hist[2 * tid + 1][c];
    }
    int suf = h0 + h1;  // becomes the count of keys in bins >= 2 tid
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_down(suf, o);
        if (lane + o < kWave) suf += t;
    }
    if (lane == 0) sh.wave_tot[wave] = suf;
    __syncthreads();
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {  // every total is read (independent LDS reads), the later waves' are added
        const int t = sh.wave_tot[w];
        if (w > wave) suf += t;
    }
    // exactly one bin satisfies excl < remaining <= incl (the keys under the prefix number at least `remaining`)
    const int incl1 = suf - h0, excl1 = incl1 - h1;  // bin 2 tid + 1
    const int incl0 = suf, excl0 = incl1;            // bin 2 tid
    if (excl1 < remaining && remaining <= incl1) {
        sh.prefix = prefix | ((uint32_t)(2 * tid + 1) << shift);
        sh.remaining = remaining - excl1;
        sh.ties = h1;
    } else if (excl0 < remaining && remaining <= incl0) {
        sh.prefix = prefix | ((uint32_t)(2 * tid) << shift);
        sh.remaining = remaining - excl0;
        sh.ties = h0;
    }
    __syncthreads();
    prefix = sh.prefix;
    remaining = sh.remaining;
}

// The least of the threads' values, of either of two, uniform; ends with a barrier. By row shifts and broadcasts inside a wave, over the
// waves by one LDS read per lane: with shuffles, and every thread reading all waves' values, it took half a microsecond longer.
template <int CTRL>
__device__ __forceinline__ void fold_lanes(uint32_t& a, uint32_t& b) {  // lanes without a source keep their own
    a = min(a, (uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)a, CTRL, 0xF, 0xF, false));
    b = min(b, (uint32_t)__builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ void fold_row(uint32_t& a, uint32_t& b) {  // of 16 lanes, into its last
    fold_lanes<0x111>(a, b);  // row_shr:1, 2, 4, 8
    fold_lanes<0x112>(a, b);
    fold_lanes<0x114>(a, b);
    fold_lanes<0x118>(a, b);
}
__device__ __forceinline__ void least_of_all(SelectShared& sh, uint32_t& a, uint32_t& b) {
    static_assert(kSelectThreads / kWave == 16, "a row of lanes per wave's values");
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    fold_row(a, b);
    fold_lanes<0x142>(a, b);  // row_bcast:15, 31: a row's last lane to the next row, the second row's to the last two
    fold_lanes<0x143>(a, b);
    if (lane == kWave - 1) sh.least[wave] = make_uint2(a, b);
    __syncthreads();
    const uint2 w = sh.least[lane % 16];
    a = w.x;
    b = w.y;
    fold_row(a, b);
    a = (uint32_t)__builtin_amdgcn_readlane((int)a, 15);
    b = (uint32_t)__builtin_amdgcn_readlane((int)b, 15);
}

// The cut: rows with a key above T are kept, and of the `same` ones at T the first `quota`.
struct TopkCut {
    uint32_t T;
    int quota;
    bool rank_ties;  // more rows tie with the K-th key than may be kept: tie_base is filled
};
constexpr int topk_chunks(int B) { return B * kSelectThreads / kWave; }

// Key u of thread t is row u * 1024 + t's, no_key for rows that are no candidates; bit u of `cand`: it is one. n_cand candidates, of
// which k_cand are kept. tie_base[topk_chunks(B)]: ties in all chunks before chunk u * 16 + w, which is what wave w holds at step u.
template <int B>
__device__ __forceinline__ TopkCut select_cut(SelectShared& sh, int* tie_base, const uint32_t (&key)[B], uint32_t cand, int n_cand,
                                              int k_cand, int keep_low) {
    constexpr int kWaves = kSelectThreads / kWave, kChunks = topk_chunks(B);
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    // nothing unprotected survives: no key exceeds the threshold and no tie is kept
    uint32_t T = 0xFFFFFFFFu;
    int quota = 0;
    bool rank_ties = false;
    if (k_cand > 0) {
        // Keys of interest are those with key - base <= span, `same` of them: at first every score's.
        uint32_t base = keep_low ? 0u : 1u, span = 0xFFFFFFFEu;
        int remaining = k_cand, same = n_cand;
        if (tid == 0) sh.n_list = 0;
#pragma unroll 1
        for (;;) {
            // The bins cover their own range: 2048 equal steps from the smallest to the largest. (Unsigned distances from either
            // end are beyond span for all other keys.)
            uint32_t lead = 0xFFFFFFFFu, trail = 0xFFFFFFFFu;
#pragma unroll
            for (int u = 0; u < B; ++u) {
                lead = min(lead, key[u] - base);
                trail = min(trail, base + span - key[u]);
            }
            clear_hist(sh);
            least_of_all(sh, lead, trail);  // ends with a barrier
            base += lead;
            span -= lead + trail;
            if (span == 0u) break;  // one value
            const int shift = max(0, 21 - __clz((int)span));
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (key[u] - base <= span) hist_add(sh, (key[u] - base) >> shift);
            __syncthreads();
            uint32_t bin = 0u;
            select_bin(sh, 0, bin, remaining);
            base += bin << shift;
            span = min((1u << shift) - 1u, span - (bin << shift));  // never beyond the largest key, so never at no_key
            same = sh.ties;
            if (span == 0u || same <= kListMax) break;
        }
        if (span > 0u) {
            // few keys are left: the wanted one by counting
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (key[u] - base <= span) sh.list[atomicAdd(&sh.n_list, 1)] = key[u];
            __syncthreads();
            if (tid < same) {
                const uint32_t mine = sh.list[tid];
                int greater = 0, equal = 0;
                for (int i = 0; i < same; ++i) {
                    greater += sh.list[i] > mine;
                    equal += sh.list[i] == mine;
                }
                if (greater < remaining && remaining <= greater + equal) {  // every holder of that key writes the same
                    sh.prefix = mine;
                    sh.remaining = remaining - greater;
                    sh.ties = equal;
                }
            }
            __syncthreads();
            base = sh.prefix;
            remaining = sh.remaining;
            same = sh.ties;
        }
        T = base;
        quota = remaining;           // >= 1: ties (key == T) still to be kept
        rank_ties = same > remaining;  // more rows tie with the K-th key than may be kept
    }
    if (rank_ties) {
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const unsigned long long m = __ballot(((cand >> u) & 1u) && key[u] == T);
            if (lane == 0) tie_base[u * kWaves + wave] = __popcll(m);
        }
        __syncthreads();
        if (wave == 0) {  // exclusive prefix over the chunks in row order: B/4 consecutive chunks per lane
            constexpr int kPer = kChunks / kWave;
            int v[kPer], tot = 0;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                v[j] = tie_base[lane * kPer + j];
                tot += v[j];
            }
            int incl = tot;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int t = __shfl_up(incl, o);
                if (lane >= o) incl += t;
            }
            int run = incl - tot;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                tie_base[lane * kPer + j] = run;
                run += v[j];
            }
        }
        __syncthreads();
    }
    return TopkCut{T, quota, rank_ties};
}

// Whether the row of key u (of this thread) is kept; called by whole waves.
template <int B>
__device__ __forceinline__ bool cut_keeps(const TopkCut& cut, const int* tie_base, const uint32_t (&key)[B], uint32_t cand, int u, bool in_range) {
    const int lane = threadIdx.x % kWave, chunk = u * (kSelectThreads / kWave) + threadIdx.x / kWave;
    const bool is_cand = (cand >> u) & 1u, tie = is_cand && key[u] == cut.T;
    const bool keep = in_range && (!is_cand || key[u] > cut.T);
    const unsigned long long tie_mask = __ballot(tie);
    // unranked: every tie is kept when any is (quota 0 only with the all-halt state, where no key is kept)
    if (!tie) return keep;
    return cut.rank_ties ? tie_base[chunk] + __popcll(tie_mask & ((1ull << lane) - 1ull)) < cut.quota : cut.quota > 0;
}

}  // namespace dash
