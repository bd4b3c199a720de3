// Stream compaction of the surviving rows (Alg. 1 step 4; Sec. 3.4: each block runs on the
// compacted active sequence). HBM-bound: the row gather moves 2 * row_bytes per kept row.
//
// Layout: one workgroup per 64-row chunk (x column splits). The chunk's output offset is the sum of
// the kept counts of all earlier chunks (written by the decision kernel, one wave ballot each), so no
// cross-workgroup waiting is needed; ranks inside the chunk come from ballot + popcount.
#include "common.h"
#include "publish.h"
#include "score_rows.h"
#include "topk_select.h"

namespace dash {

__global__ __launch_bounds__(256) void chunk_counts_kernel(const uint8_t* __restrict__ halt, int n,
                                                           int32_t* __restrict__ counts) {
    const int chunk = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int lane = threadIdx.x % kWave;
    const int n_chunks = (n + kChunkRows - 1) / kChunkRows;
    if (chunk >= n_chunks) return;
    const int row = chunk * kChunkRows + lane;
    const bool keep = row < n && halt[row] == 0;
    const unsigned long long m = __ballot(keep);
    if (lane == 0) counts[chunk] = __popcll(m);
}

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Gathered rows go by the caches (non-temporal loads and stores): each is read and written once, and what they
// displaced, the rows that are still to be gathered or scattered and the next launches' operands, is worth more there. Measured
// with inputs that change from pass to pass, plain / loads and stores by the caches, us: block-level signal path (scores, TopK, gather, scatter) of
// 16384 rows of 3584 109 / 88, with a reader of the gathered rows behind it 149 / 142, 60000 rows 365 / 304 and 531 / 493, 1000 rows
// 24 / 22 and 27 / 25.5; the chain of eight layers from 32768 rows the same (23.13 ms). In the layer call's one launch (THRESHOLD, 28 heads, width
// 3584) it depends on what comes next. Three calls in turn on inputs and weights of their own, which the caches hold between them: 333
// rows the same, 1000 65.1 / 63.7, 2120 120 / 113, 3000 167 / 153, 6000 394 / 393. Layers one behind the other, 16 with weights of
// their own and the next one's norm reading the gathered rows, us a layer: 64 rows 45.3 / 46.1, 333 75.4 / 75.5, 1000 134.4 / 134.2,
// 2120 200 / 201, 3000 260 / 259, 6000 587 / 582; of width 512 (60 layers) 333 rows 29.9 / 30.0, 3000 61.3 / 61.6, 6000 105.1 / 105.1: within
// a percent either way but for the fewest rows. (Both in one kernel, plain up to 4 MB of rows: 64 rows 45.5, but 0.3 us more in a call by itself.)
__device__ __forceinline__ uint4 load_once(const uint4* p) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store_once(uint4* p, uint4 v) {
    const u32x4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p));
}

constexpr int kCompactThreads = 256;
constexpr int kCompactWaves = kCompactThreads / kWave;

__global__ __launch_bounds__(kCompactThreads) void compact_kernel(
    const uint8_t* __restrict__ halt, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ active_idx, const uint4* __restrict__ x_next, int n, int row_vecs,
    int vecs_per_split, uint4* __restrict__ x_compact, int32_t* __restrict__ new_idx,
    int32_t* __restrict__ n_out) {
    __shared__ int wave_part[kCompactWaves];
    __shared__ int kept_rows[kChunkRows];
    const int chunk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;

    // exclusive offset of this chunk: integer sum of earlier chunk counts (order does not matter)
    int part = 0;
    for (int c = tid; c < chunk; c += kCompactThreads) part += counts[c];
    part = wave_sum_int(part);
    if (lane == 0) wave_part[wave] = part;

    const int row = chunk * kChunkRows + lane;
    const bool keep = row < n && halt[row] == 0;
    const unsigned long long mask = __ballot(keep);
    const int rank = __popcll(mask & ((1ull << lane) - 1ull));
    const int cnt = __popcll(mask);
    if (wave == 0 && keep) kept_rows[rank] = row;
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int w = 0; w < kCompactWaves; ++w) base += wave_part[w];

    if (blockIdx.y == 0 && wave == 0) {
        if (keep) new_idx[base + rank] = active_idx[row];
        if (chunk == (int)gridDim.x - 1 && lane == 0) *n_out = base + cnt;
    }

    // gather: a wave copies its kept rows four at a time (four independent 16-byte loads per lane in
    // flight before the first store); lanes stride over this split's vectors
    const int v0 = blockIdx.y * vecs_per_split;
    const int v1 = min(row_vecs, v0 + vecs_per_split);
    constexpr int R = 4;
    for (int r0 = wave * R; r0 < cnt; r0 += kCompactWaves * R) {
        const uint4* src[R];
        uint4* dst[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int r = min(r0 + i, cnt - 1);  // a clamped duplicate rewrites the same bytes
            src[i] = x_next + (size_t)kept_rows[r] * row_vecs;
            dst[i] = x_compact + (size_t)(base + r) * row_vecs;
        }
        for (int c = v0 + lane; c < v1; c += kWave) {
            uint4 val[R];
#pragma unroll
            for (int i = 0; i < R; ++i) val[i] = load_once(src[i] + c);
#pragma unroll
            for (int i = 0; i < R; ++i) store_once(dst[i] + c, val[i]);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Score, decision and compaction in ONE launch (rules NONE and THRESHOLD of the layer call).
//
// Grid (chunks of 64 rows, column splits), 256 threads. Workgroup (c, 0) finishes the scores of chunk c from the
// norm partials, writes scores and halt flags and PUBLISHES the chunk's kept mask and count; every workgroup
// (c, y) takes its chunk's mask and the counts of all earlier chunks from the published words, then gathers its
// columns of the kept rows as compact_kernel does. Nothing is computed twice and nothing waits for a kernel boundary.
//
// Published words: publish.h. They must be zero when the kernel starts (the attention kernel of the same layer call clears
// them).
//
// Waiting. Workgroups are dispatched in the order of their linear index (x fastest), and the publishers (c, 0) are the first of
// the grid: a workgroup (c, y) waits for publishers (c', 0) with c' <= c only, which have a smaller linear index and publish without
// having waited. Each XCD takes its share of the grid in that order, at its own pace: where other streams' kernels fill one, its publishers
// come later than readers elsewhere.
// Every wait is bounded (kPubSpinLimit), and one that ends without its word fails the call: whoever gives up gathers nothing and writes
// the survivor count -1.
// The count is 0 when the kernel starts (cleared with the words), and its writer, one thread of the last chunk's publisher,
// exchanges the 0 for the count: a -1 that is there already stays, and one that comes later replaces the count.
// ------------------------------------------------------------------------------------------------
constexpr int kPubSpinLimit = 1 << 20;

__device__ __forceinline__ unsigned long long wait_published(const unsigned long long* word, bool& bad) {
    unsigned long long v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int spins = 0;
    while (!pub_ready(v)) {
        __builtin_amdgcn_s_sleep(4);
        if (++spins > kPubSpinLimit) break;
        v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!pub_ready(v)) bad = true;
    return v;
}

__global__ __launch_bounds__(kCompactThreads) void score_decide_compact_kernel(
    const float* __restrict__ partials, int cols, int fold, int n, int score_kind, int rule, float tau, int n_first,
    int n_last, float* __restrict__ scores, uint8_t* __restrict__ halt, unsigned long long* __restrict__ published,
    const int32_t* __restrict__ active_idx, const uint4* __restrict__ x_next, int row_vecs, int vecs_per_split,
    uint4* __restrict__ x_compact, int32_t* __restrict__ new_idx, int32_t* __restrict__ n_out) {
    __shared__ float2 red[4][kChunkRows];
    __shared__ int wave_part[kCompactWaves];
    __shared__ int wave_bad[kCompactWaves];
    __shared__ int kept_rows[kChunkRows];
    const int chunk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int row = chunk * kChunkRows + lane;
    bool bad = false;
    unsigned long long mask;
    if (blockIdx.y == 0) {
        // publisher: scores, flags, the chunk's kept mask
        const float2 t = row_sums_256(partials, cols, fold, n, chunk * kChunkRows, red);
        bool keep = false;
        if (row < n) {  // every wave holds the sums of the chunk's rows (row = lane): every wave gets the same mask
            const float sc = score_from_sums(t, score_kind);
            const bool h = rule == DASH_RULE_THRESHOLD && !row_protected(row, n, n_first, n_last) && sc < tau;
            keep = !h;
            if (wave == 0) {
                scores[row] = sc;
                halt[row] = h ? 1 : 0;
            }
        }
        mask = __ballot(keep);
        if (tid == 0) {
            __hip_atomic_store(published + 2 * chunk, pub_word0(mask, __popcll(mask)), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(published + 2 * chunk + 1, pub_word1(mask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    } else {
        // the chunk's mask from its publisher (every lane reads the same two words: one request per wave)
        const unsigned long long w0 = wait_published(published + 2 * chunk, bad);
        const unsigned long long w1 = wait_published(published + 2 * chunk + 1, bad);
        mask = pub_mask(w0, w1);
    }
    // exclusive offset of this chunk: kept counts of all earlier chunks (integer sum, order does not matter)
    int part = 0;
    for (int c = tid; c < chunk; c += kCompactThreads)
        part += pub_count(wait_published(published + 2 * c, bad));
    part = wave_sum_int(part);
    const unsigned long long any_bad = __ballot(bad);
    if (lane == 0) {
        wave_part[wave] = part;
        wave_bad[wave] = any_bad != 0ull;
    }
    const bool keep = (mask >> lane) & 1ull;
    const int rank = __popcll(mask & ((1ull << lane) - 1ull));
    const int cnt = __popcll(mask);
    if (wave == 0 && keep) kept_rows[rank] = row;
    __syncthreads();
    int base = 0, failed = 0;
#pragma unroll
    for (int w = 0; w < kCompactWaves; ++w) {
        base += wave_part[w];
        failed |= wave_bad[w];
    }
    if (failed) {  // uniform: every thread read the same LDS words
        if (tid == 0) __hip_atomic_store(n_out, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (chunk == (int)gridDim.x - 1 && blockIdx.y == 0 && tid == 0) {
        int cleared = 0;
        (void)__hip_atomic_compare_exchange_strong(n_out, &cleared, base + cnt, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    }
    if (blockIdx.y == 0 && wave == 0 && keep) new_idx[base + rank] = active_idx[row];
    const int v0 = ((int)gridDim.y - 1 - (int)blockIdx.y) * vecs_per_split;
    const int v1 = min(row_vecs, v0 + vecs_per_split);
    constexpr int R = 4;
    for (int r0 = wave * R; r0 < cnt; r0 += kCompactWaves * R) {
        const uint4* src[R];
        uint4* dst[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int r = min(r0 + i, cnt - 1);  // a clamped duplicate rewrites the same bytes
            src[i] = x_next + (size_t)kept_rows[r] * row_vecs;
            dst[i] = x_compact + (size_t)(base + r) * row_vecs;
        }
        for (int c = v0 + lane; c < v1; c += kWave) {
            uint4 val[R];
#pragma unroll
            for (int i = 0; i < R; ++i) val[i] = load_once(src[i] + c);
#pragma unroll
            for (int i = 0; i < R; ++i) store_once(dst[i] + c, val[i]);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// TOPK of few rows: scores, decision and compaction in one launch without any exchange. Each workgroup (c, y) finishes the
// scores of ALL rows, one of its waves selects, and the workgroup gathers its columns of its chunk's kept rows. Repeated is little
// (at width 3584 the pairs of 256 rows are 115 KB, through the L2); saved are two round trips between workgroups (keys, masks), and no word has to be cleared. Thread (r, q)
// of 256 x 4 adds a quarter of the pairs of rows r, r + 256, ...
// The selection, 4 RPT keys per lane of one wave: the k_cand-th greatest key bit by bit (the greatest T that k_cand keys reach),
// counted by ballots, without a barrier; where exactly k_cand keys reach a T the set is found, so only rows that tie with the
// last one kept take all 32 steps.
// Bound by latency: norms, selection (about a microsecond), gather. (Counting, for each row, the candidates before it was as fast
// up to 128 rows and 1 us slower at 256.) Figures: few_topk.
// ------------------------------------------------------------------------------------------------
constexpr int kFewThreads = 1024;

template <int RPT>
__global__ __launch_bounds__(kFewThreads) void topk_compact_few_kernel(
    const float* __restrict__ partials, int cols, int fold, int n, int score_kind, int k_keep, int n_first, int n_last,
    float* __restrict__ scores, uint8_t* __restrict__ halt, const int32_t* __restrict__ active_idx,
    const uint4* __restrict__ x_next, int row_vecs, int vecs_per_split, uint4* __restrict__ x_compact,
    int32_t* __restrict__ new_idx, int32_t* __restrict__ n_out) {
    static_assert(RPT <= 2, "rows of a launch");
    constexpr int kRows = 256 * RPT, kChunks = kRows / kChunkRows;
    __shared__ float2 red[4][kRows];
    __shared__ uint32_t keys[kRows];
    __shared__ unsigned long long masks[kChunks];
    __shared__ int kept_rows[kChunkRows];
    const int chunk = blockIdx.x, tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
        const int r = u * 256 + tid % 256;
        red[tid / 256][r] = row_quarter(partials, cols, fold, n, r, tid / 256);
    }
    __syncthreads();
    const int lo = min(n_first, n), hi = max(lo, n - n_last);  // candidates are rows [lo, hi)
    if (tid < kRows) {
        const float sc = score_from_sums(add_quarters(red[0][tid], red[1][tid], red[2][tid], red[3][tid]), score_kind);
        keys[tid] = tid >= lo && tid < hi ? order_key(sc) : 0u;  // 0, which no score's key is: no candidate
        if (blockIdx.y == 0 && wave == chunk && tid < n) scores[tid] = sc;
    }
    __syncthreads();
    if (wave == 0) {
        const int k_cand = max(0, min(k_keep - (n - (hi - lo)), hi - lo));
        uint32_t k[kChunks], T = 0u;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) k[c] = keys[c * kChunkRows + lane];
        int reach = k_cand == 0 ? 0 : hi - lo;  // keys that reach T
#pragma unroll 1
        for (uint32_t bit = 0x80000000u; bit != 0u && reach != k_cand; bit >>= 1) {
            int cnt = 0;
#pragma unroll
            for (int c = 0; c < kChunks; ++c) cnt += __popcll(__ballot(k[c] >= (T | bit)));
            if (cnt >= k_cand) {
                T |= bit;
                reach = cnt;
            }
        }
        int over = reach - k_cand;  // of the rows at T itself the last ones go, this many
#pragma unroll
        for (int c = kChunks - 1; c >= 0; --c) {
            const int r = c * kChunkRows + lane;
            unsigned long long kept = k_cand == 0 ? 0ull : __ballot(k[c] != 0u && k[c] >= T);
            if (over > 0) {
                const unsigned long long tie = __ballot(k[c] == T);
                kept &= ~__ballot(k[c] == T && __popcll(tie >> lane) <= over);  // this row and the ties behind it in the chunk
                over -= min(over, (int)__popcll(tie));
            }
            kept |= __ballot(r < n && row_protected(r, n, n_first, n_last));
            if (lane == 0) masks[c] = kept;
            if (c == chunk) {
                const bool keep = (kept >> lane) & 1ull;
                if (keep) kept_rows[__popcll(kept & ((1ull << lane) - 1ull))] = r;
                if (blockIdx.y == 0 && r < n) halt[r] = keep ? 0 : 1;
            }
        }
    }
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) base += c < chunk ? __popcll(masks[c]) : 0;
    const int cnt = __popcll(masks[chunk]);
    if (blockIdx.y == 0) {
        if (tid < cnt) new_idx[base + tid] = active_idx[kept_rows[tid]];
        if (chunk == (int)gridDim.x - 1 && tid == 0) *n_out = base + cnt;
    }
    const int v0 = (int)blockIdx.y * vecs_per_split, v1 = min(row_vecs, v0 + vecs_per_split);
    constexpr int R = 4;
    for (int r0 = wave * R; r0 < cnt; r0 += kFewThreads / kWave * R) {
        const uint4* from[R];
        uint4* to[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int r = min(r0 + i, cnt - 1);  // a clamped duplicate rewrites the same bytes
            from[i] = x_next + (size_t)kept_rows[r] * row_vecs;
            to[i] = x_compact + (size_t)(base + r) * row_vecs;
        }
        for (int c = v0 + lane; c < v1; c += kWave) {
            uint4 val[R];
#pragma unroll
            for (int i = 0; i < R; ++i) val[i] = load_once(from[i] + c);
#pragma unroll
            for (int i = 0; i < R; ++i) store_once(to[i] + c, val[i]);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// TOPK of more rows in one launch. The first workgroups, one per 64 rows, finish scores and share them as order-preserving keys
// (one 32-bit word per row, cleared by the attention kernel of the same call; no key is 0, so a word is its own READY flag);
// they wait for nothing and are done. Each of the others (chunk, column split) takes the keys of ALL rows, finds the cut with all of its
// 1024 threads (select_cut, keys in registers), and gathers its columns of its chunk's kept rows. The cut is found in as many
// places as there are workgroups, all resident at once, so it costs its time once; saved are the launches of score, decision and
// compaction and two trips of flags and counts through memory.
// Waiting: a key that does not come in time is computed where it is missing (take_keys, publish.h), so no workgroup depends on another
// and the call cannot fail (a bounded wait that failed it, with the count exchanged for a -1, was no faster: 640 rows of width 512 23.0 -> 22.4 us
// a layer, 2120 of 3584 107.2 -> 106.8). All threads ask for their keys at once and again while one is missing: with one wave
// asking for the last row first, a trip to memory more, 640 rows of width 512 took 23.9 us and not 23.1.
// Bound by latency: pairs, key out and back, cut, gather. Figures: kFusedTopkRows.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kSelectThreads, 8) void topk_compact_kernel(
    const float* __restrict__ partials, int cols, int fold, int n, int n_chunks, int score_kind, int k_keep, int n_first, int n_last,
    float* __restrict__ scores, uint8_t* __restrict__ halt, uint32_t* __restrict__ words, const int32_t* __restrict__ active_idx,
    const uint4* __restrict__ x_next, int row_vecs, int vecs_per_split, uint4* __restrict__ x_compact,
    int32_t* __restrict__ new_idx, int32_t* __restrict__ n_out) {
    constexpr int B = kFusedTopkRows / kSelectThreads;  // keys of a thread
    static_assert(kSelectThreads >= 4 * kChunkRows, "a thread per row of a chunk and quarter");
    __shared__ SelectShared sh;
    __shared__ float2 red[4][kChunkRows];
    __shared__ int tie_base[topk_chunks(B)];
    __shared__ unsigned long long masks[topk_chunks(B)];
    __shared__ int kept_rows[kChunkRows];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    if ((int)blockIdx.x < n_chunks) {  // publisher
        const int row = (int)blockIdx.x * kChunkRows + lane;
        if (wave < 4) red[wave][lane] = row_quarter(partials, cols, fold, n, row, wave);
        __syncthreads();
        if (wave == 0 && row < n) {
            const float sc = score_from_sums(add_quarters(red[0][lane], red[1][lane], red[2][lane], red[3][lane]), score_kind);
            __hip_atomic_store(words + row, order_key(sc), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            scores[row] = sc;
        }
        return;
    }
    const int chunk = ((int)blockIdx.x - n_chunks) % n_chunks, split = ((int)blockIdx.x - n_chunks) / n_chunks;
    const int lo = min(n_first, n), hi = max(lo, n - n_last);  // candidates are rows [lo, hi)
    const int k_cand = max(0, min(k_keep - (n - (hi - lo)), hi - lo));
    uint32_t key[B];
    take_keys<B>(
        key, tid, kSelectThreads, n,
        [&](int r) { return __hip_atomic_load(words + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
        [&](int r) { return order_key(score_from_sums(row_sums(partials, cols, fold, n, r), score_kind)); },
        [] { __builtin_amdgcn_s_sleep(2); });
    uint32_t cand = 0u;  // bit u: row u * 1024 + tid is a candidate; 0, which no score's key is, for others
#pragma unroll
    for (int u = 0; u < B; ++u) {
        const int r = u * kSelectThreads + tid;
        if (r >= lo && r < hi) cand |= 1u << u;
        else key[u] = 0u;
    }
    const TopkCut cut = select_cut<B>(sh, tie_base, key, cand, hi - lo, k_cand, 0);
#pragma unroll
    for (int u = 0; u < B; ++u) {
        const unsigned long long m = __ballot(cut_keeps<B>(cut, tie_base, key, cand, u, u * kSelectThreads + tid < n));
        if (lane == 0) masks[u * (kSelectThreads / kWave) + wave] = m;
    }
    __syncthreads();
    int base = 0;
    for (int c = lane; c < chunk; c += kWave) base += __popcll(masks[c]);
    base = wave_sum_int(base);
    const unsigned long long mask = masks[chunk];
    const int cnt = __popcll(mask), rank = __popcll(mask & ((1ull << lane) - 1ull)), row = chunk * kChunkRows + lane;
    const bool keep = (mask >> lane) & 1ull;
    if (wave == 0) {
        if (keep) kept_rows[rank] = row;
        if (split == 0) {
            if (row < n) halt[row] = keep ? 0 : 1;
            if (keep) new_idx[base + rank] = active_idx[row];
            if (chunk == n_chunks - 1 && lane == 0) *n_out = base + cnt;
        }
    }
    __syncthreads();
    const int v0 = split * vecs_per_split, v1 = min(row_vecs, v0 + vecs_per_split);
    constexpr int R = 4;
    for (int r0 = wave * R; r0 < cnt; r0 += kSelectThreads / kWave * R) {
        const uint4* from[R];
        uint4* to[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int r = min(r0 + i, cnt - 1);  // a clamped duplicate rewrites the same bytes
            from[i] = x_next + (size_t)kept_rows[r] * row_vecs;
            to[i] = x_compact + (size_t)(base + r) * row_vecs;
        }
        for (int c = v0 + lane; c < v1; c += kWave) {
            uint4 val[R];
#pragma unroll
            for (int i = 0; i < R; ++i) val[i] = load_once(from[i] + c);
#pragma unroll
            for (int i = 0; i < R; ++i) store_once(to[i] + c, val[i]);
        }
    }
}

__global__ void write_zero_kernel(int32_t* p) { *p = 0; }

__global__ __launch_bounds__(256) void validate_idx_kernel(const int32_t* __restrict__ idx, int n, int N,
                                                           int32_t* __restrict__ violations) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int v = idx[i];
    bool bad = v < 0 || (N >= 0 && v >= N);
    if (i > 0 && idx[i - 1] >= v) bad = true;
    if (bad) atomicAdd(violations, 1);
}

constexpr int kGatherGroups = 2048;  // of 256 threads
constexpr int kTopkGatherGroups = 384;  // of 1024 threads, of which the chip holds 512
// Column splits of the gather: whole wave-widths (64 vectors), enough workgroups to fill 256 CUs several times over (`wanted`).
static void gather_splits(int n_chunks, int row_vecs, int wanted, int& splits, int& vecs_per_split) {
    const int wave_cols = (row_vecs + kWave - 1) / kWave;
    splits = (wanted + n_chunks - 1) / n_chunks;
    if (splits > wave_cols) splits = wave_cols;
    if (splits < 1) splits = 1;
    vecs_per_split = ((wave_cols + splits - 1) / splits) * kWave;
    splits = (row_vecs + vecs_per_split - 1) / vecs_per_split;
}

dash_status launch_chunk_counts(const uint8_t* halt, int n, int32_t* chunk_counts, hipStream_t s) {
    const int n_chunks = (n + kChunkRows - 1) / kChunkRows;
    if (n_chunks == 0) return DASH_OK;
    const int blocks = (n_chunks * kWave + 255) / 256;
    hipLaunchKernelGGL(chunk_counts_kernel, dim3(blocks), dim3(256), 0, s, halt, n, chunk_counts);
    return launch_status();
}

dash_status launch_compact(const uint8_t* halt, const int32_t* chunk_counts, const int32_t* active_idx,
                           const void* x_next, int n, int row_bytes, void* x_compact,
                           int32_t* new_active_idx, int32_t* n_active_out, hipStream_t s) {
    if (n == 0) {
        hipLaunchKernelGGL(write_zero_kernel, dim3(1), dim3(1), 0, s, n_active_out);
        return launch_status();
    }
    const int n_chunks = (n + kChunkRows - 1) / kChunkRows;
    const int row_vecs = row_bytes / 16;
    int splits, vecs_per_split;
    gather_splits(n_chunks, row_vecs, kGatherGroups, splits, vecs_per_split);
    hipLaunchKernelGGL(compact_kernel, dim3(n_chunks, splits), dim3(kCompactThreads), 0, s, halt,
                       chunk_counts, active_idx, (const uint4*)x_next, n, row_vecs, vecs_per_split,
                       (uint4*)x_compact, new_active_idx, n_active_out);
    return launch_status();
}

// words of the one-launch kernels: two per chunk, for TOPK a key per row
size_t published_bytes(int n, bool topk) {
    return topk ? (size_t)n * sizeof(uint32_t) : (size_t)((n + kChunkRows - 1) / kChunkRows) * 2 * sizeof(unsigned long long);
}

// Scores, decision and compaction in one launch (TOPK: n <= kFusedTopkRows). `published` (published_bytes, 8-byte aligned) must have been
// cleared on this stream before (launch_flash_fwd does it for the layer call), except for TOPK where few_topk holds, which hands
// nothing over; for NONE and THRESHOLD the count too.
dash_status launch_score_decide_compact(const dash_layer_params& p, const NormSums& sums, int n, float* scores, uint8_t* halt, void* published, const int32_t* active_idx,
                                        const void* x_next, int row_bytes, void* x_compact, int32_t* new_active_idx,
                                        int32_t* n_active_out, hipStream_t s) {
    const int n_chunks = (n + kChunkRows - 1) / kChunkRows;
    const int row_vecs = row_bytes / 16;
    int splits, vecs_per_split;
    const bool topk = p.rule == DASH_RULE_TOPK, few = topk && few_topk(n, sums.cols);
    gather_splits(n_chunks, row_vecs, topk && !few ? kTopkGatherGroups : kGatherGroups, splits, vecs_per_split);
    if (few) {
        hipLaunchKernelGGL(n <= 256 ? topk_compact_few_kernel<1> : topk_compact_few_kernel<2>,
                           dim3(n_chunks, splits), dim3(kFewThreads), 0, s, sums.pairs, sums.cols, sums.fold, n, p.score_kind,
                           topk_keep(p, n), p.keep_first_n, p.keep_last_n, scores, halt, active_idx, (const uint4*)x_next,
                           row_vecs, vecs_per_split, (uint4*)x_compact, new_active_idx, n_active_out);
        return launch_status();
    }
    if (topk) {
        hipLaunchKernelGGL(topk_compact_kernel, dim3(n_chunks * (1 + splits)), dim3(kSelectThreads), 0, s, sums.pairs, sums.cols, sums.fold, n, n_chunks, p.score_kind, topk_keep(p, n),
                           p.keep_first_n, p.keep_last_n, scores, halt, (uint32_t*)published, active_idx, (const uint4*)x_next,
                           row_vecs, vecs_per_split, (uint4*)x_compact, new_active_idx, n_active_out);
        return launch_status();
    }
    hipLaunchKernelGGL(score_decide_compact_kernel, dim3(n_chunks, splits), dim3(kCompactThreads), 0, s, sums.pairs, sums.cols,
                       sums.fold, n, p.score_kind, p.rule, p.tau, p.keep_first_n, p.keep_last_n, scores, halt,
                       (unsigned long long*)published, active_idx, (const uint4*)x_next, row_vecs, vecs_per_split,
                       (uint4*)x_compact, new_active_idx, n_active_out);
    return launch_status();
}

dash_status launch_validate_idx(const int32_t* idx, int n, int N, int32_t* violations, hipStream_t s) {
    hipLaunchKernelGGL(write_zero_kernel, dim3(1), dim3(1), 0, s, violations);
    if (n > 0)
        hipLaunchKernelGGL(validate_idx_kernel, dim3((n + 255) / 256), dim3(256), 0, s, idx, n, N,
                           violations);
    return launch_status();
}

// Halted tokens keep the state they had when they halted (Sec. 3.4): selected rows are written to a
// full-length buffer at their original positions. One wave per row, 16-byte vectors; rows whose position
// lies outside [0, N) are skipped. The buffer is read when the prompt is done: its rows are stored by the caches (with the signal's
// x_old loaded so, the signal path of 16384 rows 118 -> 107.5 us).
template <typename T>
__global__ __launch_bounds__(256) void scatter_rows_kernel(const T* __restrict__ rows, const int32_t* __restrict__ idx,
                                                           const uint8_t* __restrict__ sel, int sel_value, int n,
                                                           int d, int N, T* __restrict__ full) {
    constexpr int VEC = 16 / (int)sizeof(T);
    const int row = (int)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) / kWave);
    const int lane = threadIdx.x % kWave;
    if (row >= n) return;
    if (sel && sel[row] != (uint8_t)sel_value) return;
    const int p = idx[row];
    if (p < 0 || p >= N) return;
    const u32x4* src = reinterpret_cast<const u32x4*>(rows + (size_t)row * d);
    u32x4* dst = reinterpret_cast<u32x4*>(full + (size_t)p * d);
    for (int c = lane; c < d / VEC; c += kWave) __builtin_nontemporal_store(src[c], dst + c);
}

dash_status launch_scatter_rows(const void* rows, const int32_t* idx, const uint8_t* sel, int sel_value, int n,
                                int d, int dtype, int N, void* full, hipStream_t s) {
    if (n == 0) return DASH_OK;
    const int blocks = (int)(((size_t)n * kWave + 255) / 256);
    if (dtype == DASH_BF16)
        hipLaunchKernelGGL(scatter_rows_kernel<__bf16>, dim3(blocks), dim3(256), 0, s, (const __bf16*)rows, idx, sel,
                           sel_value, n, d, N, (__bf16*)full);
    else
        hipLaunchKernelGGL(scatter_rows_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float*)rows, idx, sel,
                           sel_value, n, d, N, (float*)full);
    return launch_status();
}

}  // namespace dash
