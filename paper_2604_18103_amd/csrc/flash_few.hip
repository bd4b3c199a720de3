// Attention over few rows (bf16): the same operator as flash_fwd.hip, for sequences so short that the time is a workgroup's
// chain of latencies and not the chip's throughput.
#include "common.h"
#include "flash_map.h"
#include "lds_ops.h"
#include "staging_addr.h"

namespace dash {

// ------------------------------------------------------------------------------------------------
// A workgroup owns 32 query rows of one head; its KW waves split the KEYS: wave w takes the 32-key blocks w, w + KW, ... Each
// wave fetches its blocks into LDS of its own (global -> LDS loads, one K and one V stage), so the loop has no barrier, and
// the waves meet once, at the end: O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w, in the order of w.
//
// The products are those of the tiled kernels (S^T = K Q^T, then O^T += V^T P^T with the score registers as P's operand;
// layouts in flash_fwd.hip). The scale is applied to the fp32 scores, so Q is not rounded a second time (error against 64 bits
// 2.2e-3 of a row, the rounding of P and O). The softmax reference of a row moves only when a block's maximum exceeds it by
// more than 2^8: any reference gives the same quotient.
//
// One K and one V stage per wave do: K of the next block is requested when this block's scores have read theirs, V when its
// P V has; either is in flight while the other product and the softmax run, and a SIMD has a second wave.
//
// What bounds it: at a few hundred rows the chain launch (3 us), arguments and first loads (1 us), one or two blocks (0.8 us
// each), exchange through LDS (0.7 us) and store, so 177 rows of 28 heads of 128 take 7.2 us where the tiled kernels, with
// 64-key tiles for 128 rows and barriers between the waves' phases, take 10.6; from two workgroups per unit on the
// key blocks' way from the L2 into LDS, 16 KB per 32 x 32 scores. Where the rule lies: few_waves (staging_addr.h).
// ------------------------------------------------------------------------------------------------
template <int DH>
struct FewSmem {
    static constexpr int kStage = kFewKeys * DH;  // elements of a K or V stage, and of the 32 query rows
    // the query rows; per wave a K and a V stage, where its sums are left in the end (32 rows of DH fp32: the same bytes);
    // per wave the sums' statistics and the limits of its masked block
    static constexpr int bytes(int KW) { return kStage * (int)sizeof(__bf16) + KW * (2 * kStage * (int)sizeof(__bf16) + 32 * 8 + 32 * 4); }
    static_assert(2 * kStage * sizeof(__bf16) == 32 * DH * sizeof(float), "a wave's sums take its stages' place");
};

// PARTS: the keys are cut over gridDim.y workgroups as well (few_tail_parts), `blocks_per_part` blocks each; a part leaves its rows' sums
// [part][row - row_base][head][DH] in `sums` and their (reference, sum of weights) behind all of them, for few_parts_kernel to add.
template <int DH, int KW, bool PARTS>
__global__ __launch_bounds__(KW * kWave, 2) void flash_few(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                                                            const __bf16* __restrict__ v, const int32_t* __restrict__ pos,
                                                            __bf16* __restrict__ o, int n, int Hq, int Hkv, float scale_log2,
                                                            int causal, int n_qtiles, FaMap mp, uint32_t* __restrict__ clear_words,
                                                            int n_clear, int row_base, int32_t* __restrict__ clear_count,
                                                            float* __restrict__ sums, int blocks_per_part) {
    using SM = FewSmem<DH>;
    constexpr int KC = DH / 16, DB = DH / 32;
    constexpr int LOADS = few_loads(DH);
    constexpr float kMove = 8.f;  // how far (log2) a score may exceed the reference
    extern __shared__ __attribute__((aligned(16))) unsigned char few_smem_raw[];
    if (blockIdx.x == 0)  // scratch of the kernels that follow in the layer call
        for (int c = threadIdx.x; c <= n_clear; c += KW * kWave) {
            if (c < n_clear) clear_words[c] = 0u;
            else if (clear_count) *clear_count = 0;
        }
    int qt, head;
    if (!fa_map_block(mp, (int)blockIdx.x, n_qtiles, Hq, Hkv, qt, head)) return;  // whole workgroup
    const int g = head / (Hq / Hkv);
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int j = lane % 32, h = lane / 32;
    const int tg = lane / 16, ti = lane % 16;
    const int row0 = row_base + qt * 32, row = min(row0 + j, n - 1);
    __bf16* Qs = reinterpret_cast<__bf16*>(few_smem_raw);
    __bf16* Ks = Qs + SM::kStage + wave * 2 * SM::kStage;
    __bf16* Vs = Ks + SM::kStage;
    float2* stat = reinterpret_cast<float2*>(Qs + (1 + 2 * KW) * SM::kStage);  // [KW][32]
    int* limit = reinterpret_cast<int*>(stat + KW * 32) + wave * 32;

    // block b: rows 32 b .. 32 b + 31 of a sequence; the lane offsets are those of a whole block, rows beyond the end are clamped
    const int kend = causal ? min(n, row0 + 32) : n, n_blocks = (kend + kFewKeys - 1) / kFewKeys;
    const int first = PARTS ? (int)blockIdx.y * blocks_per_part : 0, end = PARTS ? min(n_blocks, first + blocks_per_part) : n_blocks;
    // the query rows, once for all waves (a wave's own fragments from memory are 32-byte pieces of 32 rows per instruction: four
    // waves kept the address unit busy with them for most of the prologue)
#pragma unroll
    for (int u = 0; u < few_q_loads(DH, KW); ++u) {
        const int i = few_q_index(wave, u, DH, KW);
        if (LOADS % KW != 0 && i >= LOADS) continue;
        dma_load16(reinterpret_cast<const char*>(q) + few_q_base(row0, Hq, DH),
                   few_q_voff(row0, n, few_row(i, lane, DH), lane, head, Hq, DH), lds_addr(Qs) + (uint32_t)(i * 1024));
    }
    uint32_t k_off[LOADS], v_off[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int r = few_row(i, lane, DH);
        k_off[i] = fa_dma_voff(r, lane, g, Hkv, DH, true);
        v_off[i] = fa_dma_voff(r, lane, g, Hkv, DH, false);
    }
    const size_t block_bytes = few_block_bytes(Hkv, DH);
    auto request = [&](const __bf16* src, const uint32_t* off, const __bf16* stage, int b) {
        const char* base = reinterpret_cast<const char*>(src) + (size_t)b * block_bytes;
        const uint32_t lds = lds_addr(stage);
        const int rows_left = n - b * kFewKeys;
        if (rows_left >= kFewKeys) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) dma_load16(base, off[i], lds + (uint32_t)(i * 1024));
        } else {
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                dma_load16(base, fa_dma_voff_tail(off[i], few_row(i, lane, DH), rows_left, Hkv, DH), lds + (uint32_t)(i * 1024));
        }
    };
    // A row's last block is the only one with keys that it may not see: those at later positions (the block at the diagonal), or,
    // without a causal mask, those beyond the last key. Key j of that block is masked for the rows below its limit.
    const int pos_q = causal ? pos[row] : 0;
    const bool masked = causal || n % kFewKeys != 0;
    if (first + wave < end) {
        request(k, k_off, Ks, first + wave);
        request(v, v_off, Vs, first + wave);
        dma_wait_keep<2 * LOADS>();
    } else {
        dma_wait();
    }
    limit[j] = (n_blocks - 1) * kFewKeys + j >= n ? 0x7FFFFFFF : pos_q;  // causal: key j is row j; both halves of the wave write the same
    __syncthreads();
    bf16x8 Qf[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
        Qf[kc] = *reinterpret_cast<const bf16x8*>(&Qs[j * DH + ((2 * kc + h) ^ fa_k_swz(j, DH)) * 8]);
    f32x16 O[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[db][r] = 0.f;
    float m = -INFINITY, l = 0.f;
    // Q stays in registers
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) asm volatile("" : "+v"(Qf[kc]));

    for (int b = first + wave; b < end; b += KW) {
        const bool more = b + KW < end;  // wave-uniform
        dma_wait_keep<LOADS>();  // K(b); V(b), requested after it, may be in flight
        wave_sync_lds();
        f32x16 S;
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            const bf16x8 Kf = *reinterpret_cast<const bf16x8*>(&Ks[j * DH + ((2 * kc + h) ^ fa_k_swz(j, DH)) * 8]);
            S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Kf, Qf[kc], S, 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // K(b) is read
        if (more) request(k, k_off, Ks, b + KW);
        if (masked && b == n_blocks - 1) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const int4 lim = *reinterpret_cast<const int4*>(&limit[8 * rg + 4 * h]);
                const int lm[4] = {lim.x, lim.y, lim.z, lim.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) S[4 * rg + e] = lm[e] > pos_q ? -INFINITY : S[4 * rg + e];
            }
        }
        float c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = fmaxf(fmaxf(S[e], S[4 + e]), fmaxf(S[8 + e], S[12 + e]));
        float mx = fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * scale_log2;
        const bool moves = mx > m + kMove;  // m = -inf: at the first finite maximum
        if (__any(moves)) {
            const float alpha = moves ? __builtin_amdgcn_exp2f(m - mx) : 1.f;
            m = moves ? mx : m;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) O[db][r] *= alpha;
        }
        const float ref = m == -INFINITY ? 0.f : m;  // nothing visible yet, or only scores of -inf
        uint32_t Pw[2][4];
        float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(S[r], scale_log2, -ref));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(S[r + 1], scale_log2, -ref));
            ps[(r / 2) % 4] += p0;
            ps[(r / 2 + 2) % 4] += p1;
            const bf16x2 pk = {(__bf16)p0, (__bf16)p1};
            Pw[r / 8][(r % 8) / 2] = __builtin_bit_cast(uint32_t, pk);
        }
        l += (ps[0] + ps[1]) + (ps[2] + ps[3]);
        if (more)
            dma_wait_keep<LOADS>();  // V(b); K of the next block may be in flight
        else
            dma_wait();
        wave_sync_lds();
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const u32x4 pw = {Pw[kk][0], Pw[kk][1], Pw[kk][2], Pw[kk][3]};
            const bf16x8 Pf = __builtin_bit_cast(bf16x8, pw);
            const int krow = 16 * kk + 4 * (tg / 2) + ti / 4;  // and krow + 8: the same swizzle
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int col = 32 * db + 16 * (tg % 2) + 4 * (ti % 4);
                const int scol = ((col / 8) ^ fa_v_swz(krow, DH)) * 8 + col % 8;
                const s16x4 lo = lds_read_tr16(&Vs[krow * DH + scol]);
                const s16x4 hi = lds_read_tr16(&Vs[(krow + 8) * DH + scol]);
                const bf16x8 Vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                O[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Vf, Pf, O[db], 0, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // V(b) is read
        if (more) request(v, v_off, Vs, b + KW);
    }

    // The results of the waves that had a block meet: 16-byte unit u = 4 db + rg of lane (j, h) is dims 8 u + 4 h .. + 3 of row j.
    constexpr int UNITS = 4 * DB, OWN = UNITS / KW;
    const int n_waves = min(KW, end - first);
    if (wave < n_waves) {
        l += __shfl_xor(l, 32);
        if (h == 0) stat[wave * 32 + j] = make_float2(m, l);
        f32x4* mine = reinterpret_cast<f32x4*>(Ks);  // this wave's stages: read, and nothing is in flight
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
                mine[(4 * db + rg) * kWave + lane] = f32x4{O[db][4 * rg], O[db][4 * rg + 1], O[db][4 * rg + 2], O[db][4 * rg + 3]};
    }
    __syncthreads();
    float a[KW], M = -INFINITY, L = 0.f;
    f32x4 t[OWN];
#pragma unroll
    for (int i = 0; i < OWN; ++i) t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < KW; ++w)
        if (w < n_waves) M = fmaxf(M, stat[w * 32 + j].x);
    const float ref = PARTS && M == -INFINITY ? 0.f : M;  // no finite score in this part: sums of 0
    const f32x4* all = reinterpret_cast<const f32x4*>(Qs + SM::kStage);
#pragma unroll
    for (int w = 0; w < KW; ++w)
        if (w < n_waves) {
            const float2 s = stat[w * 32 + j];
            a[w] = __builtin_amdgcn_exp2f(s.x - ref);
            L = fmaf(a[w], s.y, L);
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                const f32x4 x = all[(w * UNITS + wave * OWN + i) * kWave + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) t[i][e] = fmaf(a[w], x[e], t[i][e]);
            }
        }
    if (row0 + j >= n) return;
    if constexpr (PARTS) {
        const size_t rows = n - row_base, item = ((size_t)blockIdx.y * rows + (row - row_base)) * Hq + head;
#pragma unroll
        for (int i = 0; i < OWN; ++i) *reinterpret_cast<f32x4*>(sums + item * DH + 8 * (wave * OWN + i) + 4 * h) = t[i];
        if (wave == 0 && h == 0) reinterpret_cast<float2*>(sums + (size_t)gridDim.y * rows * Hq * DH)[item] = make_float2(M, L);
        return;
    }
    const float inv = 1.0f / L;
    __bf16* op = o + ((size_t)row * Hq + head) * DH + 4 * h;
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        bf16x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(t[i][e] * inv);
        *reinterpret_cast<bf16x4*>(op + 8 * (wave * OWN + i)) = ov;
    }
}

// Adds the parts of each row and head, in their order; a thread has four dims.
__global__ __launch_bounds__(256) void few_parts_kernel(const float* __restrict__ sums, int parts, int items, int DH, __bf16* __restrict__ o) {
    const int u = blockIdx.x * 256 + threadIdx.x, item = u / (DH / 4);
    if (item >= items) return;
    const float2* stat = reinterpret_cast<const float2*>(sums + (size_t)parts * items * DH) + item;
    const float* src = sums + (size_t)u * 4;
    float M = -INFINITY, L = 0.f;
    for (int p = 0; p < parts; ++p) M = fmaxf(M, stat[(size_t)p * items].x);
    f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int p = 0; p < parts; ++p) {
        const float2 s = stat[(size_t)p * items];
        const f32x4 x = *reinterpret_cast<const f32x4*>(src + (size_t)p * items * DH);
        const float a = __builtin_amdgcn_exp2f(s.x - M);
        L = fmaf(a, s.y, L);
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = fmaf(a, x[e], t[e]);
    }
    const float inv = 1.0f / L;
    bf16x4 ov;
#pragma unroll
    for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(t[e] * inv);
    *reinterpret_cast<bf16x4*>(o + (size_t)u * 4) = ov;
}

template <int DH, int KW, bool PARTS = false>
static hipError_t set_few_lds_size() {
    return hipFuncSetAttribute((const void*)flash_few<DH, KW, PARTS>, hipFuncAttributeMaxDynamicSharedMemorySize, FewSmem<DH>::bytes(KW));
}

dash_status init_few_kernels() {
    static const hipError_t err = [] {
        hipError_t e = set_few_lds_size<64, 4>();
        if (e == hipSuccess) e = set_few_lds_size<64, 8>();
        if (e == hipSuccess) e = set_few_lds_size<128, 4>();
        if (e == hipSuccess) e = set_few_lds_size<128, 8>();
        if (e == hipSuccess) e = set_few_lds_size<64, 8, true>();
        if (e == hipSuccess) e = set_few_lds_size<128, 8, true>();
        return e;
    }();
    return err == hipSuccess ? DASH_OK : DASH_ERR_HIP;
}

template <int DH, int KW>
static void launch_few(const dash_layer_params& p, const __bf16* q, const __bf16* k, const __bf16* v, const int32_t* pos, int n,
                       int row0, __bf16* o, float scale_log2, uint32_t* clear_words, int n_clear, int32_t* clear_count, hipStream_t s) {
    const int n_qtiles = (n - row0 + 31) / 32;
    unsigned blocks = 0;
    const FaMap mp = fa_map(n_qtiles, p.n_q_heads, p.n_kv_heads, blocks);
    hipLaunchKernelGGL((flash_few<DH, KW, false>), dim3(blocks), dim3(KW * kWave), FewSmem<DH>::bytes(KW), s, q, k, v, pos, o, n,
                       p.n_q_heads, p.n_kv_heads, scale_log2, p.causal, n_qtiles, mp, clear_words, n_clear, row0, clear_count, nullptr, 0);
}
template <int DH>
static void launch_few_parts(const dash_layer_params& p, const __bf16* q, const __bf16* k, const __bf16* v, const int32_t* pos, int n,
                             int row0, __bf16* o, float scale_log2, const FewParts& g, float* sums, hipStream_t s) {
    constexpr int KW = kFewTailWaves;
    const int n_qtiles = (n - row0 + 31) / 32, Hq = p.n_q_heads, items = (n - row0) * Hq;
    unsigned blocks = 0;
    const FaMap mp = fa_map(n_qtiles, Hq, p.n_kv_heads, blocks);
    hipLaunchKernelGGL((flash_few<DH, KW, true>), dim3(blocks, g.parts), dim3(KW * kWave), FewSmem<DH>::bytes(KW), s, q, k, v, pos, o, n, Hq,
                       p.n_kv_heads, scale_log2, p.causal, n_qtiles, mp, nullptr, 0, row0, nullptr, sums, g.blocks_per_part);
    hipLaunchKernelGGL(few_parts_kernel, dim3((items * (DH / 4) + 255) / 256), dim3(256), 0, s, sums, g.parts, items, DH, o + (size_t)row0 * Hq * DH);
}

// The rows beyond the last whole tile, without a causal mask, their keys cut into parts (few_tail_parts).
dash_status launch_flash_few_parts(const dash_layer_params& p, const __bf16* q, const __bf16* k, const __bf16* v, const int32_t* pos, int n,
                                   int row0, __bf16* o, float scale_log2, const FewParts& g, float* sums, hipStream_t s) {
    if (init_few_kernels() != DASH_OK) return DASH_ERR_HIP;
    (p.head_dim == 64 ? launch_few_parts<64> : launch_few_parts<128>)(p, q, k, v, pos, n, row0, o, scale_log2, g, sums, s);
    return launch_status();
}

// Query rows [row0, n), row0 a multiple of 32, against all keys. waves: 4 or 8 (few_waves, staging_addr.h)
dash_status launch_flash_few(const dash_layer_params& p, const __bf16* q, const __bf16* k, const __bf16* v,
                             const int32_t* pos, int n, int row0, __bf16* o, float scale_log2, int waves, uint32_t* clear_words,
                             int n_clear, int32_t* clear_count, hipStream_t s) {
    if (init_few_kernels() != DASH_OK) return DASH_ERR_HIP;
    if (p.head_dim == 64)
        (waves == 8 ? launch_few<64, 8> : launch_few<64, 4>)(p, q, k, v, pos, n, row0, o, scale_log2, clear_words, n_clear, clear_count, s);
    else
        (waves == 8 ? launch_few<128, 8> : launch_few<128, 4>)(p, q, k, v, pos, n, row0, o, scale_log2, clear_words, n_clear, clear_count, s);
    return launch_status();
}

}  // namespace dash
