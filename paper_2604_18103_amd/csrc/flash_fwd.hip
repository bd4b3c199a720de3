// Causal grouped-query attention forward over the compacted active rows (Attn of Eq. 1, before the
// output projection). Tiled online-softmax: the probability matrix is never written to HBM, which is
// the property the paper needs from its attention operator (no attention matrix is materialised).
//
// Causality is defined on ORIGINAL positions (active_idx). Because active_idx is strictly increasing,
// "position of key <= position of query" equals "rank of key <= rank of query"; whole tiles are
// skipped by rank and the elements of diagonal tiles are masked by comparing positions.
//
// Kernels:
//   flash_fwd_mfma<DH, KG> bf16, MFMA 32x32x16, fp32 softmax and accumulation (the hot kernel); few rows: flash_few.hip
//   flash_fwd_f32<DH> fp32, MFMA 16x16x4 fp32, keys split over the waves of a workgroup
#include "common.h"
#include "flash_map.h"
#include "lds_ops.h"
#include "staging_addr.h"

namespace dash {

// ------------------------------------------------------------------------------------------------
// fp32 kernel: v_mfma_f32_16x16x4_f32 (fp32 operands, products and sums), exact expf.
//
// A workgroup owns 16 query rows of one head; its 8 waves split the KEYS (wave w takes the 32-key blocks w, w + 8,
// ...) and meet once, at the end, in LDS. The prompts of this path are short (hundreds to a few thousand rows): with a
// wave per query row and all of its keys in series the kernel waited for memory and for its own chain of adds. Splitting
// the keys makes that chain eight times shorter and needs no barrier inside the loop.
//
// S^T = K Q^T, then O^T += V^T P^T: in the 16x16 accumulator layout (lane 16 g + i: rows 4 g .. 4 g + 3 of column i) lane
// (i, g) holds the scores of query i for keys 4 g + r, and taking key 4 g + r as k-slot g of step r makes those registers
// the B operand of the second product as they are. The contraction of the first product and the dims of the second are
// numbered so that every operand is a 16-byte global load: step s of dim chunk c contracts dims 16 c + 4 g + s, and
// output block (hf, e) holds dims 64 hf + 4 i + e. No LDS in the loop: K and V come from the L2.
//
// Bound by latency at a few hundred rows, by the fp32 matrix rate and the L2 from a few thousand on. Measured, causal, 4 / 1
// heads of 64: n = 512 12 us, 2048 39 us, 8192 451 us (a wave per row and head: 72, 409, 5378 us); 4 / 2 heads of 128: 19,
// 70, 868 us (96, 809, 11795 us). Error against 64 bits 2.2e-7 instead of 2.7e-7 at 512, 3.2e-7 instead of 6.3e-7 at 8192.
// Two 16-row blocks per wave, which read K and V half as often, were 10 % faster from 4096 rows on, 40 % slower at 2048
// and less, and spill at head_dim 128.
// ------------------------------------------------------------------------------------------------
constexpr int kF32Waves = 8;
constexpr int kF32Keys = 32;  // keys per wave and step

template <int DH>
__global__ __launch_bounds__(kF32Waves * kWave) void flash_fwd_f32(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    const int32_t* __restrict__ pos, float* __restrict__ o, int n, int Hq, int Hkv, float scale, int causal, int n_qtiles,
    uint32_t* __restrict__ clear_words, int n_clear, int32_t* __restrict__ clear_count) {
    constexpr int KC = DH / 16, HF = DH / 64, OSTR = DH + 4;
    __shared__ float part_o[kF32Waves][16][OSTR];
    __shared__ float part_m[kF32Waves][16], part_l[kF32Waves][16];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    if (blockIdx.x == 0)  // scratch of the kernels that follow in the layer call
        for (int c = tid; c <= n_clear; c += kF32Waves * kWave) {
            if (c < n_clear) clear_words[c] = 0u;
            else if (clear_count) *clear_count = 0;
        }
    const int qt = n_qtiles - 1 - (int)blockIdx.x / Hq, head = (int)blockIdx.x % Hq;  // longest rows first
    const int kvh = head / (Hq / Hkv);
    const int i = lane % 16, g = lane / 16;
    const int row0 = qt * 16;
    const size_t kv_stride = (size_t)Hkv * DH;
    const float* kh = k + (size_t)kvh * DH;
    const float* vh = v + (size_t)kvh * DH;

    f32x4 Qf[KC], O[HF * 4];
    float m = -INFINITY, l = 0.f;
    const int row = min(row0 + i, n - 1);
    {
        const float* qp = q + ((size_t)row * Hq + head) * DH + 4 * g;
#pragma unroll
        for (int c = 0; c < KC; ++c) Qf[c] = *reinterpret_cast<const f32x4*>(qp + 16 * c);
#pragma unroll
        for (int d = 0; d < HF * 4; ++d) O[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int pos_q = pos[row];
    const int kend = causal ? min(n, row0 + 16) : n;
    // Only the last block of keys is masked. The positions that its masks compare are asked for here: inside the loop they were one
    // more trip to memory, behind the scores (4 / 2 heads of 128, 63 rows 7.7 -> 7.2 us; 16 of 64, 257 rows 10.7 -> 9.7; 28 of
    // 128, 333 rows 28.4 -> 26.9).
    int pos_k[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) pos_k[e] = pos[min((kend - 1) / kF32Keys * kF32Keys + 16 * (e / 4) + 4 * g + e % 4, n - 1)];
    for (int key0 = wave * kF32Keys; key0 < kend; key0 += kF32Waves * kF32Keys) {
        f32x4 S[2];
        f32x4 Vf[2][4][HF];
        {
            f32x4 Kf[2][KC];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const float* kp = kh + (size_t)min(key0 + 16 * kb + i, n - 1) * kv_stride + 4 * g;
#pragma unroll
                for (int c = 0; c < KC; ++c) Kf[kb][c] = *reinterpret_cast<const f32x4*>(kp + 16 * c);
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float* vp = vh + (size_t)min(key0 + 16 * kb + 4 * g + r, n - 1) * kv_stride + 4 * i;
#pragma unroll
                    for (int hf = 0; hf < HF; ++hf) Vf[kb][r][hf] = *reinterpret_cast<const f32x4*>(vp + 64 * hf);
                }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) S[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < KC; ++c)
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
                        S[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(Kf[kb][c][s], Qf[c][s], S[kb], 0, 0, 0);
        }
        // the block that ends beyond the first row's key, or beyond the last key (the last one): -inf where a key is not visible
        const bool masked = (causal && key0 + kF32Keys - 1 > row0) || key0 + kF32Keys > n;
        uint32_t seen = 0xFFu;  // bit 4 kb + r: the key is visible to this lane's query
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) S[kb] *= scale;
        if (masked) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int key = key0 + 16 * kb + 4 * g + r;
                    if (key >= n || (causal && (key > row0 + i || pos_k[4 * kb + r] > pos_q))) {
                        seen &= ~(1u << (4 * kb + r));
                        S[kb][r] = -INFINITY;
                    }
                }
        }
        {
            float mx = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, S[kb][r]);
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx);
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // nothing visible to this query yet
            const float alpha = expf(m - m_ref);
            m = m_new;
            float ps = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    S[kb][r] = (seen >> (4 * kb + r)) & 1u ? expf(S[kb][r] - m_ref) : 0.f;
                    ps += S[kb][r];
                }
            l = l * alpha + ps;
#pragma unroll
            for (int d = 0; d < HF * 4; ++d) O[d] *= alpha;
        }
        // A key that a query does not see has probability 0, but 0 times an infinite or NaN value is NaN: such a block
        // is added key by key, reading only what is visible. (Wave-uniform, never taken on finite values.)
        bool odd = false;
        if (masked) {
            float t = 0.f;  // stays 0 unless some value is not finite
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int hf = 0; hf < HF; ++hf)
#pragma unroll
                        for (int e = 0; e < 4; ++e) t = fmaf(Vf[kb][r][hf][e], 0.f, t);
            odd = __any(t != 0.f);  // NaN != 0
        }
        if (!odd) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int hf = 0; hf < HF; ++hf)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            O[4 * hf + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(Vf[kb][r][hf][e], S[kb][r], O[4 * hf + e], 0, 0, 0);
        } else {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll 1
                    for (int gg = 0; gg < 4; ++gg) {
                        const float* vp = vh + (size_t)min(key0 + 16 * kb + 4 * gg + r, n - 1) * kv_stride + 16 * g;
                        const float p = __shfl(S[kb][r], 16 * gg + i);
                        const uint32_t sees = __shfl(seen, 16 * gg + i);
                        if ((sees >> (4 * kb + r)) & 1u)
#pragma unroll
                            for (int hf = 0; hf < HF; ++hf)
#pragma unroll
                                for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                                    for (int e = 0; e < 4; ++e)
                                        O[4 * hf + e][rr] = fmaf(p, vp[64 * hf + 4 * rr + e], O[4 * hf + e][rr]);
                    }
        }
    }
    // the eight partial results of each query meet: O = sum_w e^(m_w - M) O_w / sum_w e^(m_w - M) l_w, in the order of w
    float lt = l;
    lt += __shfl_xor(lt, 16);
    lt += __shfl_xor(lt, 32);
    if (g == 0) {
        part_m[wave][i] = m;
        part_l[wave][i] = lt;
    }
    // block (hf, e), register rr: dim 64 hf + 4 (4 g + rr) + e
#pragma unroll
    for (int hf = 0; hf < HF; ++hf)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
            *reinterpret_cast<f32x4*>(&part_o[wave][i][64 * hf + 16 * g + 4 * rr]) =
                f32x4{O[4 * hf][rr], O[4 * hf + 1][rr], O[4 * hf + 2][rr], O[4 * hf + 3][rr]};
    __syncthreads();
    constexpr int PER = 16 * DH / (kF32Waves * kWave);  // dims per thread: 2 or 4
    const int qi = tid / (DH / PER), d0 = (tid % (DH / PER)) * PER;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) M = fmaxf(M, part_m[w][qi]);
    float L = 0.f, acc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
        const float lw = part_l[w][qi];
        if (lw == 0.f) continue;  // this wave saw no key of the query
        const float f = expf(part_m[w][qi] - M);
        L = fmaf(f, lw, L);
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] = fmaf(f, part_o[w][qi][d0 + e], acc[e]);
    }
    if (row0 + qi < n) {
        float* op = o + ((size_t)(row0 + qi) * Hq + head) * DH + d0;
#pragma unroll
        for (int e = 0; e < PER; ++e) op[e] = acc[e] / L;
    }
}

// ------------------------------------------------------------------------------------------------
// MFMA kernel.
//
// Workgroup = 8 waves = 256 query rows of one head; wave w owns rows 32w..32w+31. Keys/values come in
// tiles of 64, staged through LDS in their natural [key][dim] layout (16-byte chunks swizzled). (KG = 2, for short
// sequences: 128 rows; waves w and w + 4 own the same rows and take every other key tile, see the launcher.)
//
//   S^T = K Q^T   (A = K fragment from LDS, B = Q fragment held in registers for the whole kernel):
//         with the 32x32 accumulator layout each lane then holds 16 scores of ONE query per 32-key
//         block, so row max / row sum are in-lane reductions plus one exchange with lane^32.
//   O^T += V^T P^T (A = V^T fragment via LDS transpose reads, B = P^T): the accumulator registers of
//         S^T, converted to bf16, already ARE the B fragment - no shuffle, no LDS round trip.
//
// A wave that runs MFMAs and softmax back to back leaves each pipe idle half the time. So the eight waves
// form two groups (waves 0-3 and 4-7; wave w and w+4 share a SIMD) that run the same loop body - an MFMA
// stretch (O += P V of the previous tile, then S = K Q^T of the next) followed by the softmax of that tile -
// but pass the one workgroup barrier of a round at different places, so that between two barriers
//     group 0 runs  MFMA stretch(t), softmax(t)        group 1 runs  softmax(t-1), MFMA stretch(t)
// and the SIMD co-executes one group's MFMAs with the other group's VALU work.
// K and V tiles go from global memory straight into LDS (no registers in between), K through two stages and
// V through three; the V fragments of a tile's first key chunk are read during the softmax phase, so the
// matrix-core phase that follows the barrier starts with MFMAs, not with an exposed LDS round trip.
//
// MFMA 32x32x16 operand layout (lane l, i = l%32, h = l/32): A holds row i, k-slots 8h..8h+7;
// B holds column i, k-slots 8h..8h+7; D register r holds row 8*(r/4) + 4h + r%4 of column i.
// ------------------------------------------------------------------------------------------------
// query rows per workgroup: kFaBM = 256, keys per tile: kFaBN = 64 (staging_addr.h)
constexpr int kFaThreads = 512;
constexpr float kMaskedScore = -1.0e30f;
// 2^20 as a float: a lane's 32-key partial row sum above this moves the softmax reference
constexpr int kRowSumLimitBits = 0x49800000;

// LDS layout of one K or V stage: 64 rows of DH bf16, unpadded (the direct global->LDS loads write 1 KB of
// consecutive LDS per wave instruction, so rows cannot be padded). Bank conflicts are avoided by an XOR
// swizzle of the 16-byte chunk index inside each row, different for K and V because they are read
// differently: K by 16-byte reads of one chunk from 16 consecutive rows, V by transpose reads that touch
// 4 consecutive rows x 4 consecutive chunks per 32 lanes.
template <int DH>
struct FaSmem {
    static constexpr int CPR = DH / 8;             // 16-byte chunks per row
    static constexpr int RP = 256 / (DH * 2);      // rows per 256 bytes of LDS (one pass over all banks)
    static constexpr int STAGE_ELEMS = kFaBN * DH;
    // one key group: two stages of K, three of V; two key groups: two of each for either group
    static constexpr size_t bytes(int KG) { return (KG == 1 ? 5 : 8) * STAGE_ELEMS * sizeof(__bf16); }
    // the result rows of 8 waves, and with two key groups the halves they exchange before that, take the stages' place
    static_assert(bytes(1) >= 8 * 32 * (DH + 8) * sizeof(__bf16), "result rows fit");
    static_assert(bytes(2) >= 32 * DH * 16 + 2048 + 8 * 32 * (DH / 2 + 8) * sizeof(__bf16), "exchange and result rows fit");
    __device__ static constexpr int k_swz(int row) { return fa_k_swz(row, DH); }
    __device__ static constexpr int v_swz(int row) { return fa_v_swz(row, DH); }
};


// Where the key loop lies in the code. The loop body is branches and short stretches between them, two waves per SIMD are
// fetched from one instruction cache, and what a taken branch costs depends on where its target lies in a 32-byte fetch: the
// same instructions shifted by 4 bytes at a time take from 0.98 to 1.10 times as long at head size 64 with one key group
// (4097 to 12001 rows), up to 1.03 with two. So the loop starts at a stated distance from a 64-byte line (no-ops before
// it), and so does what follows the rarely taken branch of the softmax (no-ops at its end). Steps of 4 bytes, measured; to be
// measured again when the loop changes.
constexpr int fa_loop_pad(int DH, int KG) { return KG == 2 ? (DH == 64 ? 10 : 4) : (DH == 64 ? 6 : 1); }
constexpr int fa_branch_pad(int DH, int KG) { return DH == 64 && KG == 1 ? 3 : 4; }

// A wave's 32 result rows of W elements go out through LDS (rows of W + 8 elements, written 8 bytes per lane as the
// accumulators lie): a store instruction then covers whole rows instead of 8-byte pieces of 32 of them.
__device__ constexpr int out_row(int W) { return W + 8; }
template <int W>
__device__ __forceinline__ void store_rows(const __bf16* rows, int lane, int q0, int n, __bf16* o, size_t stride) {
    constexpr int LPR = W / 8, RPI = kWave / LPR;  // lanes per row, rows per instruction
    wave_sync_lds();
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += RPI) {
        const int r = r0 + lane / LPR, c = 8 * (lane % LPR);
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(rows + r * out_row(W) + c);
        if (q0 + r < n) *reinterpret_cast<bf16x8*>(o + (size_t)(q0 + r) * stride + c) = v;
    }
}

template <int DH, int KG>
__global__ __launch_bounds__(kFaThreads, 1) void flash_fwd_mfma(const __bf16* __restrict__ q,
                                                                const __bf16* __restrict__ k,
                                                                const __bf16* __restrict__ v,
                                                                const int32_t* __restrict__ pos,
                                                                __bf16* __restrict__ o, int n, int Hq,
                                                                int Hkv, float scale_log2, int causal,
                                                                int n_qtiles, FaMap mp,
                                                                uint32_t* __restrict__ clear_words, int n_clear,
                                                                int row_base, int32_t* __restrict__ clear_count) {
    using SM = FaSmem<DH>;
    constexpr int KC = DH / 16;  // contraction chunks of Q K^T
    constexpr int DB = DH / 32;  // 32-wide output blocks of O^T
    constexpr int BM = kFaBM / KG;            // query rows of the workgroup
    constexpr int V_STAGES = KG == 1 ? 3 : 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char fa_smem_raw[];
    __shared__ __attribute__((aligned(16))) int pos_blk[BM];  // original positions of this workgroup's rows

    if (blockIdx.x == 0)  // scratch of the kernels that follow in the layer call: cleared here, no launch of its own
        for (int c = threadIdx.x; c <= n_clear; c += kFaThreads) {
            if (c < n_clear) clear_words[c] = 0u;
            else if (clear_count) *clear_count = 0;
        }
    int qt, head;
    if (!fa_map_block(mp, (int)blockIdx.x, n_qtiles, Hq, Hkv, qt, head)) return;  // whole workgroup exits
    const int g = head / (Hq / Hkv);
    const int tid = threadIdx.x, lane = tid % kWave;
    // the wave index is made provably uniform: the role branches below must be scalar branches, never
    // exec-masked regions (MFMA ignores the exec mask)
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int grp = wave >> 2;
    // two K stages, then the V stages; with two key groups either group has its own
    __bf16* Kst = reinterpret_cast<__bf16*>(fa_smem_raw) + (KG == 1 ? 0 : grp * 4 * SM::STAGE_ELEMS);
    __bf16* Vst = Kst + 2 * SM::STAGE_ELEMS;
    const int j = lane % 32, h = lane / 32;
    const int tg = lane / 16, ti = lane % 16;
    const int tile_row0 = (KG == 1 ? 0 : row_base) + qt * BM;  // this workgroup's first query row
    const int q0 = tile_row0 + (KG == 1 ? wave : wave & 3) * 32;
    const int qrow = q0 + j;
    const int qrow_c = min(qrow, n - 1);
    const int pos_q = pos[qrow_c];

    bf16x8 Qf[KC];
    {
        const __bf16* qp = q + ((size_t)qrow_c * Hq + head) * DH + 8 * h;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) Qf[kc] = *reinterpret_cast<const bf16x8*>(qp + 16 * kc);
        // Q is scaled once by softmax_scale * log2(e) (rounded to bf16 again), so the MFMA result is already the
        // exponent in the log2 domain. Rounding the scaled row r = bf16(x) changes its length along x by the
        // factor <r, x> / <x, x>, which acts on every logit of the row like a change of the softmax temperature
        // and, for a fixed scale constant, has a common sign for most rows (measured: 3e-4 of systematic relative
        // error in ||delta||). The row is therefore rounded a second time from x scaled by the inverse of that
        // factor, which cancels the systematic part; what is left is the random part of one rounding.
        // Head size 128: the two sums are taken over bf16 pairs (fp32 products and sums): with q the unscaled row and s the
        // scale, <x, x> = s^2 <q, q> and <r, x> = s <r, q>. A third of the prologue's instructions less: 1 % at 4096 rows. At
        // head size 64 the same text leaves the compiler a main loop that is 3 % slower, so it keeps the plain form.
        if constexpr (DH == 128) {
            float qq = 0.f, rq = 0.f;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const bf16x2 qp2 = {Qf[kc][e], Qf[kc][e + 1]};
                    const bf16x2 r2 = {(__bf16)((float)Qf[kc][e] * scale_log2), (__bf16)((float)Qf[kc][e + 1] * scale_log2)};
                    qq = __builtin_amdgcn_fdot2_f32_bf16(qp2, qp2, qq, false);
                    rq = __builtin_amdgcn_fdot2_f32_bf16(r2, qp2, rq, false);
                }
            qq += __shfl_xor(qq, 32);  // lanes j and j + 32 hold the two halves of the row
            rq += __shfl_xor(rq, 32);
            const float sqq = qq * scale_log2;
            // 1 / (1 + a) to first order, a = rq / sqq - 1 (rows of zeros, or too long to measure: 1), and the scale itself
            const float scale_comp = (sqq > 0.f && sqq < INFINITY ? 2.0f - rq / sqq : 1.0f) * scale_log2;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int e = 0; e < 8; ++e) Qf[kc][e] = (__bf16)((float)Qf[kc][e] * scale_comp);
        } else {
            float xs[KC][8];
            float sxx = 0.f, srx = 0.f;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = (float)Qf[kc][e] * scale_log2;
                    xs[kc][e] = x;
                    sxx = fmaf(x, x, sxx);
                    srx = fmaf((float)(__bf16)x, x, srx);
                }
            sxx += __shfl_xor(sxx, 32);  // lanes j and j + 32 hold the two halves of the row
            srx += __shfl_xor(srx, 32);
            const float comp = sxx > 0.f ? 2.0f - srx / sxx : 1.0f;  // 1 / (1 + a) to first order, a = srx / sxx - 1
#pragma unroll
            for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                for (int e = 0; e < 8; ++e) Qf[kc][e] = (__bf16)(xs[kc][e] * comp);
        }
    }
    f32x16 Oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) Oacc[db][r] = 0.f;
    f32x16 S[2];
    uint32_t Pw[4][4];  // P^T of the previous tile as packed bf16 pairs: Pw[c] is the B fragment of key chunk c
    // m is the softmax reference (log2 domain); Cneg holds -m in all 16 accumulator slots and is what every
    // score accumulation starts from, so S arrives as (score - m) and the common tile needs no subtraction.
    // It changes only when the reference moves; the empty asm keeps it a register block instead of 16
    // re-materialised moves per tile.
    float m = 0.f, lsum = 0.f;
    int sum_limit = kRowSumLimitBits;  // wave-uniform; -1 (a NaN: no sum lies below it) while some row waits for a key that counts
    f32x16 Cneg;
#pragma unroll
    for (int r = 0; r < 16; ++r) Cneg[r] = 0.f;
    asm volatile("" : "+v"(Cneg));

    const int kv_end = causal ? min(n, tile_row0 + BM) : n;
    const int all_tiles = (kv_end + kFaBN - 1) / kFaBN;
    // tile t of this wave is key tile t, or, with two key groups, key tile 2 t + grp
    const int n_tiles = KG == 1 ? all_tiles : fa_group_tiles(all_tiles, grp);
    const int n_rounds = KG == 1 ? all_tiles : (all_tiles + 1) / 2;
    auto first_key = [&](int t) { return fa_first_key(t, grp, KG); };
    // keys at or beyond this rank are masked for the whole wave; a wave whose rows all lie beyond the end does nothing
    const int wave_kend = q0 >= n ? 0 : (causal ? min(n, q0 + 32) : n);

    // Staging by direct global->LDS loads, no registers in between: the four waves of group 0 fetch the K
    // tiles, those of group 1 the V tiles. One wave instruction moves 1 KB = ROWS_PER_DMA rows; lane l
    // lands in physical chunk l % CPR of row l / CPR, so it fetches the logical chunk that the swizzle maps
    // there. The address of a load is a scalar tile base (advanced by scalar arithmetic) plus a 32-bit lane offset
    // that is the same for every whole tile (the launcher checks the tensors are below 2 GiB); only the last,
    // partly filled tile recomputes the offsets, with rows beyond the end clamped to the last row.
    constexpr int DMAS = fa_dmas(DH);                           // loads per wave and tile: 4 (DH 128) or 2 (DH 64)
    const int gw = wave & 3;                                    // wave inside its group
    const uint32_t tile_bytes = (uint32_t)fa_tile_bytes(Hkv, DH);
    // byte offset of this lane's 16 bytes from the start of a whole tile: this group's operand (one key group), or K and
    // V (two key groups, either of which fetches its own tiles)
    uint32_t dma_voff[KG][DMAS];
#pragma unroll
    for (int i = 0; i < DMAS; ++i) {
        dma_voff[0][i] = fa_dma_voff(fa_dma_row(gw, i, lane, DH), lane, g, Hkv, DH, KG == 2 || grp == 0);
        if (KG == 2) dma_voff[KG - 1][i] = fa_dma_voff(fa_dma_row(gw, i, lane, DH), lane, g, Hkv, DH, false);
    }
    auto fetch_tile = [&](const char* base, const uint32_t* voff, uint32_t lds, int key0) {
        const char* tile_base = base + (size_t)(key0 / kFaBN) * tile_bytes;
        const int rows_left = n - key0;  // >= 1: only tiles that hold a row are fetched
        if (rows_left >= kFaBN) {
#pragma unroll
            for (int i = 0; i < DMAS; ++i) dma_load16(tile_base, voff[i], lds + (uint32_t)(i * 1024));
        } else {
#pragma unroll
            for (int i = 0; i < DMAS; ++i)
                dma_load16(tile_base, fa_dma_voff_tail(voff[i], fa_dma_row(gw, i, lane, DH), rows_left, Hkv, DH),
                           lds + (uint32_t)(i * 1024));
        }
    };
    // one key group: tiles of this group's operand are fetched strictly in order: 0, 1, 2, ...
    const char* dma_base = reinterpret_cast<const char*>(grp == 0 ? k : v);
    const uint32_t lds_stage0 = lds_addr(KG == 2 || grp == 0 ? Kst : Vst) + (uint32_t)(gw * DMAS * 1024);
    int dma_tile = 0;
    auto dma_next_tile = [&](int stage) {
        fetch_tile(dma_base, dma_voff[0], lds_stage0 + (uint32_t)(stage * SM::STAGE_ELEMS * 2), dma_tile++ * kFaBN);
    };
    // two key groups: K or V of this group's tile t
    auto fetch_k = [&](int t) {
        fetch_tile(reinterpret_cast<const char*>(k), dma_voff[0], lds_stage0 + (uint32_t)((t & 1) * SM::STAGE_ELEMS * 2),
                   first_key(t));
    };
    auto fetch_v = [&](int t) {
        fetch_tile(reinterpret_cast<const char*>(v), dma_voff[KG - 1],
                   lds_stage0 + (uint32_t)((2 + (t & 1)) * SM::STAGE_ELEMS * 2), first_key(t));
    };

    // A fragment of O^T += V^T P^T: V^T block (32 dims of block db) x (16 keys of chunk c) by transpose reads
    auto v_frag = [&](const __bf16* Vs, int c, int db) {
        const int kbase_row = 16 * c + 4 * (tg / 2) + ti / 4;  // key row this lane addresses
        const int col = 32 * db + 16 * (tg % 2) + 4 * (ti % 4);
        // rows kbase_row and kbase_row + 8 have the same swizzle (it repeats every 4 * RP <= 8 rows)
        const int scol = ((col / 8) ^ SM::v_swz(kbase_row)) * 8 + col % 8;
        const s16x4 lo = lds_read_tr16(&Vs[kbase_row * DH + scol]);
        const s16x4 hi = lds_read_tr16(&Vs[(kbase_row + 8) * DH + scol]);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // The fragments of key chunk 0 are read during the softmax phase, before the barrier that opens the
    // matrix-core phase, so that phase starts with MFMAs instead of an exposed LDS round trip.
    bf16x8 Vpre[DB];
    auto prefetch_v = [&](int t) {
        const __bf16* Vs = Vst + (t % V_STAGES) * SM::STAGE_ELEMS;
#pragma unroll
        for (int db = 0; db < DB; ++db) Vpre[db] = v_frag(Vs, 0, db);
    };
    // O^T += V^T(t) P^T(t): A = V^T fragment, B = packed P
    auto pv_mfma = [&](int t) {
        const __bf16* Vs = Vst + (t % V_STAGES) * SM::STAGE_ELEMS;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const u32x4 pw = {Pw[c][0], Pw[c][1], Pw[c][2], Pw[c][3]};
            const bf16x8 Pf = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
            for (int db = 0; db < DB; ++db)
                Oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c == 0 ? Vpre[db] : v_frag(Vs, c, db), Pf,
                                                                   Oacc[db], 0, 0, 0);
        }
        // issue order: operand reads run DB MFMAs ahead, so no MFMA waits for a read issued just before it
        constexpr int NM = 4 * DB;
#pragma unroll
        for (int i = 0; i < NM - DB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, DB, 0);
    };
    // S^T = K(t) Q^T. A fragment: key row 32 kb + j, chunk 2 kc + h; rows j and 32 + j swizzle alike, so the key
    // block only adds a constant to the element offset k_elem[kc].
    static_assert((32 / SM::RP) % SM::CPR == 0, "rows j and j + 32 must share the K swizzle");
    int k_elem[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) k_elem[kc] = j * DH + ((2 * kc + h) ^ SM::k_swz(j)) * 8;
    auto qk_mfma = [&](int t) {
        const __bf16* Ks = Kst + (t & 1) * SM::STAGE_ELEMS;
        // the two key blocks take turns, so that no MFMA accumulates into the result of the one issued just before it
        // (eight in a row on one block measured 0.6 % slower)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) S[kb][r] = Cneg[r];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const bf16x8 Kf = *reinterpret_cast<const bf16x8*>(&Ks[k_elem[kc] + 32 * kb * DH]);
                S[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Kf, Qf[kc], S[kb], 0, 0, 0);
            }
        constexpr int NM = 2 * KC;
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < NM - 4; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    };
    auto tile_active = [&](int t) { return t >= 0 && t < n_tiles && first_key(t) < wave_kend; };  // wave-uniform

    // matrix-core phase of tile t: finish the previous tile's P V, start this tile's scores
    auto mfma_phase = [&](int t) {
        // While a wave is in its matrix-core phase it gets issue priority over the wave of the other group
        // on the same SIMD: an MFMA is issued as soon as the pipe frees, VALU work fills the gaps.
        __builtin_amdgcn_s_setprio(3);
        if (tile_active(t - 1)) {
            if (KG == 2) prefetch_v(t - 1);
            pv_mfma(t - 1);
        }
        if (tile_active(t)) qk_mfma(t);
        __builtin_amdgcn_s_setprio(0);
    };
    // probabilities of the tile from S = score - m (minus `shift` when the reference has just moved), packed
    // to bf16 pairs into Pw; returns this lane's part of the row sum. fp32 adds on four chains: a bf16 dot2
    // would halve the instruction count, but it executes on the matrix pipe and (measured) serialises
    // with the other group's MFMAs.
    auto exp_pack = [&](bool shifted, float shift) {
        float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float p0 = __builtin_amdgcn_exp2f(shifted ? S[kb][r] - shift : S[kb][r]);
                const float p1 = __builtin_amdgcn_exp2f(shifted ? S[kb][r + 1] - shift : S[kb][r + 1]);
                ps[(r / 2) % 4] += p0;
                ps[(r / 2 + 2) % 4] += p1;
                const bf16x2 pk = {(__bf16)p0, (__bf16)p1};
                Pw[2 * kb + r / 8][(r % 8) / 2] = __builtin_bit_cast(uint32_t, pk);
            }
        return (ps[0] + ps[1]) + (ps[2] + ps[3]);
    };
    // VALU phase of tile t: softmax numerators in the log2 domain on S, leaves packed P in Pw
    auto valu_phase = [&](int t) {
        if (!tile_active(t)) return;
        const int key0 = first_key(t);
        // Causal masks are only ever needed on tiles that lie inside the workgroup's own row range, whose
        // original positions sit in LDS (pos_blk); masking compares positions, not ranks.
        const bool diag = causal && key0 + kFaBN - 1 > q0;  // wave-uniform
        if (diag || key0 + kFaBN > n) {
            const int kl0 = key0 - tile_row0;  // >= 0 whenever diag holds
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    const int kl = 32 * kb + 8 * rg + 4 * h;  // four consecutive keys of this lane
                    int4 kp = make_int4(0, 0, 0, 0);
                    if (diag) kp = *reinterpret_cast<const int4*>(&pos_blk[kl0 + kl]);
                    const int kpe[4] = {kp.x, kp.y, kp.z, kp.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool bad = (key0 + kl + e >= n) || (diag && kpe[e] > pos_q);
                        S[kb][4 * rg + e] = bad ? kMaskedScore : S[kb][4 * rg + e];
                    }
                }
        }
        // Probabilities are taken against a reference m that is NOT the running maximum: any reference
        // gives the same O / sum, it only has to keep exp2 in range. The common tile therefore computes
        // no row maximum at all: it exponentiates S (already relative to m) and looks at the row sums;
        // only if a sum is not a modest finite number (a score far above the reference), and always while a
        // row of the wave has no reference yet, the reference moves to the true running maximum, what was accumulated is
        // rescaled, and the tile's probabilities are redone.
        if (KG == 1) prefetch_v(t);
        float psum = exp_pack(false, 0.f);
        if (t == 0 || __any(!(psum < __builtin_bit_cast(float, sum_limit)))) {
            float c0 = fmaxf(S[0][0], S[1][0]), c1 = fmaxf(S[0][1], S[1][1]);
            float c2 = fmaxf(S[0][2], S[1][2]), c3 = fmaxf(S[0][3], S[1][3]);
#pragma unroll
            for (int r = 4; r < 16; r += 4) {
                c0 = fmaxf(fmaxf(c0, S[0][r]), S[1][r]);  // v_max3_f32
                c1 = fmaxf(fmaxf(c1, S[0][r + 1]), S[1][r + 1]);
                c2 = fmaxf(fmaxf(c2, S[0][r + 2]), S[1][r + 2]);
                c3 = fmaxf(fmaxf(c3, S[0][r + 3]), S[1][r + 3]);
            }
            float mx = fmaxf(fmaxf(c0, c1), fmaxf(c2, c3));  // tile maximum relative to m
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            // A row for which nothing has been accumulated takes the tile's maximum as its reference outright; later the
            // reference only rises. A tile may hold no key that counts for a row (every score -inf, or masked): the row
            // then keeps 0, adds nothing and waits for its next tile.
            const bool first = t == 0 || lsum + __shfl_xor(lsum, 32) == 0.f;
            const bool none = first && !(mx > 0.5f * kMaskedScore);
            const float shift = none ? 0.f : (first ? mx : fmaxf(mx, 0.f));
            const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(-shift);
            sum_limit = __builtin_amdgcn_readfirstlane(__any(none)) ? -1 : kRowSumLimitBits;
            m += shift;
#pragma unroll
            for (int r = 0; r < 16; ++r) Cneg[r] = -m;
            asm volatile("" : "+v"(Cneg));
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) Oacc[db][r] *= alpha;
            psum = exp_pack(true, shift);
            asm volatile(".rept %0\n\ts_nop 0\n\t.endr" : : "n"(fa_branch_pad(DH, KG)));
        }
        lsum += psum;
    };

    if (KG == 2) {
        // K(0) is waited for; group 1 has K(1) and V(0) in flight behind it
        if (n_tiles > 0) fetch_k(0);
        if (grp == 1 && n_tiles > 1) {
            fetch_k(1);
            fetch_v(0);
            dma_wait_keep<2 * DMAS>();
        } else {
            if (grp == 1 && n_tiles > 0) fetch_v(0);
            dma_wait();
        }
    } else {
        // K(0) by group 0; V(0) and V(1) by group 1, which waits for V(0) only
        dma_next_tile(0);
        if (grp == 1 && n_tiles > 1) {
            dma_next_tile(1);
            dma_wait_keep<DMAS>();
        } else {
            dma_wait();
        }
    }
    if (tid < BM) pos_blk[tid] = pos[min(tile_row0 + tid, n - 1)];
    // The Q fragments have to be in registers before the loop: if their loads were still in flight at
    // loop entry, the first MFMAs of every tile would also wait for the staging loads (issued later,
    // returned in order). An empty asm that "uses" them pins the wait here.
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) asm volatile("" : "+v"(Qf[kc]));
    __syncthreads();

    // Every wave passes the same number of barriers: waves whose rows cannot see a tile skip its work, not its
    // barriers. The extra round t = n_tiles only drains P V of the final tile.
    // barrier that orders LDS traffic only: the staging loads in flight must not be waited for here
    auto lds_barrier = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // One barrier per round and wave, at different places of the same loop: group 0 passes it after its softmax
    // phase, group 1 between its MFMA and softmax phases. Round r (between barriers r-1 and r) is therefore
    //     group 0: MFMA stretch of tile r (P V of tile r-1, S of tile r), then softmax of tile r
    //     group 1: softmax of tile r-1, then the MFMA stretch of tile r
    // so a SIMD sees the two roles in opposite order, and where one stretch outlasts the other the two MFMA
    // stretches may overlap instead of waiting for each other.
    //   K(r+1) is requested by group 0 in the middle of round r (after its matrix-core phase) and complete before
    //   barrier r; K(r) is read in round r only, K(r-1) was last read before barrier r-1: two stages. V(r+1) is
    //   requested by group 1 at the start of round r (V(0) and V(1) before the loop) and complete before barrier r;
    //   V(r) is read in round r (first fragments, group 0's softmax) and in round r+1 (P V of tile r, group 1's first
    //   fragments): three stages, and V(r-2) was last read before barrier r-1.
    //
    // Two key groups (KG = 2): the same rounds, but group grp works on the key tiles 2 t + grp of the workgroup's 128 rows
    // and fetches its own K and V. Group 0 requests K(t+1) and V(t) at the start of softmax(t) - V(t-2) was last read
    // before barrier t-1 - and waits for them before barrier t, the first reads of both following it. Group 1 requests
    // K(t+2) and V(t+1) after barrier t and waits for them before barrier t+1: K(t) and V(t-1) were last read before
    // barrier t. Two stages of each do for either group.
    asm volatile(".p2align 6\n\t.rept %0\n\ts_nop 0\n\t.endr" : : "n"(fa_loop_pad(DH, KG)));
    if (KG == 2) {
        for (int t = 0; t <= n_rounds; ++t) {
            mfma_phase(t);
            if (grp == 1) {
                dma_wait();
                lds_barrier();
                if (t + fa_k_lead(1) < n_tiles) fetch_k(t + fa_k_lead(1));
                if (t + fa_v_lead(1) < n_tiles) fetch_v(t + fa_v_lead(1));
            } else {
                if (t + fa_k_lead(0) < n_tiles) fetch_k(t + fa_k_lead(0));
                if (t + fa_v_lead(0) < n_tiles) fetch_v(t + fa_v_lead(0));
            }
            valu_phase(t);
            if (grp == 0) {
                dma_wait();
                lds_barrier();
            }
        }
    } else {
        for (int t = 0; t <= n_rounds; ++t) {
            mfma_phase(t);
            if (grp == 1) {
                dma_wait();  // V(t+1)
                lds_barrier();
                if (t + 2 < n_tiles) dma_next_tile((t + 2) % 3);  // V(t+2)
            }
            // Both groups request their tile at the START OF THEIR SOFTMAX PHASE, while the other group runs MFMAs: the
            // compute unit's one address unit takes 16 cycles per request and holds few, so a wave queues behind its
            // group's 16 requests, and ahead of a matrix-core phase that wait leaves the matrix pipe idle (K requested
            // before group 0's matrix-core phase, where it also met group 1's V requests: 3 % slower).
            if (grp == 0 && t + 1 < n_tiles) dma_next_tile((t + 1) & 1);  // K(t+1)
            valu_phase(t);
            if (grp == 0) {
                dma_wait();  // K(t+1)
                lds_barrier();
            }
        }
    }

    lsum += __shfl_xor(lsum, 32);
    float inv = 1.0f / lsum;
    if (KG == 2) {
        // The two key groups' results for the same rows meet in LDS (all tiles are read, nothing is in flight): group 0
        // finishes the first half of the dims, group 1 the second, either with the other's half of its sums.
        constexpr int HB = DB / 2;
        f32x4* xo = reinterpret_cast<f32x4*>(fa_smem_raw);                                          // [4][2][4 HB][64]
        float2* xm = reinterpret_cast<float2*>(fa_smem_raw + 4 * 2 * 4 * HB * kWave * sizeof(f32x4));  // [4][2][32]
        const float m_own = lsum == 0.f ? -INFINITY : m;  // no key of this group is visible to the row
#pragma unroll
        for (int b = 0; b < HB; ++b)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                f32x4 t;
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] = grp == 0 ? Oacc[HB + b][4 * rg + e] : Oacc[b][4 * rg + e];
                xo[((gw * 2 + grp) * 4 * HB + 4 * b + rg) * kWave + lane] = t;
            }
        if (h == 0) xm[(gw * 2 + grp) * 32 + j] = make_float2(m_own, lsum);
        __syncthreads();
        const float2 other = xm[(gw * 2 + 1 - grp) * 32 + j];
        const float M = fmaxf(m_own, other.x);
        const float a_own = __builtin_amdgcn_exp2f(m_own - M), a_oth = __builtin_amdgcn_exp2f(other.x - M);
        inv = grp == 0 ? 1.0f / (lsum * a_own + other.y * a_oth) : 1.0f / (other.y * a_oth + lsum * a_own);
        __bf16* mine = reinterpret_cast<__bf16*>(xm + 4 * 2 * 32) + wave * 32 * out_row(32 * HB);
        {
#pragma unroll
            for (int b = 0; b < HB; ++b)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    const f32x4 t = xo[((gw * 2 + 1 - grp) * 4 * HB + 4 * b + rg) * kWave + lane];
                    bf16x4 ov;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float own = grp == 0 ? Oacc[b][4 * rg + e] : Oacc[HB + b][4 * rg + e];
                        ov[e] = (__bf16)((own * a_own + t[e] * a_oth) * inv);
                    }
                    *reinterpret_cast<bf16x4*>(mine + j * out_row(32 * HB) + 32 * b + 8 * rg + 4 * h) = ov;
                }
        }
        store_rows<32 * HB>(mine, lane, q0, n, o + (size_t)head * DH + grp * 32 * HB, (size_t)Hq * DH);
        return;
    }
    // all tiles are read, nothing is in flight: every wave passes its rows through a piece of LDS of its own
    __bf16* mine = reinterpret_cast<__bf16*>(fa_smem_raw) + wave * 32 * out_row(DH);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            bf16x4 ov;
#pragma unroll
            for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(Oacc[db][4 * rg + e] * inv);
            *reinterpret_cast<bf16x4*>(mine + j * out_row(DH) + 32 * db + 8 * rg + 4 * h) = ov;
        }
    store_rows<DH>(mine, lane, q0, n, o + (size_t)head * DH, (size_t)Hq * DH);
}

template <int DH>
static dash_status launch_f32(const dash_layer_params& p, const float* q, const float* k, const float* v,
                              const int32_t* pos, int n, float* o, float scale, uint32_t* clear_words, int n_clear, int32_t* clear_count,
                              hipStream_t s) {
    const int n_qtiles = (n + 15) / 16;
    hipLaunchKernelGGL((flash_fwd_f32<DH>), dim3((unsigned)n_qtiles * p.n_q_heads), dim3(kF32Waves * kWave), 0, s, q, k, v,
                       pos, o, n, p.n_q_heads, p.n_kv_heads, scale, p.causal, n_qtiles, clear_words, n_clear, clear_count);
    return launch_status();
}

// One-time launch attribute of the MFMA kernels: their dynamic LDS size.
template <int DH, int KG>
static hipError_t set_flash_lds_size() {
    return hipFuncSetAttribute((const void*)flash_fwd_mfma<DH, KG>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)FaSmem<DH>::bytes(KG));
}

dash_status init_flash_kernels() {
    static const hipError_t err = [] {
        hipError_t e = set_flash_lds_size<64, 1>();
        if (e == hipSuccess) e = set_flash_lds_size<64, 2>();
        if (e == hipSuccess) e = set_flash_lds_size<128, 1>();
        if (e == hipSuccess) e = set_flash_lds_size<128, 2>();
        return e;
    }();
    return err == hipSuccess ? DASH_OK : DASH_ERR_HIP;
}

// Query rows [row0, row1) against all keys (row0 = 0 with one key group).
template <int DH, int KG>
static dash_status launch_mfma(const dash_layer_params& p, const __bf16* q, const __bf16* k, const __bf16* v,
                               const int32_t* pos, int n, int row0, int row1, __bf16* o, float scale_log2,
                               uint32_t* clear_words, int n_clear, int32_t* clear_count, hipStream_t s) {
    const int n_qtiles = (row1 - row0 + kFaBM / KG - 1) / (kFaBM / KG);
    const int Hq = p.n_q_heads, Hkv = p.n_kv_heads;
    unsigned blocks = 0;
    const FaMap mp = p.causal ? fa_map_later(n_qtiles, Hq, Hkv, DH, KG, compute_units(), blocks) : fa_map(n_qtiles, Hq, Hkv, blocks);
    hipLaunchKernelGGL((flash_fwd_mfma<DH, KG>), dim3(blocks), dim3(kFaThreads), FaSmem<DH>::bytes(KG), s, q, k, v, pos, o, n,
                       Hq, Hkv, scale_log2, p.causal, n_qtiles, mp, clear_words, n_clear, row0, clear_count);
    return launch_status();
}

dash_status launch_flash_fwd(const dash_layer_params& p, const void* q, const void* k, const void* v,
                             const int32_t* active_idx, int n, void* o, uint32_t* clear_words, int n_clear,
                             int32_t* clear_count, void* scratch, size_t scratch_bytes, hipStream_t s) {
    if (n == 0) return DASH_OK;
    const float scale = p.softmax_scale > 0.f ? p.softmax_scale : 1.0f / sqrtf((float)p.head_dim);
    if (p.dtype == DASH_F32) {
        const float *fq = (const float*)q, *fk = (const float*)k, *fv = (const float*)v;
        return p.head_dim == 64 ? launch_f32<64>(p, fq, fk, fv, active_idx, n, (float*)o, scale, clear_words, n_clear, clear_count, s)
                                : launch_f32<128>(p, fq, fk, fv, active_idx, n, (float*)o, scale, clear_words, n_clear, clear_count, s);
    }
    // the MFMA kernel addresses K and V with 32-bit byte offsets
    if ((size_t)n * p.n_kv_heads * p.head_dim * 2 >= (size_t)1 << 31) return DASH_ERR_UNSUPPORTED;
    if (init_flash_kernels() != DASH_OK || compute_units() <= 0) return DASH_ERR_HIP;
    const float scale_log2 = scale * 1.4426950408889634f;
    const __bf16 *bq = (const __bf16*)q, *bk = (const __bf16*)k, *bv = (const __bf16*)v;
    const int waves = few_waves(n, p.n_q_heads, p.head_dim, p.causal != 0, compute_units());
    if (waves > 0)
        return launch_flash_few(p, bq, bk, bv, active_idx, n, 0, (__bf16*)o, scale_log2, waves, clear_words, n_clear, clear_count, s);
    const FaForm form = fa_form(n, p.n_q_heads, p.head_dim, p.causal != 0, compute_units());  // staging_addr.h
    const int one_end = form == FA_TWO ? 0 : (form == FA_ONE ? n : n - n % kFaBM);  // rows of the one-group form
    dash_status st = DASH_OK;
    if (one_end > 0)
        st = p.head_dim == 64 ? launch_mfma<64, 1>(p, bq, bk, bv, active_idx, n, 0, one_end, (__bf16*)o, scale_log2, clear_words, n_clear, clear_count, s)
                              : launch_mfma<128, 1>(p, bq, bk, bv, active_idx, n, 0, one_end, (__bf16*)o, scale_log2, clear_words, n_clear, clear_count, s);
    if (st != DASH_OK || one_end == n) return st;
    if (one_end > 0) {  // cleared by the first launch
        n_clear = 0;
        clear_count = nullptr;
    }
    if (form == FA_ONE_AND_TAIL && fa_few_tail(n, p.n_q_heads, p.head_dim, compute_units())) {
        const FewParts parts = few_tail_parts(n, p.n_q_heads, p.head_dim, compute_units(), scratch ? scratch_bytes : 0);
        if (parts.parts > 1)
            return launch_flash_few_parts(p, bq, bk, bv, active_idx, n, one_end, (__bf16*)o, scale_log2, parts, (float*)scratch, s);
        return launch_flash_few(p, bq, bk, bv, active_idx, n, one_end, (__bf16*)o, scale_log2, kFewTailWaves, clear_words, n_clear, clear_count, s);
    }
    return p.head_dim == 64 ? launch_mfma<64, 2>(p, bq, bk, bv, active_idx, n, one_end, n, (__bf16*)o, scale_log2, clear_words, n_clear, clear_count, s)
                            : launch_mfma<128, 2>(p, bq, bk, bv, active_idx, n, one_end, n, (__bf16*)o, scale_log2, clear_words, n_clear, clear_count, s);
}

}  // namespace dash
