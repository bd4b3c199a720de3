// Output projection fused with the residual update and the row norms:
//   delta = O @ W_o            (completes U of Eq. 1: the attention output before the residual add)
//   x_next = x + delta         (Sec. 3.1, Alg. 1 step 6)
//   partial sums of delta^2 and x^2 per row, from the fp32 accumulators (feeds Eq. 2)
// delta never goes to HBM (unless the caller asks for the debug copy): the score is taken before the
// bf16 rounding of x_next, which would otherwise cancel catastrophically for large-norm rows.
//
// Also here: the front end used by a chain of layers (RMSNorm + q/k/v projections), which shares the
// MFMA main loop with a plain store epilogue.
//
// norm_partials layout: [P][n][2] fp32, P = column tiles of the kernel in use (256 columns; 64 in the fp32 kernel).
#include "common.h"
#include "lds_ops.h"
#include "staging_addr.h"

namespace dash {

// ------------------------------------------------------------------------------------------------
// fp32 kernel: v_mfma_f32_16x16x4_f32 on a tile of 32 rows x 64 columns; the 8 waves split K (wave w takes the 16-wide
// chunks w, w + 8, ...) and their sums are added in the order of w through LDS. The products of this path have few rows
// and few columns, so a larger tile would leave the chip idle and a wave with all of K a long serial chain. Step s of
// chunk c contracts 16 c + 4 g + s (lane = 16 g + i) and column block e holds columns 4 i + e, so that every operand is a
// 16-byte global load; no LDS and no barrier in the loop. Latency-bound at a few hundred rows, then bound by the L2
// reads (96 words per 32 x 64 products and step). Measured, with K = N (in parentheses with 64 x 64 tiles staged through LDS): 2048 rows
// of 512 15 us (97), 8192 of 512 46 us (127); the error against 64 bits fell from 2.9e-7 to 1.2e-7, the chains of adds being shorter.
// Fewer rows: wo_f32_few_kernel.
// ------------------------------------------------------------------------------------------------
constexpr int kF32TileM = 32, kF32TileN = 64;
constexpr int kF32Split = 8;

__global__ __launch_bounds__(kF32Split * kWave) void wo_f32_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                                   const float* __restrict__ x, int M, int K, int N,
                                                                   float* __restrict__ x_next, float* __restrict__ partials,
                                                                   float* __restrict__ delta_dbg) {
    __shared__ float part[kF32Split][16][kF32TileN + 4];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int i = lane % 16, g = lane / 16;
    const int64_t tile_m = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;  // the last slice of row tiles may be padded
    if (tile_m * kF32TileM >= M) return;                                  // the whole workgroup
    const int m0 = (int)tile_m * kF32TileM, n0 = blockIdx.x * kF32TileN;
    f32x4 acc[2][4];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[rb][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    // rows beyond M and columns beyond N are computed on clamped addresses and never stored (K % 16 == 0, N % 4 == 0)
    const float* ap[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) ap[rb] = A + (size_t)min(m0 + 16 * rb + i, M - 1) * K + 4 * g;
    const float* bp = B + (size_t)(4 * g) * N + min(n0 + 4 * i, N - 4);
    struct Chunk {
        f32x4 a[2], b[4];
    };
    auto load = [&](int k0) {
        Chunk c;
#pragma unroll
        for (int s = 0; s < 4; ++s) c.b[s] = *reinterpret_cast<const f32x4*>(bp + (size_t)(k0 + s) * N);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) c.a[rb] = *reinterpret_cast<const f32x4*>(ap[rb] + k0);
        return c;
    };
    int k0 = 16 * wave;
    if (k0 < K) {
        Chunk cur = load(k0);
        for (; k0 < K; k0 += 16 * kF32Split) {
            // the next chunk is in flight while this one is multiplied (after the last one: this one again, unused)
            const Chunk next = load(k0 + 16 * kF32Split < K ? k0 + 16 * kF32Split : k0);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[rb][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.a[rb][s], cur.b[s][e], acc[rb][e], 0, 0, 0);
            cur = next;
        }
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        if (rb > 0) __syncthreads();  // the readers of the block before are done
#pragma unroll
        for (int r = 0; r < 4; ++r)  // register r of a block: row 4 g + r; blocks e = columns 4 i + e
            *reinterpret_cast<f32x4*>(&part[wave][4 * g + r][4 * i]) = f32x4{acc[rb][0][r], acc[rb][1][r], acc[rb][2][r], acc[rb][3][r]};
        __syncthreads();
        if (tid < 256) {  // 16 threads per row, four columns each (whole waves)
            const int lr = tid / 16, gm = m0 + 16 * rb + lr, gn = n0 + 4 * (tid % 16);
            f32x4 d = *reinterpret_cast<const f32x4*>(&part[0][lr][4 * (tid % 16)]);
#pragma unroll
            for (int w = 1; w < kF32Split; ++w) d += *reinterpret_cast<const f32x4*>(&part[w][lr][4 * (tid % 16)]);
            float sd = 0.f, sx = 0.f;
            if (gm < M && gn < N) {
                const f32x4 xv = *reinterpret_cast<const f32x4*>(x + (size_t)gm * N + gn);
                *reinterpret_cast<f32x4*>(x_next + (size_t)gm * N + gn) = xv + d;
                if (delta_dbg) *reinterpret_cast<f32x4*>(delta_dbg + (size_t)gm * N + gn) = d;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sd = fmaf(d[e], d[e], sd);
                    sx = fmaf(xv[e], xv[e], sx);
                }
            }
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                sd += __shfl_xor(sd, off);
                sx += __shfl_xor(sx, off);
            }
            if (tid % 16 == 0 && gm < M)
                *reinterpret_cast<float2*>(partials + ((size_t)blockIdx.x * M + gm) * 2) = make_float2(sd, sx);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same on tiles of 16 rows x 64 columns, where those are no more than the compute units: with 32-row tiles 512 rows of 256
// occupied 64 units with twice the serial work. The same split of K, so the same sums. A wave has four chunks in flight (in the
// kernel above the compiler moves the next chunk's loads to their use; where many workgroups share a unit, that and the fewer
// registers are the faster way: four chunks in flight there cost 10 to 35 %), and x is asked for before the product. Measured, 32-row
// tiles / these, us, K = N: 512 rows of 256 6.2 / 4.9, of 512 8.9 / 6.8, 177 of 1024 13.7 / 10.4, 63 of 3584 42 / 27.6; with more tiles
// than units 257 rows of 1024 13.8 / 16.1, 1100 of 256 6.4 / 7.2.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kF32Split * kWave) void wo_f32_few_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                                       const float* __restrict__ x, int M, int K, int N,
                                                                       float* __restrict__ x_next, float* __restrict__ partials,
                                                                       float* __restrict__ delta_dbg) {
    __shared__ float part[kF32Split][16][kF32TileN + 4];
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int i = lane % 16, g = lane / 16;
    const int m0 = (int)blockIdx.y * 16, n0 = blockIdx.x * kF32TileN;
    // the epilogue's thread: 16 per row, four columns each; x is asked for before the product
    const int lr = tid / 16, gm = m0 + lr, gn = n0 + 4 * (tid % 16);
    const bool has_row = tid < 256, ok = has_row && gm < M && gn < N;
    f32x4 xv = f32x4{0.f, 0.f, 0.f, 0.f};
    if (ok) xv = *reinterpret_cast<const f32x4*>(x + (size_t)gm * N + gn);
    f32x4 acc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    // rows beyond M and columns beyond N are computed on clamped addresses and never stored (K % 16 == 0, N % 4 == 0)
    const float* ap = A + (size_t)min(m0 + i, M - 1) * K + 4 * g;
    const float* bp = B + (size_t)(4 * g) * N + min(n0 + 4 * i, N - 4);
    struct Chunk {
        f32x4 a, b[4];
    };
    auto load = [&](int k0, Chunk& c) {
#pragma unroll
        for (int s = 0; s < 4; ++s) c.b[s] = *reinterpret_cast<const f32x4*>(bp + (size_t)(k0 + s) * N);
        c.a = *reinterpret_cast<const f32x4*>(ap + k0);
    };
    auto multiply = [&](const Chunk& c) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.a[s], c.b[s][e], acc[e], 0, 0, 0);
    };
    // The chunks of a wave in order, kAhead of them in flight; the conditions are scalar, so each is a load of its own kind and not
    // moved to its use.
    constexpr int kAhead = 4, kStep = 16 * kF32Split;
    Chunk c[kAhead];
    int k0 = 16 * wave;
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
        if (k0 + u * kStep < K) load(k0 + u * kStep, c[u]);
    for (; k0 < K; k0 += kAhead * kStep) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (k0 + u * kStep < K) {
                multiply(c[u]);
                if (k0 + (u + kAhead) * kStep < K) load(k0 + (u + kAhead) * kStep, c[u]);
            }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(&part[wave][4 * g + r][4 * i]) = f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
    __syncthreads();
    if (!has_row) return;  // whole waves
    f32x4 d = *reinterpret_cast<const f32x4*>(&part[0][lr][4 * (tid % 16)]);
#pragma unroll
    for (int w = 1; w < kF32Split; ++w) d += *reinterpret_cast<const f32x4*>(&part[w][lr][4 * (tid % 16)]);
    float sd = 0.f, sx = 0.f;
    if (ok) {
        *reinterpret_cast<f32x4*>(x_next + (size_t)gm * N + gn) = xv + d;
        if (delta_dbg) *reinterpret_cast<f32x4*>(delta_dbg + (size_t)gm * N + gn) = d;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sd = fmaf(d[e], d[e], sd);
            sx = fmaf(xv[e], xv[e], sx);
        }
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        sd += __shfl_xor(sd, off);
        sx += __shfl_xor(sx, off);
    }
    if (tid % 16 == 0 && gm < M)
        *reinterpret_cast<float2*>(partials + ((size_t)blockIdx.x * M + gm) * 2) = make_float2(sd, sx);
}

// ------------------------------------------------------------------------------------------------
// MFMA kernel (bf16): C[M,N] = A[M,K] B[K,N], A and B row-major.
// Workgroup tile 256x256, K step 64; 8 waves in 2 (M) x 4 (N), two per SIMD, each wave 128x64 = 8x4 blocks of
// v_mfma_f32_16x16x32_bf16 (128 fp32 accumulator registers per lane). On normally distributed operands the part
// is power-limited, and this shape moves fewer accumulator registers per flop than 32x32x16: the same tiles and
// LDS traffic finish 1-2 % sooner end to end, although twice the MFMA instructions cost cycles at the full
// clock. A fragments are 16-byte LDS reads from the [m][k] tile; B fragments come from the natural [k][n] tile
// through LDS transpose reads.
// The tiles of a K step go from global memory straight into LDS (no registers in between). Such a load
// writes 1 KB of consecutive LDS per wave instruction, so rows cannot be padded; bank conflicts are avoided
// by an XOR swizzle of the 16-byte chunk index inside a row: A (128-byte rows, 16-byte reads of one chunk
// from 16 consecutive rows) by (row / 2) % 8, B (512-byte rows; 32 lanes read 4 k-rows and the 4 k-rows 8
// below them, 32 bytes of each) by 4 * (row % 4) + 2 * ((row / 8) % 2).
// ------------------------------------------------------------------------------------------------
constexpr int kGThreads = kGWaves * kWave;  // tile constants kGM, kGN, kGK: staging_addr.h
constexpr int kGBElems = kGK * kGN;
// Operand stages in LDS: a stage holds the A tile (32 RB rows, whole load instructions of every wave: the 224-row tile fetches 256)
// and the B tile of one K step. The 256-row tile has
// two stages (128 KB): the tiles of step k + 2 are requested once every wave is done with step k. The 128-row half
// tile has three (144 KB) and requests three steps ahead: its steps are half as long, and with only one step of
// lead it waited for memory latency at every step.
constexpr int gemm_stages(int RB) { return RB == 4 ? 3 : 2; }
constexpr int gemm_stage_elems(int RB) { return 8 * kGWaves * gemm_adma(32 * RB) * kGK + kGBElems; }
constexpr size_t gemm_smem_bytes(int RB) { return (size_t)gemm_stages(RB) * gemm_stage_elems(RB) * sizeof(__bf16); }
constexpr int kEpiStr = 64 + 4;  // fp32 words per staged epilogue row (conflict-free 16-byte reads of two rows by 16 lanes)
static_assert(gemm_smem_bytes(6) >= 8 * 32 * kEpiStr * sizeof(float) + 4 * kGM * 2 * sizeof(float) &&
                  gemm_smem_bytes(4) >= 8 * 32 * kEpiStr * sizeof(float) + 4 * kGM * 2 * sizeof(float),
              "epilogue staging and the row-sum exchange must fit");


// EPI_SWIGLU: B holds gate and up columns interleaved in blocks of 32 (columns 64c..64c+31 = gate features
// 32c..32c+31, columns 64c+32..64c+63 = the up columns of the same features), so a wave's two 32-column
// accumulator blocks are gate and up of the same 32 features and the epilogue writes silu(gate) * up,
// N / 2 columns per row.
// EPI_SPLITK: the workgroup covers only the K steps of split blockIdx.y and writes its fp32 accumulators to
// f32_out[split][M][N]; a reduction kernel adds the splits in order and applies one of the other epilogues.
// EPI_QKV: a plain store whose columns are routed to three outputs (the q, k and v projections as one product
// over the concatenated weight).
// EPI_QKV_ROPE: the same with the q and k columns rotated on the way (rotary embedding), from the fp32 sums and a table
// of cosines and sines that the row norm's launch leaves: q and k are not read and written once more.
enum { EPI_RESIDUAL_NORM = 0, EPI_STORE = 1, EPI_SWIGLU = 2, EPI_SPLITK = 3, EPI_QKV = 4, EPI_QKV_ROPE = 5 };
constexpr bool epi_qkv(int EPI) { return EPI == EPI_QKV || EPI == EPI_QKV_ROPE; }

// Output routing of EPI_QKV: columns [0, Dq) go to `out` (row stride Dq), [Dq, Dq + Dkv) to k and the rest to v
// (row stride Dkv). Dq and Dkv are multiples of 8, so the 8 columns a lane stores never straddle two outputs.
struct QkvOut {
    __bf16* k;
    __bf16* v;
    int Dq, Dkv;
    const float2* table;  // EPI_QKV_ROPE: [n][half] cosine and sine of each row's angles
    int half;             // head_dim / 2
};
// The 8 columns of a row that start at `col` (v) rotated with their partners `half` columns away in the same head.
__device__ __forceinline__ void rope8(const QkvOut& o, int row, int col, const float* partner, float* v) {
    const int i0 = col % o.half;  // col is a multiple of 8, half 32 or 64: the eight columns lie on one side
    const bool hi = col % (2 * o.half) >= o.half;
    const float4* t = reinterpret_cast<const float4*>(o.table + (size_t)row * o.half + i0);
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const float4 cs = t[e / 2];  // cos, sin of two neighbouring frequencies
        const float s0 = hi ? cs.y : -cs.y, s1 = hi ? cs.w : -cs.w;
        v[e] = fmaf(partner[e], s0, v[e] * cs.x);
        v[e + 1] = fmaf(partner[e + 1], s1, v[e + 1] * cs.z);
    }
}
__device__ __forceinline__ __bf16* qkv_dst(__bf16* q, const QkvOut& o, int row, int col) {
    if (col < o.Dq) return q + (size_t)row * o.Dq + col;
    col -= o.Dq;
    if (col < o.Dkv) return o.k + (size_t)row * o.Dkv + col;
    return o.v + (size_t)row * o.Dkv + (col - o.Dkv);
}

// How the workgroups of a launch map to tiles (staging_addr.h: GemmPlan, gemm_index_of, gemm_tile_of).
struct GemmLaunch {
    int mt, nt, ksteps;
    int full, plain, seg;   // the launch of whole tiles: tile order and indices per XCD
    int first_tile;         // half tiles start at this tile index
    int row0;               // first row of the tiles (not half tiles)
    int ksteps_per_split;   // EPI_SPLITK: K steps per part (part = blockIdx.y)
};

// RB = 16-row blocks per wave: 8 gives the 256-row tile, 7 and 6 tiles of 224 and 192 rows (RowPlan), 4 a 128-row half tile. Half
// tiles finish the grid: when the 256-row tiles do not fill a whole number of rounds over the compute units, the tiles of
// the last, partly filled round are cut in two so that twice as many units share them: workgroup b of that
// second launch handles half b % 2 of tile first_tile + b / 2.
template <int EPI, int RB>
__global__ __launch_bounds__(kGThreads, 1) void gemm_mfma_kernel(const __bf16* __restrict__ A,
                                                                 const __bf16* __restrict__ B, int M, int K,
                                                                 int N, const __bf16* __restrict__ x,
                                                                 __bf16* __restrict__ out,  // x_next or C
                                                                 float* __restrict__ partials,
                                                                 float* __restrict__ f32_out,  // delta (debug) or split sums
                                                                 GemmLaunch L, QkvOut qkv) {
    constexpr int BM = 32 * RB;   // rows of this workgroup's tile
    constexpr int WM = 16 * RB;   // rows of a wave's tile
    constexpr bool HALF = RB == 4;
    constexpr int NS = gemm_stages(RB), kStageElems = gemm_stage_elems(RB), kAElems = kStageElems - kGBElems;
    extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem_raw[];
    __bf16* smem = reinterpret_cast<__bf16*>(gemm_smem_raw);
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave / 4, wn = wave % 4;
    // this workgroup's tile and K steps
    int tile_idx, ks0 = 0, n_ksteps = L.ksteps;
    if (EPI == EPI_SPLITK) {
        tile_idx = HALF ? L.first_tile + (int)blockIdx.x / 2 : (int)blockIdx.x;
        ks0 = (int)blockIdx.y * L.ksteps_per_split;
        n_ksteps = min(L.ksteps_per_split, L.ksteps - ks0);
    } else if (HALF) {
        tile_idx = L.first_tile + (int)blockIdx.x / 2;
    } else {
        tile_idx = gemm_index_of((int)blockIdx.x, L.full, L.plain != 0, L.seg);
        if (tile_idx < 0) return;  // padding of the last stretch: the whole workgroup leaves
    }
    int tile_m, tile_n;
    gemm_tile_of(tile_idx, L.mt, L.nt, L.plain != 0, tile_m, tile_n);
    const int m0 = HALF ? tile_m * kGM + ((int)blockIdx.x % 2) * BM : L.row0 + tile_m * BM, n0 = tile_n * kGN;

    f32x4 acc[RB][4];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.f;

    // Staging. A tile: BM rows of 128 bytes, one load instruction = 8 rows; B tile: 64 rows of 512 bytes,
    // one instruction = 2 rows. Lane l lands in physical chunk l % (chunks per row) of its row and therefore
    // fetches the logical chunk that the swizzle maps there. Rows beyond M and columns beyond N are clamped:
    // they are computed on valid data and never stored.
    // The address of a load is a scalar base (this workgroup's tile at the current K step, advanced by scalar
    // arithmetic) plus a 32-bit lane offset that never changes.
    constexpr int ADMA = gemm_adma(BM), BDMA = gemm_bdma();  // load instructions per wave and K step
    uint32_t a_off[ADMA], b_off[BDMA];
#pragma unroll
    for (int i = 0; i < ADMA; ++i) {
        const int row = gemm_a_row(wave, i, lane, ADMA);
        a_off[i] = gemm_a_off(m0, M, K, row, gemm_a_lchunk(row, lane));
    }
#pragma unroll
    for (int i = 0; i < BDMA; ++i) {
        const int row = gemm_b_row(wave, i, lane);
        b_off[i] = gemm_b_off(n0, N, row, gemm_b_lchunk(row, lane));
    }
    const char* a_base = reinterpret_cast<const char*>(A + gemm_a_base_elem(m0, M, K, ks0));
    const char* b_base = reinterpret_cast<const char*>(B + gemm_b_base_elem(n0, N, ks0));
    const size_t b_step = gemm_b_step_bytes(N);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)gemm_smem_raw;
    const uint32_t lds_a = lds0 + (uint32_t)(wave * ADMA * 1024);
    const uint32_t lds_b = lds0 + (uint32_t)(kAElems * 2 + wave * BDMA * 1024);
    // K steps are fetched strictly in order; the A and the B tile of a step are requested separately
    auto dma_next_a = [&](int stage) {
        const uint32_t so = (uint32_t)(stage * kStageElems * 2);
#pragma unroll
        for (int i = 0; i < ADMA; ++i) dma_load16(a_base, a_off[i], lds_a + so + i * 1024);
        a_base += gemm_a_step_bytes();
    };
    auto dma_next_b = [&](int stage) {
        const uint32_t so = (uint32_t)(stage * kStageElems * 2);
#pragma unroll
        for (int i = 0; i < BDMA; ++i) dma_load16(b_base, b_off[i], lds_b + so + i * 1024);
        b_base += b_step;
    };

    // barrier that orders LDS traffic only
    auto lds_barrier = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // Fragments of one 32-wide slice for v_mfma_f32_16x16x32_bf16: RB A fragments (rows 16 rb + i, k-slots
    // 8 g .. 8 g + 7: one 16-byte read) and four B fragments (columns 16 cb + i, the same k-slots: two transpose
    // reads of a 4 x 16 block each), lane = 16 g + i.
    const int fi = lane % 16, fg = lane / 16;
    bf16x8 Af[2][RB], Bf[2][4];
    auto read_frags = [&](int st, int ks, bf16x8* af, bf16x8* bfr) {
        const __bf16* sa = smem + st * kStageElems;
        const __bf16* sb = sa + kAElems;
        // B first: the MFMAs of a slice go through the row blocks in order and need every B fragment at once
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int krow = 32 * ks + 8 * fg + fi / 4;  // and krow + 4: the same swizzle
            const int col = wn * 64 + 16 * b + 4 * (fi % 4);
            const int scol = ((col / 8) ^ gemm_b_swz(krow)) * 8 + col % 8;
            const s16x4 lo = lds_read_tr16(&sb[krow * kGN + scol]);
            const s16x4 hi = lds_read_tr16(&sb[(krow + 4) * kGN + scol]);
            bfr[b] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int a = 0; a < RB; ++a) {
            const int row = wm * WM + 16 * a + fi;
            af[a] = *reinterpret_cast<const bf16x8*>(&sa[row * kGK + ((4 * ks + fg) ^ ((row / 2) % 8)) * 8]);
        }
    };
    auto mfma_slice = [&](const bf16x8* af, const bf16x8* bfr) {
#pragma unroll
        for (int a = 0; a < RB; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
    };
    // issue order of one slice: the fragment reads of the slice after it spread between its MFMAs
    constexpr int RD = RB + 8, MF = 4 * RB;  // LDS reads and MFMAs per slice: 16 and 32 (256 rows), 15 and 28, 14 and 24, 12 and 16
    auto pin_slice = [] {
#pragma unroll
        for (int i = 0; i < 2 * RD - MF; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < MF - RD; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };
    constexpr int kStepLoads = ADMA + BDMA;
    const int n_pre = min(NS, n_ksteps);
    for (int j = 0; j < n_pre; ++j) {
        dma_next_a(j);
        dma_next_b(j);
    }
    if (n_pre == NS) {
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NS - 1) * kStepLoads) : "memory");  // step 0 has landed
    } else {
        dma_wait();
    }
    __syncthreads();
    read_frags(0, 0, Af[0], Bf[0]);
    // One round per K step of two 32-wide slices. The fragments of a slice are read while the MFMAs of the slice
    // before it run, across the step boundary too: the wait for the next step's tiles and the barrier that
    // publishes them sit before the second slice's MFMAs, whose fragments are in registers by then, and the
    // first slice of the next step is read from the next stage while those MFMAs run. After that barrier every
    // wave is done reading this step's stage, so the tiles of step kt + NS are requested into it.
    //
    // Second half of a step. The tile requests are dealt out between its MFMAs, one every three: the compute
    // unit's one address unit takes 16 cycles per request and holds few of them, so after a burst of requests every
    // wave queues behind it and issues no MFMA meanwhile (a burst after the barrier: 5 % slower; one request per
    // MFMA, per 2, per 4: 3, 1.5 and 0.5 % slower than per 3). The requests are opaque to the compiler's scheduler
    // and fence its LDS reads, so this half is placed by hand: requests, the fragment reads of the next slice (B
    // first) at even distances, MFMAs, pinned in eight groups (224 rows: seven of four, 28 having no eighth).
    auto read_b_frag = [&](int st, int ks, int b, bf16x8* bfr) {
        const __bf16* sb = smem + st * kStageElems + kAElems;
        const int krow = 32 * ks + 8 * fg + fi / 4;
        const int col = wn * 64 + 16 * b + 4 * (fi % 4);
        const int scol = ((col / 8) ^ gemm_b_swz(krow)) * 8 + col % 8;
        const s16x4 lo = lds_read_tr16(&sb[krow * kGN + scol]);
        const s16x4 hi = lds_read_tr16(&sb[(krow + 4) * kGN + scol]);
        bfr[b] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_a_frag = [&](int st, int ks, int a, bf16x8* af) {
        const __bf16* sa = smem + st * kStageElems;
        const int row = wm * WM + 16 * a + fi;
        af[a] = *reinterpret_cast<const bf16x8*>(&sa[row * kGK + ((4 * ks + fg) ^ ((row / 2) % 8)) * 8]);
    };
    constexpr int kGroup = MF % 8 == 0 ? MF / 8 : 4;
    constexpr int kRequestEvery = 3;  // MFMAs from one tile request to the next
    static_assert((kStepLoads - 1) * kRequestEvery < MF, "the requests of a step fit into its second half");
    auto second_half = [&](int st_next, bool request, int st_free) {
        constexpr int UNITS = 4 + RB;  // fragments of the next slice: 4 B, RB A
        const uint32_t so = (uint32_t)(st_free * kStageElems * 2);
#pragma unroll
        for (int m = 0; m < MF; ++m) {
#pragma unroll
            for (int l = 0; l < kStepLoads; ++l)
                if (m == l * kRequestEvery && request) {
                    if (l < ADMA) dma_load16(a_base, a_off[l], lds_a + so + l * 1024);
                    else dma_load16(b_base, b_off[l - ADMA], lds_b + so + (l - ADMA) * 1024);
                }
#pragma unroll
            for (int u = 0; u < UNITS; ++u)  // fragment u before the first MFMA m with u * MF <= m * UNITS
                if (u * MF <= m * UNITS && (m == 0 || u * MF > (m - 1) * UNITS)) {
                    if (u < 4) read_b_frag(st_next, 0, u, Bf[0]);
                    else read_a_frag(st_next, 0, u - 4, Af[0]);
                }
            acc[m / 4][m % 4] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Af[1][m / 4], Bf[1][m % 4], acc[m / 4][m % 4], 0, 0, 0);
            if (m % kGroup == kGroup - 1) __builtin_amdgcn_sched_barrier(0);
        }
        if (request) {
            a_base += gemm_a_step_bytes();
            b_base += b_step;
        }
    };
    int kt = 0, st = 0;  // st = kt % NS
    for (; kt + NS < n_ksteps; ++kt) {
        const int st_next = st + 1 == NS ? 0 : st + 1;
        read_frags(st, 1, Af[1], Bf[1]);
        mfma_slice(Af[0], Bf[0]);
        pin_slice();
        // the tiles of step kt + 1 have landed; those of the steps after it may still be in flight
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NS - 2) * kStepLoads) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // the second slice's fragments are in registers
        lds_barrier();
        second_half(st_next, true, st);
        st = st_next;
    }
    const int e_row = lane / 8, e_c8 = lane % 8;
    const int gn_e = n0 + wn * 64 + 8 * e_c8;
    const bool col_ok = gn_e < N;
    constexpr int EB = (RB + 1) / 2;  // the epilogue's 32-row blocks, the last one of 16 rows where RB is odd
    bf16x8 xv[EB][4];
    auto fetch_x = [&](int a) {
#pragma unroll
        for (int step = 0; step < 4; ++step) {
            const int gm = min(m0 + wm * WM + 32 * a + 8 * step + e_row, M - 1);
            xv[a][step] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(x + (size_t)gm * N + min(gn_e, N - 8)));
        }
    };
    for (; kt < n_ksteps; ++kt) {  // the last NS steps request nothing
        const int st_next = st + 1 == NS ? 0 : st + 1;
        if (EPI == EPI_RESIDUAL_NORM && kt + 1 == n_ksteps) fetch_x(0);
        read_frags(st, 1, Af[1], Bf[1]);
        mfma_slice(Af[0], Bf[0]);
        pin_slice();
        if (kt + 1 < n_ksteps) dma_wait();  // no tiles are in flight in the last one
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        lds_barrier();
        second_half(st_next, false, st);  // after the last step the fragments read are stale data, never used
        st = st_next;
    }
    __syncthreads();  // the stale fragment reads of slower waves are harmless, but keep the epilogue's reuse simple
    // all waves are past the last barrier: the operand stages are free and are reused by the epilogue

    // Epilogue, per 32-row block of the wave's tile: stage the fp32 accumulators in LDS, then every lane
    // handles 8 consecutive columns of one row - 16-byte x loads, 16-byte x_next stores, in-row sums over
    // 8 lanes. The x vectors of the first block are asked for in the last K step, the others all at once ahead of the epilogue, in the
    // operands' registers (a block ahead each: K = N = 3584 one round of tiles, 4096 rows 85.4 -> 83.2 us, 3000 67.5 -> 66.4; several rounds
    // the same, inside the power limit).
    float* stage = reinterpret_cast<float*>(gemm_smem_raw) + wave * 32 * kEpiStr;
    float2* nrm = reinterpret_cast<float2*>(gemm_smem_raw + kGWaves * 32 * kEpiStr * sizeof(float));  // [4 wave columns][BM rows]
    if (EPI == EPI_RESIDUAL_NORM)
#pragma unroll
        for (int a = 1; a < EB; ++a) fetch_x(a);
#pragma unroll
    for (int a = 0; a < EB; ++a) {
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r)  // accumulator register r of a 16x16 block: row 4 g + r, column i
                    if (2 * a + sb < RB) stage[(16 * sb + 4 * fg + r) * kEpiStr + 16 * b + fi] = acc[2 * a + sb < RB ? 2 * a + sb : 0][b][r];
        __syncthreads();  // every wave runs the same epilogue schedule, so the barrier is uniform
        if (EPI == EPI_SWIGLU) {
            // 4 lanes per row: lane c takes gate columns 8c..8c+7 and the up columns 32 + 8c..
            const int s_row = lane / 4, s_c = lane % 4;
            const int gcol = n0 / 2 + wn * 32 + 8 * s_c;  // output column
#pragma unroll
            for (int step = 0; step < 2; ++step) {
                const int lr = 16 * step + s_row;
                if (32 * a + 16 * step >= WM) break;
                const int gm = m0 + wm * WM + 32 * a + lr;
                const f32x4 g0 = *reinterpret_cast<const f32x4*>(&stage[lr * kEpiStr + 8 * s_c]);
                const f32x4 g1 = *reinterpret_cast<const f32x4*>(&stage[lr * kEpiStr + 8 * s_c + 4]);
                const f32x4 u0 = *reinterpret_cast<const f32x4*>(&stage[lr * kEpiStr + 32 + 8 * s_c]);
                const f32x4 u1 = *reinterpret_cast<const f32x4*>(&stage[lr * kEpiStr + 32 + 8 * s_c + 4]);
                const float gv[8] = {g0[0], g0[1], g0[2], g0[3], g1[0], g1[1], g1[2], g1[3]};
                const float uv[8] = {u0[0], u0[1], u0[2], u0[3], u1[0], u1[1], u1[2], u1[3]};
                if (gm < M && gcol < N / 2) {
                    bf16x8 ov;
#pragma unroll
                    for (int e = 0; e < 8; ++e) ov[e] = (__bf16)(gv[e] / (1.0f + __expf(-gv[e])) * uv[e]);
                    *reinterpret_cast<bf16x8*>(out + (size_t)gm * (N / 2) + gcol) = ov;
                }
            }
            __syncthreads();
            continue;
        }
#pragma unroll
        for (int step = 0; step < 4; ++step) {
            const int lr = 8 * step + e_row;
            if (32 * a + 8 * step >= WM) break;
            const int gm = m0 + wm * WM + 32 * a + lr;
            const f32x4 d0 = *reinterpret_cast<const f32x4*>(&stage[lr * kEpiStr + 8 * e_c8]);
            const f32x4 d1 = *reinterpret_cast<const f32x4*>(&stage[lr * kEpiStr + 8 * e_c8 + 4]);
            const float dv[8] = {d0[0], d0[1], d0[2], d0[3], d1[0], d1[1], d1[2], d1[3]};
            const bool ok = gm < M && col_ok;
            if (EPI == EPI_RESIDUAL_NORM) {
                float sd = 0.f, sx = 0.f;
                if (ok) {
                    const bf16x8 xr = xv[a][step];
                    bf16x8 ov;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float xf = (float)xr[e];
                        ov[e] = (__bf16)(xf + dv[e]);
                        sd = fmaf(dv[e], dv[e], sd);
                        sx = fmaf(xf, xf, sx);
                    }
                    *reinterpret_cast<bf16x8*>(out + (size_t)gm * N + gn_e) = ov;
                    if (f32_out) {
                        *reinterpret_cast<f32x4*>(f32_out + (size_t)gm * N + gn_e) = d0;
                        *reinterpret_cast<f32x4*>(f32_out + (size_t)gm * N + gn_e + 4) = d1;
                    }
                }
#pragma unroll
                for (int off = 4; off > 0; off >>= 1) {
                    sd += __shfl_xor(sd, off);
                    sx += __shfl_xor(sx, off);
                }
                // the four wave columns of the tile meet in LDS; one pair per row and tile is written after the loop
                if (e_c8 == 0) nrm[wn * BM + wm * WM + 32 * a + lr] = make_float2(sd, sx);
            } else if (EPI == EPI_SPLITK) {
                if (ok) {
                    // whole products: [part][M][N]; left-over half tiles: [part][half tile][128][256]
                    float* dst = HALF ? f32_out + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * rest_sum_elems() +
                                               (size_t)(gm - m0) * kGN + (gn_e - n0)
                                         : f32_out + ((size_t)blockIdx.y * M + gm) * N + gn_e;
                    *reinterpret_cast<f32x4*>(dst) = d0;
                    *reinterpret_cast<f32x4*>(dst + 4) = d1;
                }
            } else if (ok) {
                float v[8] = {dv[0], dv[1], dv[2], dv[3], dv[4], dv[5], dv[6], dv[7]};
                if (EPI == EPI_QKV_ROPE && gn_e < qkv.Dq + qkv.Dkv) {
                    // the partner columns: in the neighbouring wave's staged block (head size 128) or in this one (64)
                    const float* src = qkv.half == 64 ? reinterpret_cast<const float*>(gemm_smem_raw) + (wave ^ 1) * 32 * kEpiStr +
                                                            lr * kEpiStr + 8 * e_c8
                                                      : stage + lr * kEpiStr + ((8 * e_c8) ^ 32);
                    float partner[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) partner[e] = src[e];
                    rope8(qkv, gm, gn_e, partner, v);
                }
                bf16x8 ov;
#pragma unroll
                for (int e = 0; e < 8; ++e) ov[e] = (__bf16)v[e];
                __bf16* dst = epi_qkv(EPI) ? qkv_dst(out, qkv, gm, gn_e) : out + (size_t)gm * N + gn_e;
                *reinterpret_cast<bf16x8*>(dst) = ov;
            }
        }
        __syncthreads();
    }
    if (EPI == EPI_RESIDUAL_NORM) {
        // row sums of the tile's 256 columns: the wave columns in the fixed order 0..3
        for (int r = tid; r < BM; r += kGThreads) {
            const int gm = m0 + r;
            if (gm < M) {
                float2 t = nrm[r];
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    t.x += nrm[w * BM + r].x;
                    t.y += nrm[w * BM + r].y;
                }
                *reinterpret_cast<float2*>(partials + ((size_t)tile_n * M + gm) * 2) = t;
            }
        }
    }
}

// Epilogue of STAGED rows of a small tile's BN columns, whose KW groups' sums lie in LDS one behind the other (rows of BN + 4 words): a
// thread has 8 consecutive columns of one row (16-byte stores). row_of: the product's row of a staged one; x_of: a thread's p-th piece of x,
// row gm from column gn on.
template <int EPI, int BN, int STAGED, int KW, int THREADS, class RowOf, class XOf>
__device__ __forceinline__ void small_epilogue(const float* stage, int tid, RowOf row_of, int n0, int part, int M, int N,
                                               XOf x_of, __bf16* __restrict__ out, float* __restrict__ partials,
                                               float* __restrict__ split_sums, const QkvOut& qkv) {
    constexpr int STR = BN + 4;
    auto sum8 = [&](const float* src, float* v) {  // eight columns, the K groups' parts in their order
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = src[e];
#pragma unroll
        for (int g = 1; g < KW; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += src[g * STAGED * STR + e];
    };
    if (EPI == EPI_SWIGLU) {
        // lane group of 4 per row and 64 columns: lane c takes gate columns 8c..8c+7 and the up columns 32 + 8c..
        constexpr int LPR = BN / 16, ROWS = THREADS / LPR;
#pragma unroll
        for (int p = 0; p < (STAGED + ROWS - 1) / ROWS; ++p) {
            const int sr = p * ROWS + tid / LPR, l = tid % LPR;
            if (sr >= STAGED) break;
            const int gm = row_of(sr);
            const int gcol = (n0 + 64 * (l / 4)) / 2 + 8 * (l % 4);
            float gv[8], uv[8];
            sum8(&stage[sr * STR + 64 * (l / 4) + 8 * (l % 4)], gv);
            sum8(&stage[sr * STR + 64 * (l / 4) + 8 * (l % 4) + 32], uv);
            if (gm < M && gcol < N / 2) {
                bf16x8 ov;
#pragma unroll
                for (int e = 0; e < 8; ++e) ov[e] = (__bf16)(gv[e] / (1.0f + __expf(-gv[e])) * uv[e]);
                *reinterpret_cast<bf16x8*>(out + (size_t)gm * (N / 2) + gcol) = ov;
            }
        }
    } else {
        constexpr int LPR = BN / 8, ROWS = THREADS / LPR;
#pragma unroll
        for (int p = 0; p < (STAGED + ROWS - 1) / ROWS; ++p) {
            const int sr = p * ROWS + tid / LPR, l = tid % LPR;
            if (sr >= STAGED) break;
            const int gm = row_of(sr), gn = n0 + 8 * l;
            float dv[8];
            sum8(&stage[sr * STR + 8 * l], dv);
            const bool ok = gm < M && gn < N;
            if (EPI == EPI_RESIDUAL_NORM) {
                float sd = 0.f, sx = 0.f;
                if (ok) {
                    const bf16x8 xr = x_of(p, gm, gn);
                    bf16x8 ov;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float xf = (float)xr[e];
                        ov[e] = (__bf16)(xf + dv[e]);
                        sd = fmaf(dv[e], dv[e], sd);
                        sx = fmaf(xf, xf, sx);
                    }
                    *reinterpret_cast<bf16x8*>(out + (size_t)gm * N + gn) = ov;
                }
                if (partials) {
#pragma unroll
                    for (int off = 4; off > 0; off >>= 1) {
                        sd += __shfl_xor(sd, off);
                        sx += __shfl_xor(sx, off);
                    }
                    if (l % 8 == 0 && ok)
                        *reinterpret_cast<float2*>(partials + ((size_t)(gn / 64) * M + gm) * 2) = make_float2(sd, sx);
                }
            } else if (EPI == EPI_SPLITK) {
                if (ok) {
                    float* dst = split_sums + ((size_t)part * M + gm) * N + gn;
                    *reinterpret_cast<f32x4*>(dst) = f32x4{dv[0], dv[1], dv[2], dv[3]};
                    *reinterpret_cast<f32x4*>(dst + 4) = f32x4{dv[4], dv[5], dv[6], dv[7]};
                }
            } else if (ok) {
                if (EPI == EPI_QKV_ROPE && gn < qkv.Dq + qkv.Dkv) {  // a head lies in one tile (the launcher's choice)
                    float partner[8];
                    sum8(&stage[sr * STR + ((8 * l) ^ qkv.half)], partner);
                    rope8(qkv, gm, gn, partner, dv);
                }
                bf16x8 ov;
#pragma unroll
                for (int e = 0; e < 8; ++e) ov[e] = (__bf16)dv[e];
                __bf16* dst = epi_qkv(EPI) ? qkv_dst(out, qkv, gm, gn) : out + (size_t)gm * N + gn;
                *reinterpret_cast<bf16x8*>(dst) = ov;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same product on small tiles: BM x BN (64, 128 or 192 x 64 or 128), KW groups of 4 waves in 2 x 2. One workgroup per compute unit (96 to
// 144 KB of LDS), of the second 128 x 128 form two.
// Few rows leave the 256 x 256 tiles with a handful of workgroups, which then have to be cut along K and summed in a
// second pass: with 177 rows the fp32 sums written and read back were more bytes than the weight. Small tiles fill the
// chip without that: 177 rows of K = N = 3584 take 15.5 us instead of 26, 333 rows of 512 4.8 instead of 15 (small_plan).
// The KW groups share a workgroup's tile and split its K steps (group kg: steps kg, kg + KW, ...), each with NS
// operand stages of its own; their sums meet in the epilogue, in the order of kg. One barrier per round: a step is
// multiplied from registers while the next one's fragments are read and the step NS ahead is requested. What bounds it: per
// 64 x 64 step 48 KB through LDS (16 written, 32 read), 384 cycles of it, of the 500 that a step takes; more stages or K
// groups do not shorten it.
// 128 x 128 tiles, one workgroup per unit (KW 1, NS 3): four waves, one per SIMD, so what a wave does one after the other is not covered
// by another: requests, fragment reads and MFMAs are dealt out among one another as the large tiles do it, with two steps of lead for
// the requests to land in. Per step 96 KB through LDS and 512 cycles each of requests and MFMAs, 0.45 us. As two K groups of two
// stages, each requesting a step at once and ahead of its fragment reads, a step took 0.50 us on cached weights and 0.70 on weights from memory,
// which then had one round to land: K = N = 3584 with a row norm's launch, weights from memory, 640 rows 48.5 -> 44.0 us, 995 48.8 -> 44.7, 1150
// 50.6 -> 46.5; 4096 700 rows 52.9 -> 44.9; cached 640 34.5 -> 32.9, 995 the same. Four or five stages are no faster. (Four waves
// that request and read in turn, without the interleaving: 0.66 us a step whatever the stages.)
// Two workgroups per unit (NS 2) cover each other's gaps and keep the plain order: a step has one round to land, so it is requested
// first (interleaved: 1400 rows 47.5 -> 46.1 us, 2120 57.0 -> 57.8).
// Row norms (EPI_RESIDUAL_NORM) come as one pair per 64 columns, as a wave column of the large tiles sums them;
// fold_partials_kernel adds them up to 256 columns for callers that see them.
// ------------------------------------------------------------------------------------------------
constexpr size_t small_smem_bytes(int BM, int BN, int KW, int NS) { return (size_t)KW * NS * (BM + BN) * kGK * sizeof(__bf16); }

// 192 rows: with x in flight as well the registers of two waves per SIMD are too few (1153 rows of 3584 48.0 us for 44.0), while the other
// epilogues' loops are the faster ones with them (front end, 1000 rows, 42.4 us for 52.1).
template <int EPI, int BM, int BN, int KW, int NS>
__global__ __launch_bounds__(KW * kSWaves * kWave, BM > 128 && EPI == EPI_RESIDUAL_NORM ? 1 : 2) void gemm_small_kernel(const __bf16* __restrict__ A, const __bf16* __restrict__ B,
                                                                  int M, int K, int N, const __bf16* __restrict__ x,
                                                                  __bf16* __restrict__ out, float* __restrict__ partials,
                                                                  float* __restrict__ split_sums, int mt, int tiles, int parts,
                                                                  int ksteps, int ksteps_per_split, QkvOut qkv) {
    constexpr int kThreads = KW * kSWaves * kWave;
    constexpr int RB = BM / 32, CB = BN / 32;  // 16-row and 16-column blocks of a wave
    constexpr int kAElems = BM * kGK, kStageElems = (BM + BN) * kGK;
    constexpr int STR = BN + 4;
    static_assert(small_smem_bytes(BM, BN, KW, NS) >= KW * 64 * STR * sizeof(float), "the epilogue's 64 staged rows fit");
    extern __shared__ __attribute__((aligned(16))) unsigned char small_smem_raw[];
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int kg = KW == 1 ? 0 : wave_all / kSWaves, wave = wave_all % kSWaves;  // K group, wave inside it
    const int wm = wave / 2, wn = wave % 2;
    __bf16* smem = reinterpret_cast<__bf16*>(small_smem_raw) + kg * NS * kStageElems;  // this group's stages
    int idx, part;
    if (!small_work_of((int)blockIdx.x, tiles, EPI == EPI_SPLITK ? parts : 1, idx, part)) return;  // padding: the whole workgroup
    const int tile_m = idx % mt, tile_n = idx / mt;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int ks0 = EPI == EPI_SPLITK ? part * ksteps_per_split : 0;
    const int n_ksteps = EPI == EPI_SPLITK ? min(ksteps_per_split, ksteps - ks0) : ksteps;
    const int n_rounds = (n_ksteps + KW - 1) / KW, n_mine = (n_ksteps - kg + KW - 1) / KW;  // group kg: steps kg, kg + KW, ...

    f32x4 acc[RB][CB];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    constexpr int ADMA = small_adma(BM), BDMA = small_bdma(BN);
    uint32_t a_off[ADMA], b_off[BDMA];
#pragma unroll
    for (int i = 0; i < ADMA; ++i) {
        const int row = small_a_row(wave, i, lane, BM);
        a_off[i] = gemm_a_off(m0, M, K, row, gemm_a_lchunk(row, lane));
    }
#pragma unroll
    for (int i = 0; i < BDMA; ++i) {
        const int row = small_b_row(wave, i, lane, BN);
        b_off[i] = gemm_b_off(n0, N, row, small_b_lchunk(row, lane, BN));
    }
    const char* a_base = reinterpret_cast<const char*>(A + gemm_a_base_elem(m0, M, K, ks0 + kg));
    const char* b_base = reinterpret_cast<const char*>(B + gemm_b_base_elem(n0, N, ks0 + kg));
    const size_t b_step = gemm_b_step_bytes(N);
    const uint32_t lds_a = lds_addr(smem) + (uint32_t)(wave * ADMA * 1024);
    const uint32_t lds_b = lds_addr(smem) + (uint32_t)(kAElems * 2 + wave * BDMA * 1024);
    auto request = [&](int stage) {  // a group's K steps are requested strictly in order
        const uint32_t so = (uint32_t)(stage * kStageElems * 2);
#pragma unroll
        for (int i = 0; i < ADMA; ++i) dma_load16(a_base, a_off[i], lds_a + so + i * 1024);
#pragma unroll
        for (int i = 0; i < BDMA; ++i) dma_load16(b_base, b_off[i], lds_b + so + i * 1024);
        a_base += KW * gemm_a_step_bytes();
        b_base += KW * b_step;
    };
    const int fi = lane % 16, fg = lane / 16;
    struct Frags {  // operands of one K step
        bf16x8 a[2][RB], b[2][CB];
    };
    auto read_a = [&](int st, int ks, int a) {
        const int row = wm * (BM / 2) + 16 * a + fi;
        return *reinterpret_cast<const bf16x8*>(&smem[st * kStageElems + row * kGK + ((4 * ks + fg) ^ ((row / 2) % 8)) * 8]);
    };
    auto read_b = [&](int st, int ks, int b) {
        const __bf16* sb = smem + st * kStageElems + kAElems;
        const int krow = 32 * ks + 8 * fg + fi / 4;  // and krow + 4: the same swizzle
        const int col = wn * (BN / 2) + 16 * b + 4 * (fi % 4);
        const int scol = ((col / 8) ^ small_b_swz(krow, BN)) * 8 + col % 8;
        const s16x4 lo = lds_read_tr16(&sb[krow * BN + scol]);
        const s16x4 hi = lds_read_tr16(&sb[(krow + 4) * BN + scol]);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_slice = [&](int st, int ks, bf16x8* af, bf16x8* bfr) {
#pragma unroll
        for (int b = 0; b < CB; ++b) bfr[b] = read_b(st, ks, b);
#pragma unroll
        for (int a = 0; a < RB; ++a) af[a] = read_a(st, ks, a);
    };
    auto read_frags = [&](int st, Frags& f) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) read_slice(st, ks, f.a[ks], f.b[ks]);
    };
    auto mfmas = [&](const Frags& f) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int a = 0; a < RB; ++a)
#pragma unroll
                for (int b = 0; b < CB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[ks][a], f.b[ks][b], acc[a][b], 0, 0, 0);
    };
    // barrier that orders LDS traffic only: the tile requests in flight are not waited for
    auto lds_barrier = [] {
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // this wave's fragment reads are in registers
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    constexpr int kStepLoads = ADMA + BDMA;
    // One workgroup per unit: the epilogue's x is asked for during the K loop, all of it at once. In the epilogue nothing covers its way from
    // memory, once per 64 rows (K = N = 3584 with attention and score, 640 rows 51.1 -> 50.4 us, with x and weights from memory 60.6 -> 57.5,
    // 1000 70.6 -> 67.0). The waits of the steps count the tiles' requests alone: with x in flight they wait for more than they need, never
    // for less. Two workgroups per unit cover it, and asking early costs them 2 to 3 % (2120 rows 112.7 -> 116.1).
    constexpr bool kEarlyX = EPI == EPI_RESIDUAL_NORM && NS > 2 && KW == 1;
    constexpr int kXRows = kThreads / (BN / 8), XP = 64 / kXRows;  // small_epilogue's rows at a time
    auto epi_row = [&](int a, int sr) { return m0 + (sr / 32) * (BM / 2) + 32 * a + sr % 32; };
    bf16x8 xr[kEarlyX ? BM / 64 : 1][kEarlyX ? XP : 1];
    auto load_x = [&] {  // rows and columns beyond the end: the last ones, never used
        if constexpr (kEarlyX)
#pragma unroll
            for (int a = 0; a < BM / 64; ++a)
#pragma unroll
                for (int p = 0; p < XP; ++p)
                    xr[a][p] = *reinterpret_cast<const bf16x8*>(x + (size_t)min(epi_row(a, p * kXRows + tid / (BN / 8)), M - 1) * N +
                                                                min(n0 + 8 * (tid % (BN / 8)), N - 8));
    };
    for (int j = 0; j < min(NS, n_mine); ++j) request(j);
    if (n_mine >= NS)
        dma_wait_keep<(NS - 1) * kStepLoads>();  // the first step has landed
    else
        dma_wait();
    lds_barrier();
    Frags f[2];
    int st = 0;  // t % NS
    if constexpr (NS > 2 && KW == 1) {
        // The large tiles' round (gemm_mfma_kernel): two 32-wide slices a step, the fragments of a slice read while the MFMAs of the one
        // before it run; the wait for the next step and the barrier sit before the second slice's MFMAs, among which the step
        // NS ahead is requested into the stage that every wave has read by then. The last NS steps request nothing.
        constexpr int RD = RB + 2 * CB, MF = RB * CB, UNITS = RB + CB;
        constexpr int kRequestEvery = MF / kStepLoads;
        static_assert(kRequestEvery >= 1 && RD <= MF && MF <= 2 * RD, "reads and requests of a half step fit between its MFMAs");
        auto second_half = [&](int st_next, bool ask) {
            const uint32_t so = (uint32_t)(st * kStageElems * 2);
#pragma unroll
            for (int m = 0; m < MF; ++m) {
#pragma unroll
                for (int l = 0; l < kStepLoads; ++l)
                    if (m == l * kRequestEvery && ask) {
                        if (l < ADMA) dma_load16(a_base, a_off[l], lds_a + so + l * 1024);
                        else dma_load16(b_base, b_off[l - ADMA], lds_b + so + (l - ADMA) * 1024);
                    }
#pragma unroll
                for (int u = 0; u < UNITS; ++u)  // fragment u before the first MFMA m with u * MF <= m * UNITS
                    if (u * MF <= m * UNITS && (m == 0 || u * MF > (m - 1) * UNITS)) {
                        if (u < CB) f[0].b[0][u] = read_b(st_next, 0, u);
                        else f[0].a[0][u - CB] = read_a(st_next, 0, u - CB);
                    }
                acc[m / CB][m % CB] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[0].a[1][m / CB], f[0].b[1][m % CB], acc[m / CB][m % CB], 0, 0, 0);
                if (m % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
            if (ask) {
                a_base += gemm_a_step_bytes();
                b_base += b_step;
            }
        };
        auto step = [&](bool ask) {
            const int st_next = st + 1 == NS ? 0 : st + 1;
            read_slice(st, 1, f[0].a[1], f[0].b[1]);
#pragma unroll
            for (int a = 0; a < RB; ++a)
#pragma unroll
                for (int b = 0; b < CB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[0].a[0][a], f[0].b[0][b], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 2 * RD - MF; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
#pragma unroll
            for (int i = 0; i < MF - RD; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            if (ask) dma_wait_keep<(NS - 2) * kStepLoads>();
            else dma_wait();
            lds_barrier();
            second_half(st_next, ask);
            st = st_next;
        };
        if (n_ksteps > 0) read_slice(0, 0, f[0].a[0], f[0].b[0]);
        int kt = 0;
        const int x_step = max(0, n_ksteps - NS - 2);  // as the last steps are requested
        if (n_ksteps <= NS) load_x();
        for (; kt + NS < n_ksteps; ++kt) {
            if (kt == x_step) load_x();
            step(true);
        }
        for (; kt < n_ksteps; ++kt) step(false);
    } else {
        // Round t multiplies its step from registers while the next step's fragments are read. Before barrier t this wave's
        // part of step t + 1 has landed (the NS - 2 steps after it may be in flight) and its fragments of step t are in
        // registers; so after it every wave's part of step t + 1 is there, and the stage of step t takes step t + NS.
        // Every group passes the same number of barriers.
        if (n_mine > 0) read_frags(0, f[0]);
        auto round = [&](int t, const Frags& cur, Frags& next) {
            if (t + NS <= n_mine)
                dma_wait_keep<(NS - 2) * kStepLoads>();
            else
                dma_wait();
            lds_barrier();
            if (t + NS < n_mine) request(st);
            st = st + 1 == NS ? 0 : st + 1;
            if (t + 1 < n_mine) read_frags(st, next);
            if (t < n_mine) mfmas(cur);
        };
        for (int t = 0; t < n_rounds; t += 2) {
            round(t, f[0], f[1]);
            if (t + 1 < n_rounds) round(t + 1, f[1], f[0]);
        }
    }
    __syncthreads();  // the operand stages are free and are reused

    // Epilogue, 32 rows of either wave row at a time: the accumulators go to LDS first.
    float* stage = reinterpret_cast<float*>(small_smem_raw);
#pragma unroll
    for (int a = 0; a < BM / 64; ++a) {
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r)  // accumulator register r of a 16x16 block: row 4 g + r, column i
                    stage[(64 * kg + 32 * wm + 16 * sb + 4 * fg + r) * STR + wn * (BN / 2) + 16 * b + fi] = acc[2 * a + sb][b][r];
        __syncthreads();
        small_epilogue<EPI, BN, 64, KW, kThreads>(
            stage, tid, [&](int sr) { return epi_row(a, sr); }, n0, part, M, N,
            [&](int p, int gm, int gn) {
                if constexpr (kEarlyX) return xr[a][p];
                else return *reinterpret_cast<const bf16x8*>(x + (size_t)gm * N + gn);
            },
            out, partials, split_sums, qkv);
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------------
// The same product for the fewest rows: 16 RB x 64 tiles whose 8 waves split the K steps and share nothing until the end: wave w takes
// the steps w, w + 8, ... of the whole tile, fetches their operands into LDS of its own (one stage, A and B) and asks for the next
// step as soon as this one's fragments are in registers. No barrier in the loop, every byte of a stage is read once, and the
// lowest tile that a launch's workgroups take in one round is used (few_tile_plan).
// A compute unit has at most 64 KB in flight, and a step's first bytes come from the last-level cache or memory, so a step takes 1.0 to 1.7 us
// whatever the tile, of a launch of 2.5 to 4.5 us. K = N = 3584, weight in the last-level cache, us, the forms above / this: 177 rows
// 15.1 / 13.0, 16 in four K parts with their second pass 12.6 / 10.8; 333 rows of 512 x 512 4.0 / 3.2, of 1024 x 1024 5.4 / 4.5. Two stages, 5 or 10
// waves, and fragments straight from memory (22 us; 8-byte loads have half the rate) are no faster; all 177 rows on one 192-row tile in four K parts
// took 16.7 without the second pass.
// ------------------------------------------------------------------------------------------------
template <int EPI, int RB>
__global__ __launch_bounds__(kFewTileWaves * kWave, 2) void gemm_few_kernel(const __bf16* __restrict__ A, const __bf16* __restrict__ B, int M, int K,
                                                                  int N, const __bf16* __restrict__ x, __bf16* __restrict__ out,
                                                                  float* __restrict__ partials, float* __restrict__ split_sums, int mt,
                                                                  int tiles, int parts, int ksteps, int ksteps_per_split, QkvOut qkv) {
    constexpr int BM = 16 * RB, BN = kFewTileN, CB = BN / 16, W = kFewTileWaves;
    constexpr int kAElems = BM * kGK, kStageElems = (BM + BN) * kGK, STR = BN + 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char few_tile_smem_raw[];
    const int tid = threadIdx.x, lane = tid % kWave, fi = lane % 16, fg = lane / 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    int idx, part;
    if (!small_work_of((int)blockIdx.x, tiles, EPI == EPI_SPLITK ? parts : 1, idx, part)) return;  // padding: the whole workgroup
    const int m0 = (idx % mt) * BM, n0 = (idx / mt) * BN;
    const int ks0 = EPI == EPI_SPLITK ? part * ksteps_per_split : 0;
    const int n_ksteps = EPI == EPI_SPLITK ? min(ksteps_per_split, ksteps - ks0) : ksteps, n_mine = (n_ksteps - wave + W - 1) / W;
    __bf16* sa = reinterpret_cast<__bf16*>(few_tile_smem_raw) + wave * kStageElems;  // this wave's stage
    __bf16* sb = sa + kAElems;

    f32x4 acc[RB][CB];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int ADMA = BM / 8, BDMA = kGK / 8;  // load instructions of a step, 8 rows each
    uint32_t a_off[ADMA], b_off[BDMA];
#pragma unroll
    for (int i = 0; i < ADMA; ++i) a_off[i] = gemm_a_off(m0, M, K, few_tile_row(i, lane), gemm_a_lchunk(few_tile_row(i, lane), lane));
#pragma unroll
    for (int i = 0; i < BDMA; ++i) b_off[i] = gemm_b_off(n0, N, few_tile_row(i, lane), small_b_lchunk(few_tile_row(i, lane), lane, BN));
    const char* a_base = reinterpret_cast<const char*>(A + gemm_a_base_elem(m0, M, K, ks0 + wave));
    const char* b_base = reinterpret_cast<const char*>(B + gemm_b_base_elem(n0, N, ks0 + wave));
    const size_t b_step = W * gemm_b_step_bytes(N);
    const uint32_t lds_a = lds_addr(sa), lds_b = lds_addr(sb);
    auto request = [&] {  // the wave's steps strictly in order
#pragma unroll
        for (int i = 0; i < BDMA; ++i) dma_load16(b_base, b_off[i], lds_b + i * 1024);
#pragma unroll
        for (int i = 0; i < ADMA; ++i) dma_load16(a_base, a_off[i], lds_a + i * 1024);
        a_base += W * gemm_a_step_bytes();
        b_base += b_step;
    };
    if (n_mine > 0) request();
    for (int t = 0; t < n_mine; ++t) {
        dma_wait();
        wave_sync_lds();
        bf16x8 af[2][RB], bfr[2][CB];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const int krow = 32 * ks + 8 * fg + fi / 4;  // and krow + 4: the same swizzle
                const int col = 16 * b + 4 * (fi % 4), scol = ((col / 8) ^ small_b_swz(krow, BN)) * 8 + col % 8;
                const s16x4 lo = lds_read_tr16(&sb[krow * BN + scol]);
                const s16x4 hi = lds_read_tr16(&sb[(krow + 4) * BN + scol]);
                bfr[ks][b] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
#pragma unroll
            for (int a = 0; a < RB; ++a) {
                const int row = 16 * a + fi;
                af[ks][a] = *reinterpret_cast<const bf16x8*>(&sa[row * kGK + ((4 * ks + fg) ^ ((row / 2) % 8)) * 8]);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // the stage is in registers
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < n_mine) request();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int a = 0; a < RB; ++a)
#pragma unroll
                for (int b = 0; b < CB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks][a], bfr[ks][b], acc[a][b], 0, 0, 0);
    }
    __syncthreads();  // every wave's stage is read and nothing is in flight
    float* stage = reinterpret_cast<float*>(few_tile_smem_raw);
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)  // accumulator register r of a 16x16 block: row 4 g + r, column i
                stage[(BM * wave + 16 * a + 4 * fg + r) * STR + 16 * b + fi] = acc[a][b][r];
    __syncthreads();
    small_epilogue<EPI, BN, BM, W, W * kWave>(stage, tid, [&](int sr) { return m0 + sr; }, n0, part, M, N,
        [&](int, int gm, int gn) { return *reinterpret_cast<const bf16x8*>(x + (size_t)gm * N + gn); }, out, partials, split_sums, qkv);
}

// Row norms of a small-tile product, kNormFold neighbouring columns of pairs to one: fine[cols][M] -> partials[P][M].
__global__ __launch_bounds__(256) void fold_partials_kernel(const float2* __restrict__ fine, int cols, int M,
                                                            float2* __restrict__ partials) {
    const int row = blockIdx.x * 256 + threadIdx.x, c0 = blockIdx.y * kNormFold;
    if (row >= M) return;
    float2 v[kNormFold];
#pragma unroll
    for (int c = 0; c < kNormFold; ++c) v[c] = c0 + c < cols ? fine[(size_t)(c0 + c) * M + row] : make_float2(0.f, 0.f);
#pragma unroll
    for (int c = 1; c < kNormFold; ++c) {
        v[0].x += v[c].x;
        v[0].y += v[c].y;
    }
    partials[(size_t)blockIdx.y * M + row] = v[0];
}

// Second pass of a split-K product: adds the S split sums of sums[S][M][N] in the order s = 0..S-1 and applies
// the epilogue EPI (same results layout as the one-pass kernel). A wave works on one row; a lane owns 8
// consecutive columns, so the 32 lanes of a 256-column tile hold that tile's row sums for the norm partials.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ sums, int S, int M, int N,
                                                            const __bf16* __restrict__ x, __bf16* __restrict__ out,
                                                            float* __restrict__ partials, QkvOut qkv) {
    const int lane = threadIdx.x % kWave;
    const int wave_global = (int)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) / kWave);
    if (EPI == EPI_SWIGLU) {
        // 4 lanes per 64-column group (32 gate + 32 up columns): 16 groups = 1024 input columns per wave
        const int segs = (N + 1023) / 1024;
        const int row = wave_global / segs, seg = wave_global % segs;
        if (row >= M) return;
        const int grp = seg * 16 + lane / 4, c = lane % 4;
        const int gcol = grp * 64 + 8 * c;  // gate columns gcol..gcol+7, up columns gcol+32..
        if (gcol >= N) return;
        float g[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, u[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int sp = 0; sp < S; ++sp) {
            const float* src = sums + ((size_t)sp * M + row) * N + gcol;
            const f32x4 g0 = *reinterpret_cast<const f32x4*>(src), g1 = *reinterpret_cast<const f32x4*>(src + 4);
            const f32x4 u0 = *reinterpret_cast<const f32x4*>(src + 32), u1 = *reinterpret_cast<const f32x4*>(src + 36);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                g[e] += g0[e];
                g[4 + e] += g1[e];
                u[e] += u0[e];
                u[4 + e] += u1[e];
            }
        }
        bf16x8 ov;
#pragma unroll
        for (int e = 0; e < 8; ++e) ov[e] = (__bf16)(g[e] / (1.0f + __expf(-g[e])) * u[e]);
        *reinterpret_cast<bf16x8*>(out + (size_t)row * (N / 2) + grp * 32 + 8 * c) = ov;
        return;
    }
    const int segs = (N + 511) / 512;  // 8 groups of 64 columns per wave
    const int row = wave_global / segs, seg = wave_global % segs;
    if (row >= M) return;
    const int grp = seg * 8 + lane / 8;
    const int col = grp * 64 + 8 * (lane % 8);
    const bool ok = col < N;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (ok) {
        for (int sp = 0; sp < S; ++sp) {
            const float* src = sums + ((size_t)sp * M + row) * N + col;
            const f32x4 a0 = *reinterpret_cast<const f32x4*>(src), a1 = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[e] += a0[e];
                acc[4 + e] += a1[e];
            }
        }
    }
    if (EPI == EPI_STORE || epi_qkv(EPI)) {
        if (EPI == EPI_QKV_ROPE) {  // the partner columns belong to the lane half / 8 away
            float partner[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) partner[e] = __shfl_xor(acc[e], qkv.half / 8);
            if (ok && col < qkv.Dq + qkv.Dkv) rope8(qkv, row, col, partner, acc);
        }
        if (ok) {
            bf16x8 ov;
#pragma unroll
            for (int e = 0; e < 8; ++e) ov[e] = (__bf16)acc[e];
            __bf16* dst = epi_qkv(EPI) ? qkv_dst(out, qkv, row, col) : out + (size_t)row * N + col;
            *reinterpret_cast<bf16x8*>(dst) = ov;
        }
        return;
    }
    float sd = 0.f, sx = 0.f;
    if (ok) {
        const bf16x8 xr = *reinterpret_cast<const bf16x8*>(x + (size_t)row * N + col);
        bf16x8 ov;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float xf = (float)xr[e];
            ov[e] = (__bf16)(xf + acc[e]);
            sd = fmaf(acc[e], acc[e], sd);
            sx = fmaf(xf, xf, sx);
        }
        *reinterpret_cast<bf16x8*>(out + (size_t)row * N + col) = ov;
    }
    // one partial pair per 256-column tile, as the one-pass kernel writes them: the 32 lanes of a tile in fixed order
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
        sd += __shfl_xor(sd, off);
        sx += __shfl_xor(sx, off);
    }
    const int tile = seg * 2 + lane / 32;
    if (lane % 32 == 0 && tile < (N + kGN - 1) / kGN)
        *reinterpret_cast<float2*>(partials + ((size_t)tile * M + row) * 2) = make_float2(sd, sx);
}

// Second pass over left-over half tiles that were cut along K: adds sums[part][half tile][128][256] in the order of the
// parts and applies the epilogue EPI. 8 columns per lane: 32 lanes per row (gating: 16, with the gate and up columns of 8
// features each).
template <int EPI>
__global__ __launch_bounds__(256) void rest_reduce_kernel(const float* __restrict__ sums, int parts, int M, int N,
                                                          const __bf16* __restrict__ x, __bf16* __restrict__ out,
                                                          float* __restrict__ partials, GemmLaunch L, QkvOut qkv) {
    constexpr int LPR = EPI == EPI_SWIGLU ? 16 : 32, ROWS = 256 / LPR;
    const int half = (int)blockIdx.x, lr = (int)blockIdx.y * ROWS + (int)threadIdx.x / LPR, l = (int)threadIdx.x % LPR;
    int tile_m, tile_n;
    gemm_tile_of(L.first_tile + half / 2, L.mt, L.nt, L.plain != 0, tile_m, tile_n);
    const int gm = tile_m * kGM + (half % 2) * (kGM / 2) + lr, n0 = tile_n * kGN;
    const size_t part_stride = (size_t)gridDim.x * rest_sum_elems();
    auto add_parts = [&](int col, float* v) {
        const float* src = sums + (size_t)half * rest_sum_elems() + (size_t)lr * kGN + col;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.f;
#pragma unroll 4
        for (int p = 0; p < parts; ++p) {
            const f32x4 a0 = *reinterpret_cast<const f32x4*>(src + p * part_stride);
            const f32x4 a1 = *reinterpret_cast<const f32x4*>(src + p * part_stride + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] += a0[e];
                v[4 + e] += a1[e];
            }
        }
    };
    if (EPI == EPI_SWIGLU) {
        const int col = 64 * (l / 4) + 8 * (l % 4), gcol = (n0 + 64 * (l / 4)) / 2 + 8 * (l % 4);
        if (gm >= M || gcol >= N / 2) return;
        float g[8], u[8];
        add_parts(col, g);
        add_parts(col + 32, u);
        bf16x8 ov;
#pragma unroll
        for (int e = 0; e < 8; ++e) ov[e] = (__bf16)(g[e] / (1.0f + __expf(-g[e])) * u[e]);
        *reinterpret_cast<bf16x8*>(out + (size_t)gm * (N / 2) + gcol) = ov;
        return;
    }
    const int gn = n0 + 8 * l;
    const bool ok = gm < M && gn < N;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, sd = 0.f, sx = 0.f;
    if (ok) add_parts(8 * l, v);
    if (EPI == EPI_QKV_ROPE) {  // the partner columns belong to the lane half / 8 away
        float partner[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) partner[e] = __shfl_xor(v[e], qkv.half / 8);
        if (ok && gn < qkv.Dq + qkv.Dkv) rope8(qkv, gm, gn, partner, v);
    }
    if (ok) {
        bf16x8 ov;
        if (EPI == EPI_RESIDUAL_NORM) {
            const bf16x8 xr = *reinterpret_cast<const bf16x8*>(x + (size_t)gm * N + gn);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float xf = (float)xr[e];
                ov[e] = (__bf16)(xf + v[e]);
                sd = fmaf(v[e], v[e], sd);
                sx = fmaf(xf, xf, sx);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) ov[e] = (__bf16)v[e];
        }
        __bf16* dst = epi_qkv(EPI) ? qkv_dst(out, qkv, gm, gn) : out + (size_t)gm * N + gn;
        *reinterpret_cast<bf16x8*>(dst) = ov;
    }
    if (EPI == EPI_RESIDUAL_NORM) {
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            sd += __shfl_xor(sd, off);
            sx += __shfl_xor(sx, off);
        }
        if (l == 0 && gm < M) *reinterpret_cast<float2*>(partials + ((size_t)tile_n * M + gm) * 2) = make_float2(sd, sx);
    }
}

// h = x / sqrt(mean(x^2) + 1e-6), unit gain; one wave per row. Rows of up to 512 * CH elements are held in
// registers between the two passes (one read of x); longer rows are read twice (CH = 0).
// HALF > 0: the wave also leaves the cosine and sine of its row's HALF rotary angles pos * theta^(-2i / (2 HALF)) in
// table[row][HALF], from fp64 angles as rope_qk_kernel forms them; the arithmetic hides behind the row's loads.
struct RopeTable {
    const int32_t* pos;
    float2* table;
    double neg_log2_theta_2_over_dh;
};
template <int CH, int HALF>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const __bf16* __restrict__ x, int n, int d,
                                                      __bf16* __restrict__ hout, RopeTable rope) {
    const int row = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int lane = threadIdx.x % kWave;
    if (row >= n) return;
    const __bf16* xr = x + (size_t)row * d;
    __bf16* hr = hout + (size_t)row * d;
    float ss = 0.f;
    auto leave_angles = [&] {
        if (HALF > 0 && lane < HALF) {
            double a = (double)rope.pos[row] * exp2((double)lane * rope.neg_log2_theta_2_over_dh);
            a -= 6.283185307179586476925286766559 * rint(a * 0.15915494309189533576888376337251);
            double s, c;
            sincos(a, &s, &c);
            rope.table[(size_t)row * HALF + lane] = make_float2((float)c, (float)s);
        }
    };
    if (CH > 0) {
        bf16x8 v[CH > 0 ? CH : 1];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = (i * kWave + lane) * 8;
            if (c < d) v[i] = *reinterpret_cast<const bf16x8*>(xr + c);
        }
        leave_angles();  // while the row is on its way
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = (i * kWave + lane) * 8;
            if (c < d) {
#pragma unroll
                for (int e = 0; e < 8; ++e) ss = fmaf((float)v[i][e], (float)v[i][e], ss);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
        const float inv = 1.0f / sqrtf(ss / (float)d + 1e-6f);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = (i * kWave + lane) * 8;
            if (c < d) {
                bf16x8 ov;
#pragma unroll
                for (int e = 0; e < 8; ++e) ov[e] = (__bf16)((float)v[i][e] * inv);
                *reinterpret_cast<bf16x8*>(hr + c) = ov;
            }
        }
        return;
    }
    leave_angles();
    for (int c = lane * 8; c < d; c += kWave * 8) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf((float)v[e], (float)v[e], ss);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    const float inv = 1.0f / sqrtf(ss / (float)d + 1e-6f);
    for (int c = lane * 8; c < d; c += kWave * 8) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c);
        bf16x8 ov;
#pragma unroll
        for (int e = 0; e < 8; ++e) ov[e] = (__bf16)((float)v[e] * inv);
        *reinterpret_cast<bf16x8*>(hr + c) = ov;
    }
}

template <int HALF>
static void launch_rmsnorm(const __bf16* x, int n, int d, __bf16* h, const RopeTable& rope, hipStream_t s) {
    const int blocks = (int)(((size_t)n * kWave + 255) / 256);
    if (d <= 512 * 4)
        hipLaunchKernelGGL((rmsnorm_kernel<4, HALF>), dim3(blocks), dim3(256), 0, s, x, n, d, h, rope);
    else if (d <= 512 * 8)
        hipLaunchKernelGGL((rmsnorm_kernel<8, HALF>), dim3(blocks), dim3(256), 0, s, x, n, d, h, rope);
    else
        hipLaunchKernelGGL((rmsnorm_kernel<0, HALF>), dim3(blocks), dim3(256), 0, s, x, n, d, h, rope);
}
static void launch_rmsnorm(const __bf16* x, int n, int d, __bf16* h, hipStream_t s) {
    launch_rmsnorm<0>(x, n, d, h, RopeTable{nullptr, nullptr, 0.0}, s);
}

int norm_partials_per_row(int d, int dtype) {
    if (dtype == DASH_F32) return (d + kF32TileN - 1) / kF32TileN;
    return (d + kGN - 1) / kGN;
}

// Number of compute units of the current device (queried once; the library serves one GPU).
int compute_units() {
    static const int n = [] {
        int dev = 0, cu = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 0;
        if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        return cu;
    }();
    return n;
}

// One-time launch attribute of every instantiation of the MFMA kernel: its dynamic LDS (112 to 144 KB).
template <int EPI, int RB>
static hipError_t set_gemm_lds_size(hipError_t e) {
    return e != hipSuccess ? e : hipFuncSetAttribute((const void*)gemm_mfma_kernel<EPI, RB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)gemm_smem_bytes(RB));
}
template <int EPI>
static hipError_t set_gemm_lds_sizes() {
    hipError_t e = set_gemm_lds_size<EPI, 4>(set_gemm_lds_size<EPI, 8>(hipSuccess));
    if constexpr (EPI != EPI_SPLITK) e = set_gemm_lds_size<EPI, 6>(set_gemm_lds_size<EPI, 7>(e));
    return e;
}

template <int EPI, int F>
static hipError_t set_small_lds_size() {
    constexpr SmallForm f = kSmallForms[F];
    return hipFuncSetAttribute((const void*)gemm_small_kernel<EPI, f.BM, f.BN, f.KW, f.NS>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)small_smem_bytes(f.BM, f.BN, f.KW, f.NS));
}
template <int EPI, int RB>
static hipError_t set_few_tile_lds_size(hipError_t e) {
    return e != hipSuccess ? e : hipFuncSetAttribute((const void*)gemm_few_kernel<EPI, RB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)few_tile_smem_bytes(16 * RB));
}
template <int EPI>
static hipError_t set_few_tile_lds_sizes() {
    return set_few_tile_lds_size<EPI, 3>(set_few_tile_lds_size<EPI, 2>(set_few_tile_lds_size<EPI, 1>(hipSuccess)));
}
template <int EPI>
static hipError_t set_small_lds_sizes() {
    hipError_t e = set_few_tile_lds_sizes<EPI>();
    if (e == hipSuccess) e = set_small_lds_size<EPI, 0>();
    if (e == hipSuccess) e = set_small_lds_size<EPI, 1>();
    if (e == hipSuccess) e = set_small_lds_size<EPI, 2>();
    if (e == hipSuccess) e = set_small_lds_size<EPI, 3>();
    if (e == hipSuccess) e = set_small_lds_size<EPI, kTallForm>();
    return e;
}

dash_status init_gemm_kernels() {
    static const hipError_t err = [] {
        hipError_t e = set_gemm_lds_sizes<EPI_RESIDUAL_NORM>();
        if (e == hipSuccess) e = set_gemm_lds_sizes<EPI_STORE>();
        if (e == hipSuccess) e = set_gemm_lds_sizes<EPI_SWIGLU>();
        if (e == hipSuccess) e = set_gemm_lds_sizes<EPI_SPLITK>();
        if (e == hipSuccess) e = set_gemm_lds_sizes<EPI_QKV>();
        if (e == hipSuccess) e = set_gemm_lds_sizes<EPI_QKV_ROPE>();
        if (e == hipSuccess) e = set_small_lds_sizes<EPI_QKV_ROPE>();
        if (e == hipSuccess) e = set_small_lds_sizes<EPI_RESIDUAL_NORM>();
        if (e == hipSuccess) e = set_small_lds_sizes<EPI_STORE>();
        if (e == hipSuccess) e = set_small_lds_sizes<EPI_SWIGLU>();
        if (e == hipSuccess) e = set_small_lds_sizes<EPI_QKV>();
        if (e == hipSuccess) e = set_few_tile_lds_sizes<EPI_SPLITK>();
        if (e == hipSuccess) e = set_small_lds_size<EPI_SPLITK, 0>();
        if (e == hipSuccess) e = set_small_lds_size<EPI_SPLITK, 1>();
        return e;
    }();
    return err == hipSuccess && compute_units() > 0 ? DASH_OK : DASH_ERR_HIP;
}

struct GemmArgs {
    const __bf16 *A, *B;
    int M, K, N;
    const __bf16* x;
    __bf16* out;
    float *partials, *split_sums;
    QkvOut qkv;
};

template <int EPI, int F>
static void launch_small_form(const SmallPlan& g, const GemmArgs& a, hipStream_t s) {
    constexpr SmallForm f = kSmallForms[F];
    hipLaunchKernelGGL((gemm_small_kernel<EPI, f.BM, f.BN, f.KW, f.NS>), dim3(g.grid), dim3(f.KW * kSWaves * kWave),
                       small_smem_bytes(f.BM, f.BN, f.KW, f.NS), s, a.A, a.B, a.M, a.K, a.N, a.x, a.out, a.partials,
                       a.split_sums, g.mt, g.tiles, g.parts, a.K / kGK, g.ksteps_per_part, a.qkv);
}

template <int EPI, int RB>
static void launch_few_tile_rows(const SmallPlan& g, const GemmArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((gemm_few_kernel<EPI, RB>), dim3(g.grid), dim3(kFewTileWaves * kWave), few_tile_smem_bytes(16 * RB), s, a.A, a.B, a.M,
                       a.K, a.N, a.x, a.out, a.partials, a.split_sums, g.mt, g.tiles, g.parts, a.K / kGK, g.ksteps_per_part, a.qkv);
}
template <int EPI>
static void launch_few_tiles(const SmallPlan& g, const GemmArgs& a, hipStream_t s) {
    switch (g.few_rows) {
        case 16: launch_few_tile_rows<EPI, 1>(g, a, s); break;
        case 32: launch_few_tile_rows<EPI, 2>(g, a, s); break;
        default: launch_few_tile_rows<EPI, kFewTileMostRows / 16>(g, a, s); break;
    }
}

// Adds the K parts (staging_addr.h: splitk_parts, gemm_plan), whose fp32 sums lie in the scratch, in a fixed order and applies the epilogue.
template <int EPI>
static void launch_splitk_reduce(const float* sums, int parts, const GemmArgs& a, hipStream_t s) {
    const int cols_per_wave = EPI == EPI_SWIGLU ? 1024 : 512;
    const size_t waves = (size_t)a.M * ((a.N + cols_per_wave - 1) / cols_per_wave);
    hipLaunchKernelGGL((splitk_reduce_kernel<EPI>), dim3((unsigned)((waves * kWave + 255) / 256)), dim3(256), 0, s, sums,
                       parts, a.M, a.N, a.x, a.out, a.partials, a.qkv);
}

// A small-tile product (g.form >= 0, or g.few_rows > 0). scratch: the K parts' sums, or the fine row norms, which `sums` then describes or,
// without it, are folded into a.partials; a.partials = nullptr: the caller has no use for row norms.
template <int EPI>
static dash_status launch_small(const SmallPlan& g, GemmArgs a, void* scratch, NormSums* sums, hipStream_t s) {
    if (g.parts >= 2) {
        GemmArgs part = a;
        part.split_sums = reinterpret_cast<float*>(scratch);
        if (g.few_rows > 0)
            launch_few_tiles<EPI_SPLITK>(g, part, s);
        else if (g.form == 0)
            launch_small_form<EPI_SPLITK, 0>(g, part, s);
        else
            launch_small_form<EPI_SPLITK, 1>(g, part, s);
        launch_splitk_reduce<EPI>(part.split_sums, g.parts, a, s);
        return launch_status();
    }
    float* coarse = a.partials;
    if (EPI == EPI_RESIDUAL_NORM && coarse) a.partials = reinterpret_cast<float*>(scratch);
    if (g.few_rows > 0)
        launch_few_tiles<EPI>(g, a, s);
    else switch (g.form) {
        case 0: launch_small_form<EPI, 0>(g, a, s); break;
        case 1: launch_small_form<EPI, 1>(g, a, s); break;
        case 2: launch_small_form<EPI, 2>(g, a, s); break;
        case 3: launch_small_form<EPI, 3>(g, a, s); break;
        default: launch_small_form<EPI, kTallForm>(g, a, s); break;
    }
    if (EPI == EPI_RESIDUAL_NORM && coarse) {
        static_assert(kGN == 64 * kNormFold, "a fine pair covers 64 columns");
        const int cols = (a.N + 63) / 64;
        if (sums)
            *sums = NormSums{a.partials, cols, kNormFold};
        else
            hipLaunchKernelGGL(fold_partials_kernel, dim3((a.M + 255) / 256, (cols + kNormFold - 1) / kNormFold), dim3(256), 0, s,
                               (const float2*)a.partials, cols, a.M, (float2*)coarse);
    }
    return launch_status();
}

// Rows [row0, row1) of a product on tiles of 32 RB rows.
template <int EPI, int RB>
static void launch_rows(const GemmArgs& a, int row0, int row1, float* delta_dbg, hipStream_t s) {
    GemmLaunch L{};
    L.mt = (row1 - row0 + 32 * RB - 1) / (32 * RB);
    L.nt = (a.N + kGN - 1) / kGN;
    L.ksteps = a.K / kGK;
    L.plain = rows_plain(L.mt, RB);
    L.full = L.mt * L.nt;
    L.seg = (L.full + 7) / 8;
    L.row0 = row0;
    hipLaunchKernelGGL((gemm_mfma_kernel<EPI, RB>), dim3(L.plain ? L.full : 8 * L.seg), dim3(kGThreads), gemm_smem_bytes(RB), s, a.A,
                       a.B, a.M, a.K, a.N, a.x, a.out, a.partials, delta_dbg, L, a.qkv);
}

// Products of few rows: the small tiles (small_plan). Otherwise
// 256x256 tiles for every whole round over the compute units, in an order that keeps the tiles an XCD runs at one
// time close together (GemmPlan); if the tiles left over would occupy at most half of the units, they are run as
// 128-row half tiles by a second launch (same kernel, RB = 4). Products with few tiles are split along K when
// `split_ws` (device scratch of `split_bytes`) allows.
template <int EPI>
static dash_status launch_gemm(const __bf16* A, const __bf16* B, int M, int K, int N, const __bf16* x,
                               __bf16* out, float* partials, float* delta_dbg, void* split_ws, size_t split_bytes,
                               hipStream_t s, QkvOut qkv = QkvOut{}, bool want_norms = true,
                               NormSums* sums_out = nullptr) {
    // the staging loads address a tile with 32-bit lane offsets: 256 rows of A, 64 rows of B
    if ((size_t)kGM * K * 2 >= ((size_t)1 << 32) || (size_t)kGK * N * 2 + 2 * kGN >= ((size_t)1 << 32)) return DASH_ERR_UNSUPPORTED;
    if (init_gemm_kernels() != DASH_OK) return DASH_ERR_HIP;
    const GemmPlan g = gemm_plan(M, K, N, compute_units(), split_ws != nullptr && !delta_dbg, split_bytes);
    const GemmArgs args{A, B, M, K, N, x, out, partials, nullptr, qkv};
    const bool norms = EPI == EPI_RESIDUAL_NORM && want_norms;
    if (sums_out) *sums_out = NormSums{partials, (N + kGN - 1) / kGN, 1};
    // the debug output keeps the product off K parts and small tiles: with and without scratch it has the same bits
    const int head = EPI == EPI_QKV_ROPE ? 2 * qkv.half : 0;
    const SmallPlan small = product_plan(g, M, K, N, compute_units(), norms, head, split_ws != nullptr, split_ws ? split_bytes : 0);
    if ((small.form >= 0 || small.few_rows > 0) && !delta_dbg) {
        GemmArgs a = args;
        if (!norms && small.parts < 2) a.partials = nullptr;
        return launch_small<EPI>(small, a, split_ws, sums_out, s);
    }
    GemmLaunch L{};
    L.mt = g.mt;
    L.nt = g.nt;
    L.ksteps = g.ksteps;
    L.plain = g.plain;
    if (g.parts >= 2) {
        float* sums = reinterpret_cast<float*>(split_ws);
        L.ksteps_per_split = g.ksteps_per_part;
        hipLaunchKernelGGL((gemm_mfma_kernel<EPI_SPLITK, 8>), dim3(g.tiles, g.parts), dim3(kGThreads), gemm_smem_bytes(8), s,
                           A, B, M, K, N, nullptr, nullptr, nullptr, sums, L, qkv);
        launch_splitk_reduce<EPI>(sums, g.parts, args, s);
        return launch_status();
    }
    const RowPlan rows = row_plan(g, M, compute_units());
    if (rows.rb > 0) {
        if (rows.whole > 0) launch_rows<EPI, 8>(args, 0, rows.whole * kGM, delta_dbg, s);
        (rows.rb == 6 ? launch_rows<EPI, 6> : launch_rows<EPI, 7>)(args, rows.whole * kGM, M, delta_dbg, s);
        return launch_status();
    }
    L.full = g.full;
    L.seg = g.seg;
    if (g.full > 0)
        hipLaunchKernelGGL((gemm_mfma_kernel<EPI, 8>), dim3(g.grid), dim3(kGThreads), gemm_smem_bytes(8), s, A, B, M, K, N, x,
                           out, partials, delta_dbg, L, qkv);
    if (g.rest > 0) {
        L.first_tile = g.full;
        const int parts = split_ws && !delta_dbg ? rest_parts(g, compute_units(), split_bytes) : 1;
        if (parts >= 2) {
            float* sums = reinterpret_cast<float*>(split_ws);
            L.ksteps_per_split = (g.ksteps + parts - 1) / parts;
            hipLaunchKernelGGL((gemm_mfma_kernel<EPI_SPLITK, 4>), dim3(2 * g.rest, parts), dim3(kGThreads), gemm_smem_bytes(4), s,
                               A, B, M, K, N, nullptr, nullptr, nullptr, sums, L, qkv);
            constexpr int kRows = 256 / (EPI == EPI_SWIGLU ? 16 : 32);
            hipLaunchKernelGGL((rest_reduce_kernel<EPI>), dim3(2 * g.rest, kGM / 2 / kRows), dim3(256), 0, s, sums, parts, M, N,
                               x, out, partials, L, qkv);
            return launch_status();
        }
        hipLaunchKernelGGL((gemm_mfma_kernel<EPI, 4>), dim3(2 * g.rest), dim3(kGThreads), gemm_smem_bytes(4), s, A, B, M, K, N,
                           x, out, partials, delta_dbg, L, qkv);
    }
    return launch_status();
}

size_t wo_splitk_bytes(const dash_layer_params& p, int n) {
    return p.dtype == DASH_BF16 ? wo_scratch_bytes(n, p.n_q_heads * p.head_dim, p.d) : 0;
}

dash_status launch_wo_residual_rownorm(const dash_layer_params& p, const void* o, const void* w_o,
                                       const void* x, int n, void* x_next, float* partials,
                                       float* delta_dbg, void* split_ws, size_t split_bytes, NormSums* sums,
                                       hipStream_t s) {
    if (n == 0) return DASH_OK;
    const int K = p.n_q_heads * p.head_dim, N = p.d;
    if (p.dtype == DASH_F32) {
        const int64_t col_tiles = (N + kF32TileN - 1) / kF32TileN;
        if (((int64_t)n + 15) / 16 * col_tiles <= compute_units()) {
            hipLaunchKernelGGL(wo_f32_few_kernel, dim3((unsigned)col_tiles, (n + 15) / 16), dim3(kF32Split * kWave), 0, s, (const float*)o,
                               (const float*)w_o, (const float*)x, n, K, N, (float*)x_next, partials, delta_dbg);
            if (sums) *sums = NormSums{partials, norm_partials_per_row(N, p.dtype), 1};
            return launch_status();
        }
        // a launch has at most 65535 workgroups along y: more row tiles go along z in slices
        constexpr int64_t kSlice = 32768;
        const int64_t row_tiles = ((int64_t)n + kF32TileM - 1) / kF32TileM;
        const dim3 grid((N + kF32TileN - 1) / kF32TileN, (unsigned)(row_tiles < kSlice ? row_tiles : kSlice),
                        (unsigned)((row_tiles + kSlice - 1) / kSlice));
        hipLaunchKernelGGL(wo_f32_kernel, grid, dim3(kF32Split * kWave), 0, s, (const float*)o, (const float*)w_o,
                           (const float*)x, n, K, N, (float*)x_next, partials, delta_dbg);
        if (sums) *sums = NormSums{partials, norm_partials_per_row(N, p.dtype), 1};
        return launch_status();
    }
    return launch_gemm<EPI_RESIDUAL_NORM>((const __bf16*)o, (const __bf16*)w_o, n, K, N, (const __bf16*)x,
                                          (__bf16*)x_next, partials, delta_dbg, split_ws, split_bytes, s,
                                          QkvOut{}, true, sums);
}

static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

size_t ffn_workspace_bytes(const dash_layer_params& p, int n, int m) {
    return up256((size_t)n * p.d * 2) + up256((size_t)n * m * 2) +
           up256((size_t)n * norm_partials_per_row(p.d, p.dtype) * 2 * sizeof(float)) +
           max(gemm_splitk_bytes(n, p.d, 2 * m), gemm_splitk_bytes(n, m, p.d));
}

// out = x + (silu(h W_gate) * (h W_up)) W_down with h = RMSNorm(x) (Alg. 1 step 7): row norm, one GEMM over
// the interleaved gate/up weight with the gating in its epilogue, one GEMM with the residual epilogue.
dash_status launch_ffn_swiglu(const dash_layer_params& p, const void* x, const void* w_gate_up, const void* w_down,
                              int n, int m, void* x_out, void* ws, hipStream_t s) {
    if (n == 0) return DASH_OK;
    char* base = reinterpret_cast<char*>(ws);
    __bf16* h = reinterpret_cast<__bf16*>(base);
    __bf16* act = reinterpret_cast<__bf16*>(base + up256((size_t)n * p.d * 2));
    float* partials = reinterpret_cast<float*>(base + up256((size_t)n * p.d * 2) + up256((size_t)n * m * 2));
    char* split_ws = reinterpret_cast<char*>(partials) +
                     up256((size_t)n * norm_partials_per_row(p.d, p.dtype) * 2 * sizeof(float));
    const size_t split_bytes = max(gemm_splitk_bytes(n, p.d, 2 * m), gemm_splitk_bytes(n, m, p.d));
    launch_rmsnorm((const __bf16*)x, n, p.d, h, s);
    dash_status st = launch_gemm<EPI_SWIGLU>(h, (const __bf16*)w_gate_up, n, p.d, 2 * m, nullptr, act, nullptr,
                                             nullptr, split_ws, split_bytes, s);
    if (st != DASH_OK) return st;
    return launch_gemm<EPI_RESIDUAL_NORM>(act, (const __bf16*)w_down, n, m, p.d, (const __bf16*)x,
                                          (__bf16*)x_out, partials, nullptr, split_ws, split_bytes, s,
                                          QkvOut{}, false);
}

size_t rope_table_bytes(const dash_layer_params& p, int n);

size_t qkv_workspace_bytes(const dash_layer_params& p, int n) {
    if (p.dtype != DASH_BF16) return 0;
    const int Dq = p.n_q_heads * p.head_dim, Dkv = p.n_kv_heads * p.head_dim;
    // the rotary table, and the widest of the three separate projections or the one product over the concatenated weight
    return rope_table_bytes(p, n) + max(gemm_splitk_bytes(n, p.d, Dq), gemm_splitk_bytes(n, p.d, Dq + 2 * Dkv));
}

dash_status launch_rmsnorm_qkv(const dash_layer_params& p, const void* x, const void* w_q, const void* w_k,
                               const void* w_v, int n, void* q, void* k, void* v, void* hbuf, void* split_ws,
                               size_t split_bytes, hipStream_t s) {
    if (n == 0) return DASH_OK;
    const int d = p.d, Dq = p.n_q_heads * p.head_dim, Dkv = p.n_kv_heads * p.head_dim;
    launch_rmsnorm((const __bf16*)x, n, d, (__bf16*)hbuf, s);
    const __bf16* h = (const __bf16*)hbuf;
    dash_status st = launch_gemm<EPI_STORE>(h, (const __bf16*)w_q, n, d, Dq, nullptr, (__bf16*)q, nullptr, nullptr,
                                            split_ws, split_bytes, s);
    if (st != DASH_OK) return st;
    st = launch_gemm<EPI_STORE>(h, (const __bf16*)w_k, n, d, Dkv, nullptr, (__bf16*)k, nullptr, nullptr, split_ws,
                                split_bytes, s);
    if (st != DASH_OK) return st;
    return launch_gemm<EPI_STORE>(h, (const __bf16*)w_v, n, d, Dkv, nullptr, (__bf16*)v, nullptr, nullptr, split_ws,
                                  split_bytes, s);
}

// The same front end as one product over w_qkv = [w_q | w_k | w_v] ([d, Dq + 2 Dkv]): one pass over the
// normalised rows instead of three, and no launches that fill a fraction of the chip for the narrow k and v.
dash_status launch_rmsnorm_qkv_fused(const dash_layer_params& p, const void* x, const void* w_qkv, int n, void* q,
                                     void* k, void* v, void* hbuf, void* split_ws, size_t split_bytes,
                                     hipStream_t s) {
    if (n == 0) return DASH_OK;
    const int d = p.d, Dq = p.n_q_heads * p.head_dim, Dkv = p.n_kv_heads * p.head_dim;
    launch_rmsnorm((const __bf16*)x, n, d, (__bf16*)hbuf, s);
    return launch_gemm<EPI_QKV>((const __bf16*)hbuf, (const __bf16*)w_qkv, n, d, Dq + 2 * Dkv, nullptr, (__bf16*)q,
                                nullptr, nullptr, split_ws, split_bytes, s, QkvOut{(__bf16*)k, (__bf16*)v, Dq, Dkv, nullptr, 0});
}

// ... and with the rotary embedding of q and k in the product's epilogue: the row norm's launch leaves the angles' cosines
// and sines at the start of the scratch, the rest of it serves the product.
size_t rope_table_bytes(const dash_layer_params& p, int n) { return up256((size_t)n * (p.head_dim / 2) * sizeof(float2)); }

dash_status launch_rmsnorm_qkv_rope(const dash_layer_params& p, const void* x, const void* w_qkv, const int32_t* active_idx,
                                    double theta, int n, void* q, void* k, void* v, void* hbuf, void* ws, size_t ws_bytes,
                                    hipStream_t s) {
    if (n == 0) return DASH_OK;
    const int d = p.d, Dq = p.n_q_heads * p.head_dim, Dkv = p.n_kv_heads * p.head_dim, half = p.head_dim / 2;
    const size_t used = rope_table_bytes(p, n);
    const RopeTable rope{active_idx, (float2*)ws, -log2(theta) * 2.0 / (double)p.head_dim};
    if (half == 32)
        launch_rmsnorm<32>((const __bf16*)x, n, d, (__bf16*)hbuf, rope, s);
    else
        launch_rmsnorm<64>((const __bf16*)x, n, d, (__bf16*)hbuf, rope, s);
    return launch_gemm<EPI_QKV_ROPE>((const __bf16*)hbuf, (const __bf16*)w_qkv, n, d, Dq + 2 * Dkv, nullptr, (__bf16*)q, nullptr,
                                     nullptr, (char*)ws + used, ws_bytes - used, s,
                                     QkvOut{(__bf16*)k, (__bf16*)v, Dq, Dkv, rope.table, half});
}

}  // namespace dash
