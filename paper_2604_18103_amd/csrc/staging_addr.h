// Address arithmetic of the direct global->LDS staging loads of the two MFMA kernels, and the way a GEMM is
// cut into launches. Plain C++ that compiles for the host and for the device: the kernels and launchers use
// these functions, and a host program (staging_check.cpp) enumerates every load of a launch with the same
// functions and checks it against the operand sizes, so a change of the addressing is checked on the CPU
// before it runs on a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define DASH_HD __host__ __device__ __forceinline__
#else
#define DASH_HD inline
#endif

namespace dash {

DASH_HD int sa_min(int a, int b) { return a < b ? a : b; }
DASH_HD int sa_max(int a, int b) { return a > b ? a : b; }

// ------------------------------------------------------------------------------------------------
// GEMM: workgroup tile 256 x 256, K step 64, 8 waves. A tile rows are 128 bytes (one load instruction = 8
// rows), B tile rows 512 bytes (one instruction = 2 rows). A load's address is a uniform base (the tile at the
// current K step) plus a 32-bit lane offset that never changes.
// ------------------------------------------------------------------------------------------------
constexpr int kGM = 256, kGN = 256, kGK = 64;
constexpr int kGWaves = 8;

DASH_HD constexpr int gemm_adma(int BM) { return (BM / 8 + kGWaves - 1) / kGWaves; }  // A load instructions per wave and K step
DASH_HD constexpr int gemm_bdma() { return kGK / 2 / 8; }         // B load instructions per wave and K step

DASH_HD int gemm_a_row(int wave, int i, int lane, int adma) { return (wave * adma + i) * 8 + lane / 8; }
DASH_HD int gemm_b_row(int wave, int i, int lane) { return (wave * gemm_bdma() + i) * 2 + lane / 32; }
// logical 16-byte chunk that lands in physical chunk lane % (chunks per row) of the row (XOR swizzle)
DASH_HD int gemm_a_lchunk(int row, int lane) { return (lane % 8) ^ ((row / 2) % 8); }
DASH_HD int gemm_b_swz(int row) { return 4 * (row % 4) + 2 * ((row / 8) % 2); }
DASH_HD int gemm_b_lchunk(int row, int lane) { return (lane % 32) ^ gemm_b_swz(row); }

// First row of the A base. The second half tile of a last row tile may lie wholly beyond M: the base is
// clamped like the rows, so every lane offset stays non-negative. Rows beyond M and columns beyond N are
// computed on valid (clamped) data and never stored.
DASH_HD int gemm_a_base_row(int m0, int M) { return sa_min(m0, M - 1); }
DASH_HD size_t gemm_a_base_elem(int m0, int M, int K, int ks0) {
    return (size_t)gemm_a_base_row(m0, M) * K + (size_t)ks0 * kGK;
}
DASH_HD uint32_t gemm_a_off(int m0, int M, int K, int row, int lchunk) {
    return (uint32_t)(((size_t)(sa_min(m0 + row, M - 1) - gemm_a_base_row(m0, M)) * K + lchunk * 8) * 2);
}
DASH_HD size_t gemm_b_base_elem(int n0, int N, int ks0) { return (size_t)ks0 * kGK * N + n0; }
DASH_HD uint32_t gemm_b_off(int n0, int N, int row, int lchunk) {
    return (uint32_t)(((size_t)row * N + (sa_min(n0 + lchunk * 8, N - 8) - n0)) * 2);
}
DASH_HD size_t gemm_a_step_bytes() { return (size_t)kGK * 2; }
DASH_HD size_t gemm_b_step_bytes(int N) { return (size_t)kGK * N * 2; }

// Split-K: a product with few output tiles and a long contraction (few active rows) leaves most compute units
// idle and the few busy ones with a long serial loop. Such a product is cut along K into parts that run side
// by side. Used when the tiles would occupy at most half of the units; a part has at least kSplitMinSteps K steps.
constexpr int kSplitMinSteps = 4;
inline int splitk_parts(int tiles, int ksteps, int cu) {
    if (cu <= 0 || 2 * tiles > cu) return 1;
    const int s = sa_min(cu / tiles, ksteps / kSplitMinSteps);
    return s < 2 ? 1 : s;
}
// Scratch bytes that let every product of up to M_cap rows with this K and N split as far as it would like to.
constexpr int kSplitSizingUnits = 256;  // unit count assumed when sizing the scratch (the launch uses the real one)
inline size_t gemm_splitk_bytes(int M_cap, int K, int N) {
    const int nt = (N + kGN - 1) / kGN, ksteps = K / kGK;
    size_t best = 0;
    for (int mt = 1; mt <= (M_cap + kGM - 1) / kGM; ++mt) {
        const int parts = splitk_parts(mt * nt, ksteps, kSplitSizingUnits);
        if (parts < 2) break;  // more row tiles only split less
        const size_t bytes = (size_t)parts * sa_min(mt * kGM, M_cap) * N * sizeof(float);
        best = bytes > best ? bytes : best;
    }
    return (best + 255) / 256 * 256;
}
// The layer call's: as well the fine row norms of a small-tile projection (one pair per row and 64 columns); products of more than 1 MB of
// them are no small ones, and one that finds less scratch takes the large tiles.
inline size_t wo_scratch_bytes(int n, int K, int N) {
    const size_t fine = ((size_t)n * ((N + 63) / 64) * 2 * sizeof(float) + 255) / 256 * 256, most = (size_t)1 << 20;
    const size_t norms = fine < most ? fine : most, split = gemm_splitk_bytes(n, K, N);
    return split > norms ? split : norms;
}

// Order in which the output tiles of a product are handed out ("tile index" below), and which workgroup takes which
// index. Workgroup b of a launch runs on XCD b % 8, and each XCD has its own L2: what the 32 workgroups that an XCD
// runs at one time share in that L2 is decided here.
//  - row tiles a multiple of 8 ("plain"): tile index = column-major position (row tile fastest), workgroup b takes
//    index b. An XCD then holds row tiles b % 8, b % 8 + 8, ... of four consecutive tile columns: 8 A panels and
//    4 B panels for 32 tiles, and all XCDs are in the same four tile columns at the same time.
//  - otherwise: column panels of 4 tile columns (the last one narrower), row by row inside a panel, so that 32
//    consecutive indices are a block of 8 x 4 tiles; the indices are dealt to the XCDs as 8 contiguous stretches
//    (workgroup b takes index (b % 8) * seg + b / 8), equally many per XCD. With the plain order a row-tile count
//    that is not a multiple of 8 would scatter an XCD's 32 tiles over up to 32 row panels.
constexpr int kGPanel = 4;
DASH_HD void gemm_tile_of(int idx, int mt, int nt, bool plain, int& tile_m, int& tile_n) {
    if (plain) {
        tile_m = idx % mt;
        tile_n = idx / mt;
        return;
    }
    const int per_panel = mt * kGPanel, whole = nt / kGPanel;
    const int p = idx / per_panel;
    if (p < whole) {
        const int r = idx - p * per_panel;
        tile_m = r / kGPanel;
        tile_n = p * kGPanel + r % kGPanel;
    } else {
        const int w = nt - whole * kGPanel;  // >= 1: idx < mt * nt
        const int r = idx - whole * per_panel;
        tile_m = r / w;
        tile_n = whole * kGPanel + r % w;
    }
}

// How launch_gemm cuts a product into launches: either `parts` >= 2 split-K parts over all tiles, or `full`
// 256-row tiles (a grid of `grid` workgroups: gemm_index_of) followed by `rest` tiles run as 128-row half tiles
// (when the tiles left over after the whole rounds would occupy at most half of the units).
struct GemmPlan {
    int mt, nt, tiles, ksteps;
    int parts, ksteps_per_part;  // parts >= 2: split-K launch
    int full, rest;              // otherwise
    int plain, seg, grid;        // tile order of the whole tiles, indices per XCD, workgroups of their launch
};
inline GemmPlan gemm_plan(int M, int K, int N, int cu, bool may_split, size_t split_bytes) {
    GemmPlan g{};
    g.mt = (M + kGM - 1) / kGM;
    g.nt = (N + kGN - 1) / kGN;
    g.tiles = g.mt * g.nt;
    g.ksteps = K / kGK;
    g.parts = 1;
    g.ksteps_per_part = g.ksteps;
    g.plain = g.mt % 8 == 0 ? 1 : 0;
    if (may_split) {
        int parts = splitk_parts(g.tiles, g.ksteps, cu);
        const size_t per_part = (size_t)M * N * sizeof(float);
        if ((size_t)parts * per_part > split_bytes) parts = (int)(split_bytes / per_part);
        if (parts >= 2) {
            const int per = (g.ksteps + parts - 1) / parts;
            g.parts = (g.ksteps + per - 1) / per;  // every part has at least one K step
            g.ksteps_per_part = per;
            return g;
        }
    }
    g.rest = cu > 0 ? g.tiles % cu : 0;
    if (2 * g.rest > cu) g.rest = 0;
    g.full = g.tiles - g.rest;
    g.seg = (g.full + 7) / 8;
    g.grid = g.plain ? g.full : 8 * g.seg;
    return g;
}

// Lower tiles for a round that 256-row tiles would fill by more than half but not quite: its workgroups then take 32 rb / 256 of the
// time, on more units. On the workload's data the part is power-limited and runs faster while units idle, so half of that is
// what is gained, less a launch where whole rounds go before it.
//  - products of one round: the lowest tile that still fits it. Measured, 256-row tiles / these, us, K = N = 3584: 2400 rows 82 / 67,
//    3000 78 / 71, 3400 80 / 76 (192 rows), 3700 84 / 82.5 (224); K = 18944 2400 330 / 281, 3700 410 / 400; 3584 x 4608 with the row
//    norm's launch 1800 74 / 64; 1024 x 1024 9000 30.5 / 26.7. Not 224 rows where the row tiles are a multiple of 8 and the columns
//    few: the plain tile order, which lets an XCD share row panels, is worth more (8192 x 1024 x 1536 34.6 / 36.0).
//  - the last of several rounds, for long contractions: K = 18944, N = 3584: 7500 rows 853 / 792, 8192 860 / 845, 11885 1312 / 1239,
//    13000 1339 / 1300; at K = 3584 it is within the noise (11885 260 / 253, 8192 169 / 175).
//    Not 224 rows where they fill every unit, so that none idles: 14336 x 4096 7635 rows 648 / 658, 11731 978 / 1009, 15827 1310 / 1371.
//    (As the only round they gain there too: 3539 rows of 4096 x 4096 100.9 / 95.7, 7123 of 1024 x 2048 38.9 / 34.6.)
// All rounds on lower tiles is slower: 10000 rows of K = 18944 1046 / 1169.
struct RowPlan {
    int rb, whole;  // 16-row blocks per wave of the lower tiles (0: none), 256-row row tiles before them
};
// Tile order of a launch over whole rows of tiles. Lower tiles are one round, so each XCD holds all of its tiles at once: in the plain
// order mt / 8 row tiles and every column, in column panels blocks of 8 x 4 tiles. With 8 row tiles the plain order gives an XCD one of them
// and the whole weight, and panels are faster whatever the weight; from 16 on an operand that has just been written is read through one L2
// and not two, which is worth more. 256-row tiles / lower ones plain / in panels, us, operand written before each call: 1491 rows of 256 x
// 8192 21.5 / 19.9 / 19.4, of 1024 x 6144 34.2 / 32.1 / 30.3, of 4096 x 6144 97.7 / 94.2 / 89.9, of 8192 x 8192 177 / 185 / 165; 6099 of 512 x 1536
// 26.5 / 23.6 / 26.4, 4563 of 1024 x 2048 37.4 / 31.1 / 32.9, 3027 of 2048 x 4096 56.1 / 52.5 / 53.7, of 18944 x 3584 431 / 401 / 410, 3027 of 14336 x
// 4096 and 4563 of 4096 x 2048 the same. (Repeated on operands that stay in the L2s panels are up to 4 % faster there too.)
DASH_HD bool rows_plain(int mt, int rb) { return mt % 8 == 0 && (rb == 8 || mt > 8); }
inline RowPlan row_plan(const GemmPlan& g, int M, int cu) {
    if (cu <= 0 || g.parts >= 2 || g.rest > 0) return RowPlan{0, 0};
    const int rounds = (g.tiles + cu - 1) / cu, whole = (int)((long long)(rounds - 1) * cu / g.nt);
    for (int rb = 6; rb <= 7; ++rb) {
        const long long t = (long long)((M - whole * kGM + 32 * rb - 1) / (32 * rb)) * g.nt;
        const double gain_us = 0.5 * (1.0 - rb / 8.0) * g.ksteps * 1.66;
        if (rb == 7 && ((g.plain && g.nt < 8) || (whole > 0 && t == cu))) continue;
        if (t <= cu && (whole == 0 || gain_us > 20.0)) return RowPlan{rb, whole};
    }
    return RowPlan{0, 0};
}

// Tile index that workgroup b of the whole-tile launch takes, or -1 (padding of the last stretch: the workgroup leaves).
DASH_HD int gemm_index_of(int b, int full, bool plain, int seg) {
    if (plain) return b;
    const int idx = (b % 8) * seg + b / 8;
    return (b / 8 < seg && idx < sa_min(((b % 8) + 1) * seg, full)) ? idx : -1;
}

// ------------------------------------------------------------------------------------------------
// Small tiles: workgroup tile BM x BN (64 or 128 each), K step 64, 4 waves. A tile rows are 128 bytes (one load
// instruction = 8 rows, swizzled as above), B tile rows 2 BN bytes (one instruction = 512 / BN rows). The bases and lane
// offsets are those of the large tiles (gemm_a_base_elem, gemm_a_off, gemm_b_base_elem, gemm_b_off).
// ------------------------------------------------------------------------------------------------
constexpr int kSWaves = 4;
DASH_HD constexpr int small_adma(int BM) { return BM / 8 / kSWaves; }
DASH_HD constexpr int small_bdma(int BN) { return BN / 8 / kSWaves; }
DASH_HD int small_a_row(int wave, int i, int lane, int BM) { return (wave * small_adma(BM) + i) * 8 + lane / 8; }
DASH_HD int small_b_row(int wave, int i, int lane, int BN) {
    return (wave * small_bdma(BN) + i) * (512 / BN) + lane / (BN / 8);
}
// 32 lanes of a transpose read touch rows r .. r + 3 and r + 8 .. r + 11, 32 bytes of each: the swizzle spreads these
// eight pieces over the 256 bytes that the banks cover (one row of 128 columns, two rows of 64)
DASH_HD int small_b_swz(int row, int BN) {
    return BN == 64 ? 2 * ((row / 2) % 2) + 4 * ((row / 8) % 2) : 2 * (row % 4) + 8 * ((row / 8) % 2);
}
DASH_HD int small_b_lchunk(int row, int lane, int BN) { return (lane % (BN / 8)) ^ small_b_swz(row, BN); }
// Tile (and K part) of workgroup b: the parts one after the other, in each the column tiles in order, row tiles of a column
// next to each other; all of it dealt to the XCDs (b % 8) as 8 contiguous stretches, so that the row tiles of a weight column
// are read through one L2 and no XCD gets more than an eighth of the workgroups. (Stretches of each part by itself, rounded up,
// gave 33 workgroups to XCDs of 32 units where 84 tiles run in 3 parts, and the launch two rounds.) False: padding, no tile.
DASH_HD bool small_work_of(int b, int tiles, int parts, int& tile, int& part) {
    const int work = tiles * parts, seg = (work + 7) / 8, idx = (b % 8) * seg + b / 8;
    part = parts == 1 ? 0 : idx / tiles;
    tile = idx - part * tiles;
    return b / 8 < seg && idx < work;
}

// Which form a product takes: the large tiles (gemm_plan) or one of five small-tile forms (the fifth: tall_tile_plan). Small tiles are for products of few
// rows (at most two large row tiles), and for others while the large tiles would occupy at most half of the units (their
// alternative is then K parts and a second pass). From there on they save nothing worth a second rule: of 300 products
// measured beyond that line, small tiles were up to 1.3 times as slow where they had been chosen, and never more than 8 %
// faster. Otherwise the form expected to be fastest is taken. (With few rows of a wide product the large form may also
// cut its left-over half tiles along K, which large_tiles_us leaves out: at 257 to 384 rows of 3584 x 37888 that estimate would
// turn to the large tiles, which measured 2 to 4 % slower.) The expectation is a count of rounds over the compute units times
// the K steps times what one step was measured to take, plus what a launch costs (us, 256 compute units at their usual clock
// under matrix work; the forms differ by 10 to 300 %, so the figures only have to be roughly right):
//   small form       KW NS  per unit  step alone, step of a full unit   (weight from memory, not from the last-level cache)
//   64 x  64          2  3     1        0.205                             0.23
//   64 x 128          2  3     1        0.31                              0.35
//  128 x 128          1  3     1        0.45                              0.61
//  128 x 128          1  2     2        0.64,  0.875 (two workgroups)     0.80, 0.95
//   large tile 1.35 (units two thirds busy or less) to 1.66 (all busy), half tile 0.65 to 0.98
//   a second pass over K parts: 4 + 8 bytes per partial sum at 8 TB/s; several rounds of small tiles: a factor 1.3 (the L2)
// The launcher cannot know where the weight is, and the figures taken are the cached ones: with those of the last column the
// choice gains 1 % on weights from memory and loses 1 % on cached ones.
// Measured over 916 products (17 to 12001 rows, K 512 to 4096, N 512 to 6144; each repeated on one weight, and the shorter ones
// on weights from memory): below the line 0.62 and 0.64 times the large tiles' time on average; at worst 1.09 times on cached
// weights and, at K = 4096 on weights from memory, 1.18. (Beyond those ranges: five K steps, 2201 x 320 x 3584, 14 / 18; a column
// tile for 8 columns, 6600 x 3584 x 520, 50 / 66.) Large tiles / this choice, us, K = N = 3584 with a row norm's launch of about
// 5, cached and from memory: 63 rows 24.6 / 14.9 and 25.1 / 17.7, 511 40 / 28 and 41 / 35, 901 48 / 37 and 48 / 43, 1401 58 / 49.5
// and 58 / 58.6, 2201 75 / 60 and 75 / 65; from 2305 on large. Feed-forward 3584 x 18944: 17 rows 133 / 103, 63 133 / 113.
struct SmallForm {
    int BM, BN, KW, NS, per_cu;
    double step_us, full_us;
};
constexpr SmallForm kSmallForms[5] = {{64, 64, 2, 3, 1, 0.205, 0.205},
                                      {64, 128, 2, 3, 1, 0.31, 0.31},
                                      {128, 128, 1, 3, 1, 0.45, 0.45},
                                      {128, 128, 1, 2, 2, 0.64, 0.875},
                                      {192, 128, 1, 3, 1, 0.65, 0.65}};  // tall_tile_plan
constexpr int kSmallSplitMinSteps = 6;  // K steps of a part, at least

struct SmallPlan {
    int form;                              // index into kSmallForms, -1: the large tiles
    int mt, nt, tiles, grid;               // grid = workgroups of all parts, padded to a multiple of 8
    int parts, ksteps_per_part;            // parts >= 2: fp32 sums and a second pass
    int few_rows;                          // few_tile_plan: rows of its tiles, 0: the form above
    double us;                             // estimate
};
inline double sa_busy(int wgs, int cu) {  // 0 up to two thirds of the units busy, 1 from all of them on
    const double b = ((double)wgs / cu - 0.65) / 0.35;
    return b < 0 ? 0 : (b > 1 ? 1 : b);
}
inline double second_pass_us(int parts, int M, int N) { return 4.0 + (double)parts * M * N * 8.0 / 8.0e6; }
inline double large_tiles_us(const GemmPlan& g, int M, int N, int cu) {
    if (g.parts >= 2) return g.ksteps_per_part * 1.35 + 9.0 + second_pass_us(g.parts, M, N);
    const int rounds = (g.full + cu - 1) / cu;
    double t = rounds * (g.ksteps * (1.35 + 0.31 * sa_busy(g.full, cu)) + 5.0);
    if (g.rest > 0) t += g.ksteps * (0.65 + 0.33 * sa_busy(2 * g.rest, cu)) + 5.0;  // in one part
    return t;
}
// The tiles left over after the whole rounds (g.rest, run as 128-row half tiles on 2 g.rest units) cut along K as well when
// that leaves units idle: fp32 sums [part][half tile][128][256] and a second pass over those tiles only. Returns the parts, 1
// where the second pass costs more than it gives. Measured, whole product, one pass / cut, us: K = N = 3584 with 10
// left-over tiles 140 / 125, 24 140 / 128, 38 143 / 137; K = 18944: 10 625 / 480, 38 644 / 534. From about 64 on (two parts) it
// no longer pays.
constexpr int kRestMinSteps = 4;
DASH_HD constexpr size_t rest_sum_elems() { return (size_t)(kGM / 2) * kGN; }
inline int rest_parts(const GemmPlan& g, int cu, size_t scratch_bytes) {
    if (g.parts >= 2 || g.rest == 0 || cu <= 0) return 1;
    auto launch_us = [&](int per, int parts) { return per * (0.65 + 0.33 * sa_busy(2 * g.rest * parts, cu)) + 5.0; };
    int best = 1;
    double best_us = 0.9 * launch_us(g.ksteps, 1);
    const int most = sa_min(cu / (2 * g.rest), g.ksteps / kRestMinSteps);
    for (int p = 2; p <= most; ++p) {
        const int per = (g.ksteps + p - 1) / p;
        const size_t need = (size_t)p * 2 * g.rest * rest_sum_elems() * sizeof(float);
        if ((g.ksteps + per - 1) / per != p || need > scratch_bytes) continue;
        const double t = launch_us(per, p) + 4.0 + 2.0 * (double)need / 8.0e6;
        if (t < best_us) {
            best_us = t;
            best = p;
        }
    }
    return best;
}
// norms: the product returns row norms, whose fine pairs need scratch too. Without scratch a product adds its K steps in
// one order, whatever its width: large tiles.
// head: columns that have to lie in one tile unless a second pass follows (0: none).
inline SmallPlan small_plan(int M, int K, int N, int cu, bool norms, int head, bool scratch, size_t scratch_bytes, double large_us) {
    SmallPlan best{};
    best.form = -1;
    best.us = large_us;
    const long long large_tiles = (long long)((M + kGM - 1) / kGM) * ((N + kGN - 1) / kGN);
    if (cu <= 0 || !scratch || (M > 2 * kGM && 2 * large_tiles > cu)) return best;
    double best_us = 0.95 * large_us - 0.5;  // so close, the large tiles were the faster ones (few K steps)
    const int ksteps = K / kGK;
    for (int f = 0; f < 4; ++f) {
        const SmallForm& s = kSmallForms[f];
        const int mt = (M + s.BM - 1) / s.BM, nt = (N + s.BN - 1) / s.BN;
        const long long tiles = (long long)mt * nt;
        if (tiles > 8LL * cu) continue;
        const int most = f < 2 ? sa_min(cu / (int)tiles, ksteps / kSmallSplitMinSteps) : 1;
        for (int parts = 1; parts <= sa_max(most, 1); ++parts) {
            const int per = (ksteps + parts - 1) / parts;
            if (parts == 1 && head > s.BN) continue;
            if ((ksteps + per - 1) / per != parts) continue;  // every part has a K step, and no two plans are alike
            const size_t need = parts > 1 ? (size_t)parts * M * N * sizeof(float) : (norms ? (size_t)((N + 63) / 64) * M * 2 * sizeof(float) : 0);
            if (need > scratch_bytes) continue;
            const int rounds = (int)((tiles + cu * s.per_cu - 1) / (cu * s.per_cu));
            const double twice = tiles <= cu ? 0.0 : (tiles < 2LL * cu ? (double)(tiles - cu) / cu : 1.0);  // units with two
            double t = rounds * per * (s.step_us + (s.full_us - s.step_us) * twice) * (rounds > 1 ? 1.3 : 1.0) + 4.0;
            if (parts > 1) t += second_pass_us(parts, M, N);
            if (t < best_us) {
                best_us = t;
                best = SmallPlan{f, mt, nt, (int)tiles, 8 * (((int)tiles * parts + 7) / 8), parts, per, 0, t};
            }
        }
    }
    return best;
}

// 192 x 128 tiles, one workgroup per unit and all three stages' lead, in place of two 128 x 128 workgroups per unit (form 3), whose steps
// have one round to land, where they fit one round. us, two workgroups / these; with a row norm's launch, weight cached: K = N = 3584 1153 rows
// 46.4 / 44.0, 1400 48.0 / 46.0, 1728 50.6 / 48.9; 4096 1025 49.3 / 45.1, 1536 55.0 / 51.8; 1024 (16 steps) 4097 24.4 / 21.9, 5000 26.2 / 24.3, 6144 27.1 /
// 27.2; front end of 3584 x 4608 1000 rows 46.3 / 42.4, 1344 50.9 / 47.1. Weights and x from memory: layer of 3584 1220 rows 86.8 / 72.2, 1700 100.8 / 91.2;
// front end 1000 55.7 / 43.4. Fewer than 16 steps: 12000 rows of 512 x 512 19.7 / 20.4. 256 x 128 tiles: 2120 rows of 3584 the same from the caches and
// from memory, 8192 of 1024 30.5 / 33.6.
constexpr int kTallForm = 4, kTallMinSteps = 16;
inline SmallPlan tall_tile_plan(int M, int N, int cu, const SmallPlan& other) {
    const SmallForm& s = kSmallForms[kTallForm];
    const int mt = (M + s.BM - 1) / s.BM, nt = (N + s.BN - 1) / s.BN, tiles = mt * nt, ksteps = other.ksteps_per_part;
    if (other.form != 3 || (long long)mt * nt > cu || ksteps < kTallMinSteps) return other;
    return SmallPlan{kTallForm, mt, nt, tiles, 8 * ((tiles + 7) / 8), 1, ksteps, 0, ksteps * s.step_us + 4.0};
}

// ------------------------------------------------------------------------------------------------
// Tiles for the fewest rows: 16, 32 or 48 rows x 64 columns, 8 waves that take K steps of their own (wave w: w, w + 8, ...). A load
// instruction is 8 rows of 128 bytes of either operand; swizzles, bases and lane offsets are those of the tiles above.
// ------------------------------------------------------------------------------------------------
constexpr int kFewTileN = 64, kFewTileWaves = 8;
DASH_HD int few_tile_row(int i, int lane) { return 8 * i + lane / 8; }
DASH_HD constexpr size_t few_tile_smem_bytes(int bm) {  // the waves' stages; in the end their sums, rows of 64 + 4 words
    const size_t stages = (size_t)kFewTileWaves * (bm + kFewTileN) * kGK * 2, sums = (size_t)kFewTileWaves * bm * (kFewTileN + 4) * 4;
    return stages > sums ? stages : sums;
}
// These tiles for products of up to kFewTileRows rows, where they are expected to be faster than `other`, the form chosen so far. One round
// of workgroups; in K parts where the tiles leave units idle, every wave with a step at least. The expectation (us): a launch with one
// step per wave, 2.6 + 0.035 per row; every step more 1.05 + 0.01 per row, 0.2 more where a quarter of the units or less share the
// weight's way from the last-level cache; K parts (of either) 2.4 beside the second pass. Where the other form is in K parts and this one is
// not, 4.8 against it: the parts' sums leave fewer norm pairs to read, and a weight from memory goes through more units at a time.
// No more than eight steps per wave: a longer contraction's weight comes from memory, and more slowly so (18944 x 3584 in four parts, 16 rows,
// with the gate and up product 96.9 / 99.5).
// Measured, the other forms / these: layer calls, weights in the last-level cache, width 3584 16 rows 21.9 / 20.3, 48 23.9 / 22.8, 177 28.6 /
// 27.1; 4096 177 29.5 / 28.5; 512 16 12.2 / 11.35, 333 17.6 / 16.5, 700 21.5 / 20.6; 1024 16 14.0 / 12.4, 177 16.7 / 15.0, 511 20.4 / 19.8; weights from
// memory 3584 16 23.3 / 22.3, 177 37.1 / 33.7. Front end of width 1024 with heads of 64, 150 rows 9.55 / 8.05; feed-forward 512 x 1408 64 rows 14.2 /
// 11.4, 600 19.05 / 18.3. Left out, being no faster: 64 rows a tile (256 rows of 3584 30.3 / 30.5), more than 1024 rows (1500 of 512 x 512 6.8 / 7.0),
// one pass over 64 rows of 3584 where the others take four parts (22.7 / 22.75, from memory 26.4 / 27.6).
constexpr int kFewTileRows = 1024, kFewTileMostRows = 48, kFewTileMostSteps = 8;
inline SmallPlan few_tile_plan(int M, int K, int N, int cu, bool norms, int head, bool scratch, size_t scratch_bytes, const SmallPlan& other) {
    SmallPlan best = other;
    if (cu <= 0 || !scratch || M > kFewTileRows) return best;
    const int nt = (N + kFewTileN - 1) / kFewTileN, ksteps = K / kGK;
    best.us += other.parts > 1 ? 2.4 : 0.0;
    for (int bm = 16; bm <= kFewTileMostRows; bm += 16) {
        const int mt = (M + bm - 1) / bm;
        const long long tiles = (long long)mt * nt;
        if (tiles > cu) continue;
        const int most = sa_min(cu / (int)tiles, ksteps / kFewTileWaves);
        for (int parts = 1; parts <= sa_max(most, 1); ++parts) {
            const int per = (ksteps + parts - 1) / parts;
            if ((parts == 1 && head > kFewTileN) || (ksteps + per - 1) / per != parts || per > kFewTileMostSteps * kFewTileWaves) continue;
            const size_t need = parts > 1 ? (size_t)parts * M * N * sizeof(float) : (norms ? (size_t)((N + 63) / 64) * M * 2 * sizeof(float) : 0);
            if (need > scratch_bytes) continue;
            const double step = 1.05 + 0.01 * bm + (4 * tiles * parts <= cu ? 0.2 : 0.0);
            double t = 2.6 + 0.035 * bm + ((per + kFewTileWaves - 1) / kFewTileWaves - 1) * step;
            t += parts > 1 ? 2.4 + second_pass_us(parts, M, N) : (other.parts > 1 ? 4.8 : 0.0);
            if (t < best.us) best = SmallPlan{-1, mt, nt, (int)tiles, 8 * (((int)tiles * parts + 7) / 8), parts, per, bm, t};
        }
    }
    return best;
}

// The form a product takes (form < 0 and no few_rows: the large tiles), for the launcher and for the checks.
inline SmallPlan product_plan(const GemmPlan& g, int M, int K, int N, int cu, bool norms, int head, bool scratch, size_t scratch_bytes) {
    const SmallPlan small = small_plan(M, K, N, cu, norms, head, scratch, scratch_bytes, large_tiles_us(g, M, N, cu));
    return few_tile_plan(M, K, N, cu, norms, head, scratch, scratch_bytes, tall_tile_plan(M, N, cu, small));
}

// ------------------------------------------------------------------------------------------------
// Attention: K/V tiles of 64 keys, rows of DH bf16, unpadded, 16-byte chunks XOR-swizzled inside a row. One
// load instruction moves 1 KB = 64 / CPR rows; lane l lands in physical chunk l % CPR of row l / CPR. The four
// waves of a group fetch a tile; a load's address is a uniform tile base plus a 32-bit lane offset that is the
// same for every whole tile; in the last, partly filled tile rows beyond the end are clamped to the last row.
// ------------------------------------------------------------------------------------------------
constexpr int kFaBM = 256;  // query rows per workgroup (two key groups: 128)
constexpr int kFaBN = 64;   // keys per tile

DASH_HD constexpr int fa_cpr(int DH) { return DH / 8; }            // 16-byte chunks per row
DASH_HD constexpr int fa_rp(int DH) { return 256 / (DH * 2); }     // rows per 256 bytes of LDS
DASH_HD constexpr int fa_k_swz(int row, int DH) { return (row / fa_rp(DH)) % fa_cpr(DH); }
DASH_HD constexpr int fa_v_swz(int row, int DH) { return 4 * ((row / fa_rp(DH)) % (fa_cpr(DH) / 4)); }
DASH_HD constexpr int fa_rows_per_dma(int DH) { return 64 / fa_cpr(DH); }
DASH_HD constexpr int fa_dmas(int DH) { return kFaBN / fa_rows_per_dma(DH) / 4; }  // per wave and tile

// row in the tile that load i of wave gw (0..3 inside its group) fetches for this lane
DASH_HD int fa_dma_row(int gw, int i, int lane, int DH) {
    return (gw * fa_dmas(DH) + i) * fa_rows_per_dma(DH) + lane / fa_cpr(DH);
}
// lane offset inside a whole tile: row r of the tile, KV head g, the logical chunk that the swizzle maps to
// this lane's physical chunk (is_k selects the K or the V swizzle)
DASH_HD uint32_t fa_dma_voff(int r, int lane, int g, int Hkv, int DH, bool is_k) {
    const int pchunk = lane % fa_cpr(DH);
    const int lchunk = pchunk ^ (is_k ? fa_k_swz(r, DH) : fa_v_swz(r, DH));
    return (uint32_t)r * ((uint32_t)Hkv * DH * 2u) + ((uint32_t)g * DH + lchunk * 8) * 2u;
}
// the same for a tile that holds only rows_left (1..63) rows
DASH_HD uint32_t fa_dma_voff_tail(uint32_t voff, int r, int rows_left, int Hkv, int DH) {
    const int beyond = sa_max(r - (rows_left - 1), 0);  // rows past the last one
    return voff - (uint32_t)beyond * ((uint32_t)Hkv * DH * 2u);
}
DASH_HD size_t fa_tile_bytes(int Hkv, int DH) { return (size_t)kFaBN * Hkv * DH * 2; }

// Which key tiles a wave group works on: tile t of group grp is key tile t, or with two key groups (KG = 2) key tile 2 t + grp.
DASH_HD constexpr int fa_first_key(int t, int grp, int KG) { return (KG == 1 ? t : 2 * t + grp) * kFaBN; }
DASH_HD constexpr int fa_group_tiles(int all_tiles, int grp) { return (all_tiles - grp + 1) / 2; }  // KG = 2
// Two key groups: how many tiles ahead of the round a group requests K and V. Group 0 requests K(t + lead) and V(t + lead) in
// round t before its barrier t, group 1 after it; tiles below the lead are requested before the loop.
DASH_HD constexpr int fa_k_lead(int grp) { return grp == 0 ? 1 : 2; }
DASH_HD constexpr int fa_v_lead(int grp) { return grp == 0 ? 0 : 1; }

// Two key groups (128 query rows and half of the serial key loop per workgroup) where the loop's length or the last round
// of workgroups decides the time; one (256 rows) where the chip is full anyway, because either group of the split form
// fetches its own K and V tiles and its rounds take 14 % longer.
//  - causal: while the 128-row workgroups number at most two (head size 64: two and a half) per compute unit: the long ones
//    start first, the short ones fill up behind them. 28 heads of 128, us, one group / two: n = 177 13.6 / 11.5, 804 26.8 /
//    19.7, 2304 (504 workgroups) 56.4 / 51.6, 2400 (532) 56.0 / 59.2; 4 heads of 128: 16384 (512) 328 / 263; 16 heads of 64:
//    4096 (512) 65 / 49, 5000 (640) 78 / 76.
//  - otherwise all workgroups are equally long, so whole rounds are counted, a round of the split form being half as many
//    tiles: 28 heads of 128: 1152 (252 workgroups of 128 rows) 31 / 25, 1500 (336) 41 / 56; 16 heads of 64: 4300 (272 of 256
//    rows, 544 of 128) 137 / 122. A form whose count is less than 6 % (head size 64: 4 %) lower is not the faster one,
//    its last round being as likely a nearly empty one: 28 heads of 128, counts 4 / 3.99, 8001 758 / 823; 3 / 2.85, 5500 384 /
//    406; 16 heads of 64, 3 / 2.85, 9700 433 / 418; 4 / 3.99, 14001 1 / 1.03. The rows beyond the
//    last whole 256-row tile may also run as a launch of their own in the split form, so that a few of them do not cost a
//    round of all (4 % lower will do: the whole tiles keep their form): 28 heads of 128: 2400 111 / 101, 14001 7 / 6.67
//    rounds, 0.967 times; 32 of 128: 4100 298 / 270; 16 of 64: 4097 112 / 107, 8200 354 / 341.
//    Where the workgroups of those rows are all resident at once, the last rows run in the few-row form (32 rows and 8
//    key-splitting waves per workgroup, flash_few.hip): a quarter of a round and less. In the split form / so, us: 28 heads of
//    128 2305 102 / 88, 2559 111 / 95, 4700 317 / 288; 32 of 128 4100 284 / 260; 16 of 64 4097 108 / 91, 4351 114 / 94, 8200 336 / 303.
enum FaForm { FA_ONE = 0, FA_TWO = 1, FA_ONE_AND_TAIL = 2 };
inline bool fa_few_tail(int n, int Hq, int head_dim, int cu) {
    return (long long)((n % kFaBM + 31) / 32) * Hq <= (long long)cu * (head_dim == 64 ? 2 : 1);
}
inline FaForm fa_form(int n, int Hq, int head_dim, bool causal, int cu) {
    auto rounds = [&](long long wgs) { return (double)((wgs + cu - 1) / cu); };
    const long long one = (long long)((n + kFaBM - 1) / kFaBM) * Hq, two = (long long)((n + kFaBM / 2 - 1) / (kFaBM / 2)) * Hq;
    if (causal) return 2 * two <= (head_dim == 64 ? 5 : 4) * cu ? FA_TWO : FA_ONE;
    const double t_one = rounds(one), t_two = 0.57 * rounds(two);
    const int tail = n % kFaBM;
    if (tail > 0 && n > kFaBM) {
        const double t_tail = rounds(one - Hq) + (fa_few_tail(n, Hq, head_dim, cu) ? 0.25 : 0.57 * rounds(tail <= kFaBM / 2 ? Hq : 2 * Hq)) + 0.1;
        if (t_tail < 0.96 * t_one && t_tail < t_two) return FA_ONE_AND_TAIL;
    }
    return t_two < (head_dim == 64 ? 0.96 : 0.94) * t_one ? FA_TWO : FA_ONE;
}

// Order in which the tiled kernels' workgroups start under a causal mask (their lengths fall linearly): heaviest first, but with 2.25
// to 3.5 workgroups per unit the `later` heaviest may start in the second round and not in the first. Heaviest first, a unit that began
// with one of the longest gets no third workgroup and the others one too many: the last end 5 to 10 % after an even deal would.
// Started second, behind the middle ones, the longest fill up to a common end. By list scheduling that ends up to 8 % earlier
// and nowhere later (1 to 16 heads, 8 to 160 row tiles, a workgroup's fixed cost 0.5 or 0.8 of a tile); from 3.5 per unit on there are
// short ones enough to fill up with, and with few more than 2 it is the longest that end last. On the card it gains less, and only (fa_deal_pays)
//  - with 13 row tiles or more (two key groups: 24 of 128 rows), so that the lengths are graded finely enough to fill up with: 64
//    heads of 64 2779 rows (11) 83.8 / 86.5, 64 of 128 3035 rows (12) 142 / 145, 32 of 64 2445 rows (20 of 128) 45.5 / 46.1;
//  - up to 3.1 per unit, of head size 128 with 24 tiles or more up to 3.5: 40 heads of 128 5339 rows (3.3) 247 / 252, 24 of 64
//    9435 (3.5) 279 / 283; 16 of 128 13531 (3.3) 598 / 590;
//  - at head size 64, one key group, from 2.45 on and with the XCD map: 16 heads 9435 rows (2.3) 196 / 199, 12 heads of 3 groups,
//    without that map, 13019 rows 273 / 277.
// Measured, us, repeated for some milliseconds, heaviest first / this: head size 128, 8 heads 20443 rows 700 / 668, 16 heads 10203 361 / 340,
// 28 heads (4 KV) 5851 218 / 212, 6107 235 / 226, 6875 287 / 284, 32 heads 5083 191 / 180, 5339 208 / 196, 6107 261 / 255, 48 heads 3291
// 130 / 125, 12 of 3 groups 14811 560 / 547; head size 64, one key group, 16 heads 12251 316 / 312, 24 heads 7387 185 / 181, 40 heads
// 4059 105 / 102; two key groups, single calls, 16 heads 4935 72.9 / 68.1, 12 heads 6595 92.5 / 85.0, 8 heads 10081 135 / 122.
// slots: workgroups in that order on `units` units, one at a time each.
inline int fa_later(int slots, int units) {
    if (4 * slots <= 9 * units || 2 * slots >= 7 * units) return 0;
    return sa_min((int)((3.5 * units - slots) / 1.4 + 0.5), units);
}
// groups: key groups of the form; xcd_map: the workgroups of a KV head share XCDs
inline bool fa_deal_pays(int slots, int units, int n_qtiles, int head_dim, int groups, bool xcd_map) {
    const double per_unit = (double)slots / units;
    if (n_qtiles < (groups == 2 ? 24 : 13)) return false;
    if (head_dim == 64 && groups == 1 && (per_unit < 2.45 || !xcd_map)) return false;
    return per_unit < (head_dim == 128 && n_qtiles >= 24 ? 3.5 : 3.1);
}
// A launch's workgroups in one order: those of an XCD with the XCD map, else all.
DASH_HD bool fa_xcd_map(int Hkv) { return (Hkv <= 8 && 8 % Hkv == 0) || Hkv % 8 == 0; }
inline int fa_slots(int n_qtiles, int Hq, int Hkv) {
    if (!fa_xcd_map(Hkv)) return n_qtiles * Hq;
    const int items = n_qtiles * (Hq / Hkv);  // per KV head
    return Hkv <= 8 ? (items * Hkv + 7) / 8 : items * (Hkv / 8);
}
// How many of the heaviest start later in a causal launch of n_qtiles row tiles on cu units.
inline int fa_launch_later(int n_qtiles, int Hq, int Hkv, int head_dim, int groups, int cu) {
    const bool xcds = fa_xcd_map(Hkv);
    const int slots = fa_slots(n_qtiles, Hq, Hkv), units = xcds ? cu / 8 : cu;
    return units > 0 && fa_deal_pays(slots, units, n_qtiles, head_dim, groups, xcds) ? fa_later(slots, units) : 0;
}
DASH_HD int fa_item_of(int slot, int later, int units) {
    return slot < units ? slot + later : (slot < units + later ? slot - units : slot);
}

// ------------------------------------------------------------------------------------------------
// Attention over few rows: workgroups of 32 query rows whose waves take 32-key blocks of their own. A wave fetches whole
// blocks (few_loads instructions of fa_rows_per_dma rows each); lane offsets and clamping as above.
// ------------------------------------------------------------------------------------------------
constexpr int kFewKeys = 32;
DASH_HD constexpr int few_loads(int DH) { return kFewKeys / fa_rows_per_dma(DH); }
DASH_HD int few_row(int i, int lane, int DH) { return i * fa_rows_per_dma(DH) + lane / fa_cpr(DH); }
DASH_HD size_t few_block_bytes(int Hkv, int DH) { return (size_t)kFewKeys * Hkv * DH * 2; }
// The 32 query rows come the same way, dealt to the KW waves: instruction u (< few_q_loads) of a wave is the i-th of the few_loads, or none.
DASH_HD constexpr int few_q_loads(int DH, int KW) { return (few_loads(DH) + KW - 1) / KW; }
DASH_HD int few_q_index(int wave, int u, int DH, int KW) { return wave * few_q_loads(DH, KW) + u; }
DASH_HD size_t few_q_base(int row0, int Hq, int DH) { return (size_t)(row0 / kFewKeys) * few_block_bytes(Hq, DH); }
DASH_HD uint32_t few_q_voff(int row0, int n, int r, int lane, int head, int Hq, int DH) {
    return fa_dma_voff_tail(fa_dma_voff(r, lane, head, Hq, DH, true), r, sa_min(n - row0, kFewKeys), Hq, DH);
}
// Waves per workgroup of that form, 0: the tiled kernels (fa_form). Its workgroups fetch a key block for 32 rows where those fetch
// it for 128 or 256, so it pays while latencies and not the L2 decide: counted in its workgroups per compute unit, with a
// causal mask (half of the blocks, long rows first) up to 3, at head size 64 (half the bytes) 5; without one, where a third
// workgroup per unit is a whole round, 2. Measured, us, this form / the tiled ones; causal, 28 heads of 128: n = 64 5.7 / 8.4, 192
// 7.3 / 10.6, 512 10.8 / 15.2, 832 (2.8 per unit) 18.1 / 18.8, 960 (3.3) 20.8 / 20.2; 14 heads 2048 (3.5) 31.9 / 33.1, 8 heads 3072
// (3) 35.3 / 44.1, 4096 (4) 58 / 57; the longest that take it, 4 heads 6144 (3) 65 / 79, 2 heads 11000 (2.7) 110 / 134, one head 16385 (2)
// 151 / 191, one of 64 24577 (3) 162 / 188; 16 heads of 64: 64 4.7 / 6.8, 1024 9.8 / 15.2, 2560 (5) 27.2 / 27.8, 2816 34.1 / 29.8; 32 heads
// of 64: 1280 (5) 18.8 / 18.9. Without a mask, 28 heads of 128: 576 (2) 12.9 / 14.5, 640 (2.2) 20.6 / 15.4; 16 heads of 64: 1024 (2)
// 12.0 / 13.9, 1152 16.1 / 15.1.
// Eight waves, which halve the serial loop, while all workgroups are resident at once (one per unit, at head size 64 two): 4 heads of
// 128, causal, four waves / eight: 512 9.0 / 8.8, 2048 21.3 / 17.7; beyond that the smaller workgroups overlap better: 28 heads
// of 128 320 (1.1 per unit) 8.6 / 9.7.
inline int few_waves(int n, int Hq, int head_dim, bool causal, int cu) {
    const long long wgs = (long long)((n + 31) / 32) * Hq;
    if (wgs > (long long)cu * (causal ? (head_dim == 64 ? 5 : 3) : 2)) return 0;
    return wgs <= (long long)cu * (head_dim == 64 ? 2 : 1) ? 8 : 4;
}

// The rows beyond the last whole tile (fa_few_tail), keys cut over several workgroups per 32 rows and head: a unit fetches a key block in
// 0.9 us (head size 128: 1.7) per wave's turn whatever its waves, so a few workgroups that each go through all keys leave the chip idle.
// Parts of at least a block per wave, one workgroup per unit in all, and another launch to add them, 4 us; where that is expected to
// be shorter and the sums fit the scratch. 1: not cut. Layer calls without a causal mask, not cut / cut, us: 16 heads of 64 4097 rows 119.7 / 112.4,
// 4129 120.4 / 114.5, 4319 125.7 / 122.4, 8193 337.6 / 317.8; 28 of 128 2305 156.9 / 149.9, 2400 159.8 / 157.2, 4609 410 / 392; 32 of 128 4100 398.4 / 384.7.
// (Twice the waves per workgroup instead of twice the workgroups: 88.1 / 87.9 us of attention at 4097 rows.)
constexpr int kFewTailWaves = 8;
struct FewParts {
    int parts, blocks_per_part;
};
DASH_HD size_t few_part_bytes(int rows, int Hq, int DH) { return (size_t)rows * Hq * (DH + 2) * sizeof(float); }
inline FewParts few_tail_parts(int n, int Hq, int head_dim, int cu, size_t scratch_bytes) {
    const int rows = n % kFaBM, wgs = (rows + 31) / 32 * Hq, blocks = (n + kFewKeys - 1) / kFewKeys;
    FewParts best{1, blocks};
    if (rows == 0) return best;
    const double turn = head_dim == 64 ? 0.9 : 1.7;
    auto turns = [](int b) { return (b + kFewTailWaves - 1) / kFewTailWaves; };
    double best_us = turn * turns(blocks);
    for (int parts = 2; parts * wgs <= cu; ++parts) {
        const int per = kFewTailWaves * turns((blocks + parts - 1) / parts);
        const double us = turn * turns(per) + 4.0;
        if ((blocks + per - 1) / per != parts || parts * few_part_bytes(rows, Hq, head_dim) > scratch_bytes || us >= best_us) continue;
        best = FewParts{parts, per};
        best_us = us;
    }
    return best;
}

}  // namespace dash
