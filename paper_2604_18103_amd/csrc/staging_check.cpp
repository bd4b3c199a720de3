// Host-side check of the staging addresses (test infrastructure, CPU only; built as its own small library).
// Enumerates the direct global->LDS loads of a GEMM or attention launch with the functions the kernels use
// (staging_addr.h), forms each address the way the hardware does (64-bit uniform base + zero-extended 32-bit
// lane offset) and compares it with the address stated from first principles: the clamped row and column of
// the operand the lane is meant to fetch. A wrapped offset, a wrong clamp or a load outside the operand fails.
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "staging_addr.h"

using namespace dash;

namespace {

struct Counter {
    long long loads = 0;
    int status = 0;
    void fail(int code) {
        if (status == 0) status = code;
    }
};

// one GEMM workgroup: tile (tile_m, tile_n), half (0/1, used when MB == 2), K steps ks0 .. ks0 + n_ksteps - 1
void check_gemm_workgroup(int M, int K, int N, int MB, int tile_m, int tile_n, int half, int ks0, int n_ksteps,
                          Counter& c) {
    const int BM = 64 * MB;
    const int m0 = tile_m * kGM + (MB == 4 ? 0 : half * BM), n0 = tile_n * kGN;
    const int adma = gemm_adma(BM), bdma = gemm_bdma();
    const uint64_t a_bytes = (uint64_t)M * K * 2, b_bytes = (uint64_t)K * N * 2;
    for (int wave = 0; wave < kGWaves; ++wave)
        for (int lane = 0; lane < 64; ++lane) {
            for (int i = 0; i < adma; ++i) {
                const int row = gemm_a_row(wave, i, lane, adma);
                const int lchunk = gemm_a_lchunk(row, lane);
                if (row < 0 || row >= BM || lchunk < 0 || lchunk >= 8) c.fail(1);
                const uint64_t off = gemm_a_off(m0, M, K, row, lchunk);
                for (int st = 0; st < n_ksteps; ++st) {
                    const uint64_t addr = gemm_a_base_elem(m0, M, K, ks0) * 2 + (uint64_t)st * gemm_a_step_bytes() + off;
                    const int grow = sa_min(m0 + row, M - 1);
                    const uint64_t want = ((uint64_t)grow * K + (uint64_t)(ks0 + st) * kGK + lchunk * 8) * 2;
                    if (addr != want) c.fail(2);
                    if (addr + 16 > a_bytes) c.fail(3);
                    ++c.loads;
                }
            }
            for (int i = 0; i < bdma; ++i) {
                const int row = gemm_b_row(wave, i, lane);
                const int lchunk = gemm_b_lchunk(row, lane);
                if (row < 0 || row >= kGK || lchunk < 0 || lchunk >= 32) c.fail(4);
                const uint64_t off = gemm_b_off(n0, N, row, lchunk);
                for (int st = 0; st < n_ksteps; ++st) {
                    const uint64_t addr = gemm_b_base_elem(n0, N, ks0) * 2 + (uint64_t)st * gemm_b_step_bytes(N) + off;
                    const int gcol = sa_min(n0 + lchunk * 8, N - 8);
                    const uint64_t want = ((uint64_t)((ks0 + st) * kGK + row) * N + gcol) * 2;
                    if (addr != want) c.fail(5);
                    if (addr + 16 > b_bytes) c.fail(6);
                    ++c.loads;
                }
            }
        }
}

// a tile index is checked when the launch is small, or when it is the first or last tile of its row or column range
bool sampled(int idx, int count, bool all) { return all || idx == 0 || idx == count - 1; }

}  // namespace

extern "C" {

// Checks the launches that the library makes for C[M,N] = A[M,K] B[K,N] on `cu` compute units (split_bytes > 0:
// scratch for split-K is available): that the tile order visits every tile once, that the workgroups of the
// whole-tile launch take every whole tile exactly once, equally many per XCD (workgroup b runs on XCD b % 8), and
// every staging load. Products with more than 4096 tiles have their loads checked on the first and last row and
// column tiles only (the addresses are affine in the tile indices); the coverage is always checked in full.
// Returns 0 when everything is right; *n_loads = loads checked.
int dash_check_gemm_staging(int M, int K, int N, int cu, unsigned long long split_bytes, long long* n_loads) {
    Counter c;
    if (M <= 0 || K <= 0 || K % kGK != 0 || N <= 0 || N % 8 != 0) return -1;
    const GemmPlan g = gemm_plan(M, K, N, cu, split_bytes > 0, (size_t)split_bytes);
    const bool all = g.tiles <= 4096;
    const bool plain = g.plain != 0;
    // the tile order is a bijection onto the tile grid
    {
        std::vector<char> seen((size_t)g.tiles, 0);
        for (int idx = 0; idx < g.tiles; ++idx) {
            int tm = -1, tn = -1;
            gemm_tile_of(idx, g.mt, g.nt, plain, tm, tn);
            if (tm < 0 || tm >= g.mt || tn < 0 || tn >= g.nt || seen[(size_t)tn * g.mt + tm]) {
                c.fail(9);
                break;
            }
            seen[(size_t)tn * g.mt + tm] = 1;
        }
    }
    auto loads_wanted = [&](int tm, int tn) { return sampled(tm, g.mt, all) || sampled(tn, g.nt, all); };
    if (g.parts >= 2) {
        for (int tile = 0; tile < g.tiles; ++tile) {
            int tm, tn;
            gemm_tile_of(tile, g.mt, g.nt, plain, tm, tn);
            if (!loads_wanted(tm, tn)) continue;
            for (int part = 0; part < g.parts; ++part) {
                const int ks0 = part * g.ksteps_per_part;
                const int nk = sa_min(g.ksteps_per_part, g.ksteps - ks0);
                if (nk <= 0) c.fail(7);
                check_gemm_workgroup(M, K, N, 4, tm, tn, 0, ks0, nk, c);
            }
        }
    } else {
        if (g.full + g.rest != g.tiles || g.full < 0 || g.rest < 0) c.fail(8);
        if (g.full > 0 && (g.grid < g.full || g.grid > g.full + 15)) c.fail(10);
        std::vector<int> taken((size_t)g.tiles, 0);
        int per_xcd[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int b = 0; b < (g.full > 0 ? g.grid : 0); ++b) {
            const int idx = gemm_index_of(b, g.full, plain, g.seg);
            if (idx < 0) continue;
            if (idx >= g.full) {
                c.fail(11);
                continue;
            }
            ++taken[(size_t)idx];
            ++per_xcd[b % 8];
            int tm, tn;
            gemm_tile_of(idx, g.mt, g.nt, plain, tm, tn);
            if (loads_wanted(tm, tn) || idx == g.full - 1) check_gemm_workgroup(M, K, N, 4, tm, tn, 0, 0, g.ksteps, c);
        }
        for (int t = 0; t < g.full; ++t)
            if (taken[(size_t)t] != 1) c.fail(12);
        for (int x = 0; x < 8; ++x)  // no XCD has more than a stretch's worth, none is short by more than the padding
            if (per_xcd[x] > (g.full + 7) / 8 || per_xcd[x] + 8 < g.full / 8) c.fail(13);
        const int rp = split_bytes > 0 ? rest_parts(g, cu, (size_t)split_bytes) : 1, per = (g.ksteps + rp - 1) / rp;
        if (rp > 1 && (size_t)rp * 2 * g.rest * rest_sum_elems() * 4 > split_bytes) c.fail(14);
        for (int b = 0; b < 2 * g.rest; ++b) {  // half tiles: workgroup b handles half b % 2 of tile full + b / 2
            int tm, tn;
            gemm_tile_of(g.full + b / 2, g.mt, g.nt, plain, tm, tn);
            for (int part = 0; part < rp; ++part) {
                if (g.ksteps - part * per <= 0) c.fail(15);
                check_gemm_workgroup(M, K, N, 2, tm, tn, b % 2, part * per, sa_min(per, g.ksteps - part * per), c);
            }
        }
    }
    if (n_loads) *n_loads = c.loads;
    return c.status;
}

// The launch decomposition of a product as launch_gemm makes it: out[0..7] = tiles, K steps, parts (>= 2: split-K),
// K steps per part, whole 256-row tiles, tiles run as 128-row half tiles, plain tile order (1) or column panels
// dealt to the XCDs in stretches (0), workgroups of the whole-tile launch.
void dash_gemm_launch_plan(int M, int K, int N, int cu, unsigned long long split_bytes, int* out) {
    const GemmPlan g = gemm_plan(M, K, N, cu, split_bytes > 0, (size_t)split_bytes);
    out[0] = g.tiles; out[1] = g.ksteps; out[2] = g.parts; out[3] = g.ksteps_per_part; out[4] = g.full;
    out[5] = g.rest; out[6] = g.plain; out[7] = g.grid;
}

// The lower tiles of a round (row_plan): out[0..1] = 16-row blocks per wave (0: none), 256-row row tiles before them.
void dash_row_plan(int M, int K, int N, int cu, unsigned long long split_bytes, int* out) {
    const RowPlan r = row_plan(gemm_plan(M, K, N, cu, split_bytes > 0, (size_t)split_bytes), M, cu);
    out[0] = r.rb; out[1] = r.whole;
}

// Checks the launch of rows [row0, row1) on tiles of 32 rb rows: every tile is taken once, every row lies in one tile, the lower
// tiles' launch fits one round, every load of the A tile fetches the clamped row and fills the tile's rows.
int dash_check_rows(int M, int K, int N, int row0, int row1, int rb) {
    Counter c;
    const int BM = 32 * rb, mt = (row1 - row0 + BM - 1) / BM, nt = (N + kGN - 1) / kGN, full = mt * nt, seg = (full + 7) / 8;
    const bool plain = rows_plain(mt, rb);
    if (row0 % kGM != 0 || row1 > M || (row1 < M && (row1 - row0) % BM != 0)) c.fail(1);
    std::vector<int> taken((size_t)full, 0);
    for (int b = 0; b < (plain ? full : 8 * seg); ++b) {
        const int idx = gemm_index_of(b, full, plain, seg);
        if (idx < 0) continue;
        if (idx >= full) { c.fail(2); continue; }
        int tm = -1, tn = -1;
        gemm_tile_of(idx, mt, nt, plain, tm, tn);
        if (tm < 0 || tm >= mt || tn < 0 || tn >= nt) { c.fail(3); continue; }
        ++taken[(size_t)tn * mt + tm];
    }
    for (const int t : taken)
        if (t != 1) c.fail(4);
    const int adma = gemm_adma(BM), rows = 8 * kGWaves * adma;  // fetched rows: at least the tile's
    for (int tm = 0; tm < mt; ++tm) {
        const int m0 = row0 + tm * BM;
        if (m0 >= M) c.fail(5);
        std::vector<char> seen((size_t)rows * 8, 0);
        for (int wave = 0; wave < kGWaves; ++wave)
            for (int lane = 0; lane < 64; ++lane)
                for (int i = 0; i < adma; ++i) {
                    const int row = gemm_a_row(wave, i, lane, adma), lchunk = gemm_a_lchunk(row, lane);
                    if (row < 0 || row >= rows || lchunk < 0 || lchunk >= 8) { c.fail(6); continue; }
                    seen[(size_t)row * 8 + lchunk] = 1;
                    const uint64_t addr = (uint64_t)gemm_a_base_elem(m0, M, K, 0) * 2 + gemm_a_off(m0, M, K, row, lchunk);
                    if (addr != ((uint64_t)sa_min(m0 + row, M - 1) * K + lchunk * 8) * 2) c.fail(7);
                    if (addr + (uint64_t)(K / kGK - 1) * gemm_a_step_bytes() + 16 > (uint64_t)M * K * 2) c.fail(8);
                }
        for (const char s : seen)
            if (!s) c.fail(9);
    }
    if (rows < BM || (rb == 8 && rows != BM)) c.fail(10);
    return c.status;
}

// Column tiles that one XCD reads in the launch of rows [row0, row1) on tiles of 32 rb rows: the most.
int dash_rows_columns(int N, int row0, int row1, int rb) {
    const int mt = (row1 - row0 + 32 * rb - 1) / (32 * rb), nt = (N + kGN - 1) / kGN, full = mt * nt, seg = (full + 7) / 8;
    const bool plain = rows_plain(mt, rb);
    int most = 0;
    for (int xcd = 0; xcd < 8; ++xcd) {
        std::vector<char> seen((size_t)nt, 0);
        for (int b = xcd; b < (plain ? full : 8 * seg); b += 8) {
            const int idx = gemm_index_of(b, full, plain, seg);
            int tm = 0, tn = 0;
            if (idx >= 0) {
                gemm_tile_of(idx, mt, nt, plain, tm, tn);
                seen[(size_t)tn] = 1;
            }
        }
        int columns = 0;
        for (const char c : seen) columns += c;
        most = sa_max(most, columns);
    }
    return most;
}

// The workgroups of a small-tile launch of `tiles` tiles in `parts` K parts: the most that one XCD gets, or -1 if some tile of
// some part is not taken exactly once.
int dash_small_deal(int tiles, int parts) {
    std::vector<int> taken((size_t)tiles * parts, 0), xcd(8, 0);
    for (int b = 0; b < 8 * ((tiles * parts + 7) / 8); ++b) {
        int tile = -1, part = -1;
        if (!small_work_of(b, tiles, parts, tile, part)) continue;
        if (tile < 0 || tile >= tiles || part < 0 || part >= parts) return -1;
        ++taken[(size_t)part * tiles + tile];
        ++xcd[(size_t)(b % 8)];
    }
    for (const int t : taken)
        if (t != 1) return -1;
    return *std::max_element(xcd.begin(), xcd.end());
}

// Checks the small-tile product in form `form` on every shape: that the workgroups take every tile exactly once and that
// every staging load of every K group fetches the clamped row and column its lane is meant to.
int dash_check_small_staging(int M, int K, int N, int form, long long* n_loads) {
    Counter c;
    if (M <= 0 || K <= 0 || K % kGK != 0 || N <= 0 || N % 8 != 0 || form < 0 || form > kTallForm) return -1;
    const SmallForm& f = kSmallForms[form];
    const int mt = (M + f.BM - 1) / f.BM, nt = (N + f.BN - 1) / f.BN, tiles = mt * nt;
    const uint64_t a_bytes = (uint64_t)M * K * 2, b_bytes = (uint64_t)K * N * 2;
    if (dash_small_deal(tiles, 1) < 0) c.fail(2);
    std::vector<char> a_seen((size_t)f.BM * 8, 0), b_seen((size_t)kGK * (f.BN / 8), 0);
    for (int tm = 0; tm < mt; ++tm)
        for (int tn = 0; tn < nt; ++tn) {
            if (tm != 0 && tm != mt - 1 && tn != 0 && tn != nt - 1) continue;  // the addresses are affine in the tile
            const int m0 = tm * f.BM, n0 = tn * f.BN;
            for (int wave = 0; wave < kSWaves; ++wave)
                for (int lane = 0; lane < 64; ++lane) {
                    for (int i = 0; i < small_adma(f.BM); ++i) {
                        const int row = small_a_row(wave, i, lane, f.BM), lchunk = gemm_a_lchunk(row, lane);
                        if (row < 0 || row >= f.BM || lchunk < 0 || lchunk >= 8) { c.fail(3); continue; }
                        a_seen[(size_t)row * 8 + lchunk] = 1;
                        const uint64_t off = gemm_a_off(m0, M, K, row, lchunk);
                        for (int ks = 0; ks < K / kGK; ++ks) {
                            const uint64_t addr = gemm_a_base_elem(m0, M, K, ks % f.KW) * 2 + (uint64_t)(ks - ks % f.KW) * gemm_a_step_bytes() + off;
                            if (addr != ((uint64_t)sa_min(m0 + row, M - 1) * K + (uint64_t)ks * kGK + lchunk * 8) * 2) c.fail(4);
                            if (addr + 16 > a_bytes) c.fail(5);
                            ++c.loads;
                        }
                    }
                    for (int i = 0; i < small_bdma(f.BN); ++i) {
                        const int row = small_b_row(wave, i, lane, f.BN), lchunk = small_b_lchunk(row, lane, f.BN);
                        if (row < 0 || row >= kGK || lchunk < 0 || lchunk >= f.BN / 8) { c.fail(6); continue; }
                        b_seen[(size_t)row * (f.BN / 8) + lchunk] = 1;
                        const uint64_t off = gemm_b_off(n0, N, row, lchunk);
                        for (int ks = 0; ks < K / kGK; ++ks) {
                            const uint64_t addr = gemm_b_base_elem(n0, N, ks % f.KW) * 2 + (uint64_t)(ks - ks % f.KW) * gemm_b_step_bytes(N) + off;
                            if (addr != ((uint64_t)(ks * kGK + row) * N + sa_min(n0 + lchunk * 8, N - 8)) * 2) c.fail(7);
                            if (addr + 16 > b_bytes) c.fail(8);
                            ++c.loads;
                        }
                    }
                }
        }
    for (char v : a_seen) if (!v) c.fail(9);
    for (char v : b_seen) if (!v) c.fail(10);
    if (n_loads) *n_loads = c.loads;
    return c.status;
}

// Checks the tiles of `bm` rows and 64 columns whose waves take K steps of their own: every load fetches the clamped row and column of its
// wave's step, a step's loads fill the stage, and the waves' steps are all steps of all `parts`.
int dash_check_few_tiles(int M, int K, int N, int bm, int parts, long long* n_loads) {
    Counter c;
    if (M <= 0 || K <= 0 || K % kGK != 0 || N <= 0 || N % 8 != 0 || bm % 16 != 0 || bm > 64 || parts < 1) return -1;
    const int mt = (M + bm - 1) / bm, nt = (N + kFewTileN - 1) / kFewTileN, ksteps = K / kGK, per = (ksteps + parts - 1) / parts;
    const uint64_t a_bytes = (uint64_t)M * K * 2, b_bytes = (uint64_t)K * N * 2;
    if (dash_small_deal(mt * nt, parts) < 0) c.fail(2);
    if (few_tile_smem_bytes(bm) > 160 * 1024) c.fail(3);
    std::vector<char> a_seen((size_t)bm * 8, 0), b_seen((size_t)kGK * (kFewTileN / 8), 0), step_seen((size_t)ksteps, 0);
    for (int tm = 0; tm < mt; ++tm)
        for (int tn = 0; tn < nt; ++tn) {
            if (tm != 0 && tm != mt - 1 && tn != 0 && tn != nt - 1) continue;
            const int m0 = tm * bm, n0 = tn * kFewTileN;
            for (int part = 0; part < parts; ++part)
                for (int wave = 0; wave < kFewTileWaves; ++wave) {
                    const int ks0 = part * per, steps = sa_min(per, ksteps - ks0), mine = (steps - wave + kFewTileWaves - 1) / kFewTileWaves;
                    uint64_t a_base = gemm_a_base_elem(m0, M, K, ks0 + wave) * 2, b_base = gemm_b_base_elem(n0, N, ks0 + wave) * 2;
                    for (int t = 0; t < mine; ++t) {
                        const int ks = ks0 + wave + t * kFewTileWaves;
                        if (ks >= ksteps || ks >= ks0 + per) { c.fail(4); continue; }
                        step_seen[(size_t)ks] = 1;
                        for (int lane = 0; lane < 64; ++lane) {
                            for (int i = 0; i < bm / 8; ++i) {
                                const int row = few_tile_row(i, lane), lchunk = gemm_a_lchunk(row, lane);
                                if (row < 0 || row >= bm || lchunk < 0 || lchunk >= 8) { c.fail(5); continue; }
                                a_seen[(size_t)row * 8 + lchunk] = 1;
                                const uint64_t addr = a_base + gemm_a_off(m0, M, K, row, lchunk);
                                if (addr != ((uint64_t)sa_min(m0 + row, M - 1) * K + (uint64_t)ks * kGK + lchunk * 8) * 2) c.fail(6);
                                if (addr + 16 > a_bytes) c.fail(7);
                                ++c.loads;
                            }
                            for (int i = 0; i < kGK / 8; ++i) {
                                const int row = few_tile_row(i, lane), lchunk = small_b_lchunk(row, lane, kFewTileN);
                                if (row < 0 || row >= kGK || lchunk < 0 || lchunk >= kFewTileN / 8) { c.fail(8); continue; }
                                b_seen[(size_t)row * (kFewTileN / 8) + lchunk] = 1;
                                const uint64_t addr = b_base + gemm_b_off(n0, N, row, lchunk);
                                if (addr != ((uint64_t)(ks * kGK + row) * N + sa_min(n0 + lchunk * 8, N - 8)) * 2) c.fail(9);
                                if (addr + 16 > b_bytes) c.fail(10);
                                ++c.loads;
                            }
                        }
                        a_base += kFewTileWaves * gemm_a_step_bytes();
                        b_base += kFewTileWaves * gemm_b_step_bytes(N);
                    }
                }
        }
    for (char v : a_seen) if (!v) c.fail(11);
    for (char v : b_seen) if (!v) c.fail(12);
    for (char v : step_seen) if (!v) c.fail(13);
    if (n_loads) *n_loads = c.loads;
    return c.status;
}

// K parts of the left-over half tiles, 1: one pass.
int dash_rest_parts(int M, int K, int N, int cu, unsigned long long scratch) {
    return rest_parts(gemm_plan(M, K, N, cu, scratch > 0, (size_t)scratch), cu, (size_t)scratch);
}

// How a product whose columns have to lie in one tile by heads of `head` columns (0: none) is launched: out[0..4] = small form (-1: large
// or few-row tiles), tiles, K parts, K steps per part, rows of the few-row tiles (0: not those); out[5..7] = if on large tiles, their K parts,
// the half tiles left over, and those tiles' K parts.
void dash_product_plan(int M, int K, int N, int cu, int norms, int head, unsigned long long scratch, int* out) {
    const GemmPlan g = gemm_plan(M, K, N, cu, scratch > 0, (size_t)scratch);
    const SmallPlan p = product_plan(g, M, K, N, cu, norms != 0, head, scratch > 0, (size_t)scratch);
    out[0] = p.form; out[1] = p.tiles; out[2] = p.parts; out[3] = p.ksteps_per_part; out[4] = p.few_rows;
    out[5] = g.parts; out[6] = g.rest; out[7] = rest_parts(g, cu, (size_t)scratch);
}

// The item that each of `slots` workgroups takes on `units` units.
void dash_fa_order(int slots, int units, int* out) {
    for (int s = 0; s < slots; ++s) out[s] = fa_item_of(s, fa_later(slots, units), units);
}

// The workgroups of a causal launch in one order, and how many of them start later.
int dash_fa_launch_later(int n_qtiles, int Hq, int Hkv, int head_dim, int groups, int cu, int* slots) {
    *slots = fa_slots(n_qtiles, Hq, Hkv);
    return fa_launch_later(n_qtiles, Hq, Hkv, head_dim, groups, cu);
}

// The form attention takes among the tiled kernels (dash_few_waves = 0): 0 one key group, 1 two, 2 one with the rows beyond the last whole tile as a launch of their own.
int dash_fa_form(int n, int Hq, int head_dim, int causal, int cu) { return (int)fa_form(n, Hq, head_dim, causal != 0, cu); }

// Checks every K and V staging load of the attention launch over n rows (K, V: [n][Hkv][DH] bf16): for each
// query tile of 256 rows, the tiles of 64 keys it fetches. Returns 0 when all loads are right.
int dash_check_flash_staging(int n, int Hkv, int DH, int causal, long long* n_loads) {
    Counter c;
    if (n <= 0 || Hkv <= 0 || (DH != 64 && DH != 128)) return -1;
    const uint64_t kv_bytes = (uint64_t)n * Hkv * DH * 2;
    const int n_qtiles = (n + 255) / 256;
    const int dmas = fa_dmas(DH), cpr = fa_cpr(DH);
    // the tiles a query tile fetches are a prefix of those of the last query tile: the last two are checked
    for (int qt = n_qtiles - 1; qt >= 0 && qt >= n_qtiles - 2; --qt) {
        const int kv_end = causal ? sa_min(n, qt * 256 + 256) : n;
        const int n_tiles = (kv_end + kFaBN - 1) / kFaBN;
        for (int g = 0; g < Hkv; ++g)
            for (int is_k = 0; is_k < 2; ++is_k)
                for (int gw = 0; gw < 4; ++gw)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int i = 0; i < dmas; ++i) {
                            const int r = fa_dma_row(gw, i, lane, DH);
                            if (r < 0 || r >= kFaBN) c.fail(1);
                            const uint32_t voff = fa_dma_voff(r, lane, g, Hkv, DH, is_k != 0);
                            const int swz = is_k ? fa_k_swz(r, DH) : fa_v_swz(r, DH);
                            const int lchunk = (lane % cpr) ^ swz;
                            if (lchunk < 0 || lchunk >= cpr) c.fail(2);
                            for (int t = 0; t < n_tiles; ++t) {
                                const int rows_left = n - t * kFaBN;
                                if (rows_left < 1) c.fail(3);
                                const uint32_t off = rows_left >= kFaBN ? voff : fa_dma_voff_tail(voff, r, rows_left, Hkv, DH);
                                const uint64_t addr = (uint64_t)t * fa_tile_bytes(Hkv, DH) + off;
                                const int grow = sa_min(t * kFaBN + r, n - 1);
                                const uint64_t want = ((uint64_t)grow * Hkv + g) * DH * 2 + (uint64_t)lchunk * 16;
                                if (addr != want) c.fail(4);
                                if (addr + 16 > kv_bytes) c.fail(5);
                                ++c.loads;
                            }
                        }
    }
    if (n_loads) *n_loads = c.loads;
    return c.status;
}

// The same for the form with two key groups over the query rows [row0, row1) (128-row tiles; row0 > 0: the launch of the last
// rows alone): every key tile is fetched once as K and once as V, by its group; every load is inside the operand and fetches the
// clamped row; the positions that a causal mask reads lie in the workgroup's own 128; and a stage is written only after the
// barrier that follows the last read of what it held, and read only after a barrier that follows the wait for it. (Reads:
// round t reads K(t) and V(t - 1), after barrier t - 1. A request of round t lies before barrier t in group 0 and is waited
// for before it, after barrier t in group 1 and waited for before barrier t + 1.)
int dash_check_flash_groups(int n, int Hkv, int DH, int causal, int row0, int row1, long long* n_loads) {
    Counter c;
    if (n <= 0 || Hkv <= 0 || (DH != 64 && DH != 128) || row0 < 0 || row0 % kFaBM != 0 || row1 <= row0 || row1 > n) return -1;
    constexpr int KG = 2, BM = kFaBM / KG;
    const uint64_t kv_bytes = (uint64_t)n * Hkv * DH * 2;
    const int n_qtiles = (row1 - row0 + BM - 1) / BM, dmas = fa_dmas(DH), cpr = fa_cpr(DH);
    for (int qt = 0; qt < n_qtiles; ++qt) {
        if (qt > 1 && qt < n_qtiles - 2) continue;
        const int tile_row0 = row0 + qt * BM;
        const int kv_end = causal ? sa_min(n, tile_row0 + BM) : n;
        const int all_tiles = (kv_end + kFaBN - 1) / kFaBN, n_rounds = (all_tiles + 1) / 2;
        std::vector<int> fetched((size_t)all_tiles * 2, 0);
        for (int grp = 0; grp < 2; ++grp) {
            const int n_tiles = fa_group_tiles(all_tiles, grp);
            if (n_tiles > n_rounds) c.fail(6);
            for (int is_k = 0; is_k < 2; ++is_k)
                for (int t = 0; t < n_tiles; ++t) {
                    const int key0 = fa_first_key(t, grp, KG), rows_left = n - key0;
                    if (key0 / kFaBN >= all_tiles) {
                        c.fail(7);
                        continue;
                    }
                    ++fetched[(size_t)(key0 / kFaBN) * 2 + is_k];
                    if (rows_left < 1) c.fail(3);
                    const int lead = is_k ? fa_k_lead(grp) : fa_v_lead(grp);
                    auto requested = [&](int u) { return u < lead ? -1 : u - lead + grp; };      // barriers passed by then
                    const int readable = requested(t) < 0 ? (is_k && t == 0 ? 0 : 1) : requested(t) + 1;
                    const int read = is_k ? t : t + 1;
                    if (readable > read) c.fail(8);
                    if (t + 2 < n_tiles && requested(t + 2) <= read) c.fail(9);
                    if (t > 2 && t < n_tiles - 2) continue;  // the addresses are affine in the tile
                    for (int g = 0; g < Hkv; ++g)
                        for (int gw = 0; gw < 4; ++gw)
                            for (int lane = 0; lane < 64; ++lane)
                                for (int i = 0; i < dmas; ++i) {
                                    const int r = fa_dma_row(gw, i, lane, DH);
                                    const uint32_t voff = fa_dma_voff(r, lane, g, Hkv, DH, is_k != 0);
                                    const int lchunk = (lane % cpr) ^ (is_k ? fa_k_swz(r, DH) : fa_v_swz(r, DH));
                                    const uint32_t off = rows_left >= kFaBN ? voff : fa_dma_voff_tail(voff, r, rows_left, Hkv, DH);
                                    const uint64_t addr = (uint64_t)(key0 / kFaBN) * fa_tile_bytes(Hkv, DH) + off;
                                    const int grow = sa_min(key0 + r, n - 1);
                                    if (addr != ((uint64_t)grow * Hkv + g) * DH * 2 + (uint64_t)lchunk * 16) c.fail(4);
                                    if (addr + 16 > kv_bytes) c.fail(5);
                                    ++c.loads;
                                }
                }
            for (int w = 0; w < 4 && causal; ++w)  // a wave's masked tiles: those that reach beyond its first row
                for (int t = 0; t < n_tiles; ++t) {
                    const int q0 = tile_row0 + 32 * w, key0 = fa_first_key(t, grp, KG);
                    const int wave_kend = q0 >= n ? 0 : sa_min(n, q0 + 32);
                    if (key0 < wave_kend && key0 + kFaBN - 1 > q0 && (key0 < tile_row0 || key0 + kFaBN > tile_row0 + BM)) c.fail(10);
                }
        }
        for (const int f : fetched)
            if (f != 1) c.fail(11);
    }
    if (n_loads) *n_loads = c.loads;
    return c.status;
}

// Attention over few rows (workgroups of 32 query rows, `waves` waves): over all query tiles every 32-key block that a tile can see
// is fetched by exactly one wave, once as K and once as V; every load is inside the operand, fetches the clamped row, and
// together they fill a stage; the positions that a causal mask reads are those of the tile's own rows.
int dash_check_flash_few(int n, int Hkv, int DH, int causal, int waves, long long* n_loads) {
    Counter c;
    if (n <= 0 || Hkv <= 0 || (DH != 64 && DH != 128) || waves <= 0) return -1;
    const uint64_t kv_bytes = (uint64_t)n * Hkv * DH * 2;
    const int cpr = fa_cpr(DH);
    for (int qt = 0; qt < (n + 31) / 32; ++qt) {
        const int row0 = 32 * qt, kend = causal ? sa_min(n, row0 + 32) : n, n_blocks = (kend + kFewKeys - 1) / kFewKeys;
        std::vector<int> taken((size_t)n_blocks, 0);
        for (int w = 0; w < waves; ++w)
            for (int b = w; b < n_blocks; b += waves) {
                ++taken[(size_t)b];
                const int rows_left = n - b * kFewKeys;
                if (rows_left < 1) c.fail(3);
                if (causal && b * kFewKeys + kFewKeys - 1 > row0 && b * kFewKeys != row0) c.fail(10);
                for (int g = 0; g < Hkv; ++g)
                    for (int is_k = 0; is_k < 2; ++is_k) {
                        std::vector<char> filled((size_t)kFewKeys * cpr, 0);
                        for (int lane = 0; lane < 64; ++lane)
                            for (int i = 0; i < few_loads(DH); ++i) {
                                const int r = few_row(i, lane, DH);
                                if (r < 0 || r >= kFewKeys || r * cpr + lane % cpr != i * 64 + lane) { c.fail(1); continue; }
                                filled[(size_t)r * cpr + lane % cpr] = 1;
                                const int lchunk = (lane % cpr) ^ (is_k ? fa_k_swz(r, DH) : fa_v_swz(r, DH));
                                if (lchunk < 0 || lchunk >= cpr) c.fail(2);
                                const uint32_t voff = fa_dma_voff(r, lane, g, Hkv, DH, is_k != 0);
                                const uint32_t off = rows_left >= kFewKeys ? voff : fa_dma_voff_tail(voff, r, rows_left, Hkv, DH);
                                const uint64_t addr = (uint64_t)b * few_block_bytes(Hkv, DH) + off;
                                const int grow = sa_min(b * kFewKeys + r, n - 1);
                                if (addr != ((uint64_t)grow * Hkv + g) * DH * 2 + (uint64_t)lchunk * 16) c.fail(4);
                                if (addr + 16 > kv_bytes) c.fail(5);
                                ++c.loads;
                            }
                        for (const char f : filled)
                            if (!f) c.fail(6);
                    }
            }
        for (const int t : taken)
            if (t != 1) c.fail(11);
    }
    if (n_loads) *n_loads = c.loads;
    return c.status;
}

// ... and the query rows of its launch over rows [row_base, n): in every workgroup each of the 32 rows' pieces is fetched once by one
// wave, clamped, in range, to its place.
int dash_check_few_queries(int n, int Hq, int DH, int waves, int row_base, long long* n_loads) {
    Counter c;
    if (n <= row_base || row_base % 32 != 0 || Hq <= 0 || (DH != 64 && DH != 128) || waves <= 0) return -1;
    const int cpr = fa_cpr(DH), loads = few_loads(DH);
    for (int qt = 0; qt < (n - row_base + 31) / 32; ++qt)
        for (int head = 0; head < Hq; ++head) {
            const int row0 = row_base + 32 * qt;
            std::vector<int> filled((size_t)32 * cpr, 0);
            for (int wave = 0; wave < waves; ++wave)
                for (int u = 0; u < few_q_loads(DH, waves); ++u) {
                    const int i = few_q_index(wave, u, DH, waves);
                    if (loads % waves != 0 && i >= loads) continue;  // as the kernel
                    for (int lane = 0; lane < 64; ++lane) {
                        const int r = few_row(i, lane, DH), place = i * 64 + lane;  // 16-byte pieces of the stage
                        if (i >= loads || r < 0 || r >= 32 || place / cpr != r) { c.fail(1); continue; }
                        ++filled[(size_t)place];
                        const int lchunk = (place % cpr) ^ fa_k_swz(r, DH);
                        const uint64_t addr = (uint64_t)few_q_base(row0, Hq, DH) + few_q_voff(row0, n, r, lane, head, Hq, DH);
                        if (addr != ((uint64_t)sa_min(row0 + r, n - 1) * Hq + head) * DH * 2 + (uint64_t)lchunk * 16) c.fail(4);
                        if (addr + 16 > (uint64_t)n * Hq * DH * 2) c.fail(5);
                        ++c.loads;
                    }
                }
            for (const int f : filled)
                if (f != 1) c.fail(6);
        }
    if (n_loads) *n_loads = c.loads;
    return c.status;
}

// Parts of the keys of the rows beyond the last whole tile, and the key blocks of a part.
int dash_few_tail_parts(int n, int Hq, int head_dim, int cu, size_t scratch_bytes, int* blocks_per_part) {
    const FewParts g = few_tail_parts(n, Hq, head_dim, cu, scratch_bytes);
    *blocks_per_part = g.blocks_per_part;
    return g.parts;
}
// Bytes of the layer call's scratch that the projection and those parts share.
size_t dash_wo_scratch_bytes(int n, int K, int N) { return wo_scratch_bytes(n, K, N); }
// Whether the rows beyond the last whole tile take the few-row form (where dash_fa_form is 2).
int dash_fa_few_tail(int n, int Hq, int head_dim, int cu) { return fa_few_tail(n, Hq, head_dim, cu); }

// Waves of the few-row form, 0 where the tiled kernels run.
int dash_few_waves(int n, int Hq, int head_dim, int causal, int cu) { return few_waves(n, Hq, head_dim, causal != 0, cu); }

}  // extern "C"
