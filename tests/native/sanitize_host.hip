// Driver for a sanitizer pass over the HOST code of the library (argument validation, grid
// preparation, the launch plan and its scratch layout), built with AddressSanitizer and
// UndefinedBehaviorSanitizer on the host side only.  Runs with or without a GPU: without one
// every compute entry point must stop at PLOGP_EDEVICE after its host-side work.
#include "../../include/plogp.h"
#include "../../include/plogp_profile.h"
#include "../../paper_cs_0408034_amd/csrc/plogp_internal.hpp"

#include <cstdio>
#include <cstdlib>
#include <vector>

static unsigned long long state = 0x243F6A8885A308D3ull;
static unsigned long long next_u64()
{
    unsigned long long z = (state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static int pick(int lo, int hi) { return lo + (int)(next_u64() % (unsigned long long)(hi - lo + 1)); }

#define CHECK(cond)                                                            \
    do {                                                                       \
        if (!(cond)) { std::printf("check failed at line %d: %s\n", __LINE__, #cond); return 1; } \
    } while (0)

int main()
{
    // ---- the C ABI: refused arguments, then valid ones (PLOGP_OK with a GPU, PLOGP_EDEVICE without)
    plogp_table *tab = nullptr;
    plogp_grid *grid = nullptr;
    const double x[4] = {1.0, 8.0, 64.0, 4096.0}, y[4] = {3.0, 3.5, 5.0, 40.0}, ybad[4] = {3.0, -1.0, 5.0, 40.0};
    CHECK(plogp_load_table(nullptr, y, 4, 1.0, &tab) == PLOGP_EINVAL);
    CHECK(plogp_load_table(x, ybad, 4, 1.0, &tab) == PLOGP_EINVAL);
    CHECK(plogp_load_table(x, y, 1, 1.0, &tab) == PLOGP_EINVAL);
    const int st_tab = plogp_load_table(x, y, 4, 7.25, &tab);
    CHECK(st_tab == PLOGP_OK || st_tab == PLOGP_EDEVICE);
    std::vector<uint64_t> m, s;
    std::vector<uint32_t> P;
    for (int i = 0; i < 300; ++i) m.push_back(8ull * (1 + next_u64() % 100000));
    for (int i = 0; i < 40; ++i) m.push_back(m[i]);                     // repeats
    for (uint32_t p = 2; p < 3000; p += 1 + p / 7) P.push_back(p);
    for (uint64_t v = 8; v <= (1u << 20); v *= 2) s.push_back(v);
    plogp_grid_desc d = {m.data(), m.size(), P.data(), P.size(), s.data(), s.size(), PLOGP_NO_CAP, 8, PLOGP_MASK_EVERY};
    const int st_grid = plogp_grid_create(&d, &grid);
    CHECK(st_grid == PLOGP_OK || st_grid == PLOGP_EDEVICE);
    plogp_grid_desc bad = d;
    bad.strategy_mask = 1u << 18;
    CHECK(plogp_grid_create(&bad, &grid) == PLOGP_EINVAL);
    bad = d;
    bad.n_P = 0;
    CHECK(plogp_grid_create(&bad, &grid) == PLOGP_EINVAL);
    std::vector<uint64_t> big = {1ull << 40};
    std::vector<uint32_t> bigP = {2, 1u << 14};
    plogp_grid_desc rng = {big.data(), 1, bigP.data(), 2, s.data(), s.size(), PLOGP_NO_CAP, 8, PLOGP_MASK_ALL};
    CHECK(plogp_grid_create(&rng, &grid) == PLOGP_ERANGE);
    CHECK(plogp_tune_grid(nullptr, nullptr, nullptr, 0, nullptr) == PLOGP_EINVAL);
    CHECK(plogp_tune_grid_static(nullptr, nullptr, nullptr, 0, nullptr) == PLOGP_EINVAL);
    float ms5[5];
    CHECK(plogp_tune_grid_profile(nullptr, nullptr, nullptr, 0, nullptr, 1, ms5) == PLOGP_EINVAL);
    CHECK(plogp_decision_table_bytes(3, nullptr) == 0);
    if (st_tab == PLOGP_OK && st_grid == PLOGP_OK) {
        CHECK(plogp_grid_ops(grid) == 4);
        CHECK(plogp_decision_table_bytes(1, grid) == 4 * m.size() * P.size() * 16);
        plogp_grid_free(grid);
        plogp_free_table(tab);
    }

    // ---- the launch plan and its scratch layout over many shapes (host arithmetic only)
    long plans = 0, leaner = 0;
    for (int it = 0; it < 20000; ++it) {
        plogp::DeviceTables T = {};
        plogp::DeviceGrid G = {};
        const int nts[] = {1, 1, 2, 5, 64, 100, 10000, 1 << 20};
        const int nsam[] = {2, 21, 64, 512, 1100, 4096};
        T.n_tables = nts[pick(0, 7)];
        T.n = nsam[pick(0, 5)];
        T.shared_x = pick(0, 1);
        G.n_m = pick(0, 3) == 0 ? pick(1, 1 << 24) : pick(1, 5000);
        G.n_mu = pick(1, G.n_m);
        G.n_P = pick(0, 3) == 0 ? pick(1, 1 << 20) : pick(1, 1200);
        G.n_s = pick(0, 4) == 0 ? 0 : (pick(0, 3) == 0 ? pick(1, 1 << 16) : pick(1, 300));
        const int p_top = 1 << (pick(0, 1) ? 24 : 12);
        const unsigned Pmax = (unsigned)pick(G.n_P + 1, p_top > G.n_P + 1 ? p_top : G.n_P + 1);
        G.n_blk = (int)((Pmax - 1) / 64) + 1;
        G.last_terms = (int)((Pmax - 1) - 64u * (unsigned)(G.n_blk - 1));
        G.cl_max = 0;
        while ((1u << G.cl_max) < Pmax) ++G.cl_max;
        const unsigned mask = (unsigned)pick(1, PLOGP_MASK_EVERY);
        G.mask = mask & PLOGP_MASK_ALL;
        G.extra = mask >> 13;
        G.need = (((mask >> 11) | (mask >> 14)) & 1u) << 11 | (((mask >> 12) | (mask >> 15)) & 1u) << 12;
        G.n_ops = ((mask & 0x3FFu) != 0) + ((mask & 0x1C00u) != 0) + ((mask & 0xE000u) != 0) + ((mask & 0x30000u) != 0);
        G.blk_is_prefix = G.n_blk > 32;
        for (int terms_only = 0; terms_only < 2; ++terms_only) {
            plogp::TunePlan plan;
            if (!plogp::plan_tune(T, G, terms_only != 0, plan))
                continue;                                        // too large for one launch: refused, not wrapped
            ++plans;
            const plogp::ScratchLayout &l = plan.lay;
            const size_t offs[] = {l.g1, l.gs, l.gm, l.sum2, l.blk, l.pre, l.part, l.rcp, l.segC, l.segA, l.segB,
                                   l.amin, l.minG, l.nv, l.rec, l.tab, l.batch_ys, l.score_rows};
            for (size_t o : offs)
                CHECK(o < l.total && o % 256 == 0);
            CHECK(plan.path >= 0 && plan.path <= 3);
            // rows beyond the tables: the staged path, a row to a workgroup, or the table-lane kernel when
            // the Gather rows are enabled exactly as the Scatter rows are (or one of the two is absent)
            const unsigned scatter_rows = G.mask & 0x1C00u, gather_rows = (G.extra & 7u) << 10;
            const bool lanes_may = gather_rows == 0 || scatter_rows == 0 || gather_rows == scatter_rows;
            if (terms_only)
                CHECK(plan.path == plogp::TUNE_STAGED);
            else if (G.extra != 0)
                CHECK(plan.path == plogp::TUNE_STAGED || plan.path == plogp::TUNE_ROW ||
                      (plan.path == plogp::TUNE_TABLE_LANES && lanes_may));
            // without room for scratch: the same plan, rows where there are some beyond the tables, or tiles
            // of a big table
            plogp::TunePlan lean;
            CHECK(plogp::plan_tune(T, G, terms_only != 0, lean, 0));
            if (lean.path != plan.path) {
                ++leaner;
                CHECK(plan.path == plogp::TUNE_STAGED && !terms_only && lean.lay.total == 256);
                if (G.extra != 0)
                    CHECK(lean.path == plogp::TUNE_ROW && lean.row_lds <= 64 * 1024);
                else
                    CHECK(lean.path == plogp::TUNE_TILE && T.n > 512 && lean.tile_lds <= 160 * 1024 - 256);
            }
            if (G.extra != 0 && !terms_only && plan.path == plogp::TUNE_STAGED && T.n <= 512 && G.n_blk <= 32 &&
                G.n_s <= 64 && (long)T.n_tables * G.n_m <= 65535 * 16)
                CHECK(lean.path == plogp::TUNE_ROW);
            if (plan.path == plogp::TUNE_STAGED && plan.pairs)
                CHECK(l.segA != 0 && l.segB != 0 && l.amin != 0 && G.n_s > 0);
            if (plan.path == plogp::TUNE_STAGED && plan.lanes_s && !terms_only)
                CHECK(l.minG != 0 && l.nv - l.minG >= (size_t)T.n_tables * ((G.n_s + 63) / 64) * sizeof(double));
        }
    }
    CHECK(leaner > 0);

    // ---- scratch of the cut-over extraction: rows taken whole stay within their limit (or take no more than
    // a counter, its prefix and the flags of each tile of 16 sizes), and a tighter limit never takes more
    for (int it = 0; it < 20000; ++it) {
        plogp::DeviceGrid G = {};
        G.n_m = pick(0, 1) ? pick(1, 40) : pick(1, 513);
        G.n_ops = pick(1, 4);
        G.n_P = pick(0, 1) ? pick(1, 50) : pick(1, 5000);
        const int n_tables = 1 + (int)(next_u64() % (1ull << pick(0, 24)));
        const size_t n_rows = (size_t)n_tables * G.n_ops * G.n_P, per_tile = 12 * plogp::cutover_items(G, n_tables);
        plogp::CutScratch C = {};
        const size_t bytes = plogp::cutover_scratch(G, n_tables, plogp::CUT_SCRATCH_MOST, nullptr, &C);
        const size_t limit = per_tile > plogp::CUT_SCRATCH_MOST ? per_tile : plogp::CUT_SCRATCH_MOST;
        CHECK(bytes <= limit + (limit >> 6));
        CHECK(C.slice_rows >= 1 && C.slice_rows <= n_rows && (C.slice_rows == n_rows || C.slice_rows % 64 == 0));
        // a group's starts fit the scratch and a workgroup's LDS, or, where they are too many, its threads' counts do
        for (int k = 0; k < 8 && G.n_m <= plogp::CUT_ROWS_MAX_M; ++k) {
            const size_t rows = k == 0 ? C.slice_rows : 1 + next_u64() % C.slice_rows;
            const plogp::CutRowsShape c = plogp::cutover_rows_shape(G, rows, C.entries);
            CHECK(c.groups << c.row_bits >= rows && c.groups * c.cap <= C.entries && c.seg * c.parts >= G.n_m);
            CHECK(64 * c.waves == c.parts << c.row_bits && c.waves <= plogp::CUT_ROWS_MAX_WAVES && c.seg % 16 == 0);
            CHECK(14 * c.cap + 4 * 64 * c.waves + 512 <= 160 * 1024 && c.cap <= G.n_m << c.row_bits && c.cap < 65536);
            CHECK(c.cap == G.n_m << c.row_bits || 64 * c.waves * sizeof(uint32_t) <= (size_t)c.cap * 8);
        }
        for (size_t most = bytes / 4, before = bytes;; most = before / 4) {
            const size_t fewer = plogp::cutover_scratch(G, n_tables, most, nullptr, &C);
            CHECK(fewer <= before && C.slice_rows >= 1 && C.slice_rows <= n_rows);
            if (fewer == before) {                    // the shortest slices
                CHECK(G.n_m > plogp::CUT_ROWS_MAX_M || C.slice_rows == n_rows || C.slice_rows == plogp::CUT_SLICE_LEAST);
                break;
            }
            before = fewer;
        }
    }

    // starts per row that are kept (reading a group of rows again more than doubles the call)
    const struct { int n_m; size_t rows; int kept; } keeps[] = {{16, 96000, 16}, {128, 480000, 26}, {256, 480000, 40},
                                                                {256, 96000, 40}, {512, 384000, 77}, {512, 19200, 77},
                                                                {512, 48, 512}, {512, 4096, 512}, {256, 960, 256}};
    for (const auto &k : keeps) {
        plogp::DeviceGrid G = {};
        G.n_m = k.n_m;
        const plogp::CutRowsShape c = plogp::cutover_rows_shape(G, k.rows, SIZE_MAX);
        CHECK(c.cap >> c.row_bits >= k.kept);
    }

    // masks with Gather or Barrier rows: whole rows to a workgroup where that is the faster path
    const struct { unsigned mask; int n_m, n_P, p_max, by_row; } routes[] = {
        {PLOGP_MASK_EVERY, 4000, 5, 6, 1},      {PLOGP_MASK_EVERY, 8000, 5, 6, 0},      {PLOGP_MASK_EVERY, 8000, 100, 1500, 1},
        {PLOGP_MASK_EVERY, 16000, 300, 1500, 1}, {PLOGP_MASK_EVERY, 50000, 600, 2000, 1}, {PLOGP_MASK_GATHER, 2000, 12, 200, 1},
        {PLOGP_MASK_GATHER, 5000, 12, 200, 0},  {PLOGP_MASK_BARRIER, 2000, 5, 6, 1},    {PLOGP_MASK_BARRIER, 5000, 5, 6, 0},
        {PLOGP_MASK_BARRIER, 5000, 100, 1500, 0}, {PLOGP_MASK_BARRIER, 50000, 512, 513, 0},
        {PLOGP_MASK_ALL | PLOGP_MASK_BARRIER, 5000, 36, 1500, 0}, {PLOGP_MASK_BCAST | PLOGP_MASK_GATHER, 5000, 12, 200, 0},
        {PLOGP_MASK_BARRIER, 50000, 1500, 2048, 1}};
    for (const auto &r : routes) {
        plogp::DeviceTables T = {};
        plogp::DeviceGrid G = {};
        T.n_tables = 1;
        T.n = 64;
        G.n_m = G.n_mu = r.n_m;
        G.n_P = r.n_P;
        G.n_s = 15;
        G.n_blk = (r.p_max - 1) / 64 + 1;
        while ((1 << G.cl_max) < r.p_max) ++G.cl_max;
        G.mask = r.mask & PLOGP_MASK_ALL;
        G.extra = r.mask >> 13;
        G.need = (((r.mask >> 11) | (r.mask >> 14)) & 1u) << 11 | (((r.mask >> 12) | (r.mask >> 15)) & 1u) << 12;
        G.n_ops = 4;
        plogp::TunePlan plan;
        CHECK(plogp::plan_tune(T, G, false, plan) && (plan.path == plogp::TUNE_ROW) == (r.by_row != 0));
    }

    // ---- slices of tables of the robustness summary: a launch dimension, at any number of tables
    const int n_robust[] = {1, 2, 9, 2001, 16776960, 16776961, 16776962, 1 << 24};
    for (int n : n_robust)
        for (size_t cells = 1; cells <= ((size_t)1 << 32) - 256; cells = cells * 3 + 5) {
            const int chunk = plogp::robust_chunk(cells, n);
            CHECK(chunk >= 1 && (n - 1 + (long)chunk - 1) / chunk <= 65535);
        }
    std::printf("host sanitizer pass: %ld plans laid out\n", plans);
    return 0;
}
