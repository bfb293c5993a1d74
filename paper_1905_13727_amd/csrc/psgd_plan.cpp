// Host side of the library: plan construction (flat layout, effective ranks,
// tile work-lists, workspace layout, traffic model) and the C ABI entry points.
// No HIP call is made in this file.
#include <algorithm>
#include <cstring>
#include <functional>
#include <new>
#include <queue>

#include "psgd_internal.h"

namespace psgd {

static int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
static int64_t ceil_div(int64_t x, int64_t a) { return (x + a - 1) / a; }

// Split `total` items into `parts` consecutive ranges whose sizes differ by at most one.
static void even_split(int64_t total, int64_t parts, int64_t idx, int64_t* begin, int64_t* count) {
    const int64_t base = total / parts, rem = total % parts;
    *begin = idx * base + std::min(idx, rem);
    *count = base + (idx < rem ? 1 : 0);
}

// Column chunks of a row of `nvec` vectors when one wavefront lane owns at most
// `nv` vectors: chunks are whole multiples of 64 vectors except the last.
static int64_t col_chunks(int64_t nvec, int64_t nv) { return ceil_div(nvec, (int64_t)kWave * nv); }

static void col_chunk_range(int64_t nvec, int64_t nchunk, int64_t c, int32_t* vec0, int32_t* cnt) {
    const int64_t units = ceil_div(nvec, kWave);
    int64_t u0, un;
    even_split(units, nchunk, c, &u0, &un);
    const int64_t v0 = u0 * kWave;
    const int64_t v1 = std::min(nvec, (u0 + un) * kWave);
    *vec0 = (int32_t)v0;
    *cnt = (int32_t)(v1 - v0);
}

// Rows per workgroup tile of the three sweeps when the tuning leaves them to the planner (0), from sweeps on the
// three kinds of sets.  First sweep: a tile of about 8192 elements per column vector a lane owns (16 rows of
// 4-wide vectors, 32 of 2-wide, 64 of scalars).  Second sweep: 128 rows, but 1024 for matrices that are both tall
// and wide (>= 2048 each way), where fewer partial Q pay more than more workgroups.  Third sweep: 16 rows.  A small
// set (under 16 M matrix elements over all workers: each sweep lasts a few tens of microseconds) takes tiles twice
// as tall in the first and third sweep: fewer, longer-lived workgroups.  Not the first sweep of the mean over the workers, which is
// launched once for all of them: us a step, each worker by itself / 32 rows / 16, rank 2 or less: 3 matrices of 2.0 M elements, 4
// workers 50.3 / 53.1 / 48.6; ResNet18-shaped, 2.1 M elements, 4 workers 57.8 / 61.5 / 57.2; 60 matrices of 1.2 M elements, 9 workers
// 69.3 / 73.6 / 64.2 (of 48 such sets at four to twelve workers none lost more than 1 % at 16).
static bool small_set(const psgd_plan* plan) {
    return (int64_t)plan->workers * plan->sizes.n_mat_elems < (int64_t(16) << 20);
}
static int64_t rows_first_sweep(const psgd_plan* plan, const MatDesc& d, int64_t forced, bool mean = false) {
    return forced > 0 ? forced : (small_set(plan) && !mean ? 2 : 1) * (64 / d.vec);
}
static int64_t rows_second_sweep(const MatDesc& d, int64_t forced) {
    return forced > 0 ? forced : (d.n >= 2048 && d.m >= 2048 ? 1024 : 128);
}
static int64_t rows_third_sweep(const psgd_plan* plan, int64_t forced) {
    return forced > 0 ? forced : (small_set(plan) ? 32 : 16);
}

// sweep: 1, 2, 3, or 0 for the first one over the mean (rows per tile by the rules above when rows_forced is 0)
static void streaming_tiles(const psgd_plan* plan, int sweep, int64_t rows_forced, int64_t nv, bool by_col_part,
                            std::vector<Tile>* out, std::vector<int32_t>* n_rblock,
                            std::vector<int32_t>* n_cchunk) {
    out->clear();
    for (size_t i = 0; i < plan->mats.size(); ++i) {
        const MatDesc& d = plan->mats[i];
        const int64_t rows_per_tile = sweep <= 1 ? rows_first_sweep(plan, d, rows_forced, sweep == 0)
                                      : (sweep == 2 ? rows_second_sweep(d, rows_forced) : rows_third_sweep(plan, rows_forced));
        const int64_t nvec = d.m / d.vec;
        const int64_t ncc = col_chunks(nvec, nv);
        const int64_t nrb = ceil_div(d.n, rows_per_tile);
        if (n_rblock) (*n_rblock)[i] = (int32_t)nrb;
        if (n_cchunk) (*n_cchunk)[i] = (int32_t)ncc;
        for (int64_t b = 0; b < nrb; ++b) {
            int64_t r0, rn;
            even_split(d.n, nrb, b, &r0, &rn);
            for (int64_t c = 0; c < ncc; ++c) {
                Tile t{};
                t.mat = (int32_t)i;
                t.row0 = (int32_t)r0;
                t.nrows = (int32_t)rn;
                col_chunk_range(nvec, ncc, c, &t.vec0, &t.nvec);
                t.part = (int32_t)(by_col_part ? c : b);
                out->push_back(t);
            }
        }
    }
}

// Workgroups are handed to the 8 accelerator dies (XCDs, one L2 each) round robin by their linear index.  With
// the tile list permuted so that entry b is the (b / 8)-th tile of the b % 8-th contiguous eighth of the list,
// each die works through one contiguous range of tiles: neighbouring tiles (column chunks of the same rows, the
// next row block) share cache lines at their edges when rows are not multiples of the line size, and those lines
// then stay within one L2 instead of being fetched and partially written back by two.
static void order_for_xcds(std::vector<Tile>& tiles) {
    constexpr size_t X = 8;
    const size_t nb = tiles.size();
    if (nb < 2 * X) return;
    const size_t per = nb / X, rem = nb % X;
    std::vector<Tile> out(nb);
    for (size_t b = 0; b < nb; ++b) {
        const size_t x = b % X, k = b / X;
        out[b] = tiles[x * per + std::min(x, rem) + k];
    }
    tiles.swap(out);
}

// The same within groups of consecutive matrices: a group is closed once it holds `min_tiles` tiles, so that a large
// matrix is spread over all dies by itself (the dies then work on the same matrix at the same time) while small
// ones are ordered together.  Slices of the vector region (mat < 0) are left where they are.
static void order_for_xcds_grouped(std::vector<Tile>& tiles, size_t min_tiles) {
    size_t b = 0;
    while (b < tiles.size()) {
        if (tiles[b].mat < 0) { ++b; continue; }
        size_t e = b;
        while (e < tiles.size() && tiles[e].mat >= 0) {
            // extend by one whole matrix
            const int32_t m = tiles[e].mat;
            while (e < tiles.size() && tiles[e].mat == m) ++e;
            if (e - b >= min_tiles) break;
        }
        std::vector<Tile> run(tiles.begin() + b, tiles.begin() + e);
        order_for_xcds(run);
        std::copy(run.begin(), run.end(), tiles.begin() + b);
        b = e;
    }
}

// xcd_order: 0 leaves a list as built, 1 orders it as a whole, k >= 2 in groups of at least k tiles.
static void order_tiles(std::vector<Tile>& tiles, int64_t xcd_order) {
    if (xcd_order >= 2) order_for_xcds_grouped(tiles, (size_t)xcd_order);
    else if (xcd_order == 1) order_for_xcds(tiles);
}

// The planner's own group size (xcd_order = -1): about 4096 workgroups per group, counting the W workers that
// every tile is launched for; between 128 and 2048 tiles.  Measured on the ResNet18-shaped set: at W = 16 groups of
// 64...256 tiles are 3-4 % faster than groups of 2048 (the sweeps' first and third kernel), at W = 4 and W = 1 the
// size makes no difference; LSTM-shaped set at W = 4: 1.5 %.
static int64_t group_tiles(const psgd_plan* plan) {
    return std::min<int64_t>(2048, std::max<int64_t>(128, 4096 / plan->workers));
}


static void build_one_wide(psgd_plan* plan);

// Matrix-core path: its own tilings and workspace layout.
static psgd_status build_hr_tables(psgd_plan* plan) {
    const Tuning& tu = plan->tuning;
    if (tu.hr_k3_rows < 64 || tu.hr_k1_rows < 64 || tu.hr_k1_rows > 256 || tu.hr_k1_rows % 64 != 0 ||
        tu.hr_k1_cols < 64 || tu.hr_k1_cols % 64 != 0 || (tu.hr_k4_rows != 0 && (tu.hr_k4_rows < 16 || tu.hr_k4_rows > 1024)) ||
        tu.stream_hints < -1 || tu.stream_hints > 1 || tu.xcd_order < -1 || tu.gram_fused < -1 || tu.gram_fused > 2 || tu.gram_spin < 1 ||
        tu.gram_spin > (1 << 24))
        return PSGD_EINVAL;
    for (const MatDesc& d : plan->mats)   // 16-byte accesses along the rows, 31-bit byte offsets within a tile
        if (d.m % 4 != 0 || d.m > kHrMaxCols || d.n > kHrMaxRows) return PSGD_EUNSUPPORTED;
    const int64_t W = plan->workers;
    const size_t nm = plan->mats.size();
    plan->tiles1.clear(); plan->tiles3.clear(); plan->tiles4.clear(); plan->tiles4u.clear(); plan->tilesp.clear();
    plan->tiles1m.clear(); plan->mats_mean.clear();
    plan->small_mats.clear(); plan->tiles_gram.clear(); plan->tilesq.clear();
    plan->hr_tiles1.clear(); plan->hr_tiles3.clear(); plan->hr_tiles4.clear();
    plan->p_pre_reduce = plan->p_pre_reduce_mean = false;
    plan->mean_first = plan->update_around = false;   // the streaming kernels' choices, should a tuning key have moved the plan here
    const int64_t right_rows = tu.hr_k1_rows;
    // rows per workgroup of the decompression: measured best on the 24-layer transformer set at ranks 16, 32, 64
    // (one, two, four rank tiles of 16)
    // measured on the 24-layer transformer-shaped set (k_hr_decomp, ms): rank 16: 2.16 at 64 rows, 2.22 at 128, 2.25 at
    // 256; rank 32: 2.54 at 64, 2.28 at 128...256, 2.36 at 512; rank 64: 3.04 at 128, 2.62 at 256, 2.48 at 512
    const int64_t decomp_rows = tu.hr_k4_rows ? tu.hr_k4_rows : (plan->rank <= 16 ? 64 : (plan->rank <= 32 ? 256 : 512));
    int64_t pp = 0, qp = 0, gp = 0, cp = 0;
    for (size_t i = 0; i < nm; ++i) {
        MatDesc& d = plan->mats[i];
        d.n_cchunk = (int32_t)ceil_div(d.m, tu.hr_k1_cols);
        const int64_t nrb = ceil_div(d.n, tu.hr_k3_rows);
        d.n_rblock = (int32_t)nrb;   // one partial Q per row block (the workgroup adds its four strips itself)
        // Gram blocks: 128 rows each, more for very tall panels so that the one workgroup that adds up a matrix's
        // blocks has at most 64 of them
        const int64_t gram_rows = kHrGramTileRows * ceil_div(d.n, (int64_t)kHrGramTileRows * 64);
        d.n_gblock = (int32_t)ceil_div(d.n, gram_rows);
        d.ppart_off = pp;
        pp += round_up(W * d.n_cchunk * d.n * d.r, kAlignElems);
        d.gram_off = gp;
        gp += round_up((int64_t)d.n_gblock * d.r * d.r, 32);
        d.chol_off = cp;
        cp += round_up((int64_t)d.r * d.r + d.r, 32);
        for (int64_t r0 = 0; r0 < d.n; r0 += right_rows)
            for (int64_t cc = 0; cc < d.n_cchunk; ++cc) {
                Tile t{};
                t.mat = (int32_t)i; t.row0 = (int32_t)r0; t.nrows = (int32_t)std::min<int64_t>(right_rows, d.n - r0);
                t.vec0 = (int32_t)(cc * tu.hr_k1_cols);
                t.nvec = (int32_t)std::min<int64_t>(tu.hr_k1_cols, d.m - t.vec0);
                t.part = (int32_t)cc;
                plan->hr_tiles1.push_back(t);
            }
        for (int64_t b = 0; b < nrb; ++b)
            for (int64_t c0 = 0; c0 < d.m; c0 += 128) {
                Tile t{};
                t.mat = (int32_t)i; t.row0 = (int32_t)(b * tu.hr_k3_rows);
                t.nrows = (int32_t)std::min<int64_t>(tu.hr_k3_rows, d.n - t.row0);
                t.vec0 = (int32_t)c0; t.nvec = (int32_t)std::min<int64_t>(128, d.m - c0);
                t.part = (int32_t)b;
                plan->hr_tiles3.push_back(t);
            }
        for (int64_t r0 = 0; r0 < d.n; r0 += decomp_rows)
            for (int64_t c0 = 0; c0 < d.m; c0 += 128) {
                Tile t{};
                t.mat = (int32_t)i; t.row0 = (int32_t)r0; t.nrows = (int32_t)std::min<int64_t>(decomp_rows, d.n - r0);
                t.vec0 = (int32_t)c0; t.nvec = (int32_t)std::min<int64_t>(128, d.m - c0);
                plan->hr_tiles4.push_back(t);
            }
        for (int32_t b = 0; b < d.n_gblock; ++b) {
            Tile t{};
            t.mat = (int32_t)i; t.row0 = (int32_t)(b * gram_rows); t.nrows = (int32_t)std::min<int64_t>(gram_rows, d.n - t.row0);
            t.part = b;
            plan->tiles_gram.push_back(t);
        }
    }
    for (size_t i = 0; i < nm; ++i) {
        MatDesc& d = plan->mats[i];
        d.qpart_off = pp + qp;
        qp += round_up(W * d.n_rblock * d.m * d.r, kAlignElems);
        // a matrix with a single partial Q (one worker, one row block) has it written straight into Q
        const int64_t total = W * d.n_rblock > 1 ? (int64_t)d.m * d.r : 0;
        for (int64_t e = 0; e < total; e += kWave) {
            Tile t{};
            t.mat = (int32_t)i; t.elem0 = e; t.nelem = std::min<int64_t>(kWave, total - e);
            plan->tilesq.push_back(t);
        }
    }
    plan->ws_ppart_floats = pp;
    plan->ws_qpart_floats = qp;
    plan->ws_gram_doubles = gp;
    plan->ws_chol_doubles = cp;
    plan->sizes.workspace_bytes =
        std::max<int64_t>(256, round_up((pp + qp) * (int64_t)sizeof(float), 256) + (gp + cp) * (int64_t)sizeof(double));
    plan->stream_hints = tu.stream_hints < 0 ? W * plan->sizes.n_mat_elems * (int64_t)sizeof(float) > kStreamHintBytes
                                             : tu.stream_hints != 0;
    plan->resident_ok = false;
    plan->res_tiles.clear(); plan->res_mats.clear();
    plan->res_ws_floats = 0; plan->res_blocks = 0; plan->res_mail_slots = 0; plan->res_sync_words = 0;
    // Whole-list order for P = M Q and the decompression was 3 % faster than groups in one process with the buffers
    // held fixed, and no faster with the benchmark's own allocations: groups, as on the streaming path.
    const int64_t order = tu.xcd_order < 0 ? group_tiles(plan) : tu.xcd_order;
    order_tiles(plan->hr_tiles1, order);
    order_tiles(plan->hr_tiles3, order);
    order_tiles(plan->hr_tiles4, order);
    build_one_wide(plan);
    plan->tables_built = true;
    return PSGD_OK;
}

// One walk over M (k_one_sweep): what a row costs its workgroup, in elements: halfway between its own and those that the lanes
// of its wavefronts could take (a row of 139 elements keeps a wavefront for 512 waiting almost as long as a full one does).  With
// blocks of equal elements instead, sets of many matrices lost up to 16 % to the other route that now gain (60 matrices of 15 M
// elements, rank 4: 100 us by the other route, 115 with equal elements, 87 with equal costs).
static int64_t one_row_cost(const OneMat& o, bool mean) {
    return (o.m + ((int64_t)kWave << o.waves_log2) * one_nv(o.vec, mean) * o.vec) / 2;
}

// Row blocks per matrix, `deals` for each of the `slots` workgroups that the device holds at once.  With one deal there are no more of
// them than slots (a second generation of workgroups adds its first loads and last sums, 6 us, and where the elements divide evenly
// was never faster), and within that as little in the largest as can be.  With several, the hardware deals them out, largest first.
//
// A group of wavefronts walks two steps at least: every block leaves a partial S behind.  One where that makes so few blocks that much
// of the chip is idle (below half of the slots on sets under 2^19 elements from eight workers on, whose steps are long, below a quarter
// with one worker at ranks whose ring holds one step).  Whole steps, us, two steps / one: 32 workers, rank 2, five matrices of 0.2 M elements 128 / 89, 20 of 0.4 M 167 / 124; 8 workers, the same
// 40 / 30 and 52 / 43, but ResNet18-shaped of 0.9 M, 8 / 16 workers 53.5 / 57.7 and 92 / 104; one worker, rank 4, 900 x 640 (57) 24.2 / 22.5, but 12 of 300 x 400 (228) 25.2 / 27.5,
// 8 of 512 x 320 24.4 / 27.4, 900 x 2048 32.1 / 36.4.
static void one_sweep_blocks(const psgd_plan* plan, int waves, int64_t slots, int deals, std::vector<int64_t>* blocks) {
    const bool mean = plan->workers > 1;
    const bool many = plan->workers >= kOneStepWorkers && plan->sizes.n_mat_elems < kOneStepElems;
    const int64_t few = many ? slots / 2 : (one_depth(plan->rank, mean) == 1 ? slots / 4 : 0);
    int64_t steps = 2, at_two = 0;
    for (const OneMat& o : plan->one_mats) at_two += ceil_div(o.n, (waves >> o.waves_log2) * kOneRows * 2);
    if (at_two < few) steps = 1;
    int64_t total = 0;
    for (const OneMat& o : plan->one_mats) total += o.n * one_row_cost(o, mean);
    auto blocks_of = [&](const OneMat& o, int64_t cost) {
        const int64_t groups = waves >> o.waves_log2;
        const int64_t most = ceil_div(o.n, groups * kOneRows * steps);
        return std::min(most, ceil_div(o.n * one_row_cost(o, mean), cost));
    };
    int64_t cost = std::max<int64_t>(1, ceil_div(total, slots * deals));
    while (deals == 1) {
        int64_t tiles = 0;
        for (const OneMat& o : plan->one_mats) tiles += blocks_of(o, cost);
        if (tiles <= slots || cost >= total) break;
        cost += ceil_div(cost, 64);
    }
    blocks->clear();
    for (const OneMat& o : plan->one_mats) blocks->push_back(blocks_of(o, cost));
}

// When the last block is done, in elements: every workgroup takes the next one of the list, largest first, as it ends one, and pays
// `extra` for the new one's first loads and the old one's last sums.
static double one_sweep_span(const psgd_plan* plan, int64_t slots, const std::vector<int64_t>& blocks, double extra) {
    const bool mean = plan->workers > 1;
    std::vector<double> costs;
    for (size_t i = 0; i < blocks.size(); ++i) {
        const OneMat& o = plan->one_mats[i];
        costs.insert(costs.end(), (size_t)blocks[i], (double)(ceil_div(o.n, blocks[i]) * one_row_cost(o, mean)));
    }
    std::sort(costs.begin(), costs.end(), std::greater<double>());
    std::priority_queue<double, std::vector<double>, std::greater<double>> ends;
    double last = 0;
    for (size_t i = 0; i < costs.size(); ++i) {
        double at = 0;
        if ((int64_t)i >= slots) {
            at = ends.top() + extra;
            ends.pop();
        }
        ends.push(at + costs[i]);
        last = std::max(last, at + costs[i]);
    }
    return last;
}

static void push_solve_tiles(psgd_plan* plan, int32_t mat, const OneMat& o) {
    // columns of Q per workgroup: fewer, with more threads to a column, where there are many blocks to add
    const int cl = o.n_blocks >= 16 ? 4 : (o.n_blocks >= 4 ? 6 : 8);
    for (int64_t c = 0; c < o.m; c += 1 << cl)
        plan->solve_tiles.push_back({mat, (int32_t)c, (int32_t)std::min<int64_t>(1 << cl, o.m - c), 0, (int16_t)cl});
    for (int64_t c = 0; c < o.n; c += kBlock)
        plan->solve_tiles.push_back({mat, (int32_t)c, (int32_t)std::min<int64_t>(kBlock, o.n - c), 1, 8});
}

// Whether the one walk is also the faster one (the planner's own choice; `partial`: bytes of the partial S).  Us, two walks / one:
//  - one worker, rows of 4 or 2 columns a lane that leave two thirds of the lanes idle: M is then read again from the caches faster than
//    the idle lanes' instructions pass.  Rows of even lengths at every size: 20 of 500 x 250, rank 2 25.3 / 30.8; 20 of 2000 x 66 33.8 / 40.2; LSTM-shaped, rows
//    of 130, 4.3 M elements 45 / 54; of 250, 4 M 34.3 / 37.4 (9 M 60.3 / 60.6; rows of 301, 5.2 M 46.4 / 40.6).  Multiples of 4 up to 4 M elements from rank 2 on: LSTM-shaped, rows of 100,
//    1.2 M, rank 2 / 4 27.8 / 29.7 and 30.8 / 34.1; of 200, 3 M 31.4 / 32.9 and 34.2 / 37.1 (9 M 59.4 / 56.2 and 63.7 / 62.9).
//  - partial S that weigh as much as what the second walk would read: one worker, rank 2, 6 of 256 x 2304 (3.5 M elements, 7 MB) 30.5 / 32.3, 20 of 128 x
//    1152 28.1 / 31.1, 10 of 20 x 6144 22.1 / 28.7; rank 4, 10 of 100 x 3000 31.8 / 36.0, 900 x 2048 29.0 / 32.1, ResNet18-shaped, 1.8, 2.8 and 6.3 M 29.2 / 31.9, 32.7 / 35.1 and 44.5 / 46.4.
//    Two workers, rank 4, 10 of 100 x 3000 (3 M elements, 24 MB) 41.0 / 45.5, 900 x 4095 50.6 / 57.0; but ResNet18-shaped, 2.8 M, 14 MB 46.0 / 42.5, 900 x 3000, 22 MB 44.6 / 42.8.
//  - sets that otherwise take the mean first, beyond the memory-side cache: storing and reading the mean is 8 of 12 W + 8 bytes an element, so what the one walk saves
//    is little with many workers, and rows of eight wavefronts, which wait for each other at every step, cost more.  Rank 2, ResNet18-shaped,
//    8.5 M elements, 16 / 32 workers 512 / 525 and 1003 / 1051, 2.8 M, 32 workers 413 / 472; 40 of 256 x 1024, 16 / 32 579 / 593 and 1141 / 1189; 6 of 2000 x 4096, 4 / 16
//    719 / 753 and 2584 / 2878, 110 of 100 x 4096, 8 workers 1289 / 1344; up to eight workers other rows 289 / 283 (ResNet18-shaped, 8), 320 / 311 (256 x 1024, 8).  Rows that do
//    not fill the mean's chunks of 256 columns gain at any number: of 648, 16 workers 2137 / 2045, of 300, 16 / 32 441 / 396 and
//    846 / 756, of 2052, 16 1092 / 1006.
//  - small sets of more than sixteen workers with most elements in rows that are not multiples of 4: a group's walk over all workers is a chain of
//    narrow accesses.  32 workers, rank 2, five matrices of 0.2 M elements 67 / 89, 20 of 0.4 M 114 / 124, 40 of 1 M 289 / 314 (16 workers 47 / 50, 69.9 / 68.9 and
//    139 / 147); but 24 of 9 M 1559 / 1442, and in rows of multiples of 4, 1.1 and 1.3 M, 288 / 266 and 175 / 150.
static bool one_sweep_pays(const psgd_plan* plan, int64_t partial) {
    const int64_t W = plan->workers, N = plan->sizes.n_mat_elems;
    const int R = plan->rank;
    const bool mean = W > 1;
    int64_t thin2 = 0, thin4 = 0, eight = 0, filled = 0, narrow = 0;
    for (const OneMat& o : plan->one_mats) {
        const int64_t chunks = ceil_div(o.m, kWave * o.vec);   // of the mean's walk: one column vector a lane
        if ((int64_t)o.m * 16 >= chunks * kWave * o.vec * 15) filled += (int64_t)o.n * o.m;
        if ((1 << o.waves_log2) == kOneMaxWaves) eight += (int64_t)o.n * o.m;
        if (o.vec != 4) narrow += (int64_t)o.n * o.m;
        if (o.vec == 1 || (int64_t)o.m * 3 > (int64_t)kWave * one_nv(o.vec, mean) * o.vec) continue;
        (o.vec == 2 ? thin2 : thin4) += (int64_t)o.n * o.m;
    }
    if (W == 1 && N >= kOneThinElems && (thin2 > N / 2 || (R >= 2 && N < kOneThin4Elems && thin2 + thin4 > N / 2))) return false;
    if (W > 16 && N < kMeanElemsPerWorker * W && narrow > N / 2) return false;
    if (plan->mean_first && W * N * (int64_t)sizeof(float) > kStreamHintBytes && filled > N / 2 && (W > kOneMeanWorkers || eight > N / 2)) return false;
    if (partial <= kOnePartialBytes) return true;
    if (W == 1) return (double)partial <= 1.9 * N || N >= (R <= 2 ? kOnePartialElems : kOnePartialElems4);
    return partial <= 3 * W * N;
}

// Whether a plan's sets go through one walk over M per iteration instead of two (see k_one_sweep), and its tables.  Ranks up to
// kOneMaxRank, every row short enough for the registers of one workgroup, partial sums of at most kOneMaxBytes.  Whole steps, us, two
// walks / one: LSTM-shaped set, rank 4, 1 / 2 / 4 workers 171 / 337 / 718 and 157 / 287 / 632; rank 1, 2, 3 167, 169, 171 and 149, 154, 153;
// two transformer layers (42 M elements), rank 2, bf16, 1 / 2 workers 183 / 365 and 168 / 305; 24 matrices of 9 M, 3 workers, two
// iterations 209 / 172; 3 to 80 matrices of 0.04 to 24 M elements in rows of any length, 1 and 3 workers: 1.00 to 1.33 and 1.09 to 1.41
// times as fast; ResNet18-shaped, 0.7 to 2.8 M, 2 and 4 workers 1.07 to 1.24 times.  Beyond rank 4 the registers hold less of a row: at rank
// 6 and 8 it gained 3 % on the LSTM-shaped set and nothing elsewhere.
static void build_one_sweep(psgd_plan* plan) {
    plan->one_sweep = false;
    plan->one_mats.clear(); plan->one_tiles.clear(); plan->solve_tiles.clear();
    const Tuning& tu = plan->tuning;
    const int R = plan->rank;
    const int64_t W = plan->workers;
    const bool mean = W > 1;
    // keys that ask for a particular kernel of the two walks, or for its tiles, get it
    const bool two = tu.k1_rows || tu.k1_nv != 2 || tu.k3_rows || tu.k3_nv != 1 || tu.ortho_rows || tu.gram_fused >= 0 || tu.worker_mean >= 0;
    if (!tu.one_sweep || (tu.one_sweep < 0 && two) || R > kOneMaxRank || plan->mats.empty()) return;
    int max_log2 = 0;
    for (const MatDesc& d : plan->mats) {
        const int64_t lanes = ceil_div(d.m / d.vec, one_nv(d.vec, mean));
        int l2 = 0;
        while ((1 << l2) <= kOneMaxWaves && ((int64_t)kWave << l2) < lanes) ++l2;
        if ((1 << l2) > kOneMaxWaves || (int64_t)d.n * d.r * 4 >= (int64_t(1) << 31)) {
            plan->one_mats.clear();
            return;
        }
        max_log2 = std::max(max_log2, l2);
        OneMat o{};
        o.off = d.off; o.p_off = d.p_off; o.q_off = d.q_off;
        o.n = d.n; o.m = d.m; o.r = d.r; o.vec = d.vec; o.waves_log2 = l2;
        plan->one_mats.push_back(o);
    }
    // Two workgroups of four wavefronts on a compute unit, or one of eight, which writes half the partial S (LSTM-shaped set, rank 4, 1 / 2
    // workers 159 / 302 and 157 / 287 us) but divides the matrices more coarsely (80 matrices of 24 M elements 128 / 133); and one, two
    // or four blocks for each: the cheapest by the time to the last block, of the partial S written and read, and of the longest sum
    // over blocks.  More than one where the matrices are so many that a block for each of the workgroups divides the large ones too
    // coarsely: whole steps, two walks / one block / several, rank 2: 600 of 64 x 9 and one of 1000 x 2560 61 / 576 / 57 us (3 workers 129 / 1849 /
    // 97), 400 of 32 x 9 and 20 of 512 x 2304 132 / 137 / 124, 600 of 64 ... 1024 rows and columns 497 / 605 / 434, 300 of 1000 x 1000 1555 / 1593 / 1439,
    // 1000 of 100 x 100 90 / 96 / 79.
    const double bytes = (double)W * ((plan->grad_dtype == PSGD_BF16 ? 2 : 4) + 8);
    double best = 0;
    std::vector<int64_t> blocks, trial;
    for (int waves : {4, 8}) {
        if ((1 << max_log2) > waves) continue;
        const int64_t slots = (int64_t)kResCUs * (kOneMaxWaves / waves);
        const double per_us = 6e6 / (slots * bytes);   // elements that a workgroup walks in a microsecond while all of them do
        for (int deals : {1, 2, 4}) {
            one_sweep_blocks(plan, waves, slots, deals, &trial);
            double partial = 0;
            int64_t longest = 0;
            for (size_t i = 0; i < trial.size(); ++i) {
                partial += 16.0 * trial[i] * plan->one_mats[i].m * plan->one_mats[i].r;
                longest = std::max(longest, trial[i]);
            }
            const double us = one_sweep_span(plan, slots, trial, 6.0 * per_us) / per_us + partial / 6e6 + 0.025 * longest + (waves == 8 ? 2.0 : 0.0);
            if (deals > 1 && partial / 2 > 0.99 * kOneMaxBytes) break;   // with the Gram matrices, more than the plan may hold
            if (blocks.empty() || us < best) {
                best = us;
                blocks = trial;
                plan->one_waves = waves;
            }
        }
    }
    const int64_t NG = R * (R + 1) / 2;
    int64_t sd = 0, gd = 0, lds = 0;
    for (size_t i = 0; i < plan->one_mats.size(); ++i) {
        OneMat& o = plan->one_mats[i];
        o.n_blocks = (int32_t)blocks[i];
        o.s_off = sd;
        sd += (int64_t)o.n_blocks * o.m * o.r;
        o.g_off = gd;
        gd += (int64_t)o.n_blocks * NG;
        lds = std::max<int64_t>(lds, ((int64_t)kWave << o.waves_log2) * one_q_floats(R, o.vec, mean) * (int64_t)sizeof(float));
        lds = std::max<int64_t>(lds, (int64_t)one_deposit(R, o.vec, mean) * o.vec * R * (plan->one_waves * kWave + 1) * (int64_t)sizeof(double));
        for (int64_t b = 0; b < o.n_blocks; ++b) {
            int64_t r0, rn;
            even_split(o.n, o.n_blocks, b, &r0, &rn);
            plan->one_tiles.push_back({(int32_t)i, (int32_t)r0, (int32_t)rn, (int32_t)b});
        }
        push_solve_tiles(plan, (int32_t)i, o);
    }
    if ((int64_t)plan->one_tiles.size() > (int64_t)kResCUs * (kOneMaxWaves / plan->one_waves))   // dealt out: what is left for the end is small
        std::stable_sort(plan->one_tiles.begin(), plan->one_tiles.end(), [&](const OneTile& a, const OneTile& b) {
            return a.nrows * one_row_cost(plan->one_mats[a.mat], mean) > b.nrows * one_row_cost(plan->one_mats[b.mat], mean);
        });
    plan->one_s_doubles = round_up(sd, 32);
    plan->one_lds_bytes = (int32_t)lds;
    plan->one_bytes = (plan->one_s_doubles + gd) * (int64_t)sizeof(double);
    plan->one_sweep = plan->one_bytes <= kOneMaxBytes && (tu.one_sweep > 0 || one_sweep_pays(plan, sd * (int64_t)sizeof(double)));
}

// psgd_step on a matrix-core plan in one walk over M that stores nothing but P (k_one_sweep_wide): one worker, bf16 gradients, rank 4, a
// set beyond the memory-side cache, rows of at most 8192 elements.  The partial S lie in `out`, each matrix's within its own region,
// which the decompression writes afterwards; the partial Gram matrices in the workspace.  24-layer transformer-shaped set, us a step:
// 5234 on the matrix cores, 4227 this way (k_one_sweep_wide 1559, k_hr_decomp with g added again 2677, where k_hr_right, k_hr_left and
// k_hr_decomp took 2166, 796 and 2154).  Other sets, before / after: transformers of 77, 91, 127, 138, 203, 216 and 304 M elements 357 / 309,
// 465 / 398, 706 / 506, 924 / 678, 1083 / 771, 1104 / 894 and 1367 / 1121; 200 matrices of 500 x 1000 678 / 465; 300000 x 300 772 / 563; 21000 x 4096
// 448 / 382.  Rows that take all eight wavefronts, which then wait for each other at every row, lose where they are all there is (6
// of 2000 x 8192 470 / 532, 110 of 100 x 8192 417 / 511) and are a third of the transformers': the line is at half of the elements.
// Rows that leave three quarters of a wavefront's 1024 columns empty lose too where they are most (1000000 x 100 897 / 980, 3000000 x 32 2021 /
// 2578, 2200 of 200 x 200 637 / 703, 600000 x 160 753 / 754; 400000 x 256 625 / 549, 1000 of 300 x 300 672 / 558).
// Above rank 4 a row of 8192 and its S do not fit a compute unit's registers.
static void build_one_wide(psgd_plan* plan) {
    plan->one_wide = false;
    plan->one_mats.clear(); plan->one_tiles.clear(); plan->solve_tiles.clear();
    const Tuning& tu = plan->tuning;
    const Tuning def;
    const int R = plan->rank;
    // keys that ask for the matrix-core kernels or for their tiles get them
    const bool others = tu.bf16_valu >= 0 || tu.hr_k1_rows != def.hr_k1_rows || tu.hr_k1_cols != def.hr_k1_cols || tu.hr_k3_rows != def.hr_k3_rows;
    if (R != kOneMaxRank || plan->workers != 1 || plan->grad_dtype != PSGD_BF16 || plan->mats.empty() || !tu.one_sweep ||
        !tu.stream_hints || (tu.one_sweep < 0 && (others || !plan->stream_hints)))   // its accesses are non-temporal
        return;
    const int64_t osz = plan->out_dtype == PSGD_BF16 ? 2 : 4;
    int64_t total = 0, eight = 0, thin = 0;
    for (const MatDesc& d : plan->mats) {
        if (d.m > (int64_t)kOneMaxWaves * kWave * kOneWideNV * 4 || (int64_t)d.n * osz < (int64_t)d.r * (int64_t)sizeof(double)) return;
        total += (int64_t)d.n * d.m;
        if (d.m > (int64_t)kOneMaxWaves / 2 * kWave * kOneWideNV * 4) eight += (int64_t)d.n * d.m;
        if (d.m < kWave * kOneWideNV) thin += (int64_t)d.n * d.m;
    }
    if ((eight > total / 2 || thin > total / 2) && tu.one_sweep < 0) return;
    // Four blocks for every compute unit, dealt largest first: what one block too many costs in the last generation is a quarter of a
    // compute unit's share, and the partial S (70 MB of the 24-layer set's 26 GB) are little.
    const int64_t elems = ceil_div(total, (int64_t)kResCUs * 4);
    int64_t gd = 0;
    for (size_t i = 0; i < plan->mats.size(); ++i) {
        const MatDesc& d = plan->mats[i];
        OneMat o{};
        o.off = d.off; o.p_off = d.p_off; o.q_off = d.q_off;
        o.n = d.n; o.m = d.m; o.r = d.r; o.vec = 4;
        while (((int64_t)kWave << o.waves_log2) * kOneWideNV * 4 < d.m) ++o.waves_log2;
        const int64_t groups = kOneMaxWaves >> o.waves_log2;
        const int64_t want = std::max<int64_t>(1, ((int64_t)o.n * o.m + elems / 2) / elems);
        const int64_t room = (int64_t)d.n * osz / ((int64_t)d.r * (int64_t)sizeof(double));   // blocks whose S the matrix's part of `out` holds
        o.n_blocks = (int32_t)std::min(std::min(ceil_div(o.n, groups * kOneWideDepth), want), room);
        o.s_off = d.off * osz / (int64_t)sizeof(double);   // d.off is a multiple of 64 elements
        o.g_off = gd;
        gd += (int64_t)o.n_blocks * (R * (R + 1) / 2);
        for (int64_t b = 0; b < o.n_blocks; ++b) {
            int64_t r0, rn;
            even_split(o.n, o.n_blocks, b, &r0, &rn);
            plan->one_tiles.push_back({(int32_t)i, (int32_t)r0, (int32_t)rn, (int32_t)b});
        }
        push_solve_tiles(plan, (int32_t)i, o);
        plan->one_mats.push_back(o);
    }
    std::stable_sort(plan->one_tiles.begin(), plan->one_tiles.end(), [&](const OneTile& a, const OneTile& b) {
        return (int64_t)a.nrows * plan->one_mats[a.mat].m > (int64_t)b.nrows * plan->one_mats[b.mat].m;
    });
    plan->one_waves = kOneMaxWaves;
    plan->one_lds_bytes = kOneWideLds;
    plan->one_wide = gd * (int64_t)sizeof(double) <= plan->sizes.workspace_bytes;
}

// Whether a call's buffers let it: `out` is scratch for fp64 values before it is written, and g is read after that.
static bool one_wide_call(const psgd_plan* plan, const void* grad, const void* out) {
    if (!plan->one_wide || reinterpret_cast<uintptr_t>(out) % 16) return false;
    const char *g = static_cast<const char*>(grad), *o = static_cast<const char*>(out);
    const int64_t gb = plan->sizes.grad_stride * 2, ob = plan->sizes.out_elems * (plan->out_dtype == PSGD_BF16 ? 2 : 4);
    return g + gb <= o || o + ob <= g;
}

psgd_status build_tables(psgd_plan* plan) {
    const Tuning& tu = plan->tuning;
    // Ranks above 8 run on the matrix-core kernels; bf16 data at the lower ranks on either (bf16_valu).  The planner's
    // own choice for bf16 data: matrix cores at rank >= 4 on a set beyond the memory-side cache, if its shapes are ones
    // those kernels take (24-layer transformer-shaped set, ms per step, streaming / matrix cores: rank 2: 5.17 / 5.15,
    // rank 4: 5.28 / 5.17, rank 8: 6.43 / 5.19).
    const bool bf16 = plan->grad_dtype != PSGD_F32 || plan->out_dtype != PSGD_F32;
    if (tu.bf16_valu < -1 || tu.bf16_valu > 1 || tu.worker_mean < -1 || tu.worker_mean > 1 || tu.one_sweep < -1 || tu.one_sweep > 1)
        return PSGD_EINVAL;
    bool hr_low = bf16 && tu.bf16_valu == 0;
    if (bf16 && tu.bf16_valu < 0 && plan->rank >= 4 &&
        plan->workers * plan->sizes.n_mat_elems * (int64_t)sizeof(float) > kStreamHintBytes) {
        hr_low = true;
        for (const MatDesc& d : plan->mats)
            if (d.m % 4 != 0 || d.m > kHrMaxCols || d.n > kHrMaxRows) hr_low = false;
    }
    plan->hr = plan->rank > kValuMaxRank || hr_low;
    plan->one_sweep = plan->one_wide = plan->iter_mean = false;
    if (plan->hr) return build_hr_tables(plan);
    if (plan->out_dtype != PSGD_F32 && tu.k4_nv != 1) return PSGD_EINVAL;   // bf16 output: one column vector per lane
    if (tu.k1_rows < 0 || tu.k3_rows < 0 || tu.k4_rows < 0 || tu.k1_nv < 1 ||
        tu.k1_nv > kMaxVecPerLaneK1 || tu.k3_nv < 1 || tu.k3_nv > kMaxVecPerLaneK3 || tu.k4_nv < 1 ||
        tu.k4_nv > kMaxVecPerLaneK3 || tu.res_rows < 0 || tu.res_rows > kResRows || tu.resident < 0 || tu.resident > 2 ||
        tu.res_spin < 1 || tu.res_spin > (int64_t(1) << 30) || tu.res_max_blocks < 0 || tu.res_max_blocks > 65535 ||
        tu.stream_hints < -1 || tu.stream_hints > 1 || tu.xcd_order < -1 || tu.gram_fused < -1 || tu.gram_fused > 2 || tu.gram_spin < 1 ||
        tu.gram_spin > (1 << 24) || tu.ortho_rows < 0 || tu.ortho_rows > kOrthoMaxRows)
        return PSGD_EINVAL;
    const size_t nm = plan->mats.size();
    // k_ef_right and k_left address the rows of a wavefront's strip (a quarter of the tile's rows) with 31-bit
    // byte offsets
    for (const MatDesc& d : plan->mats)
        if (ceil_div(std::max(rows_first_sweep(plan, d, tu.k1_rows), rows_second_sweep(d, tu.k3_rows)), kWavesPerBlock) * d.m * 4 >=
            (int64_t(1) << 31))
            return PSGD_EUNSUPPORTED;
    std::vector<int32_t> nrb(nm, 0), ncc(nm, 0);
    plan->mean_first = plan->workers >= kMeanWorkers &&
                       plan->sizes.n_mat_elems >= std::max<int64_t>(kMeanElems, plan->workers * kMeanElemsPerWorker);
    int64_t narrow = 0;   // elements in rows that are not multiples of 4: a small share (a first layer's rows of 27) does not count
    for (const MatDesc& d : plan->mats)
        if (d.vec != 4) narrow += (int64_t)d.n * d.m;
    if (narrow > plan->sizes.n_mat_elems / 16) plan->mean_first = false;
    if (tu.worker_mean >= 0) plan->mean_first = tu.worker_mean == 1 && plan->workers > 1;
    if (tu.gram_fused == 0) plan->mean_first = false;
    streaming_tiles(plan, 1, tu.k1_rows, tu.k1_nv, true, &plan->tiles1, nullptr, &ncc);
    // The mean first: a list of its own with one column vector per lane, as the sums over the workers take the registers of the
    // second.  Half as wide chunks at most double the partial P of one product, and there is one product instead of W >= 2: the
    // slices lie within those of the workers' own products, whose list stays for when the mean cannot be had.
    std::vector<int32_t> ncc_mean(nm, 0);
    plan->tiles1m.clear();
    if (plan->mean_first) streaming_tiles(plan, 0, tu.k1_rows, 1, true, &plan->tiles1m, nullptr, &ncc_mean);
    streaming_tiles(plan, 2, tu.k3_rows, tu.k3_nv, false, &plan->tiles3, &nrb, nullptr);
    streaming_tiles(plan, 3, tu.k4_rows, tu.k4_nv, false, &plan->tiles4, nullptr, nullptr);

    // The pass fused with the momentum / parameter update moves 20 bytes per element where the plain one moves 12 and
    // wants taller tiles on a mid-sized single-worker set (LSTM-shaped set, rank 4: 163 -> 155 us with 64 rows; the
    // ResNet18-shaped sets at 1 and 16 workers are at their optimum with the plain pass's tiles).
    // Where M fits the memory-side cache and M, momentum and parameters together do not, the last two go around it, on
    // the plain pass's 16-row tiles.  Whole steps, us, before and after: LSTM-shaped set (31.8 M elements) rank 2 bf16 244 / 230, rank 4
    // 254 / 246; rows of 800, 39 M elements 326 / 286; with inputs that change from step to step the first is 259 / 242.
    // Below the line ordinary accesses and 64 rows stay (21 M elements: 209 against 217).
    plan->update_around = plan->workers == 1 && 3 * plan->sizes.n_mat_elems * (int64_t)sizeof(float) > kStreamHintBytes &&
                          plan->sizes.n_mat_elems * (int64_t)sizeof(float) <= kStreamHintBytes && tu.stream_hints < 0 && tu.k4_nv == 1;
    plan->tiles4u.clear();
    if (tu.k4_rows == 0 && !plan->update_around && plan->workers == 1 && !small_set(plan) &&
        plan->sizes.n_mat_elems * (int64_t)sizeof(float) <= kStreamHintBytes)
        streaming_tiles(plan, 3, 64, tu.k4_nv, false, &plan->tiles4u, nullptr, nullptr);

    // vector region: slices appended to the decompress work-list
    const int64_t L = plan->sizes.n_vec_elems;
    const int64_t vec_slice = (int64_t)kBlock * 4 * 4;
    for (int64_t e = 0; e < L; e += vec_slice) {
        Tile t{};
        t.mat = -1;
        t.elem0 = e;
        t.nelem = std::min(vec_slice, L - e);
        plan->tiles4.push_back(t);
        if (!plan->tiles4u.empty()) plan->tiles4u.push_back(t);
    }

    // workspace: partial P of every matrix ([W * n_cchunk][n][r] each), then partial Q
    // ([W * n_rblock][m][r] each), then (doubles) the Gram partials of the tall panels
    const int64_t W = plan->workers;
    int64_t pp = 0, qp = 0, gp = 0;
    plan->tiles_gram.clear();
    plan->small_mats.clear();
    for (size_t i = 0; i < nm; ++i) {
        MatDesc& d = plan->mats[i];
        d.n_cchunk = ncc[i];
        d.n_rblock = nrb[i];
        d.ppart_off = pp;
        pp += round_up(W * d.n_cchunk * d.n * d.r, kAlignElems);
        if ((int64_t)d.n * d.r <= kPanelFloats && d.n <= tu.ortho_rows) {
            d.n_gblock = 0;
            d.gram_off = 0;
            plan->small_mats.push_back((int32_t)i);
        } else {
            d.n_gblock = (int32_t)ceil_div(d.n, kGramRows);
            d.gram_off = gp;
            gp += round_up((int64_t)d.n_gblock * d.r * d.r, 32);
            for (int32_t b = 0; b < d.n_gblock; ++b) {
                Tile t{};
                t.mat = (int32_t)i;
                t.row0 = b * kGramRows;
                t.nrows = std::min<int32_t>(kGramRows, d.n - t.row0);
                t.part = b;
                plan->tiles_gram.push_back(t);
            }
        }
    }
    for (size_t i = 0; i < nm; ++i) {
        MatDesc& d = plan->mats[i];
        d.qpart_off = pp + qp;
        qp += round_up(W * d.n_rblock * d.m * d.r, kAlignElems);
    }
    plan->ws_ppart_floats = pp;
    plan->ws_qpart_floats = qp;
    plan->ws_gram_doubles = gp;
    plan->sizes.workspace_bytes =
        std::max<int64_t>(256, round_up((pp + qp) * (int64_t)sizeof(float), 256) + gp * (int64_t)sizeof(double));

    plan->mats_mean.clear();
    if (plan->mean_first) plan->mats_mean = plan->mats;
    for (size_t i = 0; i < plan->mats_mean.size(); ++i) plan->mats_mean[i].n_cchunk = ncc_mean[i];

    // the same slicing of the n x r panels, used when a matrix has many partial-P slices
    plan->tilesp.clear();
    plan->p_pre_reduce = plan->p_pre_reduce_mean = false;
    for (size_t i = 0; i < nm; ++i) {
        const MatDesc& d = plan->mats[i];
        if (ncc_mean[i] > 2 * kPreReduceParts) plan->p_pre_reduce_mean = true;   // half as wide chunks
        if (W * d.n_cchunk > kPreReduceParts) plan->p_pre_reduce = true;
        const int64_t total = (int64_t)d.n * d.r;
        for (int64_t e = 0; e < total; e += kWave) {
            Tile t{};
            t.mat = (int32_t)i;
            t.elem0 = e;
            t.nelem = std::min<int64_t>(kWave, total - e);
            plan->tilesp.push_back(t);
        }
    }
    // Q reduction: slices of 64 elements of each matrix's m x r panel (4 part-slices per element in a workgroup)
    plan->tilesq.clear();
    for (size_t i = 0; i < nm; ++i) {
        const MatDesc& d = plan->mats[i];
        const int64_t total = (int64_t)d.m * d.r;
        for (int64_t e = 0; e < total; e += kWave) {
            Tile t{};
            t.mat = (int32_t)i;
            t.elem0 = e;
            t.nelem = std::min<int64_t>(kWave, total - e);
            plan->tilesq.push_back(t);
        }
    }
    plan->stream_hints = tu.stream_hints < 0 ? W * plan->sizes.n_mat_elems * (int64_t)sizeof(float) > kStreamHintBytes
                                             : tu.stream_hints != 0;
    build_one_sweep(plan);
    plan->iter_mean = plan->one_sweep && tu.one_sweep < 0 && plan->mean_first && W * plan->sizes.n_mat_elems > kIterMeanElems;
    build_resident(plan, (int64_t)kResCUs * kResBlocksPerCU);
    plan->sizes.workspace_bytes =
        std::max<int64_t>(plan->sizes.workspace_bytes, plan->res_ws_floats * (int64_t)sizeof(float));
    // The planner's own choice: groups; for one worker and a set beyond the memory-side cache the whole list instead
    // (24-layer transformer set, rank 4: k_left 880 -> 842 us, k_decomp 2186 -> 2143 us, k_ef_right 2203 -> 2217 us,
    // the step 5.34 -> 5.28 ms; with the first sweep alone left in groups the second sweep's gain is lost; at 16
    // workers whole-list order loses 1-3 % in every sweep).
    const int64_t order = tu.xcd_order >= 0 ? tu.xcd_order : (W == 1 && plan->stream_hints ? 1 : group_tiles(plan));
    order_tiles(plan->tiles1, order);
    order_tiles(plan->tiles1m, order);
    order_tiles(plan->tiles3, order);
    order_tiles(plan->tiles4, order);
    order_tiles(plan->tiles4u, order);
    plan->tables_built = true;
    return PSGD_OK;
}

// Resident tiling: every matrix is cut into strips of at most `h` rows and chunks of 64 column
// vectors; one wavefront keeps one (strip, chunk) tile in registers for the whole step.  The model
// qualifies when all tiles fit the wavefront slots of one co-resident grid.
static int64_t resident_tiles_for(const psgd_plan* plan, int h) {
    int64_t total = 0;
    for (const MatDesc& d : plan->mats) total += ceil_div(d.n, h) * ceil_div(d.m / d.vec, kWave);
    return total;
}

void build_resident(psgd_plan* plan, int64_t device_blocks) {
    plan->resident_ok = false;
    plan->res_tiles.clear();
    plan->res_mats.clear();
    plan->res_ws_floats = 0;
    plan->res_blocks = 0;
    const Tuning& tu = plan->tuning;
    if (!tu.resident || plan->workers != 1 || plan->rank > kResMaxRank || plan->mats.empty()) return;
    if (plan->grad_dtype != PSGD_F32 || plan->out_dtype != PSGD_F32) return;
    for (const MatDesc& d : plan->mats)
        if (d.n > kResMaxN) return;
    const int64_t max_blocks = tu.res_max_blocks > 0 ? tu.res_max_blocks : device_blocks;
    const int64_t L = plan->sizes.n_vec_elems;
    const int64_t vec_slice = (int64_t)kWave * 4 * 8;   // elements of the vector region per wavefront
    const int64_t vec_tiles = ceil_div(L, vec_slice);

    // The matrices keep model order in the tile list (largest first, so that the matrices with the most strips and
    // column chunks sit in the first workgroups, was 1 % slower on the ResNet18-shaped set).
    auto layout = [&](int h, std::vector<RTile>* tiles, std::vector<MatDesc>* mats, int32_t* n_cntq,
                      int32_t* n_cnts) -> int64_t {
        // returns the number of workgroups, fills the tables when tiles != nullptr
        int64_t slots = 0;            // wavefront slots used so far (multiple of 4 at block boundaries)
        int32_t cntq = 0, cnts = 0;
        int cur_vec = 0;
        if (mats) mats->assign(plan->mats.size(), MatDesc{});
        auto pad_block = [&]() {
            while (slots % kWavesPerBlock) {
                if (tiles) { RTile t{}; t.mat = -2; tiles->push_back(t); }
                ++slots;
            }
        };
        for (size_t i = 0; i < plan->mats.size(); ++i) {
            const MatDesc& d0 = plan->mats[i];
            if (d0.vec != cur_vec) { pad_block(); cur_vec = d0.vec; }
            const int64_t nvec = d0.m / d0.vec;
            const int64_t nchunk = ceil_div(nvec, kWave);
            const int64_t nstrip = ceil_div(d0.n, h);
            int32_t max_runs = 0;
            const size_t first_tile = tiles ? tiles->size() : 0;
            for (int64_t c = 0; c < nchunk; ++c) {
                int32_t runs = 0;
                size_t run_leader = 0;
                const size_t chunk_first = tiles ? tiles->size() : 0;
                for (int64_t sidx = 0; sidx < nstrip; ++sidx) {
                    int64_t r0, rn;
                    even_split(d0.n, nstrip, sidx, &r0, &rn);
                    const bool new_run = (sidx == 0) || (slots % kWavesPerBlock == 0);
                    if (tiles) {
                        RTile t{};
                        t.mat = (int32_t)i;
                        t.row0 = (int32_t)r0;
                        t.nrows = (int32_t)rn;
                        t.vec0 = (int32_t)(c * kWave);
                        t.nvec = (int32_t)std::min<int64_t>(kWave, nvec - c * kWave);
                        t.ppart = (int32_t)c;
                        t.cntq = cntq;
                        t.cnts = cnts + (int32_t)sidx;
                        if (new_run) {
                            run_leader = tiles->size();
                            t.qrun_len = 1;
                            t.qpart = runs;
                        } else {
                            (*tiles)[run_leader].qrun_len += 1;
                        }
                        tiles->push_back(t);
                    }
                    if (new_run) ++runs;
                    ++slots;
                }
                if (tiles)
                    for (size_t k = chunk_first; k < tiles->size(); ++k) (*tiles)[k].nqparts = runs;
                max_runs = std::max(max_runs, runs);
                ++cntq;
            }
            if (tiles) {
                for (size_t k = first_tile; k < tiles->size(); ++k)
                    if ((*tiles)[k].mat == (int32_t)i) (*tiles)[k].nstrips_mat = (int32_t)nstrip;
                MatDesc d = d0;
                d.n_cchunk = (int32_t)nchunk;
                d.n_rblock = max_runs;
                (*mats)[i] = d;
            }
            cnts += (int32_t)nstrip;
        }
        if (vec_tiles) {
            pad_block();
            for (int64_t v = 0; v < vec_tiles; ++v) {
                if (tiles) {
                    RTile t{};
                    t.mat = -1;
                    t.elem0 = v * vec_slice;
                    t.nelem = std::min(vec_slice, L - v * vec_slice);
                    tiles->push_back(t);
                }
                ++slots;
            }
        }
        pad_block();
        if (n_cntq) *n_cntq = cntq;
        if (n_cnts) *n_cnts = cnts;
        return slots / kWavesPerBlock;
    };

    int h = 0;
    const int max_rows = res_rows_for_rank(plan->rank);
    if (tu.res_rows > 0) {
        if (tu.res_rows > max_rows) return;
        h = (int)tu.res_rows;
        if (layout(h, nullptr, nullptr, nullptr, nullptr) > max_blocks) return;
    } else {
        for (int cand = kResMinRows; cand <= max_rows; ++cand) {
            if (layout(cand, nullptr, nullptr, nullptr, nullptr) <= max_blocks) { h = cand; break; }
        }
        if (!h) return;
    }
    int32_t n_cntq = 0, n_cnts = 0;
    const int64_t blocks = layout(h, &plan->res_tiles, &plan->res_mats, &n_cntq, &n_cnts);
    plan->res_strip_rows = h;
    plan->res_blocks = (int32_t)blocks;
    plan->res_n_cntq = n_cntq;
    plan->res_n_cnts = n_cnts;
    // mailbox of the resident kernel (64-bit slots): per matrix [partial P | mean P | P_hat], then per
    // matrix [partial Q | Q]; the offsets are kept in res_mats
    int64_t off = 0;
    for (MatDesc& d : plan->res_mats) {
        d.ppart_off = off;
        off += round_up(((int64_t)d.n_cchunk + 2) * d.n * d.r, kAlignElems);
    }
    for (MatDesc& d : plan->res_mats) {
        d.qpart_off = off;
        off += round_up(((int64_t)d.n_rblock + 1) * d.m * d.r, kAlignElems);
    }
    plan->res_mail_slots = off;
    plan->res_ws_floats = 0;   // nothing of the caller's workspace is used
    plan->res_sync_words = kResSyncWords;
    plan->resident_ok = true;
}

}  // namespace psgd

using namespace psgd;

extern "C" {

psgd_status psgd_plan_create(const psgd_shape* shapes, int32_t n_tensors, int32_t rank, int32_t workers,
                             psgd_dtype grad_dtype, psgd_dtype out_dtype, psgd_plan** out_plan) {
    if (!out_plan) return PSGD_EINVAL;
    *out_plan = nullptr;
    if (!shapes || n_tensors < 1 || rank < 1 || workers < 1) return PSGD_EINVAL;
    if ((grad_dtype != PSGD_F32 && grad_dtype != PSGD_BF16) ||
        (out_dtype != PSGD_F32 && out_dtype != PSGD_BF16))
        return PSGD_EINVAL;
    for (int32_t t = 0; t < n_tensors; ++t) {
        if (shapes[t].rows < 1 || shapes[t].cols < 1) return PSGD_EINVAL;
        if (shapes[t].rows > INT32_MAX || shapes[t].cols > INT32_MAX) return PSGD_EUNSUPPORTED;
    }
    if (rank > PSGD_MAX_RANK) return PSGD_EUNSUPPORTED;
    // the matrix-core kernels (ranks above 8) need row lengths that are multiples of 4 and short enough for 32-bit
    // byte offsets within a tile of rows
    const bool needs_hr = rank > kValuMaxRank;
    if (needs_hr)
        for (int32_t t = 0; t < n_tensors; ++t)
            if (shapes[t].cols != 1 && (shapes[t].cols % 4 != 0 || shapes[t].cols > kHrMaxCols ||
                                        shapes[t].rows > kHrMaxRows))
                return PSGD_EUNSUPPORTED;

    psgd_plan* plan = new (std::nothrow) psgd_plan();
    if (!plan) return PSGD_ENOMEM;
    try {
        plan->rank = rank;
        plan->workers = workers;
        plan->hr = rank > kValuMaxRank;   // settled in build_tables
        plan->hr_nt = rank <= 16 ? 1 : (rank <= 32 ? 2 : 4);
        plan->grad_dtype = grad_dtype;
        plan->out_dtype = out_dtype;
        plan->shapes.assign(shapes, shapes + n_tensors);
        plan->tensor_flat_off.assign(n_tensors, 0);
        plan->tensor_mat.assign(n_tensors, -1);

        const int64_t gsz = grad_dtype == PSGD_BF16 ? 2 : 4;
        const int64_t osz = out_dtype == PSGD_BF16 ? 2 : 4;
        int64_t N = 0, P = 0, Q = 0, payload = 0, compressed = 0, kept_total = 0;
        // matrices first
        for (int32_t t = 0; t < n_tensors; ++t) {
            if (shapes[t].cols == 1) continue;
            MatDesc d{};
            d.n = (int32_t)shapes[t].rows;
            d.m = (int32_t)shapes[t].cols;
            d.r = std::min<int32_t>(rank, std::min(d.n, d.m));
            d.vec = (d.m % 4 == 0) ? 4 : (d.m % 2 == 0 ? 2 : 1);
            d.off = N;
            d.p_off = P;
            d.q_off = Q;
            d.tensor = t;
            plan->tensor_flat_off[t] = N;
            const int32_t mi = (int32_t)plan->mats.size();
            plan->tensor_mat[t] = mi;
            plan->max_n = std::max(plan->max_n, d.n);
            const int64_t elems = (int64_t)d.n * d.m;
            // Appendix G baselines: b = (n + m) r entries per matrix "to match rank-r PowerSGD", at most all of them
            d.kept = std::min(((int64_t)d.n + d.m) * rank, elems);
            d.kept_off = kept_total;
            kept_total += d.kept;
            plan->mats.push_back(d);
            for (int64_t j0 = 0; j0 < d.kept; j0 += kBlock) {
                plan->kept_slice_mat.push_back(mi);
                plan->kept_slice_first.push_back(j0);
            }
            plan->mat_tensor.push_back(t);
            // slices of the flattened matrix for their elementwise sweep: only their running count is kept (the
            // kernel finds its matrix by bisection), not a table of a million entries for a large model
            plan->flat_first.push_back(plan->flat_tiles);
            plan->flat_tiles += ceil_div(elems, kFlatTileElems);
            N += round_up(elems, kAlignElems);
            P += round_up((int64_t)d.n * d.r, kFactorAlignElems);   // every factor starts 16-byte aligned
            Q += round_up((int64_t)d.m * d.r, kFactorAlignElems);
            payload += elems;
            compressed += (int64_t)d.r * ((int64_t)d.n + d.m);
        }
        int64_t L = 0;
        int64_t nvec_t = 0;
        for (int32_t t = 0; t < n_tensors; ++t) {
            if (shapes[t].cols != 1) continue;
            plan->tensor_flat_off[t] = N + L;
            L += shapes[t].rows;
            ++nvec_t;
        }
        plan->flat_first.push_back(plan->flat_tiles);   // one past the last matrix: where the vector region's slices start
        plan->flat_vec_tiles = ceil_div(L, kFlatTileElems);
        psgd_sizes& s = plan->sizes;
        s.kept_elems = kept_total;
        plan->kept_slices = (int64_t)plan->kept_slice_mat.size();
        s.n_mat_elems = N;
        s.n_vec_elems = L;
        s.grad_stride = round_up(N + L, kAlignElems);
        s.err_stride = N;
        s.out_elems = N + L;
        s.p_elems = P;
        s.q_elems = Q;
        s.n_matrices = (int64_t)plan->mats.size();
        s.n_vectors = nvec_t;
        s.payload_elems = payload + L;
        s.compressed_elems = compressed + L;
        const int64_t W = workers;
        s.bytes_min = payload * (W * (gsz + 4 + 4) + osz) + L * (W * gsz + osz);
        s.bytes_stream = s.bytes_min + payload * W * 12;
        psgd_status st = build_tables(plan);
        if (st != PSGD_OK) {
            delete plan;
            return st;
        }
    } catch (const std::bad_alloc&) {
        delete plan;
        return PSGD_ENOMEM;
    }
    *out_plan = plan;
    return PSGD_OK;
}

void psgd_plan_destroy(psgd_plan* plan) {
    if (!plan) return;
    free_tables(plan);
    delete plan;
}

psgd_status psgd_plan_sizes(const psgd_plan* plan, psgd_sizes* out_sizes) {
    if (!plan || !out_sizes) return PSGD_EINVAL;
    *out_sizes = plan->sizes;
    return PSGD_OK;
}

psgd_status psgd_plan_offsets(const psgd_plan* plan, int32_t tensor, int64_t* flat_off, int64_t* p_off,
                              int64_t* q_off, int32_t* eff_rank) {
    if (!plan || tensor < 0 || tensor >= (int32_t)plan->shapes.size()) return PSGD_EINVAL;
    if (flat_off) *flat_off = plan->tensor_flat_off[tensor];
    const int32_t mi = plan->tensor_mat[tensor];
    if (mi < 0) {
        if (p_off) *p_off = -1;
        if (q_off) *q_off = -1;
        if (eff_rank) *eff_rank = 0;
    } else {
        const MatDesc& d = plan->mats[mi];
        if (p_off) *p_off = d.p_off;
        if (q_off) *q_off = d.q_off;
        if (eff_rank) *eff_rank = d.r;
    }
    return PSGD_OK;
}

psgd_status psgd_plan_kept(const psgd_plan* plan, int32_t tensor, int64_t* kept_off, int64_t* kept) {
    if (!plan || tensor < 0 || tensor >= (int32_t)plan->shapes.size()) return PSGD_EINVAL;
    const int32_t mi = plan->tensor_mat[tensor];
    if (kept_off) *kept_off = mi < 0 ? -1 : plan->mats[mi].kept_off;
    if (kept) *kept = mi < 0 ? 0 : plan->mats[mi].kept;
    return PSGD_OK;
}

psgd_status psgd_plan_path(const psgd_plan* plan, int32_t* path) {
    if (!plan || !path) return PSGD_EINVAL;
    *path = plan->hr ? PSGD_PATH_MATRIX_CORES : (plan->resident_ok ? PSGD_PATH_RESIDENT : PSGD_PATH_STREAMING);
    return PSGD_OK;
}

psgd_status psgd_plan_worker_mean(const psgd_plan* plan, int32_t* taken, int64_t* bytes) {
    if (!plan) return PSGD_EINVAL;
    if (plan->one_sweep) {   // the mean is formed as M is walked; held for several iterations in one call alone
        if (taken) *taken = plan->workers > 1 ? 1 : 0;
        if (bytes) *bytes = (plan->uploaded ? plan->mbar != nullptr : plan->iter_mean) ? plan->sizes.n_mat_elems * (int64_t)sizeof(float) : 0;
        return PSGD_OK;
    }
    const bool held = plan->uploaded ? plan->mbar != nullptr : plan->mean_first;
    if (taken) *taken = held && (!plan->uploaded || plan->gram_fused) ? 1 : 0;
    if (bytes) *bytes = held ? plan->sizes.n_mat_elems * (int64_t)sizeof(float) : 0;
    return PSGD_OK;
}

psgd_status psgd_plan_one_sweep(const psgd_plan* plan, int32_t* taken, int64_t* bytes) {
    if (!plan) return PSGD_EINVAL;
    if (taken) *taken = plan->one_sweep || plan->one_wide ? 1 : 0;
    if (bytes) *bytes = plan->one_sweep ? plan->one_bytes : 0;
    return PSGD_OK;
}

psgd_status psgd_random_block_step(psgd_plan* plan, const void* grad, float* err, const int64_t* starts, float* vals,
                                   void* out, void* hip_stream) {
    if (!plan || !grad || !err || !starts || !vals || !out) return PSGD_EINVAL;
    if (plan->grad_dtype != PSGD_F32 || plan->out_dtype != PSGD_F32) return PSGD_EUNSUPPORTED;
    return launch_sparse_step(plan, grad, err, starts, nullptr, vals, out, hip_stream);
}

psgd_status psgd_random_k_step(psgd_plan* plan, const void* grad, float* err, const int64_t* indices, float* vals,
                               void* out, void* hip_stream) {
    if (!plan || !grad || !err || !indices || !vals || !out) return PSGD_EINVAL;
    if (plan->grad_dtype != PSGD_F32 || plan->out_dtype != PSGD_F32) return PSGD_EUNSUPPORTED;
    return launch_sparse_step(plan, grad, err, nullptr, indices, vals, out, hip_stream);
}

psgd_status psgd_plan_set_tuning(psgd_plan* plan, const char* key, int64_t value) {
    if (!plan || !key) return PSGD_EINVAL;
    if (plan->uploaded) return PSGD_EINVAL;
    Tuning tu = plan->tuning;
    if (!strcmp(key, "k1_rows")) tu.k1_rows = value;
    else if (!strcmp(key, "k1_nv")) tu.k1_nv = value;
    else if (!strcmp(key, "k3_rows")) tu.k3_rows = value;
    else if (!strcmp(key, "k3_nv")) tu.k3_nv = value;
    else if (!strcmp(key, "k4_rows")) tu.k4_rows = value;
    else if (!strcmp(key, "k4_nv")) tu.k4_nv = value;
    else if (!strcmp(key, "hr_k3_rows")) tu.hr_k3_rows = value;
    else if (!strcmp(key, "xcd_order")) tu.xcd_order = value;
    else if (!strcmp(key, "hr_k4_rows")) tu.hr_k4_rows = value;
    else if (!strcmp(key, "hr_k1_rows")) tu.hr_k1_rows = value;
    else if (!strcmp(key, "hr_k1_cols")) tu.hr_k1_cols = value;
    else if (!strcmp(key, "resident")) tu.resident = value;
    else if (!strcmp(key, "stream_hints")) tu.stream_hints = value;
    else if (!strcmp(key, "bf16_valu")) tu.bf16_valu = value;
    else if (!strcmp(key, "worker_mean")) tu.worker_mean = value;
    else if (!strcmp(key, "gram_fused")) tu.gram_fused = value;
    else if (!strcmp(key, "gram_spin")) tu.gram_spin = value;
    else if (!strcmp(key, "ortho_rows")) tu.ortho_rows = value;
    else if (!strcmp(key, "one_sweep")) tu.one_sweep = value;
    else if (!strcmp(key, "res_rows")) tu.res_rows = value;
    else if (!strcmp(key, "res_trace")) tu.res_trace = value;
    else if (!strcmp(key, "res_spin")) tu.res_spin = value;
    else if (!strcmp(key, "res_max_blocks")) tu.res_max_blocks = value;
    else return PSGD_EINVAL;
    Tuning old = plan->tuning;
    plan->tuning = tu;
    try {
        psgd_status st = build_tables(plan);
        if (st != PSGD_OK) {
            plan->tuning = old;
            build_tables(plan);
        }
        return st;
    } catch (const std::bad_alloc&) {
        return PSGD_ENOMEM;
    }
}

static bool bad_ptrs(const void* a, const void* b, const void* c, const void* d, const void* e) {
    return !a || !b || !c || !d || !e;
}

psgd_status psgd_compress(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* workspace,
                          void* hip_stream) {
    if (!plan || bad_ptrs(grad, err, q, p, workspace)) return PSGD_EINVAL;
    return launch_compress(plan, grad, err, q, p, workspace, hip_stream);
}

psgd_status psgd_decompress(psgd_plan* plan, const float* p, const float* q, float* err, const void* grad,
                            void* out, void* workspace, void* hip_stream) {
    if (!plan || bad_ptrs(p, q, err, out, workspace) || !grad) return PSGD_EINVAL;
    return launch_decompress(plan, p, q, err, grad, out, workspace, hip_stream);
}

psgd_status psgd_step(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* out,
                      void* workspace, void* hip_stream) {
    if (!plan || bad_ptrs(grad, err, q, p, workspace) || !out) return PSGD_EINVAL;
    if (plan->resident_ok || one_wide_call(plan, grad, out))   // a step of its own, not the two calls
        return launch_resident_step(plan, grad, err, q, p, out, workspace, hip_stream);
    psgd_status st = launch_compress(plan, grad, err, q, p, workspace, hip_stream);
    if (st != PSGD_OK) return st;
    return launch_decompress(plan, p, q, err, grad, out, workspace, hip_stream);
}

psgd_status psgd_step_static(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* out,
                             void* hip_stream) {
    if (!plan || !grad || !err || !q || !p || !out) return PSGD_EINVAL;
    void* ws = nullptr;
    psgd_status st = static_workspace(plan, &ws);
    if (st != PSGD_OK) return st;
    return psgd_step(plan, grad, err, q, p, out, ws, hip_stream);
}

psgd_status psgd_step_iterations(psgd_plan* plan, const void* grad, float* err, float* q, float* p, void* out,
                                 void* workspace, void* hip_stream, int32_t iterations) {
    if (!plan || bad_ptrs(grad, err, q, p, workspace) || !out || iterations < 1 || iterations > 64) return PSGD_EINVAL;
    if (plan->resident_ok) return launch_resident_step(plan, grad, err, q, p, out, workspace, hip_stream, UpdateArgs(), iterations);
    if (iterations == 1) return psgd_step(plan, grad, err, q, p, out, workspace, hip_stream);
    if (plan->iter_mean) return launch_resident_step(plan, grad, err, q, p, out, workspace, hip_stream, UpdateArgs(), iterations);
    psgd_status st = launch_compress(plan, grad, err, q, p, workspace, hip_stream);
    for (int32_t it = 1; it < iterations && st == PSGD_OK; ++it)
        st = launch_compress(plan, nullptr, err, q, p, workspace, hip_stream, false);
    if (st != PSGD_OK) return st;
    return launch_decompress(plan, p, q, err, grad, out, workspace, hip_stream);
}

psgd_status psgd_iterate(psgd_plan* plan, float* err, float* q, float* p, void* workspace, void* hip_stream) {
    if (!plan || !err || !q || !p || !workspace) return PSGD_EINVAL;
    // the gradient pointer is not dereferenced when nothing is added; err stands in so that it is never null
    return launch_compress(plan, err, err, q, p, workspace, hip_stream, false);
}

static bool update_args(const psgd_plan* plan, float* mom, float* param, float lr, float momentum, UpdateArgs* upd) {
    (void)plan;
    if (!mom || !param || !(lr == lr) || !(momentum == momentum)) return false;   // null or NaN
    upd->mom = mom;
    upd->param = param;
    upd->lr = lr;
    upd->lam = momentum;
    return true;
}

psgd_status psgd_decompress_update(psgd_plan* plan, const float* p, const float* q, float* err, const void* grad,
                                   float* mom, float* param, float lr, float momentum, void* workspace,
                                   void* hip_stream) {
    UpdateArgs upd;
    if (!plan || !p || !q || !err || !grad || !workspace || !update_args(plan, mom, param, lr, momentum, &upd))
        return PSGD_EINVAL;
    return launch_decompress(plan, p, q, err, grad, nullptr, workspace, hip_stream, upd);
}

psgd_status psgd_step_update(psgd_plan* plan, const void* grad, float* err, float* q, float* p, float* mom,
                             float* param, float lr, float momentum, void* workspace, void* hip_stream) {
    UpdateArgs upd;
    if (!plan || bad_ptrs(grad, err, q, p, workspace) || !update_args(plan, mom, param, lr, momentum, &upd))
        return PSGD_EINVAL;
    if (plan->resident_ok) return launch_resident_step(plan, grad, err, q, p, nullptr, workspace, hip_stream, upd);
    psgd_status st = launch_compress(plan, grad, err, q, p, workspace, hip_stream);
    if (st != PSGD_OK) return st;
    return launch_decompress(plan, p, q, err, grad, nullptr, workspace, hip_stream, upd);
}

psgd_status psgd_plan_set_profiling(psgd_plan* plan, int32_t enable) {
    if (!plan) return PSGD_EINVAL;
    return set_profiling(plan, enable != 0);
}

psgd_status psgd_plan_kernel_times(psgd_plan* plan, double* ms_sum, int64_t* steps) {
    if (!plan || !ms_sum || !steps) return PSGD_EINVAL;
    for (int i = 0; i < PSGD_N_KERNELS; ++i) {
        ms_sum[i] = plan->kernel_ms[i];
        plan->kernel_ms[i] = 0.0;
    }
    *steps = plan->profiled_steps;
    plan->profiled_steps = 0;
    return PSGD_OK;
}

const char* psgd_kernel_name(int32_t index) {
    static const char* const names[PSGD_N_KERNELS] = {"k_ef_right", "k_ortho",    "k_left",        "k_q_reduce",
                                                      "k_decomp",   "k_resident", "k_ef_add_zero", "k_kept_entries"};
    return (index >= 0 && index < PSGD_N_KERNELS) ? names[index] : nullptr;
}

psgd_status psgd_plan_check(psgd_plan* plan, void* hip_stream, int32_t* is_resident) {
    if (!plan) return PSGD_EINVAL;
    if (is_resident) *is_resident = plan->resident_ok ? 1 : 0;
    return check_plan(plan, hip_stream);
}

psgd_status psgd_plan_read_trace(psgd_plan* plan, uint64_t* out, int64_t capacity, int64_t* n_written) {
    if (!plan || !out || !n_written || capacity < 0) return PSGD_EINVAL;
    return read_trace(plan, out, capacity, n_written);
}

const char* psgd_status_string(psgd_status status) {
    switch (status) {
        case PSGD_OK: return "ok";
        case PSGD_EINVAL: return "invalid argument";
        case PSGD_ENOMEM: return "out of memory";
        case PSGD_EHIP: return "HIP runtime error";
        case PSGD_EUNSUPPORTED: return "unsupported";
    }
    return "unknown status";
}

const char* psgd_plan_last_error(const psgd_plan* plan) { return plan ? plan->last_error.c_str() : ""; }

}  // extern "C"
