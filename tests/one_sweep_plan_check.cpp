// Host-only check of the tables of the one walk over M (k_one_sweep, k_solve), built with g++ and the sanitizers by
// tests/test_one_sweep.py: every row of every matrix belongs to exactly one block, every row of P and Q is solved exactly once, the
// partial sums lie apart within the plan's memory, a row fits the lanes of its wavefronts and the workgroup's shared memory its uses.
#include <cstdio>
#include <cstdint>
#include <cstdlib>
#include <random>

#include "psgd_internal.h"

namespace psgd {
void free_tables(psgd_plan*) {}
psgd_status set_profiling(psgd_plan*, bool) { return PSGD_EHIP; }
psgd_status check_plan(psgd_plan*, void*) { return PSGD_EHIP; }
psgd_status launch_sparse_step(psgd_plan*, const void*, float*, const int64_t*, const int64_t*, float*, void*, void*) { return PSGD_EHIP; }
psgd_status static_workspace(psgd_plan*, void**) { return PSGD_EHIP; }
psgd_status read_trace(psgd_plan*, uint64_t*, int64_t, int64_t*) { return PSGD_EHIP; }
psgd_status launch_resident_step(psgd_plan*, const void*, float*, float*, float*, void*, void*, void*, const UpdateArgs&, int) { return PSGD_EHIP; }
psgd_status launch_compress(psgd_plan*, const void*, float*, float*, float*, void*, void*, bool) { return PSGD_EHIP; }
psgd_status launch_decompress(psgd_plan*, const float*, const float*, float*, const void*, void*, void*, void*, const UpdateArgs&) { return PSGD_EHIP; }
}  // namespace psgd

#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            std::printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c); \
            std::exit(1);                                           \
        }                                                           \
    } while (0)

using namespace psgd;

static psgd_plan* make(const std::vector<psgd_shape>& s, int rank, int W, psgd_dtype gd = PSGD_F32) {
    psgd_plan* plan = nullptr;
    CHECK(psgd_plan_create(s.data(), (int)s.size(), rank, W, gd, PSGD_F32, &plan) == PSGD_OK);
    return plan;
}

static void check(const std::vector<psgd_shape>& s, int rank, int W, psgd_dtype gd) {
    psgd_plan* plan = make(s, rank, W, gd);
    const bool mean = W > 1;
    if (plan->one_sweep) {
        CHECK(rank <= kOneMaxRank && (plan->one_waves == 4 || plan->one_waves == 8) && plan->one_mats.size() == plan->mats.size());
        const int NG = rank * (rank + 1) / 2;
        int64_t s_at = 0, g_at = 0, at = 0;
        std::vector<std::vector<int>> p_rows, q_rows;
        std::vector<size_t> first_tile;
        for (size_t i = 0; i < plan->one_mats.size(); ++i) {
            const OneMat& o = plan->one_mats[i];
            const MatDesc& d = plan->mats[i];
            CHECK(o.off == d.off && o.p_off == d.p_off && o.q_off == d.q_off && o.n == d.n && o.m == d.m && o.r == d.r && o.vec == d.vec);
            CHECK(o.m % o.vec == 0 && (1 << o.waves_log2) <= plan->one_waves);
            CHECK(o.m / o.vec <= (kWave << o.waves_log2) * one_nv(o.vec, mean));
            CHECK((int64_t)o.m * 4 < (int64_t(1) << 31) && (int64_t)o.n * o.r * 4 < (int64_t(1) << 31));
            CHECK(o.s_off == s_at && o.g_off == g_at && o.n_blocks >= 1);
            s_at += (int64_t)o.n_blocks * o.m * o.r;
            g_at += (int64_t)o.n_blocks * NG;
            CHECK(one_q_floats(rank, o.vec, mean) % 4 == 0 && one_q_floats(rank, o.vec, mean) >= one_nv(o.vec, mean) * o.vec * rank);
            CHECK((int64_t)(kWave << o.waves_log2) * one_q_floats(rank, o.vec, mean) * 4 <= plan->one_lds_bytes);
            CHECK((int64_t)one_deposit(rank, o.vec, mean) * o.vec * rank * (plan->one_waves * kWave + 1) * 8 <= plan->one_lds_bytes);
            CHECK(one_nv(o.vec, mean) % one_deposit(rank, o.vec, mean) == 0);
            int64_t row = 0;
            for (int b = 0; b < o.n_blocks; ++b, ++at) {
                const OneTile& t = plan->one_tiles[(size_t)at];
                CHECK(t.mat == (int)i && t.block == b && t.row0 == row && t.nrows >= 1);
                row += t.nrows;
            }
            CHECK(row == o.n);
            p_rows.emplace_back(o.n, 0);
            q_rows.emplace_back(o.m, 0);
        }
        CHECK(at == (int64_t)plan->one_tiles.size());
        CHECK(s_at <= plan->one_s_doubles && (plan->one_s_doubles + g_at) * 8 == plan->one_bytes && plan->one_bytes <= kOneMaxBytes);
        CHECK(plan->one_lds_bytes <= 128 << 10 && (plan->one_waves == 8 || plan->one_lds_bytes <= 72 << 10));   // two workgroups on a compute unit
        for (const SolveTile& t : plan->solve_tiles) {
            CHECK(t.mat >= 0 && t.mat < (int)plan->one_mats.size() && t.cols_log2 >= 0 && t.cols_log2 <= 8 && t.first >= 0);
            CHECK(t.count >= 1 && t.count <= (t.rows ? kBlock : 1 << t.cols_log2));
            std::vector<int>& v = t.rows ? p_rows[t.mat] : q_rows[t.mat];
            CHECK(t.first + t.count <= (int)v.size());
            for (int k = 0; k < t.count; ++k) v[t.first + k] += 1;
        }
        for (auto* part : {&p_rows, &q_rows})
            for (auto& v : *part)
                for (int x : v) CHECK(x == 1);
    }
    psgd_plan_destroy(plan);
}

// The walk of the matrix-core plans: every row in one block, partial S within the matrix's own part of `out`, blocks in falling size.
static void check_wide() {
    const std::vector<std::vector<psgd_shape>> sets = {
        {{50304, 2048}, {2048, 2048}, {8192, 2048}, {2048, 8192}, {2048, 1}}, {{21000, 4096}, {16, 8}, {32, 8192}, {5, 1}}, {{100000, 1024}}, {{6000, 8192}, {12004, 4096}}};
    for (auto& s : sets)
        for (psgd_dtype od : {PSGD_BF16, PSGD_F32}) {
            psgd_plan* plan = nullptr;
            CHECK(psgd_plan_create(s.data(), (int)s.size(), 4, 1, PSGD_BF16, od, &plan) == PSGD_OK);
            CHECK(plan->hr && plan->one_wide && !plan->one_sweep && plan->one_mats.size() == plan->mats.size());
            const int64_t osz = od == PSGD_BF16 ? 2 : 4;
            std::vector<std::vector<int>> rows, p_rows, q_rows;
            int64_t g_at = 0, last = INT64_MAX;
            for (size_t i = 0; i < plan->one_mats.size(); ++i) {
                const OneMat& o = plan->one_mats[i];
                CHECK(o.n_blocks >= 1 && o.m % 4 == 0 && o.m <= (kWave << o.waves_log2) * kOneWideNV * 4 && (1 << o.waves_log2) <= kOneMaxWaves);
                CHECK(o.s_off * 8 == plan->mats[i].off * osz && (int64_t)o.n_blocks * o.m * o.r * 8 <= (int64_t)o.n * o.m * osz);
                CHECK(o.g_off == g_at);
                g_at += (int64_t)o.n_blocks * 10;
                rows.emplace_back(o.n, 0);
                p_rows.emplace_back(o.n, 0);
                q_rows.emplace_back(o.m, 0);
            }
            CHECK(g_at * 8 <= plan->sizes.workspace_bytes);
            std::vector<std::vector<int>> block_seen(rows.size());
            for (size_t i = 0; i < rows.size(); ++i) block_seen[i].assign(plan->one_mats[i].n_blocks, 0);
            for (const OneTile& t : plan->one_tiles) {
                CHECK(t.nrows >= 1 && t.row0 >= 0 && t.row0 + t.nrows <= plan->one_mats[t.mat].n);
                for (int r = 0; r < t.nrows; ++r) rows[t.mat][t.row0 + r] += 1;
                block_seen[t.mat].at(t.block) += 1;
                const int64_t size = (int64_t)t.nrows * plan->one_mats[t.mat].m;
                CHECK(size <= last);
                last = size;
            }
            for (const SolveTile& t : plan->solve_tiles)
                for (int k = 0; k < t.count; ++k) (t.rows ? p_rows : q_rows)[t.mat].at(t.first + k) += 1;
            for (auto* part : {&rows, &p_rows, &q_rows, &block_seen})
                for (auto& v : *part)
                    for (int x : v) CHECK(x == 1);
            CHECK(psgd_plan_set_tuning(plan, "hr_k3_rows", 1024) == PSGD_OK && plan->hr && !plan->one_wide);
            CHECK(psgd_plan_set_tuning(plan, "hr_k3_rows", 2048) == PSGD_OK && plan->one_wide);
            CHECK(psgd_plan_set_tuning(plan, "one_sweep", 0) == PSGD_OK && !plan->one_wide);
            psgd_plan_destroy(plan);
        }
    struct { std::vector<psgd_shape> s; int rank, W; psgd_dtype gd; } no[] = {
        {{{50304, 2048}}, 5, 1, PSGD_BF16}, {{{50304, 2048}}, 4, 2, PSGD_BF16}, {{{50304, 2048}}, 4, 1, PSGD_F32}, {{{11000, 8196}}, 4, 1, PSGD_BF16},
        {{{50304, 2048}, {15, 64}}, 4, 1, PSGD_BF16}, {{{6000, 8192}, {12000, 4092}}, 4, 1, PSGD_BF16}};
    for (auto& c : no) {
        psgd_plan* plan = nullptr;
        CHECK(psgd_plan_create(c.s.data(), (int)c.s.size(), c.rank, c.W, c.gd, PSGD_BF16, &plan) == PSGD_OK && plan->hr && !plan->one_wide);
        psgd_plan_destroy(plan);
    }
}

int main() {
    check_wide();
    // Which plans take it, and that nothing of the other route moves: every line of the rule from both sides.
    struct { std::vector<psgd_shape> s; int rank, W; bool taken; } rule[] = {
        {{{900, 6144}}, 2, 1, true},  {{{900, 6148}}, 2, 1, false}, {{{900, 4096}}, 2, 2, true}, {{{900, 4100}}, 2, 2, false},
        {{{900, 6142}}, 2, 1, true},  {{{900, 3070}}, 2, 2, true},  {{{900, 3074}}, 2, 2, false}, {{{900, 4095}}, 2, 1, true},
        {{{900, 4097}}, 2, 1, false}, {{{900, 640}}, 4, 1, true},   {{{900, 640}}, 5, 1, false}, {{{64, 576}, {900, 6148}}, 2, 1, false},
    };
    for (auto& c : rule) {
        psgd_plan* plan = make(c.s, c.rank, c.W);
        CHECK(plan->one_sweep == c.taken);
        const int64_t ws = plan->sizes.workspace_bytes;
        int32_t taken = -1;
        int64_t bytes = -1;
        CHECK(psgd_plan_one_sweep(plan, &taken, &bytes) == PSGD_OK && taken == c.taken && (bytes > 0) == c.taken);
        for (const char* key : {"worker_mean", "gram_fused"}) {   // asks for kernels of the two walks
            CHECK(psgd_plan_set_tuning(plan, key, 0) == PSGD_OK && !plan->one_sweep && plan->sizes.workspace_bytes == ws);
            CHECK(psgd_plan_set_tuning(plan, key, -1) == PSGD_OK && plan->one_sweep == c.taken);
        }
        CHECK(psgd_plan_set_tuning(plan, "ortho_rows", 64) == PSGD_OK && !plan->one_sweep);
        CHECK(psgd_plan_set_tuning(plan, "one_sweep", 1) == PSGD_OK && plan->one_sweep == c.taken);
        CHECK(psgd_plan_set_tuning(plan, "one_sweep", 0) == PSGD_OK && !plan->one_sweep);
        for (int64_t bad : {-2, 2}) CHECK(psgd_plan_set_tuning(plan, "one_sweep", bad) == PSGD_EINVAL);
        psgd_plan_destroy(plan);
    }
    {
        psgd_plan* plan = make({{7168, 4096}}, 2, 1, PSGD_BF16);
        CHECK(plan->one_sweep && psgd_plan_set_tuning(plan, "bf16_valu", 0) == PSGD_OK && plan->hr && !plan->one_sweep);
        psgd_plan_destroy(plan);
        CHECK(psgd_plan_one_sweep(nullptr, nullptr, nullptr) == PSGD_EINVAL);
    }
    std::vector<std::vector<psgd_shape>> sets = {
        {{1, 2}, {2, 1}}, {{1, 6144}}, {{3, 2}, {2, 3}, {5, 5}}, {{33280, 650}, {2600, 650}, {2600, 650}, {650, 1}}, {{200000, 3}},
        {{64, 27}, {64, 576}, {64, 576}, {128, 576}}, {{17, 3071}, {9, 2049}, {100, 4}}, {{2048, 2048}, {100, 6000}},
    };
    std::mt19937 rng(1);
    for (int k = 0; k < 40; ++k) {
        std::vector<psgd_shape> s;
        const int n = 1 + (int)(rng() % 20);
        for (int i = 0; i < n; ++i) s.push_back({1 + (int64_t)(rng() % (k % 3 ? 300 : 5000)), 2 + (int64_t)(rng() % (k % 2 ? 700 : 4000))});
        sets.push_back(s);
    }
    for (auto& s : sets)
        for (int rank = 1; rank <= 4; ++rank)
            for (int W : {1, 2, 5}) check(s, rank, W, rank % 2 ? PSGD_F32 : PSGD_BF16);
    std::printf("OK\n");
    return 0;
}
