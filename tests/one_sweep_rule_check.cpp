// Host-only check of which sets the one walk over M takes and how it divides them, built with g++ and the sanitizers by
// tests/test_one_sweep_rule.py.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <queue>
#include <vector>

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
            std::fflush(stdout);                                    \
            std::_Exit(1);                                          \
        }                                                           \
    } while (0)

using namespace psgd;
typedef std::vector<psgd_shape> Set;

static psgd_plan* make(const Set& s, int rank, int W, psgd_dtype gd = PSGD_F32, psgd_dtype od = PSGD_F32) {
    psgd_plan* plan = nullptr;
    CHECK(psgd_plan_create(s.data(), (int)s.size(), rank, W, gd, od, &plan) == PSGD_OK);
    return plan;
}

static Set many(int n, psgd_shape s, int more = 0, psgd_shape t = {1, 1}) {
    Set v((size_t)n, s);
    v.insert(v.end(), (size_t)more, t);
    return v;
}

// Sets of more matrices than there are workgroups at once: the last workgroup to end has no more than twice its share of the elements,
// dealt in the order of the list, and every row lies in one block.
static void check_many() {
    Set powers, steps;
    for (int i = 0; i < 600; ++i) powers.push_back({64 << (i % 5), 64 << (i / 5 % 5)});
    for (int i = 0; i < 480; ++i) steps.push_back({100 + 37 * i % 900, 50 + 91 * i % 1900});
    const Set sets[] = {many(600, {64, 9}, 1, {1000, 2560}), many(400, {32, 9}, 20, {512, 2304}), many(400, {32, 9}, 100, {512, 2304}), powers, steps,
                        many(300, {1000, 1000}), many(250, {64, 9}, 1, {1000, 2560})};
    for (const Set& s : sets)
        for (int W : {1, 3}) {
            psgd_plan* plan = make(s, 2, W);
            CHECK(psgd_plan_set_tuning(plan, "one_sweep", 1) == PSGD_OK && plan->one_sweep && plan->one_bytes <= kOneMaxBytes);
            const size_t slots = (size_t)kResCUs * (kOneMaxWaves / plan->one_waves);
            std::vector<std::vector<int>> rows;
            for (const OneMat& o : plan->one_mats) rows.emplace_back(o.n, 0);
            int64_t total = 0, last = 0;
            std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> ends;
            for (const OneTile& t : plan->one_tiles) {
                int64_t at = 0;
                if (ends.size() >= slots) {
                    at = ends.top();
                    ends.pop();
                }
                at += (int64_t)t.nrows * plan->one_mats[t.mat].m;
                ends.push(at);
                last = std::max(last, at);
                total += (int64_t)t.nrows * plan->one_mats[t.mat].m;
                CHECK(t.block >= 0 && t.block < plan->one_mats[t.mat].n_blocks);
                for (int r = 0; r < t.nrows; ++r) rows[t.mat].at(t.row0 + r) += 1;
            }
            for (auto& v : rows)
                for (int x : v) CHECK(x == 1);
            CHECK(last <= 2 * total / (int64_t)slots + 4 * kOneRows * 2560);   // or a full pipeline of the longest rows
            psgd_plan_destroy(plan);
        }
}

// A finer division is not taken where its partial sums are more than the plan may hold and those of a coarser one are not.
static void check_memory() {
    Set s;
    for (int i = 0; i < 24; ++i) s.insert(s.end(), {{1024, 1024}, {1024, 1024}, {1024, 1024}, {1024, 1024}, {4096, 1024}, {1024, 4096}});
    s.push_back({50304, 1024});
    for (int rank : {1, 2, 3, 4}) {
        psgd_plan* plan = make(s, rank, 1);
        CHECK(plan->one_sweep && plan->one_bytes <= kOneMaxBytes);
        psgd_plan_destroy(plan);
    }
}

// A group of wavefronts walks two steps at least; one where two would leave fewer blocks than half of the workgroups that the device
// holds on sets under 2^19 elements from eight workers on, than a quarter with one worker at ranks 3 and 4.
static void check_steps() {
    for (const Set& s : {many(1, {37, 90}), many(3, {100, 200}), many(3, {128, 1500}), many(11, {160, 300}), many(15, {400, 300}), many(8, {512, 320}), many(20, {400, 300})})
        for (int rank : {1, 2, 3, 4})
            for (int W : {1, 2, 4, 8, 32}) {
                psgd_plan* plan = make(s, rank, W);
                CHECK(psgd_plan_set_tuning(plan, "one_sweep", 1) == PSGD_OK && plan->one_sweep);
                const int64_t slots = kResCUs * (kOneMaxWaves / plan->one_waves), rows = (plan->one_waves >> plan->one_mats[0].waves_log2) * kOneRows;
                const int64_t n = plan->one_mats[0].n, at_two = (int64_t)s.size() * ((n + 2 * rows - 1) / (2 * rows));
                const int64_t steps = at_two < (W >= 8 && plan->sizes.n_mat_elems < kOneStepElems ? slots / 2 : (W == 1 && rank >= 3 ? slots / 4 : 0)) ? 1 : 2;
                for (const OneMat& o : plan->one_mats) {
                    CHECK(o.n_blocks <= (n + steps * rows - 1) / (steps * rows));
                    if (s.size() <= 3) CHECK(o.n_blocks == (n + steps * rows - 1) / (steps * rows));
                }
                psgd_plan_destroy(plan);
            }
}

struct Line { Set s; int rank, W; bool taken; };

// Each line of the rule from both sides; a plan that is asked for the one walk gets it on either, and the two walks' workspace is not
// touched by the choice.
static void check_lines(const std::vector<Line>& lines) {
    for (const Line& c : lines) {
        psgd_plan* plan = make(c.s, c.rank, c.W);
        if (plan->one_sweep != c.taken) std::printf("%lld x %lld, %d matrices, rank %d, %d workers\n", (long long)c.s[0].rows, (long long)c.s[0].cols, (int)c.s.size(), c.rank, c.W);
        CHECK(plan->one_sweep == c.taken);
        const int64_t ws = plan->sizes.workspace_bytes;
        CHECK(psgd_plan_set_tuning(plan, "one_sweep", 1) == PSGD_OK && plan->one_sweep && plan->sizes.workspace_bytes == ws);
        CHECK(psgd_plan_set_tuning(plan, "one_sweep", 0) == PSGD_OK && !plan->one_sweep && plan->sizes.workspace_bytes == ws);
        psgd_plan_destroy(plan);
    }
}

// One worker: rows that leave two thirds of the lanes idle; partial sums as heavy as M.  Several: partial sums heavier than three words an element.
static const std::vector<Line> kOneWorker = {
    {many(20, {500, 250}), 2, 1, false}, {many(20, {500, 250}), 1, 1, false}, {many(20, {500, 258}), 2, 1, true}, {many(20, {500, 250}), 2, 2, true},
    {many(1, {50000, 250}), 2, 1, false}, {many(4, {500, 250}), 2, 1, true}, {many(20, {2000, 100}), 2, 1, false}, {many(20, {2000, 100}), 1, 1, true},
    {many(20, {3000, 100}), 2, 1, true}, {many(20, {2000, 101}), 2, 1, true}, {many(20, {500, 250}, 20, {500, 300}), 2, 1, true},
    {many(10, {100, 3000}), 4, 1, false}, {many(10, {100, 3000}), 2, 1, false}, {many(10, {1000, 3000}), 4, 1, true}, {many(1, {900, 640}), 4, 1, true},
    {many(10, {100, 3000}), 4, 2, false}, {many(10, {100, 3000}), 2, 2, true}, {many(10, {100, 3000}), 4, 3, true}};

// Sets that would take the mean first, beyond the memory-side cache: above eight workers, or rows of eight wavefronts, that fill the
// mean's chunks of columns.
static const std::vector<Line> kMeanFirst = {
    {many(40, {256, 1024}), 2, 8, true}, {many(40, {256, 1024}), 2, 9, false}, {many(18, {256, 1024}), 2, 16, true}, {many(40, {256, 648}), 2, 16, true},
    {many(40, {256, 1026}), 2, 16, true}, {many(12, {2000, 4096}), 2, 4, false}, {many(12, {2000, 2048}), 2, 4, true}, {many(12, {2000, 4096}), 2, 3, true},
    {many(2, {2000, 4096}), 2, 4, true}, {many(4, {2000, 2052}), 2, 16, true}};

// Small sets of many workers in narrow rows.
static const std::vector<Line> kNarrow = {
    {many(5, {200, 201}), 2, 17, false}, {many(5, {200, 201}), 2, 16, true}, {many(5, {200, 200}), 2, 32, true}, {many(5, {700, 601}), 2, 32, true},
    {many(5, {700, 601}), 2, 33, false}};

// Several iterations in one call go over the stored mean: where the mean would be taken first without the one walk, above 20 * 2^20
// elements of all workers.  The memory for it is reported, and none where it is not used.
static void check_iterations() {
    struct { Set s; int W; bool one, mean; } cases[] = {{many(1, {1200, 1200}), 16, true, true}, {many(1, {1200, 1000}), 16, true, false}, {many(1, {1024, 1280}), 16, true, false}, {many(1, {1028, 1280}), 16, true, true},
                                                        {many(5, {1200, 1200}), 3, true, false}, {many(5, {1200, 1200}), 4, true, true}, {many(5, {1200, 1201}), 4, true, false}};
    for (auto& c : cases) {
        psgd_plan* plan = make(c.s, 2, c.W);
        CHECK(plan->one_sweep == c.one && plan->iter_mean == c.mean);
        int32_t taken = -1;
        int64_t bytes = -1;
        CHECK(psgd_plan_worker_mean(plan, &taken, &bytes) == PSGD_OK && taken == 1 && bytes == (c.mean ? plan->sizes.n_mat_elems * 4 : 0));
        for (int64_t v : {0, 1}) CHECK(psgd_plan_set_tuning(plan, "one_sweep", v) == PSGD_OK && !plan->iter_mean);
        CHECK(psgd_plan_set_tuning(plan, "one_sweep", -1) == PSGD_OK && plan->iter_mean == c.mean);
        psgd_plan_destroy(plan);
    }
}

// The walk of the matrix-core plans: not where most elements lie in rows that leave three quarters of a wavefront's columns empty.
static void check_wide_lines() {
    struct { Set s; bool taken; } cases[] = {{many(1, {400000, 256}), true}, {many(1, {400000, 252}), false}, {many(2200, {200, 200}), false},
                                             {many(1, {300000, 200}, 1, {100000, 1024}), true}, {many(1, {600000, 200}, 1, {100000, 1024}), false}};
    for (auto& c : cases) {
        psgd_plan* plan = make(c.s, 4, 1, PSGD_BF16, PSGD_BF16);
        CHECK(plan->hr && plan->one_wide == c.taken);
        CHECK(psgd_plan_set_tuning(plan, "one_sweep", 1) == PSGD_OK && plan->one_wide);
        CHECK(psgd_plan_set_tuning(plan, "stream_hints", 0) == PSGD_OK && !plan->one_wide);   // its accesses to M are non-temporal
        CHECK(psgd_plan_set_tuning(plan, "stream_hints", 1) == PSGD_OK && plan->one_wide);
        psgd_plan_destroy(plan);
    }
}

// one_sweep out of its range is refused whatever kernels the plan runs, and leaves the plan as it was.
static void check_range() {
    for (int rank : {2, 4, 16}) {
        psgd_plan* plan = make(many(1, {50304, 2048}), rank, 1, PSGD_BF16, PSGD_BF16);
        const bool wide = plan->one_wide, one = plan->one_sweep;
        for (int64_t bad : {-9, -2, 2, 7}) CHECK(psgd_plan_set_tuning(plan, "one_sweep", bad) == PSGD_EINVAL && plan->one_wide == wide && plan->one_sweep == one);
        CHECK(psgd_plan_set_tuning(plan, "xcd_order", 1) == PSGD_OK && plan->one_wide == wide && plan->one_sweep == one);
        psgd_plan_destroy(plan);
    }
}

int main() {
    check_range();
    check_wide_lines();
    check_iterations();
    check_lines(kNarrow);
    check_lines(kMeanFirst);
    check_lines(kOneWorker);
    check_many();
    check_memory();
    check_steps();
    std::printf("OK\n");
    return 0;
}
