// bulk_mark_parts against times that were measured, and that the sizes of the GPU tests take every way.
#include <stdio.h>

#include <initializer_list>
#include <vector>

#include "cnr_mark_rule.h"

static int failed;
static void check(const char *what, const std::vector<cnr_table_job> &jobs, uint32_t index_bytes, std::initializer_list<uint32_t> good) {
    const uint32_t got = bulk_mark_parts(jobs.data(), (uint32_t)jobs.size(), index_bytes, 256);
    for (uint32_t g : good)
        if (got == g) return;
    printf("%s: %u parts\n", what, got);
    failed = 1;
}
static cnr_table_job table(uint64_t n_rows, uint64_t look_ups, bool scratch = true) {
    static char some;
    cnr_table_job j = {};
    j.n_rows = n_rows;
    j.n_indices = look_ups;
    j.mark_scratch = scratch ? &some : nullptr;
    return j;
}
static std::vector<cnr_table_job> same(uint32_t tables, uint64_t n_rows, uint64_t look_ups) {
    return std::vector<cnr_table_job>(tables, table(n_rows, look_ups));
}

int main() {
    // us through flags and through slices in 2, 4, 8 and 16 parts, with Zipf(1.05) / Zipf(1.2) / no repeats
    check("39 29 78; 8: 25 39 32", same(3, 4000000, 1500000), 8, {8});
    check("37 27 56; 8: 29 34 29", same(3, 4000000, 1000000), 8, {8});
    check("41 29 60; 8: 32 36 32", same(3, 8000000, 1000000), 8, {8});
    check("19 14 29; 8: 19 22 18", same(4, 2000000, 400000), 8, {4, 8});
    check("24 16 34; 8: 25 25 25", same(4, 4000000, 400000), 8, {4, 8});
    check("flags or four parts 13 to 15, 32: 30", same(8, 1310720, 131072), 8, {0, 2, 4, 8});
    check("7 5 10; 32: 17 19 19", same(1, 1310720, 1000000), 8, {0});
    check("14 11 19; 32: 23 24 23", same(2, 1000000, 1000000), 8, {0});
    check("35 29 59; 32: 67 67 67", same(1, 1000000, 10000000), 8, {0});
    check("77 with Zipf(1.2); 8: 201", same(2, 4000000, 10000000), 8, {0});
    check("181 with Zipf(1.2); 8: 557", same(2, 4000000, 30000000), 8, {0});
    check("one large table", same(1, 20000000, 40000000), 8, {0});
    check("27; 8: 48", same(16, 5000000, 131072), 8, {2, 4});
    check("eight tables of a window", same(8, 1000000, 8192000), 8, {32});
    // nothing to choose, and tables that the choice does not look at
    check("no tables", {}, 8, {0});
    check("short streams", same(8, 1000000, 40960), 8, {0});
    check("no scratch", {table(4000000, 1500000, false), table(4000000, 1500000, false)}, 8, {0});
    check("no rows", {table(0, 1500000)}, 8, {0});
    check("more slices than a team", same(3, 30000000, 1500000), 4, {0});
    auto mixed = same(3, 4000000, 1500000);
    mixed.push_back(table(30000000, 3000000));
    mixed.push_back(table(4000000, 1500000, false));
    mixed.push_back(table(4000000, 4000));
    check("the same three among others", mixed, 8, {8});
    check("the most there can be", same(16, 0xFFFFFFFFull, 1ull << 40), 8, {0});

    // no table gets more slabs than its scratch holds
    for (uint64_t n : {1ull, 31ull, 33ull, 1000ull, 1310719ull, 1310720ull, 1310721ull, 2621440ull, 2621441ull, 5242880ull, 5242881ull, 20971520ull, 4294967295ull})
        for (uint32_t want = 2; want <= 32; want *= 2) {
            const uint32_t p = slice_parts(n, want);
            if (p < 2 || p > want || (n + 31) / 32 * 4 * p > mark_scratch_bytes(n)) printf("%llu rows: %u parts\n", (unsigned long long)n, p), failed = 1;
        }

    // the batches of the GPU test, test_bulk_mark_of_a_batch_in_parts, go every way
    const struct { uint32_t tables; uint64_t n_rows, look_ups; } sizes[] = {
        {16, 1310720, 70661}, {16, 5000003, 85100}, {8, 1310721, 131073}, {8, 400001, 524289}, {8, 1000003, 1500000},
        {4, 1310719, 3000001}, {2, 4000000, 2000001}, {1, 1310720, 9000001}, {1, 777777, 70001}, {3, 200033, 150000}};
    uint32_t seen = 0;
    for (const auto &s : sizes)
        for (uint32_t index_bytes : {4u, 8u}) {
            std::vector<cnr_table_job> jobs;
            for (uint32_t i = 0; i < s.tables; ++i) {
                const uint64_t n = i % 3 == 0 ? s.n_rows : s.n_rows / (i % 5 + 1) - i;
                jobs.push_back(table(n < 66 ? 66 : n, s.look_ups));
            }
            const uint32_t p = bulk_mark_parts(jobs.data(), s.tables, index_bytes, 256);
            printf("%2u x %8llu rows, %8llu look-ups of %u bytes: %u parts\n", s.tables, (unsigned long long)s.n_rows, (unsigned long long)s.look_ups, index_bytes, p);
            seen |= p ? p : 1u;
        }
    if (seen != (1 | 2 | 4 | 8 | 16 | 32)) printf("ways taken: %x\n", seen), failed = 1;
    return failed;
}
