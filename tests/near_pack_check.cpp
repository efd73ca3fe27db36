// Host-side checker of packed task lists cut by kNearRule (pgh_set_plan_packing
// with the second list of a small plan), built and run by
// tests/test_planner_near_pack_cpu.py: for random item sets and wave counts a task
// holds one or two chunks of at most 64 i-particles together, every row of every
// item meets its whole list once, the parts of a split task have slots of their own,
// and the sublists cover the tasks.
#include <cstdio>
#include <random>
#include <set>
#include <string>
#include <vector>

#include "planner.h"

using namespace pgh;

static int g_pairs = 0;

static int check(const std::vector<pgh_item> &items, int ni, int nj, int waves)
{
    HostPlan hp;
    std::string err;
    if (plan_tasks(items.data(), (int)items.size(), ni, nj, near_waves(waves), hp, err, true,
                   kNearRule) != PGH_OK)
        return std::printf("plan_tasks: %s\n", err.c_str()), 1;
    std::vector<Task> t(hp.n_tasks);
    write_tasks(hp, t.data());
    if (hp.q_begin[hp.nq] != hp.n_tasks) return std::printf("sublists\n"), 1;
    std::vector<long long> seen(ni, 0), want(ni, -1), at(ni, -1);
    std::set<int> slots;
    for (const pgh_item &it : items)
        for (int r = it.i_off; r < it.i_off + it.n_i; ++r) want[r] = it.n_j, at[r] = it.j_off;
    for (const Task &k : t) {
        if (k.n_i < 1 || k.n_i2 < 0 || k.n_i + k.n_i2 > 64) return std::printf("chunk\n"), 1;
        if (k.n_parts > 1 && (k.slot + k.part >= hp.n_slots || !slots.insert(k.slot + k.part).second))
            return std::printf("slot\n"), 1;
        g_pairs += k.n_i2 > 0;
        for (int sub = 0; sub < (k.n_i2 > 0 ? 2 : 1); ++sub) {
            const int i0 = sub ? k.i_off2 : k.i_off, n = sub ? k.n_i2 : k.n_i;
            const int j0 = sub ? k.j_off2 : k.j_off, m = sub ? k.n_j2 : k.n_j;
            for (int r = i0; r < i0 + n; ++r) {
                if (want[r] < 0 || m < 0 || (m && (j0 < at[r] || j0 + m > at[r] + want[r])))
                    return std::printf("row or range outside\n"), 1;
                seen[r] += m + (k.part == 0 ? 1LL << 40 : 0);
            }
        }
    }
    for (int r = 0; r < ni; ++r)
        if (want[r] >= 0 ? seen[r] != want[r] + (1LL << 40) : seen[r] != 0)
            return std::printf("row %d\n", r), 1;
    return 0;
}

int main()
{
    std::mt19937 rng(11);
    for (int round = 0; round < 120; ++round) {
        const int n = 1 + (int)(rng() % 400), big = round % 7 == 0 ? 30000 : 1500;
        std::vector<pgh_item> items;
        int i0 = 0, j0 = 0;
        for (int k = 0; k < n; ++k) {
            pgh_item it{i0, (int)(rng() % 200), j0, (int)(rng() % big)};
            i0 += it.n_i + (int)(rng() % 3);
            j0 += it.n_j;
            items.push_back(it);
        }
        for (int waves : {1, 64, 8192})
            if (check(items, i0, j0, waves)) return 1;
    }
    if (g_pairs == 0) return std::printf("nothing was packed\n"), 1;
    std::printf("near pack checks passed\n");
    return 0;
}
