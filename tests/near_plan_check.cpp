// Host-side checker of the task lists cut by kNearRule (the table kernel that
// leaves out the pairs beyond the cutoff), built and run by
// tests/test_planner_near_cpu.py: for random item sets and wave counts every
// (i, j) pair of every item is in exactly one task, chunks hold at most 64
// i-particles and share no wave, each part of a split list has a slot of its
// own below n_slots, and the sublists cover the tasks.
#include <cstdio>
#include <random>
#include <set>
#include <string>
#include <vector>

#include "planner.h"

using namespace pgh;

static int check(const std::vector<pgh_item> &items, int ni, int nj, int waves)
{
    HostPlan hp;
    std::string err;
    if (plan_tasks(items.data(), (int)items.size(), ni, nj, near_waves(waves), hp, err, false,
                   kNearRule) != PGH_OK)
        return std::printf("plan_tasks: %s\n", err.c_str()), 1;
    std::vector<Task> t(hp.n_tasks);
    write_tasks(hp, t.data());
    if (hp.q_begin[hp.nq] != hp.n_tasks) return std::printf("sublists\n"), 1;
    std::vector<long long> seen(ni, 0), want(ni, -1);
    std::set<int> slots;
    for (const pgh_item &it : items)
        for (int r = it.i_off; r < it.i_off + it.n_i; ++r) want[r] = it.n_j;
    for (const Task &k : t) {
        if (k.n_i < 1 || k.n_i > 64 || k.n_i2 != 0) return std::printf("chunk\n"), 1;
        if (k.n_parts > 1 && (k.slot + k.part >= hp.n_slots || !slots.insert(k.slot + k.part).second))
            return std::printf("slot\n"), 1;
        for (int r = k.i_off; r < k.i_off + k.n_i; ++r) {
            if (want[r] < 0) return std::printf("row outside\n"), 1;
            seen[r] += k.n_j + (k.part == 0 ? 1LL << 40 : 0);
        }
    }
    for (int r = 0; r < ni; ++r)
        if (want[r] >= 0 ? seen[r] != want[r] + (1LL << 40) : seen[r] != 0)
            return std::printf("row %d\n", r), 1;
    return 0;
}

int main()
{
    std::mt19937 rng(7);
    for (int round = 0; round < 200; ++round) {
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
    std::printf("near plan checks passed\n");
    return 0;
}
