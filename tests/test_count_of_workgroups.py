"""The count by which a launch's last workgroup knows itself (k_count.h), on the host: launches by themselves, in any order of their workgroups, and
launches whose workgroups come in among one another's, after which the next launch by itself has to be right again."""
from test_lists_cut import run_host_check

CHECK = r"""
#include <stdio.h>
#include <algorithm>
#include <random>
#include <vector>
#include "k_count.h"
static int bad = 0;
static uint32_t word = 0;
static std::mt19937 gen(5);
// how many workgroups of `grid` take themselves for the last one, and whether it is the one that comes last
static void alone(uint32_t grid) {
    std::vector<uint32_t> order(grid);
    for (uint32_t i = 0; i < grid; ++i) order[i] = i;
    std::shuffle(order.begin(), order.end(), gen);
    for (uint32_t i = 0; i < grid; ++i) {
        const uint32_t share = usl_count_share(order[i], grid), before = word;
        word += share;
        if (usl_count_is_last(before, share) != (i + 1 == grid)) { if (bad++ < 20) printf("grid %u: workgroup %u, %u-th to come\n", grid, order[i], i); }
    }
    if (word != 0) { if (bad++ < 20) printf("grid %u leaves %u\n", grid, word); }
}
int main() {
    for (uint32_t grid : {1u, 2u, 3u, 17u, 255u, 256u, 257u, 512u, 100003u}) for (int i = 0; i < 5; ++i) alone(grid);
    for (int turn = 0; turn < 200; ++turn) {   // two to four launches at a time, then one by itself
        std::vector<uint32_t> shares;
        for (int n = 2 + (int)(gen() % 3); n > 0; --n) {
            const uint32_t grid = 1 + gen() % 300;
            for (uint32_t i = 0; i < grid; ++i) shares.push_back(usl_count_share(i, grid));
        }
        std::shuffle(shares.begin(), shares.end(), gen);
        for (uint32_t s : shares) word += s;
        alone(1 + gen() % 300);
    }
    return bad != 0;
}
"""


def test_count_of_workgroups(tmp_path):
    r = run_host_check(tmp_path, CHECK)
    assert r.returncode == 0, r.stdout
