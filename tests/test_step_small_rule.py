"""Which layers take the small step (k_step_small.h), on the host: the layers on either side of its lines, and LDS that fits."""
from test_lists_cut import run_host_check

CHECK = r"""
#include <stdio.h>
#include "k_step_small.h"
using namespace usl_small;
static int bad = 0;
static void want(bool yes, long long m, int d, int k, int b) {
    const bool got = small_step_fits(m, d, k, b) && small_step_pays(m, d, k, b, 256);
    if (got != yes) { ++bad; printf("m %lld d %d k %d b %d: %d\\n", m, d, k, b, (int)got); }
}
int main() {
    // faster so: latency-bound layers, two rounds by registers, long rows of few instances, few features
    want(true, 1024, 64, 8, 16); want(true, 16000, 64, 32, 64); want(true, 30000, 64, 18, 40); want(true, 76770, 62, 12, 4); want(true, 61269, 79, 6, 52);
    want(true, 2096, 5314, 2, 4); want(true, 1762, 6033, 6, 1); want(true, 4360, 5371, 2, 1); want(true, 137886, 16, 4, 4); want(true, 72586, 181, 3, 11);
    want(true, 3782, 747, 16, 17);
    // slower so: many labels with few slots, long rows of several groups of instances, two rounds by LDS
    want(false, 200000, 64, 3, 8); want(false, 188394, 28, 1, 3); want(false, 113303, 265, 4, 5); want(false, 98337, 252, 1, 6); want(false, 224083, 27, 2, 9);
    want(false, 15555, 1658, 24, 9); want(false, 9551, 778, 28, 28); want(false, 31147, 211, 31, 43); want(false, 31974, 843, 16, 19);
    // does not fit
    want(false, 1000, 9217, 8, 4); want(false, 1000, 64, 33, 4);
    for (int b = 1; b <= 1024; b += b < 40 ? 1 : 13)
        for (int d = 1; d < 9300; d += 1 + d / 7)
            for (int k = 1; k <= 32; ++k)
                if (small_step_fits(1000, d, k, b)) {   // no smaller batch of the same layer needs more
                    for (int s = 1; s <= b; s += 1 + b / 9)
                        if (small_lds(d, k, s, small_waves(s)).bytes > LDS_MOST) { if (bad++ < 20) printf("LDS: d %d k %d b %d of %d\\n", d, k, s, b); }
                }
    return bad != 0;
}
"""


def test_small_step_rule(tmp_path):
    r = run_host_check(tmp_path, CHECK)
    assert r.returncode == 0, r.stdout
