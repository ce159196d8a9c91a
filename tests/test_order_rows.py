"""The rows of LDS in which the slot order is made (csrc/k_lanes.h): a thread reads and writes its own row and no other, so no
lane depends on how far another one of its wavefront has come.  No GPU: the header is plain C++."""

from test_lists_cut import run_host_check

PROGRAM = r"""
#include <stdio.h>
#include "k_lanes.h"
template <int GS> int check() {
    int bad = 0, seen[256] = {0};
    for (int tid = 0; tid < 256; ++tid) {
        const int label = usl_order_label<GS>(tid);
        if (label < 0 || label > 255 || label / 32 != tid / 32 || seen[label]++) ++bad;   // every label once, within the half-wavefront
        else if (usl_order_row<GS>(label) != tid) ++bad;                                  // ... and its row is the thread's own
        if (usl_position_of_lane<GS>(usl_lane_of_position<GS>(tid & 31)) != (tid & 31)) ++bad;
    }
    return bad;
}
int main() { const int a = check<32>(), b = check<16>(); printf("%d %d\n", a, b); return a || b; }
"""


def test_a_thread_of_the_slot_order_has_its_own_row(tmp_path):
    r = run_host_check(tmp_path, PROGRAM)
    assert r.returncode == 0, r.stdout
