"""The turns of the workgroups that walk the column lists (csrc/k_lists_cut.h): every one of them once, and the first of every
chunk before the second of any, so that a launch ends with short lists.  No GPU: the header is plain C++."""

from test_lists_cut import run_host_check

PROGRAM = r"""
#include <stdio.h>
#include <vector>
#include "k_lists_cut.h"
using namespace usl_lists;
int main() {
    long bad = 0;
    const int widths[] = {1, 3, 4, 5, 31, 32, 33, 1000, 1023, 1024, 1025, 3075, 4095, 4096, 4097, 8191, 8192, 9000, 37107, 70000, 1 << 20, 1500000};
    for (int d : widths)
        for (int chunk : {1024, 4096})
            for (int per : {4, 32}) {
                const ChunkTurns turns = chunk_turns(d, chunk, per);
                const int n = (d + per - 1) / per;   // workgroups
                std::vector<char> seen(n, 0);
                int last = 0;
                for (int t = 0; t < n; ++t) {
                    const int at = turns(t), pos = at % (chunk / per);
                    if (at < 0 || at >= n || seen[at]++ || pos < last) {
                        if (bad++ < 10) printf("d=%d chunk=%d per=%d turn %d: %d\n", d, chunk, per, t, at);
                        break;
                    }
                    last = pos;
                }
            }
    return bad != 0;
}
"""


def test_every_turn_once_and_all_chunks_side_by_side(tmp_path):
    r = run_host_check(tmp_path, PROGRAM)
    assert r.returncode == 0, r.stdout
