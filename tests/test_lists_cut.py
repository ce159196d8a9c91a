"""How a layer is cut into windows of labels and blocks of features, checked on the host over the range of sizes: every
window has labels and fits LDS, the windows cover the layer, the blocks cover the features.  A window behind the last
label would make its workgroups copy with a negative length."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_03725_amd", "csrc")

CHECK = r"""
#include <stdio.h>
#include "k_lists_cut.h"
using namespace usl_lists;
static long bad = 0, seen = 0;
static void check(const char* what, Cut c, long long m, int d, int k, int most) {
    ++seen;
    const bool ok = c.nwin >= 1 && c.wl >= 1 && (c.wl % 4 == 0) && c.wl <= most && (long long)(c.nwin - 1) * c.wl < m && (long long)c.nwin * c.wl >= m &&
                    c.wl == c.run * c.S && c.vd == c.S * d && c.fpb % 32 == 0 && c.fpb <= NF && (long long)c.nfb * c.fpb >= c.vd && (long long)(c.nfb - 1) * c.fpb < c.vd;
    if (!ok && bad++ < 20) printf("%s m=%lld d=%d k=%d: nwin %d wl %d run %d S %d nfb %d fpb %d\n", what, m, d, k, c.nwin, c.wl, c.run, c.S, c.nfb, c.fpb);
}
static void both(long long m, int d, int k, int cu) {   // as the library cuts the layer
    const int Q = both_q(m, d, k, cu);
    const Cut cut = both_cut(m, d, k, cu, Q);
    check("both", cut, m, d, k, Q == 2 ? BOTH2_LABELS : both_own(Q, cut) ? BOTH4_OWN_LABELS : BOTH4_LABELS);
}
int main() {
    const long long pick[][3] = {{670000, 2048, 32}, {1000000, 8192, 64}, {1000000, 2048, 64}, {500000, 1500, 64}, {300000, 1100, 32}, {76296, 1133, 64}};
    for (auto& p : pick) both(p[0], (int)p[1], (int)p[2], 256);
    unsigned long long r = 88172645463325252ull;
    auto next = [&]() { r ^= r << 13; r ^= r >> 7; r ^= r << 17; return r; };
    const int ks[] = {1, 3, 5, 8, 16, 17, 32, 33, 48, 64};
    for (int n = 0; n < 400000; ++n) {
        const int d = 1 + (int)(next() % (1u << (1 + next() % 16)));
        const long long m = 1 + (long long)(next() % (1ull << (1 + next() % 23)));
        int k = ks[next() % 10];
        if (k > d) k = d;
        const int cu = n % 4 ? 256 : 1 + (int)(next() % 304);
        both(m, d, k, cu);
        const int dl = 1 + (int)(k * (300 + next() % 260));   // around the lines of the rule for the instances of a pass
        if (dl <= 65536) both(m, dl, k, cu);
        const long long lists = 32ll * d / k;
        if (d % NF == 0 && m % 4 == 0 && lists >= 2048 && lists <= WL) check("input gradient", bwi_cut(m, d, k, cu), m, d, k, WL);
        const int d2 = NF * (1 + (int)(next() % 32)), k2 = 32 * d2 / (int)(2048 + next() % 30721);   // shapes of that form
        if (k2 >= 1) check("input gradient", bwi_cut(m * 4, d2, k2, cu), m * 4, d2, k2, WL);
    }
    printf("%ld checked, %ld bad\n", seen, bad);
    return bad != 0;
}
"""


def run_host_check(tmp_path, text, *more):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(text)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-D__forceinline__=inline", "-I", CSRC, *more, str(src), "-o", str(exe)])
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_every_window_has_labels(tmp_path):
    r = run_host_check(tmp_path, CHECK)
    assert r.returncode == 0, r.stdout


MOST = r"""
#include <stdio.h>
#include "k_lists_cut.h"
using namespace usl_lists;
int main() {
    long bad = 0, drops = 0, at_lines[5] = {};
    unsigned long long r = 88172645463325252ull;
    auto next = [&]() { r ^= r << 13; r ^= r >> 7; r ^= r << 17; return r; };
    for (int n = 0; n < 3000; ++n) {
        long long m = n == 0 ? 13330 : 1 + (long long)(next() % (1ull << (4 + next() % 18)));
        int d = n == 0 ? 5000 : 1 + (int)(next() % (1u << (1 + next() % 16)));
        int k = n == 0 ? 32 : 1 + (int)(next() % 64);
        if (k > d) k = d;
        const bool line = n > 0 && n % 4 == 0 && k * 560 <= 65536;   // around the lines of the rule for the instances of a pass
        if (line) { d = k * (int)(424 + next() % 94); m *= 1 + (long long)(next() % 16); }
        const int max_b = n == 0 ? 128 : 1 + (int)(next() % 700), Q = both_q(m, d, k, 256), forced = n % 5 == 4 ? 1 + (int)(next() % 8) : 0;
        const int G = n == 0 || n % 3 ? max_b : 1 + (int)(next() % max_b);
        if (line && d > NT) ++at_lines[Q];
        const Cut cut = both_cut(m, d, k, 256, Q);
        const BothMost most = both_most(cut, m, k, 256, max_b, G, Q, forced);
        int last = 0;
        for (int b = 1; b <= max_b; ++b) {
            const BothPlan p = both_plan(cut, m, k, 256, b, G, Q, forced);
            const long long rows = (long long)p.sets * (b < G ? b : G);
            if (p.parts > most.parts || rows > (long long)most.rows) ++bad;
            if (p.parts < last) ++drops;
            last = p.parts;
        }
    }
    printf("%ld bad, %ld larger batches with fewer parts\n", bad, drops);
    return bad != 0 || drops == 0 || at_lines[2] == 0 || at_lines[4] == 0;
}
"""


def test_scratch_of_the_largest_need_covers_every_batch(tmp_path):
    """The parts of a batch do not grow with it; what is reserved once is what the neediest batch takes."""
    r = run_host_check(tmp_path, MOST)
    assert r.returncode == 0, r.stdout
