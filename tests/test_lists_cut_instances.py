"""Which layers take four instances a pass of the kernel for both products, and how they are cut then (csrc/k_lists_cut.h): the
window fits LDS, all labels are covered, and the shape that bench.py reports is the same.  No GPU: the header is plain C++."""
import subprocess

import numpy as np

import bench

PROGRAM = r"""
#include <cstdio>
#define __host__
#define __device__
#define __forceinline__ inline
#include "k_lists_cut.h"
using namespace usl_lists;
int main() {
    long long m; int d, k;
    while (scanf("%lld %d %d", &m, &d, &k) == 3) {
        const int Q = both_q(m, d, k, 256);
        const Cut c = both_cut(m, d, k, 256, Q);
        const bool fits = c.wl <= (Q == 2 ? BOTH2_LABELS : both_own(Q, c) ? BOTH4_OWN_LABELS : BOTH4_LABELS);
        const bool covers = (long long)c.nwin * c.wl >= m && (long long)(c.nwin - 1) * c.wl < m;
        printf("%d %d %d %d\n", Q, c.nwin, c.nfb, (int)(fits && covers));
    }
}
"""


def test_cut_of_the_chosen_instances(tmp_path):
    root = bench.__file__.rsplit("/", 1)[0]
    (tmp_path / "cut.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", root + "/paper_2306_03725_amd/csrc", "-o", tmp_path / "cut", tmp_path / "cut.cpp"], check=True)
    rng = np.random.default_rng(3)
    layers = [(670000, 16384, 32), (670000, 32768, 64), (300000, 24000, 48), (130000, 15360, 32), (300000, 14000, 32), (670000, 30000, 64), (500000, 32768, 32)]
    for _ in range(3000):
        k = int(rng.integers(1, 65))
        d = int(min(65536, max(k, rng.uniform(300, 560) * k)))   # around the lines of the rule
        layers.append((int(np.exp(rng.uniform(np.log(1), np.log(3e6)))), d, k))
    out = subprocess.run([tmp_path / "cut"], input="\n".join("%d %d %d" % l for l in layers), text=True, capture_output=True, check=True).stdout.split("\n")
    chosen = set()
    for (m, d, k), line in zip(layers, out):
        q, nwin, nfb, ok = map(int, line.split())
        assert ok, (m, d, k, line)
        chosen.add(q)
        cut = bench.one_pass_cut(type("Layer", (), dict(m=m, d=d, k=k, b=1, storage="f32")))
        assert cut is None or (cut["q"], cut["nwin"], cut["nfb"]) == (q, nwin, nfb), (m, d, k, line, cut)
    assert chosen == {2, 4}
    assert [int(l.split()[0]) for l in out[:7]] == [4, 2, 2, 2, 4, 2, 2]
