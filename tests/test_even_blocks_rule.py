"""When blocks of equal size are dealt (k_products.h), on the host: the busiest compute unit gets no workgroup more than with full blocks, the workgroups
that a compute unit holds are those of the kernel's registers, and forms that spill or batches in many parts of a large x are left alone."""
from test_lists_cut import run_host_check

CHECK = r"""
#include <stdio.h>
#include "k_products.h"
using namespace usl_products;
static long bad = 0;
#define WANT(x) do { if (!(x) && bad++ < 20) printf("line %d: %s (m %lld NT %d LPT %d parts %d res %d: %lld blocks, labels %d)\\n", __LINE__, #x, (long long)m, NT, LPT, parts, res, (long long)nblk, labels); } while (0)
int main() {
    unsigned long long r = 88172645463325252ull;
    auto next = [&]() { r ^= r << 13; r ^= r >> 7; r ^= r << 17; return r; };
    for (int n = 0; n < 300000; ++n) {
        const int NT = 256 << next() % 3, LPT = 1 << next() % 3, parts = 1 + (int)(next() % (n % 2 ? 8 : 200)), res = 1 + (int)(next() % 8), cus = n % 4 ? 256 : 1 + (int)(next() % 304);
        const int64_t m = 1 + (int64_t)(next() % (1ull << (1 + next() % 22))), per = (int64_t)NT * LPT, nblk = (m + per - 1) / per;
        const ProductKernel kern = {nullptr, nullptr, 32, LPT, NT, 0};
        const int labels = even_block_labels(m, kern, nblk, parts, cus, res);
        WANT(labels >= 32 && labels % 32 == 0 && labels <= per + 31);
        const int64_t blocks = (m + labels - 1) / labels, unit = LPT > 1 ? (int64_t)cus * res : cus;
        WANT((blocks * parts + unit - 1) / unit <= (nblk * parts + unit - 1) / unit);
    }
    const int64_t m = 0, nblk = 0;
    const int NT = 0, LPT = 0, parts = 0, res = 0, labels = 0;
    // registers of the 256-lane forms with 16, 32 and 64 slots; one wavefront a SIMD at 512, rows that fill LDS
    WANT(resident_workgroups(256, 78, 20000) == 6 && resident_workgroups(256, 147, 20000) == 3 && resident_workgroups(256, 174, 20000) == 2 && resident_workgroups(256, 40, 1000) == 8);
    WANT(resident_workgroups(512, 256, 60000) == 1 && resident_workgroups(1024, 128, 80000) == 1 && resident_workgroups(1024, 64, 80000) == 2 && resident_workgroups(1024, 128, 160000) == 1);
    WANT(even_blocks_allowed(8, 1 << 28, 44, 44) && even_blocks_allowed(9, 2 << 20, 0, 0) && even_blocks_allowed(1, 1, 76, 20));
    WANT(!even_blocks_allowed(1, 1, 184, 396) && !even_blocks_allowed(9, (2 << 20) + 1, 0, 0));
    return bad != 0;
}
"""


def test_even_blocks_rule(tmp_path):
    r = run_host_check(tmp_path, CHECK)
    assert r.returncode == 0, r.stdout
