"""The row copies of forward and weight gradient write M0 from inline assembly, which the compiler cannot be told: M0 must
appear nowhere else in these kernels.  Read from the compiler's listing of the narrowest of their files."""
import os
import re
import subprocess

from paper_2306_03725_amd import build


def test_m0_belongs_to_the_row_copies(tmp_path):
    out = str(tmp_path / "products.s")
    src = os.path.join(build.CSRC, "k_products_bf16_q1.hip")
    subprocess.check_call([build._hipcc()] + build.FLAGS + ["--cuda-device-only", "-S", src, "-o", out], stderr=subprocess.DEVNULL)
    inside, own, other = False, 0, []
    with open(out) as fh:
        for line in fh:
            if "ASMSTART" in line:
                inside = True
            elif "ASMEND" in line:
                inside = False
            elif re.search(r"\bm0\b", line.split(";")[0]):
                if inside:
                    own += 1
                else:
                    other.append(line.strip())
    assert own > 0 and not other, other[:5]
