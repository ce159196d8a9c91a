"""The float32 kernel of both backward products with two instances a pass: the groups of the first list wait for what they read, not for the second list's
activations, which are asked for after it.  Read from the compiler's listing."""
import os
import re
import subprocess

from paper_2306_03725_amd import build


def test_groups_of_the_first_list_wait_for_their_own_reads(tmp_path):
    src, out = os.path.join(build.CSRC, "k_backward_input_lds.hip"), os.path.join(build.HERE, "_build", "k_backward_input_lds.s")
    if not os.path.exists(out) or os.path.getmtime(out) < max(os.path.getmtime(os.path.join(build.CSRC, f)) for f in os.listdir(build.CSRC)):
        out = str(tmp_path / "both.s")
        subprocess.check_call([build._hipcc()] + build.FLAGS + ["--cuda-device-only", "-S", src, "-o", out], stderr=subprocess.DEVNULL)
    with open(src) as fh:
        groups = int(re.search(r"KT_BOTH = (\d+)", fh.read()).group(1)) // 4
    with open(out) as fh:
        lines = fh.read().splitlines()
    kernels = [i for i, l in enumerate(lines) if re.match(r"^_Z\w*k_both_ldsIfLi2E\w*:", l)]
    assert len(kernels) == 1
    for start in kernels:
        end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
        waits, last = [], ""
        for l in lines[start:end]:
            if "lgkmcnt" in l:
                last = l.strip()
            elif "v_lshlrev_b32_sdwa v112" in l:   # a group of four begins
                waits.append(last)
        assert len(waits) == 2 * groups and waits.count("s_waitcnt lgkmcnt(1)") == groups, (lines[start], waits)
