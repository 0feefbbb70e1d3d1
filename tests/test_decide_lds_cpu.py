"""LDS of a small call that decides in the slicing's launch (no GPU): a launch without a raised limit may ask for 64 KB in all, the tables that
follow from the call's sizes and the variables the compiler places beside them."""
import os
import re
import subprocess

import pytest

from test_kernel_isa import CSRC
from test_unit_walk_cpu import host_program


@pytest.fixture(scope="module")
def own_lds(tmp_path_factory):
    """LDS bytes the compiler gives each instance of the kernel."""
    from paper_2511_13778_amd.build import FLAGS, SOURCE_FLAGS
    out = tmp_path_factory.mktemp("lds") / "oz_esc_slice.s"
    r = subprocess.run(["hipcc", *FLAGS, *SOURCE_FLAGS["oz_esc_slice.hip"], "-S", "--cuda-device-only", os.path.join(CSRC, "oz_esc_slice.hip"),
                        "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = open(out).read()
    found = re.findall(r"\.amdhsa_kernel _ZN2oz16esc_slice_kernelILi(\d+)EE.*?\.amdhsa_group_segment_fixed_size (\d+)", text, re.S)
    assert len(found) == 3
    return max(int(x) for _, x in found)


def test_tables_and_variables_stay_below_64_kb(tmp_path_factory, own_lds):
    run = host_program(tmp_path_factory, "host_decide_lds.cpp")
    ks = [1, 64, 65, 128, 129, 192, 193, 256, 257, 320, 384, 385, 512, 513, 640, 768, 769, 1024]
    cases = [(m, n, k, b, cus) for m in range(64, 1100, 64) for n in range(64, 1100, 64) for k in ks for b in (16, 32, 48, 64, 128)
             for cus in (64, 256)]
    got = run(cases)
    taken = [(r[1] + own_lds, c) for c, r in zip(cases, got) if r[0]]
    assert len(taken) > 1000 and max(taken)[0] > 60 * 1024
    assert max(taken)[0] <= 64 * 1024 and {r[2] for r in got} == {64 * 1024}, max(taken)
    # 896 columns beside 64 rows and 9 to 12 ESC blocks: the tables alone are 256 bytes below the limit
    assert [r[0] for r in run([(64, 896, 320, 32, 256), (896, 64, 384, 32, 256), (64, 833, 192, 16, 256), (64, 832, 320, 32, 256)])] == [0, 0, 0, 1]
