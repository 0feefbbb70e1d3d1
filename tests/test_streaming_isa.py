"""Static checks on the generated gfx950 code of the kernels that stream the operands (no GPU needed): as many of their waves on a SIMD as hide
the loads, whichever storage order or slice count a call takes of what one kernel holds, and no scratch."""
import os
import re
import subprocess

import pytest

from test_kernel_isa import CSRC

# kernel: most vector registers (512 to a SIMD's lane: 64 are eight waves, 128 four)
SCAN = {"scan_kernelILb0ELb0EE": 64, "scan_kernelILb1ELb0EE": 64, "scan_kernelILb0ELb1EE": 84, "scan_kernelILb1ELb1EE": 84}
SLICING = {"slice_kernelILi8EE": 80, "slice_kernelILi16EE": 128, "slice_kernelILi26EE": 128}


def resources(source, tmp_path):
    """mangled name -> (vector registers, bytes of scratch) of a source's kernels."""
    from paper_2511_13778_amd.build import FLAGS, SOURCE_FLAGS
    out = tmp_path / (source + ".s")
    r = subprocess.run(["hipcc", *FLAGS, *SOURCE_FLAGS.get(source + ".hip", []), "-S", "--cuda-device-only", os.path.join(CSRC, source + ".hip"),
                        "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return {m.group(1): (int(m.group(3)), int(m.group(2)))
            for m in re.finditer(r"\.amdhsa_kernel (\S+).*?\.amdhsa_private_segment_fixed_size (\d+).*?\.amdhsa_next_free_vgpr (\d+)",
                                 open(out).read(), re.S)}


@pytest.mark.parametrize("kernel", SLICING)
def test_slicing_keeps_its_waves(tmp_path, kernel):
    (got,) = [v for name, v in resources("oz_slice", tmp_path).items() if kernel in name]
    assert got[0] <= SLICING[kernel] and got[1] == 0, got


@pytest.mark.parametrize("kernel", SCAN)
def test_scan_keeps_its_waves(tmp_path, kernel):
    # eight workgroups of four waves to a CU where no operand has rows of 64 k a load, six otherwise
    (got,) = [v for name, v in resources("oz_scan", tmp_path).items() if kernel in name]
    assert got[0] <= SCAN[kernel] and got[1] == 0, got
