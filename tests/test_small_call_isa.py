"""Static check on the generated gfx950 code of the slice GEMMs on small tiles (no GPU needed): their transfers take a scalar base in
an asm block, where the compiler does not keep the distance to a vector-ALU write of that register."""
import os
import subprocess

import pytest

from test_kernel_isa import CSRC, function_body, gemm_asm, shared_countdowns, step_blocks, too_close  # noqa: F401


@pytest.mark.parametrize("source,kernel", [("oz_gemm_small", "_ZN2oz17gemm_small_kernel"), ("oz_gemm_mid", "_ZN2oz15gemm_mid_kernelILi1EE"),
                                           ("oz_gemm_mid", "_ZN2oz15gemm_mid_kernelILi2EE")])
def test_transfers_never_read_a_freshly_valu_written_scalar(tmp_path, source, kernel):
    from paper_2511_13778_amd.build import FLAGS
    out = tmp_path / (source + ".s")
    r = subprocess.run(["hipcc", *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, source + ".hip"), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    asm = [ln for ln in open(out).read().splitlines() if ln.strip() and not ln.strip().startswith(";")]
    body = function_body(asm, kernel)
    seen, bad = too_close(body)
    assert seen.get("global_load_lds_dwordx4", 0) >= 2 and not bad, bad
    assert not any("scratch_" in ln for ln in body)


def test_slice_gemm_of_a_batch_keeps_the_rules_of_the_single_one(gemm_asm):
    body = function_body(gemm_asm, "_ZN2oz20gemm_i8_batch_kernel")
    seen, bad = too_close(body)
    assert seen.get("global_load_lds_dwordx4", 0) >= 40 and seen.get("global_store_dwordx4", 0) >= 60 and not bad, bad
    hot = step_blocks(body, "v_mfma_i32_16x16x64_i8")
    assert len(hot) >= 7
    for b in hot:
        assert not any("scratch_" in ln or "v_readlane" in ln or "v_writelane" in ln or "v_accvgpr" in ln for ln in b)
    seen, bad = shared_countdowns(body)
    assert seen >= 16 and not bad, bad
