"""Static checks on the generated gfx950 code of the slice GEMM's kernels and of the FP64 fallback GEMM (no GPU needed:
hipcc cross-compiles).

The kernel issues its tile transfers and epilogue stores from asm blocks whose base address is a
scalar register pair.  Inside an asm block the compiler does not insert the wait states the
hardware needs between a vector-ALU write of a scalar register (v_readlane / v_readfirstlane, e.g. a
register-allocator reload) and a memory instruction that reads it; a store issued too early uses the
stale register as its address.  These tests read the compiler's assembly of this repository's own
kernel and check that no such pair is closer than the required distance, and that the MFMA loop
itself is free of register spills."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_13778_amd", "csrc")
WAIT_STATES = 5


@pytest.fixture(scope="module")
def gemm_asm(tmp_path_factory):
    from paper_2511_13778_amd.build import FLAGS
    lines = []
    for name in ("oz_gemm_i8", "oz_gemm_few"):
        out = tmp_path_factory.mktemp("isa") / (name + ".s")
        cmd = ["hipcc", *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, name + ".hip"), "-o", str(out)]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        lines += [ln for ln in open(out).read().splitlines() if ln.strip() and not ln.strip().startswith(";")]
    return lines


def function_body(asm, mangled_prefix):
    (start,) = [i for i, ln in enumerate(asm) if ln.startswith(mangled_prefix) and ":" in ln]     # of several instances none is left out
    end = next(i for i in range(start, len(asm)) if asm[i].startswith(".Lfunc_end"))
    return asm[start:end]


def too_close(asm):
    """(memory instructions with a scalar base by opcode, those that read it within WAIT_STATES of a vector-ALU write)."""
    written = {}           # scalar register -> wait-state position of its last vector-ALU write
    pos = 0
    seen, bad = {}, []
    for ln in asm:
        pos += 1
        t = ln.split()
        if t[0] in ("v_readlane_b32", "v_readfirstlane_b32"):
            written[t[1].rstrip(",")] = pos
        elif t[0] == "s_nop":
            pos += int(t[1])
        elif t[0].startswith(("global_store", "global_load", "global_atomic")):
            m = re.search(r"s\[(\d+):(\d+)\]", ln)
            if not m:
                continue
            seen[t[0]] = seen.get(t[0], 0) + 1
            for x in range(int(m.group(1)), int(m.group(2)) + 1):
                if pos - written.get("s%d" % x, -10 ** 9) <= WAIT_STATES:
                    bad.append(ln)
    return seen, bad


def basic_blocks(asm):
    block, blocks = [], []
    for ln in asm:
        if re.match(r"^\.LBB\d+_\d+:", ln):
            blocks.append(block)
            block = []
        block.append(ln)
    blocks.append(block)
    return blocks


# the slice GEMM's kernels: the MFMA each issues, how its asm blocks write results, and how many basic blocks hold steps
# with transfers and LDS reads at least
FORMS = {"_ZN2oz14gemm_i8_kernelILb0EE": ("v_mfma_i32_16x16x64_i8", "global_store_dwordx4", 7),
         "_ZN2oz14gemm_i8_kernelILb1EE": ("v_mfma_i32_32x32x32_i8", None, 6),
         "_ZN2oz18gemm_i8_few_kernelILb0EE": ("v_mfma_i32_32x32x32_i8", "global_store_dword", 1),
         "_ZN2oz18gemm_i8_few_kernelILb1EE": ("v_mfma_i32_32x32x32_i8", "global_store_dword", 1)}


@pytest.mark.parametrize("kernel", FORMS)
def test_asm_memory_ops_never_read_a_freshly_valu_written_scalar(gemm_asm, kernel):
    seen, bad = too_close(function_body(gemm_asm, kernel))
    assert not bad, bad
    # the kernel's transfers, and the epilogue's stores where it has them, were actually looked at
    assert seen.get("global_load_lds_dwordx4", 0) >= 40
    store = FORMS[kernel][1]
    assert store is None or seen.get(store, 0) >= 60
    assert store is None or not any(op.startswith("global_store") and op != store for op in seen)


def test_the_check_sees_a_store_that_is_too_early():
    for op in ("global_store_dwordx4 v1, v[2:5], s[6:7]", "global_load_lds_dwordx4 v1, s[6:7]"):
        for nops, bad in ((3, 1), (4, 0)):
            seen, found = too_close(["\tv_readlane_b32 s7, v0, 1", "\ts_nop %d" % nops, "\t" + op])
            assert len(found) == bad and sum(seen.values()) == 1


def step_blocks(body, mfma):
    return [b for b in basic_blocks(body) if sum(mfma in ln for ln in b) >= 8
            and any("global_load_lds" in ln for ln in b) and any("ds_read_b128" in ln for ln in b)]


@pytest.mark.parametrize("kernel", FORMS)
def test_mfma_loop_has_no_spills(gemm_asm, kernel):
    # basic blocks (label to label) that hold the steps' MFMAs must not touch scratch memory, bring spilled scalars back or
    # move accumulators between the register files
    mfma, _, least = FORMS[kernel]
    body = function_body(gemm_asm, kernel)
    other = [m for m, _, _ in FORMS.values() if m != mfma][0]
    assert not any(other in ln for ln in body)          # each kernel is looked at through the MFMA it issues
    hot = step_blocks(body, mfma)
    assert len(hot) >= least
    for b in hot:
        assert not any("scratch_" in ln or "v_readlane" in ln or "v_writelane" in ln or "v_accvgpr" in ln for ln in b)


@pytest.mark.parametrize("kernel", FORMS)
def test_mfma_loop_waits_for_no_transfer_too_early(gemm_asm, kernel):
    # The transfers are invisible to the compiler.  A wait of its own for some earlier load (a reload of a spilled register,
    # say) that falls inside a step waits for the transfers in flight as well: with vmcnt below the sixteen that the steps
    # themselves wait for, this kernel lost 30 % of its rate.
    body = function_body(gemm_asm, kernel)
    waits = [int(n) for b in step_blocks(body, FORMS[kernel][0]) for ln in b for n in re.findall(r"vmcnt\((\d+)\)", ln)]
    assert all(n >= 16 for n in waits), waits


def shared_countdowns(asm):
    """(countdowns of the tile streams seen, those that keep another operand in the register they count down first)."""
    seen, bad = 0, []
    for i, ln in enumerate(asm):
        m = re.match(r"s_sub_u32 (s\d+), \1, 1$", ln.strip())
        if not m or "s_cselect_b64" not in asm[i + 2]:
            continue
        seen += 1
        r = int(m.group(1)[1:])
        by = [int(x) for x in re.findall(r"\[(\d+):", asm[i + 2])]        # by, wrap, plane: pairs
        n = re.match(r"s_cselect_b32 s\d+, s(\d+), s\d+", asm[i + 3].strip())
        if int(n.group(1)) == r or any(r in (x, x + 1) for x in by):
            bad.append(asm[i:i + 5])
    return seen, bad


def test_stream_countdown_has_its_register_to_itself(gemm_asm):
    for kernel in list(FORMS)[:2]:
        seen, bad = shared_countdowns(function_body(gemm_asm, kernel))
        assert seen >= 16 and not bad, bad
    alias = ["s_sub_u32 s4, s4, 1", "s_cmp_eq_u32 s4, 0", "s_cselect_b64 s[6:7], s[8:9], s[10:11]", "s_cselect_b32 s4, s4, s4"]
    assert shared_countdowns(alias + ["s_subb_u32 s5, s5, 0"])[1]


@pytest.fixture(scope="module")
def dgemm_asm(tmp_path_factory):
    from paper_2511_13778_amd.build import FLAGS
    out = tmp_path_factory.mktemp("isa") / "oz_dgemm_f64.s"
    cmd = ["hipcc", *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, "oz_dgemm_f64.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return [ln for ln in open(out).read().splitlines() if ln.strip() and not ln.strip().startswith(";")]


@pytest.mark.parametrize("mode", [0, 1])
def test_fp64_gemm_k_loop_has_no_vector_address_arithmetic(dgemm_asm, mode):
    # The K loop of the FP64 fallback GEMM (128 x 128 tiles, interior and ragged modes) loads its tiles
    # through a buffer descriptor: 16 buffer loads and 64 MFMAs per K step, and no 64-bit vector adds.  With
    # plain pointer loads the compiler rebuilt sixteen 64-bit per-lane addresses in every K step, which
    # cost the matrix unit 4 % of its issue slots; this guards the code generation the speed depends on.
    body = function_body(dgemm_asm, "_ZN2oz16dgemm_f64_kernelILb1ELb0ELi%dELi128EEE" % mode)
    # the K loop: the block that branches back to its own label (a peeled first K step may precede it);
    # what follows the back branch belongs to the code after the loop
    loops = []
    for b in basic_blocks(body):
        label = b[0].split(":")[0] if b and b[0].startswith(".LBB") else None
        back = [i for i, ln in enumerate(b) if label and ln.split()[0].startswith("s_cbranch") and ln.split()[1] == label]
        if back:
            loops.append(b[:back[0] + 1])
    loops = [b for b in loops if sum("v_mfma_f64_16x16x4" in ln for ln in b) == 64]
    assert len(loops) == 1
    loop = loops[0]
    assert sum("buffer_load_dwordx2" in ln for ln in loop) == 16
    assert not any(ln.split()[0].startswith(("v_lshl_add_u64", "v_add_co_u32", "v_addc_co_u32", "global_load")) for ln in loop)
    assert not any("scratch_" in ln for ln in loop)


def touched_in_flight(lines):
    """Loads written as asm whose target is read or written before the next full wait: (loads seen, offending lines)."""
    def registers(text):
        out = set()
        for m in re.finditer(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
            lo, hi = (m.group(1), m.group(2)) if m.group(1) else (m.group(3), m.group(3))
            out.update(range(int(lo), int(hi) + 1))
        return out

    loads, bad, flying, in_asm = 0, [], set(), False
    for ln in lines:
        t = ln.strip()
        if t.startswith(";"):
            in_asm = (in_asm or "#ASMSTART" in t) and "#ASMEND" not in t
            continue
        code = t.split(";")[0]
        if re.search(r"s_waitcnt\b.*vmcnt\(0\)", code):
            flying = set()
        elif in_asm and code.startswith("global_load"):
            target, rest = code.split(",", 1)
            if registers(rest) & flying or registers(target) & flying:
                bad.append(ln)
            loads += 1
            flying |= registers(target)
        elif registers(code) & flying:
            bad.append(ln)
    return loads, bad


def test_esc_loads_written_as_asm_are_not_touched_in_flight(tmp_path):
    # The ESC kernel requests the operands of its next step in asm, so that they stay ahead of the arithmetic, and awaits them
    # in a later asm statement.  To the compiler they have arrived at once: a copy or a spill in between would take what
    # the registers held before, and a register freed in between would be overwritten when the data comes.
    from paper_2511_13778_amd.build import FLAGS, SOURCE_FLAGS
    out = tmp_path / "oz_esc.s"
    cmd = ["hipcc", *FLAGS, *SOURCE_FLAGS["oz_esc.hip"], "-S", "--cuda-device-only", os.path.join(CSRC, "oz_esc.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    loads, bad = touched_in_flight(function_body([ln for ln in open(out).read().splitlines() if ln.strip()], "_ZN2oz10esc_kernel"))
    assert loads >= 24 and not bad, bad
    # the check itself
    load = ["\t;;#ASMSTART", "\tglobal_load_dwordx4 v[4:7], v[0:1], off", "\t;;#ASMEND"]
    assert touched_in_flight(load + ["\tv_mov_b32_e32 v9, v5"])[1] and touched_in_flight(load + ["\tv_mov_b32_e32 v6, v9"])[1]
    assert touched_in_flight(load + ["\ts_waitcnt vmcnt(0)", "\tv_mov_b32_e32 v9, v5"]) == (1, [])
